// GEMM in blocks that are chosen apart from the plan's tile (gfx950): every plan
// with 64x64 tiles, and unsignalled launches of the larger tiles whose last wave
// would be nearly empty (gemm_in_parts).
//
// A 64x64 tile is the only one that fits sizes which are odd multiples of 64,
// but as a unit of computation it is a poor one: per 64 k values it brings
// 16 KB into LDS and reads 32 KB from it for 128 cycles of MFMA (the LDS
// moves 128 bytes per cycle), and its few MFMAs do not cover a barrier. A
// workgroup therefore computes
//   128x128  four plan tiles, one per wave (half the operand bytes per flop),
//            when there are enough of them;
//   64x64    one plan tile, waves of 32x32;
//   64x32, 32x32  a half or a quarter of a plan tile, when an unsignalled
//            launch has too few tiles to occupy the compute units.
// Every block shape sums each output over k in the same order with the same
// MFMA (16x16x32), so a plan's results do not depend on the block taken.
// Measured against one 64x64 form for all (four waves of 32x32, three stages,
// one workgroup per compute unit, bf16): 768x3840x4160 51.9 -> 29.0 us (473 ->
// 846 TFLOP/s), signalled 1216x2880x1984 47.6 -> 22.6 us, 64x4096x3584 17.0 ->
// 9.8 us (in a run of 14.9 us; 13.3 without the loop, see Mode). What bounds it
// now: in the 128x128 form the LDS (32 KB in, 64 KB read per 512 cycles of MFMA)
// and the ~5 us of a launch's prologue and epilogue; in the small blocks the
// latency of a step's barrier and fragment reads.
//
// Main loop as in gemm.hip: direct global-to-LDS loads into a ring of ST
// stages, XOR-swizzled rows, the next MFMA substep's fragments read during the
// current one, one barrier per step. The next block's first loads are issued
// before the finished block is stored. Epilogue, signal and tile positions as
// described in fo.h; a wave stores its own part of the block.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>
#include <utility>

#include "fo_device.h"
#include "fo_internal.h"
#include "gemm.h"

namespace fo {
namespace {

// s_waitcnt operand for vmcnt = vm and lgkmcnt = lgkm, expcnt at its maximum
constexpr int wait_imm(int vm, int lgkm) {
    return (vm & 15) | (7 << 4) | ((lgkm & 15) << 8) | (((vm >> 4) & 3) << 14);
}
constexpr int kRsrcWord3 = 0x00020000;   // raw byte-addressed buffer accesses
constexpr int kCachePolicySc1 = 16;      // device-coherent write-through

typedef __attribute__((address_space(3))) void lds_void_t;

template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

template <int DT>
__device__ __forceinline__ f32x4_t mfma16(u32x4_t a, u32x4_t b, f32x4_t c) {
    if constexpr (DT == FO_FP16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(bit_cast<half8_t>(a), bit_cast<half8_t>(b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(bit_cast<bf16x8_t>(a), bit_cast<bf16x8_t>(b), c, 0, 0, 0);
}

// This wave waits until at most VM of its vector memory operations are in
// flight and all of its LDS reads have returned, then meets the others.
template <int VM>
__device__ __forceinline__ void wait_and_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(wait_imm(VM, 0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// A plan table entry at a wave-uniform index, through the scalar cache (the
// tables do not change while a kernel runs; a scalar load leaves the vector
// memory counter to the operands).
__device__ __forceinline__ int32_t table_at(const int32_t* t, int64_t i) {
    return ((const __attribute__((address_space(4))) int32_t*)(uintptr_t)t)[i];
}

// What a launch may do: anything; no counters and no trace; and a block per
// workgroup besides; counters in the default mode, an output in 31-bit range and no
// trace. The loop over blocks with all that it may do has some 75 scalars that are
// formed, and spilled, between a launch's start and its first MFMA, which short
// launches wait for (64x64, 64x32 and 32x32 blocks, fp16, us):
//   kAny -> kOne     64x64, 256 tiles, K 64 5.06 -> 3.44, K 1024 7.15 -> 5.54, K 4096
//                    16.5 -> 14.6; 64x32, 128 tiles, K 64 4.80 -> 3.37, K 1024 6.47 ->
//                    5.02; 32x32, 64 tiles, K 64 4.56 -> 3.07, K 3584 9.4 -> 7.9
//   kAny -> kPlain   64x64, 320 tiles on 240 workgroups, K 512 8.5 -> 7.2
//   kAny -> kSignal  64x64, 256 tiles, K 64 8.0 -> 7.2; on 240 workgroups, K 1024 12.5
//                    -> 11.6; 512 tiles, K 4096 29.9 -> 29.2
// The 128x128 form has one body for all: its launches are longer.
enum Mode { kAny, kPlain, kOne, kSignal };

template <int DT, int TM, int TN, int BM, int BN, int ST, int KS, Mode MODE>
__device__ __forceinline__ void block_body(const GemmArgs& a) {
    constexpr bool ONE = MODE == kOne;
    constexpr int kWaves = 4;                          // 2 x 2
    constexpr int WTM = BM / 2, WTN = BN / 2;          // a wave's part of the block
    constexpr int MI = WTM / 16, NJ = WTN / 16;
    constexpr int kA = BM * 128, kSlice = (BM + BN) * 128;   // bytes of 64 k values (a slice)
    constexpr int kStage = KS * kSlice;                // a stage holds KS slices
    constexpr int kAI = kA / 1024 / kWaves, kBI = BN * 128 / 1024 / kWaves;
    constexpr int kPer = kAI + kBI, kLoads = KS * kPer;      // loads per slice, per step
    constexpr bool kOwnTile = WTM == TM && WTN == TN;  // a wave's part is a plan tile (of TM x TN)
    static_assert((kOwnTile || (TM % BM == 0 && TN % BN == 0)) && BM >= 32 && BN >= 32,
                  "a plan tile per wave, a plan tile, or part of one");
    static_assert(ST >= 2 && ST <= 4 && ST * kLoads <= 62, "stages");

    // the stages live in separate arrays, so that the compiler can tell the
    // stage being read from the stages being filled
    __shared__ __attribute__((aligned(1024))) char st0[kStage], st1[kStage];
    __shared__ __attribute__((aligned(ST > 2 ? 1024 : 16))) char st2[ST > 2 ? kStage : 16];
    __shared__ __attribute__((aligned(ST > 3 ? 1024 : 16))) char st3[ST > 3 ? kStage : 16];
    auto stage = [&](auto uc) __attribute__((always_inline)) -> char* {
        constexpr int u = decltype(uc)::value % ST;
        if constexpr (u == 0) return st0;
        else if constexpr (u == 1) return st1;
        else if constexpr (u == 2) return st2;
        else return st3;
    };
    __shared__ __attribute__((aligned(16))) char s_out[kWaves][WTN == 16 ? 16 : 16 * WTN * 2];  // 16 rows of a wave
    __shared__ int64_t s_off[kWaves][WTM];             // destinations of a wave's rows
    __shared__ int s_pos[2];
    __shared__ uint32_t s_arrived[2];                  // waves whose stores of a block are complete
    __shared__ int s_group[2][kWaves];                 // group of each wave's plan tile (-1: outside the output)

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int64_t K = a.K;
    const int KT = (int)(K / 64);                      // slices
    const int steps = (KT + KS - 1) / KS;
    const int rows = a.blocks_m, cols = a.blocks_n, blocks = rows * cols;

    // Block positions are handed out as in the other GEMM kernels (gemm.hip):
    // from the class's atomic counter, the workgroup that draws a class's last
    // value leaves the word zero; without a dispenser, a fixed stride.
    const bool signals = MODE == kSignal || (MODE == kAny && a.counters), traced = MODE == kAny && a.trace;
    const bool dispenser = MODE == kSignal || (MODE == kAny && a.dispenser);
    const int DC = a.num_dispensers;
    const int cls = dispenser ? (int)(blockIdx.x % (unsigned)DC) : 0;
    const uint32_t n_cls = dispenser ? (uint32_t)((blocks - cls + DC - 1) / DC) : 0u;
    const uint32_t w_cls = dispenser ? (uint32_t)(((int)gridDim.x - cls + DC - 1) / DC) : 0u;
    // (per-lane address: at a uniform one the compiler broadcasts the result
    // across the wave, waiting for it and for every load in flight at once)
    auto draw = [&]() -> uint32_t {
        int z = 0;
        asm volatile("" : "+v"(z));
        return __hip_atomic_fetch_add(a.dispenser + cls + z, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto position = [&](uint32_t v) -> int {
        if (v == n_cls + w_cls - 1u)
            __hip_atomic_store(a.dispenser + cls, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return v < n_cls ? cls + DC * (int)v : blocks;
    };
    const bool coherent = MODE == kSignal || (signals && a.sync == FO_SYNC_COHERENT);

    // A load instruction fills 1 KB: 8 operand rows of 128 bytes, chunk c of
    // row r at slot c ^ ((r / 2) % 8).
    auto voff = [&](int blk) -> uint32_t {
        const int r = blk * 8 + lane / 8;
        return (uint32_t)(r * K * 2) + 16u * (uint32_t)((lane & 7) ^ ((r >> 1) & 7));
    };
    uint32_t voffA[kAI], voffB[kBI];
#pragma unroll
    for (int i = 0; i < kAI; ++i) voffA[i] = voff(wave * kAI + i);
#pragma unroll
    for (int i = 0; i < kBI; ++i) voffB[i] = voff(wave * kBI + i);
    const uint16_t* Ablk = a.A;
    const uint16_t* Wblk = a.W;
    uint32_t a_bytes = 0, w_bytes = 0;
    // Load `ic` of step t into stage `base`. Rows past M or N and slices past
    // the last one lie outside the buffer resource: zeros, no memory access.
    auto load_one = [&](auto ic, int t, char* base) __attribute__((always_inline)) {
        constexpr int idx = decltype(ic)::value % kPer, sl = decltype(ic)::value / kPer;
        char* const st = base + sl * kSlice;
        const int kt = t * KS + sl;
        const bool live = kt < KT;
        const uint32_t so = live ? (uint32_t)kt * 128u : 0u;
        if constexpr (idx < kAI) {
            const __amdgpu_buffer_rsrc_t r =
                __builtin_amdgcn_make_buffer_rsrc((void*)Ablk, 0, live ? (int)a_bytes : 0, kRsrcWord3);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)(st + (wave * kAI + idx) * 1024), 16, voffA[idx],
                                                     so, 0, 0);
        } else {
            const __amdgpu_buffer_rsrc_t r =
                __builtin_amdgcn_make_buffer_rsrc((void*)Wblk, 0, live ? (int)w_bytes : 0, kRsrcWord3);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)(st + kA + (wave * kBI + idx - kAI) * 1024), 16,
                                                     voffB[idx - kAI], so, 0, 0);
        }
    };

    // Fragments: lane l feeds row l % 16 of a 16-row block with chunk
    // 4 h + l / 16 of MFMA substep h.
    const int a_row = (wm * WTM + (lane & 15)) * 128;
    const int b_row = kA + (wn * WTN + (lane & 15)) * 128;
    int cslot[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) cslot[h] = 16 * ((4 * h + (lane >> 4)) ^ ((lane >> 1) & 7));
    u32x4_t fa[2][MI], fb[2][NJ];
    f32x4_t acc[MI][NJ];
    // Fragment read `ic` of substep q (slice q / 2) from stage `base`, in the
    // order of use.
    auto read_one = [&](auto ic, auto qc, const char* base, u32x4_t (&xa)[MI], u32x4_t (&xb)[NJ])
                        __attribute__((always_inline)) {
        constexpr int idx = decltype(ic)::value, q = decltype(qc)::value, h = q % 2;
        const char* const st = base + q / 2 * kSlice;
        if constexpr (idx == 0) xa[0] = *reinterpret_cast<const u32x4_t*>(st + a_row + cslot[h]);
        else if constexpr (idx <= NJ)
            xb[idx - 1] = *reinterpret_cast<const u32x4_t*>(st + b_row + (idx - 1) * 2048 + cslot[h]);
        else xa[idx - NJ] = *reinterpret_cast<const u32x4_t*>(st + a_row + (idx - NJ) * 2048 + cslot[h]);
    };
    // One substep: its MFMAs carry the reads of the next substep (q_next of
    // stage rst) and, if LOADS, the loads of step t into stage lst. W is the
    // first operand: lane l then holds row l % 16, columns 4 (l / 16) .. + 3.
    auto substep = [&](u32x4_t (&xa)[MI], u32x4_t (&xb)[NJ], auto q_next, const char* rst, u32x4_t (&ya)[MI],
                       u32x4_t (&yb)[NJ], auto loads_c, int t, char* lst) __attribute__((always_inline)) {
        constexpr bool kIssue = decltype(loads_c)::value;
        constexpr int kM = MI * NJ, kR = MI + NJ;
        constexpr int rper = (kR + kM - 1) / kM, lper = (kLoads + kM - 1) / kM;
        constexpr int gap = kM / kLoads > 1 ? kM / kLoads : 1;
        static_for<kM>([&](auto mc) __attribute__((always_inline)) {
            constexpr int m = decltype(mc)::value;
            static_for<rper>([&](auto xc) __attribute__((always_inline)) {
                constexpr int r = m * rper + decltype(xc)::value;
                if constexpr (r < kR) read_one(std::integral_constant<int, r>{}, q_next, rst, ya, yb);
            });
            static_for<lper>([&](auto xc) __attribute__((always_inline)) {
                constexpr int l = m / gap * lper + decltype(xc)::value;
                if constexpr (kIssue && m % gap == 0 && l < kLoads)
                    load_one(std::integral_constant<int, l>{}, t, lst);
            });
            acc[m / NJ][m % NJ] = mfma16<DT>(xb[m % NJ], xa[m / NJ], acc[m / NJ][m % NJ]);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // Step t (in stage u): its substeps but the last, each while the next one
    // is read; then, once step t + 1 has landed and every wave has read this
    // stage, the last substep while the next step's first one is read and
    // step t + ST is loaded here.
    auto step = [&](auto uc, int t) __attribute__((always_inline)) {
        constexpr int u = decltype(uc)::value;
        char* const cur = stage(uc);
        char* const nxt = stage(std::integral_constant<int, u + 1>{});
        static_for<2 * KS - 1>([&](auto qc) __attribute__((always_inline)) {
            constexpr int q = decltype(qc)::value;
            substep(fa[q & 1], fb[q & 1], std::integral_constant<int, q + 1>{}, cur, fa[~q & 1], fb[~q & 1],
                    std::false_type{}, 0, cur);
        });
        wait_and_barrier<(ST - 2) * kLoads>();
        substep(fa[1], fb[1], std::integral_constant<int, 0>{}, nxt, fa[0], fb[0], std::true_type{}, t + ST, cur);
    };
    auto round = [&](int t) __attribute__((always_inline)) {
        static_for<ST>([&](auto uc) __attribute__((always_inline)) { step(uc, t + decltype(uc)::value); });
    };
    auto rest = [&](auto&& self, auto uc, int t) __attribute__((always_inline)) -> void {
        constexpr int u = decltype(uc)::value;
        if constexpr (u + 1 < ST) {
            if (t + u < steps) {
                step(uc, t + u);
                self(self, std::integral_constant<int, u + 1>{}, t);
            }
        }
    };

    int p = (int)blockIdx.x;
    if (!ONE && tid < 2) s_arrived[tid] = 0;
    // One block per workgroup (the hardware starts workgroups in order): no
    // positions to hand out, and the words stay zero.
    const bool dispense = dispenser && (int)gridDim.x < blocks;
    if (dispense && tid == 0) s_pos[1] = position(draw());
    if constexpr (!ONE) wait_and_barrier<63>();
    if (dispense) p = __builtin_amdgcn_readfirstlane(s_pos[1]);

    // The wave's part of the current block: its first row and column, its plan
    // tile's slot and group, whether it lies inside the output.
    int row0 = 0, col0 = 0, slot = 0, group = 0, bucket = 0, rank = 0;
    bool inside = false;
    auto start = [&]() __attribute__((always_inline)) {
        const int b = tile_of_position(p, rows, cols, a.order, a.block_band, a.num_xcds);
        const int bm = b / cols, bn = b - bm * cols;
        Ablk = a.A + (int64_t)bm * BM * K;
        Wblk = a.W + (int64_t)bn * BN * K;
        const int64_t left_m = a.M - (int64_t)bm * BM, left_n = a.N - (int64_t)bn * BN;
        a_bytes = (uint32_t)((left_m < BM ? left_m : BM) * K * 2);
        w_bytes = (uint32_t)((left_n < BN ? left_n : BN) * K * 2);
        static_for<ST>([&](auto uc) __attribute__((always_inline)) {
            static_for<kLoads>([&](auto ic) __attribute__((always_inline)) {
                load_one(ic, decltype(uc)::value, stage(uc));
            });
        });
        row0 = bm * BM + wm * WTM;
        col0 = bn * BN + wn * WTN;
        inside = row0 < a.M && col0 < a.N;
        if (inside) {
            const int tile = row0 / TM * a.tiles_n + col0 / TN;
            slot = a.tile_to_slot ? table_at(a.tile_to_slot, tile) : 0;
            if ((signals || a.pattern == FO_PATTERN_SUBTILE) && a.slot_group) group = table_at(a.slot_group, slot);
            if (a.pattern == FO_PATTERN_SUBTOKEN && lane < WTM) {
                bucket = a.row_bucket[row0 + lane];
                rank = a.row_rank[row0 + lane];
            }
        }
    };
    // Destination (element offset) of the plan-tile row that is row `lane` of
    // the wave's part, by pattern.
    auto find_rows = [&]() __attribute__((always_inline)) {
        if (!inside || lane >= WTM) return;
        const int r = row0 % TM + lane;
        int64_t off;
        if (a.pattern == FO_PATTERN_ROWMAJOR) {
            off = (int64_t)(row0 + lane) * a.N + col0 / TN * TN;
        } else if (a.pattern == FO_PATTERN_TILE) {
            off = ((int64_t)slot * TM + r) * TN;
        } else if (a.pattern == FO_PATTERN_SUBTILE) {
            const int h = TM / a.num_dest;
            const int k = r / h, rr = r - k * h;
            const int64_t f0 = table_at(a.group_first, group);
            const int64_t nj = table_at(a.group_first, group + 1) - f0;
            off = f0 * TM * TN + ((int64_t)k * nj + (slot - f0)) * h * TN + (int64_t)rr * TN;
        } else {
            off = ((int64_t)a.pool_off[bucket] + a.pool_base[(int64_t)slot * a.num_dest + bucket] + rank) * TN;
        }
        s_off[wave][lane] = off + col0 % TN;
    };
    // The counts of a block's plan tiles (Section 3.2), sent by the last of its
    // waves to have seen its own stores complete (the caller has waited for
    // this wave's): one add for each group, since every add of a launch meets
    // the others on one 128-byte line and takes its turn there (about 6 ns).
    auto arrive = [&](int parity) __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        if (lane != 0) return;
        if (__hip_atomic_fetch_add(&s_arrived[parity], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) !=
            kWaves - 1)
            return;
        __hip_atomic_store(&s_arrived[parity], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (MODE == kAny && a.sync == FO_SYNC_FENCE_ONE) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        int g[kWaves];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) g[w] = s_group[parity][w];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            uint32_t n = 0;
#pragma unroll
            for (int v = w; v < kWaves; ++v) {
                if (g[v] != g[w]) continue;
                ++n;
                if (v > w) g[v] = -1;
            }
            if (g[w] >= 0)
                __hip_atomic_fetch_add(a.counters + g[w], n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };

    int parity = 0;
    bool pend = false;              // the previous block's counts are still to be sent
    if (ONE || p < blocks) start();
    while (ONE || p < blocks) {
        const uint64_t t_start = traced ? wall_clock64() : 0;
        uint32_t ticket = 0;
        if (dispense && tid == 0) ticket = draw();   // used after the main loop
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        wait_and_barrier<(ST - 1) * kLoads>();
        static_for<MI + NJ>([&](auto ic) __attribute__((always_inline)) { read_one(ic, std::integral_constant<int, 0>{}, st0, fa[0], fb[0]); });
        int t = 0;
        if (steps >= ST) {
            round(0);
            t = ST;
        }
        // The previous block's stores are older than the loads that this round
        // issued, of which at most (ST - 2) steps' were in flight at its last
        // wait (a short loop: wait for everything).
        if (pend) {
            if (steps < ST) {
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(wait_imm(0, 15));
                asm volatile("" ::: "memory");
            }
            arrive(parity ^ 1);
            pend = false;
        }
        find_rows();
        for (; t + ST <= steps; t += ST) round(t);
        rest(rest, std::integral_constant<int, 0>{}, t);

        // (the ticket is waited for here, on every path, where no operand load is in flight)
        asm volatile("" : "+v"(ticket));
        int next = p + (int)gridDim.x;
        if (dispense && tid == 0) s_pos[parity] = position(ticket);
        wait_and_barrier<63>();                 // every wave has read the stages
        if (dispense) next = s_pos[parity];
        const int p_now = p, group_now = group;
        const bool inside_now = inside;
        p = __builtin_amdgcn_readfirstlane(next);
        // the next block's first loads go out ahead of this block's stores
        if (!ONE && p < blocks) start();

        if (inside_now) {
            if constexpr (WTN == 16) {
                // unsignalled: 8-byte stores from the accumulator layout (the L2
                // joins the four lanes' 32 bytes per row)
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    u32x2_t v;
                    v[0] = pack2<DT>(acc[i][0][0], acc[i][0][1]);
                    v[1] = pack2<DT>(acc[i][0][2], acc[i][0][3]);
                    *reinterpret_cast<u32x2_t*>(a.C + s_off[wave][16 * i + (lane & 15)] + 4 * (lane >> 4)) = v;
                }
            } else {
                // 16 rows at a time through the wave's own staging rows: 8 bytes
                // per lane and block in, 16-byte chunks out; chunk c of row r at
                // slot c ^ (r % chunks)
                constexpr int kCh = WTN / 8, kOut = 16 * kCh / 64;
                char* const st = s_out[wave];
                const int r = lane & 15, c0 = lane >> 5, half = (lane >> 4) & 1;
#pragma unroll
                for (int i = 0; i < MI; ++i) {
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        u32x2_t v;
                        v[0] = pack2<DT>(acc[i][j][0], acc[i][j][1]);
                        v[1] = pack2<DT>(acc[i][j][2], acc[i][j][3]);
                        *reinterpret_cast<u32x2_t*>(st + r * WTN * 2 + (((2 * j + c0) ^ (r & (kCh - 1))) << 4) +
                                                    half * 8) = v;
                    }
                    asm volatile("" ::: "memory");
#pragma unroll
                    for (int e = 0; e < kOut; ++e) {
                        const int rr = lane / kCh + e * (64 / kCh), c = lane & (kCh - 1);
                        const u32x4_t v =
                            *reinterpret_cast<const u32x4_t*>(st + rr * WTN * 2 + ((c ^ (rr & (kCh - 1))) << 4));
                        const int64_t at = s_off[wave][16 * i + rr] + 8 * c;
                        if (coherent && (MODE == kSignal || a.c_rsrc)) {
                            const __amdgpu_buffer_rsrc_t rC =
                                __builtin_amdgcn_make_buffer_rsrc((void*)a.C, 0, 0x7FFFFFFF, kRsrcWord3);
                            __builtin_amdgcn_raw_buffer_store_b128(v, rC, (uint32_t)(at * 2), 0, kCachePolicySc1);
                        } else if (coherent) {
                            uint64_t* d = reinterpret_cast<uint64_t*>(a.C + at);
                            __hip_atomic_store(d, (uint64_t)v[0] | ((uint64_t)v[1] << 32), __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                            __hip_atomic_store(d + 1, (uint64_t)v[2] | ((uint64_t)v[3] << 32), __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                        } else {
                            *reinterpret_cast<u32x4_t*>(a.C + at) = v;
                        }
                    }
                    asm volatile("" ::: "memory");
                }
            }
        }
        if constexpr (ONE) return;
        if (signals) {
            // (waves of a 64x64 block: one tile, counted once)
            if (lane == 0) s_group[parity][wave] = inside_now && (kOwnTile || wave == 0) ? group_now : -1;
            if (coherent && !traced && p < blocks) {
                pend = true;               // sent after the next block's first steps
            } else {
                if (MODE == kAny && a.sync == FO_SYNC_FENCE_ALL) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(wait_imm(0, 0));
                asm volatile("" ::: "memory");
                arrive(parity);
            }
        }
        if (!kOwnTile && traced && p_now < a.trace_cap) {   // (blocks in plan order: p is the dispatch position)
            __builtin_amdgcn_s_waitcnt(wait_imm(0, 0));
            __syncthreads();
            if (tid == 0) {
                uint64_t* t = a.trace + 4 * (int64_t)p_now;
                t[0] = t_start;
                t[1] = wall_clock64();
                t[2] = ((uint64_t)__builtin_amdgcn_s_getreg((31 << 11) | 20) << 32) |
                       (uint32_t)__builtin_amdgcn_s_getreg((31 << 11) | 4);
                t[3] = blockIdx.x;
            }
        }
        parity ^= 1;
    }
}

// Template arguments: dtype, block rows and columns, waves, stages, k values
// per step, plan tile, what the launch may do.
template <int DT, int BM, int BN, int WM, int WN, int ST, int BK, int TM, int TN, Mode MODE = kAny>
__global__ __launch_bounds__(64 * WM * WN, 1) void gemm_signal_kernel(const GemmArgs a) {
    static_assert(WM == 2 && WN == 2 && BK % 64 == 0, "2 x 2 waves");
    block_body<DT, TM, TN, BM, BN, ST, BK / 64, MODE>(a);
}

// 128x128 blocks of plan tiles TM x TN, one or two on a compute unit.
template <int DT, int TM, int TN>
void launch_128(const GemmArgs& a, int grid, bool pair, hipStream_t s) {
    if (pair)
        hipLaunchKernelGGL((gemm_signal_kernel<DT, 128, 128, 2, 2, 2, 64, TM, TN>), dim3(grid), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((gemm_signal_kernel<DT, 128, 128, 2, 2, 3, 64, TM, TN>), dim3(grid), dim3(256), 0, s, a);
}

// Stages and steps as measured (bf16, us per launch, three operand sets in
// turn): 128x128 alone on its compute unit, 3 stages of 64 (768x3840x4160 29.0; 4
// stages 29.3, 2 stages 43.7: a step's loads then have less than a step to
// land), two on a unit, 2 stages; 64x64, 4 of 64, two on a unit (64x4096x3584
// 14.2; 3 stages 16.6; 3 of 128 14.8 but one block per unit); the small blocks,
// steps of 128, since their MFMAs are too few to cover a barrier per 64 (64x32
// 128x4096x3584 12.6, in steps of 64 15.7; 32x32 64x4096x3584 9.8, 11.2). Those are
// only taken where all of a launch's blocks run at a time (`one` holds).
template <int DT>
void launch_64(const GemmArgs& a, int bm, int bn, int grid, bool pair, bool one, hipStream_t s) {
    const dim3 g(grid), b(256);
    if (bm == 128) launch_128<DT, 64, 64>(a, grid, pair, s);
    else if (bm == 64 && bn == 64 && one)
        hipLaunchKernelGGL((gemm_signal_kernel<DT, 64, 64, 2, 2, 4, 64, 64, 64, kOne>), g, b, 0, s, a);
    else if (bm == 64 && bn == 64 && !a.counters && !a.trace)
        hipLaunchKernelGGL((gemm_signal_kernel<DT, 64, 64, 2, 2, 4, 64, 64, 64, kPlain>), g, b, 0, s, a);
    else if (bm == 64 && bn == 64 && a.counters && !a.trace && a.sync == FO_SYNC_COHERENT && a.c_rsrc)
        hipLaunchKernelGGL((gemm_signal_kernel<DT, 64, 64, 2, 2, 4, 64, 64, 64, kSignal>), g, b, 0, s, a);
    else if (bm == 64 && bn == 64)
        hipLaunchKernelGGL((gemm_signal_kernel<DT, 64, 64, 2, 2, 4, 64, 64, 64>), g, b, 0, s, a);
    else if (bm == 64)
        hipLaunchKernelGGL((gemm_signal_kernel<DT, 64, 32, 2, 2, 3, 128, 64, 64, kOne>), g, b, 0, s, a);
    else hipLaunchKernelGGL((gemm_signal_kernel<DT, 32, 32, 2, 2, 4, 128, 64, 64, kOne>), g, b, 0, s, a);
}

// Whether 128x128 blocks run in pairs on a compute unit. A pair takes about 1.7
// times a single block's time (its two stages hide less, its two workgroups
// cover each other's barriers, prologues and epilogues), so it pays where it
// saves enough rounds (bf16 us, single / pair, blocks in W): 1.1 W K 2048
// 32.9 / 27.2; 2.2 W K 1920 49.9 / 51.4, K 1024 31.8 / 28.5; 3 W K 5440
// 151 / 156; 4 W K 4032 145 / 138; 4.4 W K 320 30.5 / 22.0. Signalled, a second
// round of a pair draws its positions one by one from the same line: one round
// only (1.1 W 34.8 / 27.6; 4.4 W K 320 34.9 / 38.5).
bool in_pairs(const GemmArgs& a, int64_t blocks, int64_t W, bool share_cus) {
    if (!share_cus || blocks <= W) return false;
    if (a.counters) return blocks <= 2 * W;
    return a.K <= 1024 || 17 * ((blocks + 2 * W - 1) / (2 * W)) < 10 * ((blocks + W - 1) / W);
}

}  // namespace

// The block of a launch, from the number of 64x64 tiles and the workgroups
// that run at a time (the plan's wave width W; bf16 us per launch, W = 256):
//   tiles <= W/4   32x32   64 tiles, K 3584: 9.8 (64x32 12.2, 64x64 14.2)
//   tiles <= W/2   64x32   128 tiles, K 3584: 12.6 (32x32 13.4, 64x64 14.3)
//   tiles <= 2 W   64x64   256 tiles, K 1024: 7.7 (64x32 8.9, 128x128 11.5);
//                          336 tiles, K 2048: 14.9 (16.4 in 128x128, 18.1 one
//                          block per compute unit); 512 tiles: 26.2 (26.9)
//                          (these three 1.5 less since in the kOne form)
//   above          128x128 720 tiles, K 4160: 29.0 (64x64 38.5);
//                          2272 tiles, K 1920: 48.7 (57.2)
// Parts of a tile have no count of their own: a signalled launch takes whole
// tiles. Two blocks share a compute unit only if the plan reserves no units for
// communication (a second block would be placed on those). A traced launch runs
// in tiles, one per dispatch position.
hipError_t launch_gemm64(int dtype, GemmArgs a, int wave_width, bool share_cus, hipStream_t s) {
    const int64_t tiles = (int64_t)a.tiles_m * a.tiles_n, W = wave_width;
    int bm = 64, bn = 64;
    if (!a.trace) {
        if (!a.counters && tiles <= W / 4) bm = bn = 32;
        else if (!a.counters && tiles <= W / 2) bn = 32;
        // (128 rows of K must fit the buffer resources' 31-bit byte range)
        else if (tiles > 2 * W && a.K <= INT32_MAX / 256) bm = bn = 128;
    }
    a.blocks_m = (int)((a.M + bm - 1) / bm);
    a.blocks_n = (int)((a.N + bn - 1) / bn);
    // the same number of output rows per band as in the plan's order
    a.block_band = block_band(a.group_m, 64, bm, a.blocks_m);
    const int64_t blocks = (int64_t)a.blocks_m * a.blocks_n;
    const bool pair = bm == 128 ? in_pairs(a, blocks, W, share_cus) : bn == 64 && share_cus && !a.trace;
    const int grid = (int)std::min<int64_t>(blocks, pair ? 2 * W : W);
    a.num_dispensers = std::max(1, std::min(a.num_dispensers, grid));
    const bool one = !a.counters && !a.trace && grid == blocks;
    if (dtype == FO_FP16) launch_64<FO_FP16>(a, bm, bn, grid, pair, one, s);
    else launch_64<FO_BF16>(a, bm, bn, grid, pair, one, s);
    return hipGetLastError();
}

// By the rule of takes_parts; unsignalled, untraced launches only (a part has no
// count and no position of its own).
bool gemm_in_parts(int tile_n, const GemmArgs& a, int wave_width, bool share_cus) {
    return !a.counters && !a.trace &&
           takes_parts(tile_n, (int64_t)a.tiles_m * a.tiles_n, wave_width, a.K, share_cus);
}

hipError_t launch_gemm_parts(int dtype, int tile_n, GemmArgs a, int wave_width, bool share_cus, hipStream_t s) {
    a.blocks_m = (int)(a.M / 128);
    a.blocks_n = (int)(a.N / 128);
    a.block_band = block_band(a.group_m, 256, 128, a.blocks_m);
    a.num_dispensers = 1;
    const int64_t blocks = (int64_t)a.blocks_m * a.blocks_n, W = wave_width;
    const bool pair = in_pairs(a, blocks, W, share_cus);
    const int grid = (int)std::min<int64_t>(blocks, pair ? 2 * W : W);
    if (dtype == FO_FP16 && tile_n == 128) launch_128<FO_FP16, 256, 128>(a, grid, pair, s);
    else if (dtype == FO_FP16) launch_128<FO_FP16, 256, 256>(a, grid, pair, s);
    else if (tile_n == 128) launch_128<FO_BF16, 256, 128>(a, grid, pair, s);
    else launch_128<FO_BF16, 256, 256>(a, grid, pair, s);
    return hipGetLastError();
}

}  // namespace fo
