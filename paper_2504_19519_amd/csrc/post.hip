// Post-communication reorder fused into the following element-wise kernel
// (Section 3.3 Approach, last paragraph: the kernel after communication
// loads by the reordered index; Section 6.6 fuses it with RMSNorm).
//
// One wave per output row and four rows per workgroup, or a workgroup per row
// (post_form). A lane handles every 64th (256th) 16-byte chunk of the row. A
// chunk lies inside one tile
// column, so its source is 16 contiguous bytes of one row piece: the row's
// place in that tile's slot (tile pattern), in the slice's destination
// buffer (subtile pattern) or in the row's pool (subtoken pattern), and
// lanes of one tile column read one contiguous tile_n-wide piece.
//
// The workgroup first resolves the reorder map for its rows: for every
// (row, tile column) it writes the offset of the source piece to LDS. After
// that a chunk's source address is one LDS read and an add, so all of a
// lane's loads can be in flight at once.
//
// Two kernels:
//   post_gather_kernel  the plain restore (bit-exact copy): 16 loads per lane
//                       in flight before their stores;
//   post_norm_kernel    bias add and/or RMSNorm: the row is loaded up front
//                       and held in registers between the sum-of-squares and
//                       the scaling (rows up to 16384 wide; bias and gamma in
//                       LDS where four rows share them), or read twice for
//                       wider rows; which of bias, RMSNorm and gamma run is a
//                       compile-time choice.
// Each also in a fused form that is the consumer as well, for runs on one
// stream and for overlapped runs whose groups are consumed together: it reads
// the GEMM's output and the peer's partial and writes the consumer's buffer and
// the output. Both are bound by memory: 8192x8192 restore 49 us and fused 89 us
// (5.5 and 6.0 TB/s; a large copy reaches 5.1).
// Sources are read through the caches (the consumer has just written them,
// so part of them is still in the memory-side cache); the output is written
// nontemporal.
#include <hip/hip_runtime.h>

#include "consume.h"
#include "fo_device.h"
#include "fo_internal.h"
#include "post.h"

namespace fo {
namespace {

constexpr int kThreads = 256;
// FUSE: the restore alone; the consumer as well; and for overlapped runs, where the
// launch looks at the run's gate word and counts its workgroups (a form of its own:
// with branches on the arguments a one-stream run of 2048x4096x4096 took 75.7 us
// instead of 74.9).
enum { kApart = 0, kFused = 1, kFusedGated = 2 };
constexpr int kRsrcWord3 = 0x00020000;      // raw byte-addressed buffer accesses
constexpr int kSc1Nt = 16 | 2;              // cache policy: device-coherent and nontemporal
constexpr int kWaitVmcnt0 = 0x0F70;         // s_waitcnt operand: vmcnt(0), other counters not waited for

typedef __attribute__((address_space(3))) char lds_char_t;
typedef __attribute__((address_space(3))) uint32_t lds_u32_t;
typedef __attribute__((address_space(3))) u32x4_t lds_u32x4_t;

template <int DT>
__device__ __forceinline__ void widen8(u32x4_t v, float* f) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f[2 * e] = to_f32<DT>(v[e] & 0xFFFFu);
        f[2 * e + 1] = to_f32<DT>(v[e] >> 16);
    }
}

// Where the tile_n-wide piece of output row i in tile column tn lies, in
// 16-byte chunks: [0] in the consumer's buffer; [1] (FUSE) in the GEMM's output
// and the peer's partial.
template <int FUSE>
__device__ __forceinline__ u32x2_t piece_offset(const PostArgs& a, int64_t i, int tn) {
    const int64_t tw = a.tile_n;
    int64_t off, from;
    if (a.pattern == FO_PATTERN_ROWMAJOR) {
        off = from = i * a.N + tn * tw;
    } else {
        const int32_t tm = (int32_t)(i / a.tile_m);
        const int32_t r = (int32_t)(i - (int64_t)tm * a.tile_m);
        const int64_t slot = a.tile_to_slot[(int64_t)tm * a.tiles_n + tn];
        if (a.pattern == FO_PATTERN_TILE) {
            off = from = (slot * a.tile_m + r) * tw;
        } else if (a.pattern == FO_PATTERN_SUBTILE) {
            const int32_t h = a.tile_m / a.num_dest;
            const int32_t k = r / h;
            off = (int64_t)a.dest_perm[k] * a.per_dest + (slot * h + (r - k * h)) * tw;
            if constexpr (FUSE) {
                const int32_t j = a.slot_group[slot];
                const int64_t f0 = a.group_first[j], nj = a.group_first[j + 1] - f0;
                from = f0 * a.tile_m * tw + ((k * nj + (slot - f0)) * h + (r - k * h)) * tw;
            }
        } else {
            const int32_t b = a.row_bucket[i];
            off = from = ((int64_t)a.pool_off[b] + a.pool_base[slot * a.num_dest + b] + a.row_rank[i]) * tw;
        }
    }
    u32x2_t p;
    p[0] = (uint32_t)(off >> 3);
    p[1] = FUSE ? (uint32_t)(from >> 3) : 0u;
    return p;
}

// What a workgroup knows about its rows: the pieces of rows i0 .. i0 + ROWS - 1
// in LDS (one word per piece, or two with FUSE).
template <int FUSE>
struct Pieces {
    lds_u32_t* at;
    __device__ __forceinline__ void stage(const PostArgs& a, int64_t i0, int rows) const {
        const int n = rows * a.tiles_n;
        for (int idx = threadIdx.x; idx < n; idx += kThreads) {
            const int w = idx / a.tiles_n, tn = idx - w * a.tiles_n;
            const int64_t i = i0 + w;
            if (i < a.M) {
                const u32x2_t p = piece_offset<FUSE>(a, i, tn);
                at[FUSE ? 2 * idx : idx] = p[0];
                if constexpr (FUSE) at[2 * idx + 1] = p[1];
            }
        }
    }
    // where chunk c of the block's row w lies
    __device__ __forceinline__ u32x2_t chunk(const PostArgs& a, int w, uint32_t c) const {
        const uint32_t idx = (uint32_t)w * a.tiles_n + (c >> a.cpt_log2), in = c & ((1u << a.cpt_log2) - 1u);
        u32x2_t p;
        if constexpr (FUSE) {
            p = *reinterpret_cast<__attribute__((address_space(3))) u32x2_t*>(at + 2 * idx);
            p[1] += in;
        } else {
            p[0] = at[idx];
            p[1] = 0u;
        }
        p[0] += in;
        return p;
    }
};

// B chunks of the block's row w: chunk c0 + step t, past the row's end its last
// chunk (dropped by the caller). FUSE: the chunk is consumed on the way, as
// the consumer does it: the GEMM's output plus the peer's partial (if any),
// rounded, which is also what the consumer's buffer gets.
template <int DT, int FUSE, int B>
__device__ __forceinline__ void load_chunks(const PostArgs& a, const Pieces<FUSE>& pieces, int w, int c0, int step,
                                            int nch, u32x4_t* v) {
    if constexpr (!FUSE) {
#pragma unroll
        for (int t = 0; t < B; ++t) {
            const int c = c0 + step * t;
            v[t] = reinterpret_cast<const u32x4_t*>(a.src)[pieces.chunk(a, w, c < nch ? c : nch - 1)[0]];
        }
    } else {
        const __amdgpu_buffer_rsrc_t rc =
            __builtin_amdgcn_make_buffer_rsrc((void*)a.gemm_out, 0, (int)a.bytes, kRsrcWord3);
        const u32x4_t* q = reinterpret_cast<const u32x4_t*>(a.peer);
        const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc((void*)a.src, 0, (int)a.bytes, kRsrcWord3);
        constexpr int S = B < 8 ? B : 8;            // chunks in flight at once
#pragma unroll
        for (int b = 0; b < B; b += S) {
            u32x4_t y[S];
            uint32_t to[S];
#pragma unroll
            for (int t = 0; t < S; ++t) {
                const int c = c0 + step * (b + t);
                const u32x2_t p = pieces.chunk(a, w, c < nch ? c : nch - 1);
                to[t] = p[0];
                v[b + t] = bit_cast<u32x4_t>(__builtin_amdgcn_raw_buffer_load_b128(rc, (int)(p[1] * 16u), 0, kSc1Nt));
                if (q) y[t] = __builtin_nontemporal_load(q + p[1]);
            }
#pragma unroll
            for (int t = 0; t < S; ++t) {
                if (q) v[b + t] = add8<DT>(v[b + t], y[t]);
                if (c0 + step * (b + t) < nch)
                    __builtin_amdgcn_raw_buffer_store_b128(v[b + t], rd, (int)(to[t] * 16u), 0, kSc1Nt);
            }
        }
    }
}

// Chunk c of the output row that starts at chunk `row`. The fused form writes
// device-coherent (at the same rate), so that its workgroups can be counted.
template <int FUSE>
__device__ __forceinline__ void put_out(const PostArgs& a, u32x4_t* out4, int64_t row, int c, u32x4_t v) {
    if constexpr (FUSE) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)a.out, 0, (int)a.bytes, kRsrcWord3);
        __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)((uint32_t)(row + c) * 16u), 0, kSc1Nt);
    } else {
        __builtin_nontemporal_store(v, out4 + c);
    }
}

// The barrier behind the pieces, and whether the workgroup may write: the gate
// word still holds the run's tag (see post.h). One thread has read the word ahead
// of the pieces (`seen`), so that the two reads' latencies overlap (1216x2880x1984
// 31.6 us per run with and without the gate; with a read in every wave 33). Acquire
// is left to the gate kernel ahead on the stream.
template <int FUSE>
__device__ __forceinline__ uint32_t read_gate(const PostArgs& a) {
    if constexpr (FUSE == kFusedGated) {
        if (threadIdx.x == 0) return __hip_atomic_load(a.gate, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return 0u;
}
template <int FUSE>
__device__ __forceinline__ bool meet(const PostArgs& a, uint32_t seen) {
    if constexpr (FUSE == kFusedGated) {
        __shared__ int s_go;
        if (threadIdx.x == 0) s_go = seen == a.gate_tag;
        __syncthreads();
        return s_go != 0;
    } else {
        __syncthreads();
        return true;
    }
}

// End of a gated launch's workgroup that is counted (as the consumer's final
// launch counts its own): its write-through stores are complete.
template <int FUSE>
__device__ __forceinline__ void finished(const PostArgs& a) {
    if constexpr (FUSE == kFusedGated) {
        if (!a.done) return;
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        __syncthreads();
        if (threadIdx.x == 0) count_done(a.done, a.done_tag);
    }
}

// WPR waves per output row (one, or a whole workgroup), 4 / WPR rows per
// workgroup.
template <int DT, int WPR, int FUSE>
__global__ __launch_bounds__(kThreads) void post_gather_kernel(const PostArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int kRows = kThreads / 64 / WPR, kLanes = 64 * WPR;
    const Pieces<FUSE> pieces{reinterpret_cast<lds_u32_t*>((lds_char_t*)smem)};
    const int lane = threadIdx.x % kLanes, w = threadIdx.x / kLanes;
    const int64_t i0 = (int64_t)blockIdx.x * kRows, i = i0 + w;
    const uint32_t seen = read_gate<FUSE>(a);
    pieces.stage(a, i0, kRows);
    if (!meet<FUSE>(a, seen)) return;
    if (i < a.M) {
        const int nch = (int)(a.N >> 3);
        constexpr int B = FUSE ? 8 : 16;
        u32x4_t* out4 = reinterpret_cast<u32x4_t*>(a.out + i * a.N);
        for (int c0 = lane; c0 < nch; c0 += kLanes * B) {
            u32x4_t v[B];
            if constexpr (FUSE) {
                load_chunks<DT, FUSE, B>(a, pieces, w, c0, kLanes, nch, v);
            } else {
#pragma unroll
                for (int t = 0; t < B; ++t)
                    if (c0 + kLanes * t < nch)
                        v[t] = reinterpret_cast<const u32x4_t*>(a.src)[pieces.chunk(a, w, c0 + kLanes * t)[0]];
            }
#pragma unroll
            for (int t = 0; t < B; ++t)
                if (c0 + kLanes * t < nch) put_out<FUSE>(a, out4, i * nch, c0 + kLanes * t, v[t]);
        }
    }
    finished<FUSE>(a);
}

// y = (x + bias) [* rsqrt(mean((x + bias)^2) + eps) * gamma]. NORM, BIAS and
// GAMMA fix at compile time which parts run (GAMMA only with NORM), so that
// no per-chunk branch and no value of an unused part holds registers. CH > 0:
// chunks of the row that a lane holds; CH == 0: the row is read twice.
template <int DT, int CH, int WPR, int FUSE, bool NORM, bool BIAS, bool GAMMA>
__global__ __launch_bounds__(kThreads) void post_norm_kernel(const PostArgs a) {
    static_assert(CH > 0 || (WPR == 1 && !FUSE), "rows read twice: one wave each, not fused");
    // bias and gamma in LDS where the workgroup's waves share them
    constexpr bool kLdsAffine = (BIAS || GAMMA) && CH > 0 && WPR == 1;
    constexpr int kRows = kThreads / 64 / WPR, kLanes = 64 * WPR;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int nch = (int)(a.N >> 3);
    // LDS: [bias chunks][gamma chunks] (with kLdsAffine), then the pieces
    lds_u32x4_t* s_bias = reinterpret_cast<lds_u32x4_t*>((lds_char_t*)smem);
    lds_u32x4_t* s_gamma = s_bias + (kLdsAffine ? nch : 0);
    const Pieces<FUSE> pieces{reinterpret_cast<lds_u32_t*>(s_gamma + (kLdsAffine ? nch : 0))};
    const int lane = threadIdx.x % kLanes, w = threadIdx.x / kLanes;
    const int64_t i0 = (int64_t)blockIdx.x * kRows, i = i0 + w;
    const u32x4_t* bias4 = reinterpret_cast<const u32x4_t*>(a.bias);
    const u32x4_t* gamma4 = reinterpret_cast<const u32x4_t*>(a.gamma);
    if constexpr (kLdsAffine) {
        for (int c = threadIdx.x; c < nch; c += kThreads) {
            if constexpr (BIAS) s_bias[c] = bias4[c];
            if constexpr (GAMMA) s_gamma[c] = gamma4[c];
        }
    }
    const uint32_t seen = read_gate<FUSE>(a);
    pieces.stage(a, i0, kRows);
    if (!meet<FUSE>(a, seen)) return;
    u32x4_t* out4 = reinterpret_cast<u32x4_t*>(a.out + i * a.N);
    __shared__ float s_sum[WPR > 1 ? WPR : 1];

    // h = x + bias (fp32, no rounding); sb: where bias chunks are read
    auto shift = [&](u32x4_t xv, int c, const lds_u32x4_t* sb, float* h) {
        widen8<DT>(xv, h);
        if constexpr (BIAS) {
            float bv[8];
            widen8<DT>(kLdsAffine ? sb[c] : bias4[c], bv);
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] += bv[e];
        }
    };
    auto sumsq = [&](u32x4_t xv, int c, const lds_u32x4_t* sb) {
        float h[8];
        shift(xv, c, sb, h);
        float q = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) q += h[e] * h[e];
        return q;
    };
    auto finish = [&](int c, u32x4_t xv, float inv, const lds_u32x4_t* sb, const lds_u32x4_t* sg) -> u32x4_t {
        float h[8], gv[8];
        shift(xv, c, sb, h);
        if constexpr (GAMMA) widen8<DT>(kLdsAffine ? sg[c] : gamma4[c], gv);
        u32x4_t o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float y0 = h[2 * e], y1 = h[2 * e + 1];
            if constexpr (NORM) {
                y0 *= inv;
                y1 *= inv;
                if constexpr (GAMMA) {
                    y0 *= gv[2 * e];
                    y1 *= gv[2 * e + 1];
                }
            }
            o[e] = pack2<DT>(y0, y1);
        }
        return o;
    };
    auto rsqrt_mean = [&](float ss) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
        if constexpr (WPR > 1) {
            if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = ss;
            __syncthreads();
            ss = 0.0f;
#pragma unroll
            for (int v = 0; v < WPR; ++v) ss += s_sum[v];
        }
        return 1.0f / sqrtf(ss / (float)a.N + a.eps);
    };

    if constexpr (CH > 0) {
        // (a workgroup per row: i < M always, so its waves meet in rsqrt_mean)
        if (i < a.M) {
            // The row is loaded up front. Lanes past the row's end load its
            // last chunk (no branches around the loads: the array stays in
            // registers) and drop the result.
            u32x4_t xc[CH];
            load_chunks<DT, FUSE, CH>(a, pieces, w, lane, kLanes, nch, xc);
            float inv = 1.0f;
            if constexpr (NORM) {
                float ss = 0.0f;
#pragma unroll
                for (int t = 0; t < CH; ++t) {
                    const int c = lane + kLanes * t;
                    const float q = sumsq(xc[t], c < nch ? c : nch - 1, s_bias);
                    ss += c < nch ? q : 0.0f;
                    // one bias chunk at a time: the LDS reads are not all hoisted
                    // to the top, where their values would hold registers
                    if constexpr (kLdsAffine) asm volatile("" ::: "memory");
                }
                inv = rsqrt_mean(ss);
            }
            // The scaling pass widens the chunks again and reads bias and gamma
            // again, through pointers the compiler cannot match with the first
            // pass's, instead of keeping the first pass's values alive.
#pragma unroll
            for (int t = 0; t < CH; ++t) asm volatile("" : "+v"(xc[t]));
            // The lane index is laundered too, so that the second pass's addresses
            // are formed here and not kept live through the first pass.
            const lds_u32x4_t* sb = s_bias;
            const lds_u32x4_t* sg = s_gamma;
            int ln = lane;
            asm volatile("" : "+v"(sb), "+v"(sg), "+v"(ln));
#pragma unroll
            for (int t = 0; t < CH; ++t) {
                const int c = ln + kLanes * t;
                const u32x4_t o = finish(c < nch ? c : nch - 1, xc[t], inv, sb, sg);
                if (c < nch) put_out<FUSE>(a, out4, i * nch, c, o);
                if constexpr (kLdsAffine) asm volatile("" ::: "memory");
            }
        }
        finished<FUSE>(a);
    } else {
        if (i >= a.M) return;
        auto at = [&](int c) { return reinterpret_cast<const u32x4_t*>(a.src)[pieces.chunk(a, w, c)[0]]; };
        float inv = 1.0f;
        if constexpr (NORM) {
            float ss = 0.0f;
            for (int c = lane; c < nch; c += 64) ss += sumsq(at(c), c, s_bias);
            inv = rsqrt_mean(ss);
        }
        for (int c = lane; c < nch; c += 64)
            __builtin_nontemporal_store(finish(c, at(c), inv, s_bias, s_gamma), out4 + c);
    }
}

template <int DT, int CH, int WPR, int FUSE>
void launch_norm(const PostArgs& a, dim3 g, size_t lds, hipStream_t s) {
    const dim3 b(kThreads);
    const bool bias = a.bias != nullptr, gamma = a.do_norm && a.gamma != nullptr;
    if (!a.do_norm) hipLaunchKernelGGL((post_norm_kernel<DT, CH, WPR, FUSE, false, true, false>), g, b, lds, s, a);
    else if (bias && gamma)
        hipLaunchKernelGGL((post_norm_kernel<DT, CH, WPR, FUSE, true, true, true>), g, b, lds, s, a);
    else if (bias) hipLaunchKernelGGL((post_norm_kernel<DT, CH, WPR, FUSE, true, true, false>), g, b, lds, s, a);
    else if (gamma) hipLaunchKernelGGL((post_norm_kernel<DT, CH, WPR, FUSE, true, false, true>), g, b, lds, s, a);
    else hipLaunchKernelGGL((post_norm_kernel<DT, CH, WPR, FUSE, true, false, false>), g, b, lds, s, a);
}

template <int DT, int FUSE>
void launch_form(const PostArgs& a, const PostForm& f, hipStream_t s) {
    const dim3 g(f.blocks);
    if (f.chunks < 0) {
        if (f.waves_per_row == 1)
            hipLaunchKernelGGL((post_gather_kernel<DT, 1, FUSE>), g, dim3(kThreads), f.lds, s, a);
        else hipLaunchKernelGGL((post_gather_kernel<DT, 4, FUSE>), g, dim3(kThreads), f.lds, s, a);
    } else if (f.waves_per_row == 4) {
        if (f.chunks == 2) launch_norm<DT, 2, 4, FUSE>(a, g, f.lds, s);
        else if (f.chunks == 4) launch_norm<DT, 4, 4, FUSE>(a, g, f.lds, s);
        else launch_norm<DT, 8, 4, FUSE>(a, g, f.lds, s);
    } else if (f.chunks == 4) {
        launch_norm<DT, 4, 1, FUSE>(a, g, f.lds, s);
    } else if (f.chunks == 8) {
        launch_norm<DT, 8, 1, FUSE>(a, g, f.lds, s);
    } else if (f.chunks == 16) {
        launch_norm<DT, 16, 1, FUSE>(a, g, f.lds, s);
    } else if constexpr (!FUSE) {
        launch_norm<DT, 0, 1, kApart>(a, g, f.lds, s);
    }
}

template <int DT>
void launch_fused(const PostArgs& a, const PostForm& f, hipStream_t s) {
    if (a.gate) launch_form<DT, kFusedGated>(a, f, s);
    else launch_form<DT, kFused>(a, f, s);
}

}  // namespace

PostForm post_form(const PostArgs& a, bool fused) {
    const int64_t nch = a.N >> 3;
    PostForm f{};
    const bool norm = a.do_norm || a.bias;
    const bool affine = norm && (a.bias || a.gamma);
    // A workgroup per row where one wave could not hold the row in registers
    // (us, one wave -> four: 1280x12288 bias + RMSNorm 25.3 -> 11.8), where the
    // rows are too few to fill the device with waves (64x4096 fused 8.4 -> 5.9,
    // 512x4096 8.9 -> 7.1; 640x2560 the other way, 5.7 -> 6.7), and for long rows
    // (restore 8192x8192 52.7 -> 48.7, fused 103 -> 89; 4096x7168 with RMSNorm
    // fused 37.5 -> 36.1, with bias 21.4 -> 19.7), unless many rows share bias
    // and gamma, which four one-wave rows read from LDS (8192x8192 56.2 against
    // 59.5). Shorter rows: one wave (2048x4096 6.5 -> 6.8, 8192x2048 11.9 -> 12.9).
    const bool wide = nch > 64 * 16 || (a.M <= 512 && nch >= 256) ||
                      ((affine || fused ? nch > 512 : nch >= 1024) && (!affine || a.M <= 4096));
    f.waves_per_row = wide && (!norm || nch <= 256 * 8) ? 4 : 1;
    if (!norm) f.chunks = -1;
    else if (f.waves_per_row == 4) f.chunks = nch <= 256 * 2 ? 2 : nch <= 256 * 4 ? 4 : 8;
    else f.chunks = nch <= 64 * 4 ? 4 : nch <= 64 * 8 ? 8 : nch <= 64 * 16 ? 16 : 0;
    const int rows = kThreads / 64 / f.waves_per_row;
    f.blocks = (uint32_t)((a.M + rows - 1) / rows);
    const bool lds_affine = norm && (a.bias || a.gamma) && f.waves_per_row == 1 && f.chunks > 0;
    f.lds = (size_t)rows * a.tiles_n * sizeof(uint32_t) * (fused ? 2 : 1) + (lds_affine ? 2 * (size_t)nch * 16 : 0);
    return f;
}

bool post_fusable(const PostArgs& a) {
    const PostForm f = post_form(a, true);
    return f.chunks != 0 && f.lds <= kMaxPostLds && a.M * a.N * 2 <= INT32_MAX && a.M * a.N > 0;
}

hipError_t launch_post(int dtype, const PostArgs& a, bool fused, hipStream_t s) {
    if (a.M == 0 || a.N == 0) return hipSuccess;
    const PostForm f = post_form(a, fused);
    if (dtype == FO_FP16) {
        if (fused) launch_fused<FO_FP16>(a, f, s);
        else launch_form<FO_FP16, kApart>(a, f, s);
    } else {
        if (fused) launch_fused<FO_BF16>(a, f, s);
        else launch_form<FO_BF16, kApart>(a, f, s);
    }
    return hipGetLastError();
}

}  // namespace fo
