// Launch interface of the consumer kernels (internal to libfo).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fo {

// Largest consumer grid: one workgroup per compute unit.
constexpr int kMaxConsumeBlocks = 256;
// Segments one launch can carry (a group has R or B of them).
constexpr int kMaxConsumeSegments = 16;

// One contiguous piece of a group: `len` elements at src + src_off (and
// peer + src_off) go to dst + dst_off.
struct ConsumeSegment {
    int64_t src_off, dst_off, len;
};

struct ConsumeArgs {
    const uint16_t* src;
    const uint16_t* peer;        // nullptr: copy
    uint16_t* dst;
    const uint32_t* counter;     // nullptr: no wait
    uint32_t target;
    uint32_t* status;            // bit 0 set on a timed-out wait (may be nullptr)
    uint64_t timeout_ticks;      // wall-clock ticks
    uint32_t* done;              // non-null: done word 0; workgroup b adds 1 to word b % kDoneWords
                                 // (kDoneStride words apart) when its stores are visible, while
                                 // that word's high half equals done_tag's
    uint32_t done_tag;           // run tag of the done word (done_tag_of)
    int32_t nseg;                // 1 .. kMaxConsumeSegments
    ConsumeSegment seg[kMaxConsumeSegments];
};

// One launch: wait once for *counter >= target, then stream every segment.
// max_blocks caps the grid (1 .. kMaxConsumeBlocks); threads per workgroup:
// 64, 128 or 256. full: the launch has the device to itself (more accesses
// in flight per thread); otherwise it runs beside the GEMM and keeps its
// registers within what a SIMD running two GEMM waves has left. ring: a launch
// of one-wave workgroups may stream through LDS (coherent mode, 16-byte aligned
// buffers, one segment, not counted).
// *blocks (if non-null) receives the streaming kernel's grid size.
hipError_t launch_consume(int dtype, int sync, const ConsumeArgs& a, int max_blocks, int threads, bool full, bool ring,
                          hipStream_t s, int* blocks = nullptr);

// One wave that polls until *counter >= target (bounded by timeout_ticks;
// on timeout bit 0 of *status is raised).
hipError_t launch_wait(const uint32_t* counter, uint32_t target, uint32_t* status, uint64_t timeout_ticks,
                       hipStream_t s);

// Tags of the start handoff of an overlapped run: the run's reset kernel
// writes its tag (bit 31 and 30 bits of the run's sequence number) into the
// gate word once the counters are zero; the gate kernel on the other stream
// waits for that tag. A gate that times out while the word holds no later
// run's tag replaces it by tag | kGateTimedOut, which the reset kernel, if it
// runs later, leaves there and turns into bit 0 of the status word; a gate that
// times out after a later run's tag has arrived only raises the status bit. The
// done wait clears the word at the run's end, be it whole or timed out. So the
// word holds a run's tag only while none of its waits has given up, and a launch
// that may write what later work of the GEMM stream reads looks there first.
constexpr uint32_t kGateTag = 0x80000000u;
constexpr uint32_t kGateTimedOut = 0x40000000u;
constexpr uint32_t kGateSeqMask = kGateTimedOut - 1;
// Done words of an overlapped run: the low 16 bits of the run's sequence
// number in the high half, a count of finished final-consumer workgroups in
// the low half. The count is spread over kDoneWords words kDoneStride words
// apart (each in a 128-byte line of its own): workgroup b counts in word
// b % kDoneWords, so that at most ceil(grid / kDoneWords) device-scope adds
// meet on one address (256 adds on one word took ~8 us to drain).
constexpr int kDoneWords = 8;
constexpr int kDoneStride = 32;
__host__ __device__ inline uint32_t done_tag_of(uint32_t seq) { return (seq & 0xFFFFu) << 16; }
// Workgroups b < blocks with b % kDoneWords == k.
__host__ __device__ inline uint32_t done_share(int32_t blocks, int k) {
    return blocks > k ? (uint32_t)((blocks - 1 - k) / kDoneWords + 1) : 0u;
}
#if defined(__HIPCC__)
// One finished workgroup of the final launch (its stores complete), counted for
// its own run only: once a later run's reset has put its tag into the word, a
// late workgroup leaves it alone. (A plain add after the check: a
// compare-and-swap loop would serialise the grid's workgroups on one word,
// about a microsecond each. A late workgroup can only race with a later run's
// reset if an earlier wait of the stream pair timed out, which the sticky
// status bit already reports.)
__device__ __forceinline__ void count_done(uint32_t* done, uint32_t done_tag) {
    uint32_t* w = done + (blockIdx.x % kDoneWords) * kDoneStride;
    const uint32_t v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((v & 0xFFFF0000u) == done_tag) __hip_atomic_fetch_add(w, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
#endif
// One wave that polls the done words until word k reaches done_tag plus
// done_share(blocks, k) for every k (bounded like launch_wait), then clears the
// gate word (after a time-out if it holds the run's tag or its mark).
hipError_t launch_done_wait(const uint32_t* done, uint32_t done_tag, int32_t blocks, uint32_t* gate, uint32_t tag,
                            uint32_t* status, uint64_t timeout_ticks, hipStream_t s);
hipError_t launch_gate(uint32_t* gate, uint32_t tag, uint32_t* status, uint64_t timeout_ticks, hipStream_t s);
// One thread that counts as the only workgroup of a final launch, behind a
// launch that does not count itself; nothing unless the gate word holds the
// run's tag.
hipError_t launch_mark_done(uint32_t* done, uint32_t done_tag, const uint32_t* gate, uint32_t tag, hipStream_t s);

}  // namespace fo
