// Launch interface of the post-communication reorder kernel (internal).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fo {

struct PostArgs {
    const uint16_t* src;        // consumer destination buffer
    uint16_t* out;              // [M, N] row-major
    const uint16_t* bias;       // [N] or null
    const uint16_t* gamma;      // [N] or null
    int64_t M, N;
    int32_t tile_m, tile_n, tiles_n, pattern, num_dest;
    int32_t cpt_log2;           // log2(tile_n / 8) for reordered patterns; 31 for row-major
                                // (a row is one piece)
    int64_t per_dest;           // SUBTILE: elements of one destination buffer
    const int32_t* tile_to_slot;
    const int32_t* dest_perm;
    const int32_t* row_bucket;
    const int32_t* row_rank;
    const int32_t* pool_base;
    const int32_t* pool_off;
    float eps;
    int32_t do_norm;
    // The fused form is the consumer as well: it reads the GEMM's output (and
    // the peer's partial, if any), each of `bytes`, and fills src itself.
    const uint16_t* gemm_out;
    const uint16_t* peer;
    uint32_t bytes;
    const int32_t* slot_group;
    const int32_t* group_first;
    // Fused launches of an overlapped run: workgroups that find another value than
    // gate_tag in the gate word (a wait of the run has given up) write nothing and
    // are not counted. Null: no gate.
    const uint32_t* gate;
    uint32_t gate_tag;
    uint32_t done_tag;
    uint32_t* done;             // with a gate: counts finished workgroups (see ConsumeArgs), or null
};

// The kernel form of a launch.
struct PostForm {
    int32_t waves_per_row;      // 1 or 4
    int32_t chunks;             // 16-byte chunks of a row per lane; 0: rows read twice; -1: plain restore
    uint32_t blocks;
    size_t lds;                 // bytes per workgroup
};
constexpr size_t kMaxPostLds = 64 * 1024;
// LDS bytes per workgroup by which a size is accepted or refused, whatever form
// it then takes: four rows' piece offsets, and bias and gamma of a row of up to
// 8192 columns.
inline size_t post_lds_bound(const PostArgs& a) {
    const bool affine = (a.do_norm || a.bias) && (a.bias || a.gamma) && a.N <= 8192;
    return 16 * (size_t)a.tiles_n + (affine ? 4 * (size_t)a.N : 0);
}

PostForm post_form(const PostArgs& a, bool fused);
// Whether the fused form exists for these sizes.
bool post_fusable(const PostArgs& a);
hipError_t launch_post(int dtype, const PostArgs& a, bool fused, hipStream_t s);

}  // namespace fo
