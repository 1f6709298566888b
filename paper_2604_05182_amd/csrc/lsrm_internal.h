// Internal declarations shared by the HIP translation units of liblsrm (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/lsrm.h"

namespace lsrm {

constexpr int kBlock = 64;

struct Shape {
    int n_obj, n_views, grid, h, d, topk, window;
    int h_kv;           // key/value heads, divides h
    int gate_channels;  // 0: gates [N, H, 3]; 1: gates [N, 3, H, d]
    int own_block;      // window branch = the query's own block; `window` is then 128 (every slot of the block
                        // within reach) and the kernels treat the block as its own segment
    int kv_packed;      // the forward workspace already holds the tile images of k and v (lsrm_nsa_compress_pack)
    const int32_t *goff;   // device, nullable [ng + 1]: spatial blocks as runs of 64-slot blocks
    int ng;                // number of spatial blocks (0 without goff)
    int nbc;               // compressed pairs: ng with groups, else nb
    int group_window;      // window branch = the query's spatial block (groups with window_mode 1): the kernels take the
                           // window segment of a block from the blk_seg table and `window` is 2^30
    const int32_t *count;  // device, nullable [nb]: active tokens per block
    int nb_obj, tiles_per_view, n_tiles, nb;
    int64_t n;
    float scale;
};

// Validates params; fills `s`.  Returns LSRM_OK or an error code.
lsrm_status make_shape(const lsrm_nsa_params *p, Shape *s);

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Copies 1 KB global -> LDS: lane i's 16 bytes from src + lane_off (lane_off = 16 i) to dst + 16 i.  src and dst are
// wave-uniform.  Inline assembly on purpose: the compiler counts the builtin both as a vector-memory and as an LDS
// operation, so that while a copy is in flight every wait for an LDS read becomes lgkmcnt(0) -- a read that an MFMA
// needs then also waits for the reads requested behind it.  Copies it does not see leave its LDS waits counted
// (lgkmcnt(3) in the row queue of the dQ kernel); who waits for the copies themselves is settled by hand (vmcnt before a
// barrier), and a copy in flight that the compiler does not count can only make its own vmcnt waits longer.  Measured:
//   attention step  0.6 % at d = 32 with 196 K tokens, 0.5 % at d = 64 with 180 K, 0.2 % at d = 128 with 428 K;
//   training step   32 heads of 32 channels on 2, 196 K tokens 49.4 -> 48.1 ms; 16 heads of 64, 57 K tokens 3.79 ->
//                   3.73 ms; 16 heads of 128, 428 K tokens 164.7 -> 163.4 ms.
// The LDS address goes through m0, as an input in that register: the compiler writes it and knows what it holds.  The
// s_nop is the wait state between a scalar write of m0 and the copy that reads it, which the compiler does not add
// inside assembly.  Nor does it add the five between a vector instruction that writes a scalar register and a memory
// instruction that reads it: src has to come from scalar arithmetic, never straight from a readlane (true of every call).
__device__ __forceinline__ void copy_kb_to_lds(const char *src, uint32_t lane_off, const char *dst) {
    const uint32_t m = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)dst);
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(src), "{m0}"(m) : "memory");
}
// the same with 4 bytes per lane (256 bytes in all, lane_off = 4 i)
__device__ __forceinline__ void copy_256_to_lds(const void *src, uint32_t lane_off, const char *dst) {
    const uint32_t m = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)dst);
    asm volatile("s_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(lane_off), "s"(src), "{m0}"(m) : "memory");
}

#define LSRM_HIP_CHECK(expr)                         \
    do {                                             \
        hipError_t e_ = (expr);                      \
        if (e_ != hipSuccess) return LSRM_ERR_HIP;   \
    } while (0)

// launchers (each validates nothing: callers in api.hip have done so)
lsrm_status launch_route(const Shape &s, const float *d_pos, const lsrm_camera *d_cams, int32_t *d_idx,
                         float *d_dist2, void *d_ws, hipStream_t st);
size_t route_ws_bytes(const Shape &s);
// Same kernels, the projections going through the library's fixed per-GPU scratch; calls nothing that allocates.
lsrm_status launch_route_static(const Shape &s, const float *d_pos, const lsrm_camera *d_cams, int32_t *d_idx,
                                float *d_dist2, hipStream_t st);

lsrm_status launch_route_3d(const Shape &s, const lsrm_route3d_params &r, const float *d_pos, const float *d_pos_img,
                            const lsrm_camera *d_cams, int32_t *d_idx, float *d_dist2, void *d_ws, hipStream_t st);
size_t route3d_ws_bytes(const Shape &s);

// Tables derived from the group offsets, for the attention kernels (tab: 3 nb + ng int32 of workspace):
//   blk_grp [nb]     spatial block of every 64-slot block
//   blk_seg [nb][2]  first token and end token of that spatial block
//   grp_tok [ng]     active tokens of every spatial block
struct GroupTables {
    const int32_t *blk_grp, *blk_seg, *grp_tok;
};
inline size_t group_tables_bytes(const Shape &s) { return s.ng > 0 ? align_up(((size_t)3 * s.nb + s.ng) * 4, 256) : 0; }
inline GroupTables group_tables_in(const Shape &s, const int32_t *tab) {
    return s.ng > 0 ? GroupTables{tab, tab + s.nb, tab + 3 * (size_t)s.nb} : GroupTables{nullptr, nullptr, nullptr};
}
// Entry i of the nb + ng that the tables have, by one thread; a launch that prepares something else makes them beside it (a launch of their
// own took 5 us, in the forward and in the backward of each step).  A block's group is the last one that starts at or before it; blocks that
// no group covers (offsets that do not reach N / 64) get zero entries (an empty window).  Nothing outside the tables is
// written, whatever the offsets hold.
__device__ __forceinline__ void group_table_entry(int i, int ng, int nb, const int32_t *__restrict__ goff, const int32_t *__restrict__ count,
                                                  int32_t *__restrict__ tab) {
    if (i < nb) {
        int lo = 0, hi = ng;  // goff[lo] <= i, if any is
        while (hi - lo > 1) {
            const int mid = (lo + hi) / 2;
            if (goff[mid] <= i) lo = mid; else hi = mid;
        }
        const int b0 = max(goff[lo], 0), b1 = min(goff[lo + 1], nb);
        const bool covered = b0 <= i && i < b1;
        int32_t *blk_seg = tab + nb;
        tab[i] = covered ? lo : 0;
        blk_seg[2 * i] = covered ? b0 * kBlock : 0;
        blk_seg[2 * i + 1] = covered ? b1 * kBlock : 0;
    } else if (i < nb + ng) {
        const int g = i - nb;
        const int b0 = min(max(goff[g], 0), nb), b1 = min(goff[g + 1], nb);
        int tokens = 0;
        for (int b = b0; b < b1; ++b) tokens += count != nullptr ? count[b] : kBlock;
        tab[3 * (size_t)nb + g] = tokens > 0 ? tokens : 1;
    }
}
// What a kernel needs to make them: n entries, none where it is 0.
struct GroupTableArgs {
    int n, ng, nb;
    const int32_t *goff, *count;
    int32_t *tab;
};
inline GroupTableArgs group_table_args(const Shape &s, int32_t *tab) {
    return {s.ng > 0 ? s.nb + s.ng : 0, s.ng, s.nb, s.goff, s.count, tab};
}

lsrm_status launch_compress(const Shape &s, const uint16_t *d_k, const uint16_t *d_v, uint16_t *d_kc,
                            uint16_t *d_vc, hipStream_t st);  // honours s.count

lsrm_status launch_forward(const Shape &s, const int32_t *seg_host, int n_seg, const uint16_t *d_q,
                           const uint16_t *d_k, const uint16_t *d_v, const uint16_t *d_kc,
                           const uint16_t *d_vc, const int32_t *d_idx, const float *d_gates, uint16_t *d_out,
                           float *d_lse, uint16_t *d_out_branch, void *d_ws, hipStream_t st, hipEvent_t ev_start,
                           hipEvent_t ev_stop);
size_t forward_ws_bytes(const Shape &s);
// Pooling and packing in one pass over k and v: kc, vc as launch_compress writes them (same mean, fp32 partial sums
// added in a different order) and the tile images of (k, v) in the forward workspace d_ws.
lsrm_status launch_compress_pack(const Shape &s, const uint16_t *d_k, const uint16_t *d_v, uint16_t *d_kc,
                                 uint16_t *d_vc, void *d_ws, hipStream_t st);
lsrm_status launch_backward(const Shape &s, const int32_t *seg_host, int n_seg, const uint16_t *d_q,
                            const uint16_t *d_k, const uint16_t *d_v, const uint16_t *d_kc, const uint16_t *d_vc,
                            const int32_t *d_idx, const float *d_gates, const float *d_lse,
                            const uint16_t *d_out_branch, const uint16_t *d_dout, uint16_t *d_dq, uint16_t *d_dk,
                            uint16_t *d_dv, void *d_ws, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop);
size_t backward_ws_bytes(const Shape &s);

}  // namespace lsrm
