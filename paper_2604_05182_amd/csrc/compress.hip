// Block compression (Sec. 3.2 "Block Partitioning and Compression"; App. A "Compressed"):
// one key/value pair per 64-token block, the in-block average.
//
// HBM-streaming kernel: every element of K and V is read exactly once (4 N h d bytes)
// and 1/64 of that is written.  One thread owns 8 consecutive channels (one 16-byte
// load per token row), consecutive threads own consecutive channels, so each row of a
// block is read with fully coalesced 16-byte accesses; the 64 rows are independent
// loads kept in flight by unrolling.  fp32 accumulation in token order, one rounding
// to bf16 at the end.
#include "lsrm_internal.h"

namespace lsrm {

namespace {

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

__device__ __forceinline__ uint32_t f32_to_bf16_rne(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

// grid: (ceil(NB * row_chunks / 256), 2)   y = 0 -> K, y = 1 -> V
// count (nullable): block b averages its first count[b] rows only (1..64).
__global__ __launch_bounds__(256) void pool_blocks(int nb, int row_chunks /* h*d/8 */, const uint4 *__restrict__ k,
                                                   const uint4 *__restrict__ v, uint4 *__restrict__ kc,
                                                   uint4 *__restrict__ vc, const int32_t *__restrict__ count) {
    const size_t g = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t b = g / row_chunks;
    const int c = (int)(g % row_chunks);
    if (b >= (size_t)nb) return;
    const uint4 *src = (blockIdx.y == 0 ? k : v) + b * kBlock * (size_t)row_chunks + c;
    uint4 *dst = (blockIdx.y == 0 ? kc : vc) + b * (size_t)row_chunks + c;
    const int n_act = count != nullptr ? count[b] : kBlock;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int t0 = 0; t0 < kBlock; t0 += 16) {
        uint4 r[16];
#pragma unroll
        for (int t = 0; t < 16; ++t)
            r[t] = t0 + t < n_act ? src[(size_t)(t0 + t) * row_chunks] : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            acc[0] += bf16_lo(r[t].x); acc[1] += bf16_hi(r[t].x);
            acc[2] += bf16_lo(r[t].y); acc[3] += bf16_hi(r[t].y);
            acc[4] += bf16_lo(r[t].z); acc[5] += bf16_hi(r[t].z);
            acc[6] += bf16_lo(r[t].w); acc[7] += bf16_hi(r[t].w);
        }
    }
    const float den = (float)n_act;  // 64: the division is exact, as a multiplication by 1/64 would be
    uint4 o;
    o.x = f32_to_bf16_rne(acc[0] / den) | (f32_to_bf16_rne(acc[1] / den) << 16);
    o.y = f32_to_bf16_rne(acc[2] / den) | (f32_to_bf16_rne(acc[3] / den) << 16);
    o.z = f32_to_bf16_rne(acc[4] / den) | (f32_to_bf16_rne(acc[5] / den) << 16);
    o.w = f32_to_bf16_rne(acc[6] / den) | (f32_to_bf16_rne(acc[7] / den) << 16);
    *dst = o;
}

// Spatial blocks of several 64-slot blocks (Sec. 3.2: volume blocks of up to 512 active tokens): one pair per
// group, the mean over the active tokens of all its blocks.  One workgroup per (group, 16 chunks of 8 channels): 16
// threads side by side read 256 contiguous bytes of a row, 16 such rows are read at a time, eight deep, so that a
// block of 512 tokens is four round trips to memory; a thread adds its rows in order, the 16 partial sums of a channel are
// added in order through LDS.  (One thread per chunk walking the whole group, one dependent load after another, took
// 170 us for 21 K token slots in groups of up to eight blocks, a sixth of a training step; this takes 11 us.)
// grid: (min(ng, kPoolMaxGrid), ceil(row_chunks / 16), 2); a workgroup takes every kPoolMaxGrid-th group (a launch holds
// fewer than 2^32 threads in a direction: one workgroup each for the 2^24 groups of 2^30 tokens are too many).
constexpr int kPoolLanes = 16, kPoolRows = 16, kPoolDepth = 8, kPoolMaxGrid = 1 << 16;
__global__ __launch_bounds__(256) void pool_groups(int ng, int row_chunks, const uint4 *__restrict__ k,
                                                   const uint4 *__restrict__ v, uint4 *__restrict__ kc,
                                                   uint4 *__restrict__ vc, const int32_t *__restrict__ count,
                                                   const int32_t *__restrict__ goff) {
    __shared__ float part[kPoolRows][kPoolLanes * 8 + 1];
    __shared__ int part_tokens[kPoolRows];
    const int cl = threadIdx.x % kPoolLanes, rl = threadIdx.x / kPoolLanes;
    const int c = blockIdx.y * kPoolLanes + cl;
    const bool in_row = c < row_chunks;
    const uint4 *src = (blockIdx.z == 0 ? k : v) + (in_row ? c : 0);
    for (int grp = blockIdx.x; grp < ng; grp += gridDim.x) {
        const int s0 = goff[grp] * kBlock, s1 = goff[grp + 1] * kBlock;  // token slots of the group
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        int tokens = 0;
        for (int s = s0 + rl; s < s1; s += kPoolRows * kPoolDepth) {
            bool on[kPoolDepth];
            uint4 r[kPoolDepth];
#pragma unroll
            for (int i = 0; i < kPoolDepth; ++i) {
                const int si = s + i * kPoolRows;
                on[i] = si < s1 && (count == nullptr || (si & (kBlock - 1)) < count[si / kBlock]);
            }
#pragma unroll
            for (int i = 0; i < kPoolDepth; ++i)  // (inactive slots are never read: the caller may have left anything there)
                r[i] = on[i] ? src[(size_t)(s + i * kPoolRows) * row_chunks] : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < kPoolDepth; ++i) {
                acc[0] += bf16_lo(r[i].x); acc[1] += bf16_hi(r[i].x);
                acc[2] += bf16_lo(r[i].y); acc[3] += bf16_hi(r[i].y);
                acc[4] += bf16_lo(r[i].z); acc[5] += bf16_hi(r[i].z);
                acc[6] += bf16_lo(r[i].w); acc[7] += bf16_hi(r[i].w);
                tokens += on[i] ? 1 : 0;
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) part[rl][cl * 8 + j] = acc[j];
        if (cl == 0) part_tokens[rl] = tokens;
        __syncthreads();
        if (rl == 0 && in_row) {
            int n_tok = 0;
            for (int i = 0; i < kPoolRows; ++i) n_tok += part_tokens[i];
            const float den = (float)(n_tok > 0 ? n_tok : 1);
            uint32_t bits[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                float sum = 0.f;
                for (int i = 0; i < kPoolRows; ++i) sum += part[i][cl * 8 + j];
                bits[j] = f32_to_bf16_rne(sum / den);
            }
            uint4 *dst = (blockIdx.z == 0 ? kc : vc) + (size_t)grp * row_chunks + c;
            *dst = make_uint4(bits[0] | bits[1] << 16, bits[2] | bits[3] << 16, bits[4] | bits[5] << 16, bits[6] | bits[7] << 16);
        }
        __syncthreads();  // the partial sums have been read
    }
}

// The tables the attention kernels look blocks up in (see GroupTables): one thread per block, then one per group.
// A block's group is the last one that starts at or before it; blocks that no group covers (offsets that do not
// reach N / 64) get zero entries (an empty window).  Written by one kernel and no memset, which callers that
// capture the stream cannot replay; nothing outside the tables is written, whatever the offsets hold.
__global__ __launch_bounds__(256) void group_tables(int ng, int nb, const int32_t *__restrict__ goff,
                                                    const int32_t *__restrict__ count, int32_t *__restrict__ blk_grp,
                                                    int32_t *__restrict__ blk_seg, int32_t *__restrict__ grp_tok) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nb) {
        int lo = 0, hi = ng;  // goff[lo] <= i, if any is
        while (hi - lo > 1) {
            const int mid = (lo + hi) / 2;
            if (goff[mid] <= i) lo = mid; else hi = mid;
        }
        const int b0 = max(goff[lo], 0), b1 = min(goff[lo + 1], nb);
        const bool covered = b0 <= i && i < b1;
        blk_grp[i] = covered ? lo : 0;
        blk_seg[2 * i] = covered ? b0 * kBlock : 0;
        blk_seg[2 * i + 1] = covered ? b1 * kBlock : 0;
    } else if (i < nb + ng) {
        const int g = i - nb;
        const int b0 = min(max(goff[g], 0), nb), b1 = min(goff[g + 1], nb);
        int tokens = 0;
        for (int b = b0; b < b1; ++b) tokens += count != nullptr ? count[b] : kBlock;
        grp_tok[g] = tokens > 0 ? tokens : 1;
    }
}

}  // namespace

lsrm_status launch_group_tables(const Shape &s, int32_t *tab, GroupTables *out, hipStream_t st) {
    out->blk_grp = out->blk_seg = out->grp_tok = nullptr;
    if (s.ng <= 0) return LSRM_OK;
    int32_t *blk_grp = tab, *blk_seg = tab + s.nb, *grp_tok = tab + 3 * (size_t)s.nb;
    hipLaunchKernelGGL(group_tables, dim3((s.nb + s.ng + 255) / 256), dim3(256), 0, st, s.ng, s.nb, s.goff, s.count, blk_grp,
                       blk_seg, grp_tok);
    LSRM_HIP_CHECK(hipGetLastError());
    out->blk_grp = blk_grp;
    out->blk_seg = blk_seg;
    out->grp_tok = grp_tok;
    return LSRM_OK;
}

lsrm_status launch_compress(const Shape &s, const uint16_t *d_k, const uint16_t *d_v, uint16_t *d_kc,
                            uint16_t *d_vc, hipStream_t st) {
    if (s.nb == 0) return LSRM_OK;
    int row_chunks = s.h_kv * s.d / 8;
    if (s.ng > 0) {
        const dim3 grid_g((unsigned)(s.ng < kPoolMaxGrid ? s.ng : kPoolMaxGrid),
                          (unsigned)((row_chunks + kPoolLanes - 1) / kPoolLanes), 2);
        hipLaunchKernelGGL(pool_groups, grid_g, dim3(256), 0, st, s.ng, row_chunks, reinterpret_cast<const uint4 *>(d_k),
                           reinterpret_cast<const uint4 *>(d_v), reinterpret_cast<uint4 *>(d_kc),
                           reinterpret_cast<uint4 *>(d_vc), s.count, s.goff);
        LSRM_HIP_CHECK(hipGetLastError());
        return LSRM_OK;
    }
    dim3 grid((unsigned)(((size_t)s.nb * row_chunks + 255) / 256), 2);
    hipLaunchKernelGGL(pool_blocks, grid, dim3(256), 0, st, s.nb, row_chunks, reinterpret_cast<const uint4 *>(d_k),
                       reinterpret_cast<const uint4 *>(d_v), reinterpret_cast<uint4 *>(d_kc),
                       reinterpret_cast<uint4 *>(d_vc), s.count);
    LSRM_HIP_CHECK(hipGetLastError());
    return LSRM_OK;
}

}  // namespace lsrm
