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

// The same sums where pool_blocks would be a few workgroups: a workgroup per block and sixteen chunks, sixteen threads to a
// chunk with four rows each in flight, which go into LDS as they are; then a thread per channel adds its 64 values in token order,
// so that a block's pair has the same bits however many blocks a call has.  (Bound by latency; sixteen partial sums a channel,
// a shorter chain, took 2.6 us where this takes 2.9, 43 blocks, 3 heads of 128, and rounded differently.)  Workgroups of one block
// beside each other: whole rows are read at about the same time.  pool_blocks / this, us, blocks x heads: d = 128, 43 x 3 6.9 / 2.9; d = 64, 128 x 16
// 7.3 / 4.8, 160 x 16 9.8 / 8.5, 512 x 8 12.6 / 11.8, 128 x 32 12.4 / 11.8, 64 x 64 15.8 / 11.7; the line is where little is left to gain.
constexpr int64_t kPoolFew = 1 << 15;  // chunks in all
constexpr int kPoolFewBlocks = 2048;
__global__ __launch_bounds__(256) void pool_blocks_few(int row_chunks, const uint4 *__restrict__ k, const uint4 *__restrict__ v,
                                                       uint4 *__restrict__ kc, uint4 *__restrict__ vc,
                                                       const int32_t *__restrict__ count) {
    __shared__ uint4 rows[kBlock][16];
    const size_t b = blockIdx.y;
    const int cl = threadIdx.x % 16, rl = threadIdx.x / 16, c = blockIdx.x * 16 + cl;
    const uint4 *src = (blockIdx.z == 0 ? k : v) + b * kBlock * (size_t)row_chunks + min(c, row_chunks - 1);
    const int n_act = count != nullptr ? count[b] : kBlock;
    uint4 r[kBlock / 16];
#pragma unroll
    for (int i = 0; i < kBlock / 16; ++i)
        r[i] = rl + 16 * i < n_act ? src[(size_t)(rl + 16 * i) * row_chunks] : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < kBlock / 16; ++i) rows[rl + 16 * i][cl] = r[i];
    __syncthreads();
    const int ch = threadIdx.x, chunk = blockIdx.x * 16 + ch / 8;
    if (ch >= 128 || chunk >= row_chunks) return;
    const uint16_t *column = reinterpret_cast<const uint16_t *>(rows) + ch;
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < kBlock; ++t) sum += __uint_as_float((uint32_t)column[t * 128] << 16);
    uint16_t *dst = reinterpret_cast<uint16_t *>((blockIdx.z == 0 ? kc : vc) + b * (size_t)row_chunks + chunk);
    dst[ch % 8] = (uint16_t)f32_to_bf16_rne(sum / (float)n_act);
}

// Spatial blocks of several 64-slot blocks (Sec. 3.2: volume blocks of up to 512 active tokens): one pair per
// group, the mean over the active tokens of all its blocks.  A workgroup takes SIDE groups side by side and LANES chunks of 8
// channels of their rows; the threads of a group read 256 / (LANES SIDE) of its rows at a time, DEPTH deep.  However many
// that are, a channel's sum is that of sixteen partial sums in order, the i-th over the slots i, i + 16, ... of
// the group: a thread adds its rows in registers, then they go through LDS and a thread per channel adds them up.  The
// same bits in every layout, chosen by the shape alone (see launch_compress):
//   <16, 1, 8>   16 rows of 256 bytes at a time: 512 tokens in four round trips to memory.  What a few long groups need, where
//                the latency of the chain (offsets, rows, sums) is all there is.
//   <4, 4, 8>, <8, 2, 8>   rows of 4 or 8 chunks (a head or two of 32 channels, one of 64), which would leave 12 or 8 of
//                16 lanes idle.  8 chunks only where groups are short (under two blocks on average): with two
//                blocks a group, one group fills the loads in flight (16 M tokens of a head of 64: 680 us alone, 720 side by side).
//   <64, 1, 16>  1 KB of a row per wavefront, a whole 64-slot block in flight, the sets of chunks numbered fastest: neighbouring
//                workgroups read neighbouring pieces of the same rows.  What many groups of wide rows need, which the
//                memory bounds (428 K tokens, 16 heads of 128, 3.5 GB: 597 us = 5.9 TB/s, 676 with <16, 1, 8>).  Not
//                for few: 256 groups there 25.9 instead of 21.5 us, 500 of them 43.8 instead of 40.5.
// One thread per chunk that walked the whole group, the form before the first of these, took 158 us for 197 K tokens of
// 2 heads of 32 in groups of eight blocks (9), 26.8 us for 1 M tokens of one head of 32 in single blocks (21.5; 52 with
// <16, 1, 8>) and 628 us for the 3.5 GB above.
// A workgroup loops where there are more units than kPoolMaxGrid: a launch holds fewer than 2^32 threads in a direction, and
// there can be 2^24 groups.  (Not at fewer: 131 K groups of two blocks, one head of 64, 700 us in two turns, 645 to 680 in one.)
constexpr int kPoolSums = 16, kPoolMaxGrid = 1 << 20;
constexpr int64_t kPoolWideFrom = 1 << 17;  // groups times chunks of a row
template <int LANES, int SIDE, int DEPTH>
__global__ __launch_bounds__(256) void pool_groups(int ng, int row_chunks, const uint4 *__restrict__ k,
                                                   const uint4 *__restrict__ v, uint4 *__restrict__ kc,
                                                   uint4 *__restrict__ vc, const int32_t *__restrict__ count,
                                                   const int32_t *__restrict__ goff) {
    constexpr int COLS = LANES * SIDE, ROWS = 256 / COLS, CHANNELS = COLS * 8, PER = (CHANNELS + 255) / 256;
    constexpr int SUMS = kPoolSums / ROWS;  // of the partial sums, how many a thread holds: rows rl + ROWS m, m mod SUMS
    constexpr bool SETS_FIRST = LANES == 64;
    static_assert(SUMS * ROWS == kPoolSums && DEPTH % SUMS == 0, "");
    __shared__ __attribute__((aligned(16))) float part[ROWS][CHANNELS + 4];  // (a pitch of whole 16-byte pieces)
    __shared__ int part_tokens[ROWS][SIDE];
    const int cl = threadIdx.x % COLS, rl = threadIdx.x / COLS;
    const int n_sets = SETS_FIRST ? row_chunks / LANES : 1, set = SETS_FIRST ? blockIdx.x % n_sets : blockIdx.y;
    const int c0 = set * LANES, c = c0 + cl % LANES;
    const bool in_row = c < row_chunks;
    const uint4 *src = (blockIdx.z == 0 ? k : v) + c;
    const int stride = (int)(gridDim.x / n_sets) * SIDE;
    for (int g0 = blockIdx.x / n_sets * SIDE; g0 < ng; g0 += stride) {
        const int grp = SIDE == 1 ? g0 : min(g0 + cl / LANES, ng - 1);   // (past the end: the last group again, not stored)
        const int s0 = goff[grp] * kBlock, s1 = goff[grp + 1] * kBlock;  // token slots of the group
        float acc[SUMS][8];
#pragma unroll
        for (int m = 0; m < SUMS; ++m)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[m][j] = 0.f;
        int tokens = 0;
        for (int s = s0 + rl; s < s1; s += ROWS * DEPTH) {
            bool on[DEPTH];
            uint4 r[DEPTH];
#pragma unroll
            for (int i = 0; i < DEPTH; ++i) {
                const int si = s + i * ROWS;
                on[i] = in_row && si < s1 && (count == nullptr || (si & (kBlock - 1)) < count[si / kBlock]);
            }
#pragma unroll
            for (int i = 0; i < DEPTH; ++i)  // (inactive slots are never read: the caller may have left anything there)
                r[i] = on[i] ? src[(size_t)(s + i * ROWS) * row_chunks] : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < DEPTH; ++i) {
                float(&x)[8] = acc[i % SUMS];
                x[0] += bf16_lo(r[i].x); x[1] += bf16_hi(r[i].x);
                x[2] += bf16_lo(r[i].y); x[3] += bf16_hi(r[i].y);
                x[4] += bf16_lo(r[i].z); x[5] += bf16_hi(r[i].z);
                x[6] += bf16_lo(r[i].w); x[7] += bf16_hi(r[i].w);
                tokens += on[i] ? 1 : 0;
            }
        }
        if (cl % LANES == 0) part_tokens[rl][cl / LANES] = tokens;
        float sum[PER];
#pragma unroll
        for (int m = 0; m < SUMS; ++m) {
            if (m > 0) __syncthreads();  // the sums before these have been read
            float4 *row = reinterpret_cast<float4 *>(&part[rl][cl * 8]);
            row[0] = make_float4(acc[m][0], acc[m][1], acc[m][2], acc[m][3]);
            row[1] = make_float4(acc[m][4], acc[m][5], acc[m][6], acc[m][7]);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int ch = u * 256 + threadIdx.x;
                if (m == 0) sum[u] = 0.f;
                if (CHANNELS % 256 != 0 && ch >= CHANNELS) continue;
#pragma unroll
                for (int i = 0; i < ROWS; ++i) sum[u] += part[i][ch];
            }
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int ch = u * 256 + threadIdx.x, side = ch / (LANES * 8), channel = c0 * 8 + ch % (LANES * 8);
            if (ch >= CHANNELS || g0 + side >= ng || channel >= row_chunks * 8) continue;
            int n_tok = 0;
#pragma unroll
            for (int i = 0; i < ROWS; ++i) n_tok += part_tokens[i][side];
            reinterpret_cast<uint16_t *>(blockIdx.z == 0 ? kc : vc)[(size_t)(g0 + side) * row_chunks * 8 + channel] =
                (uint16_t)f32_to_bf16_rne(sum[u] / (float)(n_tok > 0 ? n_tok : 1));
        }
        if (g0 + stride < ng) __syncthreads();  // the partial sums have been read
    }
}

}  // namespace

lsrm_status launch_compress(const Shape &s, const uint16_t *d_k, const uint16_t *d_v, uint16_t *d_kc,
                            uint16_t *d_vc, hipStream_t st) {
    if (s.nb == 0) return LSRM_OK;
    int row_chunks = s.h_kv * s.d / 8;
    if (s.ng > 0) {
        const bool wide = row_chunks % 64 == 0 && (int64_t)s.ng * row_chunks >= kPoolWideFrom;
        const bool short_groups = s.nb < 2 * (int64_t)s.ng;
        const int lanes = wide ? 64 : row_chunks <= 4 ? 4 : row_chunks <= 8 && short_groups ? 8 : 16;
        const int side = wide ? 1 : 16 / lanes, n_sets = (row_chunks + lanes - 1) / lanes;
        const int units = (s.ng + side - 1) / side;
        const int most = !wide ? kPoolMaxGrid : n_sets < kPoolMaxGrid ? kPoolMaxGrid / n_sets : 1;
        const unsigned grid_x = units < most ? units : most;
        const auto kernel = wide         ? pool_groups<64, 1, 16>
                            : lanes == 4 ? pool_groups<4, 4, 8>
                            : lanes == 8 ? pool_groups<8, 2, 8>
                                         : pool_groups<16, 1, 8>;
        hipLaunchKernelGGL(kernel, wide ? dim3(grid_x * n_sets, 1, 2) : dim3(grid_x, n_sets, 2), dim3(256), 0, st, s.ng,
                           row_chunks, reinterpret_cast<const uint4 *>(d_k), reinterpret_cast<const uint4 *>(d_v),
                           reinterpret_cast<uint4 *>(d_kc), reinterpret_cast<uint4 *>(d_vc), s.count, s.goff);
        LSRM_HIP_CHECK(hipGetLastError());
        return LSRM_OK;
    }
    if (s.nb <= kPoolFewBlocks && (int64_t)s.nb * row_chunks <= kPoolFew) {
        hipLaunchKernelGGL(pool_blocks_few, dim3((row_chunks + 15) / 16, s.nb, 2), dim3(256), 0, st, row_chunks,
                           reinterpret_cast<const uint4 *>(d_k), reinterpret_cast<const uint4 *>(d_v),
                           reinterpret_cast<uint4 *>(d_kc), reinterpret_cast<uint4 *>(d_vc), s.count);
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
