// NSA backward on gfx950 (App. A, Eq. nsa_1 differentiated): gradients with respect to q, k, v
// of the gated sum of the compressed, selected and window branches, routing table and gate
// weights held constant, average pooling differentiated.
//
// Per branch, with P the softmax probabilities (recomputed from the saved log-sum-exp), g the
// gate, D_i = dout_i . o_branch_i and dP = dout V^T:
//     dV = (g P)^T dout        dS = (g P) o (dP - D)        dQ = scale dS K        dK = scale dS^T Q
// A per-head gate is folded into the exponent: g P = exp2(S scale log2e - (lse log2e - log2 g)); with
// per-channel gates the incoming gradient of each branch is gate o dout instead (three images of it).
// With grouped-query heads a key/value head walks the query tiles of every query head that reads it.
//
// No floating-point atomics: the work is split into passes that each own their output rows.
//   bwd_dq_kernel    one workgroup per (query block, head), or for two heads of one key/value head or two blocks of one head: walks
//                    the same key tiles as the forward (pooled, routed, window) and accumulates dQ^T in registers.
//   bwd_dkv_kernel   one workgroup per (key block, key/value head): walks the query tiles that attend it --
//                    MODE 1: pooled keys, every query tile of the sequence (split into ranges whose
//                    partial sums sum_parts adds in order); MODE 0: token keys, the query tiles
//                    of the window and of the reverse routing list (query blocks in ascending order),
//                    longest walks first -- accumulates dK^T and dV^T in registers, adds
//                    the pooled gradients / 64.  Long walks, and the heads of large groups, are dealt to several
//                    workgroups, whose sums sum_walks adds in order before finishing the rows.
// Small problems go through three launches instead (bwd_prepare, bwd_walks_small, sum_walks): their walks run beside each
// other, and all sums of token keys meet the pooled gradients in the last one.
// Every operand tile is a "tile image" (see forward.hip): MFMA A-operand fragments in row order
// (rows permuted so that an accumulator is directly the B operand of the next contraction); the
// fragments of the transposed tile are read out of the same bytes in LDS (see mfma_tr).  The
// transposed S^T = K Q^T form of the forward is
// used in the dQ pass (one query per lane: lse and D are per-lane scalars); the dK/dV pass uses
// S = Q K^T (one key per lane; lse and D of the 32 queries of the tile come from a small
// per-tile table copied to LDS with the tile).
// Steps are not software pipelined: the copy of tile t+1 (global -> LDS) overlaps the arithmetic of tile t, and
// nothing inside a loop may make the compiler wait for all memory operations (see tr_issue, run_segment).
#include "lsrm_internal.h"

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>

constexpr int kBwdNbuf = 2;         // tile buffers of the dQ kernel
// tile buffers of the dK/dV kernels (three, copies two steps ahead: slower, 51 -> 65 ms on the pooled keys at d = 128)
constexpr int kBwdDkvNbuf = 2;

namespace lsrm {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxSeg = 63;
constexpr float kLog2e = 1.4426950408889634f;

struct BwdArgs {
    const uint16_t *q, *k, *v, *kc, *vc, *dout, *out_branch;
    const int32_t *idx;
    const float *gates, *lse;
    const char *img_q, *img_k, *img_v, *img_kc, *img_vc;  // tile images
    const char *img_do[3];    // images of the gradient that reaches each branch: one shared image of dout with
                              // per-head gates (the gate is folded into the exponent), gate o dout per branch
                              // with per-channel gates (written by bwd_prep)
    float *aux;               // [3][N/32][H][64]: per query tile, 32 x (lse log2e - log2 g) then 32 x -D, rows permuted
    float *part_k, *part_v;   // [n_split][nbp][H][d] fp32 partial gradients of the pooled keys / values
    int32_t *rev_cnt, *rev_ptr, *rev_cur, *rev_idx;  // reverse routing lists
    uint16_t *dq, *dk, *dv;
    int32_t seg[kMaxSeg + 1];
    int64_t n;
    int nb, h, topk, window, n_seg;
    int nbc;        // compressed pairs (spatial blocks): nb unless blocks are grouped
    // spatial blocks of several 64-slot blocks (nullable): group of every block, its token range as the window
    // segment of the block (given only when the window is the spatial block), active tokens per group
    const int32_t *blk_grp, *blk_seg, *grp_tok;
    int own_block;  // window branch = the query's own block
    int h_kv, group;    // key/value heads; query heads per key/value head
    int gate_channels;  // gates are [N, 3, H, d]
    const int32_t *count;  // nullable [NB]: active tokens per block; the other slots are neither queries nor keys
    int nt;               // query / key tiles of 32 tokens
    int nbp, tiles_per_split, n_split;  // pooled keys, rounded up; the query ranges of their walks
    // Token keys: a key block's walk -- the query tiles of its window, then two per entry of its reverse list -- is dealt to
    // several workgroups where it is long.  The query heads of a group go to hsplit
    // workgroups, hpw heads each; and a walk of more than part_steps tiles is cut into parts of that many (cut_window = 0:
    // the window, of unknown length, goes to the first part and is not counted).  A (key block, part) is a task;
    // order / order_part [<= max_tasks] hold the tasks, longest first: the order the workgroups start in.  Where a block's
    // walk is dealt out, the workgroups leave fp32 sums [hsplit][max_slots][64][H_kv][d], those of block b's parts from slot
    // slot0[b] on, and a last pass adds them up in order: over all blocks if hsplit > 1, else over those in split_list.
    // (In the launches of small problems every walk leaves sums, and the last pass goes over all blocks.)
    int hsplit, hpw, part_steps, max_slots, cut_window;
    float *hpart_k, *hpart_v;
    int32_t *order, *order_part, *slot0, *split_list, *task_n;  // task_n: number of tasks, length of split_list
    int32_t *walk;  // [NB] counted tiles of every key block's walk
    float scale, sl2;
};

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    bf16x2 p;
    p[0] = (__bf16)a;
    p[1] = (__bf16)b;
    return *reinterpret_cast<uint32_t *>(&p);
}
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// row permutation of the tile images: bits 2 and 3 swapped
__device__ __forceinline__ int perm32(int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); }

union BFrag {
    bf16x8 v;
    uint32_t u[4];
};

// accumulator tile -> the two B operands (16-row slabs) of the next contraction
__device__ __forceinline__ void to_b_operand(const float (&x)[16], BFrag (&b)[2]) {
#pragma unroll
    for (int k = 0; k < 8; ++k) b[k / 4].u[k % 4] = pack_bf16(x[2 * k], x[2 * k + 1]);
}

// MFMAs whose accumulator stays in ordinary VGPRs, written as inline assembly.  A kernel compiled for one wavefront
// per SIMD (more than 256 registers) gets every MFMA builtin in the form that accumulates in AGPRs; results that the
// vector ALU must read (scores, dP) then travel through v_accvgpr_read/write, and the register allocator was seen to
// park them in the AGPRs of the long-lived dK/dV accumulators, saving and restoring those around every chain (about
// 100 register moves per step).  The hardware does not interlock "MFMA result read by a VALU instruction" and the
// compiler cannot pad what it does not see, so a chain ends with mfma_v_settle (24 wait states cover the 8 passes).
__device__ __forceinline__ void mfma_v_first(f32x16 &d, bf16x8 a, bf16x8 b) {
    asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_v(f32x16 &d, bf16x8 a, bf16x8 b) {
    asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_v_settle(f32x16 &d) { asm volatile("s_nop 15\n\ts_nop 7" : "+v"(d)); }

// copies n_kb KB, contiguous on both sides, global -> LDS; the WV wavefronts of the workgroup split it
template <int N_KB, int WV = 2>
__device__ __forceinline__ void copy_kb(const char *src, char *dst, int wave, uint32_t lane16) {
    static_assert(N_KB % WV == 0, "");
    src += wave * 1024;
    dst += wave * 1024;
#pragma unroll
    for (int i = 0; i < N_KB; i += WV)
        copy_kb_to_lds(src + i * 1024, lane16, dst + i * 1024);
}

// s_waitcnt vmcnt <= n (and lgkmcnt == 0), and a raw barrier.  Neither this barrier nor __syncthreads() waits
// for global -> LDS copies in flight: whoever issued them waits on vmcnt before the barrier that publishes them.
constexpr int vm_lgkm_imm(int n) { return (n & 0xF) | ((n >> 4) << 14) | 0x0070; }
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }

// A-operand fragment of the TRANSPOSE of a tile, read out of the tile's row-order fragments in LDS with
// the transposing LDS load of gfx950 (ds_read_b64_tr_b16): within each group of 16 lanes, lane j receives
// as element e the 16-bit element j % 4 of what lane 4 e + j / 4 of the group addressed.  So a lane of the
// group addresses the four channels 4 (s % 4) .. + 3 of tile row s / 4 (s its index in the group), and
// lane j ends up with one channel of four consecutive rows -- four of the eight K-values of a fragment
// whose rows are channels.  Fragment (ks2, dt): channel 32 dt + (lane & 31), tile rows 16 ks2 + 8 hh + 0..7.
// `tr_lane_offset` is the per-lane part of the address inside the row-order fragments; the fragment adds
// dt * 2048 + ks2 * 256 and the second half of the rows another 128 (rows are stored permuted).
// This halves what a step copies into LDS: the transposed halves of the tile images stay in memory.
// In the backward's tile images the 16-byte slot of (row position r, channel half h) inside a fragment is
// h * 32 + (r ^ 4 h): without the xor the two channel halves that a group of 16 lanes addresses in one
// transposing load lie 512 bytes apart, i.e. in the same banks (measured: half the LDS cycles of these
// kernels were bank conflicts); with it the group's 16 addresses cover 32 distinct banks.
__device__ __forceinline__ uint32_t tr_lane_offset(int lane) {
    const int s = lane & 15, grp = lane >> 4;
    const int c = s & 3, k_local = s >> 2, hh = grp >> 1;
    return (uint32_t)((grp & 1) * 1024 + (c >> 1) * 512 + (4 * (hh ^ (c >> 1)) + k_local) * 16 + (c & 1) * 8);
}
// per-lane offset of this lane's 16 bytes inside a row-order fragment of such an image
__device__ __forceinline__ uint32_t row_lane_offset(int lane) {
    const int r = lane & 31, hh = lane >> 5;
    return (uint32_t)((hh * 32 + (r ^ (hh << 2))) * 16);
}
// The loads are written as inline assembly on purpose.  The compiler cannot tell that a transposing load
// (the builtin) does not touch the buffer that the global -> LDS copies of the next step are filling, and puts
// an s_waitcnt vmcnt(0) before the first of them: every step then waits for the copies it has just issued,
// and nothing is prefetched (seen in the assembly and in timestamps).  Loads it does not see get no such wait;
// in exchange their results are waited for by hand: tr_take ties a counted lgkmcnt wait to the registers of a
// fragment (LDS operations complete in order, so "at most n outstanding" covers all but the last n issued).
typedef int i32x2 __attribute__((ext_vector_type(2)));
struct TrFrag {
    i32x2 lo, hi;
};
template <int OFF>
__device__ __forceinline__ void tr_issue(TrFrag &f, uint32_t addr) {
    asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"
                 : "=&v"(f.lo), "=&v"(f.hi)
                 : "v"(addr), "n"(OFF), "n"(OFF + 128)
                 : "memory");
}
template <int N>
__device__ __forceinline__ bf16x8 tr_take(TrFrag &f) {
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(f.lo), "+v"(f.hi) : "n"(N) : "memory");
    union {
        i32x2 h[2];
        bf16x8 v;
    } u;
    u.h[0] = f.lo;
    u.h[1] = f.hi;
    return u.v;
}

// acc[dt] += (fragment (ks2, dt) of the transposed tile) x b[ks2] for every dt and ks2: all 2 ND fragments are
// requested at once and each MFMA waits for its own.  rows: the tile's row-order fragments in LDS.
template <int ND, int... I>
__device__ __forceinline__ void mfma_tr_impl(f32x16 (&acc)[ND], uint32_t addr, const BFrag (&b)[2],
                                             std::integer_sequence<int, I...>) {
    TrFrag f[2 * ND];
    (tr_issue<(I % ND) * 2048 + (I / ND) * 256>(f[I], addr), ...);
    ((acc[I % ND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr_take<2 * (2 * ND - 1 - I)>(f[I]), b[I / ND].v,
                                                            acc[I % ND], 0, 0, 0)),
     ...);
}
template <int ND>
__device__ __forceinline__ void mfma_tr(f32x16 (&acc)[ND], const char *rows, uint32_t lane_off, const BFrag (&b)[2]) {
    // (the low 32 bits of a generic pointer into LDS are the LDS address)
    mfma_tr_impl<ND>(acc, (uint32_t)(uintptr_t)rows + lane_off, b, std::make_integer_sequence<int, 2 * ND>{});
}

// f(integral_constant<0>), ..., f(integral_constant<N - 1>), in order
template <typename F, int... K>
__device__ __forceinline__ void for_each_index_impl(F &f, std::integer_sequence<int, K...>) {
    (f(std::integral_constant<int, K>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void for_each_index(F &f) {
    for_each_index_impl(f, std::make_integer_sequence<int, N>{});
}

template <int D>
struct BGeo {
    static constexpr int NS = D / 16, ND = D / 32;
    static constexpr int ROW = 32 * D * 2;  // row-order fragments of a tile
    static constexpr int TB = D * 64;       // fragments of the transposed tile
    static constexpr int IMG = ROW;         // the backward's images hold the row-order fragments only
    static constexpr int OUT_ROW = 2 * D + 8;  // padded bf16 row of the output staging (bytes)
};

// rows of a [D x 32] accumulator pair set (transposed gradient tile) -> bf16 rows of `dst`
// (32 rows of this wavefront, row stride h*D elements), staged through LDS so that rows are
// written as whole 16-byte chunks.  x[dt][i]: channel 32 dt + (i/4)*8 + hh*4 + i%4, row lane%32.
template <int D>
__device__ __forceinline__ void store_rows_transposed(const float (&x)[D / 32][16], char *stage, uint16_t *dst,
                                                      int64_t row_stride, int lane) {
    using G = BGeo<D>;
    const int r = lane & 31, hh = lane >> 5;
#pragma unroll
    for (int dt = 0; dt < G::ND; ++dt)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            uint2 w2;
            w2.x = pack_bf16(x[dt][4 * gq + 0], x[dt][4 * gq + 1]);
            w2.y = pack_bf16(x[dt][4 * gq + 2], x[dt][4 * gq + 3]);
            *reinterpret_cast<uint2 *>(stage + r * G::OUT_ROW + (32 * dt + 8 * gq + 4 * hh) * 2) = w2;
        }
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wavefront's own staging writes
    constexpr int CH = D / 8, RPP = 64 / CH;
#pragma unroll
    for (int it = 0; it < 32 / RPP; ++it) {
        const int rr = it * RPP + lane / CH, ch = lane % CH;
        uint4 val = *reinterpret_cast<const uint4 *>(stage + rr * G::OUT_ROW + ch * 16);
        *reinterpret_cast<uint4 *>(dst + rr * row_stride + ch * 8) = val;
    }
}

// ---------------------------------------------------------------------------------------------
// per (token, head): the per-branch exponent offset and D = dout . o_branch, in tile-image row order, and the tile
// images of the gradient rows (dout, or gate o dout per branch with per-channel gates; padding slots as zeros).
// Threads: 8 channels each.  A workgroup takes one query tile and PREP_HB heads: thread = (head, row of the tile,
// 16-byte chunk of the row), chunks fastest, so a row's d channels are read by d / 8 neighbouring lanes (16-byte
// loads, contiguous per row) and the 32 table entries of a (tile, head) are written from one wavefront, side by side.
// The images of a tile's heads are contiguous: a workgroup writes HB of them, 4 or 8 KB, in image order out of LDS (chunk
// pitch 33 slots: neither the writes, chunks fastest, nor the reads, rows fastest, share banks).  Bound by memory:
// dout and three branch outputs read, one or three images written, with per-channel gates 12 bytes of gates per channel.
// Packing the images in passes of their own from dout (57 K tokens, 16 heads of 64: 40 us) or from three bf16
// tensors that this kernel wrote (196 K tokens, 32 heads of 32: 3 x 166 us) cost one more trip through memory each.
template <int D>
struct PrepGeo {
    static constexpr int CH = D / 8;                            // chunks = lanes per (row, head)
    static constexpr int HB = CH * 32 >= 256 ? 1 : 256 / (CH * 32);  // heads per workgroup
    static constexpr int THREADS = HB * 32 * CH;
};
template <int D>
using PrepStage = uint4[3][PrepGeo<D>::HB * PrepGeo<D>::CH * 33];
template <int D>
__device__ __forceinline__ void prep_rows(const BwdArgs &a, PrepStage<D> &stage, int64_t wg) {
    using P = PrepGeo<D>;
    constexpr int CH = P::CH, PITCH = 33;  // LDS slots of 16 bytes per chunk column
    const int c = threadIdx.x % CH, r = (threadIdx.x / CH) % 32, hb = threadIdx.x / (CH * 32);
    const int heads_x = (a.h + P::HB - 1) / P::HB;
    const int64_t tile = wg / heads_x;
    const int head0 = (int)(wg % heads_x) * P::HB;
    const bool active = head0 + hb < a.h;  // (whole groups of CH lanes)
    const int head = active ? head0 + hb : head0;
    const int64_t row = tile * 32 + r;
    // a padding slot is no query: zero probabilities (offset +inf), a zero D in every branch, a zero row in the images
    const bool padding = a.count != nullptr && (int)(row & 63) >= a.count[row >> 6];
    const uint4 raw = *reinterpret_cast<const uint4 *>(a.dout + (row * a.h + head) * D + 8 * c);
    float dov[8];
    {
        const uint32_t u[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            dov[2 * j] = bf16_lo(u[j]);
            dov[2 * j + 1] = bf16_hi(u[j]);
        }
    }
    const int pr = perm32(r);
    const int slot = (hb * CH + c) * PITCH + (pr ^ ((c & 1) << 2));
    if (!a.gate_channels) stage[0][slot] = padding ? make_uint4(0, 0, 0, 0) : raw;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const uint4 w = *reinterpret_cast<const uint4 *>(a.out_branch + (((int64_t)b * a.n + row) * a.h + head) * D + 8 * c);
        const uint32_t u[4] = {w.x, w.y, w.z, w.w};
        float dl = 0.f;
        if (a.gate_channels) {
            // the gradient reaching this branch is gate o dout, channel by channel: D uses it, and its
            // bf16 rounding is kept for the contractions
            const f32x4 *gch = reinterpret_cast<const f32x4 *>(a.gates + ((row * 3 + b) * a.h + head) * D + 8 * c);
            const f32x4 g_lo = gch[0], g_hi = gch[1];
            const float g[8] = {g_lo[0], g_lo[1], g_lo[2], g_lo[3], g_hi[0], g_hi[1], g_hi[2], g_hi[3]};
            uint32_t o4[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float g0 = g[2 * j] * dov[2 * j], g1 = g[2 * j + 1] * dov[2 * j + 1];
                dl += g0 * bf16_lo(u[j]) + g1 * bf16_hi(u[j]);
                o4[j] = pack_bf16(g0, g1);
            }
            stage[b][slot] = padding ? make_uint4(0, 0, 0, 0) : make_uint4(o4[0], o4[1], o4[2], o4[3]);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) dl += dov[2 * j] * bf16_lo(u[j]) + dov[2 * j + 1] * bf16_hi(u[j]);
        }
        // D of the row: the sum over its CH lanes, in a fixed order
#pragma unroll
        for (int m = 1; m < CH; m <<= 1) dl += __shfl_xor(dl, m);
        if (c != 0 || !active) continue;
        const float lse = a.lse[((int64_t)b * a.n + row) * a.h + head];
        // an empty key set (lse = -inf) or a zero gate gives zero probabilities: offset +inf
        float l2 = __builtin_inff();
        if (a.gate_channels) {
            if (lse > -__builtin_inff()) l2 = lse * kLog2e;
        } else {
            const float g = a.gates[(row * a.h + head) * 3 + b];
            if (g > 0.f && lse > -__builtin_inff()) l2 = lse * kLog2e - __log2f(g);
        }
        float *ax = a.aux + (((int64_t)b * a.nt + tile) * a.h + head) * 64;
        ax[pr] = padding ? __builtin_inff() : l2;
        ax[32 + pr] = padding ? 0.f : -dl;  // negated: the kernels start the dP accumulators from it
    }
    __syncthreads();
    // image of (tile, head0 + e / (32 CH)): slot e % (32 CH) = chunk column (e / 32) % CH, row slot e % 32
    const int e = threadIdx.x, e_head = e / (32 * CH);
    if (head0 + e_head >= a.h) return;
    const int64_t dst = (tile * a.h + head0) * (int64_t)BGeo<D>::IMG + (int64_t)e * 16;
    const int src = (e / 32) * PITCH + e % 32;
#pragma unroll
    for (int b = 0; b < 3; ++b)
        if (b == 0 || a.gate_channels) *reinterpret_cast<uint4 *>(const_cast<char *>(a.img_do[b]) + dst) = stage[b][src];
}
template <int D>
__global__ __launch_bounds__(PrepGeo<D>::THREADS) void bwd_prep(BwdArgs a, GroupTableArgs tables) {
    __shared__ PrepStage<D> stage;
    // (the counters of the reverse lists, which the next kernel increments, and the tables of spatial blocks: there are more threads than twice
    // the blocks)
    const int64_t gid = (int64_t)blockIdx.x * PrepGeo<D>::THREADS + threadIdx.x;
    if (gid < a.nb) a.rev_cnt[gid] = 0;
    if (gid < tables.n) group_table_entry((int)gid, tables.ng, tables.nb, tables.goff, tables.count, tables.tab);
    prep_rows<D>(a, stage, blockIdx.x);
}

// ---------------------------------------------------------------------------------------------
// Tile images of q, k, v, kc and vc in one launch (latency and launches are what a small problem pays for; a large one
// is bound by memory: read once, written once), one workgroup per (64-row block, tensor, head), heads fastest so
// that neighbouring workgroups read neighbouring pieces of the same rows.  Workgroups behind those count, per key
// block, the query blocks that list it (the reverse lists' lengths).
// Image: slot cc * 32 + rr of 16 bytes = chunk cc of tile row perm32(rr ^ 4 (cc & 1)).  Rows at or beyond the end, and
// padding slots, read as zeros.
// The workgroups are numbered over both directions of the grid: a launch holds fewer than 2^32 threads in a direction, which
// three workgroups per block and head (179 M tokens, 2 heads of 32) exceed.
constexpr int64_t kPackMaxGrid = 1 << 23;  // workgroups in the first direction
template <int D>
using PackStage = uint16_t[64][D + 16];  // (pitch: 16-byte aligned, chunks of a row spread over the banks)
template <int D, int THREADS>
__device__ __forceinline__ void pack_block(const BwdArgs &a, PackStage<D> &rows, int64_t n_token_wg, int64_t wg) {
    constexpr int CH = D / 8, IMG = BGeo<D>::IMG;
    const bool pooled = wg >= n_token_wg;
    const int y_n = pooled ? 2 * a.h_kv : a.h + 2 * a.h_kv;
    const int64_t at = pooled ? wg - n_token_wg : wg;
    const int64_t blk = at / y_n;
    int head = (int)(at % y_n), h = a.h_kv;
    const uint16_t *src;
    const char *img;
    if (!pooled && head < a.h) {
        src = a.q;
        img = a.img_q;
        h = a.h;
    } else {
        if (!pooled) head -= a.h;
        const bool second = head >= a.h_kv;
        if (second) head -= a.h_kv;
        src = pooled ? (second ? a.vc : a.kc) : (second ? a.v : a.k);
        img = pooled ? (second ? a.img_vc : a.img_kc) : (second ? a.img_v : a.img_k);
    }
    const int64_t n_rows = pooled ? a.nbc : a.n, n_tiles = pooled ? (a.nbc + 31) / 32 : a.nt;
    const int n_act = !pooled && a.count != nullptr ? a.count[blk] : 64;
    constexpr int NIT = 64 * CH / THREADS;
    uint4 in[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int e = threadIdx.x + THREADS * it, t = e / CH, cc = e % CH;
        const int64_t row = blk * 64 + t;
        in[it] = row < n_rows && t < n_act ? *reinterpret_cast<const uint4 *>(src + (row * h + head) * D + cc * 8)
                                           : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int e = threadIdx.x + THREADS * it;
        *reinterpret_cast<uint4 *>(&rows[e / CH][(e % CH) * 8]) = in[it];
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int e = threadIdx.x + THREADS * it, half = e / (32 * CH), q = e % (32 * CH), cc = q / 32, rr = q % 32;
        const int64_t tile = blk * 2 + half;
        if (tile < n_tiles)
            *reinterpret_cast<uint4 *>(const_cast<char *>(img) + (tile * h + head) * IMG + q * 16) =
                *reinterpret_cast<const uint4 *>(&rows[32 * half + perm32(rr ^ ((cc & 1) << 2))][cc * 8]);
    }
}

template <int D>
__global__ __launch_bounds__(256) void pack_rows(BwdArgs a, int64_t n_token_wg, int64_t n_wg) {
    __shared__ __attribute__((aligned(16))) PackStage<D> rows;
    const int64_t wg = (int64_t)blockIdx.y * kPackMaxGrid + blockIdx.x;
    if (wg >= n_wg) {
        const int64_t e = (wg - n_wg) * 256 + threadIdx.x;
        if (e < (int64_t)a.nb * a.topk) {
            const int v = a.idx[e];
            if (v >= 0 && v < a.nb) atomicAdd(&a.rev_cnt[v], 1);
        }
        return;
    }
    pack_block<D, 256>(a, rows, n_token_wg, wg);
}

// ---------------------------------------------------------------------------------------------
// reverse routing lists: for every key block the query blocks that list it, ascending
// The query tiles that see key block kb in the window branch: [first, first + n).
struct WindowTiles {
    int first, n;
};
__device__ __forceinline__ WindowTiles window_tiles(const BwdArgs &a, int kb) {
    const int k0 = kb * 64, half_w = a.window / 2;
    int seg_lo = 0, seg_hi = 0;
    if (a.blk_seg != nullptr) {  // the key's spatial block
        seg_lo = a.blk_seg[2 * kb];
        seg_hi = a.blk_seg[2 * kb + 1];
    } else {
        for (int s = 0; s < a.n_seg; ++s)
            if (k0 >= a.seg[s] && k0 < a.seg[s + 1]) {
                seg_lo = a.seg[s];
                seg_hi = a.seg[s + 1];
            }
    }
    if (a.own_block) {
        seg_lo = k0;
        seg_hi = k0 + 64;
    }
    // query i sees key j iff -W/2 <= j - i < W/2, i.e. j - W/2 < i <= j + W/2
    const int i_lo = max(seg_lo, k0 - half_w + 1), i_hi = min(seg_hi, k0 + 63 + half_w + 1);
    WindowTiles w;
    w.first = i_lo / 32;
    w.n = (half_w > 0 && i_hi > i_lo) ? (i_hi - 1) / 32 + 1 - w.first : 0;
    return w;
}
// Where the lists start, and the tasks of the token-key dK/dV workgroups (see BwdArgs) in order of falling length
// (within 1024 length classes; equal lengths in any order -- it only decides which workgroup starts when): the long
// walks start first instead of forming the tail of the kernel, and the round-robin of workgroups over the XCDs
// spreads them, where a contiguous range of blocks per XCD had left the popular blocks (say, all image blocks) to one or
// two XCDs.
__global__ __launch_bounds__(1024) void rev_scan_order(BwdArgs a) {
    constexpr int kHeld = 4096;  // lengths kept in LDS up to this many blocks: a round trip to memory is most of this kernel
    __shared__ int wave_total[3][16], bin[1024], n_split_blocks, held_cnt[kHeld], held_walk[kHeld];
    const int t = threadIdx.x;
    const bool held = a.nb <= kHeld;
    auto cnt = [&](int b) { return held ? held_cnt[b] : a.rev_cnt[b]; };
    auto walk = [&](int b) { return held ? held_walk[b] : a.walk[b]; };
    auto n_parts = [&](int steps) { return max(1, (steps + a.part_steps - 1) / a.part_steps); };
    auto n_slots = [&](int steps) { return a.hsplit > 1 || steps > a.part_steps ? n_parts(steps) : 0; };
    auto length_class = [](int steps) { return 1023 - min(steps >> 1, 1023); };
    bin[t] = 0;
    if (t == 0) n_split_blocks = 0;
    for (int b = t; b < a.nb; b += 1024) {  // (an even number of window tiles: a part boundary never splits a list entry)
        const int c = a.rev_cnt[b], w = 2 * c + (a.cut_window ? (window_tiles(a, b).n + 1) & ~1 : 0);
        a.walk[b] = w;
        if (held) {
            held_cnt[b] = c;
            held_walk[b] = w;
        }
    }
    __syncthreads();
    // starts of the lists and of the blocks' slots: exclusive prefix sums
    const int chunk = (a.nb + 1023) / 1024;
    const int lo = min(t * chunk, a.nb), hi = min(lo + chunk, a.nb);
    int s = 0, sl = 0;
    for (int i = lo; i < hi; ++i) {
        s += cnt(i);
        sl += n_slots(walk(i));
    }
    for (int b = t; b < a.nb; b += 1024) {
        const int steps = walk(b), np = n_parts(steps);
        if (np > 1) atomicAdd(&bin[length_class(a.part_steps)], np - 1);
        atomicAdd(&bin[length_class(steps - (np - 1) * a.part_steps)], 1);
    }
    __syncthreads();
    const int own = bin[t];
    // inclusive prefix sums over the threads: inside each wavefront, then over the wavefronts' totals
    int x[3] = {s, own, sl};
#pragma unroll
    for (int off = 1; off < 64; off <<= 1)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int y = __shfl_up(x[k], off);
            if ((t & 63) >= off) x[k] += y;
        }
    if ((t & 63) == 63)
        for (int k = 0; k < 3; ++k) wave_total[k][t >> 6] = x[k];
    __syncthreads();
    for (int w = 0; w < t >> 6; ++w)
        for (int k = 0; k < 3; ++k) x[k] += wave_total[k][w];
    const int part_t = x[0], bin_t = x[1], slots_t = x[2];
    int run = part_t - s, run_slot = slots_t - sl;
    for (int i = lo; i < hi; ++i) {
        a.rev_ptr[i] = run;
        a.rev_cur[i] = run;
        a.slot0[i] = run_slot;
        run += cnt(i);
        run_slot += n_slots(walk(i));
    }
    if (t == 1023) {
        a.rev_ptr[a.nb] = part_t;
        a.task_n[0] = bin_t;
    }
    bin[t] = bin_t - own;  // start of each class
    __syncthreads();
    for (int b = t; b < a.nb; b += 1024) {
        const int steps = walk(b), np = n_parts(steps);
        if (np > 1) {
            const int at = atomicAdd(&bin[length_class(a.part_steps)], np - 1);
            for (int p = 0; p < np - 1; ++p) {
                a.order[at + p] = b;
                a.order_part[at + p] = p;
            }
            a.split_list[atomicAdd(&n_split_blocks, 1)] = b;
        }
        const int at = atomicAdd(&bin[length_class(steps - (np - 1) * a.part_steps)], 1);
        a.order[at] = b;
        a.order_part[at] = np - 1;
    }
    __syncthreads();
    if (t == 0) a.task_n[1] = n_split_blocks;
}
__global__ void rev_fill(BwdArgs a) {
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= a.nb * a.topk) return;
    int v = a.idx[e];
    if (v >= 0 && v < a.nb) a.rev_idx[atomicAdd(&a.rev_cur[v], 1)] = e / a.topk;
}
// Puts every list in ascending order (the fill order is whatever the atomics gave; a fixed order makes the
// gradients reproducible, and ascending keeps consecutive query tiles together).  The entries of a list are
// block numbers, distinct unless a row of the table repeats a block: one wavefront per key block marks them in
// a bitmap of nb bits in LDS and reads the bitmap back in order.
__global__ __launch_bounds__(64) void rev_sort(BwdArgs a) {
    extern __shared__ uint32_t bits[];  // (nb + 31) / 32 words
    const int b = blockIdx.x, lane = threadIdx.x;
    const int words = (a.nb + 31) >> 5;
    int32_t *x = a.rev_idx + a.rev_ptr[b];
    const int len = a.rev_ptr[b + 1] - a.rev_ptr[b];
    if (len <= 1) return;
    for (int w = lane; w < words; w += 64) bits[w] = 0u;
    __syncthreads();
    for (int i = lane; i < len; i += 64) atomicOr(&bits[x[i] >> 5], 1u << (x[i] & 31));
    __syncthreads();
    // a table may list a block twice in one row (it is then attended twice): the bitmap would drop the repeat,
    // so such a list is sorted the slow way
    int marked = 0;
    for (int w = lane; w < words; w += 64) marked += __popc(bits[w]);
    for (int off = 32; off > 0; off >>= 1) marked += __shfl_xor(marked, off);
    if (marked != len) {
        if (lane == 0)
            for (int i = 1; i < len; ++i) {
                int v = x[i], j = i - 1;
                while (j >= 0 && x[j] > v) {
                    x[j + 1] = x[j];
                    --j;
                }
                x[j + 1] = v;
            }
        return;
    }
    int base = 0;
    for (int w0 = 0; w0 < words; w0 += 64) {
        const int w = w0 + lane;
        uint32_t m = w < words ? bits[w] : 0u;
        const int c = __popc(m);
        int pre = c;  // inclusive prefix sum over the lanes
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(pre, off);
            if (lane >= off) pre += t;
        }
        int at = base + pre - c;
        while (m != 0u) {
            x[at++] = (w << 5) + (__ffs(m) - 1);
            m &= m - 1u;
        }
        base += __shfl(pre, 63);
    }
}
// the same for sequences too long for the bitmap: insertion sort, one thread per list
__global__ void rev_sort_serial(BwdArgs a) {
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= a.nb) return;
    int32_t *x = a.rev_idx + a.rev_ptr[b];
    const int len = a.rev_ptr[b + 1] - a.rev_ptr[b];
    for (int i = 1; i < len; ++i) {
        int v = x[i], j = i - 1;
        while (j >= 0 && x[j] > v) {
            x[j + 1] = x[j];
            --j;
        }
        x[j + 1] = v;
    }
}

// Everything that the walks need where the routing table is small, in one launch: gradient rows and tables (prep_rows), tile images
// (pack_block) and, one workgroup per key block, the reverse list, its place and the block's tasks.  As five launches
// that is 6 + 5 + 7 + 4 + 4 us and the gaps between them for 6 K tokens of 4 heads of 64, most of them with a few workgroups; here 8.7 us.
// A workgroup counts all entries of the table by itself (in LDS), which tells it the lists, parts and lengths of all other
// blocks without another launch, then writes its list by going through the table once more: ascending, and the same in every
// run, as it is.  Eight loads of the table in flight to a wavefront: a pass of 16 K entries is eight round trips.
// Tasks as rev_scan_order puts them: longest first, whole parts, then the blocks' last parts.  all_slots: sums for every walk
// (bwd_walks_small), not only for those that are dealt out.
constexpr int kTableBlocks = 768, kTableEntries = 16384;  // (see small_table)
template <int D>
__global__ __launch_bounds__(PrepGeo<D>::THREADS) void bwd_prepare(BwdArgs a, int64_t n_prep, int64_t n_token_wg, int64_t n_pack,
                                                                    int all_slots, GroupTableArgs tables) {
    constexpr int THREADS = PrepGeo<D>::THREADS, WAVES = THREADS / 64, DEEP = 8, SUMS = 6;
    __shared__ union {
        PrepStage<D> prep;
        __attribute__((aligned(16))) PackStage<D> pack;
        struct {
            int count[kTableBlocks], of_wave[WAVES], sum[SUMS][WAVES];
        } rev;
    } lds;
    if (blockIdx.x < n_prep) {
        prep_rows<D>(a, lds.prep, blockIdx.x);
        return;
    }
    if (blockIdx.x < n_prep + n_pack) {
        pack_block<D, THREADS>(a, lds.pack, n_token_wg, blockIdx.x - n_prep);
        return;
    }
    const int kb = (int)(blockIdx.x - n_prep - n_pack), t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (kb >= a.nb) {
        const int i = (kb - a.nb) * THREADS + t;
        if (i < tables.n) group_table_entry(i, tables.ng, tables.nb, tables.goff, tables.count, tables.tab);
        return;
    }
    const int n_entries = a.nb * a.topk, per_wave = (n_entries + WAVES - 1) / WAVES;
    const int e0 = min(wave * per_wave, n_entries), e1 = min(e0 + per_wave, n_entries);
    // the entries [e0, e1) of this wavefront, 64 at a time: take(first entry, this lane's, -1 past the end)
    auto each = [&](auto take) {
        for (int e = e0; e < e1; e += 64 * DEEP) {
            int v[DEEP];
#pragma unroll
            for (int j = 0; j < DEEP; ++j) v[j] = e + 64 * j + lane < e1 ? a.idx[e + 64 * j + lane] : -1;
#pragma unroll
            for (int j = 0; j < DEEP; ++j) take(e + 64 * j, v[j]);
        }
    };
    for (int b = t; b < a.nb; b += THREADS) lds.rev.count[b] = 0;
    __syncthreads();
    int mine = 0;  // entries of this wavefront's part of the table that name kb
    each([&](int, int v) {
        if (v >= 0 && v < a.nb) atomicAdd(&lds.rev.count[v], 1);
        mine += __popcll(__ballot(v == kb));
    });
    if (lane == 0) lds.rev.of_wave[wave] = mine;
    __syncthreads();
    auto walk_of = [&](int b) { return 2 * lds.rev.count[b] + (a.cut_window ? (window_tiles(a, b).n + 1) & ~1 : 0); };
    auto parts_of = [&](int steps) { return max(1, (steps + a.part_steps - 1) / a.part_steps); };
    const int steps = walk_of(kb), np = parts_of(steps), last = steps - (np - 1) * a.part_steps;
    // of the blocks before kb: entries, slots of sums, whole parts, cut blocks; of all: whole parts, last parts that go before kb's
    int x[SUMS] = {0, 0, 0, 0, 0, 0};
    for (int b = t; b < a.nb; b += THREADS) {
        const int w = walk_of(b), n = parts_of(w), rest = w - (n - 1) * a.part_steps;
        const bool before = b < kb;
        x[0] += before ? lds.rev.count[b] : 0;
        x[1] += before && (all_slots || a.hsplit > 1 || n > 1) ? n : 0;
        x[2] += before ? n - 1 : 0;
        x[3] += before && n > 1 ? 1 : 0;
        x[4] += n - 1;
        x[5] += rest > last || (rest == last && before) ? 1 : 0;
    }
#pragma unroll
    for (int k = 0; k < SUMS; ++k) {
        for (int off = 32; off > 0; off >>= 1) x[k] += __shfl_xor(x[k], off);
        if (lane == 0) lds.rev.sum[k][wave] = x[k];
    }
    __syncthreads();
    int at = 0;
#pragma unroll
    for (int k = 0; k < SUMS; ++k) x[k] = 0;
    for (int w = 0; w < WAVES; ++w) {
#pragma unroll
        for (int k = 0; k < SUMS; ++k) x[k] += lds.rev.sum[k][w];
        at += w < wave ? lds.rev.of_wave[w] : 0;
    }
    for (int p = t; p < np; p += THREADS) {
        const int task = p < np - 1 ? x[2] + p : x[4] + x[5];
        a.order[task] = kb;
        a.order_part[task] = p;
    }
    if (t == 0) {
        a.walk[kb] = steps;
        a.slot0[kb] = x[1];
        a.rev_ptr[kb] = x[0];
        if (np > 1) a.split_list[x[3]] = kb;
        if (kb == a.nb - 1) {
            a.rev_ptr[a.nb] = x[0] + lds.rev.count[kb];
            a.task_n[0] = x[4] + a.nb;
            a.task_n[1] = x[3] + (np > 1 ? 1 : 0);
        }
    }
    at += x[0];
    each([&](int e, int v) {
        const unsigned long long m = __ballot(v == kb);
        if (v == kb) a.rev_idx[at + __popcll(m & ((1ull << lane) - 1ull))] = (e + lane) / a.topk;
        at += __popcll(m);
    });
}

// Position of the n-th (from 0) set bit of m; 0 <= result <= 63 whatever n is (meaningful for n < popcount(m)).
__device__ __forceinline__ int nth_set_bit(unsigned long long m, int n) {
    int pos = 0;
#pragma unroll
    for (int w = 32; w >= 1; w >>= 1) {
        const int below = __popcll(m & ((1ull << w) - 1ull));
        if (n >= below) {
            n -= below;
            m >>= w;
            pos += w;
        }
    }
    return pos;
}

// The partial gradients of the pooled keys / values, summed over the query ranges in order into range 0's slot,
// so that the token-key workgroups read one row per pooled pair however many ranges there were.
// (Eight ranges' rows are requested at a time: one dependent load after another took 31 us for 64 ranges.)
__global__ __launch_bounds__(256) void sum_parts(float *__restrict__ part_k, float *__restrict__ part_v, int n_split,
                                                 int64_t per_split) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= per_split) return;
    float *part = blockIdx.y == 0 ? part_k : part_v;
    f32x4 acc = *reinterpret_cast<const f32x4 *>(part + i);
    int sp = 1;
    for (; sp + 8 <= n_split; sp += 8) {
        f32x4 x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = *reinterpret_cast<const f32x4 *>(part + (sp + j) * per_split + i);
#pragma unroll
        for (int j = 0; j < 8; ++j) acc += x[j];
    }
    for (; sp < n_split; ++sp) acc += *reinterpret_cast<const f32x4 *>(part + sp * per_split + i);
    *reinterpret_cast<f32x4 *>(part + i) = acc;
}

// ---------------------------------------------------------------------------------------------
// dQ: one workgroup (2 wavefronts x 32 query rows) per (query block, head), or four wavefronts that share the copies of tiles:
//   HEADS   two heads of one key/value head, which read the same tiles in all branches
//   BLOCKS  two query blocks of one head, which share the tiles of the pooled keys; the others' each block copies for itself, and
//           the barriers are common: a block with fewer steps waits for the other at the end
// WIDE: routing rows of 65..128 entries (two per lane of the list holder instead of one).
// lds: DQ_LDS bytes.  wg, unit: numbers of the workgroup; wg: query block or pair of them, unit: head or pair of heads.
enum Pair { ALONE, HEADS, BLOCKS };
template <int D, Pair PAIR = ALONE>
constexpr int DQ_LDS = PAIR == BLOCKS  ? 2 * kBwdNbuf * 2 * BGeo<D>::ROW
                       : PAIR == HEADS ? std::max(4 * 32 * BGeo<D>::OUT_ROW, kBwdNbuf * 2 * BGeo<D>::ROW)
                                       : kBwdNbuf * 2 * BGeo<D>::ROW;
template <int D, bool WIDE, Pair PAIR>
__device__ __forceinline__ void dq_walk(const BwdArgs &a, char *lds, int wg, int unit) {
    using G = BGeo<D>;
    constexpr int NS = G::NS, ND = G::ND;
    constexpr int TILE = 2 * G::ROW;     // K rows | V rows (K^T is read out of the K rows, see mfma_tr)
    constexpr int NBUF = kBwdNbuf;  // tile buffers: copies run NBUF - 1 tiles ahead
    static_assert((G::ROW / 1024) % 2 == 0, "");
    static_assert((PAIR != ALONE ? 4 : 2) * 32 * G::OUT_ROW <= DQ_LDS<D, PAIR>, "output staging fits in the tile buffers");
    // consecutive workgroup ids go round-robin to the 8 XCDs: give each XCD a contiguous range of
    // blocks so that neighbouring blocks (overlapping windows, similar routed sets) share its L2
    const int n_units = PAIR == BLOCKS ? (a.nb + 1) / 2 : a.nb, per_xcd = (n_units + 7) / 8;
    const int place = (wg & 7) * per_xcd + (wg >> 3);
    if (place >= n_units) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int head = PAIR == HEADS ? 2 * unit + (wave >> 1) : unit;
    const int blk = PAIR == BLOCKS ? wave >> 1 : 0;             // query block inside the workgroup
    const bool active = PAIR != BLOCKS || 2 * place + blk < a.nb;  // (without one: the pooled keys for the last block once more, not stored)
    const int qb = PAIR == BLOCKS ? min(2 * place + blk, a.nb - 1) : place;
    const int r = lane & 31, hh = lane >> 5;
    const uint32_t lane16 = (uint32_t)lane * 16u;
    const int64_t row0 = (int64_t)qb * 64 + 32 * (wave & 1);
    const int half_w = a.window / 2;
    const int kvh = head / a.group;  // key/value head of this query head
    const uint32_t tr_off = tr_lane_offset(lane), row_off = row_lane_offset(lane);

    bf16x8 qf[NS], dof[NS];
    // the query rows, and the gradient rows of branch b (dout itself, or gate o dout with per-channel gates), out of
    // their tile images: 1 KB contiguous per fragment, padding slots are zeros there
    const int64_t img_off = ((row0 >> 5) * a.h + head) * (int64_t)G::IMG + (hh * 32 + (perm32(r) ^ (hh << 2))) * 16;
    auto load_dof = [&](int b) {
#pragma unroll
        for (int ks = 0; ks < NS; ++ks) dof[ks] = *reinterpret_cast<const bf16x8 *>(a.img_do[b] + img_off + ks * 1024);
    };
#pragma unroll
    for (int ks = 0; ks < NS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(a.img_q + img_off + ks * 1024);
    load_dof(0);
    float l2[3], dl[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const float *ax = a.aux + (((int64_t)b * a.nt + (row0 >> 5)) * a.h + head) * 64;
        l2[b] = ax[perm32(r)];
        dl[b] = ax[32 + perm32(r)];
    }
    f32x16 acc[ND];
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[dt][i] = 0.f;

    // ---- the tiles of this query block: pooled, routed, window
    const int tc = (a.nbc + 31) / 32;
    // the routing row, valid entries first: entry u sits in lane u % 64 of register u / 64.  Compacted with lane
    // permutes, not through LDS memory: with a second LDS object in the kernel the compiler can no longer tell the
    // tile buffers' reads from the copies in flight and puts a full vmcnt wait in front of the first read of every
    // step (measured: the kernel 8 % slower).
    constexpr int NR = WIDE ? 2 : 1;
    int packed[NR], pcount[NR], n_valid = 0;
    {
        int v[NR], nv[NR];
        unsigned long long bal[NR];
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const int col = lane + 64 * j;
            v[j] = col < a.topk ? a.idx[(int64_t)qb * a.topk + col] : -1;
            if (v[j] >= a.nb) v[j] = -1;
            bal[j] = __ballot(v[j] >= 0);
            nv[j] = __popcll(bal[j]);
            n_valid += nv[j];
        }
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            // the entry of rank lane + 64 j: the (rank)-th valid one of register 0, or the (rank - nv[0])-th of register 1
            const int rank = lane + 64 * j;
            int val = __builtin_amdgcn_ds_bpermute(4 * nth_set_bit(bal[0], rank), v[0]);
            if constexpr (WIDE) {
                const int val1 = __builtin_amdgcn_ds_bpermute(4 * nth_set_bit(bal[1], rank - nv[0]), v[1]);
                if (rank >= nv[0]) val = val1;
            }
            packed[j] = rank < n_valid ? val : -1;
        }
    }
    // active tokens of the routed blocks, held like the list itself
#pragma unroll
    for (int j = 0; j < NR; ++j) pcount[j] = a.count != nullptr && lane + 64 * j < n_valid ? a.count[packed[j]] : 64;
    auto entry = [&](const int (&reg)[NR], int u) {  // wave-uniform u
        if constexpr (WIDE) {
            const int e0 = __builtin_amdgcn_readlane(reg[0], u & 63), e1 = __builtin_amdgcn_readlane(reg[NR - 1], u & 63);
            return u < 64 ? e0 : e1;
        } else {
            return __builtin_amdgcn_readlane(reg[0], u);
        }
    };
    const int ts = active ? 2 * n_valid : 0;
    int seg_lo = 0, seg_hi = 0;
    if (a.blk_seg != nullptr) {  // the query's spatial block
        seg_lo = a.blk_seg[2 * qb];
        seg_hi = a.blk_seg[2 * qb + 1];
    } else {
        for (int s = 0; s < a.n_seg; ++s)
            if (qb * 64 >= a.seg[s] && qb * 64 < a.seg[s + 1]) {
                seg_lo = a.seg[s];
                seg_hi = a.seg[s + 1];
            }
    }
    if (a.own_block) {  // window = the query's own block: the block is its own segment (a.window is 128)
        seg_lo = qb * 64;
        seg_hi = qb * 64 + 64;  // (padding slots at its end are masked per tile below)
    }
    const int k_start = max(seg_lo, qb * 64 - half_w), k_end = min(seg_hi, qb * 64 + 63 + half_w);
    const int st0 = k_start / 32;
    // active tokens of the blocks of the window range, one per lane (a range of more than 64 blocks falls back to
    // loading the count inside the loop)
    const int wcount = a.count != nullptr && (st0 >> 1) + lane < a.nb ? a.count[(st0 >> 1) + lane] : 64;
    const int tw = active && k_end > k_start ? (k_end - 1) / 32 + 1 - st0 : 0;
    const int T = tc + ts + tw;
    const int wlo = max(seg_lo, (int)row0 + r - half_w), whi = min(seg_hi, (int)row0 + r + half_w);

    // Two tile buffers: the copy of tile t+1 is issued behind the barrier of step t and waited for before the
    // barrier of step t+1.  The walk is one pipelined loop per branch, so that everything that depends on the
    // branch (tile lookup, image, mask rule, table entries) is fixed inside a loop; the first tile of the next
    // branch is requested in the last step of the one before it, so the pipeline never drains.
    static_assert(NBUF == 2, "");
    // Two query blocks: the tiles of the compressed branch in the first buffer of either block, shared; then each block's own, from
    // its second buffer on.
    auto buffer = [&](int t) {
        if constexpr (PAIR != BLOCKS) return lds + (t & 1) * TILE;
        return lds + (t < tc ? 2 * (t & 1) : 2 * blk + ((t - tc + 1) & 1)) * TILE;
    };
    auto issue_tile = [&](auto shared, const char *kimg, const char *vimg, int tile, char *buf) {
        const int64_t off = (int64_t)((uint32_t)tile * (uint32_t)a.h_kv + (uint32_t)kvh) * G::IMG;
        if constexpr (PAIR == HEADS || (PAIR == BLOCKS && decltype(shared)::value)) {
            // K rows and V rows, one behind the other, dealt to four wavefronts
            constexpr int KB = G::ROW / 1024;
#pragma unroll
            for (int j = 0; j < 2 * KB; j += 4) {
                const int i = j + wave;
                copy_kb_to_lds((i < KB ? kimg : vimg - G::ROW) + off + i * 1024, lane16, buf + i * 1024);
            }
        } else {
            copy_kb<G::ROW / 1024>(kimg + off, buf, wave & 1, lane16);
            copy_kb<G::ROW / 1024>(vimg + off, buf + G::ROW, wave & 1, lane16);
        }
    };
    // tile of step t of the whole walk (used at the branch boundaries only)
    auto issue_any = [&](int t, char *buf) {
        if (t < tc) {
            issue_tile(std::true_type{}, a.img_kc, a.img_vc, t, buf);
        } else if (t < tc + ts) {
            const int u = t - tc;
            issue_tile(std::false_type{}, a.img_k, a.img_v, 2 * entry(packed, u >> 1) + (u & 1), buf);
        } else {
            issue_tile(std::false_type{}, a.img_k, a.img_v, st0 + (t - tc - ts), buf);
        }
    };
    // steps [t0, t1) of the walk, all of branch BR.  tile_fn(u): image tile of the u-th step of the branch;
    // mask_fn(u, &j0, &lo, &hi) -> does this tile need a mask: key j0 + (position in the tile) is attended iff
    // lo <= key < hi (per lane)
    auto run_branch = [&](int t0, int t1, auto br_c, const char *kimg, const char *vimg, auto tile_fn, auto mask_fn) {
        constexpr int BR = decltype(br_c)::value;
        const float lb = l2[BR];
        f32x16 dp0;  // -D of this lane's query: the dP accumulator starts from it, so the MFMAs leave dP - D
#pragma unroll
        for (int i = 0; i < 16; ++i) dp0[i] = dl[BR];
        for (int t = t0; t < t1; ++t) {
            // tile t has landed (this wavefront's share; the barrier covers the others'); all wavefronts are done
            // with tile t-1, whose buffer takes tile t+1
            __builtin_amdgcn_s_waitcnt(vm_lgkm_imm(0));
            wg_barrier();
            char *nbuf = buffer(t + 1);
            const char *tile_k = buffer(t);
            const char *base = tile_k + row_off;

            // The pieces of the step in a fixed order (a wavefront issues in order: what is to overlap has to alternate
            // in the program).  K and V row fragments go through one rolling queue of QD registers sets, refilled
            // behind the MFMA that consumed a set; the score chain, then the dP chain with the tile's exponentials
            // behind its MFMAs (unmasked; edge tiles are fixed up afterwards); then the transposing loads of K^T are
            // requested, dS of the first 16-key slab is formed, and the dQ MFMAs run with the second slab's dS
            // behind the first ones.
            constexpr int QD = NS < 4 ? NS : 4;
            bf16x8 fq[QD];
            auto frag = [&](int i) {  // fragment i of the K rows (i < NS) or of the V rows
                return *reinterpret_cast<const bf16x8 *>(base + (i < NS ? i * 1024 : G::ROW + (i - NS) * 1024));
            };
#pragma unroll
            for (int i = 0; i < QD; ++i) fq[i] = frag(i);
            __builtin_amdgcn_sched_barrier(0);
            // the copies of the next tile: their address arithmetic runs while the first reads land
            if (t + 1 < t1)
                issue_tile(std::integral_constant<bool, BR == 0>{}, kimg, vimg, tile_fn(t + 1 - t0), nbuf);
            else if (t + 1 < T)
                issue_any(t + 1, nbuf);
            int j0, lo, hi;
            const bool need_mask = mask_fn(t - t0, &j0, &lo, &hi);
            f32x16 s, dp;
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = 0.f;
            __builtin_amdgcn_sched_barrier(0);
            auto s_step = [&](auto kc) {
                constexpr int ks = decltype(kc)::value;
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fq[ks % QD], qf[ks], s, 0, 0, 0);
                fq[ks % QD] = frag(ks + QD);
                __builtin_amdgcn_sched_barrier(0);
            };
            for_each_index<NS>(s_step);
            constexpr int E = 16 / NS;  // exponentials per dP MFMA
            float pr[16];
            auto dp_step = [&](auto kc) {
                constexpr int ks = decltype(kc)::value;
                dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fq[ks % QD], dof[ks], ks == 0 ? dp0 : dp, 0, 0, 0);
                if constexpr (ks + QD < NS) fq[ks % QD] = frag(NS + ks + QD);
#pragma unroll
                for (int e = ks * E; e < (ks + 1) * E; ++e) {
                    pr[e] = __builtin_amdgcn_exp2f(s[e] * a.sl2 - lb);
                    asm volatile("" : "+v"(pr[e]));
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            for_each_index<NS>(dp_step);
            // with per-channel gates the gradient rows change with the branch: the next branch's are requested
            // once the last dP MFMAs of this one are issued, and have arrived by the wait at the top of the next step
            if (BR < 2 && a.gate_channels && t + 1 == t1 && t + 1 < T) load_dof(t + 1 < tc + ts ? 1 : 2);
            TrFrag ft[2 * ND];
            const uint32_t tr_k = (uint32_t)(uintptr_t)tile_k + tr_off;
            auto issue_tr = [&](auto ic) {
                constexpr int I = decltype(ic)::value;
                tr_issue<(I % ND) * 2048 + (I / ND) * 256>(ft[I], tr_k);
            };
            for_each_index<2 * ND>(issue_tr);
            if (__builtin_expect(need_mask, 0)) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int j = j0 + 16 * (i / 8) + 8 * hh + (i % 8);
                    pr[i] = ((j >= lo) & (j < hi)) ? pr[i] : 0.f;
                }
            }
            BFrag dsb[2];
#pragma unroll
            for (int k = 0; k < 4; ++k) dsb[0].u[k] = pack_bf16(pr[2 * k] * dp[2 * k], pr[2 * k + 1] * dp[2 * k + 1]);
            __builtin_amdgcn_sched_barrier(0);
            constexpr int EQ = 4 / ND > 0 ? 4 / ND : 1;  // bf16 pairs of the second slab's dS per MFMA of the first slab
            auto dq_step = [&](auto ic) {
                constexpr int I = decltype(ic)::value;
                acc[I % ND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr_take<2 * (2 * ND - 1 - I)>(ft[I]), dsb[I / ND].v,
                                                                      acc[I % ND], 0, 0, 0);
                if constexpr (I < ND) {
#pragma unroll
                    for (int k = 4 + I * EQ; k < 4 + (I + 1) * EQ && k < 8; ++k) {
                        dsb[1].u[k - 4] = pack_bf16(pr[2 * k] * dp[2 * k], pr[2 * k + 1] * dp[2 * k + 1]);
                        asm volatile("" : "+v"(dsb[1].u[k - 4]));
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            for_each_index<2 * ND>(dq_step);
        }
    };
    // padding slots at the end of a tile's block are no keys: valid keys of the tile, given its block's count
    auto valid_keys = [&](int cnt, int half) { return min(32, max(0, cnt - 32 * half)); };

    if (T > 0) issue_any(0, lds);
    int t_all = T;  // steps of the workgroup
    if constexpr (PAIR == BLOCKS) {
        int *const steps = reinterpret_cast<int *>(lds + 3 * TILE);  // (a buffer that step tc - 1 is the first to fill)
        if (lane == 0) steps[wave] = T;
        __syncthreads();
        t_all = __builtin_amdgcn_readfirstlane(max(T, steps[wave ^ 2]));
    }
    // pooled keys: only the last tile can reach past the end
    run_branch(0, tc, std::integral_constant<int, 0>{}, a.img_kc, a.img_vc, [&](int u) { return u; },
               [&](int u, int *j0, int *lo, int *hi) {
                   *j0 = 32 * u;
                   *lo = 0;
                   *hi = a.nbc;
                   return 32 * u + 32 > a.nbc;
               });
    // routed blocks: every key counts, except padding slots
    run_branch(tc, tc + ts, std::integral_constant<int, 1>{}, a.img_k, a.img_v,
               [&](int u) { return 2 * entry(packed, u >> 1) + (u & 1); },
               [&](int u, int *j0, int *lo, int *hi) {
                   *j0 = 0;
                   *lo = 0;
                   *hi = 32;
                   if (a.count == nullptr) return false;
                   *hi = valid_keys(entry(pcount, u >> 1), u & 1);
                   return *hi < 32;
               });
    // window: the band's edges and the segment's ends, and padding slots
    const int edge_lo = max(seg_lo, (int)row0 + 31 - half_w), edge_hi = min(seg_hi, (int)row0 + half_w);
    run_branch(tc + ts, T, std::integral_constant<int, 2>{}, a.img_k, a.img_v, [&](int u) { return st0 + u; },
               [&](int u, int *j0, int *lo, int *hi) {
                   const int st = st0 + u;
                   *j0 = 32 * st;
                   *lo = wlo;
                   *hi = whi;
                   bool need = 32 * st < edge_lo || 32 * st + 32 > edge_hi;
                   if (a.count != nullptr) {
                       const int wb = (st >> 1) - (st0 >> 1);  // block of the window range
                       const int cnt = wb < 64 ? __builtin_amdgcn_readlane(wcount, wb) : a.count[st >> 1];
                       const int vld = valid_keys(cnt, st & 1);
                       if (vld < 32) {
                           need = true;
                           *hi = min(*hi, 32 * st + vld);
                       }
                   }
                   return need;
               });
    for (int t = T; PAIR == BLOCKS && t < t_all; ++t) wg_barrier();  // (the other block's steps)
    __syncthreads();  // the tile buffers become the output staging
    if (!active) return;
    float x[ND][16];
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) x[dt][i] = acc[dt][i] * a.scale;
    store_rows_transposed<D>(x, lds + wave * 32 * G::OUT_ROW, a.dq + (row0 * a.h + head) * D, (int64_t)a.h * D, lane);
}
template <int D, bool WIDE, Pair PAIR>
__global__ __launch_bounds__((PAIR != ALONE ? 256 : 128), (D == 128 ? 2 : D == 64 ? 3 : 4)) void bwd_dq_kernel(BwdArgs a) {
    // (at d = 128 the 256-register budget of two workgroups per SIMD still holds: 64 accumulator registers; at d = 64 wide rows fit the 168
    // of three wavefronts only if the compiler is told to: 1536 blocks, 4 heads, rows of 80 2869 -> 2793 us the whole backward)
    __shared__ __attribute__((aligned(1024))) char lds[DQ_LDS<D, PAIR>];
    dq_walk<D, WIDE, PAIR>(a, lds, blockIdx.x, blockIdx.y);
}

// ---------------------------------------------------------------------------------------------
// dK, dV: one workgroup (WV wavefronts x 32 keys) per (key block or group of pooled keys, key/value head, range of query
// heads or of query tiles); the query tiles of each of the `group` query heads of a key/value head are walked in turn.
// SUMS (MODE 0): every walk leaves fp32 sums for a last pass, which is also where the pooled gradients come in.
// V_LDS: the value fragments of a wavefront's keys are read from LDS in every step instead of held in 32 registers.  At
// d = 128, where the two [128 x 32] sets of sums alone take 128, that is what lets two wavefronts share a SIMD (223 registers,
// in the plain order of a step), each filling the other's waits.  Done for many pooled keys (kPooledWide), with four wavefronts to a
// workgroup: they share a tile's copies, and two workgroups' buffers and values fit the LDS of a CU.  Backward before / after, ms,
// blocks x heads: 512 x 16 2.45 / 2.41, 2560 x 8 10.7 / 10.1, 4096 x 16 (2) 43.9 / 42.2, 6704 x 16 127.9 / 117.7.  Not done for
// the token keys: 9 registers more than there are, and the last of these took 121 to 122 ms either way; nor in the joint launch
// of small problems (192 x 6 305 / 300 us, 132 x 1 61 / 65).
// lds: DKV_LDS bytes.  wg: place in the order of tasks, or group of 32 * WV pooled keys; z: head range, or range of query tiles.
template <int D, int WV, bool V_LDS>
constexpr int DKV_LDS = kBwdDkvNbuf * (2 * BGeo<D>::ROW + 1024) + (V_LDS ? WV * BGeo<D>::ROW : 0);
template <int D, int MODE, bool SUMS, int WV, bool V_LDS>
__device__ __forceinline__ void dkv_walk(const BwdArgs &a, char *lds, int wg, int head, int z) {
    using G = BGeo<D>;
    constexpr int NS = G::NS, ND = G::ND;
    constexpr int AUX = 2 * G::ROW;          // Q rows | dO rows | table (64 floats); Q^T and dO^T: see mfma_tr
    constexpr int TILE = 2 * G::ROW + 1024;  // (table padded to keep the next buffer aligned)
    static_assert(2 * 32 * G::OUT_ROW <= kBwdDkvNbuf * TILE, "output staging fits in the tile buffers");
    static_assert(MODE == 1 || WV == 2, "a block of token keys");
    int kb = wg;
    int part = 0;  // of the key block's walk
    if (MODE == 0) {  // token keys: longest walk first (see rev_scan_order)
        if (wg >= a.task_n[0]) return;
        kb = a.order[wg];
        part = a.order_part[wg];
    }
    const int walk = MODE == 0 ? a.walk[kb] : 0;
    const int split = MODE == 1 ? z : 0;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, hh = lane >> 5;
    const uint32_t lane16 = (uint32_t)lane * 16u;
    const uint32_t tr_off = tr_lane_offset(lane), row_off = row_lane_offset(lane);
    const int64_t key0 = (int64_t)kb * (32 * WV) + 32 * wave;  // token index (MODE 0) or pooled-key index (MODE 1)
    const int64_t key = key0 + r;
    const int64_t limit = MODE == 0 ? a.n : (int64_t)a.nbc;
    const int half_w = a.window / 2;
    // MODE 0 with per-block counts: a padding slot is nobody's key (its probabilities are zeroed) and gets a zero gradient
    const int n_act = MODE == 0 && a.count != nullptr ? a.count[kb] : 64;
    const bool key_active = MODE == 1 || 32 * wave + r < n_act;

    bf16x8 kB[NS], vB[NS];
    char *const v_own = lds + kBwdDkvNbuf * TILE + wave * G::ROW + lane * 16;  // V_LDS: this lane's part of fragment 0, its own only
    {
        const int64_t krow_i = key < limit ? key : limit - 1;  // (rows past the end are masked below)
        const uint16_t *krow = (MODE == 0 ? a.k : a.kc) + (krow_i * a.h_kv + head) * D + 8 * hh;
        const uint16_t *vrow = (MODE == 0 ? a.v : a.vc) + (krow_i * a.h_kv + head) * D + 8 * hh;
#pragma unroll
        for (int ks = 0; ks < NS; ++ks) {
            kB[ks] = *reinterpret_cast<const bf16x8 *>(krow + 16 * ks);
            vB[ks] = *reinterpret_cast<const bf16x8 *>(vrow + 16 * ks);
            if (!key_active) {  // a padding slot reads as zeros, whatever the caller left there
                const bf16x8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
                kB[ks] = vB[ks] = zero8;
            }
            if constexpr (V_LDS) *reinterpret_cast<bf16x8 *>(v_own + ks * 1024) = vB[ks];
        }
    }
    f32x16 acck[ND], accv[ND];
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acck[dt][i] = accv[dt][i] = 0.f;

    // ---- the query tiles that attend these keys
    int tw = 0, wt0 = 0, n_e = 0, e0 = 0, T = 0;  // window / pooled: first tile, how many; reverse list: first entry, how many
    if (MODE == 1) {
        wt0 = split * a.tiles_per_split;
        T = max(0, min(a.nt, wt0 + a.tiles_per_split) - wt0);
    } else {
        const WindowTiles win = window_tiles(a, kb);
        const int lo = part * a.part_steps, hi = min(lo + a.part_steps, walk);  // this part's share of the walk
        const int counted = a.cut_window ? (win.n + 1) & ~1 : 0;                // counted window tiles
        const int w_lo = a.cut_window ? min(lo, win.n) : 0, w_hi = a.cut_window ? min(hi, win.n) : (part == 0 ? win.n : 0);
        wt0 = win.first + w_lo;
        tw = w_hi - w_lo;
        const int e_lo = max(lo - counted, 0) >> 1, e_hi = max(hi - counted, 0) >> 1;
        e0 = a.rev_ptr[kb] + e_lo;
        n_e = e_hi - e_lo;
    }
    // The walk is cut into segments with one pipelined loop each: the window tiles, then the routed tiles 64
    // reverse-list entries at a time (one entry per lane, loaded before the loop).  Inside a loop nothing is loaded
    // into registers from global memory: the wait for such a load would also wait for every tile copy in flight.
    // the query heads of the group this workgroup walks: all of them, or (token keys, heads dealt to hsplit
    // workgroups) its share
    const int gh0 = MODE == 0 && a.hsplit > 1 ? z * a.hpw : 0;
    const int grp = MODE == 0 && a.hsplit > 1 ? min(a.group, gh0 + a.hpw) - gh0 : a.group;
    constexpr bool VGPR_CHAINS = D == 128 && !V_LDS;  // (the kernel has one wavefront per SIMD: see mfma_v)
    // the step in its interleaved form (step_interleaved below).  Not with two wavefronts per SIMD; not at d = 64: there it needs more than the 168
    // registers of three wavefronts per SIMD, and with two it measured slower (config 5: 1.12 -> 1.25 ms).
    constexpr bool INTERLEAVE = D != 64 && !V_LDS;
    static_assert(kBwdDkvNbuf == 2, "the copies of a step go out one step ahead");
    // br_c: the branch whose probabilities these are (0 compressed, 1 selected, 2 window); tile_fn(t): the t-th query
    // tile of the segment (arithmetic on registers only); every tile is met by the grp query heads of this key/value
    // head in turn
    auto run_segment = [&](int n_t, auto br_c, auto tile_fn) {
        constexpr int BR = decltype(br_c)::value;
        const int U = n_t * grp;
        if (U <= 0) return;
        const char *img_do = a.img_do[BR];
        const float *aux_br = a.aux + (int64_t)BR * a.nt * a.h * 64;  // table of this branch: [tile][head][64]
        auto issue = [&](int t, int gh, char *buf) {
            // (tile, head) index in 32 bits, byte offsets by shifts: a 64-bit multiply is several scalar instructions
            const uint32_t ih = (uint32_t)tile_fn(t) * (uint32_t)a.h + (uint32_t)(head * a.group + gh0 + gh);
            const int64_t off = (int64_t)ih * G::IMG;
            copy_kb<G::ROW / 1024, WV>(a.img_q + off, buf, wave, lane16);
            copy_kb<G::ROW / 1024, WV>(img_do + off, buf + G::ROW, wave, lane16);
            if (wave == 0)
                copy_256_to_lds(aux_br + (int64_t)ih * 64, lane16 >> 2, buf + AUX);
        };
        int t = 0, gh = 0, t_nxt = 0, gh_nxt = 0;  // the step being computed, the step being copied
        auto advance = [&](int &tt, int &gg) {     // (counters instead of a division per step)
            if (++gg == grp) {
                gg = 0;
                ++tt;
            }
        };
        // ---- the pieces of a step (one 32-query tile against this wavefront's 32 keys)
        struct Tile {
            const char *buf;  // its buffer: Q rows | dO rows | table
            int q0;           // first query of the tile
            bool win;         // a window tile at the band's edge: positions outside the band are masked
            f32x16 s, dp;
            float p[16];
        };
        // S = Q K^T
        auto ph_scores = [&](Tile &x, const char *buf, int tile) {
            x.buf = buf;
            x.q0 = 32 * tile;
            // window tiles away from the band's edges (and all routed tiles) need no mask
            x.win = BR == 2 && ((int)key0 - (x.q0 + 31) < -half_w || (int)key0 + 31 - x.q0 >= half_w);
            const char *base = buf + row_off;
            if constexpr (VGPR_CHAINS) {
                mfma_v_first(x.s, *reinterpret_cast<const bf16x8 *>(base), kB[0]);
#pragma unroll
                for (int ks = 1; ks < NS; ++ks) mfma_v(x.s, *reinterpret_cast<const bf16x8 *>(base + ks * 1024), kB[ks]);
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) x.s[i] = 0.f;
#pragma unroll
                for (int ks = 0; ks < NS; ++ks)
                    x.s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8 *>(base + ks * 1024),
                                                                  kB[ks], x.s, 0, 0, 0);
            }
        };
        // dP - D = dout V^T - D: the accumulator starts from -D of the 16 query rows this lane holds (second half
        // of the table, rows (i/4)*8 + hh*4 + i%4)
        auto ph_dp = [&](Tile &x) {
            const char *base = x.buf + row_off;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 y = *reinterpret_cast<const f32x4 *>(x.buf + AUX + 128 + (8 * g + 4 * hh) * 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) x.dp[4 * g + j] = y[j];
            }
#pragma unroll
            for (int ks = 0; ks < NS; ++ks) {
                const bf16x8 rows = *reinterpret_cast<const bf16x8 *>(base + G::ROW + ks * 1024);
                if constexpr (VGPR_CHAINS)
                    mfma_v(x.dp, rows, vB[ks]);
                else
                    x.dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        rows, V_LDS ? *reinterpret_cast<const bf16x8 *>(v_own + ks * 1024) : vB[ks], x.dp, 0, 0, 0);
            }
        };
        // P = exp2(S scale log2e - offset), the offsets of the query rows from the first half of the table
        // (read right before their use: fewer registers live at once)
        auto ph_exp = [&](Tile &x) {
            float lv[16];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 y = *reinterpret_cast<const f32x4 *>(x.buf + AUX + (8 * g + 4 * hh) * 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) lv[4 * g + j] = y[j];
            }
            // Most tiles need no mask at all (wave-uniform test): routed tiles and window tiles inside the band, of
            // blocks without padding; pooled keys before the last block.
            const bool plain = MODE == 1 ? key0 + 32 <= limit : (!x.win && n_act == 64);
            if constexpr (VGPR_CHAINS) mfma_v_settle(x.s);
            if (__builtin_expect(plain, 1)) {
#pragma unroll
                for (int i = 0; i < 16; ++i) x.p[i] = __builtin_amdgcn_exp2f(x.s[i] * a.sl2 - lv[i]);
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float pi = __builtin_amdgcn_exp2f(x.s[i] * a.sl2 - lv[i]);
                    bool ok;
                    if (MODE == 1) {
                        ok = key < limit;
                    } else {
                        const int qi = x.q0 + (i % 8) + 8 * hh + 16 * (i / 8);  // the query behind accumulator row i
                        const int dj = (int)key - qi;
                        ok = key_active & (!x.win | ((dj >= -half_w) & (dj < half_w)));
                    }
                    x.p[i] = ok ? pi : 0.f;
                }
            }
        };
        // dV^T += dout^T P
        auto ph_dv = [&](Tile &x) {
            BFrag pb[2];
            to_b_operand(x.p, pb);
            mfma_tr<ND>(accv, x.buf + G::ROW, tr_off, pb);
        };
        // dS = P o (dP - D), dK^T += Q^T dS
        auto ph_dk = [&](Tile &x) {
            if constexpr (VGPR_CHAINS) mfma_v_settle(x.dp);
            float ds[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) ds[i] = x.p[i] * x.dp[i];
            BFrag dsb[2];
            to_b_operand(ds, dsb);
            mfma_tr<ND>(acck, x.buf, tr_off, dsb);
        };

        // The interleaved form of a step (INTERLEAVE).  A wavefront issues in order, and this kernel has one wavefront
        // per SIMD at d = 128: whatever is to overlap -- vector arithmetic with MFMAs, LDS latency with either -- has to
        // alternate in the program.  Scheduling barriers fix the order of the pieces:
        //   reads of the Q rows | S#0, reads of the dout rows and of the table | S#1.. | (all reads have arrived)
        //   dP#k, each followed by its share of the exponentials (unmasked; edge tiles are fixed up afterwards) and by
        //     the transposing loads of one dout^T fragment
        //   dV#i (dout^T P), each followed by its share of dS = P o (dP - D) and by the loads of one Q^T fragment
        //   dK#i (Q^T dS)
        // The transposing loads are untracked (see tr_issue): their waits are counted by hand.  Fragment i of dout^T
        // is needed at dV#i, by when fragments i+1.. of dout^T and 0..i-1 of Q^T (two loads each) have been issued
        // behind it: at most 14 younger loads whatever i is; Q^T fragment i at dK#i has the 7-i later ones behind it.
        // The tracked reads (row fragments, table) are all waited for before the first untracked load is issued, so
        // the compiler's own counted waits never meet loads it does not know of.
        auto step_interleaved = [&](const char *buf, int tile, auto issue_next) {
            static_assert(!INTERLEAVE || 16 % NS == 0, "");
            const int q0 = 32 * tile;
            const bool win = BR == 2 && ((int)key0 - (q0 + 31) < -half_w || (int)key0 + 31 - q0 >= half_w);
            const bool plain = MODE == 1 ? key0 + 32 <= limit : (!win && n_act == 64);
            const char *base = buf + row_off;
            const uint32_t tr_q = (uint32_t)(uintptr_t)buf + tr_off, tr_do = tr_q + G::ROW;
            f32x16 sc, dp;
            float lv[16], pr[16];
            bf16x8 qr[NS], rows[NS];
#pragma unroll
            for (int ks = 0; ks < NS; ++ks) qr[ks] = *reinterpret_cast<const bf16x8 *>(base + ks * 1024);
            __builtin_amdgcn_sched_barrier(0);
            issue_next();  // the copies of the next step's tile: their address arithmetic runs while the reads land
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (VGPR_CHAINS) {
                mfma_v_first(sc, qr[0], kB[0]);
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) sc[i] = 0.f;
                sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qr[0], kB[0], sc, 0, 0, 0);
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 y = *reinterpret_cast<const f32x4 *>(buf + AUX + 128 + (8 * g + 4 * hh) * 4);
                const f32x4 z = *reinterpret_cast<const f32x4 *>(buf + AUX + (8 * g + 4 * hh) * 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    dp[4 * g + j] = y[j];
                    lv[4 * g + j] = z[j];
                }
            }
#pragma unroll
            for (int ks = 0; ks < NS; ++ks) rows[ks] = *reinterpret_cast<const bf16x8 *>(base + G::ROW + ks * 1024);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 1; ks < NS; ++ks) {
                if constexpr (VGPR_CHAINS)
                    mfma_v(sc, qr[ks], kB[ks]);
                else
                    sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qr[ks], kB[ks], sc, 0, 0, 0);
            }
            // every tracked read has arrived (the empty statements make the compiler wait for them here)
#pragma unroll
            for (int ks = 0; ks < NS; ++ks) asm volatile("" : "+v"(rows[ks]));
#pragma unroll
            for (int i = 0; i < 16; ++i) asm volatile("" : "+v"(lv[i]));
            asm volatile("" : "+v"(dp));
            if constexpr (VGPR_CHAINS) mfma_v_settle(sc);
            __builtin_amdgcn_sched_barrier(0);

            TrFrag fdo[2 * ND], fq[2 * ND];
            BFrag pb[2], dsb[2];
            // dP chain with the exponentials; dout^T fragments requested on the way (fragment f after MFMA f * NS / 2ND)
            constexpr int E = 16 / NS;
            auto issue_do = [&](auto ic) {
                constexpr int I = decltype(ic)::value;
                tr_issue<(I % ND) * 2048 + (I / ND) * 256>(fdo[I], tr_do);
            };
            auto issue_q = [&](auto ic) {
                constexpr int I = decltype(ic)::value;
                tr_issue<(I % ND) * 2048 + (I / ND) * 256>(fq[I], tr_q);
            };
            auto dp_step = [&](auto kc) {
                constexpr int ks = decltype(kc)::value;
                if constexpr (VGPR_CHAINS)
                    mfma_v(dp, rows[ks], vB[ks]);
                else
                    dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows[ks], vB[ks], dp, 0, 0, 0);
#pragma unroll
                for (int e = ks * E; e < (ks + 1) * E; ++e) {
                    pr[e] = __builtin_amdgcn_exp2f(sc[e] * a.sl2 - lv[e]);
                    if (e & 1) {
                        pb[e / 8].u[(e / 2) % 4] = pack_bf16(pr[e - 1], pr[e]);
                        asm volatile("" : "+v"(pb[e / 8].u[(e / 2) % 4]));
                    }
                    asm volatile("" : "+v"(pr[e]));
                }
                // NS MFMAs, 2 ND fragments: one fragment behind every (NS / 2ND)-th MFMA (NS = 2 ND * (NS / 2ND))
                if constexpr (ks % (NS / (2 * ND)) == 0) issue_do(std::integral_constant<int, ks / (NS / (2 * ND))>{});
                __builtin_amdgcn_sched_barrier(0);
            };
            for_each_index<NS>(dp_step);
            if constexpr (VGPR_CHAINS) mfma_v_settle(dp);
            if (__builtin_expect(!plain, 0)) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    bool ok;
                    if (MODE == 1) {
                        ok = key < limit;
                    } else {
                        const int qi = q0 + (i % 8) + 8 * hh + 16 * (i / 8);  // the query behind accumulator row i
                        const int dj = (int)key - qi;
                        ok = key_active & (!win | ((dj >= -half_w) & (dj < half_w)));
                    }
                    pr[i] = ok ? pr[i] : 0.f;
                }
                to_b_operand(pr, pb);
            }
            __builtin_amdgcn_sched_barrier(0);
            // dV with dS; Q^T fragments requested on the way
            constexpr int EV = 16 / (2 * ND);
            auto dv_step = [&](auto ic) {
                constexpr int I = decltype(ic)::value;
                // younger loads behind dout^T fragment I: its 2 ND - 1 - I successors and the I fragments of Q^T
                accv[I % ND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr_take<2 * (2 * ND - 1)>(fdo[I]), pb[I / ND].v,
                                                                       accv[I % ND], 0, 0, 0);
#pragma unroll
                for (int e = I * EV; e < (I + 1) * EV; e += 2) {
                    const float d0 = pr[e] * dp[e], d1 = pr[e + 1] * dp[e + 1];
                    dsb[e / 8].u[(e / 2) % 4] = pack_bf16(d0, d1);
                    asm volatile("" : "+v"(dsb[e / 8].u[(e / 2) % 4]));
                }
                issue_q(ic);
                __builtin_amdgcn_sched_barrier(0);
            };
            for_each_index<2 * ND>(dv_step);
            auto dk_step = [&](auto ic) {
                constexpr int I = decltype(ic)::value;
                acck[I % ND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr_take<2 * (2 * ND - 1 - I)>(fq[I]), dsb[I / ND].v,
                                                                       acck[I % ND], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            };
            for_each_index<2 * ND>(dk_step);
        };

        __builtin_amdgcn_s_waitcnt(vm_lgkm_imm(0));
        __syncthreads();  // both wavefronts are done with the buffers (previous segment)
        issue(t_nxt, gh_nxt, lds);
        advance(t_nxt, gh_nxt);
        for (int u = 0, slot = 0; u < U; ++u, advance(t, gh), slot ^= 1) {
            // The barrier alone does not wait for copies in flight (they are counted by vmcnt, which a
            // workgroup-scope fence leaves alone): every wavefront first waits for its own share of the
            // step's tile, then the barrier publishes all shares; it also tells that everyone is done with the
            // buffer refilled next.
            __builtin_amdgcn_s_waitcnt(vm_lgkm_imm(0));
            wg_barrier();
            auto issue_next = [&]() {
                if (u + 1 < U) {
                    issue(t_nxt, gh_nxt, lds + (slot ^ 1) * TILE);  // the buffer of step u - 1
                    advance(t_nxt, gh_nxt);
                }
            };
            if constexpr (INTERLEAVE) {
                step_interleaved(lds + slot * TILE, tile_fn(t), issue_next);
            } else {
                // (the plain order: scores, exponentials, dV, dP, dK; at d = 64 the interleaved one does not fit the
                // registers of three wavefronts per SIMD)
                issue_next();
                if (WV > 2 && key0 >= a.nbc) continue;  // (no keys in the last workgroup: copies and barriers only)
                Tile x;
                ph_scores(x, lds + slot * TILE, tile_fn(t));
                ph_exp(x);
                ph_dv(x);
                ph_dp(x);
                ph_dk(x);
            }
        }
    };
    if (MODE == 1) {
        run_segment(T, std::integral_constant<int, 0>{}, [&](int t) { return wt0 + t; });
    } else {
        run_segment(tw, std::integral_constant<int, 2>{}, [&](int t) { return wt0 + t; });
        for (int c0 = 0; c0 < n_e; c0 += 64) {
            const int rev_held = c0 + lane < n_e ? a.rev_idx[e0 + c0 + lane] : 0;
            run_segment(2 * min(64, n_e - c0), std::integral_constant<int, 1>{}, [&](int t) {
                return 2 * __builtin_amdgcn_readlane(rev_held, t >> 1) + (t & 1);
            });
        }
    }

    if (MODE == 0 && (SUMS || a.hsplit > 1 || walk > a.part_steps)) {
        // this workgroup's sums, fp32; the last pass finishes the rows
        const int64_t slot = (int64_t)z * a.max_slots + a.slot0[kb] + part;
        const int64_t o = ((slot * 64 + 32 * wave + r) * a.h_kv + head) * D;
#pragma unroll
        for (int dt = 0; dt < ND; ++dt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4 xk, xv;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    xk[j] = acck[dt][4 * g + j];
                    xv[j] = accv[dt][4 * g + j];
                }
                *reinterpret_cast<f32x4 *>(a.hpart_k + o + 32 * dt + 8 * g + 4 * hh) = xk;
                *reinterpret_cast<f32x4 *>(a.hpart_v + o + 32 * dt + 8 * g + 4 * hh) = xv;
            }
        return;
    }
    if (SUMS) return;
    if (MODE == 1) {
        // partial sums of this query range: [split][pooled key][head][channel] fp32
        const int64_t o = (((int64_t)split * a.nbp + key) * a.h_kv + head) * D;
#pragma unroll
        for (int dt = 0; dt < ND; ++dt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4 xk, xv;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    xk[j] = acck[dt][4 * g + j];
                    xv[j] = accv[dt][4 * g + j];
                }
                *reinterpret_cast<f32x4 *>(a.part_k + o + 32 * dt + 8 * g + 4 * hh) = xk;
                *reinterpret_cast<f32x4 *>(a.part_v + o + 32 * dt + 8 * g + 4 * hh) = xv;
            }
    } else {
        // add the gradient of the pooled key / value this block went into (its query ranges are added up already),
        // divided by the number of tokens that pair averaged: the block's, or its whole spatial block's
        const int pair = a.blk_grp != nullptr ? a.blk_grp[kb] : kb;
        const float pooled_tokens = a.grp_tok != nullptr ? (float)a.grp_tok[pair] : (float)n_act;
        float xk[ND][16], xv[ND][16];
#pragma unroll
        for (int dt = 0; dt < ND; ++dt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int64_t o = ((int64_t)pair * a.h_kv + head) * D + 32 * dt + 8 * g + 4 * hh;
                const f32x4 pk = *reinterpret_cast<const f32x4 *>(a.part_k + o), pv = *reinterpret_cast<const f32x4 *>(a.part_v + o);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    // the block average was taken over its n_act active tokens; a padding slot gets nothing
                    const float inv_cnt = key_active ? 1.0f / pooled_tokens : 0.f;
                    xk[dt][4 * g + j] = (acck[dt][4 * g + j] + pk[j] * inv_cnt) * a.scale;
                    xv[dt][4 * g + j] = accv[dt][4 * g + j] + pv[j] * inv_cnt;
                }
            }
        __syncthreads();  // the tile buffers become the output staging
        char *stage = lds + wave * 32 * G::OUT_ROW;
        store_rows_transposed<D>(xk, stage, a.dk + (key0 * a.h_kv + head) * D, (int64_t)a.h_kv * D, lane);
        __builtin_amdgcn_s_waitcnt(0xC07F);  // staging reads of dK done before it is overwritten
        store_rows_transposed<D>(xv, stage, a.dv + (key0 * a.h_kv + head) * D, (int64_t)a.h_kv * D, lane);
    }
}

// Pooled keys from which a workgroup of four wavefronts takes 128 of them, two to a SIMD with the values in LDS (d = 128 only, not
// in the joint launch).  Fewer keys leave it short of work, or its second half without keys.  Backward with 64 / with 128
// keys to a workgroup, us, blocks x heads: 64 x 32 597 / 607, 128 x 16 586 / 598, 192 x 8 466 / 477, 257 x 4 401 / 411, 300 x 2 255 / 265, 400 x 1
// 203 / 206, 64 groups of 256 x 8 469 / 481; 448 x 8 1103 / 1100, 512 x 2 339 / 345, 520 x 8 1314 / 1312, 700 x 8 1843 / 1802, 896 x 8
// 2469 / 2391, 1500 x 4 2514 / 2405.
constexpr int kPooledWide = 512;
constexpr int kPooledMany = 2048;  // dQ, see launch_backward_d

// Number of a workgroup among the walks of pooled keys -> group of 32 * WV keys, key/value head, range of query tiles; false: none left.
// Equal shares of all walks for the XCDs, and to each the key groups of one (head, range) beside each other: they read the same
// query tiles, at the same pace, so that its L2 fetches those about once.  (Dealing the key groups of every (head, range) to
// the XCDs leaves some with nothing where there are few: of three groups, five of eight.  Backward, that / this, us, blocks x
// heads: d = 128, 192 x 8 404 / 363, 337 x 8 (2) 974 / 909, 896 x 2 731 / 654, 896 x 8 2549 / 2440, 4096 x 8 22570 / 21930; d = 64, 192 x
// 8 222 / 206, 896 x 8 1287 / 1224.)
template <int WV>
__device__ bool pooled_walk(const BwdArgs &a, int wg, int *group, int *head, int *z) {
    const int n_groups = a.nbp / (32 * WV), n = n_groups * a.h_kv * a.n_split, item = (wg & 7) * ((n + 7) / 8) + (wg >> 3);
    if (item >= n) return false;
    // (divided in vector registers: readfirstlane tells the compiler that the numbers are uniform all the same)
    const int y = __builtin_amdgcn_readfirstlane(item / n_groups);
    *z = __builtin_amdgcn_readfirstlane(y / a.h_kv);
    *head = y - *z * a.h_kv;
    *group = item - y * n_groups;
    return true;
}

template <int D, int MODE, int WV = 2>
__global__ __launch_bounds__(64 * WV, (D == 128 ? WV / 2 : 3)) void bwd_dkv_kernel(BwdArgs a) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    if constexpr (MODE == 0) {
        dkv_walk<D, 0, false, 2, false>(a, lds, blockIdx.x, blockIdx.y, blockIdx.z);
    } else {
        int group, head, z;
        if (!pooled_walk<WV>(a, blockIdx.x, &group, &head, &z)) return;
        dkv_walk<D, 1, false, WV, WV == 4>(a, lds, group, head, z);
    }
}

// The three kinds of walks of a small problem in one launch: none of them fills the chip, and none needs another's results (the
// gradients of the pooled pairs meet those of the token keys in sum_walks<D, true>).  Workgroups: token keys first, dQ, pooled keys; each
// kind's number is a multiple of 8 (XCDs).
template <int D, bool WIDE>
__global__ __launch_bounds__(128, (D == 128 ? 1 : 3)) void bwd_walks_small(BwdArgs a, int n_tasks, int n_dkv, int n_dq_x, int n_dq) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    // (divided in vector registers: readfirstlane tells the compiler that the numbers are uniform all the same)
    auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    int wg = blockIdx.x;
    if (wg < n_dkv) {
        const int y = uniform(wg / n_tasks), z = uniform(y / a.h_kv);
        if (z >= a.hsplit) return;  // (the number was rounded up to eight)
        dkv_walk<D, 0, true, 2, false>(a, lds, wg - y * n_tasks, y - z * a.h_kv, z);
        return;
    }
    wg -= n_dkv;
    if (wg < n_dq) {
        const int y = uniform(wg / n_dq_x);
        dq_walk<D, WIDE, ALONE>(a, lds, wg - y * n_dq_x, y);
        return;
    }
    wg -= n_dq;
    int group, head, z;
    if (pooled_walk<2>(a, wg, &group, &head, &z)) dkv_walk<D, 1, false, 2, false>(a, lds, group, head, z);
}

// The rows of the key blocks whose walks were dealt out: the sums of the parts of each head range, added in order, then
// what the token-key kernel does at the end of a walk of its own (pooled gradient, scale, rounding).  One workgroup per
// (block, key/value head, 256 groups of four channels of a token), one such group per thread, four sums of each of dk and dv in flight:
// bound by memory at size (196 K tokens, 2 key/value heads of 32, two head ranges: 201 MB of sums and those of cut walks in 71 us), by
// its chain of loads below.
// SMALL (behind bwd_walks_small): the rows of all blocks; the pooled gradient is still in n_split parts, which a workgroup adds up first,
// 256 / (D / 2) threads to a group of four channels.
template <int D, bool SMALL>
__global__ __launch_bounds__(256) void sum_walks(BwdArgs a, int n_split) {
    const int head = blockIdx.y;
    int kb = blockIdx.x;
    if (!SMALL && a.hsplit == 1) {  // only the blocks whose walk was cut
        if (kb >= a.task_n[1]) return;
        kb = a.split_list[kb];
    }
    const int np = max(1, (a.walk[kb] + a.part_steps - 1) / a.part_steps), n_sums = a.hsplit * np, slot0 = a.slot0[kb];
    const int n_act = a.count != nullptr ? a.count[kb] : 64;
    const int pair = a.blk_grp != nullptr ? a.blk_grp[kb] : kb;
    const float pooled_tokens = a.grp_tok != nullptr ? (float)a.grp_tok[pair] : (float)n_act;
    const int64_t range = (int64_t)a.max_slots * 64 * a.h_kv * D, slot = (int64_t)64 * a.h_kv * D;  // in floats
    const int e = blockIdx.z * 256 + threadIdx.x;
    const int row = e / (D / 4), c = 4 * (e % (D / 4));
    const int64_t in_slot = ((int64_t)row * a.h_kv + head) * D + c;
    const int64_t o_pair = ((int64_t)pair * a.h_kv + head) * D + c;
    f32x4 pk, pv;
    if constexpr (SMALL) {
        constexpr int COLS = D / 2, GROUPS = 256 / COLS;  // columns of four channels: of dk, then of dv
        __shared__ f32x4 parts[GROUPS][COLS];
        const int col = threadIdx.x % COLS, g = threadIdx.x / COLS;
        const float *from = (col < D / 4 ? a.part_k : a.part_v) + ((int64_t)pair * a.h_kv + head) * D + 4 * (col % (D / 4));
        const int64_t per_split = (int64_t)a.nbp * a.h_kv * D;
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int sp = g; sp < n_split; sp += GROUPS) sum += *reinterpret_cast<const f32x4 *>(from + sp * per_split);
        parts[g][col] = sum;
        __syncthreads();
        pk = parts[0][c / 4];
        pv = parts[0][D / 4 + c / 4];
#pragma unroll 4
        for (int j = 1; j < GROUPS; ++j) {
            pk += parts[j][c / 4];
            pv += parts[j][D / 4 + c / 4];
        }
    } else {
        pk = *reinterpret_cast<const f32x4 *>(a.part_k + o_pair);
        pv = *reinterpret_cast<const f32x4 *>(a.part_v + o_pair);
    }
    f32x4 sk = {0.f, 0.f, 0.f, 0.f}, sv = {0.f, 0.f, 0.f, 0.f};
    for (int i = 0; i < n_sums; i += 4) {
        f32x4 xk[4], xv[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int at = min(i + j, n_sums - 1), z = at / np;  // (past the end: the last one, not added)
            const int64_t o = z * range + (slot0 + at - z * np) * slot + in_slot;
            xk[j] = *reinterpret_cast<const f32x4 *>(a.hpart_k + o);
            xv[j] = *reinterpret_cast<const f32x4 *>(a.hpart_v + o);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (i + j < n_sums) {
                sk += xk[j];
                sv += xv[j];
            }
    }
    const float inv_cnt = row < n_act ? 1.0f / pooled_tokens : 0.f;  // a padding slot gets nothing
    uint2 wk, wv;
    wk.x = pack_bf16((sk[0] + pk[0] * inv_cnt) * a.scale, (sk[1] + pk[1] * inv_cnt) * a.scale);
    wk.y = pack_bf16((sk[2] + pk[2] * inv_cnt) * a.scale, (sk[3] + pk[3] * inv_cnt) * a.scale);
    wv.x = pack_bf16(sv[0] + pv[0] * inv_cnt, sv[1] + pv[1] * inv_cnt);
    wv.y = pack_bf16(sv[2] + pv[2] * inv_cnt, sv[3] + pv[3] * inv_cnt);
    const int64_t dst = (((int64_t)kb * 64 + row) * a.h_kv + head) * D + c;
    *reinterpret_cast<uint2 *>(a.dk + dst) = wk;
    *reinterpret_cast<uint2 *>(a.dv + dst) = wv;
}

// Whether bwd_prepare does what else takes five launches: few enough table entries to be counted by every block's workgroup, and a
// grid that one direction holds.  Backward, five launches / bwd_prepare (us; blocks x heads, entries): 96 x 4, 768 118 / 99; 192 x 8 of
// 128, 1536 430 / 412; 337 x 8 (2), 6740 532 / 511; 544 x 32 (2), 16320 3972 / 3935; 896 x 2, 14336 431 / 423; 896 x 8 1327 / 1319; 1020 x 4,
// 16320 805 / 805; 2024 x 1, 16192 550 / 564.
bool small_table(const Shape &s) {
    return s.topk > 0 && s.nb <= kTableBlocks && (int64_t)s.nb * s.topk <= kTableEntries && (int64_t)s.nb * s.h <= 1 << 20;
}

// Whether a backward goes through the launches of small problems.  They are three, bwd_prepare and the general kernels six (without
// bwd_prepare ten), and the ends of three kernels become one; they cost fp32 sums of every walk and, at d = 128, dQ walks with one
// wavefront per SIMD.  Backward, general / small (us), blocks x heads (on key/value heads):
//   d = 32   96 x 4 74 / 51, 192 x 8 147 / 116, 548 x 4 273 / 235, 337 x 8 (2) 287 / 241, 640 x 2 193 / 156, 160 x 32 (16) 515 / 478;
//            700 x 8 591 / 583, 512 x 16 774 / 776
//   d = 64   96 x 4 92 / 62, 192 x 8 214 / 186, 548 x 4 416 / 384, 337 x 8 (2) 432 / 390, 160 x 32 (16) 806 / 769; 700 x 2 290 / 278,
//            384 x 12 779 / 741, 512 x 16 1284 / 1315
//   d = 128  96 x 4 146 / 103, 132 x 1 96 / 62, 116 x 16 (1) 434 / 390, 256 x 4 377 / 387, 192 x 6 291 / 305; 192 x 8 374 / 404, 512 x 2 361 /
//            394, 160 x 32 (2) 1500 / 1567
// Over 700 drawn problems that bwd_prepare takes, the rule costs 0.1 % against the better choice for each with grouped heads at d <= 64,
// 0.4 and 1.6 % with plain ones (d = 64 and 32: the joint launch still wins a little beyond its limits), 1 % at d = 128.
bool small_backward(const Shape &s) {
    if (!small_table(s) || s.nb > 640 || (int64_t)s.nb * s.h > 1 << 16) return false;
    return s.d == 128 ? s.nb <= 256 && s.nb * s.h <= 1280 : s.nb * s.h_kv <= 3072;
}

struct WsLayout {
    size_t img_q, img_do[3], img_k, img_v, img_kc, img_vc, aux, part_k, part_v, rev_cnt, rev_ptr, rev_cur, rev_idx, total;
    int n_split, nbp, wg_keys, tiles_per_split, hsplit, hpw, part_steps, max_tasks, max_slots, max_split;
    bool small;  // bwd_walks_small
    size_t hpart_k, hpart_v, order, order_part, slot0, split_list, task_n, walk, gtab;
};

// Blocks of a spatial block, about: the mean, of all or of those that are not an image tile each.
double blocks_of_group(const Shape &s) {
    const double all = (double)s.nb / s.ng;
    return s.ng > s.n_tiles ? std::max(all, (double)s.nb_obj / (s.ng - s.n_tiles)) : all;
}

WsLayout ws_layout(const Shape &s) {
    WsLayout w;
    const size_t img = (size_t)s.d * 64;  // bytes of one (tile, head) image: row-order fragments only
    const size_t nt = (size_t)s.nb * 2, ntc = (size_t)(s.nbc + 31) / 32;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t at = off;
        off += align_up(bytes > 0 ? bytes : 1, 256);
        return at;
    };
    w.img_q = take(nt * s.h * img);
    w.img_do[0] = take(nt * s.h * img);
    if (s.gate_channels) {
        // one image of gate o dout per branch
        w.img_do[1] = take(nt * s.h * img);
        w.img_do[2] = take(nt * s.h * img);
    } else {
        w.img_do[1] = w.img_do[2] = w.img_do[0];
    }
    w.img_k = take(nt * s.h_kv * img);
    w.img_v = take(nt * s.h_kv * img);
    w.img_kc = take(ntc * s.h_kv * img);
    w.img_vc = take(ntc * s.h_kv * img);
    w.aux = take((size_t)3 * nt * s.h * 64 * 4);
    // pooled keys: enough query ranges to fill the chip
    w.small = small_backward(s);
    const int wg_keys = w.wg_keys = s.d == 128 && !w.small && s.nbc >= kPooledWide ? 128 : 64;  // pooled keys of a workgroup
    w.nbp = (s.nbc + wg_keys - 1) / wg_keys * wg_keys;
    const int wgs = (w.nbp / wg_keys) * s.h_kv;
    // The query tiles are cut into n ranges, one workgroup per (wg_keys pooled keys, key/value head, range), all equally
    // long.  The chip runs `slots` of them at a time (256 CUs x the workgroups per CU that the kernel's registers
    // allow), so the kernel takes ceil(workgroups / slots) rounds of (tiles per range) x (query heads per key/value
    // head) steps; every range also costs its partial sums, written here and read back by the token-key kernel.
    // n minimises that: e.g. at 848 workgroups per range and 512 slots, one range runs 2 rounds where 1.66 would
    // do, three ranges run 5 rounds of a third of the length (17 % less).  At most 96: 297 blocks x 8 heads (1) of 64, at most 64 / 96 / 128
    // 370 / 356 / 352 us, 499 x 3 (1) of 128 610 / 595 / 592, 1740 x 1 of 32 214 / 208 / 208, but 337 x 8 (2) of 64 354 / 353 / 358.
    {
        const int slots = 256 * (s.d == 128 ? 2 : s.d == 64 ? 6 : 8);  // workgroups the chip holds
        const int grp_q = s.h / s.h_kv;
        const double range_bytes = (double)w.nbp * s.h_kv * s.d * 4 * 2 * 2;
        const double step_seconds = wg_keys == 128 ? 1.9e-6 : 1.1e-6 * s.d / 128, range_steps = range_bytes / 4e12 / step_seconds;
        double best = 0;
        int best_n = 1;
        for (int n = 1; n <= 96; ++n) {
            const int64_t tiles = ((int64_t)nt + n - 1) / n;
            if (tiles <= 0) break;
            const int64_t n_eff = ((int64_t)nt + tiles - 1) / tiles;
            const int64_t rounds = ((int64_t)wgs * n_eff + slots - 1) / slots;
            const double cost = (double)rounds * tiles * grp_q + range_steps * n_eff;
            if (n == 1 || cost < best) {
                best = cost;
                best_n = n;
            }
        }
        const int n_split = best_n;
        w.tiles_per_split = (int)((nt + n_split - 1) / n_split);
        w.n_split = (int)((nt + w.tiles_per_split - 1) / (w.tiles_per_split > 0 ? w.tiles_per_split : 1));
        if (w.n_split < 1) w.n_split = 1;
    }
    w.part_k = take((size_t)w.n_split * w.nbp * s.h_kv * s.d * 4);
    w.part_v = take((size_t)w.n_split * w.nbp * s.h_kv * s.d * 4);
    // Token keys.  No single walk may set the kernel's time: geometric routing makes some blocks popular, and a small problem has too
    // few walks to fill the chip, which then waits for the latency of their steps (1 to 2 us each).  So long walks are cut into
    // parts, longest first, and the heads of a group may be dealt to several workgroups.  Both cost a workgroup's start and its sums
    // (32 KB at d = 64, written and read).  A "share" is the steps that all walks have for each workgroup the chip holds.
    //
    // Launches of their own: a part is half a share, a quarter with grouped-query heads, where a cut is what spreads the heads of a group
    // too, but at least 64 steps (96 with grouped heads; at d = 128 16 and 64), fewer where there is little to do.
    // The heads of a group used to be dealt to up to 8 workgroups; the sums that costs took more than it gave once walks were cut,
    // except for large groups, where two workgroups' images of q and dout are nearer to each other in memory: those are dealt to
    // two (as long as the sums stay within 2 GiB of workspace).  8 workgroups and half a share / this, us: 2069 blocks, 6 heads on 2
    // of 128 9285 / 8120, 2553 x 6 (1) of 32 3190 / 3060, 3307 x 4 (2) of 128 8390 / 7790; 3072 x 32 (2) of 32 32024 / 31900, undealt
    // 32900; spatial blocks with their own window, 115 x 16 (4) of 128 381 / 364 (with parts of at least 16 steps 430).
    //
    // The joint launch, plain heads: at least half a share as well, and 16 to 64 steps, the fewer the less there is to do (backward, parts
    // of at least 16 steps / this, us: 174 x 2 of 64 195 / 149, 178 x 4 of 32 189 / 150, 99 x 1 of 128 120 / 100, 202 x 1 of 64 85 / 75).
    // The joint launch, grouped heads: a part of L steps costs its chain, and a workgroup's place share / L starts and sums, which is
    // least at L in proportion to the root of the share: at 8 to 10 roots, over 360 problems with parts of 8 to 256 steps.  A part
    // cannot be shorter than an entry's two tiles of every head of its workgroup, nor, where the window is a spatial block, than
    // that block's tiles, which go uncut (its size is known on the device only: half as much again as the mean); so heads are
    // dealt until that fits, and until the walks take an eighth of the places.  Where whole walks take a third of the places, cuts are for
    // popular blocks only: up to 96 steps, and windows deal nothing (337 x 8 (2) of 64 below: 353 us without that).  Backward, 8
    // workgroups and at least 16 steps / undealt and up to 96 / this, us: spatial blocks with their own window 13 x 32 (2) of 32 48 / 167 /
    // 46, 85 x 16 (2) of 64 139 / 257 / 133, 90 x 8 (1) of 64 131 / 219 / 116, 337 x 8 (2) of 64 375 / 346 / 346; single blocks 18 x 32 (4)
    // of 64 60 / 104 / 58, 18 x 12 (3) of 128 59 / 108 / 56, 7 x 12 (1) of 128 54 / 72 / 44, 34 x 6 (2) of 64 53 / 93 / 54; 96 x 3 (1) of 64
    // 126 / 96 / 109 and 65 x 4 (1) of 128 91 / 78 / 94 are what this loses.  Of 800 drawn problems of the joint launch, plain heads among
    // them, the second takes more than 5 % longer than the first in 122 (20 % in 65), this in 25 (20 % in one), tables of few entries in long
    // rows above all: the host knows the length of the rows only.  On average this is 4.5 % faster than the first, 4 % than the second.
    // (Walks cut only where they are a quarter or a half longer than a part: slower.)
    {
        const int slots = 256 * (s.d == 128 ? 2 : s.d == 64 ? 6 : 8);  // workgroups the chip holds
        const int grp = s.h / s.h_kv;
        // bounds a block's counted window, an even number of tiles: no window leaves the sequence, however large the
        // caller's W (an unlimited one is 2^31 - 2: 64 bits)
        const int64_t reach = (((64 + (int64_t)s.window) / 32 + 2) + 1) & ~(int64_t)1;
        const int64_t win = s.group_window ? 0 : reach < (int64_t)nt ? reach : (int64_t)nt;
        const int64_t steps = (int64_t)s.nb * (2 * s.topk + win);  // at most, whatever the table holds
        const int64_t half_share = steps * s.h / slots / 2;
        // a row holds no more blocks than there are, unless it repeats some: the estimate leaves that out, the bounds below do not
        const double share = (double)s.nb * (2 * std::min(s.topk, s.nb) + win) * s.h / slots;
        double part;  // steps, of all heads that a workgroup has
        int ranges;
        if (w.small && grp > 1) {
            const bool many = 3 * s.nb * s.h_kv >= slots;
            part = std::max({16.0, (s.d == 32 ? 10 : 8) * std::sqrt(share), half_share / 2.0, many ? std::min(96.0, 1.5 * share) : 0.0});
            const double uncut = s.group_window && !many ? 6 * blocks_of_group(s) : 4;
            ranges = (int)std::min<double>(std::min(grp, 8), std::ceil(std::max(uncut * grp / part, slots / 8.0 / (s.nb * s.h_kv))));
        } else if (w.small) {
            part = std::max({16.0, std::min(64.0, (s.d == 128 ? 1.5 : 3) * share), (double)half_share});
            ranges = 1;
        } else {
            part = std::max(16.0, std::min<double>(s.d < 128 ? (grp > 1 ? 96 : 64) : grp > 1 ? 64 : 16, (s.d == 128 ? 4 : 8) * half_share));
            ranges = grp >= 8 ? 2 : 1;
        }
        for (; ranges >= 1; --ranges) {
            w.hpw = (grp + ranges - 1) / ranges;
            w.hsplit = (grp + w.hpw - 1) / w.hpw;
            int64_t len;
            if (w.small)
                len = std::max<int64_t>(2, 2 * (int64_t)std::floor(part / w.hpw / 2 + 0.5));
            else
                len = std::max<int64_t>(steps * s.h_kv * w.hsplit / slots / (grp > 1 ? 4 : 2), (int64_t)std::ceil(part / w.hpw));
            len = (len + 1) & ~(int64_t)1;
            if (len > 0x3ffffffe) len = 0x3ffffffe;
            w.part_steps = (int)len;
            // bounds whatever the table holds: parts beyond a block's first number at most steps / len in all, and
            // so do the blocks that are cut (steps / len is below 8 slots, or 2^20 where len is at its largest: no
            // sum below leaves 32 bits)
            const int64_t more = steps / len;
            w.max_split = (int)(more < s.nb ? more : s.nb);
            w.max_tasks = (int)(s.nb + more);
            w.max_slots = w.hsplit > 1 || w.small ? w.max_tasks : (int)(w.max_split + more);
            if ((double)w.hsplit * w.max_slots * 64 * s.h_kv * s.d * 8 <= 2147483648.0) break;
        }
    }
    const size_t sums = (size_t)w.hsplit * w.max_slots * 64 * s.h_kv * s.d * 4;
    w.hpart_k = take(sums);
    w.hpart_v = take(sums);
    w.order = take((size_t)w.max_tasks * 4);
    w.order_part = take((size_t)w.max_tasks * 4);
    w.slot0 = take((size_t)s.nb * 4);
    w.split_list = take((size_t)w.max_split * 4);
    w.task_n = take(8);
    w.walk = take((size_t)s.nb * 4);
    w.rev_cnt = take((size_t)s.nb * 4);
    w.rev_ptr = take((size_t)(s.nb + 1) * 4);
    w.rev_cur = take((size_t)s.nb * 4);
    w.rev_idx = take((size_t)s.nb * (s.topk > 0 ? s.topk : 1) * 4);
    w.gtab = take(group_tables_bytes(s));
    w.total = off;
    return w;
}

template <int D>
lsrm_status launch_backward_d(const Shape &s, BwdArgs a, const GroupTableArgs &tables, const WsLayout &w, char *ws, hipStream_t st,
                              hipEvent_t ev_start, hipEvent_t ev_stop) {
    constexpr int LDS_TOKENS = DKV_LDS<D, 2, false>;
    const int64_t n_prep = (int64_t)a.nt * ((s.h + PrepGeo<D>::HB - 1) / PrepGeo<D>::HB);
    const int64_t n_token_wg = (int64_t)s.nb * (s.h + 2 * s.h_kv), n_wg = n_token_wg + (int64_t)((s.nbc + 63) / 64) * 2 * s.h_kv;
    const bool table = small_table(s);
    if (ev_start != nullptr) LSRM_HIP_CHECK(hipEventRecord(ev_start, st));
    if (table) {
        const int n_tables = (tables.n + PrepGeo<D>::THREADS - 1) / PrepGeo<D>::THREADS;
        hipLaunchKernelGGL(bwd_prepare<D>, dim3((unsigned)(n_prep + n_wg + s.nb + n_tables)), dim3(PrepGeo<D>::THREADS), 0, st, a, n_prep,
                           n_token_wg, n_wg, w.small ? 1 : 0, tables);
        LSRM_HIP_CHECK(hipGetLastError());
    }
    if (w.small) {
        auto eights = [](int64_t x) { return (x + 7) / 8 * 8; };
        const int n_dq_x = (int)eights(s.nb);
        const int64_t n_dkv = eights((int64_t)w.max_tasks * s.h_kv * a.hsplit), n_dq = (int64_t)n_dq_x * s.h;
        const int64_t n_walks = n_dkv + n_dq + eights((int64_t)w.nbp / 64 * s.h_kv * w.n_split);
        constexpr int LDS_WALK = DKV_LDS<D, 2, false>, LDS = LDS_WALK > DQ_LDS<D> ? LDS_WALK : DQ_LDS<D>;
        auto walks = s.topk > 64 ? &bwd_walks_small<D, true> : &bwd_walks_small<D, false>;
        // (set on every call: cheap, and right whichever device is current and whichever thread calls)
        LSRM_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(walks), hipFuncAttributeMaxDynamicSharedMemorySize, LDS));
        hipLaunchKernelGGL(walks, dim3((unsigned)n_walks), dim3(128), LDS, st, a, w.max_tasks, (int)n_dkv, n_dq_x, (int)n_dq);
        LSRM_HIP_CHECK(hipGetLastError());
        hipLaunchKernelGGL((sum_walks<D, true>), dim3(s.nb, s.h_kv, D / 16), dim3(256), 0, st, a, w.n_split);
        LSRM_HIP_CHECK(hipGetLastError());
        if (ev_stop != nullptr) LSRM_HIP_CHECK(hipEventRecord(ev_stop, st));
        return LSRM_OK;
    }
    LSRM_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(&bwd_dkv_kernel<D, 0>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, LDS_TOKENS));
    if (!table) {
        hipLaunchKernelGGL(bwd_prep<D>, dim3((unsigned)n_prep), dim3(PrepGeo<D>::THREADS), 0, st, a, tables);
        LSRM_HIP_CHECK(hipGetLastError());
        const int64_t n_pack = n_wg + ((int64_t)s.nb * s.topk + 255) / 256;
        const dim3 pack_grid((unsigned)(n_pack < kPackMaxGrid ? n_pack : kPackMaxGrid),
                             (unsigned)((n_pack + kPackMaxGrid - 1) / kPackMaxGrid));
        hipLaunchKernelGGL(pack_rows<D>, pack_grid, dim3(256), 0, st, a, n_token_wg, n_wg);
        LSRM_HIP_CHECK(hipGetLastError());
        // reverse routing lists
        hipLaunchKernelGGL(rev_scan_order, dim3(1), dim3(1024), 0, st, a);
        LSRM_HIP_CHECK(hipGetLastError());
        if (s.topk > 0) {
            hipLaunchKernelGGL(rev_fill, dim3((s.nb * s.topk + 255) / 256), dim3(256), 0, st, a);
            LSRM_HIP_CHECK(hipGetLastError());
            const size_t bitmap = (size_t)((s.nb + 31) / 32) * 4;
            if (bitmap <= 48 * 1024)
                hipLaunchKernelGGL(rev_sort, dim3(s.nb), dim3(64), bitmap, st, a);
            else
                hipLaunchKernelGGL(rev_sort_serial, dim3((s.nb + 63) / 64), dim3(64), 0, st, a);
            LSRM_HIP_CHECK(hipGetLastError());
        }
    }
    // Two heads to a workgroup wherever heads that share keys and values come in pairs.  Whole backward, one head / two, us: 1536 blocks, rows
    // of 32, 16 heads on 2 of 64 6237 / 6070, 8 on 2 of 128 6175 / 5989; rows of 80, 8 on 4 of 64 5415 / 5096; 900 blocks, 4 on 2 of 64 696 / 684.
    // From 641 blocks on (257 at d = 128) 1 to 3 % in each of 126 problems but two, 257 and 300 blocks x 2 (1) of 128, 1.5 % the other way.
    const bool heads = a.group % 2 == 0;
    // Two query blocks to a workgroup for other heads where the pooled keys are many, at d >= 64.  One block / two, us: d = 128, 6688 blocks x
    // 16 heads 128.9 / 127.9 ms, 5121 x 4 16371 / 16177, 2176 x 8 9258 / 9218, 1536 x 8 6446 / 6445, 641 x 8 2300 / 2330, 257 x 8 870 / 902;
    // d = 64, 4864 x 2 3693 / 3630, 2816 x 4 3727 / 3693, 2048 x 8 3959 / 3923, 1536 x 8 3192 / 3184, 897 x 8 1670 / 1680.
    // It is little: over 46 problems of 2048 to 6700 blocks each (rows of 16 and 80; 1, 3 and 8 heads, and 3 on 1) one block takes, of
    // two's time, at d = 128 0.8 % more (-1.6 to 2.6, one of them below -0.3: 3128 x 1, rows of 80), at d = 64 0.6 % (-0.7 to 3.3, five
    // below -0.3), at d = 32 0.3 % (-1.0 to 2.6, ten below -0.3).
    const bool blocks = D >= 64 && !heads && s.nbc >= kPooledMany;
    auto choose = [&](auto wide) {
        constexpr bool WIDE = decltype(wide)::value;
        if (heads) return &bwd_dq_kernel<D, WIDE, HEADS>;
        if constexpr (D >= 64)
            if (blocks) return &bwd_dq_kernel<D, WIDE, BLOCKS>;
        return &bwd_dq_kernel<D, WIDE, ALONE>;
    };
    const auto dq = s.topk > 64 ? choose(std::true_type{}) : choose(std::false_type{});
    const int n_units = blocks ? (s.nb + 1) / 2 : s.nb;
    hipLaunchKernelGGL(dq, dim3((n_units + 7) / 8 * 8, heads ? s.h / 2 : s.h), dim3(heads || blocks ? 256 : 128), 0, st, a);
    LSRM_HIP_CHECK(hipGetLastError());
    auto pooled = [&](auto *kernel, int lds) -> lsrm_status {
        LSRM_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        hipLaunchKernelGGL(kernel, dim3((w.nbp / w.wg_keys * s.h_kv * w.n_split + 7) / 8 * 8), dim3(2 * w.wg_keys), lds, st, a);
        LSRM_HIP_CHECK(hipGetLastError());
        return LSRM_OK;
    };
    lsrm_status rc;
    if constexpr (D == 128)
        rc = w.wg_keys == 128 ? pooled(&bwd_dkv_kernel<D, 1, 4>, DKV_LDS<D, 4, true>) : pooled(&bwd_dkv_kernel<D, 1>, LDS_TOKENS);
    else
        rc = pooled(&bwd_dkv_kernel<D, 1>, LDS_TOKENS);
    if (rc != LSRM_OK) return rc;
    if (w.n_split > 1) {
        const int64_t per_split = (int64_t)w.nbp * s.h_kv * D;
        hipLaunchKernelGGL(sum_parts, dim3((unsigned)((per_split / 4 + 255) / 256), 2), dim3(256), 0, st, a.part_k, a.part_v,
                           w.n_split, per_split);
        LSRM_HIP_CHECK(hipGetLastError());
    }
    hipLaunchKernelGGL((bwd_dkv_kernel<D, 0>), dim3(w.max_tasks, s.h_kv, a.hsplit), dim3(128), LDS_TOKENS, st, a);
    LSRM_HIP_CHECK(hipGetLastError());
    // add up the sums of walks that were dealt out, in order, and finish their rows
    const int n_sum_blocks = a.hsplit > 1 ? s.nb : w.max_split;
    if (n_sum_blocks > 0) {
        hipLaunchKernelGGL((sum_walks<D, false>), dim3(n_sum_blocks, s.h_kv, D / 16), dim3(256), 0, st, a, w.n_split);
        LSRM_HIP_CHECK(hipGetLastError());
    }
    if (ev_stop != nullptr) LSRM_HIP_CHECK(hipEventRecord(ev_stop, st));
    return LSRM_OK;
}

}  // namespace

size_t backward_ws_bytes(const Shape &s) { return ws_layout(s).total; }

lsrm_status launch_backward(const Shape &s, const int32_t *seg_host, int n_seg, const uint16_t *d_q,
                            const uint16_t *d_k, const uint16_t *d_v, const uint16_t *d_kc, const uint16_t *d_vc,
                            const int32_t *d_idx, const float *d_gates, const float *d_lse,
                            const uint16_t *d_out_branch, const uint16_t *d_dout, uint16_t *d_dq, uint16_t *d_dk,
                            uint16_t *d_dv, void *d_ws, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
    if (s.nb == 0) return LSRM_OK;
    if (n_seg > kMaxSeg) return LSRM_ERR_UNSUPPORTED;
    const WsLayout w = ws_layout(s);
    char *ws = reinterpret_cast<char *>(d_ws);
    BwdArgs a{};
    a.q = d_q;
    a.k = d_k;
    a.v = d_v;
    a.kc = d_kc;
    a.vc = d_vc;
    a.dout = d_dout;
    a.out_branch = d_out_branch;
    a.idx = d_idx;
    a.gates = d_gates;
    a.lse = d_lse;
    a.img_q = ws + w.img_q;
    for (int b = 0; b < 3; ++b) a.img_do[b] = ws + w.img_do[b];
    a.img_k = ws + w.img_k;
    a.img_v = ws + w.img_v;
    a.img_kc = ws + w.img_kc;
    a.img_vc = ws + w.img_vc;
    a.aux = reinterpret_cast<float *>(ws + w.aux);
    a.part_k = reinterpret_cast<float *>(ws + w.part_k);
    a.part_v = reinterpret_cast<float *>(ws + w.part_v);
    a.rev_cnt = reinterpret_cast<int32_t *>(ws + w.rev_cnt);
    a.rev_ptr = reinterpret_cast<int32_t *>(ws + w.rev_ptr);
    a.rev_cur = reinterpret_cast<int32_t *>(ws + w.rev_cur);
    a.rev_idx = reinterpret_cast<int32_t *>(ws + w.rev_idx);
    a.dq = d_dq;
    a.dk = d_dk;
    a.dv = d_dv;
    for (int i = 0; i <= n_seg; ++i) a.seg[i] = seg_host[i];
    a.n = s.n;
    a.nb = s.nb;
    a.nbc = s.nbc;
    a.blk_grp = a.blk_seg = a.grp_tok = nullptr;
    GroupTableArgs tables{};
    if (s.ng > 0) {
        tables = group_table_args(s, reinterpret_cast<int32_t *>(ws + w.gtab));  // (the first launch makes them)
        const GroupTables gt = group_tables_in(s, tables.tab);
        a.blk_grp = gt.blk_grp;
        a.grp_tok = gt.grp_tok;
        if (s.group_window) a.blk_seg = gt.blk_seg;
    }
    a.h = s.h;
    a.h_kv = s.h_kv;
    a.group = s.h / s.h_kv;
    a.gate_channels = s.gate_channels;
    a.count = s.count;
    a.topk = s.topk;
    a.window = s.window;
    a.own_block = s.own_block;
    a.n_seg = n_seg;
    a.nt = s.nb * 2;
    a.hsplit = w.hsplit;
    a.hpw = w.hpw;
    a.hpart_k = reinterpret_cast<float *>(ws + w.hpart_k);
    a.hpart_v = reinterpret_cast<float *>(ws + w.hpart_v);
    a.part_steps = w.part_steps;
    a.cut_window = s.group_window ? 0 : 1;
    a.walk = reinterpret_cast<int32_t *>(ws + w.walk);
    a.max_slots = w.max_slots;
    a.order = reinterpret_cast<int32_t *>(ws + w.order);
    a.order_part = reinterpret_cast<int32_t *>(ws + w.order_part);
    a.slot0 = reinterpret_cast<int32_t *>(ws + w.slot0);
    a.split_list = reinterpret_cast<int32_t *>(ws + w.split_list);
    a.task_n = reinterpret_cast<int32_t *>(ws + w.task_n);
    a.nbp = w.nbp;
    a.tiles_per_split = w.tiles_per_split;
    a.n_split = w.n_split;
    a.scale = s.scale;
    a.sl2 = s.scale * kLog2e;
    if (s.d == 32) return launch_backward_d<32>(s, a, tables, w, ws, st, ev_start, ev_stop);
    if (s.d == 64) return launch_backward_d<64>(s, a, tables, w, ws, st, ev_start, ev_stop);
    return launch_backward_d<128>(s, a, tables, w, ws, st, ev_start, ev_stop);
}

}  // namespace lsrm
