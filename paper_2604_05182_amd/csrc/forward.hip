// NSA forward on gfx950 (App. A, Eq. nsa_1): compressed, selected and window attention,
// each its own softmax, combined by the gated sum, in one kernel.
//
// Work decomposition
//   One workgroup owns NP = 2 consecutive query blocks of one head (or, where query heads share key/value
//   heads in pairs, one query block of two such heads) and carries them through all three branches.  A
//   wavefront holds 32 query rows, two wavefronts a query block.  Each of the four wavefronts of a
//   workgroup sits on its own SIMD, and as many workgroups share a CU as the registers of a wavefront
//   allow: two at d = 128, three at d = 64, four at d = 32 (the LDS of a workgroup is sized for that).
//   They meet no common barrier, so one's start, epilogues, window edges and waits are filled by the
//   others.  In the compressed branch every K/V tile is copied to LDS once and used by both query blocks;
//   in the selected and the window branch each query block streams its own tiles (two heads share those
//   too).  Workgroups are numbered so that each of the 8 XCDs walks a contiguous range of (head, query
//   block) units: the L2 of an XCD then holds one head's pooled keys/values and the neighbouring windows /
//   routed blocks.  With grouped-query heads the query heads that share a key/value head are
//   consecutive, hence run back to back on the same tile images.
//
// Per 32-key step, per wavefront
//   S^T = K Q^T        v_mfma_f32_32x32x16_bf16, A = 32 keys x 16 channels, B = Q^T.
//                      With S transposed, each lane owns one query column, so the row
//                      max / row sum of the softmax are in-lane reductions plus one
//                      exchange between the two lane halves (v_permlane32_swap).
//   P^T -> bf16        the accumulator layout of S^T is already the B-operand layout of
//                      the next contraction once the key rows of the A operand are
//                      loaded in a fixed permutation (bits 2 and 3 of the row swapped),
//                      so P never leaves registers.
//   O^T += V^T P^T     A = 32 channels x 16 keys from a pre-transposed copy of V.
//   A wavefront issues in order and the matrix pipe takes one MFMA at a time, so MFMA and
//   VALU work only overlap if they alternate in program order.  All phases are
//   therefore software pipelined by hand over three tiles: the QK^T MFMAs of tile t+1 and
//   the PV MFMAs of tile t-1 are issued alternately, each followed by its share of the
//   exponentials of tile t (scheduling barriers keep the compiler from regrouping them).
//
// Data movement
//   K and V are repacked once per call into tile images: per (head, 32-key tile) the exact
//   bytes of an LDS slot, K fragments then V^T fragments in MFMA operand order (see
//   read_k), head-major so that one head's keys and values are one contiguous range.
//   Tiles are copied global -> LDS with global_load_lds_dwordx4 (no VGPR staging), 1 KB
//   contiguous on both sides per instruction, the copy instructions of a tile split over
//   the wavefronts that share it, s_waitcnt vmcnt placed by hand, and read back as
//   conflict-free ds_read_b128 MFMA fragments.
//   The gated sum of the branches is carried between branches in registers and LDS (fp32) at d <= 64 and, at
//   d = 128, where they do not suffice, in a bf16 scratch tile in MFMA-fragment order (fully coalesced); the
//   final tile goes through LDS so that the bf16 output rows are written as whole 16-byte chunks.
#include "lsrm_internal.h"

#include <algorithm>
#include <type_traits>

namespace lsrm {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxSeg = 63;
constexpr float kMinusHuge = -1.0e30f;  // initial running maximum: finite, so no inf - inf

struct FwdArgs {
    const uint16_t *q;
    const char *kv, *kvc;  // packed tile images of (k, v) and of the pooled (kc, vc)
    const int32_t *idx;    // routing table [NB, topk]
    const float *gates;
    int32_t seg[kMaxSeg + 1];  // window segment offsets (tokens)
    uint16_t *out;
    float *lse;
    uint16_t *out_branch;
    uint16_t *gsum;  // d = 128: scratch for the running gated sum, bf16 in accumulator-fragment order
    int64_t n;
    int nb, h, topk, window, n_seg;
    int nbc;                 // compressed pairs (spatial blocks): nb unless blocks are grouped
    const int32_t *blk_seg;  // nullable [nb][2]: window segment (first and end token) of every block, instead of `seg`
    int h_kv, group;    // key/value heads; query heads per key/value head (query head i reads head i / group)
    int gate_channels;  // gates are [N, 3, H, d] (one per output channel) instead of [N, H, 3]
    int own_block;      // the window branch sees the query's own block (App. A) instead of a sliding window
    const int32_t *count;  // nullable [NB]: active tokens per block (its first count[b] slots)
    int groups_per_head, groups_per_xcd;  // query-block groups of one head, and the share of one XCD (nsa_forward_teams: of all heads)
    int teams[3];  // nsa_forward_teams: teams of each branch
    const uint16_t *kc, *vc;  // nsa_forward_teams with PAIRS: the pooled pairs
    float scale_log2e, scale;
};

// NP = query blocks per workgroup; a wavefront holds 32 query rows, NW = 2 wavefronts a query block.
// LDS is 2 NP tile slots of 32 keys each (K fragments, then V^T fragments): one ring in the compressed phase, two
// stages of NP slots in the others; behind them the part of the running gated sum that stays on chip.
//
// Why workgroups of two query blocks: they used to be of four (one workgroup of eight wavefronts per CU at d >= 64),
// with a ring of eight tiles that all shared in the compressed and window branches.  Traced at d = 64, 57 K tokens, 16
// routed blocks, window 512: 25 % of a workgroup's time was start, epilogues and filling pipelines, with nothing else
// on the CU, and the window's 24 shared steps cost as much as 50 compressed ones, because every query block's window
// edges (masks, redone tiles, a pipeline filled or drained) held up the barrier of all.  Attention step, four query
// blocks -> six of them with three wavefronts per SIMD and first copies under the epilogues -> two:
//   16 heads of 64, 57 K tokens 1025 -> 920 -> 797 us, 180 K tokens 4.64 -> 4.12 -> 3.78 ms; 4 heads of 64, 6 K tokens
//   52 -> 53 -> 39 us; 32 heads of 32 on 2, 196 K tokens 10.8 -> 10.7 (still four) -> 10.6 ms; 16 heads of 128, 428 K
//   tokens 34.9 -> 34.4 (still four) -> 32.7 ms; 3 heads of 128, 2752 tokens 100 -> 98 (still four) -> 62 us.
// It won at every size of a sweep over 12 .. 768 blocks and 1, 4, 16 heads.  What it costs is tile copies: the compressed
// tiles are read by twice as many workgroups, and at d = 128 the routed blocks that four neighbouring rows have in
// common (about half) are no longer copied once for all four.  Two query blocks with four stages (two workgroups per
// CU at d = 64): 57 K tokens 860 us, 180 K 4.03 ms.  Three query blocks: two such workgroups do not share a CU at
// three wavefronts per SIMD, since both put two wavefronts on the same two SIMDs (180 K tokens 5.12 ms).
template <int D_>
struct Geo {
    static constexpr int D = D_, NP = 2;
    static constexpr int NW = 2;                // wavefronts per query block
    static constexpr int ROWS = 32;             // query rows per wavefront
    static constexpr int NS = D / 16;           // 16-channel slabs of the QK^T contraction
    static constexpr int ND = D / 32;           // 32-channel tiles of the PV output
    static constexpr int K_BYTES = 32 * D * 2;  // 32 key rows
    static constexpr int V_BYTES = D * 64;      // D channel rows x 32 keys
    static constexpr int TILE = K_BYTES + V_BYTES;
    static constexpr int WAVES = NW * NP;
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int WAVES_PER_SIMD = D_ == 128 ? 2 : D_ == 64 ? 3 : 4;
    static constexpr int NST = 2;  // stages per query block in the phases where each streams its own tiles
    static constexpr int NSLOT = NST * NP;
    static constexpr int LDS_BYTES = NSLOT * TILE;
    static constexpr int KQ = 2, VQ = 2;        // operand fragments kept in registers (rolling queues)
    static constexpr int OUT_ROW = 2 * D + 8;   // padded bf16 row of the output staging (bytes)
    // The running gated sum (D / 8 fragments of four values per lane).  At d <= 64 it is fp32: the first
    // GSUM_FRAGS_REGS fragments in registers, the others in LDS.  d = 32: all in LDS (16 KB beside 16 KB of tiles).
    // d = 64: five of eight in LDS (20 KB beside 32 KB), which leaves 165 of the 168 registers of three wavefronts per SIMD.
    // d = 128: bf16; that of the first GSUM_LDS_WAVES wavefronts in LDS (16 KB beside 64 KB), that of the
    // others through the scratch buffer in memory.
    static constexpr bool GSUM_F32 = D_ <= 64;
    static constexpr int GSUM_FRAGS_LDS = D_ == 32 ? 4 : 5, GSUM_FRAGS_REGS = GSUM_F32 ? 4 * ND - GSUM_FRAGS_LDS : 0;
    static constexpr int GSUM_LDS_WAVES = GSUM_F32 ? WAVES : 2;
    static constexpr int GSUM_LDS_BYTES = GSUM_F32 ? GSUM_FRAGS_LDS * 1024 : 32 * D_ * 2;  // per wavefront
    // all of it, in bytes; as many workgroups fit a CU's 160 KB as the registers allow
    static constexpr int LDS_ALL = LDS_BYTES + GSUM_LDS_WAVES * GSUM_LDS_BYTES;
    static_assert(WAVES == 4 && WAVES_PER_SIMD * LDS_ALL <= 160 * 1024, "");
    static_assert(WAVES * ROWS * OUT_ROW <= LDS_BYTES, "output staging must fit in the tile slots");
};

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    bf16x2 p;
    p[0] = (__bf16)a;
    p[1] = (__bf16)b;
    return *reinterpret_cast<uint32_t *>(&p);
}

// max / sum across the two lane halves (lanes i and i + 32 hold the same query)
__device__ __forceinline__ float half_max(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// s_waitcnt immediates (vmcnt is split over bits [3:0] and [15:14], expcnt is bits [6:4],
// lgkmcnt bits [11:8]; counters that are not waited for are left at their maxima)
constexpr int vm_lgkm_imm(int n) { return (n & 0xF) | ((n >> 4) << 14) | 0x0070; }  // vmcnt <= n, lgkmcnt == 0
constexpr int kLgkmOnly = 0xC07F;                                                   // lgkmcnt == 0, vmcnt left alone

// Waits until at most n copies of UNIT instructions each are in flight, n <= MAX at run time (wave-uniform).
template <int UNIT, int MAX>
__device__ __forceinline__ void wait_copies(int n) {
    if constexpr (MAX == 0) {
        __builtin_amdgcn_s_waitcnt(vm_lgkm_imm(0));
    } else {
        static_assert(UNIT * MAX < 64, "vmcnt has six bits");
        if (n >= MAX)
            __builtin_amdgcn_s_waitcnt(vm_lgkm_imm(UNIT * MAX));
        else
            wait_copies<UNIT, MAX - 1>(n);
    }
}

// Bare workgroup barrier.  No barrier, fenced or not, waits for global -> LDS copies in flight
// (they are counted by vmcnt, which a workgroup-scope fence leaves alone), so what must be
// visible is ordered by hand: a wavefront waits for its own copies (s_waitcnt vmcnt, counted so
// that later tiles stay in flight) and its own LDS reads (lgkmcnt) before the barrier, and reads
// what others copied only after it.
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Results of an MFMA become readable by VALU instructions only a fixed number of cycles
// after issue, and the hardware does not interlock that dependency: the compiler pads
// with s_nop, but it has been seen to misplace the padding when a branch separates the
// MFMA from its first VALU reader.  Every such (rare) path starts with this explicit
// settle instead; 24 wait states cover the 8-pass MFMA used here.
__device__ __forceinline__ void mfma_settle() { asm volatile("s_nop 15\n\ts_nop 7" ::: "memory"); }

template <class G>
struct WaveCtx {
    bf16x8 qf[G::NS];
    f32x16 o[G::ND];
    float m, l;
    // running gated sum of the branches: the fragments kept in registers (d = 64).  At d = 128 it goes
    // through a bf16 scratch tile in LDS or global memory instead (fp32 there cost 1.8 % of the kernel for 7 % less
    // rounding error in `out`, whose own bf16 rounding and that of the probabilities dominate either way)
    f32x4 g[G::GSUM_FRAGS_REGS > 0 ? G::GSUM_FRAGS_REGS : 1];
    uint32_t lane16;  // lane * 16: byte offset of this lane inside any 1 KB fragment or copy instruction
};

// A tile (32 keys of one head) is stored in global memory as the exact image of its LDS slot:
// K_BYTES of K fragments, then V_BYTES of V^T fragments, each fragment 64 lanes x 16 bytes in
// the order the MFMA A operand wants them.  A copy instruction therefore moves 1 KB that is
// contiguous on both sides, and a fragment read is one ds_read_b128 at (slot + lane * 16) plus
// an immediate offset: conflict free, no per-fragment address registers or arithmetic.
//   K fragment ks (hh = lane bit 5, r = lane & 31): key perm(r), channels 16 ks + 8 hh + 0..7,
//     perm = bits 2 and 3 of r swapped (makes the S^T accumulator the B operand of the PV MFMA);
//   V^T fragment f = ks2 * ND + dt: channel 32 dt + r, keys 16 ks2 + 8 hh + 0..7.
// (Gathering the K fragments straight from the caller's [N, H, d] tensor instead -- every copy
// instruction touching 32 rows -- was measured: the attention kernel lost more than the packing
// pass costs.)

template <class G>
__device__ __forceinline__ void reset_branch(WaveCtx<G> &c) {
    c.m = kMinusHuge;
    c.l = 0.f;
#pragma unroll
    for (int dt = 0; dt < G::ND; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) c.o[dt][i] = 0.f;
}

// ---- pieces of one 32-key step of one wavefront ------------------------------------------
template <class G>
__device__ __forceinline__ void read_k(const WaveCtx<G> &c, const char *slot, bf16x8 (&kf)[G::NS]) {
#pragma unroll
    for (int ks = 0; ks < G::NS; ++ks) kf[ks] = *reinterpret_cast<const bf16x8 *>(slot + c.lane16 + ks * 1024);
}

// S^T = K Q^T for 32 keys x the wavefront's 32 queries
template <class G>
__device__ __forceinline__ void qk_scores(const WaveCtx<G> &c, const bf16x8 (&kf)[G::NS], f32x16 &s) {
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < G::NS; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], c.qf[ks], s, 0, 0, 0);
}

// Keys outside [lo, hi) of this lane's query get a score of -inf.
__device__ __forceinline__ void mask_scores(int lo, int hi, f32x16 &s, int j0, int lane) {
    const int hh = lane >> 5;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        int j = j0 + 16 * (i / 8) + 8 * hh + (i % 8);
        if (j < lo || j >= hi) s[i] = -__builtin_inff();
    }
}

__device__ __forceinline__ float lane_max(const f32x16 &s) {
    float mx = fmaxf(s[0], s[1]);
#pragma unroll
    for (int i = 2; i < 16; i += 2) mx = fmaxf(mx, fmaxf(s[i], s[i + 1]));
    return mx;
}

// The running maximum m of a row is kept optimistically: the exponentials of a tile are taken
// against the current m without looking at the tile's own maximum first, and only their row sum
// (which the softmax needs anyway) is examined afterwards.  If it exceeds kSumLimit -- some
// probability would be above 2^10, or infinite: m starts at kMinusHuge, so the first real tile of
// a branch always lands here -- the tile is redone: m is raised to the tile's maximum, O and l are
// rescaled, the probabilities recomputed.  Otherwise every probability is at most 2^10, harmless in
// fp32 and in bf16 (same exponent range), and the step has spent nothing on the maximum: no
// in-lane reduction, no exchange between lane halves, no wait for the score MFMAs to retire.
// A fully masked tile gives zeros and never redoes; a row whose keys are all masked so far keeps
// m = kMinusHuge.
constexpr float kSumLimit = 1024.0f;

// Wave-uniform: does any lane need its tile redone?  (psum is a sum of exponentials of finite or -inf arguments: never NaN)
__device__ __forceinline__ bool sum_overflow(float psum) {
    return __builtin_amdgcn_ballot_w64(!(psum <= kSumLimit)) != 0;
}

// Redoes the exponentials of one tile (scores s, already masked) after raising m to the tile's maximum; O and l (which do
// not yet contain this tile) are rescaled.  Rare path.
template <class G>
__device__ __forceinline__ void redo_tile(WaveCtx<G> &c, const f32x16 &s, uint32_t (&pu)[8], float &psum, float sl2) {
    mfma_settle();  // the O accumulators (and, at the start of a phase, s itself) may still be in flight
    const float mx = half_max(lane_max(s));
    const float m_new = fmaxf(c.m, mx);
    const float alpha = __builtin_amdgcn_exp2f((c.m - m_new) * sl2);
    c.m = m_new;
    c.l *= alpha;
#pragma unroll
    for (int dt = 0; dt < G::ND; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) c.o[dt][i] *= alpha;
    const float mc = m_new * sl2;
    float p[16];
    psum = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        p[e] = __builtin_amdgcn_exp2f(s[e] * sl2 - mc);
        psum += p[e];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) pu[k] = pack_bf16(p[2 * k], p[2 * k + 1]);
}

// After the exponentials of a tile: redo where needed, then add the row sums to l.
template <class G>
__device__ __forceinline__ void close_tile(WaveCtx<G> &c, const f32x16 &s, uint32_t (&pu)[8], float &psum, float sl2) {
    if (__builtin_expect(sum_overflow(psum), 0)) redo_tile<G>(c, s, pu, psum, sl2);
    c.l += psum;
}

union BFrag {
    bf16x8 v;
    uint32_t u[4];
};

// The MFMA block of one step.  Up to three tiles are in flight in a wavefront:
//   QK   the QK^T MFMAs of the tile whose scores are produced now        (-> s_next)
//   exp  the exponentials of the tile whose scores `s` are complete, already masked and
//        folded into the running maximum                                  (-> pu, c.l)
//   PV   the V^T P^T MFMAs of the tile before that (probabilities pu_prev)
// A wavefront issues in order and the matrix pipe runs one MFMA at a time, so MFMA and VALU
// work only overlap when they alternate in program order: the QK and PV MFMAs are issued
// alternately and every MFMA is followed by its share of the exponentials (one v_exp, its
// fma and sum, half a bf16 pack at d = 128) -- about as many VALU cycles as the MFMA takes.
// The row sums of the tile come back in psum (not yet added to l: see close_tile).
// The empty asm statements pin each result to its place in the program (the compiler
// otherwise sinks the arithmetic to its first use) and the scheduling barriers keep the
// machine scheduler from regrouping; neither emits an instruction.
// pu[k] = bf16 pair (p[2k], p[2k+1]): pu[0..3] / [4..7] are the B operands of the two 16-key slabs of the PV
// contraction.
// The A operands come from two rolling queues of LDS fragments (kq: K rows, vq: V^T rows), which the caller primes with the
// first ones: the MFMA that consumes fragment i is followed by the ds_read of fragment i + queue depth of the same
// tile.  k_cur and v_cur are per-lane addresses: slot + lane * 16.  LDS reads are thereby spread under the MFMAs,
// and only a few fragments are live at a time.
template <class G, bool QK, bool PV>
__device__ __forceinline__ void mfma_block(WaveCtx<G> &c, const f32x16 &s, bf16x8 (&kq)[G::KQ], f32x16 &s_next,
                                           bf16x8 (&vq)[G::VQ], const uint32_t (&pu_prev)[8], uint32_t (&pu)[8],
                                           float &psum, float sl2, const char *k_cur, const char *v_cur) {
    constexpr int NQ = QK ? G::NS : 0, NPV = PV ? 2 * G::ND : 0, NG = NQ + NPV;
    constexpr int NE = 16;
    const float mc = c.m * sl2;
    float p[NE];
    psum = 0.f;
    if constexpr (NG == 0) {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            p[e] = __builtin_amdgcn_exp2f(s[e] * sl2 - mc);
            psum += p[e];
        }
#pragma unroll
        for (int k = 0; k < NE / 2; ++k) pu[k] = pack_bf16(p[2 * k], p[2 * k + 1]);
    } else {
        constexpr int E = NE / NG;  // exponentials per MFMA
        static_assert(E >= 1 && E * NG == NE, "");
        BFrag pb[2];
        if (PV) {
#pragma unroll
            for (int k = 0; k < 8; ++k) pb[k / 4].u[k % 4] = pu_prev[k];
        }
        if (QK) {
#pragma unroll
            for (int i = 0; i < 16; ++i) s_next[i] = 0.f;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const bool do_qk = QK && (!PV || (g % 2) == 0);
            if (do_qk) {
                const int ks = PV ? g / 2 : g;
                s_next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kq[ks % G::KQ], c.qf[ks], s_next, 0, 0, 0);
                asm volatile("" : "+v"(s_next));
                if (ks + G::KQ < G::NS) kq[ks % G::KQ] = *reinterpret_cast<const bf16x8 *>(k_cur + (ks + G::KQ) * 1024);
            } else {
                const int f = QK ? g / 2 : g;
                const int ks = f / G::ND, dt = f % G::ND;
                c.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vq[f % G::VQ], pb[ks].v, c.o[dt], 0, 0, 0);
                asm volatile("" : "+v"(c.o[dt]));
                if (f + G::VQ < 2 * G::ND)
                    vq[f % G::VQ] = *reinterpret_cast<const bf16x8 *>(v_cur + G::K_BYTES + (f + G::VQ) * 1024);
            }
#pragma unroll
            for (int e = g * E; e < (g + 1) * E; ++e) {
                p[e] = __builtin_amdgcn_exp2f(s[e] * sl2 - mc);
                psum += p[e];
                if (e & 1) {
                    pu[e / 2] = pack_bf16(p[e - 1], p[e]);
                    asm volatile("" : "+v"(pu[e / 2]));
                } else {
                    asm volatile("" : "+v"(p[e]));
                }
            }
            asm volatile("" : "+v"(psum));
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// O^T += V^T P^T of the last tile (pipeline drain): the queue holds its first fragments.
template <class G>
__device__ __forceinline__ void pv_drain(WaveCtx<G> &c, bf16x8 (&vq)[G::VQ], const uint32_t (&pu)[8], const char *v_cur) {
    BFrag pb[2];
#pragma unroll
    for (int k = 0; k < 8; ++k) pb[k / 4].u[k % 4] = pu[k];
#pragma unroll
    for (int f = 0; f < 2 * G::ND; ++f) {
        const int ks = f / G::ND, dt = f % G::ND;
        c.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vq[f % G::VQ], pb[ks].v, c.o[dt], 0, 0, 0);
        if (f + G::VQ < 2 * G::ND)
            vq[f % G::VQ] = *reinterpret_cast<const bf16x8 *>(v_cur + G::K_BYTES + (f + G::VQ) * 1024);
    }
}

// Every wavefront is done with the tile slots of the phase that ends here.
// (LDS reads only: no copy is in flight at the end of a phase, and stores issued earlier -- outputs, the gated-sum
// scratch -- need not have been acknowledged before the first copies of the next phase go out; they are older than
// those copies, so the counted waits of its first steps still cover them)
__device__ __forceinline__ void end_phase() {
    __builtin_amdgcn_s_waitcnt(kLgkmOnly);
    wg_barrier();
}

// A phase streams tiles of 32 keys through LDS, K and V parts copied separately.  Where a tile comes from, which slot
// it lives in and who copies it is the business of a Tiles object:
//   OwnTiles     selected and window branch: each query block streams its own tiles through NST slots of its own, its
//                two wavefronts split the copies
//   SharedTiles  compressed branch, and all branches of a workgroup of two heads: one list of tiles for all, which go
//                through one ring of NSLOT slots, copied by all wavefronts together
// Both have: n (tiles of this query block), NST (tile tau lives in slot tau mod NST), PER_STEP (copies a wavefront issues
// per step), begin() (the first copies of the phase).  begin() is separate from run_tiles so that the epilogue of the previous
// branch -- at the start of the kernel, the loads of the query rows and of the routing rows -- runs while the first
// tiles are on their way.
template <class G, typename SrcFn>
struct OwnTiles {
    static constexpr int NP = G::NP, NST = G::NST;
    static constexpr bool EXACT = false, MEET = false;
    static constexpr int KI = G::K_BYTES / 1024 / G::NW, VI = G::V_BYTES / 1024 / G::NW, PER_STEP = KI + VI;
    static_assert(G::NW == 2, "two wavefronts per query block");
    static_assert((NST & (NST - 1)) == 0 && NST >= 2, "");
    const int n;  // tiles of this query block
    const SrcFn src;  // address of the image of tile tau
    char *const lds;
    const int qbi, sub;
    const uint32_t lane16;
    __device__ __forceinline__ char *stage(int tau) const { return lds + ((tau & (NST - 1)) * NP + qbi) * G::TILE; }
    __device__ __forceinline__ void issue_part(const char *tile, char *slot, int n_inst) const {
#pragma unroll 8
        for (int j = 0; j < n_inst; ++j) {
            const int i = sub + G::NW * j;
            copy_kb_to_lds(tile + i * 1024, lane16, slot + i * 1024);
        }
    }
    __device__ __forceinline__ void issue_k(int tau) const {
        issue_part(src(tau), stage(tau), KI);
    }
    __device__ __forceinline__ void issue_v(int tau) const {
        issue_part(src(tau) + G::K_BYTES, stage(tau) + G::K_BYTES, VI);
    }
    // the first copies of the phase (the slots are free)
    __device__ __forceinline__ void begin() const {
#pragma unroll
        for (int tau = 0; tau < NST; ++tau)
            if (tau < n) issue_k(tau);
#pragma unroll
        for (int tau = 0; tau < NST - 2; ++tau)
            if (tau < n) issue_v(tau);
    }
};

template <class G, typename SrcFn>
__device__ __forceinline__ OwnTiles<G, SrcFn> own_tiles(int n, SrcFn src, char *lds, int qbi, int sub, uint32_t lane16) {
    return OwnTiles<G, SrcFn>{n, src, lds, qbi, sub, lane16};
}

template <class G, typename SrcFn>
struct SharedTiles {
    static constexpr bool EXACT = false, MEET = false;
    static constexpr int NST = G::NSLOT, KN = G::K_BYTES / 1024, VN = G::V_BYTES / 1024;
    static constexpr int KI = (KN + G::WAVES - 1) / G::WAVES, VI = (VN + G::WAVES - 1) / G::WAVES;
    static constexpr int KW = KN / KI, VW = VN / VI;  // wavefronts that copy: the first KW the K part, the last VW the V part
    // copies per wavefront and step: both parts, or (d = 32, two instructions each) one of them
    static constexpr int PER_STEP = KW + VW <= G::WAVES ? KI : KI + VI;
    static_assert(KI == VI && KW == VW && (KW == G::WAVES || KW + VW == G::WAVES), "");
    static_assert(KW * KI == KN && VW * VI == VN, "");
    const int n;
    const SrcFn src;  // address of the image of tile tau
    char *const lds;
    const int wave;
    const uint32_t lane16;
    __device__ __forceinline__ char *stage(int tau) const { return lds + (tau & (NST - 1)) * G::TILE; }
    __device__ __forceinline__ void issue_k(int tau) const {
        if (KW < G::WAVES && wave >= KW) return;
        const char *tile = src(tau);
#pragma unroll
        for (int j = 0; j < KI; ++j) {
            const int i = wave + KW * j;
            copy_kb_to_lds(tile + i * 1024, lane16, stage(tau) + i * 1024);
        }
    }
    __device__ __forceinline__ void issue_v(int tau) const {
        if (VW < G::WAVES && wave < G::WAVES - VW) return;
        const char *tile = src(tau) + G::K_BYTES;
#pragma unroll
        for (int j = 0; j < VI; ++j) {
            const int i = (VW < G::WAVES ? wave - (G::WAVES - VW) : wave) + VW * j;
            copy_kb_to_lds(tile + i * 1024, lane16, stage(tau) + G::K_BYTES + i * 1024);
        }
    }
    __device__ __forceinline__ void begin() const {
#pragma unroll
        for (int tau = 0; tau < NST; ++tau)
            if (tau < n) issue_k(tau);
#pragma unroll
        for (int tau = 0; tau < NST - 2; ++tau)
            if (tau < n) issue_v(tau);
    }
};

template <class G, typename SrcFn>
__device__ __forceinline__ SharedTiles<G, SrcFn> shared_tiles(int n, SrcFn src, char *lds, int wave, uint32_t lane16) {
    return SharedTiles<G, SrcFn>{n, src, lds, wave, lane16};
}

// Three tiles are in flight in a wavefront: step t runs
// mfma_block with QK of its tile t+1, the exponentials of tile t and PV of tile t-1, so every MFMA
// has its share of the exponentials behind it.  Scores and probabilities alternate between two register sets
// (index = tile parity), so nothing is copied from step to step.  Barrier t comes before step t; behind it K(t) and
// V(t-2) are dead, and K(t+NST) and V(t+NST-2) are copied over them, NST-1 steps ahead of their use.
// The operand queues are primed from LDS at the start of every step (the next tile's fragments may
// still be in flight while a step runs, so the queues do not roll across tiles).
// mask_tile(t, s) masks the scores of the keys of tile t that the query block does not see.
// Steps 0 .. n (the last one is the PV of tile n-1); every wavefront meets barriers 0 .. n_steps, the largest n of
// the workgroup.
template <class G, typename Tiles, typename MaskFn>
__device__ __forceinline__ void run_tiles(WaveCtx<G> &c, int n_steps, const Tiles &tiles, MaskFn mask_tile, float sl2) {
    if (n_steps <= 0) return;
    constexpr int NST = Tiles::NST;
    const int n = tiles.n;
    auto stage = [&](int tau) { return tiles.stage(tau); };
    auto lstage = [&](int tau) { return tiles.stage(tau) + c.lane16; };
    // barrier t: K(t+1) and V(t-1) have landed (both were issued behind barrier t+1-NST; what the NST-2
    // barriers since then issued may stay in flight) and every LDS read of this wavefront is done.  Every
    // wavefront waits for its own copies before the barrier, so behind it the tiles are there for all
    // wavefronts, whoever copied them; all wavefronts are at the same step, so the slots overwritten behind
    // barrier t (K of step t, V of step t-2) are dead for all of them.
    auto sync = [&](int t) {
        if (NST > 2 && t + NST - 1 < n)
            __builtin_amdgcn_s_waitcnt(vm_lgkm_imm((NST - 2) * Tiles::PER_STEP));
        else if constexpr (Tiles::EXACT)
            wait_copies<Tiles::KI, Tiles::MOST>(tiles.in_flight(t));
        else
            __builtin_amdgcn_s_waitcnt(vm_lgkm_imm(0));
        if constexpr (Tiles::MEET)
            tiles.meet(t);
        else
            wg_barrier();
        if (t + NST < n) tiles.issue_k(t + NST);
        if (t + NST - 2 < n) tiles.issue_v(t + NST - 2);
    };
    bf16x8 kq[G::KQ], vq[G::VQ];
    f32x16 S[2];
    uint32_t P[2][8];
    float psum;
    auto prime_k = [&](const char *ls) {
#pragma unroll
        for (int i = 0; i < G::KQ; ++i) kq[i] = *reinterpret_cast<const bf16x8 *>(ls + i * 1024);
    };
    auto prime_v = [&](const char *ls) {
#pragma unroll
        for (int f = 0; f < G::VQ; ++f) vq[f] = *reinterpret_cast<const bf16x8 *>(ls + G::K_BYTES + f * 1024);
    };
    auto mask_next = [&](int t, f32x16 &s_next) {  // (an empty body where no tile can need a mask)
        if (t + 1 < n) mask_tile(t + 1, s_next);
    };
    if constexpr (Tiles::EXACT)
        wait_copies<Tiles::KI, Tiles::MOST>(tiles.n_copied > 0 ? tiles.in_flight_first() : 0);
    else
        __builtin_amdgcn_s_waitcnt(vm_lgkm_imm(0));
    wg_barrier();
    if (n > 0) {
        bf16x8 kf[G::NS];
        read_k<G>(c, stage(0), kf);
        qk_scores<G>(c, kf, S[0]);
        mask_next(-1, S[0]);
    }
    auto full_step = [&](auto par, int t) {
        constexpr int A = decltype(par)::value;
        sync(t);
        const char *k_nx = lstage(t + 1), *v_pv = lstage(t - 1);
        prime_k(k_nx);
        prime_v(v_pv);
        mfma_block<G, true, true>(c, S[A], kq, S[A ^ 1], vq, P[A ^ 1], P[A], psum, sl2, k_nx, v_pv);
        mask_next(t, S[A ^ 1]);
        close_tile<G>(c, S[A], P[A], psum, sl2);
    };
    auto last_steps = [&](auto par, int t) {  // t = n - 1 >= 1: exp(t) || PV(t-1), then the PV of tile t
        constexpr int A = decltype(par)::value;
        sync(t);
        const char *v_pv = lstage(t - 1);
        prime_v(v_pv);
        mfma_block<G, false, true>(c, S[A], kq, S[A ^ 1], vq, P[A ^ 1], P[A], psum, sl2, nullptr, v_pv);
        close_tile<G>(c, S[A], P[A], psum, sl2);
        sync(t + 1);
        const char *v_last = lstage(t);
        prime_v(v_last);
        pv_drain<G>(c, vq, P[A], v_last);
    };
    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, 1>;
    int done = 0;  // barriers 0 .. done-1 are behind us
    if (n >= 2) {
        sync(0);
        const char *k1 = lstage(1);
        prime_k(k1);
        mfma_block<G, true, false>(c, S[0], kq, S[1], vq, P[1], P[0], psum, sl2, k1, nullptr);
        mask_next(0, S[1]);
        close_tile<G>(c, S[0], P[0], psum, sl2);
        int t = 1;
        for (; t + 2 < n; t += 2) {
            full_step(Odd{}, t);
            full_step(Even{}, t + 1);
        }
        if (t + 1 < n) {
            full_step(Odd{}, t);
            ++t;
        }
        if (t & 1)
            last_steps(Odd{}, t);
        else
            last_steps(Even{}, t);
        done = n + 1;
    } else if (n == 1) {
        sync(0);
        mfma_block<G, false, false>(c, S[0], kq, S[1], vq, P[1], P[0], psum, sl2, nullptr, nullptr);
        close_tile<G>(c, S[0], P[0], psum, sl2);
        sync(1);
        const char *v_last = lstage(0);
        prime_v(v_last);
        pv_drain<G>(c, vq, P[0], v_last);
        done = 2;
    }
    if constexpr (Tiles::MEET) {
        tiles.leave();
    } else {
        for (int t = done; t <= n_steps; ++t) {
            __builtin_amdgcn_s_waitcnt(vm_lgkm_imm(0));
            wg_barrier();
        }
    }
}

// Ends a branch: normalises, applies the gate and folds the result into the running
// gated sum (registers, or the scratch tile: written by branch 0, updated by branch 1,
// consumed by branch 2, which converts to bf16 and stores the output rows through LDS).
// Optionally stores the un-gated branch output and its log-sum-exp.
template <class G>
__device__ __forceinline__ void finish_branch(WaveCtx<G> &c, const FwdArgs &a, int branch, int64_t row0, int head,
                                              int64_t gtile, int wave, int lane, char *lds) {
    constexpr int D = G::D;
    const int r = lane & 31, hh = lane >> 5;
    char *tr = lds + wave * G::ROWS * G::OUT_ROW;  // output staging region of this wavefront
    const int64_t row = row0 + r;
    const float l_tot = half_sum(c.l);
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    const float w = a.gate_channels ? inv : a.gates[(row * a.h + head) * 3 + branch] * inv;
    // per-channel gates of this row, branch and head: D floats
    const f32x4 *gch = reinterpret_cast<const f32x4 *>(a.gates + ((row * 3 + branch) * a.h + head) * D) + hh;
    if (a.lse != nullptr && hh == 0) {
        float v = l_tot > 0.f ? c.m * a.scale + __logf(l_tot) : -__builtin_inff();
        a.lse[((int64_t)branch * a.n + row) * a.h + head] = v;
    }
    if (a.out_branch != nullptr) {
#pragma unroll
        for (int dt = 0; dt < G::ND; ++dt) {
            uint16_t *dst = a.out_branch + (((int64_t)branch * a.n + row) * a.h + head) * D + 32 * dt + 4 * hh;
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                uint2 w2;
                w2.x = pack_bf16(c.o[dt][4 * gq + 0] * inv, c.o[dt][4 * gq + 1] * inv);
                w2.y = pack_bf16(c.o[dt][4 * gq + 2] * inv, c.o[dt][4 * gq + 3] * inv);
                *reinterpret_cast<uint2 *>(dst + 8 * gq) = w2;
            }
        }
    }
#pragma unroll
    for (int dt = 0; dt < G::ND; ++dt) {
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            f32x4 v;
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = w * c.o[dt][4 * gq + j];
            if (a.gate_channels) v *= gch[8 * dt + 2 * gq];  // channels 32 dt + 8 gq + 4 hh + 0..3
            if constexpr (G::GSUM_F32) {
                const int f = dt * 4 + gq;
                if (f < G::GSUM_FRAGS_REGS) {
                    if (branch > 0) v += c.g[f];
                    if (branch < 2) c.g[f] = v;
                } else {
                    f32x4 *slot_lds = reinterpret_cast<f32x4 *>(lds + G::LDS_BYTES + wave * G::GSUM_LDS_BYTES) +
                                      (f - G::GSUM_FRAGS_REGS) * 64 + lane;
                    if (branch > 0) v += *slot_lds;
                    if (branch < 2) *slot_lds = v;
                }
            } else {
                // bf16 pairs in accumulator order: 8 bytes per lane and fragment, fully coalesced; in LDS for the
                // first wavefronts of the workgroup (behind the ring), in the scratch buffer for the others
                // (the scratch buffer holds the query tiles of wavefronts GSUM_LDS_WAVES .. WAVES - 1 only: number gtile)
                uint2 *slot = reinterpret_cast<uint2 *>(a.gsum) + (gtile * (G::ND * 4) + dt * 4 + gq) * 64 + lane;
                uint2 *slot_lds =
                    reinterpret_cast<uint2 *>(lds + G::LDS_BYTES + wave * G::GSUM_LDS_BYTES) + (dt * 4 + gq) * 64 + lane;
                const bool in_lds = G::GSUM_LDS_WAVES == G::WAVES || wave < G::GSUM_LDS_WAVES;
                if (branch > 0) {
                    // (address spaces spelled out: one pointer that may be either would become a flat load)
                    unsigned long long raw;
                    if (in_lds)
                        raw = *(const __attribute__((address_space(3))) unsigned long long *)slot_lds;
                    else
                        raw = *(const __attribute__((address_space(1))) unsigned long long *)slot;
                    const uint2 pv = make_uint2((uint32_t)raw, (uint32_t)(raw >> 32));
                    v[0] += __uint_as_float(pv.x << 16);
                    v[1] += __uint_as_float(pv.x & 0xffff0000u);
                    v[2] += __uint_as_float(pv.y << 16);
                    v[3] += __uint_as_float(pv.y & 0xffff0000u);
                }
                if (branch < 2) {
                    uint2 w2;
                    w2.x = pack_bf16(v[0], v[1]);
                    w2.y = pack_bf16(v[2], v[3]);
                    if (in_lds)
                        *slot_lds = w2;
                    else
                        *slot = w2;
                }
            }
            if (branch == 2) {
                uint2 w2;
                w2.x = pack_bf16(v[0], v[1]);
                w2.y = pack_bf16(v[2], v[3]);
                *reinterpret_cast<uint2 *>(tr + r * G::OUT_ROW + (32 * dt + 8 * gq + 4 * hh) * 2) = w2;
            }
        }
    }
    if (branch == 2) {
        // rows of this wavefront back from LDS as whole 16-byte chunks: 4 (d=128) or 8 (d=64) rows per pass
        constexpr int CH = D / 8;
        constexpr int RPP = 64 / CH;
#pragma unroll
        for (int it = 0; it < G::ROWS / RPP; ++it) {
            const int rr = it * RPP + lane / CH, ch = lane % CH;
            uint4 val = *reinterpret_cast<const uint4 *>(tr + rr * G::OUT_ROW + ch * 16);
            *reinterpret_cast<uint4 *>(a.out + ((row0 + rr) * a.h + head) * D + ch * 8) = val;
        }
    }
}

// Window geometry of one query block (all values uniform over its wavefronts).
struct WinRange {
    int seg_lo, seg_hi;    // segment of the block
    int full_lo, full_hi;  // keys inside [full_lo, full_hi) are visible to all 64 queries of the block
    int st0, st1;          // 32-key tiles [st0, st1) intersect the block's window
};

__device__ __forceinline__ WinRange window_range(const FwdArgs &a, int qb) {
    WinRange w;
    const int q0 = qb * 64;
    w.seg_lo = 0;
    w.seg_hi = 0;
    if (a.blk_seg != nullptr) {  // segments per block (the query's spatial block), looked up instead of scanned
        w.seg_lo = a.blk_seg[2 * qb];
        w.seg_hi = a.blk_seg[2 * qb + 1];
    } else {
        for (int s = 0; s < a.n_seg; ++s) {
            int lo = a.seg[s], hi = a.seg[s + 1];
            if (q0 >= lo && q0 < hi) {
                w.seg_lo = lo;
                w.seg_hi = hi;
            }
        }
    }
    if (a.own_block) {
        // the block is its own segment (a.window is 128 in this mode: every query reaches every slot);
        // with counts, the segment ends at the last active token
        w.seg_lo = q0;
        w.seg_hi = q0 + (a.count != nullptr ? a.count[qb] : 64);
    }
    const int half = a.window / 2;
    const int k_start = max(w.seg_lo, q0 - half);
    const int k_end = min(w.seg_hi, q0 + 63 + half);  // exclusive
    w.full_lo = max(w.seg_lo, q0 + 63 - half);
    w.full_hi = min(w.seg_hi, q0 + half);
    w.st0 = k_start / 32;
    w.st1 = k_end > k_start ? (k_end - 1) / 32 + 1 : w.st0;
    return w;
}

// CNT: a.count is given (variable number of active tokens per block).
// WIDE: routing rows of 65..128 entries (two per lane of the list holder instead of one).
// HEADS: the workgroup has two query heads of one key/value head and one query block, instead of one head and two query
// blocks: all three branches then read the same tiles, which are copied to LDS once for both, four stages deep.  What that
// saves is the copies (they take instructions and the LDS; the images come from L2 either way); what it gave stands at
// its rule in launch_forward_d.
template <class G, bool CNT, bool WIDE, bool HEADS>
__global__ __launch_bounds__((G::THREADS), (G::WAVES_PER_SIMD)) void nsa_forward_kernel(FwdArgs a) {
    constexpr int D = G::D, NP = HEADS ? 1 : G::NP;  // query blocks of the workgroup
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    // XCD-aware numbering: hardware deals consecutive workgroups round-robin to the 8 XCDs
    // and runs them roughly in launch order.  All XCDs work on the same head at the same time (so the
    // K/V working set of the moment is one head: it fits the last-level cache and the pooled
    // keys/values fit every L2), each XCD on its own contiguous eighth of the head's query blocks
    // (so neighbouring windows and routed blocks meet in its L2).
    const int xcd = blockIdx.x & 7, slot_id = blockIdx.x >> 3;
    const int unit = slot_id / a.groups_per_xcd;  // head, or pair of heads
    const int group = xcd * a.groups_per_xcd + slot_id % a.groups_per_xcd;
    if (group >= a.groups_per_head) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sub = wave % G::NW;              // wavefront inside the block
    const int qbi = HEADS ? 0 : wave / G::NW;  // query block inside the group
    const int head = HEADS ? 2 * unit + wave / G::NW : unit;
    const int64_t gtile = (int64_t)(2 * group + wave - G::GSUM_LDS_WAVES) * (HEADS ? a.h / 2 : a.h) + unit;
    const int r = lane & 31, hh = lane >> 5;
    const int qb = group * NP + qbi;
    const bool active = qb < a.nb;  // a trailing group may have fewer than NP query blocks
    const int64_t row0 = (int64_t)(active ? qb : 0) * 64 + G::ROWS * sub;
    const int kvh = head / a.group;                         // key/value head of this query head
    // images are stored head-major: the tiles of one head are contiguous
    const int64_t tile_stride = G::TILE;
    const int64_t head_kv = (int64_t)kvh * (2 * a.nb) * G::TILE, head_kvc = (int64_t)kvh * ((a.nbc + 31) / 32) * G::TILE;
    const float sl2 = a.scale_log2e;

    WaveCtx<G> c;
    c.lane16 = (uint32_t)lane * 16u;
    // The first copies go out before anything else.  (Slots that no copy fills hold anything: run_tiles reads the tiles of
    // the phase only.)
    const int n_cmp = (a.nbc + 31) / 32;
    const char *const base_c = a.kvc + head_kvc;
    const auto cmp_tiles = shared_tiles<G>(n_cmp, [=](int t) { return base_c + (int64_t)t * G::TILE; }, lds, wave, c.lane16);
    cmp_tiles.begin();
    {
        // (an inactive wavefront reads the rows of block 0: finite values, results discarded)
        const uint16_t *qrow = a.q + ((row0 + r) * a.h + head) * D + 8 * hh;
#pragma unroll
        for (int ks = 0; ks < G::NS; ++ks) c.qf[ks] = *reinterpret_cast<const bf16x8 *>(qrow + 16 * ks);
    }

    // ---------------- this query block's routing row, read while the first compressed tiles are copied;
    // valid entries first: entry u sits in lane u % 64 of register u / 64
    constexpr int NR = WIDE ? 2 : 1;
    int packed[NR], pcount[NR], my_valid = 0, max_valid = 0;
#pragma unroll
    for (int j = 0; j < NR; ++j) packed[j] = -1, pcount[j] = 0;
    {
        // rows of the routing table: compacted through 512 bytes per wavefront of the LDS that will hold gated sums
        static_assert(G::GSUM_LDS_WAVES * G::GSUM_LDS_BYTES >= 512 * G::WAVES, "");
        int *scratch = reinterpret_cast<int *>(lds + G::LDS_BYTES + wave * 512);
        int raw[NP][NR];  // (all loads in flight together; lanes past the end of a row read its first entry)
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int j = 0; j < NR; ++j) {
                const int col = lane + 64 * j;
                raw[p][j] = a.topk > 0 ? a.idx[(int64_t)min(group * NP + p, a.nb - 1) * a.topk + (col < a.topk ? col : 0)] : -1;
            }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int qbp = group * NP + p;
            int v[NR], n_valid = 0;
            unsigned long long bal[NR];
#pragma unroll
            for (int j = 0; j < NR; ++j) {
                v[j] = (qbp < a.nb && lane + 64 * j < a.topk) ? raw[p][j] : -1;
                if (v[j] >= a.nb) v[j] = -1;
                bal[j] = __ballot(v[j] >= 0);
                n_valid += __popcll(bal[j]);
            }
            max_valid = max(max_valid, n_valid);
            if (p == qbi) {
                int before = 0;
#pragma unroll
                for (int j = 0; j < NR; ++j) {
                    if (v[j] >= 0) scratch[before + __popcll(bal[j] & ((1ull << lane) - 1ull))] = v[j];
                    before += __popcll(bal[j]);
                }
                // (LDS operations of a wavefront complete in order: the reads below see the writes above)
#pragma unroll
                for (int j = 0; j < NR; ++j) packed[j] = lane + 64 * j < n_valid ? scratch[lane + 64 * j] : -1;
                my_valid = n_valid;
            }
        }
    }
    if constexpr (CNT) {
#pragma unroll
        for (int j = 0; j < NR; ++j) pcount[j] = lane + 64 * j < my_valid ? a.count[packed[j]] : 0;
    }

    // ---------------- compressed branch: all NB pooled pairs
    {
        reset_branch<G>(c);
        auto mask_tile = [&](int t, f32x16 &sc) {
            if (32 * t + 32 > a.nbc) {
                mfma_settle();
                mask_scores(0, a.nbc, sc, 32 * t, lane);
            }
        };
        run_tiles<G>(c, n_cmp, cmp_tiles, mask_tile, sl2);
    }

    auto tiles_of = [&](int n, auto src) {
        if constexpr (HEADS)
            return shared_tiles<G>(n, src, lds, wave, c.lane16);
        else
            return own_tiles<G>(n, src, lds, qbi, sub, c.lane16);
    };
    // ---------------- selected branch: every token of the routed blocks
    {
        // entry u of the row / of the counts (wave-uniform u)
        auto entry = [&](int u) {
            if constexpr (WIDE) {
                const int e0 = __builtin_amdgcn_readlane(packed[0], u & 63), e1 = __builtin_amdgcn_readlane(packed[NR - 1], u & 63);
                return u < 64 ? e0 : e1;
            } else {
                return __builtin_amdgcn_readlane(packed[0], u);
            }
        };
        const char *base = a.kv + head_kv;
        auto src = [&](int t) { return base + (2 * entry(t >> 1) + (t & 1)) * tile_stride; };
        auto valid = [&](int t) {  // active keys of tile t of this query block's list
            const int u = t >> 1;
            int cnt;
            if constexpr (WIDE) {
                const int c0 = __builtin_amdgcn_readlane(pcount[0], u & 63), c1 = __builtin_amdgcn_readlane(pcount[NR - 1], u & 63);
                cnt = u < 64 ? c0 : c1;
            } else {
                cnt = __builtin_amdgcn_readlane(pcount[0], u);
            }
            return min(32, max(0, cnt - 32 * (t & 1)));
        };
        auto mask_tile = [&](int t, f32x16 &sc) {
            if constexpr (CNT) {
                const int vld = valid(t);
                if (vld < 32) {
                    mfma_settle();
                    mask_scores(0, vld, sc, 0, lane);
                }
            }
        };
        const auto tiles = tiles_of(2 * my_valid, src);
        end_phase();
        tiles.begin();
        if (active) finish_branch<G>(c, a, 0, row0, head, gtile, wave, lane, lds);
        reset_branch<G>(c);
        run_tiles<G>(c, 2 * max_valid, tiles, mask_tile, sl2);
    }

    // ---------------- window branch: keys j with -W/2 <= j - i < W/2 inside the segment
    {
        const WinRange mine = window_range(a, active ? qb : 0);
        int n_max = 0;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int qbp = group * NP + p;
            if (qbp < a.nb) {
                const WinRange w = window_range(a, qbp);
                n_max = max(n_max, w.st1 - w.st0);
            }
        }
        // the keys that this lane's query sees
        const int i = (int)row0 + r, half_w = a.window / 2;
        const int lo = max(mine.seg_lo, i - half_w), hi = min(mine.seg_hi, i + half_w);
        const char *base = a.kv + head_kv;
        auto src = [&](int t) { return base + (mine.st0 + t) * tile_stride; };
        auto mask_tile = [&](int t, f32x16 &sc) {
            const int j0 = 32 * (mine.st0 + t);
            bool need = j0 < mine.full_lo || j0 + 32 > mine.full_hi;
            int cap = 0x7fffffff;
            if constexpr (CNT) {
                // slots of the tile's block beyond its active tokens (in own-block mode the segment already ends there)
                if (!a.own_block) {
                    const int vld = min(32, max(0, a.count[j0 >> 6] - (j0 & 32)));
                    if (vld < 32) {
                        need = true;
                        cap = j0 + vld;
                    }
                }
            }
            if (need) {
                mfma_settle();
                mask_scores(lo, min(hi, cap), sc, j0, lane);
            }
        };
        const auto tiles = tiles_of(active ? mine.st1 - mine.st0 : 0, src);
        end_phase();
        tiles.begin();
        if (active) finish_branch<G>(c, a, 1, row0, head, gtile, wave, lane, lds);
        reset_branch<G>(c);
        run_tiles<G>(c, n_max, tiles, mask_tile, sl2);
        __builtin_amdgcn_s_waitcnt(vm_lgkm_imm(0));
        wg_barrier();  // the tile slots are about to be reused for the output rows
        if (active) finish_branch<G>(c, a, 2, row0, head, gtile, wave, lane, lds);
    }
}

// The same layer for few query blocks: the three branches run beside each other instead of one after the other, in one workgroup
// per query block and head (or two query blocks).  NT teams of two wavefronts share the tiles of a query block: every
// branch has teams of its own, the longest branches the most (FwdArgs::teams), and a team streams a contiguous part of its
// branch's tiles.  All run the same code (the tiles' addresses and masks differ), so that its instructions are fetched once
// and not three times.  The teams' running maxima, sums and outputs meet in LDS in fp32.
// A lone workgroup of nsa_forward_kernel is a chain: 6 K tokens, 4 heads of 64, 8 routed blocks, window 512
// (3 + 16 + 18 steps) took 39.5 K cycles, 3.1 K of them for the routing row, 4.1 / 8.7 / 13.9 K for the branches at 500 to 800 a step, 2 to
// 3 K for each epilogue, on SIMDs with one wavefront or none.
// Attention step, nsa_forward_kernel and this: that problem 19.9 -> 14.8 us; 43 blocks, 3 heads of 128, 9 routed blocks, window
// 192: 33.8 -> 15.6 us (what remains is the copies' latency, two stages deep: 2000 cycles a step, 1400 without copies).
// PAIRS: the workgroups make the images of the pooled pairs by themselves (FwdArgs::kc, vc), all of them, behind the slots.
// MEET: the two wavefronts of a team wait for each other only in a step, not for all teams, by two numbers a team (TeamTiles::meet).
// A barrier keeps all in step, copying and computing at the same times, as slow as the slowest: with packing, out of a graph, us, 16
// blocks x 1 head of 32 13.2 / 12.5, 128 x 2 19.2 / 18.3; of 64 33 x 4 16.6 / 15.8, 65 x 4 24.0 / 22.8, 200 x 1 26.8 / 25.6, 96 x 4 the
// same.  Not at d = 128 (128 x 2 34.8 / 34.4, 33 x 4 22.4 / 22.7).
template <class G, int NB_, int NT_, int NST_, bool PAIRS_>
struct Teams {
    static constexpr bool PAIRS = PAIRS_, MEET = G::D <= 64;
    static constexpr int NB = NB_, NT = NT_, NST = NST_;  // query blocks of a workgroup; teams of one; stages of a team
    static constexpr int THREADS = 64 * G::NW * NT * NB;
    static constexpr int PITCH = G::D + 4;  // floats of a row of a team's result: 16-byte aligned, rows spread over the banks
    static constexpr int TILES_BYTES = NB * NT * NST * G::TILE, SUM_BYTES = NB * NT * kBlock * (PITCH + 2) * 4;
    static constexpr int LDS_ALL = TILES_BYTES > SUM_BYTES ? TILES_BYTES : SUM_BYTES;
    // Tiles of pooled pairs that fit a CU's LDS behind the slots (what the teams add up at the end takes their place): 16 at d = 32, 8
    // at d = 64, 2 at d = 128.
    static constexpr int MAX_PAIRS = (160 * 1024 - TILES_BYTES) / G::TILE;
    // Where the numbers of MEET are: behind everything else, or, with PAIRS, in the slots of team 0, a team of the pooled pairs, which
    // copies nothing there.
    static constexpr int STEPS_AT = PAIRS ? 0 : LDS_ALL;
    static constexpr int lds_bytes(int tiles) {
        return PAIRS ? (tiles * G::TILE > LDS_ALL - TILES_BYTES ? TILES_BYTES + tiles * G::TILE : LDS_ALL) : LDS_ALL + (MEET ? NB * NT * 8 : 0);
    }
    static constexpr int WAVES_PER_SIMD = (THREADS / 64 + 3) / 4;  // (one workgroup per CU)
    static_assert(LDS_ALL <= 160 * 1024 && NT >= 3, "");
};

template <class G, class TM, typename SrcFn>
struct TeamTiles {
    static constexpr int NST = TM::NST;
    static constexpr bool EXACT = true, MEET = TM::MEET;
    static constexpr int KI = G::K_BYTES / 1024 / G::NW, VI = G::V_BYTES / 1024 / G::NW, PER_STEP = KI + VI;
    const int n;
    const int n_copied;  // n, or 0: the tiles are there already, one behind the other from `lds` on
    const SrcFn src;
    char *const lds;  // the slots of the team
    int *const steps;  // [2] in LDS: steps that the team's wavefronts have come to
    const int sub;
    const uint32_t lane16;
    __device__ __forceinline__ char *stage(int tau) const { return lds + (!TM::PAIRS || n_copied > 0 ? tau & (NST - 1) : tau) * G::TILE; }
    __device__ __forceinline__ void issue_part(const char *tile, char *slot, int n_inst) const {
#pragma unroll 8
        for (int j = 0; j < n_inst; ++j) {
            const int i = sub + G::NW * j;
            copy_kb_to_lds(tile + i * 1024, lane16, slot + i * 1024);
        }
    }
    __device__ __forceinline__ void issue_k(int tau) const {
        if (!TM::PAIRS || n_copied > 0) issue_part(src(tau), stage(tau), KI);
    }
    __device__ __forceinline__ void issue_v(int tau) const {
        if (!TM::PAIRS || n_copied > 0) issue_part(src(tau) + G::K_BYTES, stage(tau) + G::K_BYTES, VI);
    }
    // The barrier of a team: a wavefront says that it has come to step t (its copies and reads are waited for) and looks until the
    // other has, which runs as many steps.  After its last it says so for all: each has read the routing row for itself, and if a
    // caller lets the table be written meanwhile, the rows may differ and the result is worthless, but no wavefront may wait for ever.
    __device__ __forceinline__ void say(int t) const {
        asm volatile("ds_write_b32 %0, %1" ::"v"((uint32_t)(uintptr_t)steps + 4 * sub), "v"(t) : "memory");
    }
    __device__ __forceinline__ void leave() const { say(0x7fffffff); }
    __device__ __forceinline__ void meet(int t) const {
        const uint32_t at = (uint32_t)(uintptr_t)steps;
        say(t + 1);
        int other;
        do {
            asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(other) : "v"(at + 4 * (1 - sub)) : "memory");
        } while (__builtin_amdgcn_readfirstlane(other) <= t);
    }
    // in the order K(0), K(1), V(0), K(2), V(1), ..
    __device__ __forceinline__ void begin() const {
#pragma unroll
        for (int tau = 0; tau < NST; ++tau) {
            if (tau < n_copied) issue_k(tau);
            if (tau >= 1 && tau < NST - 1 && tau - 1 < n_copied) issue_v(tau - 1);
        }
    }
    // Copies that may be in flight at barrier t, in units of KI instructions: behind K(t + 1) and V(t - 1) those of K(t + 2 ..) and
    // V(t ..) that were issued before it; ahead of the first step all but K(0).
    static constexpr int MOST = 2 * NST - 3;
    static_assert(KI == VI, "");
    __device__ __forceinline__ int in_flight(int t) const { return min(NST - 2, max(0, n_copied - 2 - t)) + min(NST - 2, max(0, n_copied - t)); }
    __device__ __forceinline__ int in_flight_first() const { return min(NST - 1, n_copied - 1) + min(NST - 2, n_copied); }
};

template <class G, bool CNT, bool WIDE, class TM>
__global__ __launch_bounds__((TM::THREADS), (TM::WAVES_PER_SIMD)) void nsa_forward_teams(FwdArgs a) {
    constexpr int D = G::D, NB = TM::NB, NT = TM::NT;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    // Equal shares of all workgroups for the XCDs, of 32 CUs each: the chip holds them together only if none gets more.  (An eighth
    // of every head's, rounded up, is 36 for 17 blocks x 12 heads; with packing, general kernel, that deal, this one, us: d = 32 26.6, 29.8,
    // 16.8; 9 x 28 26.7, 30.8, 17.3; one block x 256 heads of 64 59.9, 80.3, 16.7.)
    const int item = (blockIdx.x & 7) * a.groups_per_xcd + (blockIdx.x >> 3);
    const int head = item / a.groups_per_head, group = item - head * a.groups_per_head;
    if (head >= a.h) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int team = wave % NT, sub = wave / NT % G::NW, qbi = wave / (NT * G::NW);
    const int branch = team < a.teams[0] ? 0 : team < a.teams[0] + a.teams[1] ? 1 : 2;
    const int part = branch == 0 ? team : branch == 1 ? team - a.teams[0] : team - a.teams[0] - a.teams[1];
    const int n_parts = a.teams[branch];
    const int r = lane & 31, hh = lane >> 5;
    const int qb = min(group * NB + qbi, a.nb - 1);  // (the last group may be short: its last wavefronts have no keys)
    const bool active = group * NB + qbi < a.nb;
    const int64_t row0 = (int64_t)qb * 64 + G::ROWS * sub, row = row0 + r;
    const int kvh = head / a.group;
    const float sl2 = a.scale_log2e;
    char *const slots = lds + (qbi * NT + team) * TM::NST * G::TILE;

    // the routing row, valid entries first (entry u in lane u % 64 of register u / 64), compacted in the part of the branch's
    // slots that this wavefront copies to
    constexpr int NR = WIDE ? 2 : 1;
    int packed[NR], pcount[NR], n_valid = 0;
#pragma unroll
    for (int j = 0; j < NR; ++j) packed[j] = -1, pcount[j] = 0;
    if (branch == 1) {
        int *scratch = reinterpret_cast<int *>(slots + sub * 1024);
        int v[NR];
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            v[j] = lane + 64 * j < a.topk ? a.idx[(int64_t)qb * a.topk + lane + 64 * j] : -1;
            if (v[j] >= a.nb) v[j] = -1;
        }
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const unsigned long long bal = __ballot(v[j] >= 0);
            if (v[j] >= 0) scratch[n_valid + __popcll(bal & ((1ull << lane) - 1ull))] = v[j];
            n_valid += __popcll(bal);
        }
        // (LDS operations of a wavefront complete in order: the reads see the writes)
#pragma unroll
        for (int j = 0; j < NR; ++j) packed[j] = lane + 64 * j < n_valid ? scratch[lane + 64 * j] : -1;
        if constexpr (CNT) {
#pragma unroll
            for (int j = 0; j < NR; ++j) pcount[j] = lane + 64 * j < n_valid ? a.count[packed[j]] : 0;
        }
    }
    WaveCtx<G> c;
    c.lane16 = (uint32_t)lane * 16u;
    const uint16_t *qrow = a.q + (row * a.h + head) * D + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < G::NS; ++ks) c.qf[ks] = *reinterpret_cast<const bf16x8 *>(qrow + 16 * ks);
    auto of_row = [&](const int (&x)[NR], int u) {  // (u is wave-uniform)
        const int e0 = __builtin_amdgcn_readlane(x[0], u & 63);
        if constexpr (WIDE) {
            const int e1 = __builtin_amdgcn_readlane(x[NR - 1], u & 63);
            return u < 64 ? e0 : e1;
        } else {
            return e0;
        }
    };

    // the keys of this team: tiles first .. first + n - 1 of an image, or entries of the routing row; lane's query sees [lo, hi),
    // all queries [full_lo, full_hi)
    const WinRange win = window_range(a, qb);
    const int n_cmp = (a.nbc + 31) / 32;
    const bool cmp = branch == 0;
    const int n_branch = !active ? 0 : cmp ? n_cmp : branch == 1 ? 2 * n_valid : win.st1 - win.st0;
    const int t0 = n_branch * part / n_parts, n = n_branch * (part + 1) / n_parts - t0;
    const int i = (int)row, half_w = a.window / 2;
    const int first = (cmp ? 0 : branch == 1 ? 0 : win.st0) + t0;
    const int full_lo = cmp ? 0 : win.full_lo, full_hi = cmp ? a.nbc : win.full_hi;
    const int lo = cmp ? 0 : max(win.seg_lo, i - half_w), hi = cmp ? a.nbc : min(win.seg_hi, i + half_w);
    // no fewer steps than any wavefront of the workgroup has
    int n_win = win.st1 - win.st0;
    if (NB == 2) {
        const WinRange other = window_range(a, min(group * NB + 1 - qbi, a.nb - 1));
        n_win = max(n_win, other.st1 - other.st0);
    }
    const int n_steps = max(max((n_cmp + a.teams[0] - 1) / a.teams[0], (2 * a.topk + a.teams[1] - 1) / a.teams[1]),
                            (n_win + a.teams[2] - 1) / a.teams[2]);
    const char *base = cmp ? a.kvc + (int64_t)kvh * n_cmp * G::TILE : a.kv + (int64_t)kvh * (2 * a.nb) * G::TILE;
    auto src = [&](int t) {
        const int tile = branch == 1 ? 2 * of_row(packed, (first + t) >> 1) + ((first + t) & 1) : first + t;
        return base + (int64_t)tile * G::TILE;
    };
    auto mask_tile = [&](int t, f32x16 &sc) {
        // (masks of their own for the selected branch: with counts most tiles need one, and one bound is half the work of two; 171 x 2 of
        // d = 32, 64 partly filled blocks routed, 113 -> 94 us)
        if (branch == 1) {
            if constexpr (CNT) {
                const int vld = min(32, max(0, of_row(pcount, (first + t) >> 1) - 32 * ((first + t) & 1)));
                if (vld < 32) {
                    mfma_settle();
                    mask_scores(0, vld, sc, 0, lane);
                }
            }
            return;
        }
        const int j0 = 32 * (first + t);
        int to = hi;
        bool need = j0 < full_lo || j0 + 32 > full_hi;
        if constexpr (CNT) {
            if (branch == 2 && !a.own_block) {
                const int vld = min(32, max(0, a.count[j0 >> 6] - (j0 & 32)));
                if (vld < 32) {
                    need = true;
                    to = min(hi, j0 + vld);
                }
            }
        }
        if (need) {
            mfma_settle();
            mask_scores(lo, to, sc, j0, lane);
        }
    };
    const bool there = TM::PAIRS && cmp;
    char *const pairs = lds + TM::TILES_BYTES;
    int *const steps = reinterpret_cast<int *>(lds + TM::STEPS_AT) + 2 * (qbi * NT + team);
    if (TM::MEET && lane == 0) steps[sub] = 0;
    const TeamTiles<G, TM, decltype(src)> tiles{n, there ? 0 : n, src, there ? pairs + t0 * G::TILE : slots, steps, sub, c.lane16};
    tiles.begin();
    if constexpr (TM::PAIRS) {
        // The images of all pooled pairs of this key/value head (see pack_block), rows past the end as zeros: a launch of its own took 3 us
        // and the time to enqueue it.  The first barrier of run_tiles publishes them.  A thread turns eight rows of V by eight channels.
        constexpr int CHUNKS = D / 8;
        auto chunk = [&](const uint16_t *from, int pair, int ch) {
            return pair < a.nbc ? *reinterpret_cast<const uint4 *>(from + ((int64_t)pair * a.h_kv + kvh) * D + 8 * ch) : make_uint4(0, 0, 0, 0);
        };
        for (int e = threadIdx.x; e < n_cmp * 4 * CHUNKS; e += TM::THREADS) {
            const int pair = e / CHUNKS * 8, ch = e % CHUNKS, r32 = pair % 32;
            uint4 row[8];
#pragma unroll
            for (int x = 0; x < 8; ++x) row[x] = chunk(a.vc, pair + x, ch);
            char *vt = pairs + pair / 32 * G::TILE + G::K_BYTES + (r32 / 16 * G::ND + ch / 4) * 1024 + (r32 / 8 % 2 * 32 + ch % 4 * 8) * 16;
#pragma unroll
            for (int x = 0; x < 8; ++x) {  // channel 8 ch + x of the eight rows
                uint32_t w[4];
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    const uint4 &r0 = row[2 * y], &r1 = row[2 * y + 1];
                    const uint32_t lo = x / 2 == 0 ? r0.x : x / 2 == 1 ? r0.y : x / 2 == 2 ? r0.z : r0.w;
                    const uint32_t hi = x / 2 == 0 ? r1.x : x / 2 == 1 ? r1.y : x / 2 == 2 ? r1.z : r1.w;
                    w[y] = x % 2 == 0 ? (lo & 0xffffu) | hi << 16 : lo >> 16 | (hi & 0xffff0000u);
                }
                *reinterpret_cast<uint4 *>(vt + x * 16) = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
#pragma unroll 2
        for (int e = threadIdx.x; e < n_cmp * 32 * CHUNKS; e += TM::THREADS) {
            const int pair = e / CHUNKS, ch = e % CHUNKS, r32 = pair % 32;
            *reinterpret_cast<uint4 *>(pairs + pair / 32 * G::TILE + ch * 512 + ((r32 & ~12) | ((r32 & 4) << 1) | ((r32 & 8) >> 1)) * 16) =
                chunk(a.kc, pair, ch);
        }
    }
    // A thread finishes 8 channels of NIT rows: their gates are requested now.
    constexpr int CH = D / 8, NIT = (NB * kBlock * CH + TM::THREADS - 1) / TM::THREADS;
    const int n_rows = kBlock * min(NB, a.nb - group * NB);
    const int64_t out0 = (int64_t)group * NB * kBlock;
    // (One of three by a number known at run time: out of an array of floats that is a load from scratch, 64 x 4 of d = 64, with
    // packing, 20.2 us for 19.4.)
    f32x4 gate[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int rr = (threadIdx.x + TM::THREADS * it) / CH;
#pragma unroll
        for (int b = 0; b < 3; ++b)
            gate[it][b] = !a.gate_channels && rr < n_rows ? a.gates[((out0 + rr) * a.h + head) * 3 + b] : 1.f;
    }
    reset_branch<G>(c);
    run_tiles<G>(c, n_steps, tiles, mask_tile, sl2);

    // The teams of a branch bring their results to the branch's maximum and sum.
    float *sums = reinterpret_cast<float *>(lds);     // [query block][team][row][PITCH]
    float *ml = sums + NB * NT * kBlock * TM::PITCH;  // [query block][team][row][2]: running maximum, row sum
    const int my_row = (qbi * NT + team) * kBlock + G::ROWS * sub + r;
    const float l_part = half_sum(c.l);
    __builtin_amdgcn_s_waitcnt(vm_lgkm_imm(0));
    wg_barrier();  // (the tile slots are reused)
    if (hh == 0) {
        ml[2 * my_row] = c.m;
        ml[2 * my_row + 1] = l_part;
    }
    __syncthreads();
    float m = c.m, l = l_part, f = 1.f;
    if (n_parts > 1) {
        const int of_branch = my_row - part * kBlock;
        m = kMinusHuge;
        for (int j = 0; j < n_parts; ++j) m = fmaxf(m, ml[2 * (of_branch + j * kBlock)]);
        l = 0.f;
        for (int j = 0; j < n_parts; ++j) {
            const int at = of_branch + j * kBlock;
            l += ml[2 * at + 1] * __builtin_amdgcn_exp2f((ml[2 * at] - m) * sl2);
        }
        f = __builtin_amdgcn_exp2f((c.m - m) * sl2);
    }
    f = l > 0.f ? f / l : 0.f;
    if (a.lse != nullptr && part == 0 && hh == 0 && active)
        a.lse[((int64_t)branch * a.n + row) * a.h + head] = l > 0.f ? m * a.scale + __logf(l) : -__builtin_inff();
#pragma unroll
    for (int dt = 0; dt < G::ND; ++dt)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq)
            *reinterpret_cast<f32x4 *>(sums + my_row * TM::PITCH + 32 * dt + 8 * gq + 4 * hh) =
                f32x4{f * c.o[dt][4 * gq], f * c.o[dt][4 * gq + 1], f * c.o[dt][4 * gq + 2], f * c.o[dt][4 * gq + 3]};
    __syncthreads();
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int e = threadIdx.x + TM::THREADS * it, rr = e / CH, ch = e % CH;
        if (rr >= n_rows) break;
        const float *at = sums + (rr / kBlock * NT * kBlock + rr % kBlock) * TM::PITCH + 8 * ch;
        f32x4 part_of[NT][2], total[2], of_branch[2];
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int q4 = 0; q4 < 2; ++q4) part_of[j][q4] = *reinterpret_cast<const f32x4 *>(at + j * kBlock * TM::PITCH + 4 * q4);
        int b = 0, end = a.teams[0];  // branch of team j and the first team of the next one
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const bool opens = j == 0 || j == end;
            if (j > 0 && j == end) end += a.teams[++b];
#pragma unroll
            for (int q4 = 0; q4 < 2; ++q4) of_branch[q4] = opens ? part_of[j][q4] : of_branch[q4] + part_of[j][q4];
            if (j + 1 < end) continue;
            if (a.out_branch != nullptr)
                *reinterpret_cast<uint4 *>(a.out_branch + (((int64_t)b * a.n + out0 + rr) * a.h + head) * D + ch * 8) =
                    make_uint4(pack_bf16(of_branch[0][0], of_branch[0][1]), pack_bf16(of_branch[0][2], of_branch[0][3]),
                               pack_bf16(of_branch[1][0], of_branch[1][1]), pack_bf16(of_branch[1][2], of_branch[1][3]));
            const float g = b == 0 ? gate[it][0] : b == 1 ? gate[it][1] : gate[it][2];
#pragma unroll
            for (int q4 = 0; q4 < 2; ++q4) {
                f32x4 v = of_branch[q4] * g;
                if (a.gate_channels)
                    v *= *reinterpret_cast<const f32x4 *>(a.gates + (((out0 + rr) * 3 + b) * a.h + head) * D + ch * 8 + 4 * q4);
                total[q4] = b == 0 ? v : total[q4] + v;
            }
        }
        *reinterpret_cast<uint4 *>(a.out + ((out0 + rr) * a.h + head) * D + ch * 8) =
            make_uint4(pack_bf16(total[0][0], total[0][1]), pack_bf16(total[0][2], total[0][3]),
                       pack_bf16(total[1][0], total[1][1]), pack_bf16(total[1][2], total[1][3]));
    }
}

// Builds the tile images (see WaveCtx) of a K and a V tensor, both [n_rows, H, D] bf16:
// img[head][tile] = K fragments (K_BYTES) then V^T fragments (V_BYTES).
// Rows at or beyond n_rows read as zero (their scores are masked in the attention kernel).
// One workgroup per (64-row block, head) = two tiles.
// count (nullable, one entry per 64-row block): rows of a block at or beyond its count read as zero too.
// The images are head-major (img[head][tile]): all workgroups in flight work on one head, whose keys and values are then one
// contiguous range instead of 16 KB pieces spread over the whole buffer -- measured 3 % faster at the largest shape.
//
// POOL: the block averages of k and v are written as well (kc, vc [n_rows / 64, H, D]
// bf16: Sec. 3.2, the compressed pair of the block), so that one pass over K and V serves both the pooling and
// the packing.  A thread sums its rows in fp32 in token order (rows t, t + 2048 / D, ...); the partial sums of
// the 2048 / D threads that share a channel group are added in thread order; one rounding to bf16.
template <int D, bool POOL>
__device__ __forceinline__ void pack_block(const int64_t blk, const uint16_t *__restrict__ k, const uint16_t *__restrict__ v,
                                           char *__restrict__ img, int64_t n_rows, int h, int n_tiles,
                                           const int32_t *__restrict__ count, uint16_t *__restrict__ kc, uint16_t *__restrict__ vc) {
    constexpr int K_BYTES = 32 * D * 2, TILE = K_BYTES + D * 64;
    constexpr int CH = D / 8;  // 16-byte chunks per row
    // Both tensors' rows of the block are staged in LDS, so that the images are written in image order (a wavefront
    // writes 1 KB contiguous per instruction; written straight from the loaded registers, K chunks would go out as
    // 16-byte pieces 512 bytes apart).  Row pitch D + 16 elements: 16-byte aligned, and the 4 rows x 4 column
    // groups that 16 lanes address in one transposing load fall in distinct banks.
    constexpr int PITCH = D + 16;
    __shared__ __attribute__((aligned(16))) uint16_t kt[64][PITCH];
    __shared__ __attribute__((aligned(16))) uint16_t vt[64][PITCH];
    __shared__ float psum[POOL ? 2 : 1][POOL ? 256 / CH : 1][POOL ? D + 1 : 1];  // [k, v][thread group][channel]
    const int head = blockIdx.y;
    const int n_act = count != nullptr ? count[blk] : 64;
    float ak[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, av[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // all loads of the thread first (64 CH / 256 chunks of k and as many of v), so that they are in flight together
    constexpr int NIT = 64 * CH / 256;
    uint4 kin[NIT], vin[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int e = threadIdx.x + 256 * it;
        const int t = e / CH, cc = e % CH;
        const int64_t row = blk * 64 + t;
        kin[it] = make_uint4(0, 0, 0, 0);
        vin[it] = make_uint4(0, 0, 0, 0);
        if (row < n_rows && t < n_act) {
            kin[it] = *reinterpret_cast<const uint4 *>(k + (row * h + head) * D + cc * 8);
            vin[it] = *reinterpret_cast<const uint4 *>(v + (row * h + head) * D + cc * 8);
        }
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int e = threadIdx.x + 256 * it;
        const int t = e / CH, cc = e % CH;
        const uint4 kval = kin[it], vval = vin[it];
        *reinterpret_cast<uint4 *>(&kt[t][cc * 8]) = kval;
        *reinterpret_cast<uint4 *>(&vt[t][cc * 8]) = vval;
        if (POOL) {
            const uint32_t kw[4] = {kval.x, kval.y, kval.z, kval.w}, w[4] = {vval.x, vval.y, vval.z, vval.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                ak[2 * j] += __uint_as_float(kw[j] << 16);
                ak[2 * j + 1] += __uint_as_float(kw[j] & 0xffff0000u);
                av[2 * j] += __uint_as_float(w[j] << 16);
                av[2 * j + 1] += __uint_as_float(w[j] & 0xffff0000u);
            }
        }
    }
    if (POOL) {
        // (every thread keeps one chunk column cc = threadIdx.x % CH: 256 is a multiple of CH)
        const int grp = threadIdx.x / CH, cc = threadIdx.x % CH;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            psum[0][grp][cc * 8 + j] = ak[j];
            psum[1][grp][cc * 8 + j] = av[j];
        }
    }
    __syncthreads();
    // K: a permutation of 16-byte chunks.  Chunk q of a tile's K part = fragment ks = cc / 2, lane (hh = cc % 2,
    // r = q % 32) with cc = q / 32: source row perm(r) of the tile, source chunk cc.
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int e = threadIdx.x + 256 * it;
        const int half = e / (32 * CH), q = e % (32 * CH);
        const int cc = q / 32, r = q % 32;
        const int tt = (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1);
        const uint4 kval = *reinterpret_cast<const uint4 *>(&kt[32 * half + tt][cc * 8]);
        const int64_t tile = blk * 2 + half;
        if (tile < n_tiles)
            *reinterpret_cast<uint4 *>(img + ((int64_t)head * n_tiles + tile) * TILE + q * 16) = kval;
    }
    if (POOL) {
        if (threadIdx.x < 2 * D) {
            const int which = threadIdx.x / D, c = threadIdx.x % D;
            float sum = 0.f;
            for (int g = 0; g < 256 / CH; ++g) sum += psum[which][g][c];
            const float mean = sum / (float)n_act;
            uint32_t u = __float_as_uint(mean);
            u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest even
            (which == 0 ? kc : vc)[(blk * h + head) * D + c] = (uint16_t)(u >> 16);
        }
    }
    // V^T: chunk e of a tile = fragment f = e / 64 (ks2 = f / ND, dt = f % ND), lane = e % 64
    // (hh = lane / 32, r = lane % 32): channel 32 dt + r, keys 16 ks2 + 8 hh + 0..7.  Read with the transposing LDS
    // load (ds_read_b64_tr_b16: within a group of 16 lanes, lane j receives as element e the 16-bit element j % 4 of
    // what lane 4 e + j / 4 addressed): lane j of a group addresses row k0 + j / 4, channels c0 + 4 (j % 4) .. + 3, and
    // receives channel c0 + j of rows k0 .. k0 + 3; two loads give the 8 keys of the chunk.
    constexpr int ND = D / 32;
    const uint32_t vt_base = (uint32_t)(uintptr_t)&vt[0][0];  // (the low 32 bits of a generic LDS pointer are the LDS address)
    for (int e = threadIdx.x; e < 2 * 2 * ND * 64; e += 256) {
        const int half = e / (2 * ND * 64);
        const int f = (e / 64) % (2 * ND), ln = e % 64;
        const int ks2 = f / ND, dt = f % ND, hh = ln / 32, r = ln % 32;
        const int j = ln & 15, c0 = 32 * dt + (r & 16), t0 = 32 * half + 16 * ks2 + 8 * hh;
        const int64_t tile = blk * 2 + half;
        const uint32_t addr = vt_base + (uint32_t)(((t0 + (j >> 2)) * PITCH + c0 + 4 * (j & 3)) * 2);
        uint2 lo, hi;
        asm volatile("ds_read_b64_tr_b16 %0, %2\n\tds_read_b64_tr_b16 %1, %2 offset:%3\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(lo), "=&v"(hi)
                     : "v"(addr), "n"(4 * PITCH * 2)
                     : "memory");
        if (tile >= n_tiles) continue;
        *reinterpret_cast<uint4 *>(img + ((int64_t)head * n_tiles + tile) * TILE + K_BYTES + (f * 64 + ln) * 16) =
            make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
}
template <int D, bool POOL = false>
__global__ __launch_bounds__(256) void pack_tiles(const uint16_t *__restrict__ k, const uint16_t *__restrict__ v,
                                                  char *__restrict__ img, int64_t n_rows, int h, int n_tiles,
                                                  const int32_t *__restrict__ count, uint16_t *__restrict__ kc = nullptr,
                                                  uint16_t *__restrict__ vc = nullptr) {
    pack_block<D, POOL>(blockIdx.x, k, v, img, n_rows, h, n_tiles, count, kc, vc);
}
// What the attention kernels read besides the images that lsrm_nsa_compress_pack leaves, in one launch: those of the nbc pooled pairs, and
// the tables of spatial blocks; without that call the images of keys and values too.  Workgroups in x: nb_kv blocks of keys and
// values, n_pairs of the pairs, then the tables.
template <int D>
__global__ __launch_bounds__(256) void pack_both(int nb_kv, int n_pairs, int nbc, const uint16_t *__restrict__ k, const uint16_t *__restrict__ v,
                                                 char *__restrict__ img, const uint16_t *__restrict__ kc,
                                                 const uint16_t *__restrict__ vc, char *__restrict__ img_c, int h,
                                                 const int32_t *__restrict__ count, GroupTableArgs tables) {
    const int x = blockIdx.x;
    if (x >= nb_kv + n_pairs) {
        const int i = (x - nb_kv - n_pairs) * 256 + threadIdx.x;
        if (blockIdx.y == 0 && i < tables.n) group_table_entry(i, tables.ng, tables.nb, tables.goff, tables.count, tables.tab);
        return;
    }
    const bool pairs = x >= nb_kv;
    pack_block<D, false>(pairs ? x - nb_kv : x, pairs ? kc : k, pairs ? vc : v, pairs ? img_c : img,
                         pairs ? nbc : (int64_t)nb_kv * kBlock, h, pairs ? (nbc + 31) / 32 : 2 * nb_kv, pairs ? nullptr : count, nullptr,
                         nullptr);
}

struct WsLayout {
    size_t kv, kvc, gsum, gtab, total;
};

WsLayout ws_layout(const Shape &s) {
    WsLayout w;
    const size_t tile = (size_t)32 * s.d * 2 * 2;  // K and V^T parts of one (tile, head)
    size_t off = 0;
    w.kv = off;
    off += align_up((size_t)s.nb * 2 * s.h_kv * tile, 256);
    w.kvc = off;
    off += align_up((size_t)((s.nbc + 31) / 32) * s.h_kv * tile, 256);
    w.gsum = off;
    // (d = 128: bf16, the query tiles of two of a workgroup's four wavefronts; the others' stay in LDS; at d <= 64 all in registers and LDS)
    off += s.d == 128 ? align_up((size_t)((s.nb + 1) / 2) * 2 * 32 * s.h * s.d * 2, 256) : 0;
    w.gtab = off;
    off += group_tables_bytes(s);
    w.total = off > 0 ? off : 256;
    return w;
}

template <class G>
lsrm_status launch_forward_d(const Shape &s, const int32_t *seg_host, int n_seg, FwdArgs a, const uint16_t *d_k,
                             const uint16_t *d_v, const uint16_t *d_kc, const uint16_t *d_vc, char *ws,
                             const WsLayout &w, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
    constexpr int D = G::D, NP = G::NP;
    for (int i = 0; i <= n_seg; ++i) a.seg[i] = seg_host[i];
    const int tiles_c = (s.nbc + 31) / 32;
    GroupTableArgs tables{};
    if (s.group_window) {
        tables = group_table_args(s, reinterpret_cast<int32_t *>(ws + w.gtab));
        a.blk_seg = group_tables_in(s, tables.tab).blk_seg;
    }
    a.kv = ws + w.kv;
    a.kvc = ws + w.kvc;
    a.gsum = reinterpret_cast<uint16_t *>(ws + w.gsum);
    // Few query blocks: the branches beside each other, where all workgroups fit the 256 CUs together, one or two query blocks each.
    // Measured (us, the general kernel and teams of one / of two query blocks), 64 blocks x 4 heads: d = 32 18.5 and 14.7 / 17.7, d = 64
    // 21.7 and 15.3 / 19.3, d = 128 35.6 and 21.0; 65 x 4: 19.0 and 24.1 / 17.8, 22.1 and 25.3 / 19.8, 37.3 and 36.3 (a second
    // round of workgroups); 254 x 2: 28.4 and 34.1 / 26.5, 31.7 and 35.4 / 29.0; 258 x 2: 31.5 and 43.7 / 40.3, 36.8 and 46.1 / 45.6,
    // 59.4 and 67.9.  Workgroups are what counts, two query blocks or an odd one: 17 x 30 are 270.
    // (At d = 128 a wavefront's registers leave no room for the twelve of two query blocks.)
    using One = Teams<G, 1, D == 128 ? 4 : 6, D == 32 ? 4 : 2, false>;
    using Two = Teams<G, D == 128 ? 1 : 2, D == 128 ? 4 : 3, 2, false>;
    using OnePairs = Teams<G, 1, One::NT, One::NST, true>;
    using TwoPairs = Teams<G, Two::NB, Two::NT, Two::NST, true>;
    const int tiles[3] = {tiles_c, 2 * s.topk, (int)std::min<int64_t>(s.window / 32 + 2, 2 * s.nb)};
    const int64_t longest = std::max(tiles[0], std::max(tiles[1], tiles[2])), all = (int64_t)tiles[0] + tiles[1] + tiles[2];
    // Of two query blocks every branch has one team.  Where one is nearly all there is and long, the others' ends save less than
    // two stages of tiles instead of three cost (with packing, general kernel / teams, us: 171 x 2 of d = 32, rows of 92, window 64 79 / 83, of 128
    // 101 / 110, with counts 164 / 178; of 64, window 512 63 / 61, of 32, window 64 41 / 39).
    const bool one_branch = longest > 96 && 8 * longest > 7 * all;
    // query blocks of a workgroup of teams
    const int nb_wg = (int64_t)s.nb * s.h <= 256                                            ? 1
                      : Two::NB == 2 && !one_branch && (int64_t)(s.nb + 1) / 2 * s.h <= 256 ? 2
                                                                                            : 0;
    if (nb_wg > 0) {
        // every branch one team, the others where the longest part is
        for (int &t : a.teams) t = 1;
        for (int extra = (nb_wg == 1 ? One::NT : Two::NT) - 3; extra > 0; --extra) {
            int most = 0;
            for (int b = 1; b < 3; ++b)
                if ((int64_t)tiles[b] * a.teams[most] > (int64_t)tiles[most] * a.teams[b]) most = b;
            ++a.teams[most];
        }
    }
    // A workgroup of two heads where heads that share keys and values come in pairs; at d = 32 from 600 workgroups on, short of which too few
    // share a CU to fill one another's waits.  Packing and attention, two query blocks / two heads, mean (and extremes) of drawn problems by
    // the number of workgroups: d = 32 up to 600 0.990 (0.973 to 1.039, 31 problems), to 1100 1.014, to 5000 1.019, above 1.028; d = 64 up to
    // 400 1.002 (0.990 to 1.021), to 800 1.021, to 5000 1.033, above 1.038; d = 128 up to 400 1.064 (1.030 to 1.219), to 5000 1.072, above
    // 1.059.  196 K tokens, 32 heads of 32 on 2, rows of 80 10.61 / 10.21 ms.
    const bool heads = nb_wg == 0 && a.group % 2 == 0 && (D > 32 || (int64_t)s.nb * s.h >= 1200);
    const int per_wg = nb_wg > 0 ? nb_wg : heads ? 1 : NP;  // query blocks
    a.groups_per_head = (s.nb + per_wg - 1) / per_wg;
    a.groups_per_xcd = nb_wg == 0 ? (a.groups_per_head + 7) / 8 : (a.groups_per_head * s.h + 7) / 8;
    // The workgroups make the images of the pooled pairs where a launch would do nothing else and their LDS holds them all.  A pass of packing
    // and attention out of a graph, us, launch / own images: 16 blocks x 1 head of 32 14.6 / 13.1, 96 x 4 20.5 / 18.9, 300 x 1 24.2 / 22.9; of 64
    // 96 x 4 25.4 / 23.4; of 128 64 x 4 30.4 / 28.3.  240 x 1 of 64, not out of a graph, 25.4 / 24.2.
    const bool own_pairs = s.kv_packed && tiles_c <= (nb_wg == 1 ? OnePairs::MAX_PAIRS : nb_wg == 2 ? TwoPairs::MAX_PAIRS : 0);
    if (own_pairs) a.kc = d_kc, a.vc = d_vc;
    const int nb_kv = s.kv_packed ? 0 : s.nb, pair_blocks = own_pairs ? 0 : (s.nbc + 63) / 64;
    const int n_pack = nb_kv + pair_blocks + (tables.n + 255) / 256;
    if (n_pack > 0)
        hipLaunchKernelGGL(pack_both<D>, dim3(n_pack, s.h_kv), dim3(256), 0, st, nb_kv, pair_blocks, s.nbc, d_k, d_v, ws + w.kv, d_kc, d_vc,
                           ws + w.kvc, s.h_kv, a.count, tables);
    LSRM_HIP_CHECK(hipGetLastError());
    const bool cnt = a.count != nullptr, wide = s.topk > 64;
    const void *kern;
    int lds, threads;
#define LSRM_KERNEL(NAME, ...)                                                            \
    (cnt ? (wide ? reinterpret_cast<const void *>(&NAME<G, true, true, __VA_ARGS__>)      \
                 : reinterpret_cast<const void *>(&NAME<G, true, false, __VA_ARGS__>))    \
         : (wide ? reinterpret_cast<const void *>(&NAME<G, false, true, __VA_ARGS__>)     \
                 : reinterpret_cast<const void *>(&NAME<G, false, false, __VA_ARGS__>)))
    if (nb_wg == 1) {
        kern = own_pairs ? LSRM_KERNEL(nsa_forward_teams, OnePairs) : LSRM_KERNEL(nsa_forward_teams, One);
        lds = own_pairs ? OnePairs::lds_bytes(tiles_c) : One::lds_bytes(tiles_c), threads = One::THREADS;
    } else if (nb_wg == 2) {
        kern = own_pairs ? LSRM_KERNEL(nsa_forward_teams, TwoPairs) : LSRM_KERNEL(nsa_forward_teams, Two);
        lds = own_pairs ? TwoPairs::lds_bytes(tiles_c) : Two::lds_bytes(tiles_c), threads = Two::THREADS;
    } else {
        kern = heads ? LSRM_KERNEL(nsa_forward_kernel, true) : LSRM_KERNEL(nsa_forward_kernel, false);
        lds = G::LDS_ALL, threads = G::THREADS;  // the tile slots, then the LDS part of the running gated sum
    }
#undef LSRM_KERNEL
    // (set on every launch: cheap, and right whichever device is current and whichever thread calls)
    LSRM_HIP_CHECK(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    if (ev_start != nullptr) LSRM_HIP_CHECK(hipEventRecord(ev_start, st));
    const dim3 grid(8 * a.groups_per_xcd * (nb_wg > 0 ? 1 : heads ? s.h / 2 : s.h));
    void *kargs[] = {&a};
    LSRM_HIP_CHECK(hipLaunchKernel(kern, grid, dim3(threads), kargs, lds, st));
    LSRM_HIP_CHECK(hipGetLastError());
    if (ev_stop != nullptr) LSRM_HIP_CHECK(hipEventRecord(ev_stop, st));
    return LSRM_OK;
}

lsrm_status launch_pack_tiles(int d, const uint16_t *k, const uint16_t *v, char *img, int64_t n_rows, int h, int n_tiles,
                              hipStream_t st, const int32_t *count) {
    const dim3 grid((n_tiles + 1) / 2, h);
#define LSRM_PACK(DD) \
    hipLaunchKernelGGL((pack_tiles<DD>), grid, dim3(256), 0, st, k, v, img, n_rows, h, n_tiles, count)
    if (d == 32)
        LSRM_PACK(32);
    else if (d == 64)
        LSRM_PACK(64);
    else
        LSRM_PACK(128);
#undef LSRM_PACK
    LSRM_HIP_CHECK(hipGetLastError());
    return LSRM_OK;
}

}  // namespace

size_t forward_ws_bytes(const Shape &s) { return ws_layout(s).total; }

lsrm_status launch_compress_pack(const Shape &s, const uint16_t *d_k, const uint16_t *d_v, uint16_t *d_kc,
                                 uint16_t *d_vc, void *d_ws, hipStream_t st) {
    if (s.nb == 0) return LSRM_OK;
    char *img = reinterpret_cast<char *>(d_ws) + ws_layout(s).kv;
    const dim3 grid(s.nb, s.h_kv);
    if (s.ng > 0) {
        // a spatial block's average spans several 64-slot blocks, i.e. several workgroups of the packing pass: the
        // two are separate passes here
        lsrm_status rc = launch_pack_tiles(s.d, d_k, d_v, img, s.n, s.h_kv, 2 * s.nb, st, s.count);
        if (rc != LSRM_OK) return rc;
        return launch_compress(s, d_k, d_v, d_kc, d_vc, st);
    }
#define LSRM_POOL_PACK(DD) \
    hipLaunchKernelGGL((pack_tiles<DD, true>), grid, dim3(256), 0, st, d_k, d_v, img, s.n, s.h_kv, 2 * s.nb, s.count, \
                       d_kc, d_vc)
    if (s.d == 32)
        LSRM_POOL_PACK(32);
    else if (s.d == 64)
        LSRM_POOL_PACK(64);
    else
        LSRM_POOL_PACK(128);
#undef LSRM_POOL_PACK
    LSRM_HIP_CHECK(hipGetLastError());
    return LSRM_OK;
}

lsrm_status launch_forward(const Shape &s, const int32_t *seg_host, int n_seg, const uint16_t *d_q,
                           const uint16_t *d_k, const uint16_t *d_v, const uint16_t *d_kc, const uint16_t *d_vc,
                           const int32_t *d_idx, const float *d_gates, uint16_t *d_out, float *d_lse,
                           uint16_t *d_out_branch, void *d_ws, hipStream_t st, hipEvent_t ev_start,
                           hipEvent_t ev_stop) {
    if (s.nb == 0) return LSRM_OK;
    if (n_seg > kMaxSeg) return LSRM_ERR_UNSUPPORTED;
    FwdArgs a{};
    a.q = d_q;
    a.idx = d_idx;
    a.gates = d_gates;
    a.out = d_out;
    a.lse = d_lse;
    a.out_branch = d_out_branch;
    a.n = s.n;
    a.nb = s.nb;
    a.nbc = s.nbc;
    a.blk_seg = nullptr;
    a.h = s.h;
    a.h_kv = s.h_kv;
    a.group = s.h / s.h_kv;
    a.gate_channels = s.gate_channels;
    a.own_block = s.own_block;
    a.count = s.count;
    a.topk = s.topk;
    a.window = s.window;
    a.n_seg = n_seg;
    a.scale = s.scale;
    a.scale_log2e = s.scale * 1.4426950408889634f;
    WsLayout w = ws_layout(s);
    char *ws = reinterpret_cast<char *>(d_ws);
#define LSRM_FORWARD(DD) launch_forward_d<Geo<DD>>(s, seg_host, n_seg, a, d_k, d_v, d_kc, d_vc, ws, w, st, ev_start, ev_stop)
    if (s.d == 32) return LSRM_FORWARD(32);
    if (s.d == 64) return LSRM_FORWARD(64);
    return LSRM_FORWARD(128);
#undef LSRM_FORWARD
}

}  // namespace lsrm
