// 3D-aware block routing on gfx950 (Sec. 3.3 of the paper, block-level reading).
//
// Kernels:
//   project_blocks  one workgroup per sixteen object blocks: centroid of their 64 positions, then
//                   its pinhole projection (u, v) into every view.
//   select_topk     one 256-thread workgroup per query block (object block or image
//                   tile): evaluates the squared 2-D distance to every candidate once
//                   (keys parked in LDS) and extracts the K smallest (distance, id)
//                   keys: K rounds of a minimum per wave, then a merge of the four lists.
//   select_topk_few the two in one, for few object blocks: a workgroup projects what its query needs.
// and, for the four selection rules (volume/image query -> volume/image blocks):
//   block_points    one workgroup per sixteen blocks of either modality: centroid of their 64 points.
//   select_3d       one 256-thread workgroup per query block: a wave per view projects the
//                   query point, keeps the B^i tiles with the nearest 2-D centres and
//                   measures each one's point set (64 lanes = 64 points, minimum squared 3-D
//                   distance); the workgroup then extracts the nearest volume blocks by
//                   centre distance and the nearest of the surviving tiles.
//   select_3d_many  the same for many queries (per token): 16 lanes a query.
// The whole file is built with floating-point contraction off: every product and sum
// below is rounded to fp32 exactly as written, which is what makes the indices
// reproducible bit for bit.  Plain ALU work, latency bound and tiny next to attention.
#include "lsrm_internal.h"

#include <mutex>

// Fixed scratch of lsrm_route_blocks_static, the entry point for callers that cannot allocate: the
// projections project_blocks hands to select_topk ([n_obj/64, n_views] float2).  One copy per GPU, held
// until the process ends.  In host code this name is only a handle for hipGetSymbolAddress -- never a
// device address; kernels receive the address looked up in static_scratch() below.
static __device__ __align__(256) unsigned char scratch[LSRM_STATIC_ROUTE_SCRATCH_BYTES];

namespace lsrm {

namespace {

// Pinhole projection of (cx, cy, cz) in patch units; x = +inf marks a point at or behind the
// image plane (infinitely far from every tile of that view).
__device__ __forceinline__ float2 project(const lsrm_camera &c, float cx, float cy, float cz) {
    float x = ((c.R[0] * cx + c.R[1] * cy) + c.R[2] * cz) + c.t[0];
    float y = ((c.R[3] * cx + c.R[4] * cy) + c.R[5] * cz) + c.t[1];
    float z = ((c.R[6] * cx + c.R[7] * cy) + c.R[8] * cz) + c.t[2];
    float2 r;
    if (!(z > 1e-6f)) {
        r.x = __builtin_inff();
        r.y = 0.0f;
    } else {
        r.x = c.fx * (x / z) + c.cx;
        r.y = c.fy * (y / z) + c.cy;
    }
    return r;
}

// Centroids of blocks b0 .. b0 + n - 1 (n <= kCentBlocks) into cent[.][0..2], by a workgroup of 256 threads: the points come
// in whole lines into LDS, then a thread per (block, coordinate) adds its 64 values left to right.  Bound by latency:
// with one thread per block that loaded its 192 floats itself, 768 bytes apart from its neighbours', the whole kernel
// waited for strided loads (4096 blocks into 18 views 20 -> 4 us; a whole forward step of 6 K tokens
// 34.8 -> 33.1 us, four-rule routing of 57 K tokens 303 -> 298 us).  The pitch of 195 puts the 48 threads of the sum in 48 banks.
// point_at(b) = the first coordinate of block b.
constexpr int kCentBlocks = 16, kCentPitch = 3 * kBlock + 3;
template <class PointAt>
__device__ __forceinline__ void block_centroids(int b0, int n, PointAt point_at, float (&cent)[kCentBlocks][3]) {
    __shared__ float pts[kCentBlocks * kCentPitch];
    const int tid = threadIdx.x;
    float v[kCentBlocks * 3 * kBlock / 256];
#pragma unroll
    for (int u = 0; u < kCentBlocks * 3 * kBlock / 256; ++u) {
        const int i = u * 256 + tid, b = i / (3 * kBlock);
        v[u] = b < n ? point_at(b0 + b)[i % (3 * kBlock)] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kCentBlocks * 3 * kBlock / 256; ++u) {
        const int i = u * 256 + tid;
        pts[i / (3 * kBlock) * kCentPitch + i % (3 * kBlock)] = v[u];
    }
    __syncthreads();
    if (tid < 3 * kCentBlocks) {
        const float *p = pts + tid / 3 * kCentPitch + tid % 3;
        float s = p[0];
#pragma unroll 16
        for (int t = 1; t < kBlock; ++t) s = s + p[3 * t];
        cent[tid / 3][tid % 3] = s * (1.0f / 64.0f);
    }
    __syncthreads();
}

__global__ __launch_bounds__(256) void project_blocks(int nb_obj, int n_views, const float *__restrict__ pos,
                                                      const lsrm_camera *__restrict__ cams,
                                                      float2 *__restrict__ uv /* [nb_obj, n_views] */) {
    __shared__ float cent[kCentBlocks][3];
    const int b0 = blockIdx.x * kCentBlocks, n = min(kCentBlocks, nb_obj - b0);
    block_centroids(b0, n, [&](int b) { return pos + (size_t)b * kBlock * 3; }, cent);
    for (int i = threadIdx.x; i < n * n_views; i += 256) {
        const float *c = cent[i / n_views];
        uv[(size_t)b0 * n_views + i] = project(cams[i % n_views], c[0], c[1], c[2]);
    }
}

__device__ __forceinline__ float dist2(float2 p, int ti, int tj) {
    if (__builtin_isinf(p.x) && p.x > 0.0f) return __builtin_inff();
    float ut = (float)(8 * tj + 4);
    float vt = (float)(8 * ti + 4);
    float du = p.x - ut;
    float dv = p.y - vt;
    float d2 = du * du + dv * dv;
    if (d2 != d2) d2 = __builtin_inff();
    return d2;
}

// 64-bit selection key: non-negative fp32 bit patterns order like unsigned integers, so
// (distance bits, candidate id) compares lexicographically as one integer.
__device__ __forceinline__ unsigned long long make_key(float d2, unsigned id) {
    return ((unsigned long long)__float_as_uint(d2) << 32) | id;
}

// Wave-wide minima without the LDS crossbar: four data-parallel-primitive steps fold each row of
// 16 lanes (lane xor 1, xor 2, mirror within 8, mirror within 16), then the four row results are
// read as scalars.  All 64 lanes must be active.  The result is wave-uniform.
template <class Op>
__device__ __forceinline__ unsigned row_fold(unsigned v, Op op) {
    v = op(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
    v = op(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
    v = op(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));  // row_half_mirror
    v = op(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));  // row_mirror
    return v;
}

__device__ __forceinline__ unsigned wave_min_u32(unsigned v) {
    v = row_fold(v, [](unsigned a, unsigned b) { return a < b ? a : b; });
    unsigned r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
    unsigned r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
    unsigned a = r0 < r1 ? r0 : r1, b = r2 < r3 ? r2 : r3;
    return a < b ? a : b;
}

// Non-negative floats order like their bit patterns.
__device__ __forceinline__ float wave_min_nonneg_f32(float v) { return __uint_as_float(wave_min_u32(__float_as_uint(v))); }

__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
    const unsigned hi = (unsigned)(v >> 32), lo = (unsigned)v;
    const unsigned hi_min = wave_min_u32(hi);
    // one lane holds it, unless distances tie: no second fold then
    const unsigned long long at = __ballot(hi == hi_min);
    const unsigned lo_min = (at & (at - 1)) == 0 ? (unsigned)__builtin_amdgcn_readlane(lo, __builtin_ctzll(at))
                                                 : wave_min_u32(hi == hi_min ? lo : 0xffffffffu);
    return ((unsigned long long)hi_min << 32) | lo_min;
}

constexpr unsigned long long kNoKey = ~0ull;

// What a lane holds of a set of distinct keys (none equal to all-ones) whose smallest are taken one by one: the two
// smallest of its own candidates me, me + step, ... below n_cand that were not taken yet.  Only the lane that owned the
// taken key and has none left rescans, which serialises the wave (never, up to two candidates per lane).
struct LaneKeys {
    unsigned long long mine, next;

    template <class KeyAt>
    __device__ __forceinline__ void scan(int me, int step, int n_cand, KeyAt key_at, bool have_floor,
                                         unsigned long long floor_key) {
        mine = next = kNoKey;
        for (int c = me; c < n_cand; c += step) {
            // (selects, no branches: written with branches the two keys were once kept in scratch memory)
            unsigned long long key = key_at(c);
            key = have_floor && key <= floor_key ? kNoKey : key;
            const unsigned long long larger = key < mine ? mine : key;
            mine = key < mine ? key : mine;
            next = larger < next ? larger : next;
        }
    }
    template <class KeyAt>
    __device__ __forceinline__ void take(unsigned long long best, int me, int step, int n_cand, KeyAt key_at) {
        if (mine != best) return;
        if (next != kNoKey || n_cand <= 2 * step) {
            mine = next;
            next = kNoKey;
        } else {
            scan(me, step, n_cand, key_at, true, best);
        }
    }
};

// The k smallest of a set of distinct keys (none equal to all-ones), in ascending order, found by
// one wave: lane l looks at candidates first + l', first + l' + step, ... below n_cand, where l' is
// `me` (the lane id for a wave working alone, the thread id when the four waves of a workgroup
// each take a quarter).  A round is one wave-wide minimum.  emit(r, key) is called by every lane for
// r = 0 .. count-1; returns count.
template <class KeyAt, class Emit>
__device__ __forceinline__ int wave_extract(int me, int step, int n_cand, KeyAt key_at, int k, Emit emit) {
    LaneKeys held;
    held.scan(me, step, n_cand, key_at, false, 0);
    int n = 0;
    for (; n < k; ++n) {
        const unsigned long long best = wave_min_u64(held.mine);
        if (best == kNoKey) break;
        emit(n, best);
        held.take(best, me, step, n_cand, key_at);
    }
    return n;
}

// The k smallest of n_cand distinct keys (all-ones: no candidate), by one wave that counts, for each key, the smaller
// ones: put(r, key) is called by the lane that holds the key of rank r.  Returns the number of keys put.  About four
// instructions per 64 pairs of keys, no chain from one result to the next.
template <class KeyAt, class Put>
__device__ __forceinline__ int wave_rank(int lane, int n_cand, KeyAt key_at, int k, Put put) {
    int n = 0;
    for (int c0 = 0; c0 < n_cand; c0 += 64) {
        const unsigned long long key = c0 + lane < n_cand ? key_at(c0 + lane) : kNoKey;
        int rank = 0;
#pragma unroll 4
        for (int j = 0; j < n_cand; ++j) rank += key_at(j) < key ? 1 : 0;
        if (key != kNoKey && rank < k) put(rank, key);
        n += __popcll(__ballot(key != kNoKey));
    }
    return n < k ? n : k;
}

// Top-k over the whole workgroup (256 threads): every wave extracts the k smallest keys of its
// quarter into `stage` (LDS, 4 * k entries), then every key finds its place among all four lists -- its own position
// plus the number of smaller keys in each of the others, by bisection -- and the lane that holds it calls put(r, key).
// (One wave that extracted the k smallest of the 4 k again took as long as the first step, the others idle.)
// Bound by instructions issued; with LaneKeys, wave_rank and the tile keys kept between picks: four-rule routing of 57 K
// tokens, 8 of 512 volume blocks and 24 tiles of 6 views each, 493 -> 302 us.
// Returns, in wave 0 only, the number of keys put; the other waves get -1 and have nothing left to do for this list.
template <class KeyAt, class Put>
__device__ __forceinline__ int wg_topk(int n_cand, KeyAt key_at, int k, unsigned long long *stage, Put put) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long *mine = stage + (size_t)wave * k;
    int n = wave_extract(threadIdx.x, 256, n_cand, key_at, k, [&](int r, unsigned long long key) {
        if (lane == 0) mine[r] = key;
    });
    for (int r = n + lane; r < k; r += 64) mine[r] = kNoKey;
    __syncthreads();
    for (int r = lane; r < n; r += 64) {
        const unsigned long long key = mine[r];
        int rank = r;
#pragma unroll
        for (int o = 1; o < 4; ++o) {
            const unsigned long long *list = stage + (size_t)((wave + o) & 3) * k;
            int below = 0;
            for (int step = 1 << (31 - __builtin_clz(k)); step > 0; step >>= 1) {
                const int to = below + step;
                if (to <= k && list[to - 1] < key) below = to;
            }
            rank += below;
        }
        if (rank < k) put(rank, key);
    }
    if (wave != 0) return -1;
    return n_cand < k ? n_cand : k;
}

// One workgroup per query block.  The squared distances of all candidates are computed once into
// LDS (the candidate id is the array index), then extracted with wg_topk.  `cache_keys` is false
// when they do not fit: distances are then recomputed on every scan (same results, slower).
// Dynamic LDS: [n_cand floats if cache_keys, padded to 8 bytes][4 * topk keys].
// obj_uv(m): projection of an object query into view m; tile_uv(b): that of object block b into the view qm of a tile query.
template <class ObjUv, class TileUv>
__device__ __forceinline__ void select_row(int nb_obj, int n_views, int tg, int topk, int cache_keys, ObjUv obj_uv, TileUv tile_uv,
                                           unsigned long long *lds_base, int32_t *__restrict__ idx, float *__restrict__ dist2_out) {
    const int row = blockIdx.x;  // query block
    const int tpv = tg * tg;
    const int n_tiles = n_views * tpv;
    const bool obj_row = row < nb_obj;
    const int n_cand = obj_row ? n_tiles : nb_obj;
    const int id_base = obj_row ? nb_obj : 0;
    const int max_cand = nb_obj > n_tiles ? nb_obj : n_tiles;
    float *d2_cache = reinterpret_cast<float *>(lds_base);
    unsigned long long *stage = lds_base + (cache_keys ? (max_cand + 1) / 2 : 0);
    int qm = 0, qi = 0, qj = 0;
    if (!obj_row) {
        int t = row - nb_obj;
        qm = t / tpv;
        int r = t % tpv;
        qi = r / tg;
        qj = r % tg;
    }
    auto d2_of = [&](int c) {
        if (obj_row) {
            int m = c / tpv, r = c % tpv;
            return dist2(obj_uv(m), r / tg, r % tg);
        }
        return dist2(tile_uv(c, qm), qi, qj);
    };
    int32_t *idx_row = idx + (size_t)row * topk;
    float *d2_row = dist2_out ? dist2_out + (size_t)row * topk : nullptr;
    auto put = [&](int r, unsigned long long key) {
        idx_row[r] = id_base + (int)(unsigned)(key & 0xffffffffu);
        if (d2_row) d2_row[r] = __uint_as_float((unsigned)(key >> 32));
    };
    int n;
    if (cache_keys) {
        // every thread reads back only the entries it wrote itself: no barrier needed
        for (int c = threadIdx.x; c < n_cand; c += blockDim.x) d2_cache[c] = d2_of(c);
        n = wg_topk(n_cand, [&](int c) { return make_key(d2_cache[c], (unsigned)c); }, topk, stage, put);
    } else {
        n = wg_topk(n_cand, [&](int c) { return make_key(d2_of(c), (unsigned)c); }, topk, stage, put);
    }
    if (n < 0) return;
    for (int k = n + (threadIdx.x & 63); k < topk; k += 64) {  // fewer candidates than topk
        idx_row[k] = -1;
        if (d2_row) d2_row[k] = __builtin_inff();
    }
}

__global__ __launch_bounds__(256) void select_topk(int nb_obj, int n_views, int tg, int topk, int cache_keys,
                                                   const float2 *__restrict__ uv, int32_t *__restrict__ idx,
                                                   float *__restrict__ dist2_out) {
    extern __shared__ unsigned long long lds_base[];
    select_row(
        nb_obj, n_views, tg, topk, cache_keys, [&](int m) { return uv[(size_t)blockIdx.x * n_views + m]; },
        [&](int b, int m) { return uv[(size_t)b * n_views + m]; }, lds_base, idx, dist2_out);
}

// The same without project_blocks, for few object blocks: a workgroup works out the projections it needs by itself (an object
// query's own into every view, a tile query's of all blocks into its view), by the same sums.  A launch less, where that
// is most of the time: 25 blocks, 2 views 4.8 and 4.4 us and the gap between them -> 6.9 us; with 64 blocks a step of 6 K tokens gained nothing.
constexpr int kRouteFew = 32, kRouteFewRows = 256;  // object blocks (25 KB of points in LDS); queries, as every tile's reads all points
__global__ __launch_bounds__(256) void select_topk_few(int nb_obj, int n_views, int tg, int topk,
                                                       const float *__restrict__ pos, const lsrm_camera *__restrict__ cams,
                                                       int32_t *__restrict__ idx, float *__restrict__ dist2_out) {
    extern __shared__ unsigned long long lds_base[];
    __shared__ float pts[kRouteFew * kCentPitch], cent[kRouteFew][3];
    __shared__ float2 uv[kRouteFew];  // of an object query per view (as many as there are threads for, else worked out again)
    const int row = blockIdx.x, tid = threadIdx.x;
    const bool obj_row = row < nb_obj;
    const int b0 = obj_row ? row : 0, n = obj_row ? 1 : nb_obj;
    constexpr int NIT = kRouteFew * 3 * kBlock / 4 / 256;
    // (four floats in a row to a thread, loaded one by one: the array may start at any multiple of four bytes)
    float v[NIT][4];
    const float *src = pos + (size_t)b0 * kBlock * 3;
#pragma unroll
    for (int u = 0; u < NIT; ++u) {
        const int i = 4 * (u * 256 + tid);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[u][j] = i < n * 3 * kBlock ? src[i + j] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < NIT; ++u) {
        const int i = 4 * (u * 256 + tid), b = i / (3 * kBlock);  // (192 is a multiple of four: one block)
        if (b < n) {
#pragma unroll
            for (int j = 0; j < 4; ++j) pts[b * kCentPitch + i % (3 * kBlock) + j] = v[u][j];
        }
    }
    __syncthreads();
    if (tid < 3 * n) {
        const float *p = pts + tid / 3 * kCentPitch + tid % 3;
        float s = p[0];
#pragma unroll 16
        for (int t = 1; t < kBlock; ++t) s = s + p[3 * t];
        cent[tid / 3][tid % 3] = s * (1.0f / 64.0f);
    }
    __syncthreads();
    const int qm = obj_row ? 0 : (row - nb_obj) / (tg * tg);
    if (obj_row ? tid < min(n_views, kRouteFew) : tid < n) {
        const float *c = cent[obj_row ? 0 : tid];
        uv[tid] = project(cams[obj_row ? tid : qm], c[0], c[1], c[2]);
    }
    __syncthreads();
    select_row(
        nb_obj, n_views, tg, topk, 1,
        [&](int m) { return m < kRouteFew ? uv[m] : project(cams[m], cent[0][0], cent[0][1], cent[0][2]); },
        [&](int b, int) { return uv[b]; }, lds_base, idx, dist2_out);
}

// ---------------------------------------------------------------- four selection rules (Sec. 3.3)

// Centroid of each block's 64 points, summed left to right.  Blocks [0, nb_obj) read `pos`,
// the others `pos_img`; the result is padded to float4.
__global__ __launch_bounds__(256) void block_points(int nb_obj, int nb, const float *__restrict__ pos,
                                                    const float *__restrict__ pos_img, float4 *__restrict__ cent) {
    __shared__ float c[kCentBlocks][3];
    const int b0 = blockIdx.x * kCentBlocks, n = min(kCentBlocks, nb - b0);
    block_centroids(
        b0, n,
        [&](int b) {
            return b < nb_obj ? pos + (size_t)b * kBlock * 3 : pos_img + (size_t)(b - nb_obj) * kBlock * 3;
        },
        c);
    if ((int)threadIdx.x < n) {
        const float *m = c[threadIdx.x];
        cent[b0 + threadIdx.x] = make_float4(m[0], m[1], m[2], 0.0f);
    }
}

__device__ __forceinline__ float sqdist3(float ax, float ay, float az, float bx, float by, float bz) {
    float dx = ax - bx, dy = ay - by, dz = az - bz;
    return (dx * dx + dy * dy) + dz * dz;
}

struct Route3d {
    int nb_obj, n_views, tg, width, prefilter, k_v2v, k_v2i, k_i2v, k_i2i, cache_keys;
    int per_token, n_obj;  // queries are tokens (point = own coordinate) instead of blocks (point = centroid)
};

// Dynamic LDS: [n_views * prefilter candidate keys][4 * max(k_v2v, k_i2v) staged keys]
// [nb_obj floats if cache_keys].
__global__ __launch_bounds__(256) void select_3d(Route3d a, const float4 *__restrict__ cent,
                                                 const float *__restrict__ pos, const float *__restrict__ pos_img,
                                                 const lsrm_camera *__restrict__ cams, int32_t *__restrict__ idx,
                                                 float *__restrict__ dist2_out) {
    extern __shared__ unsigned long long lds_base[];
    unsigned long long *img_keys = lds_base;
    unsigned long long *stage = img_keys + (size_t)a.n_views * a.prefilter;
    float *vol_d2 = reinterpret_cast<float *>(stage + 4 * (size_t)(a.k_v2v > a.k_i2v ? a.k_v2v : a.k_i2v));
    const int row = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tpv = a.tg * a.tg;
    const bool obj_row = row < (a.per_token ? a.n_obj : a.nb_obj);
    const int kv = obj_row ? a.k_v2v : a.k_i2v;
    const int ki = obj_row ? a.k_v2i : a.k_i2i;
    float4 p;
    if (a.per_token) {
        const float *q = obj_row ? pos + (size_t)row * 3 : pos_img + (size_t)(row - a.n_obj) * 3;
        p = make_float4(q[0], q[1], q[2], 0.0f);
    } else {
        p = cent[row];
    }

    // image rule, first two steps: a wave per view
    if (ki > 0) {
        for (int m = wave; m < a.n_views; m += 4) {
            const float2 uv = project(cams[m], p.x, p.y, p.z);
            unsigned long long *out = img_keys + (size_t)m * a.prefilter;
            if (dist2(uv, 0, 0) == __builtin_inff()) {  // no tile of this view is a candidate
                for (int c = lane; c < a.prefilter; c += 64) out[c] = kNoKey;
                continue;
            }
            // candidates in groups of four: pick four tiles, then fetch and measure their point sets
            // together so that the memory latency is paid once per group
            // every tile's key is worked out once (a division by the row length each), not once per pick
            auto tile_key = [&](int t) { return make_key(dist2(uv, t / a.tg, t % a.tg), (unsigned)t); };
            LaneKeys held;
            held.scan(lane, 64, tpv, tile_key, false, 0);
            for (int c0 = 0; c0 < a.prefilter; c0 += 4) {
                int tile[4];
                float d[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    tile[u] = -1;
                    if (c0 + u < a.prefilter) {
                        const unsigned long long best = wave_min_u64(held.mine);
                        held.take(best, lane, 64, tpv, tile_key);
                        tile[u] = m * tpv + (int)(unsigned)(best & 0xffffffffu);
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    d[u] = 0.0f;
                    if (tile[u] >= 0) {
                        const float *q = pos_img + ((size_t)tile[u] * kBlock + lane) * 3;
                        d[u] = sqdist3(p.x, p.y, p.z, q[0], q[1], q[2]);
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (tile[u] >= 0) {
                        float dmin = wave_min_nonneg_f32(d[u]);
                        if (lane == 0) out[c0 + u] = make_key(dmin, (unsigned)(a.nb_obj + tile[u]));
                    }
                }
            }
        }
    }

    // volume rule: per-wave extraction, every wave places its own keys (the barrier inside also publishes img_keys)
    int32_t *idx_row = idx + (size_t)row * a.width;
    float *d2_row = dist2_out ? dist2_out + (size_t)row * a.width : nullptr;
    auto vol_d2_of = [&](int j) {
        float4 c = cent[j];
        return sqdist3(p.x, p.y, p.z, c.x, c.y, c.z);
    };
    int at = 0;
    auto put = [&](int r, unsigned long long key) {
        idx_row[at + r] = (int)(unsigned)(key & 0xffffffffu);
        if (d2_row) d2_row[at + r] = __uint_as_float((unsigned)(key >> 32));
    };
    if (kv > 0) {
        int n;
        if (a.cache_keys) {
            // every thread reads back only the entries it wrote itself
            for (int j = threadIdx.x; j < a.nb_obj; j += blockDim.x) vol_d2[j] = vol_d2_of(j);
            n = wg_topk(a.nb_obj, [&](int j) { return make_key(vol_d2[j], (unsigned)j); }, kv, stage, put);
        } else {
            n = wg_topk(a.nb_obj, [&](int j) { return make_key(vol_d2_of(j), (unsigned)j); }, kv, stage, put);
        }
        if (n < 0) return;
        at = n;
    } else {
        __syncthreads();
        if (wave != 0) return;
    }
    // wave 0 alone: the image budget out of the surviving candidates, then the padding
    if (ki > 0) {
        const int n_img = a.n_views * a.prefilter;
        auto key_of = [&](int c) { return img_keys[c]; };
        // Ranking costs about 4 instructions per candidate and 64 of them, an extraction about 60 per result, one
        // waiting for the other: the line is where they are equal.
        if ((n_img + 63) / 64 * n_img <= 16 * ki)
            at += wave_rank(lane, n_img, key_of, ki, put);
        else
            at += wave_extract(lane, 64, n_img, key_of, ki, [&](int r, unsigned long long key) {
                if (lane == 0) put(r, key);
            });
    }
    for (int k = at + lane; k < a.width; k += 64) {
        idx_row[k] = -1;
        if (d2_row) d2_row[k] = __builtin_inff();
    }
}

// The same selection for many queries (57 K tokens of a scene, say): a workgroup takes kManyQueries of them that follow one
// another, 16 lanes a query, so that a minimum over a query's lanes is four data-parallel-primitive steps without a scalar
// read, four queries a wavefront side by side.  select_3d gives a workgroup to a query: chains of minima over 64
// lanes, most lanes with nothing of their own.  Bound by instructions issued (the vector pipe is busy all the time), as
// that one is, with a fifth of them per query: what several queries have in common is done once.
// 57 K tokens, 8 of 512 volume blocks and 24 tiles of 6 views each: 322 -> 87 us, 3330 -> 680 vector instructions a query; with a lane for a
// view's nearest tiles (tile_window) and four lanes for a tile's points, 570, the whole call 77.7 -> 71.8 us.
constexpr int kManyQueries = 16;
constexpr int kNearList = 128, kNearFrom = 48;  // listed blocks of a query, the largest volume budget that a list is made for
constexpr int kCommonList = 256, kCommonFrom = 256;  // listed blocks of a workgroup, the fewest blocks it is made from

// Minimum over the 16 lanes of a row; every lane of the row gets it.
__device__ __forceinline__ unsigned row_min_u32(unsigned v) {
    return row_fold(v, [](unsigned a, unsigned b) { return a < b ? a : b; });
}
__device__ __forceinline__ unsigned row_max_u32(unsigned v) {
    return row_fold(v, [](unsigned a, unsigned b) { return a > b ? a : b; });
}
__device__ __forceinline__ unsigned long long row_min_u64(unsigned long long v) {
    const unsigned hi = (unsigned)(v >> 32), lo = (unsigned)v;
    const unsigned hi_min = row_min_u32(hi);
    return ((unsigned long long)hi_min << 32) | row_min_u32(hi == hi_min ? lo : 0xffffffffu);
}

struct __attribute__((packed, aligned(4))) FourPoints {
    float v[12];
};

// The window of 4 x 4 tiles of a view around a projection in which its nearest tiles are looked for, by one lane.  Squares and sums
// round monotonically, so a tile outside the window is no nearer than `beside`, the smallest of the tiles just outside its four
// borders in the row or column of the window's smallest difference: tiles of the window that are strictly nearer than
// that are the nearest of the view.
// (A lane keeps the four nearest of the 16 in order, 20 instructions a tile for 64 projections; 16 lanes that took minima of one
// projection's tiles needed as many for four of them.)
constexpr int kNoTiles = -1, kLookAtAll = 0, kPicked = 1 << 16;
struct TileWindow {
    float u, v;
    int first;  // first row << 16 | first column
    int picks;  // kNoTiles: no tile of the view is a candidate; kLookAtAll; or kPicked and the nearest tiles, four bits each: row, column
};
__device__ __forceinline__ TileWindow tile_window(float2 uv, int tg, int prefilter) {
    TileWindow w;
    w.u = uv.x;
    w.v = uv.y;
    w.first = 0;
    w.picks = kNoTiles;
    if (dist2(uv, 0, 0) == __builtin_inff()) return w;
    w.picks = kLookAtAll;
    if (prefilter > 4) return w;
    const int top = max(tg - 4, 0);
    const float fi = floorf((fminf(fmaxf(uv.y, -1.0e6f), 1.0e6f) - 4.0f) * 0.125f);
    const float fj = floorf((fminf(fmaxf(uv.x, -1.0e6f), 1.0e6f) - 4.0f) * 0.125f);
    const int i0 = min(max((int)fi - 1, 0), top), j0 = min(max((int)fj - 1, 0), top);
    w.first = i0 << 16 | j0;
    auto du2_at = [&](int j) { const float du = uv.x - (float)(8 * j + 4); return du * du; };
    auto dv2_at = [&](int i) { const float dv = uv.y - (float)(8 * i + 4); return dv * dv; };
    float du2[4], dv2[4], du2_min = __builtin_inff(), dv2_min = __builtin_inff();
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        du2[t] = du2_at(j0 + t);
        dv2[t] = dv2_at(i0 + t);
        if (t < tg) {
            du2_min = fminf(du2_min, du2[t]);
            dv2_min = fminf(dv2_min, dv2[t]);
        }
    }
    float beside = __builtin_inff();
    if (i0 > 0) beside = fminf(beside, du2_min + dv2_at(i0 - 1));
    if (i0 + 4 < tg) beside = fminf(beside, du2_min + dv2_at(i0 + 4));
    if (j0 > 0) beside = fminf(beside, du2_at(j0 - 1) + dv2_min);
    if (j0 + 4 < tg) beside = fminf(beside, du2_at(j0 + 4) + dv2_min);
    // the four smallest, equal ones in the order of the tiles
    unsigned d[4], at[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) d[r] = 0xffffffffu, at[r] = 0;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        const unsigned x = t / 4 < tg && t % 4 < tg ? __float_as_uint(du2[t % 4] + dv2[t / 4]) : 0xffffffffu;
        bool less[4];  // (of the four in order, the first that x is less than and all behind it move on)
#pragma unroll
        for (int r = 0; r < 4; ++r) less[r] = x < d[r];
#pragma unroll
        for (int r = 3; r >= 0; --r) {
            const bool moved = r > 0 && less[r > 0 ? r - 1 : 0];
            d[r] = moved ? d[r > 0 ? r - 1 : 0] : less[r] ? x : d[r];
            at[r] = moved ? at[r > 0 ? r - 1 : 0] : less[r] ? (unsigned)t : at[r];
        }
    }
    const unsigned last = prefilter == 1 ? d[0] : prefilter == 2 ? d[1] : prefilter == 3 ? d[2] : d[3];
    if (last < __float_as_uint(beside)) w.picks = (int)(kPicked | at[0] | at[1] << 4 | at[2] << 8 | at[3] << 12);
    return w;
}

// Dynamic LDS: [Q][n_views] windows, [Q][n_views * prefilter] keys, [Q][width] ids and distances.
template <int Q>
__global__ __launch_bounds__(16 * Q) void select_3d_many(Route3d a, int n_queries, const float4 *__restrict__ cent,
                                                         const float *__restrict__ pos, const float *__restrict__ pos_img,
                                                         const lsrm_camera *__restrict__ cams, int32_t *__restrict__ idx,
                                                         float *__restrict__ dist2_out) {
    extern __shared__ unsigned long long lds_base[];
    __shared__ float4 points[Q], common[kCommonList];
    __shared__ unsigned long long near_keys[Q * kNearList];
    __shared__ int n_common;
    __shared__ unsigned wave_bound[Q / 4];
    const int n_img = a.n_views * a.prefilter;
    TileWindow *windows = reinterpret_cast<TileWindow *>(lds_base);
    unsigned long long *img_keys = reinterpret_cast<unsigned long long *>(windows + Q * a.n_views);
    int *out_idx = reinterpret_cast<int *>(img_keys + Q * n_img);
    float *out_d2 = reinterpret_cast<float *>(out_idx + Q * a.width);
    const int q0 = blockIdx.x * Q, nq = min(Q, n_queries - q0);
    const int g = threadIdx.x >> 4, l = threadIdx.x & 15, lane = threadIdx.x & 63;
    const int tpv = a.tg * a.tg, n_obj_rows = a.per_token ? a.n_obj : a.nb_obj;
    const bool any_img = a.k_v2i > 0 || a.k_i2i > 0;
    const int kv_max = max(a.k_v2v, a.k_i2v);
    if ((int)threadIdx.x < Q) {
        const int row = q0 + min((int)threadIdx.x, nq - 1);
        if (a.per_token) {
            const float *q = row < a.n_obj ? pos + (size_t)row * 3 : pos_img + (size_t)(row - a.n_obj) * 3;
            points[threadIdx.x] = make_float4(q[0], q[1], q[2], 0.0f);
        } else {
            points[threadIdx.x] = cent[row];
        }
    }
    if (threadIdx.x == 0) n_common = 0;
    for (int i = threadIdx.x; i < nq * a.width; i += 16 * Q) {
        out_idx[i] = -1;
        out_d2[i] = __builtin_inff();
    }
    __syncthreads();
    for (int i = threadIdx.x; any_img && i < nq * a.n_views; i += 16 * Q) {
        const int q = i / a.n_views;
        const float4 p = points[q];
        windows[i] = tile_window(project(cams[i - q * a.n_views], p.x, p.y, p.z), a.tg, a.prefilter);
    }

    // The volume blocks that any of the workgroup's queries can select.  With R the largest distance of a query from the
    // middle one and D a bound on that one's kv-th smallest block distance, every query has kv blocks within D + R, and
    // those lie within D + 2 R of the middle one.  (Distances are off by less than 1e-6 of themselves, far below the
    // allowance; one that is not finite leaves the list empty.)
    const bool listing = kv_max > 0 && kv_max <= kNearFrom && a.nb_obj >= kCommonFrom;
    bool listed = false;
    if (listing) {
        const float4 p0 = points[nq / 2], pl = points[l & (Q - 1)];
        const float r2 = __uint_as_float(row_max_u32(__float_as_uint(sqdist3(p0.x, p0.y, p0.z, pl.x, pl.y, pl.z))));
        auto d2_bits = [&](int j) {
            const float4 c = cent[j];
            return __float_as_uint(sqdist3(p0.x, p0.y, p0.z, c.x, c.y, c.z));
        };
        unsigned m = ~0u, bound = 0;
        for (int j = threadIdx.x; j < a.nb_obj; j += 16 * Q) m = min(m, d2_bits(j));
        for (int r = 0; r < kv_max; ++r) {  // (equal ones go together: the bound is then a larger one)
            bound = wave_min_u32(m);
            m = m == bound ? ~0u : m;
        }
        if (lane == 0) wave_bound[threadIdx.x >> 6] = bound;
        __syncthreads();
        for (int w = 0; w < Q / 4; ++w) bound = min(bound, wave_bound[w]);
        const float reach = (sqrtf(__uint_as_float(bound)) + 2.0f * sqrtf(r2)) * 1.0001f + 1.0e-17f, reach2 = reach * reach;
        if (reach2 < __builtin_inff()) {
            for (int j = threadIdx.x; j < a.nb_obj; j += 16 * Q)
                if (__uint_as_float(d2_bits(j)) <= reach2) {
                    const int at = atomicAdd(&n_common, 1);
                    if (at < kCommonList) {
                        float4 c = cent[j];
                        c.w = __int_as_float(j);
                        common[at] = c;
                    }
                }
            listed = true;
        }
    }
    __syncthreads();
    if (n_common > kCommonList) listed = false;
    if (g >= nq) return;  // (from here on a query's lanes are on their own; the last barrier is behind)

    const float4 p = points[g];
    const bool obj_row = q0 + g < n_obj_rows;
    const int kv = obj_row ? a.k_v2v : a.k_i2v, ki = obj_row ? a.k_v2i : a.k_i2i;
    unsigned long long *keys = img_keys + g * n_img;
    auto put = [&](int at, unsigned long long key) {
        out_idx[g * a.width + at] = (int)(unsigned)(key & 0xffffffffu);
        out_d2[g * a.width + at] = __uint_as_float((unsigned)(key >> 32));
    };

    // image rule, first two steps: the prefilter nearest tiles of every view by 2-D distance, then their point sets
    for (int m = 0; ki > 0 && m < a.n_views; ++m) {
        const TileWindow w = windows[g * a.n_views + m];
        unsigned long long *out = keys + m * a.prefilter;
        if (w.picks == kNoTiles) {
            for (int c = l; c < a.prefilter; c += 16) out[c] = kNoKey;
            continue;
        }
        // smallest distance of four points of a tile in a row
        auto measure = [&](int tile, int point) {
            const FourPoints pts = *reinterpret_cast<const FourPoints *>(pos_img + ((size_t)tile * kBlock + point) * 3);
            unsigned d = 0xffffffffu;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                d = min(d, __float_as_uint(sqdist3(p.x, p.y, p.z, pts.v[3 * i], pts.v[3 * i + 1], pts.v[3 * i + 2])));
            return d;
        };
        if (w.picks != kLookAtAll) {
            // four lanes a tile, 16 points each, four in a row at a time
            const int r = l >> 2, at = (w.picks >> (4 * (r < a.prefilter ? r : 0))) & 15;
            const int tile = m * tpv + ((w.first >> 16) + (at >> 2)) * a.tg + (w.first & 0xffff) + (at & 3);
            unsigned d = 0xffffffffu;
#pragma unroll
            for (int k = 0; k < 4; ++k) d = min(d, measure(tile, 16 * k + 4 * (l & 3)));
            d = min(d, (unsigned)__builtin_amdgcn_update_dpp(0, (int)d, 0xB1, 0xF, 0xF, false));  // quad_perm [1,0,3,2]
            d = min(d, (unsigned)__builtin_amdgcn_update_dpp(0, (int)d, 0x4E, 0xF, 0xF, false));  // quad_perm [2,3,0,1]
            if ((l & 3) == 0 && r < a.prefilter) out[r] = ((unsigned long long)d << 32) | (unsigned)(a.nb_obj + tile);
        } else {
            const float2 uv = make_float2(w.u, w.v);
            auto tile_key = [&](int t) { return make_key(dist2(uv, t / a.tg, t % a.tg), (unsigned)t); };
            LaneKeys held;
            held.scan(l, 16, tpv, tile_key, false, 0);
            for (int c = 0; c < a.prefilter; ++c) {
                const unsigned long long best = row_min_u64(held.mine);
                held.take(best, l, 16, tpv, tile_key);
                const int tile = m * tpv + (int)(unsigned)(best & 0xffffffffu);
                const unsigned d = row_min_u32(measure(tile, 4 * l));
                if (l == 0) out[c] = ((unsigned long long)d << 32) | (unsigned)(a.nb_obj + tile);
            }
        }
    }

    // volume rule
    const int n_vol = min(kv, a.nb_obj);
    if (n_vol > 0) {
        auto key_of = [&](int j) {
            const float4 c = cent[j];
            return ((unsigned long long)__float_as_uint(sqdist3(p.x, p.y, p.z, c.x, c.y, c.z)) << 32) | (unsigned)j;
        };
        // The blocks (those of the list, or all) are dealt to 4 x 16 sets; the kv-th smallest of the sets' smallest distances
        // bounds the kv-th smallest of all, and few blocks are below it (about 64 ln(64 / (64 - kv)) of many).  Those are listed
        // and ranked.  More of them than the list holds (equal distances, say): the blocks are taken one by one.
        int n_near = kNearList + 1;
        unsigned long long *near = near_keys + g * kNearList;
        auto narrow = [&](int n_src, auto src_key) {
            unsigned m[4] = {~0u, ~0u, ~0u, ~0u};
            for (int j0 = l; j0 < n_src; j0 += 64) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = j0 + 16 * u;
                    const unsigned x = (unsigned)(src_key(min(j, n_src - 1)) >> 32);
                    m[u] = j < n_src ? min(m[u], x) : m[u];
                }
            }
            unsigned bound = 0;
            for (int r = 0; r < kv; ++r) {  // (equal ones go together, as above)
                bound = row_min_u32(min(min(m[0], m[1]), min(m[2], m[3])));
#pragma unroll
                for (int u = 0; u < 4; ++u) m[u] = m[u] == bound ? ~0u : m[u];
            }
            n_near = 0;
            const int row_shift = threadIdx.x & 48;
            for (int j0 = l; j0 - l < n_src; j0 += 16) {
                const unsigned long long key = src_key(min(j0, n_src - 1));
                const bool on = j0 < n_src && (unsigned)(key >> 32) <= bound;
                const unsigned in_row = (unsigned)(__ballot(on) >> row_shift) & 0xffffu;
                if (in_row != 0) {
                    const int at = n_near + __popc(in_row & ((1u << l) - 1u));
                    if (on && at < kNearList) near[at] = key;
                    n_near += __popc(in_row);
                }
            }
        };
        if (listed)
            narrow(n_common, [&](int i) {
                const float4 c = common[i];
                return ((unsigned long long)__float_as_uint(sqdist3(p.x, p.y, p.z, c.x, c.y, c.z)) << 32) |
                       (unsigned)__float_as_int(c.w);
            });
        else if (kv <= kNearFrom)
            narrow(a.nb_obj, key_of);
        if (n_near <= kNearList) {
            // (LDS operations of a wavefront complete in order, and a query's lanes are in one wavefront)
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            for (int c = l; c < n_near; c += 16) {
                const unsigned long long key = near[c];
                int rank = 0;
#pragma unroll 4
                for (int j = 0; j < n_near; ++j) rank += near[j] < key ? 1 : 0;
                if (rank < n_vol) put(rank, key);
            }
        } else {
            LaneKeys held;
            held.scan(l, 16, a.nb_obj, key_of, false, 0);
            for (int r = 0; r < n_vol; ++r) {
                const unsigned long long best = row_min_u64(held.mine);
                if (l == 0) put(r, best);
                held.take(best, l, 16, a.nb_obj, key_of);
            }
        }
    }

    // image rule: the budget out of the surviving candidates
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (ki > 0) {
        // ranking costs about 4 instructions per candidate and 16 of them, an extraction about 25 per result: the line is
        // where they are equal
        if ((n_img + 15) / 16 * n_img <= 6 * ki + 64) {
            for (int c = l; c < n_img; c += 16) {
                const unsigned long long key = keys[c];
                int rank = 0;
#pragma unroll 4
                for (int j = 0; j < n_img; ++j) rank += keys[j] < key ? 1 : 0;
                if (key != kNoKey && rank < ki) put(n_vol + rank, key);
            }
        } else {
            auto key_of = [&](int c) { return keys[c]; };
            LaneKeys held;
            held.scan(l, 16, n_img, key_of, false, 0);
            for (int r = 0; r < ki; ++r) {
                const unsigned long long best = row_min_u64(held.mine);
                if (best == kNoKey) break;
                if (l == 0) put(n_vol + r, best);
                held.take(best, l, 16, n_img, key_of);
            }
        }
    }
    // the row, 64 bytes at a time
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const size_t row0 = (size_t)(q0 + g) * a.width;
    for (int i = l; i < a.width; i += 16) {
        idx[row0 + i] = out_idx[g * a.width + i];
        if (dist2_out) dist2_out[row0 + i] = out_d2[g * a.width + i];
    }
}

}  // namespace

size_t route3d_ws_bytes(const Shape &s) {
    size_t n = (size_t)s.nb * sizeof(float4);
    return align_up(n > 0 ? n : 256, 256);
}

// Whether select_3d_many is the faster one (all figures: us, select_3d / select_3d_many).
static bool many_pay(const Route3d &a, unsigned n_queries) {
    constexpr unsigned kFillsChip = 6144;  // queries, 24 for every CU, from which the slower parts below pay at all
    const int n_img = a.n_views * a.prefilter, k_vol = min(max(a.k_v2v, a.k_i2v), a.nb_obj), k_img = max(a.k_v2i, a.k_i2i);
    // A query's 16 lanes do in turn what select_3d gives to 256: many queries are needed to fill the chip, and the more
    // blocks there are to look at, or candidate tiles, the more of them.  57344 queries of 512 blocks 322 / 87, 70144 of 1024
    // 936 / 331, 12288 of 64 128 / 64, 4096 of 64 16 / 11, 1280 of 16 11 / 11; but 640 of 512 11 / 21, 3072 of 2048 57 / 80,
    // 4672 of 4096 71 / 108.  64 of 120 tiles, 4384 queries 99 / 95; of 160, 2592 queries 80 / 109.
    if (n_queries < (k_img > 0 && n_img > 64 ? 4096u : 2048u) + 2u * a.nb_obj) return false;
    // Above kNearFrom there is no list of near blocks, they are taken one by one.  Of 64 blocks 48 92 / 22, 49 94 / 46, 64 113 / 57,
    // of 256 blocks 64 317 / 279; but of 128 blocks 96 113 / 125, of 512 49 671 / 802, of 2048 49 2301 / 6544; 2656 queries of 64
    // blocks, 49 59 / 67.
    if (k_vol > kNearFrom && (k_vol > 64 || a.nb_obj > 256 || n_queries < kFillsChip)) return false;
    // Above four tiles a view there is no window, all tiles are looked at.  Eight of 64 tiles a view 410 / 212, of 144 798 / 206; but
    // of 256, four views, 323 / 505; 2320 queries, eight of 144 57 / 108, 4384, five of 144 116 / 127.
    if (k_img > 0 && a.prefilter > 4 && (a.tg > 12 || n_queries < kFillsChip)) return false;
    // Too many candidates to rank and too many results to take one by one.  64 of 144 532 / 393, 120 of 96 958 / 652; but 120
    // of 144 558 / 769.
    return k_img <= 64 || n_img <= 96;
}

lsrm_status launch_route_3d(const Shape &s, const lsrm_route3d_params &r, const float *d_pos, const float *d_pos_img,
                            const lsrm_camera *d_cams, int32_t *d_idx, float *d_dist2, void *d_ws, hipStream_t st) {
    if (s.nb == 0 || s.topk == 0) return LSRM_OK;
    float4 *cent = reinterpret_cast<float4 *>(d_ws);
    hipLaunchKernelGGL(block_points, dim3((s.nb + kCentBlocks - 1) / kCentBlocks), dim3(256), 0, st, s.nb_obj, s.nb, d_pos, d_pos_img,
                       cent);
    LSRM_HIP_CHECK(hipGetLastError());
    Route3d a;
    a.nb_obj = s.nb_obj;
    a.n_views = s.n_views;
    a.tg = s.grid / 8;
    a.width = s.topk;
    a.prefilter = r.prefilter < s.tiles_per_view ? r.prefilter : s.tiles_per_view;
    a.k_v2v = r.k_v2v;
    a.k_v2i = r.k_v2i;
    a.k_i2v = r.k_i2v;
    a.k_i2i = r.k_i2i;
    a.per_token = r.per_token;
    a.n_obj = s.n_obj;
    if (a.prefilter < 1) a.k_v2i = a.k_i2i = 0;  // no tiles at all
    const int k_vol = a.k_v2v > a.k_i2v ? a.k_v2v : a.k_i2v;
    const size_t cand_bytes = ((size_t)s.n_views * (a.prefilter > 0 ? a.prefilter : 0) + 4 * (size_t)k_vol) *
                              sizeof(unsigned long long);
    const size_t vol_bytes = (size_t)s.nb_obj * sizeof(float);
    if (cand_bytes > 36 * 1024) return LSRM_ERR_UNSUPPORTED;  // api.hip has bounded both terms below this
    a.cache_keys = vol_bytes + cand_bytes <= 60 * 1024 ? 1 : 0;
    const size_t lds = cand_bytes + (a.cache_keys ? vol_bytes : 0);
    const unsigned n_queries = r.per_token ? (unsigned)s.n : (unsigned)s.nb;
    const size_t many_lds = kManyQueries * (16 * (size_t)s.n_views + 8 * (size_t)s.n_views * a.prefilter + 8 * (size_t)s.topk);
    if (many_lds <= 40 * 1024 && many_pay(a, n_queries)) {
        hipLaunchKernelGGL(select_3d_many<kManyQueries>, dim3((n_queries + kManyQueries - 1) / kManyQueries),
                           dim3(16 * kManyQueries), many_lds, st, a, (int)n_queries, cent, d_pos, d_pos_img, d_cams, d_idx,
                           d_dist2);
        LSRM_HIP_CHECK(hipGetLastError());
        return LSRM_OK;
    }
    hipLaunchKernelGGL(select_3d, dim3(n_queries), dim3(256), lds, st, a, cent, d_pos, d_pos_img, d_cams, d_idx,
                       d_dist2);
    LSRM_HIP_CHECK(hipGetLastError());
    return LSRM_OK;
}

// Device address of `scratch` on the current device, looked up once per device (every GPU holds its
// own copy of the array at its own address).
static lsrm_status static_scratch(void **out) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = -1;
    LSRM_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return LSRM_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(mu);
    if (addr[dev] == nullptr) {
        void *ptr = nullptr;
        LSRM_HIP_CHECK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (ptr == nullptr) return LSRM_ERR_HIP;
        addr[dev] = ptr;
    }
    *out = addr[dev];
    return LSRM_OK;
}

lsrm_status launch_route_static(const Shape &s, const float *d_pos, const lsrm_camera *d_cams, int32_t *d_idx,
                                float *d_dist2, hipStream_t st) {
    if (route_ws_bytes(s) > (size_t)LSRM_STATIC_ROUTE_SCRATCH_BYTES) return LSRM_ERR_TOO_LARGE;
    void *ws = nullptr;
    lsrm_status rc = static_scratch(&ws);
    if (rc != LSRM_OK) return rc;
    // project_blocks writes every projection select_topk reads, so nothing of the previous call's
    // contents needs clearing.
    return launch_route(s, d_pos, d_cams, d_idx, d_dist2, ws, st);
}

size_t route_ws_bytes(const Shape &s) {
    size_t n = (size_t)s.nb_obj * (size_t)s.n_views * sizeof(float2);
    return align_up(n > 0 ? n : 256, 256);
}

lsrm_status launch_route(const Shape &s, const float *d_pos, const lsrm_camera *d_cams, int32_t *d_idx,
                         float *d_dist2, void *d_ws, hipStream_t st) {
    float2 *uv = reinterpret_cast<float2 *>(d_ws);
    const bool few = s.nb_obj > 0 && s.nb_obj <= kRouteFew && s.nb <= kRouteFewRows && s.n_views > 0 && s.topk > 0;
    if (s.nb_obj > 0 && s.n_views > 0 && !few) {
        const int grid = (s.nb_obj + kCentBlocks - 1) / kCentBlocks;
        hipLaunchKernelGGL(project_blocks, dim3(grid), dim3(256), 0, st, s.nb_obj, s.n_views, d_pos, d_cams, uv);
        LSRM_HIP_CHECK(hipGetLastError());
    }
    if (s.nb > 0 && s.topk > 0) {
        const int max_cand = s.nb_obj > s.n_tiles ? s.nb_obj : s.n_tiles;
        const size_t stage_bytes = 4 * (size_t)s.topk * sizeof(unsigned long long);
        const size_t cache_bytes = (size_t)((max_cand + 1) / 2) * sizeof(unsigned long long);
        // default dynamic-LDS limit; beyond it distances are recomputed
        const int cache_keys = cache_bytes + stage_bytes <= 60 * 1024 ? 1 : 0;
        const size_t lds = stage_bytes + (cache_keys ? cache_bytes : 0);
        if (few) {  // (at most 5 KB: the keys are always kept)
            hipLaunchKernelGGL(select_topk_few, dim3(s.nb), dim3(256), lds, st, s.nb_obj, s.n_views, s.grid / 8, s.topk, d_pos,
                               d_cams, d_idx, d_dist2);
            LSRM_HIP_CHECK(hipGetLastError());
            return LSRM_OK;
        }
        hipLaunchKernelGGL(select_topk, dim3(s.nb), dim3(256), lds, st, s.nb_obj, s.n_views,
                           s.grid / 8, s.topk, cache_keys, uv, d_idx, d_dist2);
        LSRM_HIP_CHECK(hipGetLastError());
    }
    return LSRM_OK;
}

}  // namespace lsrm
