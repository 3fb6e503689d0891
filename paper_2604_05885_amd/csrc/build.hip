// Tree construction on gfx950 (paper: section "Z-order trees").
//
//  1. bounding box + finiteness check
//  2. Morton keys (21 bits per dimension, dimension 0 most significant in
//     each bit triple; set id above them for forests) fused with the digit
//     histograms of every radix pass
//  3. stable LSD radix sort of (key, input index), one kernel per 8-bit digit
//     with decoupled look-back across tiles (one read + one write per pass)
//  4. gather of the sorted points into float4 (x, y, z, input index)
//  5. leaf plane: gap levels (Eq. 7 on keys) and the windowed test
//     n > N_max^(0) over +-N_max^(0) neighbouring gaps, compacted in order
//  6. exact node sizes n at the leaf splits by galloping binary search
//     (the left/right search of the plane-hierarchy section)
//  7. coarser planes: keep the splits with n > N_max^(p) (Eq. 8)
//  8. node geometry: tight member boxes, first point, count
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <vector>

#include "jz_device.h"
#include "jz_internal.h"

namespace {

constexpr int kSentinelLevel = 255;
constexpr int kBoundaryLevel = 254;

// float <-> order-preserving int for atomic min/max
__device__ __forceinline__ int f2o(float f) {
    int i = __float_as_int(f);
    return i >= 0 ? i : i ^ 0x7FFFFFFF;
}
__device__ __forceinline__ float o2f(int i) { return __int_as_float(i >= 0 ? i : i ^ 0x7FFFFFFF); }

// bbox[0..2] = min (ordered int), bbox[3..5] = max, bbox[6] = non-finite flag
__global__ __launch_bounds__(256) void k_bbox(const float *__restrict__ pts, int64_t n,
                                              int *__restrict__ bbox) {
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    int bad = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float v = pts[3 * i + a];
            bad |= !isfinite(v);
            lo[a] = fminf(lo[a], v);
            hi[a] = fmaxf(hi[a], v);
        }
    }
    // one atomic per block and value (same-address atomics serialize in L2)
    __shared__ float s_v[4][7];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = wave_min(lo[a]);
        hi[a] = wave_max(hi[a]);
    }
    bad = wave_sum(bad);
    const int w = threadIdx.x >> 6;
    if (lane_id() == 0) {
        s_v[w][0] = lo[0]; s_v[w][1] = lo[1]; s_v[w][2] = lo[2];
        s_v[w][3] = hi[0]; s_v[w][4] = hi[1]; s_v[w][5] = hi[2];
        s_v[w][6] = bad ? 1.0f : 0.0f;
    }
    __syncthreads();
    if (threadIdx.x < 7) {
        const int a = threadIdx.x;
        float v = s_v[0][a];
        for (int ww = 1; ww < 4; ++ww) v = a < 3 ? fminf(v, s_v[ww][a]) : fmaxf(v, s_v[ww][a]);
        if (a < 3) atomicMin(bbox + a, f2o(v));
        else if (a < 6) atomicMax(bbox + a, f2o(v));
        else if (v != 0.0f) atomicOr(bbox + 6, 1);
    }
}

__device__ __forceinline__ uint64_t spread3(uint32_t v) {
    uint64_t x = v & 0x1fffffull;
    x = (x | x << 32) & 0x1f00000000ffffull;
    x = (x | x << 16) & 0x1f0000ff0000ffull;
    x = (x | x << 8) & 0x100f00f00f00f00full;
    x = (x | x << 4) & 0x10c30c30c30c30c3ull;
    x = (x | x << 2) & 0x1249249249249249ull;
    return x;
}

constexpr int kMaxPass = 8;

// Morton key + input index, and the digit histograms of all radix passes.
// Quantization per dimension: q = min(2^bits - 1, trunc(fl(fl(x - lo) * inv)))
// with inv = fl(2^bits / ext), ext = the largest extent of the bounding box.
__global__ __launch_bounds__(256) void k_morton(const float *__restrict__ pts, int64_t n,
                                                const int *__restrict__ bbox, int bits,
                                                const int64_t *__restrict__ set_off, int nsets,
                                                int npass, uint64_t *__restrict__ keys,
                                                uint32_t *__restrict__ vals,
                                                uint32_t *__restrict__ hist) {
    __shared__ uint32_t s_h[kMaxPass * 256];
    for (int i = threadIdx.x; i < npass * 256; i += blockDim.x) s_h[i] = 0;
    __syncthreads();
    float lo[3], ext = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = o2f(bbox[a]);
        ext = fmaxf(ext, o2f(bbox[3 + a]) - lo[a]);
    }
    float inv = ext > 0.0f ? (float)(1u << bits) / ext : 0.0f;
    if (!isfinite(inv)) inv = 0.0f;
    const uint32_t qmax = (1u << bits) - 1u;
    const int bits3 = 3 * bits;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        uint32_t q[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float t = (pts[3 * i + a] - lo[a]) * inv;
            uint32_t u = (t >= 0.0f) ? (uint32_t)fminf(t, 4294967040.0f) : 0u;
            q[a] = u < qmax ? u : qmax;
        }
        uint64_t key = (spread3(q[0]) << 2) | (spread3(q[1]) << 1) | spread3(q[2]);
        if (nsets > 1) {
            int lo_s = 0, hi_s = nsets - 1;  // largest s with set_off[s] <= i
            while (lo_s < hi_s) {
                int m = (lo_s + hi_s + 1) >> 1;
                if (set_off[m] <= i) lo_s = m; else hi_s = m - 1;
            }
            key |= (uint64_t)lo_s << bits3;
        }
        keys[i] = key;
        vals[i] = (uint32_t)i;
        for (int p = 0; p < npass; ++p) atomicAdd(&s_h[p * 256 + ((key >> (8 * p)) & 255u)], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < npass * 256; i += blockDim.x)
        if (s_h[i]) atomicAdd(hist + i, s_h[i]);
}

constexpr int RS_THREADS = 256;
constexpr int RS_WAVES = RS_THREADS / 64;
// Keys per thread and tile: 32 for large sorts (8192 keys: two tiles are what a
// CU's LDS and registers hold); fewer where those tiles would leave CUs idle
// (see rs_items).
constexpr int RS_ITEMS = 32;
constexpr uint64_t FLAG_AGG = 1ull << 62;
constexpr uint64_t FLAG_INC = 2ull << 62;
constexpr uint64_t VAL_MASK = (1ull << 62) - 1;

__device__ __forceinline__ uint64_t ld_u64(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_u64(uint64_t *p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One stable counting pass over the 8-bit digit at `shift`. Tiles take their
// id from an atomic counter (so every lower id belongs to a workgroup that has
// started); each tile ranks its keys per wave with ballots, publishes its digit
// counts, looks back over earlier tiles for its global offsets, stages the
// tile in LDS in digit order and writes it out with coalesced runs, keys first
// and then values through the same LDS. What bounds it is the writes, a run of
// tile / 256 keys per digit that begins and ends within a line another tile
// writes too: longer tiles are faster though fewer fit (2^24 keys: 138 us with
// 8192 keys, 147 with 5120, three per CU; tiles of 6144, keys and values staged
// at once, took 5 % longer than 8192; the 0.4 GB of a pass would take 85 us at
// the rate of a copy). `hist`: the
// pass's 256 digit counts over all keys, whose exclusive scan every tile takes
// for itself (a launch of its own took as long as a small pass).
template <int ITEMS>
__global__ __launch_bounds__(RS_THREADS, ITEMS <= 20 ? 3 : 2) void k_onesweep(
    const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin, uint64_t *__restrict__ kout,
    uint32_t *__restrict__ vout, int64_t n, int shift, const uint32_t *__restrict__ hist,
    uint64_t *__restrict__ status, int *__restrict__ tile_ctr) {
    constexpr int RS_TILE = RS_THREADS * ITEMS;
    __shared__ uint64_t s_k[RS_TILE];
    __shared__ __align__(4) uint16_t s_wh[RS_WAVES][256];
    static_assert(__alignof__(s_wh) >= alignof(uint32_t), "cleared in words of 32 bits");
    __shared__ uint32_t s_gb[256];  // a digit's first place, less its first in the tile
    uint32_t *s_v = reinterpret_cast<uint32_t *>(s_k);
    __shared__ int s_tmp[RS_WAVES], s_hist[RS_WAVES];
    __shared__ int s_tile;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (tid == 0) s_tile = atomicAdd(tile_ctr, 1);
    for (int i = tid; i < RS_WAVES * 128; i += RS_THREADS)
        reinterpret_cast<uint32_t *>(s_wh)[i] = 0;
    const int hv = (int)hist[tid];
    const int hinc = wave_incl_scan(hv);
    if (lane == 63) s_hist[w] = hinc;
    __syncthreads();
    const int tile = s_tile;
    int doff = hinc - hv;  // keys of the lower digits
    for (int ww = 0; ww < w; ++ww) doff += s_hist[ww];
    const int64_t base = (int64_t)tile * RS_TILE;
    const int tn = (int)((n - base) < RS_TILE ? (n - base) : RS_TILE);

    uint64_t k[ITEMS];
    uint32_t v[ITEMS];
    uint32_t rk[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int li = w * (ITEMS * 64) + i * 64 + lane;
        const bool valid = li < tn;
        k[i] = valid ? kin[base + li] : 0ull;
        v[i] = valid ? vin[base + li] : 0u;
    }
    const uint64_t ltm = lanemask_lt();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int li = w * (ITEMS * 64) + i * 64 + lane;
        const bool valid = li < tn;
        const uint32_t d = (uint32_t)(k[i] >> shift) & 255u;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t before = s_wh[w][d];
        rk[i] = (d << 16) | (before + (uint32_t)__popcll(peers & ltm));
        const bool leader = valid && ((peers & ltm) == 0ull);
        wave_lds_sync();
        if (leader) s_wh[w][d] = (uint16_t)(before + (uint32_t)__popcll(peers));
        wave_lds_sync();
    }
    __syncthreads();

    // per digit: wave prefix, tile total, look-back over earlier tiles
    const uint32_t c0 = s_wh[0][tid], c1 = s_wh[1][tid], c2 = s_wh[2][tid], c3 = s_wh[3][tid];
    const uint32_t tot = c0 + c1 + c2 + c3;
    // (s_wh becomes the wave's first place of the digit in the tile)
    uint32_t texcl;
    {
        const int inc = wave_incl_scan((int)tot);
        if (lane == 63) s_tmp[w] = inc;
        __syncthreads();
        texcl = (uint32_t)inc - tot;
        for (int ww = 0; ww < w; ++ww) texcl += (uint32_t)s_tmp[ww];
    }
    s_wh[0][tid] = (uint16_t)texcl;
    s_wh[1][tid] = (uint16_t)(texcl + c0);
    s_wh[2][tid] = (uint16_t)(texcl + c0 + c1);
    s_wh[3][tid] = (uint16_t)(texcl + c0 + c1 + c2);
    uint64_t *mine = status + (size_t)tile * 256 + tid;
    uint64_t excl = 0;
    if (tile == 0) {
        st_u64(mine, FLAG_INC | tot);
    } else {
        st_u64(mine, FLAG_AGG | tot);
        int j = tile - 1;
        while (true) {
            const uint64_t sv = ld_u64(status + (size_t)j * 256 + tid);
            const uint64_t flag = sv >> 62;
            if (flag == 0) {  // predecessor not published yet
                __builtin_amdgcn_s_sleep(1);
                continue;
            }
            excl += sv & VAL_MASK;
            if (flag == 2 || j == 0) break;
            --j;
        }
        st_u64(mine, FLAG_INC | (excl + tot));
    }
    s_gb[tid] = (uint32_t)doff + (uint32_t)excl - texcl;
    __syncthreads();
    // keys, then values through the same LDS
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int li = w * (ITEMS * 64) + i * 64 + lane;
        rk[i] = (uint32_t)s_wh[w][rk[i] >> 16] + (rk[i] & 0xffffu);
        if (li < tn) s_k[rk[i]] = k[i];
    }
    __syncthreads();
    uint32_t dest[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int e = i * RS_THREADS + tid;
        if (e < tn) {
            const uint64_t key = s_k[e];
            dest[i] = s_gb[(uint32_t)(key >> shift) & 255u] + (uint32_t)e;
            kout[dest[i]] = key;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int li = w * (ITEMS * 64) + i * 64 + lane;
        if (li < tn) s_v[rk[i]] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int e = i * RS_THREADS + tid;
        if (e < tn) vout[dest[i]] = s_v[e];
    }
}

// digit histograms of npass 8-bit passes over n 64-bit keys
__global__ __launch_bounds__(256) void k_digit_hist(const uint64_t *__restrict__ keys, int64_t n,
                                                    int npass, uint32_t *__restrict__ hist) {
    __shared__ uint32_t s_h[kMaxPass * 256];
    for (int i = threadIdx.x; i < npass * 256; i += blockDim.x) s_h[i] = 0;
    __syncthreads();
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint64_t key = keys[i];
        for (int p = 0; p < npass; ++p) atomicAdd(&s_h[p * 256 + ((key >> (8 * p)) & 255u)], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < npass * 256; i += blockDim.x)
        if (s_h[i]) atomicAdd(hist + i, s_h[i]);
}

__global__ __launch_bounds__(256) void k_gather(const float *__restrict__ pts,
                                                const uint32_t *__restrict__ order, int64_t n,
                                                float4 *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t j = order[i];
    out[i] = make_float4(pts[3 * (int64_t)j], pts[3 * (int64_t)j + 1], pts[3 * (int64_t)j + 2],
                         __int_as_float((int)j));
}

// Level of gap g (between sorted points g-1 and g), Eq. 7 on keys extended by
// the sorted position: 32 + bitlen(key xor) for different keys, bitlen of the
// position xor for equal keys, 254 where the set changes, 255 at both ends.
__device__ __forceinline__ int gap_level(const uint64_t *__restrict__ keys, int64_t n, int64_t g,
                                         int bits3, int has_sets) {
    if (g <= 0 || g >= n) return kSentinelLevel;
    const uint64_t x = keys[g - 1] ^ keys[g];
    if (has_sets && (x >> bits3)) return kBoundaryLevel;
    if (x) return 32 + (int)bitlen64(x);
    return (int)bitlen64((uint64_t)(g - 1) ^ (uint64_t)g);
}

// level of the smallest node holding sorted points i < j
__device__ __forceinline__ int pair_level(const uint64_t *__restrict__ keys, int64_t i, int64_t j,
                                          int bits3, int has_sets) {
    const uint64_t x = keys[i] ^ keys[j];
    if (has_sets && (x >> bits3)) return kBoundaryLevel;
    if (x) return 32 + (int)bitlen64(x);
    return (int)bitlen64((uint64_t)i ^ (uint64_t)j);
}

constexpr int LF_TILE = 1024;
constexpr int LF_MAXW = 64;

// Leaf-plane split flags: gap g is a split iff the node spanning it holds
// more than nmax0 points, i.e. the nearest strictly greater gap on one side
// lies farther than the window, or both lie within it but r - l > nmax0.
// The nearest greater gaps are found by binary lifting over a table of range
// maxima of the tile (mx[k][i] = max of the 2^k levels from i), so every
// thread takes the same ~2 x 7 steps instead of a scan of up to 2 x nmax0.
constexpr int LF_SPAN = LF_TILE + 2 * LF_MAXW + 2;
constexpr int LF_LOG = 7;  // 2^6 = LF_MAXW: levels 0..6
// whether the gap at position c of the tables (mx(k): the table of the 2^k) is
// a split, with a window of W gaps on either side
template <class MX>
__device__ __forceinline__ bool leaf_split(MX &&mx, int c, int W, int nmax0) {
    const int lv = mx(0)[c];
    if (lv >= kBoundaryLevel) return true;
    // left: move cur down while [cur - 2^k, cur) holds no greater level
    int cur = c;
    for (int k = LF_LOG - 1; k >= 0; --k)
        if (cur - (1 << k) >= c - W && mx(k)[cur - (1 << k)] <= lv) cur -= 1 << k;
    const int dl = cur - 1 >= c - W ? c - (cur - 1) : 0;
    if (dl == 0) return true;
    // right: move cur up while [cur, cur + 2^k) holds no greater level
    cur = c + 1;
    for (int k = LF_LOG - 1; k >= 0; --k)
        if (cur + (1 << k) - 1 <= c + W && mx(k)[cur] <= lv) cur += 1 << k;
    const int dr = cur <= c + W ? cur - c : 0;
    return dr == 0 || dl + dr > nmax0;
}
__global__ __launch_bounds__(256) void k_leaf_flags(const uint64_t *__restrict__ keys, int64_t n,
                                                    int bits3, int has_sets, int nmax0,
                                                    uint8_t *__restrict__ flags,
                                                    int *__restrict__ blk_cnt) {
    __shared__ uint8_t s_mx[LF_LOG][LF_SPAN];
    __shared__ int s_c[4];
    const int W = nmax0;
    const int span = LF_TILE + 2 * W + 1;
    const int64_t g0 = (int64_t)blockIdx.x * LF_TILE;
    for (int t = threadIdx.x; t < span; t += blockDim.x)
        s_mx[0][t] = (uint8_t)gap_level(keys, n, g0 - W + t, bits3, has_sets);
    __syncthreads();
    for (int k = 1; k < LF_LOG; ++k) {
        const int h = 1 << (k - 1);
        for (int t = threadIdx.x; t + 2 * h <= span; t += blockDim.x)
            s_mx[k][t] = max(s_mx[k - 1][t], s_mx[k - 1][t + h]);
        __syncthreads();
    }
    int cnt = 0;
    for (int t = threadIdx.x; t < LF_TILE; t += blockDim.x) {
        const int64_t g = g0 + t;
        if (g > n) break;
        // t + W: g's position in the tile
        const uint8_t f = leaf_split([&](int k) { return s_mx[k]; }, t + W, W, nmax0) ? 1 : 0;
        flags[g] = f;
        cnt += f;
    }
    cnt = wave_sum(cnt);
    if (lane_id() == 0) s_c[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) blk_cnt[blockIdx.x] = s_c[0] + s_c[1] + s_c[2] + s_c[3];
}

// exclusive offsets of per-block counts; total to *total (one block)
__global__ __launch_bounds__(1024) void k_scan_counts(const int *__restrict__ cnt, int nb,
                                                      int *__restrict__ off,
                                                      int *__restrict__ total) {
    __shared__ int s_w[16];
    const int t = threadIdx.x;
    const int per = (nb + 1023) / 1024;
    const int b0 = t * per;
    int sum = 0;
    for (int i = 0; i < per; ++i)
        if (b0 + i < nb) sum += cnt[b0 + i];
    const int inc = wave_incl_scan(sum);
    if (lane_id() == 63) s_w[t >> 6] = inc;
    __syncthreads();
    int add = 0;
    for (int w = 0; w < (t >> 6); ++w) add += s_w[w];
    int run = inc - sum + add;
    for (int i = 0; i < per; ++i)
        if (b0 + i < nb) {
            off[b0 + i] = run;
            run += cnt[b0 + i];
        }
    if (t == 1023) *total = inc + add;
}

// ordered compaction of flagged items: out[pos] = item, and, if given,
// out2[pos] = map[item] (map NULL: item)
__global__ __launch_bounds__(256) void k_compact(const uint8_t *__restrict__ flags,
                                                 int64_t nitems_max,
                                                 const int *__restrict__ nitems_dev,
                                                 const int *__restrict__ off,
                                                 int *__restrict__ out,
                                                 const int *__restrict__ map,
                                                 int *__restrict__ out2) {
    __shared__ int s_w[4];
    const int64_t nitems = nitems_dev ? (int64_t)(*nitems_dev) : nitems_max;
    const int64_t base = (int64_t)blockIdx.x * LF_TILE;
    int run = off[blockIdx.x];
    const int t = threadIdx.x, w = t >> 6;
    for (int c = 0; c < LF_TILE / 256; ++c) {
        const int64_t item = base + c * 256 + t;
        const bool f = item < nitems && flags[item];
        const uint64_t m = __ballot(f);
        const int pre = __popcll(m & lanemask_lt());
        if (lane_id() == 0) s_w[w] = __popcll(m);
        __syncthreads();
        int add = 0, tot = 0;
        for (int ww = 0; ww < 4; ++ww) {
            if (ww < w) add += s_w[ww];
            tot += s_w[ww];
        }
        if (f) {
            const int pos = run + add + pre;
            out[pos] = (int)item;
            if (out2) out2[pos] = map ? map[item] : (int)item;
        }
        run += tot;
        __syncthreads();
    }
}

// Exact size of the node spanning each leaf split (galloping search for the
// nearest strictly greater gap on both sides). Sentinels and set boundaries
// get INT_MAX so that they stay splits on every plane.
__global__ __launch_bounds__(256) void k_split_sizes(const uint64_t *__restrict__ keys, int64_t n,
                                                     int bits3, int has_sets,
                                                     const int *__restrict__ spl0,
                                                     const int *__restrict__ cnt0, int gallop0,
                                                     int *__restrict__ nsz,
                                                     uint8_t *__restrict__ slv) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t m = *cnt0;  // L0 + 1 entries
    if (s >= m) return;
    const int64_t g = spl0[s];
    const int lv = gap_level(keys, n, g, bits3, has_sets);
    slv[s] = (uint8_t)lv;
    if (lv >= kBoundaryLevel) {
        nsz[s] = INT_MAX;
        return;
    }
    // left: first j in [0, g-1] with pair_level(j, g) <= lv (monotone in j)
    int64_t good = g - 1, bad = -1, step = gallop0;
    while (good - bad > 1) {
        const int64_t j = good - step;
        if (j <= bad) break;
        if (pair_level(keys, j, g, bits3, has_sets) <= lv) {
            good = j;
            step <<= 1;
        } else {
            bad = j;
            break;
        }
    }
    while (good - bad > 1) {
        const int64_t mid = bad + (good - bad) / 2;
        if (pair_level(keys, mid, g, bits3, has_sets) <= lv) good = mid; else bad = mid;
    }
    const int64_t lb = good;
    // right: first j in [g, n) with pair_level(g-1, j) > lv, else n
    good = g;
    bad = n;
    step = gallop0;
    while (bad - good > 1) {
        const int64_t j = good + step;
        if (j >= bad) break;
        if (pair_level(keys, g - 1, j, bits3, has_sets) <= lv) {
            good = j;
            step <<= 1;
        } else {
            bad = j;
            break;
        }
    }
    while (bad - good > 1) {
        const int64_t mid = good + (bad - good) / 2;
        if (pair_level(keys, g - 1, mid, bits3, has_sets) <= lv) good = mid; else bad = mid;
    }
    const int64_t rb = bad;
    nsz[s] = (int)(rb - lb);
}

// Plane p flags over the plane p-1 splits: keep the ends and every split
// whose node size exceeds N_max^(p). lsi_prev: their leaf splits (NULL: the
// plane below is the leaf plane).
__global__ __launch_bounds__(256) void k_plane_flags(const int *__restrict__ lsi_prev,
                                                     const int *__restrict__ cnt_prev,
                                                     const int *__restrict__ nsz, int64_t nmax,
                                                     const uint8_t *__restrict__ slv, int lvl_max,
                                                     uint8_t *__restrict__ flags,
                                                     int *__restrict__ blk_cnt) {
    __shared__ int s_c[4];
    const int64_t m = *cnt_prev;
    int cnt = 0;
    const int64_t base = (int64_t)blockIdx.x * LF_TILE;
    for (int t = threadIdx.x; t < LF_TILE; t += blockDim.x) {
        const int64_t j = base + t;
        if (j >= m) break;
        const int ls = lsi_prev ? lsi_prev[j] : (int)j;
        const uint8_t f = (j == 0 || j == m - 1 || (int64_t)nsz[ls] > nmax ||
                           (int)slv[ls] > lvl_max) ? 1 : 0;
        flags[j] = f;
        cnt += f;
    }
    cnt = wave_sum(cnt);
    if (lane_id() == 0) s_c[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) blk_cnt[blockIdx.x] = s_c[0] + s_c[1] + s_c[2] + s_c[3];
}

// Regularization (paper: section on regularization): points per node level
// over the nodes of a plane. Node i spans the sorted points between leaf
// splits lsi[i] and lsi[i + 1] (lsi = NULL: the leaf plane itself); its level
// is that of its first and last point (the largest gap level inside it).
__global__ __launch_bounds__(256) void k_level_hist(const uint64_t *__restrict__ keys,
                                                    const int *__restrict__ spl0,
                                                    const int *__restrict__ lsi,
                                                    const int *__restrict__ cnt, int bits3,
                                                    int has_sets,
                                                    unsigned long long *__restrict__ hist) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i + 1 >= *cnt) return;
    const int64_t a = spl0[lsi ? lsi[i] : i], e = spl0[lsi ? lsi[i + 1] : i + 1];
    const int lv = e - a > 1 ? pair_level(keys, a, e - 1, bits3, has_sets) : 0;
    atomicAdd(hist + lv, (unsigned long long)(e - a));
}

// leaf plane: also split every gap whose level exceeds lvl_max; per-block
// counts as k_leaf_flags
__global__ __launch_bounds__(256) void k_reg_leaf_flags(const uint64_t *__restrict__ keys,
                                                        int64_t n, int bits3, int has_sets,
                                                        int lvl_max, uint8_t *__restrict__ flags,
                                                        int *__restrict__ blk_cnt) {
    __shared__ int s_c[4];
    int cnt = 0;
    const int64_t g0 = (int64_t)blockIdx.x * LF_TILE;
    for (int t = threadIdx.x; t < LF_TILE; t += blockDim.x) {
        const int64_t g = g0 + t;
        if (g > n) break;
        uint8_t f = flags[g];
        if (!f && gap_level(keys, n, g, bits3, has_sets) > lvl_max) {
            f = 1;
            flags[g] = 1;
        }
        cnt += f;
    }
    cnt = wave_sum(cnt);
    if (lane_id() == 0) s_c[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) blk_cnt[blockIdx.x] = s_c[0] + s_c[1] + s_c[2] + s_c[3];
}

// leaves: one wave per leaf, lanes over its points
__device__ __forceinline__ void leaf_box(const float4 *pts, int s0, int s1, Node *node) {
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i = s0 + lane_id(); i < s1; i += 64) {
        const float4 p = pts[i];
        lo[0] = fminf(lo[0], p.x); hi[0] = fmaxf(hi[0], p.x);
        lo[1] = fminf(lo[1], p.y); hi[1] = fmaxf(hi[1], p.y);
        lo[2] = fminf(lo[2], p.z); hi[2] = fmaxf(hi[2], p.z);
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        lo[d] = wave_min(lo[d]);
        hi[d] = wave_max(hi[d]);
    }
    if (lane_id() == 0) {
        Node nd;
        nd.lo[0] = lo[0]; nd.lo[1] = lo[1]; nd.lo[2] = lo[2];
        nd.hi[0] = hi[0]; nd.hi[1] = hi[1]; nd.hi[2] = hi[2];
        nd.start = s0;
        nd.count = s1 - s0;
        *node = nd;
    }
}

__global__ __launch_bounds__(256) void k_leaf_geom(const float4 *__restrict__ pts,
                                                   const int *__restrict__ spl, int64_t L,
                                                   Node *__restrict__ nodes) {
    const int64_t a = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (a >= L) return;
    leaf_box(pts, spl[a], spl[a + 1], nodes + a);
}

// coarser planes: one wave per node, lanes over its children
__global__ __launch_bounds__(256) void k_node_geom(const Node *__restrict__ child,
                                                   const int *__restrict__ spl, int64_t L,
                                                   Node *__restrict__ nodes) {
    const int64_t a = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (a >= L) return;
    const int c0 = spl[a], c1 = spl[a + 1];
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    int cnt = 0;
    for (int c = c0 + lane_id(); c < c1; c += 64) {
        const Node ch = child[c];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            lo[d] = fminf(lo[d], ch.lo[d]);
            hi[d] = fmaxf(hi[d], ch.hi[d]);
        }
        cnt += ch.count;
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        lo[d] = wave_min(lo[d]);
        hi[d] = wave_max(hi[d]);
    }
    cnt = wave_sum(cnt);
    if (lane_id() == 0) {
        Node nd;
        nd.lo[0] = lo[0]; nd.lo[1] = lo[1]; nd.lo[2] = lo[2];
        nd.hi[0] = hi[0]; nd.hi[1] = hi[1]; nd.hi[2] = hi[2];
        nd.start = child[c0].start;
        nd.count = cnt;
        nodes[a] = nd;
    }
}

// Before a build: bbox empty, the histogram, sort status and counters zero.
__global__ __launch_bounds__(256) void k_build_init(unsigned long long *__restrict__ zero, size_t n,
                                                    int *__restrict__ meta) {
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (size_t i = i0; i < n; i += (size_t)gridDim.x * blockDim.x) zero[i] = 0;
    if (i0 < 8) meta[i0] = i0 < 3 ? INT_MAX : (i0 < 6 ? INT_MIN : 0);
}

// Super nodes of ngr top nodes and their dense lists, for a single set: row i
// of the kNN list names all S super nodes, row i of the FoF list those from i
// on (Alg. 1 lines 1-2).
__global__ __launch_bounds__(256) void k_top_lists(int S, int LT, int ngr, int *__restrict__ spl,
                                                   int2 *__restrict__ kseg,
                                                   int2 *__restrict__ klist,
                                                   int2 *__restrict__ fseg,
                                                   int2 *__restrict__ flist) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    auto frow = [&](int64_t i) { return i * S - i * (i - 1) / 2; };
    for (int64_t i = t0; i <= S; i += stride) {
        spl[i] = i < S ? (int)i * ngr : LT;
        if (i == S) break;
        kseg[i] = make_int2((int)(i * S), S);
        fseg[i] = make_int2((int)frow(i), S - (int)i);
    }
    for (int64_t e = t0; e < (int64_t)S * S; e += stride) {
        const int64_t i = e / S, j = e - i * S;
        klist[e] = make_int2((int)j, 0);
        if (j >= i) flist[frow(i) + j - i] = make_int2((int)j, 0);
    }
}

// The whole leaf plane of a set of at most SMALL_N points in one workgroup:
// bounding box, keys, sort, sorted points, splits and leaf boxes, with the
// definitions of the kernels above (key and input index packed in one word,
// whose order is that of the stable radix sort). What bounds a set this small
// is the number of launches: 13 of them and three transfers, 0.25 ms of a build
// of 1000 points, against one launch of about 0.03 ms.
// hdr: leaf splits, then bounding box and non-finite flag as k_bbox leaves them.
constexpr int SMALL_N = 4096;
constexpr int SMALL_IDX_BITS = 12;  // of the input index in a packed key
constexpr int SMALL_NT = 1024;
__global__ __launch_bounds__(SMALL_NT) void k_build_small(const float *__restrict__ pts, int n,
                                                          int bits, int nmax0,
                                                          float4 *__restrict__ out,
                                                          int *__restrict__ spl,
                                                          Node *__restrict__ nodes,
                                                          int *__restrict__ hdr) {
    constexpr int NW = SMALL_NT / 64;
    constexpr int SPAN = SMALL_N + 1 + 2 * LF_MAXW;
    __shared__ uint64_t s_key[SMALL_N];  // later the upper tables of s_mx
    __shared__ uint8_t s_mx0[SPAN];
    __shared__ int s_spl[SMALL_N + 1];
    __shared__ float s_box[NW][6];
    __shared__ int s_w[NW + 1], s_bad;
    static_assert(sizeof(uint64_t) * SMALL_N >= (size_t)(LF_LOG - 1) * SPAN, "tables fit");
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // 1: bounding box
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    int bad = 0;
    for (int i = tid; i < n; i += SMALL_NT) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float v = pts[3 * i + a];
            bad |= !isfinite(v);
            lo[a] = fminf(lo[a], v);
            hi[a] = fmaxf(hi[a], v);
        }
    }
    if (tid == 0) s_bad = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = wave_min(lo[a]);
        hi[a] = wave_max(hi[a]);
    }
    if (lane < 3) {
        s_box[w][lane] = lane == 0 ? lo[0] : (lane == 1 ? lo[1] : lo[2]);
        s_box[w][3 + lane] = lane == 0 ? hi[0] : (lane == 1 ? hi[1] : hi[2]);
    }
    __syncthreads();
    if (bad) s_bad = 1;
    float ext = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = s_box[0][a];
        hi[a] = s_box[0][3 + a];
        for (int ww = 1; ww < NW; ++ww) {
            lo[a] = fminf(lo[a], s_box[ww][a]);
            hi[a] = fmaxf(hi[a], s_box[ww][3 + a]);
        }
        ext = fmaxf(ext, hi[a] - lo[a]);
    }
    // 2: keys
    float inv = ext > 0.0f ? (float)(1u << bits) / ext : 0.0f;
    if (!isfinite(inv)) inv = 0.0f;
    const uint32_t qmax = (1u << bits) - 1u;
    int M = 2 * NW;
    while (M < n) M <<= 1;
    for (int i = tid; i < M; i += SMALL_NT) {
        uint64_t key = ~0ull;
        if (i < n) {
            uint32_t q[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float t = (pts[3 * i + a] - lo[a]) * inv;
                const uint32_t u = (t >= 0.0f) ? (uint32_t)fminf(t, 4294967040.0f) : 0u;
                q[a] = u < qmax ? u : qmax;
            }
            key = (spread3(q[0]) << 2) | (spread3(q[1]) << 1) | spread3(q[2]);
            key = key << SMALL_IDX_BITS | (uint64_t)i;
        }
        s_key[i] = key;
    }
    __syncthreads();
    // 3: bitonic sort (pairs at a distance of up to PW lie within one wave's
    // range of PW pairs: those steps need no workgroup barrier)
    const int PW = (M >> 1) / NW;
    for (int k = 2; k <= M; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            const bool wide = j > PW;
            if (wide) __syncthreads();
            const int i0 = wide ? tid : w * PW + lane;
            const int i1 = wide ? (M >> 1) : (w + 1) * PW;
            const int di = wide ? SMALL_NT : 64;
            for (int i = i0; i < i1; i += di) {
                const int a = ((i & ~(j - 1)) << 1) | (i & (j - 1));
                const int b = a + j;
                const uint64_t x = s_key[a], y = s_key[b];
                const bool up = (a & k) == 0;
                if ((x > y) == up) {
                    s_key[a] = y;
                    s_key[b] = x;
                }
            }
            if (wide) __syncthreads();
            else wave_lds_sync();
        }
    }
    __syncthreads();
    // 4: sorted points; 5: gap levels (s_mx0[W + g] of gap g)
    const int W = nmax0, span = n + 1 + 2 * W;
    for (int i = tid; i < n; i += SMALL_NT) {
        const int j = (int)(s_key[i] & ((1u << SMALL_IDX_BITS) - 1u));
        out[i] = make_float4(pts[3 * j], pts[3 * j + 1], pts[3 * j + 2], __int_as_float(j));
    }
    for (int t = tid; t < span; t += SMALL_NT) {
        const int g = t - W;
        int lv = kSentinelLevel;
        if (g > 0 && g < n) {
            const uint64_t x = (s_key[g - 1] ^ s_key[g]) >> SMALL_IDX_BITS;
            lv = x ? 32 + (int)bitlen64(x) : (int)bitlen64((uint64_t)(g - 1) ^ (uint64_t)g);
        }
        s_mx0[t] = (uint8_t)lv;
    }
    __syncthreads();
    // 6: range maxima of 2^k levels, split flags, splits in order
    uint8_t *const s_up = reinterpret_cast<uint8_t *>(s_key);
    auto mx = [&](int k) { return k == 0 ? s_mx0 : s_up + (k - 1) * SPAN; };
    for (int k = 1; k < LF_LOG; ++k) {
        const int h = 1 << (k - 1);
        const uint8_t *src = mx(k - 1);
        uint8_t *dst = mx(k);
        for (int t = tid; t + 2 * h <= span; t += SMALL_NT) dst[t] = max(src[t], src[t + h]);
        __syncthreads();
    }
    const int per = (n + SMALL_NT) / SMALL_NT;  // gaps 0 .. n, `per` in a row per thread
    unsigned fl = 0;
    for (int u = 0; u < per; ++u) {
        const int g = tid * per + u;
        if (g > n) break;
        const int c = g + W;
        fl |= leaf_split(mx, c, W, nmax0) ? 1u << u : 0u;
    }
    const int cnt = __popc(fl);
    const int inc = wave_incl_scan(cnt);
    if (lane == 63) s_w[w] = inc;
    __syncthreads();
    int pos = inc - cnt;
    for (int ww = 0; ww < w; ++ww) pos += s_w[ww];
    int m0 = 0;
    for (int ww = 0; ww < NW; ++ww) m0 += s_w[ww];
    for (int u = 0; u < per; ++u)
        if ((fl >> u) & 1u) {
            spl[pos] = tid * per + u;
            s_spl[pos++] = tid * per + u;
        }
    __syncthreads();
    // 8: leaf boxes, one wave per leaf
    for (int l = w; l < m0 - 1; l += NW) leaf_box(out, s_spl[l], s_spl[l + 1], nodes + l);
    if (tid == 0) {
        hdr[0] = m0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            hdr[1 + a] = f2o(lo[a]);
            hdr[4 + a] = f2o(hi[a]);
        }
        hdr[7] = s_bad;
    }
}

// set of each node (from the key of its first point) and, for leaves, the
// first input index of that set
__global__ void k_node_sets(const Node *__restrict__ nodes, int64_t L,
                            const uint64_t *__restrict__ keys, int bits3,
                            const int64_t *__restrict__ set_off, int *__restrict__ set_of,
                            int *__restrict__ base_of) {
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= L) return;
    const int s = (int)(keys[nodes[a].start] >> bits3);
    set_of[a] = s;
    if (base_of) base_of[a] = (int)set_off[s];
}

}  // namespace

// ---------------------------------------------------------------------------

// Keys per thread of a sort of n keys, from the time of one pass in us:
//   n         5 10^4   1.5 10^5   3 10^5   6 10^5   10^6    2 10^6   4 10^6   2^24
//   4            7.1       12.2     17.3     26.7   37.1      62               345
//   8            8.6       11.0     13.6     19.4   25.4      40               221
//   12           9.3       11.3     13.8     15.6   23.0      34               188
//   20                                              22.1      30.3     46.4    147
//   32                                              25.2      29.2     42.6    138
// (small tiles fill the chip sooner, but each looks back over more tiles)
static int rs_items(int64_t n) {
    return n < 100000 ? 4 : n < 400000 ? 8 : n < 900000 ? 12 : n < 3000000 ? 20 : RS_ITEMS;
}


// Scratch of a radix sort of n keys in npass passes, to be zero before it: the
// digit counts of all passes, the tiles' status words and the tile counters.
struct SortScratch {
    DBuf buf;
    int64_t ntiles = 0;
    int npass = 0, items = RS_ITEMS;
    static constexpr size_t HIST_WORDS = kMaxPass * 256 / 2, CTR_WORDS = kMaxPass;
    jz_status get(const AllocCtx *ac, int64_t n, int np, hipStream_t s) {
        items = rs_items(n);
        ntiles = (n + RS_THREADS * items - 1) / (RS_THREADS * items);
        npass = np;
        return buf.get(ac, words() * sizeof(uint64_t), s);
    }
    size_t words() const { return HIST_WORDS + CTR_WORDS + (size_t)ntiles * 256 * npass; }
    uint32_t *hist() const { return buf.as<uint32_t>(); }
    int *ctr(int p) const { return reinterpret_cast<int *>(buf.as<uint64_t>() + HIST_WORDS) + 2 * p; }
    uint64_t *status(int p) const {
        return buf.as<uint64_t>() + HIST_WORDS + CTR_WORDS + (size_t)ntiles * 256 * p;
    }
};

// The onesweep passes over the low 8 * npass key bits, with the digit counts in
// sc; (kin, vin) -> sorted pairs, swapping with (kout, vout) after every pass
// (the result is where the last pass wrote).
static jz_status onesweep_passes(const SortScratch &sc, uint64_t *&kin, uint32_t *&vin,
                                 uint64_t *&kout, uint32_t *&vout, int64_t n, hipStream_t s) {
    const auto pass = sc.items == 4    ? k_onesweep<4>
                      : sc.items == 8  ? k_onesweep<8>
                      : sc.items == 12 ? k_onesweep<12>
                      : sc.items == 20 ? k_onesweep<20>
                                       : k_onesweep<RS_ITEMS>;
    for (int p = 0; p < sc.npass; ++p) {
        pass<<<(unsigned)sc.ntiles, RS_THREADS, 0, s>>>(kin, vin, kout, vout, n, 8 * p,
                                                        sc.hist() + 256 * p, sc.status(p), sc.ctr(p));
        std::swap(kin, kout);
        std::swap(vin, vout);
    }
    JZ_HIP(hipGetLastError());
    return JZ_OK;
}

jz_status radix_sort_pairs(const AllocCtx *ac, DBuf &k0, DBuf &v0, DBuf &k1, DBuf &v1, int64_t n,
                           int bits, hipStream_t s) {
    if (n <= 1 || bits <= 0) return JZ_OK;
    SortScratch sc;
    JZ_TRY(sc.get(ac, n, std::min(kMaxPass, (bits + 7) / 8), s));
    JZ_TRY(zero_words(sc.buf.as<unsigned long long>(), sc.words(), s));
    k_digit_hist<<<std::min<unsigned>(blocks_for(n, 256 * 8), 2048), 256, 0, s>>>(
        k0.as<uint64_t>(), n, sc.npass, sc.hist());
    uint64_t *kin = k0.as<uint64_t>(), *kout = k1.as<uint64_t>();
    uint32_t *vin = v0.as<uint32_t>(), *vout = v1.as<uint32_t>();
    JZ_TRY(onesweep_passes(sc, kin, vin, kout, vout, n, s));
    if (kin != k0.as<uint64_t>()) {
        std::swap(k0.p, k1.p);
        std::swap(v0.p, v1.p);
    }
    return JZ_OK;
}

namespace {

// source points per leaf (one wave per leaf: a leaf holds at most 64 points)
__global__ __launch_bounds__(256) void k_src_count_leaf(const Node *__restrict__ leaves, int64_t L,
                                                        const float4 *__restrict__ pts, int n_src,
                                                        int *__restrict__ cnt) {
    const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (i >= L) return;
    const Node a = leaves[i];
    const int lane = lane_id();
    const bool src = lane < a.count && __float_as_int(pts[a.start + lane].w) < n_src;
    const uint64_t m = __ballot(src);
    if (lane == 0) cnt[i] = (int)__popcll(m);
}

// source points per node of a coarser plane: the sum over its children
__global__ __launch_bounds__(256) void k_src_count_up(const int *__restrict__ child,
                                                      const int *__restrict__ spl, int64_t L,
                                                      int *__restrict__ cnt) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= L) return;
    int s = 0;
    for (int c = spl[i]; c < spl[i + 1]; ++c) s += child[c];
    cnt[i] = s;
}

}  // namespace

jz_status source_counts(jz_tree *t, hipStream_t s) {
    for (int p = 0; p < t->P; ++p) {
        JZ_TRY(t->src_cnt[p].get(&t->ac, (size_t)t->L[p] * sizeof(int), s));
        if (p == 0)
            k_src_count_leaf<<<blocks_for(t->L[0] * 64, 256), 256, 0, s>>>(
                t->nodes[0].as<Node>(), t->L[0], t->pts4.as<float4>(), (int)t->n_src,
                t->src_cnt[0].as<int>());
        else
            k_src_count_up<<<blocks_for(t->L[p], 256), 256, 0, s>>>(
                t->src_cnt[p - 1].as<int>(), t->spl[p].as<int>(), t->L[p], t->src_cnt[p].as<int>());
    }
    JZ_HIP(hipGetLastError());
    return JZ_OK;
}

// Regularization: the largest node level of a plane from its histogram of
// points per node level. V90 is the point-weighted mean volume (2^level) of
// the smallest nodes that together hold 90% of the points; nodes may not
// exceed f_max * V90, i.e. levels above floor(log2(f_max * V90)) are split.
static int reg_level_max(const unsigned long long *hist, double f_max) {
    double total = 0;
    for (int l = 0; l < 256; ++l) total += (double)hist[l];
    if (total <= 0) return 1000;
    double cum = 0, wsum = 0;
    for (int l = 0; l < 256 && cum < 0.9 * total; ++l) {
        cum += (double)hist[l];
        wsum += (double)hist[l] * std::ldexp(1.0, l);
    }
    const double v90 = wsum / cum;
    return (int)std::floor(std::log2(f_max * v90));
}

static int plan_planes(int64_t n, const jz_build_opts &o) {
    int P = 1;
    double nmax = (double)o.leaf_max;
    while (P < JZ_MAX_PLANES) {
        nmax *= o.coarsen;
        if ((double)n / (nmax / 2.0) < (double)o.n_target) break;
        ++P;
    }
    return P;
}

// The input's bounding box (ordered ints) and non-finite flag, as k_bbox leaves
// them, against what a tree takes.
static jz_status check_box(const int *bbox, const jz_build_opts &o) {
    if (bbox[6]) return jz_fail(JZ_E_NONFINITE, "input contains NaN or infinite coordinates");
    if (o.period > 0.0f) {
        // the periodic cube is [0, period)^3
        auto of = [](int v) {
            const int i = v >= 0 ? v : v ^ 0x7FFFFFFF;
            float f;
            std::memcpy(&f, &i, sizeof(f));
            return f;
        };
        for (int a = 0; a < 3; ++a)
            if (!(of(bbox[a]) >= 0.0f) || !(of(bbox[3 + a]) < o.period))
                return jz_fail(JZ_E_INVALID, "with period %g every coordinate must lie in "
                               "[0, %g)", (double)o.period, (double)o.period);
    }
    return JZ_OK;
}

static void set_stats(jz_tree *t) {
    t->st.n = t->n;
    t->st.planes = t->P;
    for (int p = 0; p < JZ_MAX_PLANES; ++p) t->st.nodes[p] = p < t->P ? t->L[p] : 0;
    t->st.super_nodes = t->S;
}

jz_status check_top(int64_t last) {
    if (last <= INT32_MAX) return JZ_OK;
    return jz_fail(JZ_E_CAPACITY, "the list of super node pairs has more than 2^31-1 entries; "
                   "raise ngr or lower n_target");
}

// Super nodes over the top plane and their dense lists: made on the device for
// a single set (no transfer), on the host for a forest, whose rows end at the
// set boundaries. Waits for the stream where host arrays are read.
static jz_status top_lists(jz_tree *t, const uint64_t *keys, int bits3, hipStream_t s) {
    const AllocCtx *ac = &t->ac;
    const jz_build_opts &o = t->opts;
    const int P = t->P, T = P - 1;
    const int64_t LT = t->L[T];
    if (t->nsets == 1) {
        const int64_t S = t->S = (LT + o.ngr - 1) / o.ngr;
        size_t bytes;
        if (!top_list_bytes(S, bytes))
            return jz_fail(JZ_E_OOM, "the list of all pairs of %lld super nodes does not fit; raise "
                           "ngr or lower n_target", (long long)S);
        t->knn_top_last = S * (S - 1);
        t->fof_top_last = (S - 1) * (S + 2) / 2;
        JZ_TRY(t->super_spl.get(ac, (S + 1) * sizeof(int), s));
        JZ_TRY(t->knn_top_seg.get(ac, S * sizeof(int2), s));
        JZ_TRY(t->knn_top_list.get(ac, bytes, s));
        JZ_TRY(t->fof_top_seg.get(ac, S * sizeof(int2), s));
        JZ_TRY(t->fof_top_list.get(ac, S * (S + 1) / 2 * sizeof(int2), s));
        k_top_lists<<<std::min<unsigned>(blocks_for(S * S + 1, 256), 4096), 256, 0, s>>>(
            (int)S, (int)LT, o.ngr, t->super_spl.as<int>(), t->knn_top_seg.as<int2>(),
            t->knn_top_list.as<int2>(), t->fof_top_seg.as<int2>(), t->fof_top_list.as<int2>());
        JZ_HIP(hipGetLastError());
        return JZ_OK;
    }
    std::vector<int> top_set(LT, 0);
    {
        JZ_TRY(t->leaf_base.get(ac, t->L[0] * sizeof(int), s));
        for (int p = 0; p < P; ++p) {
            JZ_TRY(t->node_set[p].get(ac, t->L[p] * sizeof(int), s));
            k_node_sets<<<blocks_for(t->L[p], 256), 256, 0, s>>>(
                t->nodes[p].as<Node>(), t->L[p], keys, bits3, t->d_set_off.as<int64_t>(),
                t->node_set[p].as<int>(), p == 0 ? t->leaf_base.as<int>() : nullptr);
        }
        JZ_HIP(hipMemcpyAsync(top_set.data(), t->node_set[T].p, LT * sizeof(int),
                              hipMemcpyDeviceToHost, s));
        JZ_HIP(hipStreamSynchronize(s));
    }
    std::vector<int> sspl;
    t->super_set.clear();
    for (int64_t a = 0; a < LT;) {
        int64_t b = a;
        while (b < LT && top_set[b] == top_set[a]) ++b;
        for (int64_t c = a; c < b; c += o.ngr) {
            sspl.push_back((int)c);
            t->super_set.push_back(top_set[a]);
        }
        a = b;
    }
    t->S = (int64_t)sspl.size();
    sspl.push_back((int)LT);
    // dense lists over the super nodes of each set
    std::vector<int2> kseg(t->S), fseg(t->S), klist, flist;
    for (int64_t a = 0; a < t->S;) {
        int64_t b = a;
        while (b < t->S && t->super_set[b] == t->super_set[a]) ++b;
        for (int64_t i = a; i < b; ++i) {
            t->knn_top_last = (int64_t)klist.size();
            t->fof_top_last = (int64_t)flist.size();
            kseg[i] = make_int2((int)klist.size(), (int)(b - a));
            for (int64_t j = a; j < b; ++j) klist.push_back(make_int2((int)j, 0));
            fseg[i] = make_int2((int)flist.size(), (int)(b - i));
            for (int64_t j = i; j < b; ++j) flist.push_back(make_int2((int)j, 0));
        }
        a = b;
    }
    JZ_TRY(t->super_spl.get(ac, sspl.size() * sizeof(int), s));
    JZ_TRY(t->knn_top_seg.get(ac, kseg.size() * sizeof(int2), s));
    JZ_TRY(t->knn_top_list.get(ac, klist.size() * sizeof(int2), s));
    JZ_TRY(t->fof_top_seg.get(ac, fseg.size() * sizeof(int2), s));
    JZ_TRY(t->fof_top_list.get(ac, flist.size() * sizeof(int2), s));
    JZ_HIP(hipMemcpyAsync(t->super_spl.p, sspl.data(), sspl.size() * sizeof(int),
                          hipMemcpyHostToDevice, s));
    JZ_HIP(hipMemcpyAsync(t->knn_top_seg.p, kseg.data(), kseg.size() * sizeof(int2),
                          hipMemcpyHostToDevice, s));
    JZ_HIP(hipMemcpyAsync(t->knn_top_list.p, klist.data(), klist.size() * sizeof(int2),
                          hipMemcpyHostToDevice, s));
    JZ_HIP(hipMemcpyAsync(t->fof_top_seg.p, fseg.data(), fseg.size() * sizeof(int2),
                          hipMemcpyHostToDevice, s));
    JZ_HIP(hipMemcpyAsync(t->fof_top_list.p, flist.data(), flist.size() * sizeof(int2),
                          hipMemcpyHostToDevice, s));
    JZ_HIP(hipStreamSynchronize(s));  // (the host arrays end here)
    return JZ_OK;
}

// the one-launch build of a small single set
static jz_status build_small(jz_tree *t, const float *points, int bits, hipStream_t s) {
    const AllocCtx *ac = &t->ac;
    const int64_t n = t->n;
    CallScope scope;
    DBuf d_hdr;
    JZ_TRY(d_hdr.get(ac, 8 * sizeof(int), s));
    JZ_TRY(t->pts4.get(ac, n * sizeof(float4), s));
    JZ_TRY(t->spl[0].get(ac, (n + 1) * sizeof(int), s));
    JZ_TRY(t->nodes[0].get(ac, n * sizeof(Node), s));  // (a leaf holds a point at least)
    k_build_small<<<1, SMALL_NT, 0, s>>>(points, (int)n, bits, t->opts.leaf_max,
                                         t->pts4.as<float4>(), t->spl[0].as<int>(),
                                         t->nodes[0].as<Node>(), d_hdr.as<int>());
    JZ_HIP(hipGetLastError());
    HostCopy hdr;
    JZ_TRY(hdr.read(d_hdr.p, 8 * sizeof(int), s));
    const int *h = hdr.as<int>();
    JZ_TRY(check_box(h + 1, t->opts));
    t->L[0] = h[0] - 1;
    t->P = 1;
    JZ_TRY(top_lists(t, nullptr, 0, s));
    JZ_HIP(hipStreamSynchronize(s));
    set_stats(t);
    return scope.done();
}

jz_status build_tree(jz_tree *t, const float *points, hipStream_t s) {
    const int64_t n = t->n;
    const AllocCtx *ac = &t->ac;
    const jz_build_opts &o = t->opts;
    t->P = 0;
    if (n == 0) return JZ_OK;

    const int has_sets = t->nsets > 1;
    // automatic key bits: 5 more per dimension than an even split of n
    // points needs (cells 32 times finer than the mean spacing), raised to
    // as many as the radix passes those need can hold (a pass sorts 8 key
    // bits; set bits come first), at most 21
    int bits = o.key_bits;
    if (bits == 0) {
        int lg = 0;
        while (lg < 62 && ((int64_t)1 << lg) < n) ++lg;
        const int b0 = std::max(10, (lg + 2) / 3 + 5);
        const int np = (3 * b0 + t->set_bits + 7) / 8;
        bits = std::min(21, std::max(b0, (8 * np - t->set_bits) / 3));
    }
    const int max_bits = (63 - t->set_bits) / 3;
    if (bits > max_bits) bits = max_bits;
    const int bits3 = 3 * bits;
    const int total_bits = bits3 + t->set_bits;
    const int npass = (total_bits + 7) / 8;

    const int P = plan_planes(n, o);
    const bool reg = o.reg_fmax > 0.0f;
    if (n <= SMALL_N && !has_sets && P == 1 && !reg && !o.keep_keys &&
        bits3 + SMALL_IDX_BITS <= 64)
        return build_small(t, points, bits, s);

    // 1-2: bbox, keys, histograms. d_meta: bounding box and non-finite flag
    // (8 words), then the number of splits of every plane
    CallScope scope;
    DBuf d_meta, k0, k1, v0, v1;
    SortScratch sc;
    JZ_TRY(d_meta.get(ac, (8 + JZ_MAX_PLANES + 2) * sizeof(int), s));
    int *const bbox = d_meta.as<int>(), *const cnts = bbox + 8;
    JZ_TRY(sc.get(ac, n, npass, s));
    JZ_TRY(k0.get(ac, n * sizeof(uint64_t), s));
    JZ_TRY(k1.get(ac, n * sizeof(uint64_t), s));
    JZ_TRY(v0.get(ac, n * sizeof(uint32_t), s));
    JZ_TRY(v1.get(ac, n * sizeof(uint32_t), s));
    k_build_init<<<std::min<unsigned>(blocks_for((int64_t)sc.words(), 256), 1024), 256, 0, s>>>(
        sc.buf.as<unsigned long long>(), sc.words(), bbox);
    // (a block ends in seven atomics on the same words: a block per 1024 points,
    // up to 1024 blocks, took 27 us at 10^6 points and 31 at 2^22; a block per
    // 8192, at least 128, takes 13 and 23; all 1024 at 2^24 take 53, 512 take 61)
    const int64_t bb = std::min<int64_t>(std::max<int64_t>(n / 8192, 128), 1024);
    k_bbox<<<(unsigned)std::min<int64_t>(blocks_for(n, 256 * 8), bb), 256, 0, s>>>(points, n, bbox);
    k_morton<<<std::min<unsigned>(blocks_for(n, 256 * 8), 2048), 256, 0, s>>>(
        points, n, bbox, bits, t->d_set_off.as<int64_t>(), t->nsets, npass, k0.as<uint64_t>(),
        v0.as<uint32_t>(), sc.hist());
    JZ_HIP(hipGetLastError());

    // 3: radix sort
    {
        uint64_t *kin = k0.as<uint64_t>(), *kout = k1.as<uint64_t>();
        uint32_t *vin = v0.as<uint32_t>(), *vout = v1.as<uint32_t>();
        JZ_TRY(onesweep_passes(sc, kin, vin, kout, vout, n, s));
        // sorted data is in (kin, vin)
        if (kin != k0.as<uint64_t>()) {
            std::swap(k0.p, k1.p);
            std::swap(v0.p, v1.p);
        }
    }
    const uint64_t *keys = k0.as<uint64_t>();
    const uint32_t *order = v0.as<uint32_t>();

    // 4: sorted points
    JZ_TRY(t->pts4.get(ac, n * sizeof(float4), s));
    k_gather<<<blocks_for(n, 256), 256, 0, s>>>(points, order, n, t->pts4.as<float4>());

    // 5: leaf plane
    const int64_t ngaps = n + 1;
    const unsigned nb = blocks_for(ngaps, LF_TILE);
    DBuf d_flags, d_bcnt, d_boff;
    JZ_TRY(d_flags.get(ac, ngaps, s));
    JZ_TRY(d_bcnt.get(ac, (size_t)nb * sizeof(int), s));
    JZ_TRY(d_boff.get(ac, (size_t)nb * sizeof(int), s));
    JZ_TRY(t->spl[0].get(ac, ngaps * sizeof(int), s));
    k_leaf_flags<<<nb, 256, 0, s>>>(keys, n, bits3, has_sets, o.leaf_max, d_flags.as<uint8_t>(),
                                    d_bcnt.as<int>());
    k_scan_counts<<<1, 1024, 0, s>>>(d_bcnt.as<int>(), (int)nb, d_boff.as<int>(), cnts + 0);
    k_compact<<<nb, 256, 0, s>>>(d_flags.as<uint8_t>(), ngaps, nullptr, d_boff.as<int>(),
                                 t->spl[0].as<int>(), nullptr, nullptr);
    JZ_HIP(hipGetLastError());
    // regularization: the largest level each plane's nodes may have
    DBuf d_hist2;
    int lvl_max = 1000;
    auto plane_level_max = [&](const int *lsi, const int *cnt_dev) -> jz_status {
        JZ_TRY(zero_words(d_hist2.as<unsigned long long>(), 256, s));
        k_level_hist<<<blocks_for(ngaps, 256), 256, 0, s>>>(keys, t->spl[0].as<int>(), lsi,
                                                            cnt_dev, bits3, has_sets,
                                                            d_hist2.as<unsigned long long>());
        unsigned long long h[256];
        JZ_HIP(hipMemcpyAsync(h, d_hist2.p, sizeof(h), hipMemcpyDeviceToHost, s));
        JZ_HIP(hipStreamSynchronize(s));
        lvl_max = std::max(lvl_max == 1000 ? 0 : lvl_max, reg_level_max(h, o.reg_fmax));
        return JZ_OK;
    };
    if (reg) {
        JZ_TRY(d_hist2.get(ac, 256 * sizeof(unsigned long long), s));
        JZ_TRY(plane_level_max(nullptr, cnts + 0));
        k_reg_leaf_flags<<<nb, 256, 0, s>>>(keys, n, bits3, has_sets, lvl_max,
                                            d_flags.as<uint8_t>(), d_bcnt.as<int>());
        k_scan_counts<<<1, 1024, 0, s>>>(d_bcnt.as<int>(), (int)nb, d_boff.as<int>(), cnts + 0);
        k_compact<<<nb, 256, 0, s>>>(d_flags.as<uint8_t>(), ngaps, nullptr, d_boff.as<int>(),
                                     t->spl[0].as<int>(), nullptr, nullptr);
        JZ_HIP(hipGetLastError());
    }
    HostCopy meta;  // bounding box, non-finite flag, leaf splits
    JZ_TRY(meta.read(bbox, 9 * sizeof(int), s));
    const int *hm = meta.as<int>();
    JZ_TRY(check_box(hm, o));
    const int64_t m0 = hm[8];  // L0 + 1
    t->L[0] = m0 - 1;

    // 6-7: node sizes at leaf splits, coarser planes
    if (P > 1) {
        CallScope planes;
        DBuf d_nsz, d_slv, lsiA, lsiB;
        JZ_TRY(d_nsz.get(ac, m0 * sizeof(int), s));
        JZ_TRY(d_slv.get(ac, m0, s));
        k_split_sizes<<<blocks_for(m0, 256), 256, 0, s>>>(
            keys, n, bits3, has_sets, t->spl[0].as<int>(), cnts + 0, o.leaf_max, d_nsz.as<int>(),
            d_slv.as<uint8_t>());
        JZ_TRY(lsiA.get(ac, m0 * sizeof(int), s));
        JZ_TRY(lsiB.get(ac, m0 * sizeof(int), s));
        const unsigned nbp = blocks_for(m0, LF_TILE);
        int64_t nmax = o.leaf_max;
        for (int p = 1; p < P; ++p) {
            const int *lsi = p == 1 ? nullptr : lsiA.as<int>();
            nmax *= o.coarsen;
            JZ_TRY(t->spl[p].get(ac, m0 * sizeof(int), s));
            // with regularization a plane is selected twice: by counts, then
            // also splitting the levels above its nodes' lvl_max
            for (int pass = 0; pass < (reg ? 2 : 1); ++pass) {
                k_plane_flags<<<nbp, 256, 0, s>>>(lsi, cnts + p - 1, d_nsz.as<int>(),
                                                  nmax, d_slv.as<uint8_t>(),
                                                  pass ? lvl_max : 1000, d_flags.as<uint8_t>(),
                                                  d_bcnt.as<int>());
                k_scan_counts<<<1, 1024, 0, s>>>(d_bcnt.as<int>(), (int)nbp, d_boff.as<int>(),
                                                 cnts + p);
                k_compact<<<nbp, 256, 0, s>>>(d_flags.as<uint8_t>(), m0, cnts + p - 1,
                                              d_boff.as<int>(), t->spl[p].as<int>(), lsi,
                                              lsiB.as<int>());
                if (reg && pass == 0) JZ_TRY(plane_level_max(lsiB.as<int>(), cnts + p));
            }
            std::swap(lsiA.p, lsiB.p);
        }
        JZ_HIP(hipGetLastError());
        JZ_TRY(meta.read(cnts, P * sizeof(int), s));
        hm = meta.as<int>();
        for (int p = 0; p < P; ++p) t->L[p] = hm[p] - 1;
        (void)planes.done();  // (the read has waited for them)
    }
    t->P = P;

    // 8: geometry
    for (int p = 0; p < P; ++p) {
        JZ_TRY(t->nodes[p].get(ac, t->L[p] * sizeof(Node), s));
        if (p == 0)
            k_leaf_geom<<<blocks_for(t->L[0] * 64, 256), 256, 0, s>>>(
                t->pts4.as<float4>(), t->spl[0].as<int>(), t->L[0], t->nodes[0].as<Node>());
        else
            k_node_geom<<<blocks_for(t->L[p] * 64, 256), 256, 0, s>>>(
                t->nodes[p - 1].as<Node>(), t->spl[p].as<int>(), t->L[p], t->nodes[p].as<Node>());
    }
    JZ_HIP(hipGetLastError());

    // super nodes over the top plane, per set
    JZ_TRY(top_lists(t, keys, bits3, s));
    if (o.keep_keys) {
        JZ_TRY(t->keys.get(ac, n * sizeof(uint64_t), s));
        JZ_HIP(hipMemcpyAsync(t->keys.p, keys, n * sizeof(uint64_t), hipMemcpyDeviceToDevice, s));
    }
    JZ_HIP(hipStreamSynchronize(s));

    set_stats(t);
    return scope.done();
}
