// Exact kNN by a dual walk over the tree planes (paper: kNN section, Alg. 1-3,
// Eq. 14-16, and the implementation-details subsection on r_low ordering).
//
// Level step (one wave per work item: a receiving parent and up to 4 of its
// children, the same for every lane; lanes = the children of the parent's
// sources):
//   FindRmax: R = smallest radius whose cumulative count reaches k (Alg. 3)
//   count children pairs with d_low^2 <= R
//   insert them (with r_low = d_low^2) into the next list, at an offset
//   reserved with one atomic per wave
// The paper's separate Count / prefix-sum / Insert launches become one kernel.
// Only the sources within the radii that the parent's own children give are
// expanded; a long list, put in r_low order in HBM before the level, is left
// at the first entries beyond them.
//
// Leaf stage (one wave per receiving leaf; lanes = its query points): the own
// leaf, then source leaves in r_low order, staged in LDS as float4; every lane
// keeps its top-k as packed (dist2 bits, index) u64 keys in registers.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <type_traits>
#include <vector>

#include "jz_device.h"
#include "jz_internal.h"

namespace {

constexpr int LCAP = 256;  // list entries staged (and sorted) in LDS per wave
constexpr uint64_t PAD_KEY = (0x7f800000ull << 32) | 0xffffffffull;  // (+inf, no index)

__device__ __forceinline__ uint64_t list_key(int2 e) {
    return ((uint64_t)(uint32_t)e.y << 32) | (uint32_t)e.x;  // r_low >= 0: bits order as floats
}

// Lists longer than a wave can sort in its LDS scratch are put in order in
// HBM before they are walked: k_find_long collects the receivers whose list
// length lies in (min_len, mid] and in (mid, max_len], and k_sort_lists
// sorts each such list in place in LDS, one workgroup per list: SORT_MID_WAVES
// waves for lists of at most SORT_MID entries, SORT_WAVES for longer ones (up to
// SORT_MAX). There are rarely more than a few hundred such lists, so one list's
// steps are what a launch takes: with one wave (49 us) and eight (81 us) the walk
// with its sorts took 0.46 ms at 10^6 clustered points, k = 32, now 0.39; 0.80 at
// 4 10^6 periodic ones, now 0.67; 0.19 at 3 10^5, now 0.16. (Sixteen for both, in
// one launch, is as fast there but loses 1 % of a call where a forest has
// thousands of the shorter lists.)
constexpr int SORT_MID = 1024;
constexpr int SORT_MID_WAVES = 8;
constexpr int SORT_MAX = 8192;
constexpr int SORT_WAVES = 16;

__global__ __launch_bounds__(64) void k_find_long(const int2 *__restrict__ seg, int n,
                                                  int min_len, int mid, int max_len,
                                                  int *__restrict__ ids_a,
                                                  unsigned long long *__restrict__ count_a,
                                                  int *__restrict__ ids_b,
                                                  unsigned long long *__restrict__ count_b) {
    const int lane = lane_id();
    const int i = blk_x() * 64 + lane;
    const int len = i < n ? seg[i].y : 0;
    const bool la = len > min_len && len <= mid, lb = len > mid && len <= max_len;
    const uint64_t ma = __ballot(la), mb = __ballot(lb);
    if (ma) {
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(count_a, (unsigned long long)__popcll(ma));
        base = uni((unsigned long long)__shfl(base, 0, 64));
        if (la) ids_a[base + __popcll(ma & lanemask_lt())] = i;
    }
    if (mb) {
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(count_b, (unsigned long long)__popcll(mb));
        base = uni((unsigned long long)__shfl(base, 0, 64));
        if (lb) ids_b[base + __popcll(mb & lanemask_lt())] = i;
    }
}

// The receivers whose lists are longer than min_len, in any order: the leaf
// stage runs them first, so that these long waves overlap the rest of the
// launch instead of trailing it.
__global__ __launch_bounds__(64) void k_long_first(const int2 *__restrict__ seg, int n,
                                                   int min_len, int *__restrict__ ids,
                                                   unsigned long long *__restrict__ count) {
    const int lane = lane_id();
    const int i = blk_x() * 64 + lane;
    const bool l = i < n && seg[i].y > min_len;
    const uint64_t m = __ballot(l);
    if (!m) return;
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(count, (unsigned long long)__popcll(m));
    base = uni((unsigned long long)__shfl(base, 0, 64));
    if (l) ids[base + __popcll(m & lanemask_lt())] = i;
}

// Bitonic sort of each listed segment by (r_low, source), in CAP keys of LDS,
// by NW waves. A compare-exchange step of pair distance j touches, for pair
// indices in one aligned range of PW = M / 2 / NW pairs, only the elements of
// one aligned range of 2 PW: steps with j <= PW run wave by wave without a
// workgroup barrier, so only the few steps of larger j pay one.
template <int CAP, int NW>
__global__ __launch_bounds__(64 * NW) void k_sort_lists(int2 *__restrict__ list,
                                                        const int2 *__restrict__ seg,
                                                        const int *__restrict__ ids,
                                                        const unsigned long long *__restrict__ count) {
    __shared__ uint64_t s[CAP];
    constexpr int NT = 64 * NW;
    const int tid = tid_x(), lane = tid & 63, w = tid >> 6;
    const long long nl = (long long)*count;
    for (long long jl = blk_x(); jl < nl; jl += nblk_x()) {
        const int2 sg = seg[ids[jl]];
        int2 *g = list + sg.x;
        const int len = sg.y;
        int M = 2 * NW;
        while (M < len) M <<= 1;
        for (int i = tid; i < M; i += NT) s[i] = i < len ? list_key(g[i]) : ~0ull;
        __syncthreads();
        const int PW = (M >> 1) / NW;
        for (int k = 2; k <= M; k <<= 1) {
            for (int j = k >> 1; j > 0; j >>= 1) {
                const bool wide = j > PW;
                // a wide step reads what other waves wrote in the steps before
                if (wide) __syncthreads();
                const int i0 = wide ? tid : w * PW + lane;
                const int i1 = wide ? (M >> 1) : (w + 1) * PW;
                const int di = wide ? NT : 64;
                for (int i = i0; i < i1; i += di) {
                    const int a = ((i & ~(j - 1)) << 1) | (i & (j - 1));
                    const int b = a + j;
                    const uint64_t x = s[a], y = s[b];
                    const bool up = (a & k) == 0;
                    if ((x > y) == up) {
                        s[a] = y;
                        s[b] = x;
                    }
                }
                if (wide) __syncthreads();
                else wave_lds_sync();
            }
        }
        __syncthreads();
        for (int i = tid; i < len; i += NT) {
            const uint64_t e = s[i];
            g[i] = make_int2((int)(uint32_t)e, (int)(uint32_t)(e >> 32));
        }
        __syncthreads();
    }
}

// The walk's work items: a receiving parent with more than cb children is
// split into items of cb children (each a wave of its own, reading the
// parent's list), so that the few parents with many children and long lists
// do not leave one wave running long after the rest of the level, and so
// that the upper levels, with few parents, still fill the device. cb is at
// most WALK_CB.
constexpr int WALK_CB = 4;
constexpr int WALK_CB_UP = 2;
// A parent whose list is longer than WALK_LONG entries takes items of at most
// WALK_CB_LONG children: such items run many times longer than the rest and
// would otherwise be the tail of the level.
constexpr int WALK_LONG = 1024;
constexpr int WALK_CB_LONG = 2;
__device__ __forceinline__ int item_cb(int cb, int len) {
    return len > WALK_LONG ? min(cb, WALK_CB_LONG) : cb;
}

__global__ __launch_bounds__(64) void k_walk_items(const int *__restrict__ par_spl, int n_par,
                                                   int cb, const int2 *__restrict__ seg_in,
                                                   int2 *__restrict__ items,
                                                   unsigned long long *__restrict__ count) {
    const int lane = lane_id();
    const int P = blk_x() * 64 + lane;
    int c0 = 0, nb = 0, cbe = cb;
    if (P < n_par) {
        c0 = par_spl[P];
        cbe = item_cb(cb, seg_in[P].y);
        nb = max(1, (par_spl[P + 1] - c0 + cbe - 1) / cbe);
    }
    const int incl = wave_incl_scan(nb);
    const int tot = uni(__shfl(incl, 63, 64));
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(count, (unsigned long long)tot);
    base = uni((unsigned long long)__shfl(base, 0, 64));
    for (int b = 0; b < nb; ++b)
        items[base + (unsigned long long)(incl - nb + b)] = make_int2(P, c0 + b * cbe);
}

constexpr int FCAP = 1024;  // source children listed in LDS at a time
// Lists longer than this (and up to sort_max) are put in r_low order in HBM
// before a wave walks them; a shorter one is at most 8 loads per phase.
constexpr int WALK_PRESORT = 512;

// Level step of the kNN walk: one wave per work item, a receiving parent P and
// up to WALK_CB of its children. The children's boxes are uniform, in scalar
// registers (38 of these do not fit and are read back from a lane of a vector
// register, one instruction each); the source children go through the lanes,
// 64 node records at a time.
//   phase 0  FindRmax: every lane keeps, per receiving child, the two smallest
//            (d_up^2, count) it has met; the smallest of them over the wave are
//            added up until the count reaches k (Alg. 3; leaving any out keeps
//            the radius an upper bound). P's own children come first: with the
//            radii they give, most of P's list is not expanded at all
//   phase 1  count pairs with d_low^2 <= R: a compare per 64 pairs
//   phase 2  insert them (with r_low = d_low^2) at offsets reserved with one
//            atomic per wave; a child's entries are contiguous
// The indices of the listed sources' children are expanded into LDS, FCAP at a
// time (nearly always once for all phases), each batch's records loaded while
// the one before is worked on.
// With the receiving children in the lanes and the source records staged
// through LDS, the level spent its time waiting for a chain of loads and LDS
// steps per batch of 128, and merging heaps: 0.20 + 0.27 + 0.46 + 2.21 ms from
// the top to the leaf level at 2^24 clustered points, k = 16, now 0.04 + 0.06 +
// 0.19 + 0.96 (8 children per item instead of 4: 0.05 + 0.07 + 0.27 + 0.92 to
// 1.03, and 0.11 ms instead of 0.07 for the one level of 5 10^4 points); 0.37 +
// 0.27 ms at 10^6 uniform points, now 0.09 + 0.06.
template <bool PER>
__global__ __launch_bounds__(64 * WPB) void k_knn_step(
    const int2 *__restrict__ items, const unsigned long long *__restrict__ n_items, int cb,
    const int2 *__restrict__ seg_in, const int2 *__restrict__ list_in,
    const int *__restrict__ par_spl, const Node *__restrict__ nodes, int k,
    int2 *__restrict__ seg_out, int2 *__restrict__ list_out,
    unsigned long long *__restrict__ ctr, long long cap, unsigned long long *overflow,
    int sorted_min, int sorted_max, const int *__restrict__ scnt, float Lp,
    float *__restrict__ rout) {
    __shared__ int s_fi[WPB][FCAP];
    const int w = WPB == 1 ? 0 : uni((int)(tid_x() >> 6)), lane = tid_x() & 63;
    // work item I: receiving parent it.x, its children from it.y (at most
    // item_cb(cb, list length) of them)
    const int I = xcd_block(blk_x(), nblk_x()) * WPB + w;
    if (I >= (int)uni(*n_items)) return;
    const int2 it = items[I];
    const int P = uni(it.x);
    const int2 sg = seg_in[P];
    const int2 *gl = list_in + uni(sg.x);
    const int len = uni(sg.y);
    // (a list of these lengths is in r_low order: the walk stops at the first
    // 64 entries that hold none within its radius)
    const bool sorted = len > sorted_min && len <= sorted_max;
    const int p0 = uni(par_spl[P]), p1 = uni(par_spl[P + 1]);
    const int c0 = uni(it.y), nc = uni(min(p1, it.y + item_cb(cb, len))) - c0;
    int *FI = s_fi[w];

    Node me[WALK_CB];
    bool act[WALK_CB];   // (uniform) receives anything
    float R[WALK_CB];    // (uniform) radius
    int cnt[WALK_CB];    // (uniform) entries, then insert position
    float r0[WALK_CB], r1[WALK_CB];
    int n0[WALK_CB], n1[WALK_CB];
#pragma unroll
    for (int j = 0; j < WALK_CB; ++j) {
        const int c = c0 + min(j, nc - 1);
        me[j] = nodes[c];
        // with separate point types, a child without query points receives
        // nothing
        act[j] = j < nc && (!scnt || uni(me[j].count) > uni(scnt[c]));
        R[j] = INFINITY;
        cnt[j] = 0;
        r0[j] = r1[j] = INFINITY;
        n0[j] = n1[j] = 0;
    }
    float Rw = INFINITY;  // largest radius of the receiving children
    // radii from what the lanes have kept
    auto radii = [&]() __attribute__((always_inline)) {
        Rw = -INFINITY;
#pragma unroll
        for (int j = 0; j < WALK_CB; ++j) {
            if (!act[j]) continue;
            float a = r0[j], b = r1[j];
            int na = n0[j], nb = n1[j], acc = 0;
            for (;;) {
                const float m = uni(wave_min(a));
                if (!(m < R[j])) break;
                const int l = __ffsll((unsigned long long)__ballot(a == m)) - 1;
                acc += __builtin_amdgcn_readlane(na, l);
                if (acc >= k) {
                    R[j] = m;
                    break;
                }
                const bool mine = lane == l;
                a = mine ? b : a;
                na = mine ? nb : na;
                b = mine ? INFINITY : b;
            }
            Rw = fmaxf(Rw, R[j]);
        }
    };

    // the stream of source children: P's own, then those of the listed sources
    // within Rw, in the order of the list
    int own = 0, t = 0, skip = 0, nN = 0;
    auto fill_own = [&]() __attribute__((always_inline)) {
        const int c = min(FCAP - nN, p1 - p0 - own);
        for (int f = lane; f < c; f += 64) FI[nN + f] = p0 + own + f;
        own += c;
        nN += c;
    };
    auto fill_list = [&]() __attribute__((always_inline)) {
        list_children<FCAP>(gl, len, par_spl, FI, nN, t, skip,
                            [&](const int2 &e, bool valid, bool &stop) {
                                const bool in = valid && __int_as_float(e.y) <= Rw;
                                stop = sorted && !__ballot(in);
                                return in && e.x != P;
                            });
    };
    long long base = 0;
    bool single = true;  // the whole stream fits FI
    for (int phase = 0; phase < 3; ++phase) {
        if (phase == 1) {
            // the leaf level keeps each child's radius for the leaf stage: k
            // points lie within R of every point of the child
#pragma unroll
            for (int j = 0; j < WALK_CB; ++j)
                if (rout && act[j] && lane == 0) rout[c0 + j] = R[j];
        }
        if (phase == 2) {
            int total = 0;
#pragma unroll
            for (int j = 0; j < WALK_CB; ++j) total += cnt[j];
            // segment in arena I % LIST_ARENAS (cap entries each)
            const int ar = I & (LIST_ARENAS - 1);
            unsigned long long lb = 0;
            if (lane == 0) lb = atomicAdd(ctr + ar, (unsigned long long)total);
            lb = uni(lb);
            base = (long long)((unsigned long long)ar * (unsigned long long)cap + lb);
            const bool ok = (long long)lb + total <= cap;
            // an overflowing level makes every list below it incomplete: flag
            // it, so that the leaf stage of this attempt exits at once
            if (!ok && lane == 0) *overflow = 1;
            int off = 0;
#pragma unroll
            for (int j = 0; j < WALK_CB; ++j) {
                if (j < nc && lane == 0)
                    seg_out[c0 + j] = ok ? make_int2((int)(base + off), cnt[j]) : make_int2(0, 0);
                const int c = cnt[j];
                cnt[j] = off;
                off += c;
            }
            if (!ok || total == 0) break;
        }
        int b0 = 0;
        bool first = phase == 0;  // P's own children alone, then the list
        if (phase == 0 || !single) own = t = skip = nN = 0;
        for (;;) {
            if (phase == 0 || !single) {
                if (own < p1 - p0) fill_own();
                if (!first && own == p1 - p0) fill_list();
            }
            wave_lds_sync();
            // node records of positions b + lane, loaded one batch ahead
            int x = 0, nx = 0;
            float4 ra = make_float4(0, 0, 0, 0), rb = ra, na = ra, nb = ra;
            auto load = [&](int b) __attribute__((always_inline)) {
                if (b + lane < nN) {
                    nx = FI[b + lane];
                    const float4 *rec = reinterpret_cast<const float4 *>(nodes + nx);
                    na = rec[0];
                    nb = rec[1];
                    if (scnt) nb.w = __int_as_float(scnt[nx]);  // Node.count is the last word
                }
            };
            load(b0);
            for (int b = b0; b < nN; b += 64) {
                x = nx;
                ra = na;
                rb = nb;
                load(b + 64);
                Node o;
                o.lo[0] = ra.x; o.lo[1] = ra.y; o.lo[2] = ra.z;
                o.hi[0] = rb.x; o.hi[1] = rb.y; o.hi[2] = rb.z;
                o.start = 0;
                o.count = b + lane < nN ? __float_as_int(rb.w) : 0;
#pragma unroll
                for (int j = 0; j < WALK_CB; ++j) {
                    if (!act[j]) continue;
                    if (phase == 0) {
                        float r = box_up2_m<PER>(me[j], o, Lp);
                        const bool in = o.count > 0 && r < R[j];
                        if (!__ballot(in)) continue;
                        r = in ? r : INFINITY;
                        const bool lt0 = r < r0[j];
                        const float tr = lt0 ? r0[j] : r;
                        const int tn = lt0 ? n0[j] : o.count;
                        r0[j] = lt0 ? r : r0[j];
                        n0[j] = lt0 ? o.count : n0[j];
                        const bool lt1 = tr < r1[j];
                        r1[j] = lt1 ? tr : r1[j];
                        n1[j] = lt1 ? tn : n1[j];
                    } else {
                        const float lo = box_low2_m<PER>(me[j], o, Lp);
                        const bool in = o.count > 0 && lo <= R[j];
                        const uint64_t m = __ballot(in);
                        if (phase == 2 && in)
                            list_out[base + cnt[j] + (int)__popcll(m & lanemask_lt())] =
                                make_int2(x, __float_as_int(lo));
                        cnt[j] += (int)__popcll(m);
                    }
                }
            }
            if (phase == 0) radii();
            if (phase > 0 && single) break;
            if (first && own == p1 - p0 && nN < FCAP) {
                first = false;
                b0 = nN;
                continue;
            }
            first = false;
            if (own == p1 - p0 && t >= len) break;
            wave_lds_sync();
            nN = b0 = 0;
            single = false;
        }
    }
}

// Top-k keys are (dist2 bits << 32 | index). dist2 >= 0 is never NaN, so the
// key's top 12 bits are never 0x7FF and, read as an IEEE double, every key is
// a non-negative non-NaN number (small keys are subnormal doubles, which this
// file's kernels keep). For such doubles the numeric order is the unsigned
// integer order of the bits, so the lists are kept as doubles and ordered
// with v_min_f64 / v_max_f64 (one instruction each, no 64-bit integer
// compare-and-select pairs).
__device__ __forceinline__ double key_of(float dd, int idx) {
    return __builtin_bit_cast(double, ((uint64_t)__float_as_uint(dd) << 32) | (uint32_t)idx);
}
__device__ __forceinline__ uint64_t bits_of(double k) { return __builtin_bit_cast(uint64_t, k); }
__device__ __forceinline__ float key_dist(double k) {
    return __uint_as_float((uint32_t)(bits_of(k) >> 32));
}

constexpr int next_pow2(int k) {
    int m = 1;
    while (m < k) m <<= 1;
    return m;
}

// An ascending list of K keys held in one or two vector registers tuples of
// at most 16 doubles. As a vector the list is one register tuple that the
// compiler updates in place; as an array of doubles every insertion renames
// the entries and loops pay a copy of the whole list per iteration.
template <int K>
struct TopK {
    static constexpr int W = K <= 16 ? next_pow2(K) : 16;
    static constexpr int NV = (K + W - 1) / W;
    typedef double vec __attribute__((ext_vector_type(W)));
    vec v[NV];
    __device__ __forceinline__ double get(int i) const { return v[i / W][i % W]; }
    __device__ __forceinline__ void set(int i, double x) { v[i / W][i % W] = x; }
};

// key of the lane at distance J (xor, a power of 2 below 64)
template <int J>
__device__ __forceinline__ double lane_xor_d(double v) {
    if constexpr (J == 32) return swap32_d(v);
    if constexpr (J == 16) return swap16_d(v);
    const uint64_t b = bits_of(v);
    int lo = (int)(uint32_t)b, hi = (int)(b >> 32);
    if constexpr (J == 1) {
        lo = dpp_i<DPP_XOR1>(lo);
        hi = dpp_i<DPP_XOR1>(hi);
    } else if constexpr (J == 2) {
        lo = dpp_i<DPP_XOR2>(lo);
        hi = dpp_i<DPP_XOR2>(hi);
    } else if constexpr (J == 4) {
        // the mirror inside 8 lanes of the mirror inside 4
        lo = dpp_i<DPP_HALF_MIRROR>(dpp_i<DPP_MIRROR4>(lo));
        hi = dpp_i<DPP_HALF_MIRROR>(dpp_i<DPP_MIRROR4>(hi));
    } else {
        lo = dpp_i<DPP_XOR8>(lo);
        hi = dpp_i<DPP_XOR8>(hi);
    }
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// One step of a bitonic sort of NR * 64 keys, element r * 64 + lane in x[r]:
// pairs at distance J ordered by bit KK of the element's index.
template <int NR, int KK, int J>
__device__ __forceinline__ void lane_step(double (&x)[NR], int lane) {
    if constexpr (J >= 64) {
        constexpr int D = J / 64;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if (r & D) continue;
            const bool up = ((r * 64) & KK) == 0;
            const double lo = __builtin_fmin(x[r], x[r + D]), hi = __builtin_fmax(x[r], x[r + D]);
            x[r] = up ? lo : hi;
            x[r + D] = up ? hi : lo;
        }
    } else {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const double y = lane_xor_d<J>(x[r]);
            const bool up = KK < 64 ? (lane & KK) == 0 : ((r * 64) & KK) == 0;
            const bool take_min = ((lane & J) == 0) == up;
            x[r] = (x[r] < y) == take_min ? x[r] : y;
        }
    }
}
template <int NR, int KK, int J>
__device__ __forceinline__ void lane_merge(double (&x)[NR], int lane) {
    lane_step<NR, KK, J>(x, lane);
    if constexpr (J > 1) lane_merge<NR, KK, J / 2>(x, lane);
}
// NR * 64 keys of L (the entries from n on taken as padding) sorted ascending
// across the wave: 21, 28 or 36 steps of register exchanges for NR = 1, 2, 4,
// with no LDS round trip between them
template <int NR>
__device__ __forceinline__ void lane_sort(uint64_t *L, int n) {
    // (opaque, so that the steps' lane masks are not kept in registers)
    int lane = lane_id();
    asm volatile("" : "+v"(lane));
    double x[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r)
        x[r] = __builtin_bit_cast(double, r * 64 + lane < n ? L[r * 64 + lane] : PAD_KEY);
    lane_merge<NR, 2, 1>(x, lane);
    lane_merge<NR, 4, 2>(x, lane);
    lane_merge<NR, 8, 4>(x, lane);
    lane_merge<NR, 16, 8>(x, lane);
    lane_merge<NR, 32, 16>(x, lane);
    lane_merge<NR, 64, 32>(x, lane);
    if constexpr (NR >= 2) lane_merge<NR, 128, 64>(x, lane);
    if constexpr (NR >= 4) lane_merge<NR, 256, 128>(x, lane);
#pragma unroll
    for (int r = 0; r < NR; ++r) L[r * 64 + lane] = bits_of(x[r]);
}

// Leaf lists longer than this (and up to sort_max) are put in r_low order in
// HBM before the leaf stage; shorter ones it orders itself, as far as needed.
constexpr int LEAF_PRESORT = 2048;
// Leaves with lists longer than LEAF_FIRST run first (longer than 1024 in trees
// of more than LEAF_MANY leaves, whose launch has many waves to hide them
// behind): at 3 10^5 points the slowest leaves take most of the kernel, 0.37 ms
// at k = 32 with only those above 1024 first, 0.33 with those above 256. At 2^24
// points both give the same, and the lower one starts more waves that find
// their leaf done.
constexpr int LEAF_FIRST = 256;
constexpr int LEAF_MANY = 1 << 17;
// Up to this many leaves, four waves share each one's queries: the chip has 1024
// SIMDs, and a wave's time is a serial chain of drains (leaf stage at 4096
// clustered points, k = 8: 75 us with one wave, 65 with four; at 20 000, k = 32:
// 152 and 134; at 50 000, 1356 leaves, 230 with one and more with four, each
// staging every tile again).
constexpr int LEAF_FEW = 768;
constexpr int TILE_PTS = 255; // source points staged per batch (positions fit a byte)
constexpr int FILLER = 255;   // tile position of a point at infinity with the padding index
constexpr int HALF = 128;     // tile positions filtered at a time (32 blocks of 4 per lane row)
constexpr int CQ = 32;        // queued candidate positions per lane

// Keep the K smallest of two ascending key lists a and b in a (ascending).
// With both lists padded to M = next power of two, min(a[i], b[M-1-i]) is a
// bitonic sequence holding the M smallest of the padded union (so the K
// smallest of a and b); a bitonic sorter then orders it.
template <int K>
__device__ __forceinline__ void merge_topk(TopK<K> &a, const TopK<K> &b) {
    constexpr int M = next_pow2(K);
    const double pad = __builtin_bit_cast(double, PAD_KEY);
    double c[M];
#pragma unroll
    for (int i = 0; i < M; ++i) {
        const double x = i < K ? a.get(i) : pad;
        const double y = (M - 1 - i) < K ? b.get(M - 1 - i) : pad;
        c[i] = __builtin_fmin(x, y);
    }
#pragma unroll
    for (int d = M / 2; d > 0; d >>= 1) {
#pragma unroll
        for (int i = 0; i < M; ++i) {
            if ((i & d) == 0) {
                const double x = c[i], y = c[i + d];
                c[i] = __builtin_fmin(x, y);
                c[i + d] = __builtin_fmax(x, y);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < K; ++i) a.set(i, c[i]);
}

// Sort C keys ascending in registers (Batcher's odd-even merge sort, C a power
// of 2: 19 compare-exchanges for 8 keys, 63 for 16, where the bitonic network
// takes 24 and 80).
template <int C>
__device__ __forceinline__ void sort_keys(double (&a)[C]) {
#pragma unroll
    for (int p = 1; p < C; p <<= 1) {
#pragma unroll
        for (int k = p; k > 0; k >>= 1) {
#pragma unroll
            for (int i = 0; i < C; ++i) {
                // i joins i + k where i lies in the lower half of its group
                // of 2k (counted from k mod p) and both in one block of 2p
                if (i >= k % p && ((i - k % p) / k) % 2 == 0 && i + k < C &&
                    i / (2 * p) == (i + k) / (2 * p)) {
                    const double x = a[i], y = a[i + k];
                    a[i] = __builtin_fmin(x, y);
                    a[i + k] = __builtin_fmax(x, y);
                }
            }
        }
    }
}

// Merge an ascending chunk of C keys into the top-k list (as merge_topk, the
// chunk padded to M with padding keys).
template <int K, int C>
__device__ __forceinline__ void merge_chunk(TopK<K> &a, const double (&ch)[C]) {
    constexpr int M = next_pow2(K);
    if constexpr (M == K) {
        // in place: only the last min(C, M) entries meet a chunk key (a
        // chunk longer than the list contributes its M smallest keys)
#pragma unroll
        for (int i = (M > C ? M - C : 0); i < M; ++i)
            a.set(i, __builtin_fmin(a.get(i), ch[M - 1 - i]));
#pragma unroll
        for (int d = M / 2; d > 0; d >>= 1) {
#pragma unroll
            for (int i = 0; i < M; ++i) {
                if ((i & d) == 0) {
                    const double x = a.get(i), y = a.get(i + d);
                    a.set(i, __builtin_fmin(x, y));
                    a.set(i + d, __builtin_fmax(x, y));
                }
            }
        }
        return;
    }
    const double pad = __builtin_bit_cast(double, PAD_KEY);
    double c[M];
#pragma unroll
    for (int i = 0; i < M; ++i) {
        const double x = i < K ? a.get(i) : pad;
        c[i] = (M - 1 - i) < C ? __builtin_fmin(x, ch[M - 1 - i]) : x;
    }
#pragma unroll
    for (int d = M / 2; d > 0; d >>= 1) {
#pragma unroll
        for (int i = 0; i < M; ++i) {
            if ((i & d) == 0) {
                const double x = c[i], y = c[i + d];
                c[i] = __builtin_fmin(x, y);
                c[i + d] = __builtin_fmax(x, y);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < K; ++i) a.set(i, c[i]);
}

// The matrix filter of k_leaf_knn over the m <= HALF tile positions from ap
// (this lane's row and component of the first block of 16): wd[k] of a lane
// receives the hits of its own query at positions 4 j + W h + k, W = 4 / SS,
// bit j for position 4 j + W h + k; SS lanes per query, lane h of them.
template <int SS, bool PER>
__device__ __forceinline__ void filter_words(const float *ap, int m, int h, float ac, float aL,
                                             float Lh, const float (&bq)[4], float tq,
                                             unsigned (&wd)[4]) {
    constexpr int W = 4 / SS;
    // t of the queries 16 g + l % 16, from the lane rows that hold them
    const int ti = __float_as_int(-tq);
    int tg[4] = {ti, ti, ti, ti};
    if constexpr (SS < 4) {
        const auto x = __builtin_amdgcn_permlane16_swap(ti, ti, false, false);
        tg[0] = x[0];
        tg[1] = x[1];
    }
    if constexpr (SS == 1) {
        const auto y = __builtin_amdgcn_permlane32_swap(tg[0], tg[0], false, false);
        const auto z = __builtin_amdgcn_permlane32_swap(tg[1], tg[1], false, false);
        tg[0] = y[0];
        tg[1] = z[0];
        tg[2] = y[1];
        tg[3] = z[1];
    }
    v4f cq[W];
#pragma unroll
    for (int g = 0; g < W; ++g) {
        const float v = __int_as_float(tg[g]);
        cq[g] = v4f{v, v, v, v};
    }
    const int nblk = uni((m + 15) >> 4);
    for (int b = 0; b < nblk; ++b) {
        const float av = wrap_diff<PER>(ap[64 * b] - ac, aL, aL != 0.0f ? Lh : INFINITY);
        v4f d[W];
#pragma unroll
        for (int g = 0; g < W; ++g)
            d[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bq[g], cq[g], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int g = 0; g < W; ++g)
                wd[g] = __builtin_amdgcn_alignbit(wd[g], __float_as_uint(d[g][i]), 31);
    }
    // rows and groups transposed
    if constexpr (SS < 4) {
        const auto x = __builtin_amdgcn_permlane16_swap(wd[0], wd[1], false, false);
        wd[0] = x[0];
        wd[1] = x[1];
    }
    if constexpr (SS == 1) {
        const auto x = __builtin_amdgcn_permlane16_swap(wd[2], wd[3], false, false);
        const auto y = __builtin_amdgcn_permlane32_swap(wd[0], x[0], false, false);
        const auto z = __builtin_amdgcn_permlane32_swap(wd[1], x[1], false, false);
        wd[0] = y[0];
        wd[1] = z[0];
        wd[2] = y[1];
        wd[3] = z[1];
    }
#pragma unroll
    for (int k = 0; k < W; ++k) {
        // positions from m on hold no point of this batch
        const int nv = max((m - (W * h + k) + 3) >> 2, 0);
        wd[k] = __builtin_bitreverse32(wd[k] << (32 - 4 * nblk)) & (unsigned)((1ull << nv) - 1ull);
    }
}

// The same masks from the exact distances of all positions.
template <bool PER>
__device__ __forceinline__ void dense_words(const float4 *tp, int m, int W, int h, const float4 &me,
                                            float thr, float Lp, float Lh, unsigned (&wd)[4]) {
    for (int k = W - 1; k >= 0; --k) {
        const int r = W * h + k;
        wd[3] = wd[2];
        wd[2] = wd[1];
        wd[1] = wd[0];
        wd[0] = 0;
        for (int j = 0; 4 * j < m; ++j) {
            const float4 p = tp[4 * j + r];
            const float dd = dist2_m<PER>(me.x, me.y, me.z, p.x, p.y, p.z, Lp, Lh);
            wd[0] |= (4 * j + r < m && dd <= thr) ? 1u << j : 0u;
        }
    }
}

// Leaf stage, one wave per receiving leaf. A leaf of at most 16 (32) points
// gives each query 4 (2) lanes; the lanes of a query take interleaved slices
// of every staged tile, keep their own top-k, and prune with the smallest
// k-th distance of the group (the merged k-th can only be smaller), and their
// lists are merged at the end.
// The leaf's own points come first; then the list's entries within the largest
// radius that is left, in r_low order, their points staged in one LDS tile in
// batches of what fits it. After the first batch every entry's box is tested
// against all queries (point-to-box bound <= the group's k-th distance), and
// the entries that no query needs are dropped. The walk stops at the first
// source whose r_low exceeds every query's k-th distance.
// The tests run with one entry per lane and the queries broadcast: with one
// query per lane and the entries broadcast in windows of 16, each window waited
// for its Node records and retested what the tile had no room for, and single
// waves with 8300 reachable boxes and no needed one took the whole 1.4 ms of
// the kernel at 10^6 clustered points, k = 8 (then 0.67 ms; 2^24 points, k = 16:
// 7.48 -> 7.42 ms; 2^21 uniform points, k = 30: 1.69 -> 1.58 ms).
//
// Which of the tile's points may belong to a query's list is decided on the
// matrix cores: a filter on approximate distances that never drops a point
// within the k-th distance, whose hits are then evaluated with the fixed
// float32 expression. With q' = fl(q - c), p' = fl(p - c) (c: centre of the
// receiving leaf's box), one v_mfma_f32_16x16x4_f32 computes, for 16 points x
// 16 queries, D = -2 q'.p' + w - t, with w = |p'|^2 (1 - e) of the point and
// t = kth (1 + e) - |q'|^2 (1 - e) + tiny of the query; a hit is D < 0, and
// the hits are collected by shifting the sign bit of each result into a mask
// (one v_alignbit per result).
// (jz_device.h states why no point within the k-th distance is missed; the
// coordinates that the filter does not cover take the exact dense scan below.)
// Against per-lane box tests and exact evaluations on the vector unit (12
// instructions per position and wave, 30 % of the lanes in use) the filter
// costs one matrix instruction and four shifts per 16 x 16 pairs: at 2^24
// clustered points and k = 16 the kernel issues 4.3e9 vector instructions
// instead of 6.1e9 and takes 9.5 ms instead of 10.6; 2^21 uniform points,
// k = 30: 1.95 ms instead of 2.85. (With the own leaf first, the queue, the
// sorts and the box tests as they are below: 7.0 ms. Its 3.56e9 vector
// instructions would take 81 % of that at one per 4 cycles and SIMD, a rate that
// plain float code exceeds; for a third of their time the waves wait to issue
// an instruction.)
// Hits are queued as tile positions and inserted into the register top-k in
// rounds, so insert time follows the busiest lane rather than every accepted
// candidate of any lane.
//
// k > 32 takes several passes (the paper's LeafToLeaf with at most 32
// neighbours per call, called again for the next ones): a pass with LO finds
// the K smallest keys strictly above the last key of the previous pass (read
// back from column col0 - 1 of the output row), so that equal distances
// continue by index. A pass writes columns [col0, col0 + kw) of rows of
// out_stride entries.
//
// Waves per SIMD: 4 up to K = 16, 3 above, at 128 and 168 registers. Towards
// the upper end of both ranges registers spill (open from K = 13 and 27 on, 9 at
// K = 16 and 7 at 32; periodic from 9 and 23 on, 34 and 11), but one wave fewer,
// without spills, is slower or the same, and with no bound most kernels run two
// (ms of the leaf stage, as it is / one wave fewer / no bound):
//   2^24 clustered points, k = 16        6.94 / 7.41 / 9.88
//   2^21 uniform, k = 30                 1.50 / 1.72 / 1.75
//   10^6 clustered, k = 8                0.39 / 0.42 / 0.43
//   k = 24                               0.68 / 0.68 / 0.83
//   k = 32                               0.84 / 0.93 / 0.95
//   k = 64                               1.99 / 2.20 / 2.22
//   4 10^6 periodic, k = 16              2.36 / 2.36 / 3.00
//   10^6 periodic, k = 8                 0.52 / 0.54 / 0.68
//   k = 32                               1.09 / 1.18 / 1.93
//   k = 64                               2.53 / 2.76 / 3.61
template <int K, bool LO, bool PER>
__global__ __launch_bounds__(64 * WPB, K <= 16 ? 4 : 3) void k_leaf_knn(
    const int2 *__restrict__ seg, const int2 *__restrict__ list,
    const Node *__restrict__ leaves, const float4 *__restrict__ pts, int n_leaves,
    const int *__restrict__ leaf_base,
    int32_t *__restrict__ out_idx, float *__restrict__ out_d2,
    unsigned long long *__restrict__ stats, const unsigned long long *__restrict__ overflow,
    int presorted, int out_stride, int col0, int kw,
    const int *__restrict__ scnt0, int src_hi, int qry_lo, float Lp,
    const float *__restrict__ rleaf, const int *__restrict__ first,
    const unsigned long long *__restrict__ n_first, int first_len, int row_align, int lg_parts) {
    // Lp: period of the cube (PER), Lh its half
    const float Lh = 0.5f * Lp;
    // one block per wave: the staged list (LCAP entries), the point tile
    // (x, y, z and the filter's w), the points' indices and the candidate
    // queues
    constexpr int O_TILE = LCAP, O_IDX = O_TILE + (FILLER + 1) * 2, O_Q = O_IDX + (FILLER + 1) / 2;
    constexpr int RAW = O_Q + CQ * 64 / 8;
    __shared__ __align__(16) uint64_t s_raw[WPB][RAW];
    const int w = WPB == 1 ? 0 : uni((int)(tid_x() >> 6)), lane = tid_x() & 63;
    // the first waves take the leaves with lists longer than first_len (in
    // `first`), the others every leaf in order except those
    // (2^lg_parts waves share a leaf: part p answers a run of its queries)
    const int n_blk = nblk_x() >> lg_parts, part = blk_x() / n_blk;
    const int wv = xcd_block(blk_x() - part * n_blk, n_blk) * WPB + w;
    const int nfirst = (int)uni(*n_first);
    int A;
    if (wv < nfirst) {
        A = uni(first[wv]);
    } else {
        A = wv - nfirst;
        if (A >= n_leaves || uni(seg[A].y) > first_len) return;
    }
    // a level of this attempt overflowed (it is rerun): nothing to do
    if (*overflow) return;
    const Node a = leaves[A];
    uint64_t *L = s_raw[w];
    // The leaf's query points: all its points, or, with separate point types
    // (scnt0 given), those with index >= qry_lo; query j sits at leaf
    // position sel[j] (selected through the LDS queue area, unused so far).
    int acount = uni(a.count);
    const bool types = scnt0 != nullptr;
    const uint8_t *sel = reinterpret_cast<const uint8_t *>(L + O_Q);
    if (types) {
        const bool isq = lane < acount && __float_as_int(pts[a.start + lane].w) >= qry_lo;
        const uint64_t qm = __ballot(isq);
        if (isq) reinterpret_cast<uint8_t *>(L + O_Q)[__popcll(qm & lanemask_lt())] = (uint8_t)lane;
        acount = uni((int)__popcll(qm));
        wave_lds_sync();
    }
    const int part_q = 64 >> lg_parts, first_q = part * part_q;  // this wave's queries
    acount = min(acount - first_q, part_q);
    if (acount <= 0) return;
    const int lgS = acount <= 16 ? 2 : (acount <= 32 ? 1 : 0);  // log2 lanes per query
    const int q = lane & ((64 >> lgS) - 1), h = lane >> (6 - lgS);
    const bool act = q < acount;
    const int q_leaf = first_q + (act ? q : 0);
    const int qpos = types ? (int)sel[q_leaf] : q_leaf;
    const float4 me = pts[a.start + qpos];
    const int64_t row = (int64_t)__float_as_int(me.w) - qry_lo;
    const int base = leaf_base ? leaf_base[A] : 0;
    // keys at or below lo belong to earlier passes
    double lo = -1.0;
    if constexpr (LO) {
        if (act) {
            const int pi = out_idx[row * out_stride + col0 - 1];
            const float pd = out_d2[row * out_stride + col0 - 1];
            lo = pi < 0 ? __builtin_bit_cast(double, PAD_KEY) : key_of(pd, pi + base);
        }
    }
    const int2 sg = seg[A];
    const int2 *gl = list + uni(sg.x);
    const int len = uni(sg.y);
    float4 *tile = reinterpret_cast<float4 *>(L + O_TILE);
    const float *tilef = reinterpret_cast<const float *>(tile);
    int *tidx = reinterpret_cast<int *>(L + O_IDX);

    const double pad = __builtin_bit_cast(double, PAD_KEY);
    TopK<K> best;
#pragma unroll
    for (int i = 0; i < K; ++i) best.set(i, pad);
    unsigned visited = 0, rounds = 0, steps = 0;
    unsigned long long evals = 0;

    // The filter's query side. Lane l holds component l / 16 (x, y, z, 1) of
    // query 16 g + l % 16 in bq[g] (through LDS: the tile is not in use yet).
    const float cx = uni(0.5f * a.lo[0] + 0.5f * a.hi[0]);
    const float cy = uni(0.5f * a.lo[1] + 0.5f * a.hi[1]);
    const float cz = uni(0.5f * a.lo[2] + 0.5f * a.hi[2]);
    const float mx = me.x - cx, my = me.y - cy, mz = me.z - cz;
    const float qn2 = mx * mx + my * my + mz * mz;
    const float nq = qn2 * (1.0f - FILTER_E);
    const bool qbad = __ballot(act && !(qn2 < FILTER_BIG)) != 0;
    // (periodic) farthest coordinate of a query from c
    const float qfar = PER ? fmaxf(fmaxf(fabsf(mx), fabsf(my)), fabsf(mz)) : 0.0f;
    if (h == 0) tile[q] = make_float4(-2.0f * mx, -2.0f * my, -2.0f * mz, 1.0f);
    wave_lds_sync();
    float bq[4];
#pragma unroll
    for (int g = 0; g < 4; ++g)
        bq[g] = tilef[(((16 * g + (lane & 15)) & ((64 >> lgS) - 1)) << 2) + (lane >> 4)];
    wave_lds_sync();
    // the points' side: row m of a block of 16 tile positions reads position
    // 4 (m % 4) + m / 4 of it, so that result i of lane row r is position
    // 4 i + r and bit j of that row's mask position 4 j + r
    const int arow = (((lane & 3) << 2 | ((lane >> 2) & 3)) << 2) + (lane >> 4);
    const float ac = lane < 16 ? cx : (lane < 32 ? cy : (lane < 48 ? cz : 0.0f));
    const float aL = lane < 48 ? Lp : 0.0f;  // (periodic) no wrap of w
    // candidate queue of this lane: positions at q0, q0 + 64, ... up to qp
    // (LDS-typed pointers: 32-bit arithmetic instead of 64-bit)
    typedef __attribute__((address_space(3))) uint8_t lds_u8;
    lds_u8 *const q0 = (lds_u8 *)(reinterpret_cast<uint8_t *>(L + O_Q) + lane);
    lds_u8 *qp = q0;

    // the group's k-th distance: an upper bound of the query's final k-th
    // the walk's radius of this leaf: the k-th distance of each of its
    // points is at most R (k = all passes' neighbours, so it bounds every
    // pass), so nothing farther is ever needed
    const float Rleaf = uni(rleaf[A]);
    auto group_kth = [&]() __attribute__((always_inline)) {
        float v = key_dist(best.get(K - 1));
        if (lgS >= 1) v = fminf(v, swap32_f(v));
        if (lgS >= 2) v = fminf(v, swap16_f(v));
        return fminf(v, Rleaf);
    };
    // insert the queued candidates of every lane into its top-k: 8 at a time,
    // sorted in registers and merged (the busiest lane sets the trip count,
    // so batches of 8 cost far less than one insertion per candidate)
    // (inlined: outlined, the list it updates would live in scratch memory)
    auto drain = [&]() __attribute__((always_inline)) {
        const int qn = (int)(qp - q0) >> 6;
        // a scalar trip count (a loop on a ballot compiles to a divergent
        // loop, whose exit handling copies the list every round)
        const int nr = uni(wave_max_i(qn));
        for (lds_u8 *qc = q0; qc < q0 + 64 * nr; qc += 64 * 8) {
            rounds += 8;
            double ch[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int qv = qc[64 * u];
                qc[64 * u] = FILLER;
                const float4 s = tile[qv];
                const float dd = dist2_m<PER>(me.x, me.y, me.z, s.x, s.y, s.z, Lp, Lh);
                const double kk = key_of(dd, tidx[qv]);
                ch[u] = (!LO || kk > lo) ? kk : pad;
            }
            sort_keys<8>(ch);
            merge_chunk<K, 8>(best, ch);
        }
        qp = q0;
    };

    // The receiving leaf itself comes first (its r_low is 0): its source
    // points meet an empty top-k, where every point is accepted, so they are
    // merged in sorted chunks instead of being queued (lane h of a query's S
    // takes positions h, h + S, ...).
    int own = uni(a.count);
    if (types) {
        const float4 p = pts[a.start + min(lane, uni(a.count) - 1)];
        const bool real = lane < a.count && __float_as_int(p.w) < src_hi;
        const uint64_t rm = __ballot(real);
        own = uni((int)__popcll(rm));
        if (real) {
            const int pos = (int)__popcll(rm & lanemask_lt());
            tile[pos] = p;
            tidx[pos] = __float_as_int(p.w);
        }
    } else if (lane < own) {
        const float4 p = pts[a.start + lane];
        tile[lane] = p;
        tidx[lane] = __float_as_int(p.w);
    }
    wave_lds_sync();
    {
        constexpr int C = K < 8 ? next_pow2(K) : (K <= 16 ? 8 : 16);
        for (int j0 = 0; j0 < own; j0 += C << lgS) {
            double ch[C];
#pragma unroll
            for (int u = 0; u < C; ++u) {
                const int j = j0 + (u << lgS) + h;
                const float4 p = tile[j];
                const float dd = dist2_m<PER>(me.x, me.y, me.z, p.x, p.y, p.z, Lp, Lh);
                const double kk = key_of(dd, tidx[j]);
                ch[u] = (j < own && (!LO || kk > lo)) ? kk : pad;
            }
            sort_keys<C>(ch);
            merge_chunk<K, C>(best, ch);
        }
        evals += (unsigned)own * (unsigned)acount;
        visited += own > 0;
    }
    wave_lds_sync();

    // The rest of the list, in slices of at most LCAP entries within the
    // largest radius the queries have left (after the own leaf, 47 of the 155
    // entries of an average leaf at k = 16), each put in r_low order in L.
    // Almost every leaf has one slice, sorted in registers.
    const bool sorted = len > LEAF_PRESORT && len <= presorted;
    bool fresh = true;  // no batch has run yet
    for (int i0 = 0; i0 < len;) {
        int nl = 0;
        {
            const float Rw = uni(wave_max_f(act ? group_kth() : -INFINITY));
            int2 e = make_int2(0, 0);
            if (i0 + lane < len) e = gl[i0 + lane];
            while (i0 < len && nl <= LCAP - 64) {
                const int2 x = e;
                if (i0 + 64 + lane < len) e = gl[i0 + 64 + lane];
                const bool keep = i0 + lane < len && x.x != A && __int_as_float(x.y) <= Rw;
                const uint64_t m = __ballot(keep);
                if (keep) L[nl + __popcll(m & lanemask_lt())] = list_key(x);
                nl += (int)__popcll(m);
                // (in r_low order, and not just the own leaf: nothing follows)
                if (sorted && i0 > 0 && m == 0) i0 = len;
                i0 += 64;
            }
        }
        wave_lds_sync();
        if (nl <= 64) lane_sort<1>(L, nl);
        else if (nl <= 128) lane_sort<2>(L, nl);
        else lane_sort<4>(L, nl);
        // every queue slot that holds no candidate names the filler, whose key
        // is the padding key, so a drain takes whole rounds without looking at
        // the count
#pragma unroll
        for (int i = 0; i < CQ; ++i) q0[64 * i] = FILLER;
        if (lane == 0) {
            tile[FILLER] = make_float4(INFINITY, INFINITY, INFINITY, 0.0f);
            tidx[FILLER] = -1;
        }
        wave_lds_sync();
        // The slice in chunks of 64 entries, one per lane, each staged in batches
        // of what fits the tile. The nearest batch runs unseen; before the others,
        // with the radii it leaves, every lane tests its entry's box against all
        // queries, and the entries that no query reaches are dropped.
        for (int c0 = 0; c0 < nl; c0 += 64) {
            uint64_t pend = nl - c0 >= 64 ? ~0ull : (1ull << (nl - c0)) - 1ull;
            float4 n_lo = make_float4(0, 0, 0, 0), n_hi = n_lo;  // the entry's Node record
            float e_rl = INFINITY;
            int e_sc = 0;
            if (lane < nl - c0) {
                const uint64_t e = L[c0 + lane];
                const int src = (int)(uint32_t)e;
                e_rl = __uint_as_float((uint32_t)(e >> 32));
                const float4 *rec = reinterpret_cast<const float4 *>(leaves + src);
                n_lo = rec[0];
                n_hi = rec[1];
                e_sc = types ? scnt0[src] : __float_as_int(n_hi.w);
            }
            bool tested = false;
            while (pend) {
                float kth = group_kth();
                pend &= __ballot(e_rl <= uni(wave_max_f(act ? kth : -INFINITY)));
                if (!fresh && !tested && pend) {
                    // A query whose k-th distance is below every r_low of the chunk
                    // needs none of it: of the thousands of boxes that one far query
                    // brings within the leaf's radius, the others look at none (leaf
                    // stage of 10^6 clustered points, k = 8: 0.57 ms with every query
                    // looking at every box, 0.40 ms).
                    const float rl0 = uni(wave_min((pend >> lane) & 1ull ? e_rl : INFINITY));
                    const uint64_t qm = __ballot(h == 0 && act && kth >= rl0);
                    if ((qm >> lane) & 1ull)
                        tile[__popcll(qm & lanemask_lt())] = make_float4(me.x, me.y, me.z, kth);
                    wave_lds_sync();
                    bool need = false;
                    const int nq_near = (int)__popcll(qm);
#pragma unroll 4
                    for (int i = 0; i < nq_near; ++i) {
                        const float4 p = tile[i];
                        need |= point_low2_m<PER>(p.x, p.y, p.z, n_lo.x, n_lo.y, n_lo.z, n_hi.x,
                                                  n_hi.y, n_hi.z, Lp) <= p.w;
                    }
                    pend &= __ballot(need);
                    tested = true;
                    wave_lds_sync();
                }
                fresh = false;
                // take entries in order while their points fit the tile: position f
                // of the tile is point f + delta, delta changing with the source
                // (several loads per lane in flight; separate point types need the
                // packing of each leaf's source points and go source by source)
                int npts = 0;
                bool bad = qbad;
                auto stage = [&](const float4 &p, int pos) __attribute__((always_inline)) {
                    const float dx = wrap_diff<PER>(p.x - cx, Lp, Lh);
                    const float dy = wrap_diff<PER>(p.y - cy, Lp, Lh);
                    const float dz = wrap_diff<PER>(p.z - cz, Lp, Lh);
                    const float pw = (dx * dx + dy * dy + dz * dz) * (1.0f - FILTER_E);
                    tile[pos] = make_float4(p.x, p.y, p.z, pw);
                    tidx[pos] = __float_as_int(p.w);
                    bad = bad || !(pw < FILTER_BIG);
                };
                const int e_st = __float_as_int(n_lo.w);
                int at[4] = {0, 0, 0, 0};
                while (pend) {
                    const int qq = __ffsll((unsigned long long)pend) - 1;
                    const int c = __builtin_amdgcn_readlane(e_sc, qq);
                    if (npts + c > TILE_PTS) break;
                    pend &= pend - 1ull;
                    ++visited;
                    const int st = __builtin_amdgcn_readlane(e_st, qq);
                    if (types) {
                        if (lane < __builtin_amdgcn_readlane(__float_as_int(n_hi.w), qq)) {
                            const float4 p = pts[st + lane];
                            const bool real = __float_as_int(p.w) < src_hi;
                            const int pos = npts + (int)__popcll(__ballot(real) & lanemask_lt());
                            if (real) stage(p, pos);
                        }
                    } else {
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (u * 64 + lane >= npts) at[u] = st - npts;
                    }
                    npts += c;
                }
                if (!types) {
#pragma unroll
                    for (int v = 0; v < 4; v += 2) {
                        float4 p[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u)
                            if ((v + u) * 64 + lane < npts)
                                p[u] = pts[at[v + u] + (v + u) * 64 + lane];
#pragma unroll
                        for (int u = 0; u < 2; ++u)
                            if ((v + u) * 64 + lane < npts) stage(p[u], (v + u) * 64 + lane);
                    }
                }
                bad = __ballot(bad) != 0;
                wave_lds_sync();
                evals += (unsigned)npts * (unsigned)acount;
                for (int p0 = 0; p0 < npts; p0 += HALF) {
                    const int m = min(HALF, npts - p0);
                    steps += (unsigned)((m + 15) >> 4);
                    unsigned wd[4] = {0, 0, 0, 0};
                    bool dense = bad;
                    float thr = kth;
                    if constexpr (PER) {
                        // the k-th distance raised by 2^-19 L
                        const float rt = __builtin_sqrtf(kth) * (1.0f + 0x1p-20f) + Lp * 0x1p-19f;
                        dense = dense || __ballot(act && !(qfar + rt < Lh * (1.0f - 0x1p-10f)));
                        thr = rt * rt;
                    }
                    // t of this lane's query
                    const float tq = act ? thr * (1.0f + FILTER_E) - nq + FILTER_TINY : -FILTER_BIG;
                    const float *ap = tilef + 4 * p0 + arow;
                    if (dense)
                        dense_words<PER>(tile + p0, m, 4 >> lgS, h, me, act ? kth : -1.0f, Lp, Lh, wd);
                    else if (lgS == 0) filter_words<1, PER>(ap, m, h, ac, aL, Lh, bq, tq, wd);
                    else if (lgS == 1) filter_words<2, PER>(ap, m, h, ac, aL, Lh, bq, tq, wd);
                    else filter_words<4, PER>(ap, m, h, ac, aL, Lh, bq, tq, wd);
                    // queue the hits word by word, lowest position first; the queue is
                    // drained before a word that would overflow some lane's, and
                    // after the batch's last word
                    const int W = 4 >> lgS;
                    for (int k = 0; k <= W; ++k) {
                        unsigned M = wd[0];
                        wd[0] = wd[1];
                        wd[1] = wd[2];
                        wd[2] = wd[3];
                        wd[3] = 0;
                        const bool full = __ballot(qp + 64 * __popc(M) > q0 + 64 * CQ) != 0;
                        if (full || (k == W && p0 + HALF >= npts)) drain();
                        const int pb = p0 + W * h + k;
                        while (M) {
                            *qp = (uint8_t)(pb + ((__ffs((int)M) - 1) << 2));
                            qp += 64;
                            M &= M - 1u;
                        }
                    }
                    if (p0 + HALF < npts) kth = group_kth();
                }
                wave_lds_sync();
            }
        }
    }
    // merge the partial lists of a query's lanes
    if (lgS >= 1) {
        TopK<K> other;
#pragma unroll
        for (int i = 0; i < K; ++i) other.set(i, swap32_d(best.get(i)));
        merge_topk<K>(best, other);
    }
    if (lgS >= 2) {
        TopK<K> other;
#pragma unroll
        for (int i = 0; i < K; ++i) other.set(i, swap16_d(best.get(i)));
        merge_topk<K>(best, other);
    }
    if (act && h == 0) {
        int32_t *oi = out_idx + row * out_stride + col0;
        float *od = out_d2 + row * out_stride + col0;
        // in words of V entries where the buffers and the row length allow
        // (row_align: bytes every row start is a multiple of): a row is a
        // place of its own in memory, so every store passes over 64 lines,
        // and 32 four-byte ones per query took 7.46 ms of kernel where 8 of
        // 16 bytes take 7.21 (2^24 points, k = 16)
        constexpr int V = K % 4 == 0 ? 4 : (K % 2 == 0 ? 2 : 1);
        if (V > 1 && kw == K && row_align >= 4 * V) {
            typedef int vi __attribute__((ext_vector_type(V)));
            typedef float vf __attribute__((ext_vector_type(V)));
#pragma unroll
            for (int r = 0; r < K; r += V) {
                vi wi;
                vf wf;
#pragma unroll
                for (int u = 0; u < V; ++u) {
                    const uint64_t e = bits_of(best.get(r + u));
                    const bool none = e == PAD_KEY;
                    wi[u] = none ? -1 : (int)(uint32_t)e - base;
                    wf[u] = none ? INFINITY : __uint_as_float((uint32_t)(e >> 32));
                }
                *reinterpret_cast<vi *>(oi + r) = wi;
                *reinterpret_cast<vf *>(od + r) = wf;
            }
        } else
#pragma unroll
        for (int r = 0; r < K; ++r) {
            if (r < kw) {
                const uint64_t e = bits_of(best.get(r));
                const bool none = e == PAD_KEY;
                oi[r] = none ? -1 : (int)(uint32_t)e - base;
                od[r] = none ? INFINITY : __uint_as_float((uint32_t)(e >> 32));
            }
        }
    }
    if (lane == 0) {
        unsigned long long *st = stats + (A & (STAT_SLOTS - 1));
        atomicAdd(st + 0 * STAT_SLOTS, evals);
        // (a leaf that several waves share counts its pairs in the first)
        if (part == 0) atomicAdd(st + 1 * STAT_SLOTS, (unsigned long long)visited);
        atomicAdd(st + 2 * STAT_SLOTS, (unsigned long long)rounds);
        atomicAdd(st + 3 * STAT_SLOTS, (unsigned long long)steps);
        if (len > LCAP && part == 0)
            atomicAdd(st + (len <= presorted ? 4 : 5) * STAT_SLOTS, 1ull);
    }
}

typedef void (*leaf_fn)(const int2 *, const int2 *, const Node *, const float4 *, int, const int *,
                        int32_t *, float *, unsigned long long *, const unsigned long long *, int,
                        int, int, int, const int *, int, int, float, const float *,
                        const int *, const unsigned long long *, int, int, int);

template <int K, bool LO, bool PER>
leaf_fn leaf_ptr() {
    return k_leaf_knn<K, LO, PER>;
}

template <bool PER>
leaf_fn leaf_kernel_m(int k, bool lo) {
    static const leaf_fn table[34] = {
        nullptr,
        leaf_ptr<1, false, PER>(),  leaf_ptr<2, false, PER>(),  leaf_ptr<3, false, PER>(),
        leaf_ptr<4, false, PER>(),  leaf_ptr<5, false, PER>(),  leaf_ptr<6, false, PER>(),
        leaf_ptr<7, false, PER>(),  leaf_ptr<8, false, PER>(),  leaf_ptr<9, false, PER>(),
        leaf_ptr<10, false, PER>(), leaf_ptr<11, false, PER>(), leaf_ptr<12, false, PER>(),
        leaf_ptr<13, false, PER>(), leaf_ptr<14, false, PER>(), leaf_ptr<15, false, PER>(),
        leaf_ptr<16, false, PER>(), leaf_ptr<17, false, PER>(), leaf_ptr<18, false, PER>(),
        leaf_ptr<19, false, PER>(), leaf_ptr<20, false, PER>(), leaf_ptr<21, false, PER>(),
        leaf_ptr<22, false, PER>(), leaf_ptr<23, false, PER>(), leaf_ptr<24, false, PER>(),
        leaf_ptr<25, false, PER>(), leaf_ptr<26, false, PER>(), leaf_ptr<27, false, PER>(),
        leaf_ptr<28, false, PER>(), leaf_ptr<29, false, PER>(), leaf_ptr<30, false, PER>(),
        leaf_ptr<31, false, PER>(), leaf_ptr<32, false, PER>(), leaf_ptr<32, true, PER>()};
    return table[lo ? 33 : k];
}

// The leaf kernel of one pass: K = k for k <= 32 (one pass); for k > 32 the
// first pass has K = 32 and the later ones continue after the last key of the
// pass before (LO).
leaf_fn leaf_kernel(int k, int col, bool per) {
    const int kk = k <= 32 ? k : 32;
    const bool lo = col > 0;
    return per ? leaf_kernel_m<true>(kk, lo) : leaf_kernel_m<false>(kk, lo);
}

}  // namespace

namespace {
__global__ __launch_bounds__(256) void k_zero_words(unsigned long long *__restrict__ p, size_t n) {
    for (size_t i = (size_t)blk_x() * bdim_x() + tid_x(); i < n;
         i += (size_t)nblk_x() * bdim_x())
        p[i] = 0;
}
}  // namespace

jz_status zero_words(unsigned long long *p, size_t n, hipStream_t s) {
    if (n == 0) return JZ_OK;
    k_zero_words<<<(unsigned)std::min<size_t>((n + 255) / 256, 1024), 256, 0, s>>>(p, n);
    JZ_HIP(hipGetLastError());
    return JZ_OK;
}

jz_status run_knn(jz_tree *t, int k, int32_t *idx, float *dist2, hipStream_t s,
                  const AllocCtx *scratch) {
    CallScope scope(t);
    const AllocCtx *ac = scratch ? scratch : &t->ac;
    const int P = t->P;
    // a joint tree of source and query points: rows are the query points
    const bool joint = t->n_src >= 0;
    // periodic cube (period 0: open)
    const float period = t->opts.period;
    const bool per = period > 0.0f;
    for (int p = 0; p <= JZ_MAX_PLANES; ++p) t->st.list_entries[p] = 0;
    t->st.leaf_pairs = t->st.leaf_pairs_visited = 0;
    t->st.evaluations = 0;
    t->st.leaf_ms = t->st.total_ms = 0;
    t->st.reruns = 0;
    t->st.insert_rounds = t->st.tile_steps = 0;
    t->st.lists_sorted_long = t->st.lists_unordered = 0;
    for (int p = 0; p <= JZ_MAX_PLANES; ++p) t->st.lists_presorted[p][0] = t->st.lists_presorted[p][1] = 0;
    if (t->n == 0) return scope.done();
    JZ_TRY(check_top(t->knn_top_last));

    // counters: four leaf statistics (evaluations, sources visited, insert
    // rounds, tile steps)
    // then two counters of long lists (up to SORT_MID entries, longer) per
    // walk level and for the leaf stage, and one counter of work items per
    // walk level
    DBuf d_ctr;
    const size_t c_long = ctr_words(6), c_items = c_long + 2 * (JZ_MAX_PLANES + 1);
    const size_t c_first = c_items + JZ_MAX_PLANES;  // leaves with long lists
    const size_t nctr = c_first + 1;
    JZ_TRY(d_ctr.get(ac, nctr * sizeof(unsigned long long), s));
    unsigned long long *ctr = d_ctr.as<unsigned long long>();
    JZ_TRY(zero_words(ctr, nctr, s));
    int64_t cap[JZ_MAX_PLANES];
    DBuf segs[JZ_MAX_PLANES], lists[JZ_MAX_PLANES];
    for (int p = 0; p < P; ++p) {
        cap[p] = initial_cap(t, CAP_KNN, k, p);
        JZ_TRY(segs[p].get(ac, t->L[p] * sizeof(int2), s));
    }
    // Lists longer than WALK_PRESORT in the walk and LEAF_PRESORT in the leaf
    // stage, up to sort_max, are sorted in HBM before their level.
    const int sort_max = t->opts.sort_max;
    const int walk_cap = WALK_PRESORT;
    const int first_len = t->L[0] > LEAF_MANY ? std::min(sort_max, 1024) : LEAF_FIRST;
    // work items of the walk (at most one per parent plus one per cb
    // children, or per WALK_CB_LONG children of a parent with a long list):
    // WALK_CB children per item at the leaf level, WALK_CB_UP
    // above it, where there are few parents
    auto cb_of = [&](int p) {
        const int64_t n_par = p == P - 1 ? t->S : t->L[p + 1];
        return p == 0 || n_par >= 4096 ? WALK_CB : WALK_CB_UP;
    };
    auto item_bound = [&](int p) {
        const int64_t n_par = p == P - 1 ? t->S : t->L[p + 1];
        return n_par + t->L[p] / std::min(cb_of(p), WALK_CB_LONG) + 1;
    };
    int64_t max_items = 0;
    for (int p = 0; p < P; ++p) max_items = std::max(max_items, item_bound(p));
    DBuf d_items;
    JZ_TRY(d_items.get(ac, (size_t)max_items * sizeof(int2), s));
    DBuf d_ids, d_rleaf, d_first;
    JZ_TRY(d_ids.get(ac, 2 * (size_t)t->L[0] * sizeof(int), s));
    JZ_TRY(d_rleaf.get(ac, (size_t)t->L[0] * sizeof(float), s));
    JZ_TRY(d_first.get(ac, (size_t)t->L[0] * sizeof(int), s));
    auto presort = [&](int2 *list, const int2 *seg, int64_t n, int min_len,
                       unsigned long long *count) {
        // (a list names a node at most once: none is longer than the plane)
        if (sort_max <= min_len || n <= min_len) return;
        int *ids_a = d_ids.as<int>(), *ids_b = ids_a + t->L[0];
        const int mid = std::max(min_len, std::min(sort_max, SORT_MID));
        k_find_long<<<(unsigned)((n + 63) / 64), 64, 0, s>>>(seg, (int)n, min_len, mid, sort_max,
                                                             ids_a, count, ids_b, count + 1);
        if (mid > min_len)
            k_sort_lists<SORT_MID, SORT_MID_WAVES><<<1024, 64 * SORT_MID_WAVES, 0, s>>>(list, seg, ids_a,
                                                                               count);
        if (sort_max > mid)
            k_sort_lists<SORT_MAX, SORT_WAVES><<<512, 64 * SORT_WAVES, 0, s>>>(list, seg, ids_b,
                                                                              count + 1);
    };
    EventSet ev(jz_profiling());
    HostCopy host(!scratch);  // the counters

    // Level p turns the list of plane p+1 (or of the super nodes) into the
    // list of plane p. On overflow, levels from the highest overflowing one
    // down are rerun with larger lists; the levels above are still valid.
    int start = P - 1;
    for (;;) {
        // the lists of the levels to (re)run: released bottom level first,
        // then acquired top level first (a scratch region handed out in
        // stack order takes them back and reuses the space)
        for (int p = 0; p <= start; ++p)
            if (lists[p].bytes < (size_t)cap[p] * sizeof(int2)) lists[p].release();
        for (int p = start; p >= 0; --p) JZ_TRY(lists[p].ensure(ac, cap[p] * sizeof(int2), s));
        if (ev.on) JZ_HIP(hipEventRecord(ev[0], s));
        for (int p = start; p >= 0; --p) {
            const bool top = p == P - 1;
            const int2 *seg_in = top ? t->knn_top_seg.as<int2>() : segs[p + 1].as<int2>();
            // the super-node list belongs to the tree (shared by every call):
            // it is never written, so long lists there are read unordered
            int2 *list_in = top ? t->knn_top_list.as<int2>() : lists[p + 1].as<int2>();
            const int *par_spl = top ? t->super_spl.as<int>() : t->spl[p + 1].as<int>();
            const int64_t n_par = top ? t->S : t->L[p + 1];
            if (!top) presort(list_in, seg_in, n_par, walk_cap, ctr + c_long + 2 * p);
            unsigned long long *n_items = ctr + c_items + p;
            k_walk_items<<<(unsigned)((n_par + 63) / 64), 64, 0, s>>>(
                par_spl, (int)n_par, cb_of(p), seg_in, d_items.as<int2>(), n_items);
            (per ? k_knn_step<true> : k_knn_step<false>)<<<blocks_for(item_bound(p), WPB),
                                                              64 * WPB, 0, s>>>(
                d_items.as<int2>(), n_items, cb_of(p), seg_in, list_in, par_spl,
                t->nodes[p].as<Node>(), k, segs[p].as<int2>(), lists[p].as<int2>(),
                ctr + (size_t)p * LIST_ARENAS, cap[p] / LIST_ARENAS, ctr + CTR_FLAG,
                top ? INT_MAX : walk_cap, top ? 0 : sort_max,
                joint ? t->src_cnt[p].as<int>() : nullptr, period,
                p == 0 ? d_rleaf.as<float>() : nullptr);
        }
        presort(lists[0].as<int2>(), segs[0].as<int2>(), t->L[0], LEAF_PRESORT,
                ctr + c_long + 2 * JZ_MAX_PLANES);
        // waves for every leaf plus the first ones (at most one per first_len
        // + 1 list entries)
        int64_t n_waves = t->L[0];
        if (t->L[0] > first_len) {
            k_long_first<<<(unsigned)((t->L[0] + 63) / 64), 64, 0, s>>>(
                segs[0].as<int2>(), (int)t->L[0], first_len, d_first.as<int>(), ctr + c_first);
            n_waves += std::min<int64_t>(t->L[0], cap[0] / (first_len + 1) + 1);
        }
        JZ_HIP(hipGetLastError());
        if (ev.on) JZ_HIP(hipEventRecord(ev[1], s));
        // k <= 32: one pass; larger k: passes of 32 neighbours, each after
        // the last key of the one before
        const int lg_parts = t->L[0] <= LEAF_FEW ? 2 : 0;
        const uintptr_t places = (uintptr_t)idx | (uintptr_t)dist2 | 4 * (uintptr_t)k;
        const int row_align = places & 4 ? 4 : (places & 8 ? 8 : 16);
        for (int col = 0; col < k; col += 32) {
            const leaf_fn fn = leaf_kernel(k, col, per);
            fn<<<blocks_for(n_waves, WPB) << lg_parts, 64 * WPB, 0, s>>>(
                segs[0].as<int2>(), lists[0].as<int2>(), t->nodes[0].as<Node>(),
                t->pts4.as<float4>(), (int)t->L[0], t->nsets > 1 ? t->leaf_base.as<int>() : nullptr,
                idx, dist2, ctr + CTR_STATS, ctr + CTR_FLAG, sort_max, k, col,
                std::min(32, k - col), joint ? t->src_cnt[0].as<int>() : nullptr,
                joint ? (int)t->n_src : INT_MAX, joint ? (int)t->n_src : 0, period,
                d_rleaf.as<float>(), d_first.as<int>(), ctr + c_first, first_len, row_align, lg_parts);
            JZ_HIP(hipGetLastError());
        }
        if (ev.on) JZ_HIP(hipEventRecord(ev[2], s));
        JZ_TRY(host.read(ctr, nctr * sizeof(unsigned long long), s));
        const unsigned long long *hc = host.as<unsigned long long>();
        int redo = -1;
        double sum[JZ_MAX_PLANES], need[JZ_MAX_PLANES];
        for (int p = P - 1; p >= 0; --p) arena_need(hc, p, sum[p], need[p]);
        for (int p = start; p >= 0; --p) {
            if (need[p] <= (double)(cap[p] / LIST_ARENAS * LIST_ARENAS)) continue;
            if (need[p] > (double)INT32_MAX)
                return jz_fail(JZ_E_CAPACITY, "interaction list at plane %d needs %.0f entries "
                               "(more than 2^31-1)", p, need[p]);
            if (redo < 0) redo = p;
            const double want = need[p] * 1.15 + 1024.0;
            cap[p] = want > (double)INT32_MAX ? (int64_t)INT32_MAX : (int64_t)want;
        }
        if (redo >= 0) {
            if (!t->opts.auto_regrow)
                return jz_fail(JZ_E_CAPACITY,
                               "interaction list overflow at plane %d; list_per_node must be at "
                               "least %.1f", redo, need[redo] / (double)t->L[redo]);
            t->st.reruns++;
            start = redo;
            // clear the counters of the levels to redo, the flag and the leaf
            // statistics
            JZ_TRY(zero_words(ctr, (size_t)(start + 1) * LIST_ARENAS, s));
            JZ_TRY(zero_words(ctr + CTR_FLAG, nctr - CTR_FLAG, s));
            continue;
        }
        for (int p = 0; p < P; ++p) {
            t->st.list_entries[p] = (int64_t)sum[p];
            cap_learn(CAP_KNN, k, p, need[p] / (double)std::max<int64_t>(1, t->L[p]));
        }
        t->st.leaf_pairs = t->st.list_entries[0];
        t->st.evaluations = stat_sum(hc, 0);
        t->st.leaf_pairs_visited = (int64_t)stat_sum(hc, 1);
        t->st.insert_rounds = (int64_t)stat_sum(hc, 2);
        t->st.tile_steps = (int64_t)stat_sum(hc, 3);
        t->st.lists_sorted_long = (int64_t)stat_sum(hc, 4);
        t->st.lists_unordered = (int64_t)stat_sum(hc, 5);
        for (int p = 0; p <= JZ_MAX_PLANES; ++p)
            for (int j = 0; j < 2; ++j)
                t->st.lists_presorted[p][j] = (int64_t)hc[c_long + 2 * p + j];
        if (ev.on) {
            float ms = 0;
            JZ_HIP(hipEventElapsedTime(&ms, ev[1], ev[2]));
            t->st.leaf_ms = ms;
            JZ_HIP(hipEventElapsedTime(&ms, ev[0], ev[2]));
            t->st.total_ms = ms;
        }
        return scope.done();
    }
}
