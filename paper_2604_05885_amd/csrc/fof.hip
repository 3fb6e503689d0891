// Friends-of-friends by the same dual walk (paper: FoF section, Eq. 18-19).
//
// Group state: a point-level union-find `uf` over z-order indices (root =
// smallest z-index of its group, linking higher root to lower root by CAS) plus
// one "whole" flag per node and plane: a whole node's points are known to be
// connected. The paper's ParentToNode advection (Eq. 19) becomes:
//   - a child of a whole parent is whole, and its first point is pointed at
//     the parent's first point (never touched before, so a plain store);
//   - a node whose own diagonal is within the linking length is whole.
// Node pairs (pairs are unordered: the lists hold sources >= receiver):
//   discard if d_low^2 > b^2, or both whole and already one group;
//   link    if d_up^2 <= b^2 (all member pairs linked): union the first
//           points and mark both whole (each is connected through the other);
//   descend otherwise (emit the pair into the next plane's list).
// Leaves: point pairs with dist2 <= b^2 are united; a final pass writes each
// point's group label as the smallest input index of its group.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <vector>

#include "jz_device.h"
#include "jz_internal.h"

namespace {

// A leaf's "whole" flag: its points are one group, and (OWN) their roots say so;
// (WALK) the node walk found it, and the leaf stage joins its points.
constexpr int WHOLE_WALK = 1, WHOLE_OWN = 2;

// The start of a call, one wave per leaf: its own links as a mask per lane, the
// components closed in registers, and every point's root the first of its
// component; a leaf that is one component is whole. The smallest input index of
// every group starts as its root's own (a root is a member; a point that stays
// a root of itself needs no update at all); the counters zero.
// Plain stores into a forest that nothing else has touched, from points that
// have to be read here anyway. With the components found where the pairs of
// leaves are worked on, no leaf of a dense region was joined when its
// neighbours' waves began: a source of 64 connected points was 64 groups, joined
// to the receiving leaf one after another, 2 us each, and the slowest waves set
// the leaf kernel's length (clustered, alpha = 0.2: 0.14 ms at 5 10^4 points,
// 0.23 at 10^6, 1.65 at 2^24; now 0.09, 0.15 and 1.28). At 2^24 points this
// kernel takes 0.33 ms, 64 distances a point on the vector unit, most of which
// the leaf kernel spent before; the whole FoF call went from 0.193 to 0.143 ms,
// from 0.57 to 0.50 and from 2.58 to 2.47. Its 0.4 GB of traffic would take
// 0.09. A search from member to member, which ends early in a
// dense leaf, took 0.59: a chain of scalar steps per point. Leaving out leaves
// whose box is within b gains nothing.
template <bool PER>
__global__ __launch_bounds__(64 * WPB) void k_fof_init(
    const Node *__restrict__ leaves, const float4 *__restrict__ pts, int n_leaves, float b2,
    const float *__restrict__ b2n, int *__restrict__ whole, int *__restrict__ uf,
    int *__restrict__ minidx, unsigned long long *__restrict__ ctr, int nctr, float L) {
    const float Lh = 0.5f * L;
    __shared__ float4 s_tile[WPB][64];
    grid_stride(blk_x(), 64 * WPB, nblk_x(), tid_x(), nctr, [&](size_t i) { ctr[i] = 0; });
    const int w = WPB == 1 ? 0 : uni((int)(tid_x() >> 6)), lane = tid_x() & 63;
    const int A = xcd_block(blk_x(), nblk_x()) * WPB + w;
    if (A >= n_leaves) return;
    const Node a = leaves[A];
    const int astart = uni(a.start), acount = uni(a.count);
    const bool act = lane < acount;
    const int my = astart + (act ? lane : 0);
    const float4 me = pts[my];
    const float bb = b2n ? b2n[A] : b2;
    float4 *tile = s_tile[w];
    tile[lane] = me;
    wave_lds_sync();
    // the leaf's own links, exactly (both directions, as masks of lanes; a
    // difference's sign is exact, and shifted in with one instruction)
    unsigned far[2] = {0, 0};
#pragma unroll
    for (int hf = 1; hf >= 0; --hf) {
#pragma unroll 4
        for (int f = min(acount, 32 * hf + 32) - 1; f >= 32 * hf; --f) {
            const float4 p = tile[f];
            const float dd = dist2_m<PER>(me.x, me.y, me.z, p.x, p.y, p.z, L, Lh);
            far[hf] = __builtin_amdgcn_alignbit(far[hf], __float_as_uint(bb - dd), 31);
        }
    }
    // (b^2 beyond the float range: every distance, infinite ones too, is within it)
    uint64_t adj = bb < INFINITY ? ~((uint64_t)far[1] << 32 | far[0]) : ~0ull;
    adj &= ~0ull >> (64 - acount);
    if (!act) adj = 0;
    // components: from the lowest point not yet in one, the links of all its
    // members are added until nothing changes
    int lead = lane;  // the first point of this lane's component
    bool one = acount == 1;
    uint64_t todo = __ballot((adj & ~(1ull << lane)) != 0);
    while (todo) {
        const int s = __ffsll((unsigned long long)todo) - 1;
        uint64_t reach = 1ull << s, prev = 0;
        while (reach != prev) {
            prev = reach;
            const uint64_t add = (reach >> lane) & 1ull ? adj : 0ull;
            reach |= (uint64_t)uni(wave_or((unsigned)(add >> 32))) << 32 |
                     uni(wave_or((unsigned)add));
        }
        if ((reach >> lane) & 1ull) lead = s;
        todo &= ~reach;
        one = one || reach == (acount == 64 ? ~0ull : (1ull << acount) - 1ull);
    }
    if (act) {
        uf[my] = astart + lead;
        minidx[my] = __float_as_int(me.w);
    }
    if (lane == 0) whole[A] = one ? WHOLE_OWN : 0;
}

__global__ void k_node_b2(const int *__restrict__ node_set, int64_t L,
                          const float *__restrict__ b2_set, float *__restrict__ b2n) {
    const int64_t i = (int64_t)blk_x() * bdim_x() + tid_x();
    if (i < L) b2n[i] = b2_set[node_set[i]];
}

// ParentToNode: one wave per parent, lanes over its children.
template <bool PER>
__global__ __launch_bounds__(64 * WPB) void k_fof_p2n(const int *__restrict__ par_spl,
                                                 const Node *__restrict__ nodes, int n_par,
                                                 const int *__restrict__ whole_par,
                                                 int *__restrict__ whole, int *__restrict__ uf,
                                                 float b2, const float *__restrict__ b2n, float L,
                                                 int leaf_level) {
    const int w = WPB == 1 ? 0 : uni((int)(tid_x() >> 6)), lane = tid_x() & 63;
    const int P = xcd_block(blk_x(), nblk_x()) * WPB + w;
    if (P >= n_par) return;
    const int c0 = par_spl[P], c1 = par_spl[P + 1];
    const int wp = whole_par ? whole_par[P] : 0;
    const int first = nodes[c0].start;
    for (int c = c0 + lane; c < c1; c += 64) {
        const Node me = nodes[c];
        const float bb = b2n ? b2n[c] : b2;
        const int wc = (wp || box_up2_m<PER>(me, me, L) <= bb) ? WHOLE_WALK : 0;
        if (!leaf_level) whole[c] = wc;
        else if (wc && whole[c] == 0) whole[c] = wc;
        if (wp && c != c0) uf[me.start] = first;
    }
}

// Node walk step: one wave per work item, a receiving parent and up to CB of
// its children (item I: parent I / nsub, its children from CB (I % nsub) on,
// in strides of CB nsub). The receivers' boxes are uniform, in scalar registers
// as far as those go (some 60 words of CB = 4 and 165 of CB = 8 are read back
// from lanes of vector registers, one instruction each); the source children go
// through the lanes, 64 node records at a time, their indices expanded into
// LDS.
//   phase 0  links (d_up^2 <= b^2: union of the first points, both nodes become
//            whole), and counts the pairs that geometry alone sends down
//            (within reach, not wholly within b)
//   phase 1  writes those still to be descended into (not both whole and
//            already one group): the group state only merges, so this is a
//            subset of what was counted, whatever either phase read of it
// A pair is taken at its lower node. With a wave per parent that went through
// its list source by source, the top level (a few dozen parents, 32 children
// each) was one chain of loads per source: 0.34 ms at 10^6 uniform points.
// CB = 4 or 8 receivers per wave: 4 (and two items per parent) where there are
// few parents, 8 from FOF_MANY parents on, where the items fill the device
// anyway and each repeats its parent's stream (leaf level at 2^24 clustered
// points, 52780 parents: 0.24 ms with 8, 0.35 with 4; 7477 parents: 0.081 and
// 0.073 ms; a top level of 94: 0.092 and 0.061 ms).
constexpr int FOF_MANY = 16384;
constexpr int FOF_CAP = 1024;
template <bool PER, int CB>
__global__ __launch_bounds__(64 * WPB) void k_fof_step(
    const int2 *__restrict__ seg_in, const int2 *__restrict__ list_in,
    const int *__restrict__ par_spl, const Node *__restrict__ nodes, int n_par, int nsub, float b2,
    const float *__restrict__ b2n, int *__restrict__ whole, int *__restrict__ uf,
    int2 *__restrict__ seg_out, int2 *__restrict__ list_out,
    unsigned long long *__restrict__ ctr, long long cap, unsigned long long *overflow, float L) {
    __shared__ int s_fi[WPB][FOF_CAP];
    const int w = WPB == 1 ? 0 : uni((int)(tid_x() >> 6)), lane = tid_x() & 63;
    const int I = xcd_block(blk_x(), nblk_x()) * WPB + w;
    const int P = I / nsub;
    if (P >= n_par) return;
    const int2 sg = seg_in[P];
    const int2 *gl = list_in + uni(sg.x);
    const int len = uni(sg.y);
    const int p0 = uni(par_spl[P]), p1 = uni(par_spl[P + 1]);
    int *FI = s_fi[w];
    for (int c0 = p0 + CB * (I % nsub); c0 < p1; c0 += CB * nsub) {
        const int nc = min(CB, p1 - c0);
        Node me[CB];
        float bb[CB];
        int cnt[CB];  // (uniform) pairs counted, then entries written
        int off[CB];  // (uniform) first entry
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            const int c = c0 + min(j, nc - 1);
            me[j] = nodes[c];
            bb[j] = b2n ? b2n[c] : b2;
            cnt[j] = off[j] = 0;
        }
        long long base = 0;
        bool single = true;  // the whole stream fits FI
        int t = 0, skip = 0, nN = 0;
        for (int phase = 0; phase < 2; ++phase) {
            if (phase == 1) {
                int total = 0;
#pragma unroll
                for (int j = 0; j < CB; ++j) {
                    off[j] = total;
                    total += cnt[j];
                    cnt[j] = 0;
                }
                // segment in arena I % LIST_ARENAS (cap entries each)
                const int ar = I & (LIST_ARENAS - 1);
                unsigned long long lb = 0;
                if (lane == 0) lb = atomicAdd(ctr + ar, (unsigned long long)total);
                lb = uni(lb);
                base = (long long)((unsigned long long)ar * (unsigned long long)cap + lb);
                const bool ok = (long long)lb + total <= cap;
                // lists below are incomplete: the leaf stage of this attempt exits
                if (!ok && lane == 0) *overflow = 1;
                if (!ok || total == 0) {
                    if (lane < nc) seg_out[c0 + lane] = make_int2(0, 0);
                    break;
                }
            }
            if (phase == 0 || !single) t = skip = nN = 0;
            for (;;) {
                if (phase == 0 || !single)
                    list_children<FOF_CAP>(gl, len, par_spl, FI, nN, t, skip,
                                           [](const int2 &, bool valid, bool &) { return valid; });
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
                    }
                };
                load(0);
                for (int b = 0; b < nN; b += 64) {
                    x = b + lane < nN ? nx : -1;
                    ra = na;
                    rb = nb;
                    load(b + 64);
                    Node o;
                    o.lo[0] = ra.x; o.lo[1] = ra.y; o.lo[2] = ra.z;
                    o.hi[0] = rb.x; o.hi[1] = rb.y; o.hi[2] = rb.z;
                    o.start = __float_as_int(ra.w);
                    o.count = 0;
#pragma unroll
                    for (int j = 0; j < CB; ++j) {
                        const int c = c0 + j;
                        const float lo = box_low2_m<PER>(me[j], o, L);
                        const bool in = j < nc && x >= c && lo <= bb[j];
                        if (!__ballot(in)) continue;
                        const bool down = in && !(box_up2_m<PER>(me[j], o, L) <= bb[j]);
                        // (flags only ever go from 0 to 1 and groups only
                        // merge: values read through the caches may be older,
                        // which only costs a redundant union)
                        const bool wc = ld_cached(whole + c) != 0;
                        if (phase == 0) {
                            cnt[j] += (int)__popcll(__ballot(down));
                            if (in && !down &&
                                !(wc && ld_cached(whole + x) &&
                                  uf_find_c(uf, me[j].start) == uf_find_c(uf, o.start))) {
                                uf_union_c(uf, me[j].start, o.start);
                                if (!wc) st_rel(whole + c, WHOLE_WALK);
                                if (!ld_cached(whole + x)) st_rel(whole + x, WHOLE_WALK);
                            }
                        } else {
                            bool emit = down;
                            if (emit && wc && ld_cached(whole + x))
                                emit = uf_find_c(uf, me[j].start) != uf_find_c(uf, o.start);
                            const uint64_t m = __ballot(emit);
                            if (emit)
                                list_out[base + off[j] + cnt[j] + (int)__popcll(m & lanemask_lt())] =
                                    make_int2(x, __float_as_int(lo));
                            cnt[j] += (int)__popcll(m);
                        }
                    }
                }
                if (phase > 0 && single) break;
                if (t >= len) break;
                wave_lds_sync();
                nN = 0;
                single = false;
            }
            if (phase == 1) {
#pragma unroll
                for (int j = 0; j < CB; ++j)
                    if (j < nc && lane == 0)
                        seg_out[c0 + j] = make_int2((int)(base + off[j]), cnt[j]);
            }
        }
        wave_lds_sync();
    }
}

// The matrix filter over the c <= 64 points of one staged source: the lane's
// own query's pairs as a mask over the source's points. Row m of a block of 16
// reads point Q (m / 4) + 4 b + m % 4 (Q: a quarter of the points, rounded up
// to 4), so that a lane row's results are one run of Q points and the four
// rows' masks join by shifts. NG: groups of 16 queries.
template <int NG, bool PER>
__device__ __forceinline__ uint64_t pair_mask(const float *tilef, int c, float ac, float aL,
                                              float Lh, const float (&bq)[4],
                                              const float (&tg)[4]) {
    const int lane = lane_id();
    const int nblk = uni((c + 15) >> 4), Q = 4 * nblk;
    const float *ap = tilef + 4 * (Q * ((lane >> 2) & 3) + (lane & 3)) + (lane >> 4);
    unsigned wd[4] = {0, 0, 0, 0};
    for (int b = 0; b < nblk; ++b) {
        const float av = wrap_diff<PER>(ap[16 * b] - ac, aL, aL != 0.0f ? Lh : INFINITY);
        v4f d[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const v4f cg = {tg[g], tg[g], tg[g], tg[g]};
            d[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bq[g], cg, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int g = 0; g < NG; ++g)
                wd[g] = __builtin_amdgcn_alignbit(wd[g], __float_as_uint(d[g][i]), 31);
    }
    // rows and groups transposed: word r holds row r's bits of this lane's query
    const auto x = __builtin_amdgcn_permlane16_swap(wd[0], wd[1], false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(wd[2], wd[3], false, false);
    const auto u = __builtin_amdgcn_permlane32_swap(x[0], y[0], false, false);
    const auto v = __builtin_amdgcn_permlane32_swap(x[1], y[1], false, false);
    const uint64_t m = (((((uint64_t)u[0] << Q | v[0]) << Q) | u[1]) << Q) | v[1];
    return __builtin_bitreverse64(m << (64 - 4 * Q)) & (~0ull >> (64 - c));
}

// The links of a leaf's points to one source's (lm: a mask per lane, which may
// hold pairs just beyond b), united where they join two groups; see k_leaf_fof.
template <bool PER>
__device__ __forceinline__ void link_source(uint64_t lm, bool wA, bool wB, int b0, int my,
                                            const float4 &me, const float4 *tile, int *rootT,
                                            int *uf, float bb, float L, float Lh, int &ra,
                                            int &last) {
    const int lane = lane_id();
    uint64_t linking = __ballot(lm != 0);
    if (!linking) return;
    auto linked = [&](int f) __attribute__((always_inline)) {
        const float4 p = tile[f];
        return dist2_m<PER>(me.x, me.y, me.z, p.x, p.y, p.z, L, Lh) <= bb;
    };
    if (wA && wB) {
        // both leaves are whole: a single link joins them
        const int l0 = __ffsll((unsigned long long)linking) - 1;
        if (uf_find_c(uf, __builtin_amdgcn_readlane(my, l0)) == uf_find_c(uf, b0)) return;
        while (linking) {
            const int f = lm ? __ffsll((unsigned long long)lm) - 1 : 0;
            const uint64_t ok = __ballot(lm != 0 && linked(f));
            if (ok) {
                if (lane == __ffsll((unsigned long long)ok) - 1) uf_union_c(uf, my, b0 + f);
                return;
            }
            lm &= lm - 1ull;
            linking = __ballot(lm != 0);
        }
        return;
    }
    if (wA) {
        // one group on this side: the source's groups are joined to it side by
        // side, every lane taking another of its links (from its own number on)
        while (linking) {
            const uint64_t want = (uint64_t)uni(wave_or((unsigned)(lm >> 32))) << 32 |
                                  uni(wave_or((unsigned)lm));
            int rt = -1;
            if ((want >> lane) & 1ull) rt = uf_find_c(uf, b0 + lane);
            const int r0 = uf_find_c(uf, __builtin_amdgcn_readfirstlane(my));
            rootT[lane] = rt;
            wave_lds_sync();
            lm &= __ballot(rt >= 0 && rt != r0);
            const uint64_t up = lm >> lane << lane;
            const int f = lm ? __ffsll((unsigned long long)(up ? up : lm)) - 1 : 0;
            const bool ok = lm != 0 && linked(f);
            lm &= ~(1ull << f);
            const int rj = ok ? rootT[f] : -1;
            bool first = false;
            for (uint64_t left = __ballot(ok); left;) {
                const int l0 = __ffsll((unsigned long long)left) - 1;
                left &= ~__ballot(rj == __builtin_amdgcn_readlane(rj, l0));
                first = first || lane == l0;
            }
            if (first) uf_union_c(uf, my, b0 + f);
            linking = __ballot(lm != 0);
            wave_lds_sync();
        }
        return;
    }
    // roots of the source's points that some lane links to
    const uint64_t want = (uint64_t)uni(wave_or((unsigned)(lm >> 32))) << 32 |
                          uni(wave_or((unsigned)lm));
    int rt = -1;
    if ((want >> lane) & 1ull) rt = uf_find_c(uf, wB ? b0 : b0 + lane);
    rootT[lane] = rt;
    wave_lds_sync();
    const int r0 = __builtin_amdgcn_readlane(rt, __ffsll((unsigned long long)want) - 1);
    const uint64_t eq = __ballot(rt == r0);
    if (lm && ra < 0) ra = uf_find_c(uf, my);
    uint64_t com = ra == r0 ? 0ull : lm & eq, rest = lm & ~eq;
    while (__ballot((com | rest) != 0)) {
        // each lane's next link to a group it has not joined
        int f = 0, rj = -1;
        if (com) {
            f = __ffsll((unsigned long long)com) - 1;
            com &= com - 1ull;
            rj = r0;
        } else {
            while (rest) {
                f = __ffsll((unsigned long long)rest) - 1;
                rest &= rest - 1ull;
                const int r = rootT[f];
                if (r != ra && r != last) {
                    rj = r;
                    break;
                }
            }
        }
        if (rj >= 0 && !linked(f)) rj = -1;
        // one lane per pair of groups joins them
        bool first = false;
        for (uint64_t left = __ballot(rj >= 0); left;) {
            const int l0 = __ffsll((unsigned long long)left) - 1;
            const int a0 = __builtin_amdgcn_readlane(ra, l0), j0 = __builtin_amdgcn_readlane(rj, l0);
            left &= ~__ballot(rj == j0 && ra == a0);
            first = first || lane == l0;
        }
        if (first) uf_union_c(uf, my, b0 + f);
        if (rj >= 0) {
            ra = uf_find_c(uf, min(ra, rj));
            if (rj == r0) com = 0;
            last = rj;
        }
    }
    wave_lds_sync();
}

// Leaf stage: one wave per receiving leaf A, lanes over its points, sources
// B >= A (a point links to the later points of a pair only).
//
// Every leaf's own links are joined already, but for a leaf that only the walk
// found whole: its points are joined here.
// Then source by source (skipped when A and B are both whole and already one
// group, or when no lane's point both reaches the source's box and was outside
// its group): the next source's points are loaded while the current one is
// worked on; a matrix filter gives each lane the points its own may link to, and
// only a pair that would join two groups is evaluated with the fixed float32
// expression. Two whole leaves need one link. A whole A is joined to the
// source's groups side by side; otherwise the roots of the source's linked
// points are looked up, in parallel, the points under the first one's root count
// as one (in a dense region they all are), and of the lanes that would join the
// same two groups only one does. Groups only ever merge, so equal roots, even
// looked up at different times, mean already connected.
// With box tests and distances on the vector unit, and every lane walking its
// own links (a dense source cost a lane up to 64 steps and as many lanes the
// same compare-and-swap), the kernel took 3.63 ms at 2^24 clustered points and
// alpha = 0.2, then 2.0; 1.03 ms at 10^6, then 0.34; 0.58 at 3 10^5, then 0.23.
// The chunks of a whole leaf's list grow from one entry: every wave of a dense
// region starts at the same time, when few leaves are joined, and with chunks of
// 64 each worked through all of its first 64 sources (2.0 -> 1.65 ms at 2^24,
// 0.34 -> 0.23 at 10^6; 5.6 -> 3.9 10^9 pairs tested at 2^24). With every leaf's
// points joined beforehand and a whole leaf joined to several groups at a time:
// 1.28, 0.15 and, at 3 10^5, 0.08 ms.
template <bool PER>
__global__ __launch_bounds__(64 * WPB, 6) void k_leaf_fof(
    const int2 *__restrict__ seg, const int2 *__restrict__ list, const Node *__restrict__ leaves,
    const float4 *__restrict__ pts, int n_leaves, float b2, const float *__restrict__ b2n,
    const int *__restrict__ whole, int *__restrict__ uf, unsigned long long *__restrict__ stats,
    const unsigned long long *__restrict__ overflow, float L) {
    const float Lh = 0.5f * L;
    __shared__ float4 s_tile[WPB][64];
    __shared__ int s_root[WPB][64];
    const int w = WPB == 1 ? 0 : uni((int)(tid_x() >> 6)), lane = tid_x() & 63;
    const int A = xcd_block(blk_x(), nblk_x()) * WPB + w;
    // a level of this attempt overflowed (it is rerun): nothing to do
    if (A >= n_leaves || *overflow) return;
    const Node a = leaves[A];
    const int astart = uni(a.start), acount = uni(a.count);
    const bool act = lane < acount;
    const int my = astart + (act ? lane : 0);
    const float4 me = pts[my];
    const float bb = b2n ? b2n[A] : b2;
    const int whA = uni(whole[A]);
    const bool wA = whA != 0;
    const int2 sg = seg[A];
    const int2 *gl = list + uni(sg.x);
    const int len = uni(sg.y);
    // (found whole by the walk alone: its points are joined here)
    if (whA == WHOLE_WALK && act && lane > 0) uf_union_c(uf, astart, my);
    // (the pairs within the leaf, looked at when the call began)
    unsigned long long evals = (unsigned)acount * (unsigned)acount;
    if (len == 0) {
        if (lane == 0) atomicAdd(stats + (A & (STAT_SLOTS - 1)), evals);
        return;
    }
    float4 *tile = s_tile[w];
    const float *tilef = reinterpret_cast<const float *>(tile);
    int *rootT = s_root[w];
    int ra = -1;    // this lane's point's root, as last looked up
    int last = -1;  // the last root this lane's group was joined with

    // the filter's query side: lane l holds component l / 16 (x, y, z, 1) of
    // query 16 g + l % 16 in bq[g], and minus that query's t in tg[g]
    const float cx = uni(0.5f * a.lo[0] + 0.5f * a.hi[0]);
    const float cy = uni(0.5f * a.lo[1] + 0.5f * a.hi[1]);
    const float cz = uni(0.5f * a.lo[2] + 0.5f * a.hi[2]);
    const float ac = lane < 16 ? cx : (lane < 32 ? cy : (lane < 48 ? cz : 0.0f));
    const float aL = lane < 48 ? L : 0.0f;  // (periodic) no wrap of w
    bool dense;
    float bq[4], tg[4];
    {
        const float mx = me.x - cx, my_ = me.y - cy, mz = me.z - cz;
        const float qn2 = mx * mx + my_ * my_ + mz * mz;
        float thr = bb;
        bool bad = !(qn2 < FILTER_BIG) || !(bb < FILTER_BIG);
        if constexpr (PER) {
            const float rt = __builtin_sqrtf(bb) * (1.0f + 0x1p-20f) + L * 0x1p-19f;
            const float qfar = fmaxf(fmaxf(fabsf(mx), fabsf(my_)), fabsf(mz));
            bad = bad || !(qfar + rt < Lh * (1.0f - 0x1p-10f));
            thr = rt * rt;
        }
        dense = __ballot(act && bad) != 0;
        const float t = thr * (1.0f + FILTER_E) - qn2 * (1.0f - FILTER_E) + FILTER_TINY;
        wave_lds_sync();
        tile[lane] = make_float4(-2.0f * mx, -2.0f * my_, -2.0f * mz, 1.0f);
        rootT[lane] = __float_as_int(act ? -t : FILTER_BIG);
        wave_lds_sync();
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int qq = 16 * g + (lane & 15);
            bq[g] = tilef[4 * qq + (lane >> 4)];
            tg[g] = __int_as_float(rootT[qq]);
        }
        wave_lds_sync();
    }

    for (int t0 = 0, lim; t0 < len; t0 = lim) {
        // up to 64 sources, one per lane; a whole leaf takes 1, 2, 4, ... at a
        // time, one of more than 64 sources 16, 32, 64, ..., since the first
        // ones join it to most of the others
        lim = min(t0 + (wA || len > 64 ? min(t0 + (wA ? 1 : 16), 64) : 64), len);
        int e_st = 0, e_ct = 0, e_wh = 0, e_rt = -2;
        float4 e_lo = make_float4(0, 0, 0, 0), e_hi = e_lo;
        bool keep = false;
        if (t0 + lane < lim) {
            const int B = gl[t0 + lane].x;
            const float4 *rec = reinterpret_cast<const float4 *>(leaves + B);
            e_lo = rec[0];
            e_hi = rec[1];
            e_st = __float_as_int(e_lo.w);
            e_ct = __float_as_int(e_hi.w);
            e_wh = whole[B];
            if (e_wh) e_rt = uf_find_c(uf, e_st);
            keep = B != A && !(wA && e_wh && e_rt == uf_find_c(uf, astart));
        }
        uint64_t pend = __ballot(keep);
        const uint64_t wholes = __ballot(e_wh != 0);
        int cur = -1;
        for (;;) {
            // the next source some lane's point reaches, its points loading
            int nxt = -1;
            float4 pn = make_float4(0, 0, 0, 0);
            while (pend) {
                const int qq = __ffsll((unsigned long long)pend) - 1;
                pend &= pend - 1ull;
                auto rl = [&](float v) __attribute__((always_inline)) {
                    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), qq));
                };
                bool need = act && point_low2_m<PER>(me.x, me.y, me.z, rl(e_lo.x), rl(e_lo.y),
                                                           rl(e_lo.z), rl(e_hi.x), rl(e_hi.y),
                                                           rl(e_hi.z), L) <= bb;
                // (not by a point that is in the group the whole source was in)
                if (__ballot(need)) {
                    const int rB = __builtin_amdgcn_readlane(e_rt, qq);
                    need = need && ra != rB && last != rB;
                }
                if (__ballot(need)) {
                    nxt = qq;
                    const int st = __builtin_amdgcn_readlane(e_st, qq);
                    if (lane < __builtin_amdgcn_readlane(e_ct, qq)) pn = pts[st + lane];
                    break;
                }
            }
            if (cur >= 0) {
                const int b0 = __builtin_amdgcn_readlane(e_st, cur);
                const int c = __builtin_amdgcn_readlane(e_ct, cur);
                const bool wB = (wholes >> cur) & 1ull;
                uint64_t lm = 0;  // the source's points this lane's may link to
                evals += (unsigned)acount * (unsigned)c;
                if (dense) {
                    for (int f = 0; f < c; ++f) {
                        const float4 p = tile[f];
                        const float dd = dist2_m<PER>(me.x, me.y, me.z, p.x, p.y, p.z, L, Lh);
                        lm |= dd <= bb ? 1ull << f : 0ull;
                    }
                    if (!act) lm = 0;
                } else if (acount > 48) lm = pair_mask<4, PER>(tilef, c, ac, aL, Lh, bq, tg);
                else if (acount > 32) lm = pair_mask<3, PER>(tilef, c, ac, aL, Lh, bq, tg);
                else if (acount > 16) lm = pair_mask<2, PER>(tilef, c, ac, aL, Lh, bq, tg);
                else lm = pair_mask<1, PER>(tilef, c, ac, aL, Lh, bq, tg);
                link_source<PER>(lm, wA, wB, b0, my, me, tile, rootT, uf, bb, L, Lh, ra, last);
            }
            if (nxt < 0) break;
            wave_lds_sync();
            {
                // the point and its w (in .w; the index is not needed)
                const float dx = wrap_diff<PER>(pn.x - cx, L, Lh);
                const float dy = wrap_diff<PER>(pn.y - cy, L, Lh);
                const float dz = wrap_diff<PER>(pn.z - cz, L, Lh);
                const float pw = (dx * dx + dy * dy + dz * dz) * (1.0f - FILTER_E);
                tile[lane] = make_float4(pn.x, pn.y, pn.z, pw);
                const bool far = lane < __builtin_amdgcn_readlane(e_ct, nxt) && !(pw < FILTER_BIG);
                if (__ballot(far)) dense = true;
            }
            wave_lds_sync();
            cur = nxt;
        }
    }
    if (lane == 0) atomicAdd(stats + (A & (STAT_SLOTS - 1)), evals);
}

// Root of every point (a read-only find: no other thread writes uf[i] now)
// and the smallest input index per root. Points of one group are mostly
// contiguous in z-order: the wave takes the minimum over each run of lanes
// with the same root (a segmented scan, 6 steps whatever the number of runs)
// and the last lane of a run issues one atomic for it, unless the root's
// current minimum is already no larger (values only decrease, so one read
// through the caches, even an older one, never skips a needed update).
__global__ __launch_bounds__(256) void k_flatten_min(int *__restrict__ uf,
                                                     const float4 *__restrict__ pts, int64_t n,
                                                     int *__restrict__ minidx) {
    const int64_t i = (int64_t)blk_x() * bdim_x() + tid_x();
    const bool valid = i < n;
    const int lane = lane_id();
    int root = -1 - lane, v = INT_MAX;  // invalid lanes: a root of their own
    if (valid) {
        // (a parent read through the caches may be an older one: still an
        // ancestor, so the walk still ends at the root)
        int x = (int)i;
        int p = ld_cached(uf + x);
        while (p != x) {
            x = p;
            p = ld_cached(uf + x);
        }
        root = x;
        uf[i] = x;
        v = __float_as_int(pts[i].w);
    }
    // segmented inclusive min-scan over runs of equal roots
    const int prev_root = __shfl_up(root, 1, 64);
    bool head = lane == 0 || prev_root != root;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int vu = __shfl_up(v, o, 64);
        const bool hu = __shfl_up((int)head, o, 64) != 0;
        if (lane >= o && !head) v = min(v, vu);
        if (lane >= o) head = head || hu;
    }
    const int next_root = __shfl_down(root, 1, 64);
    const bool tail = lane == 63 || next_root != root;
    if (valid && tail && v < ld_cached(minidx + root)) atomicMin(minidx + root, v);
}

__global__ void k_labels(const int *__restrict__ uf, const float4 *__restrict__ pts, int64_t n,
                         const int *__restrict__ minidx, const int64_t *__restrict__ set_off,
                         int nsets, int32_t *__restrict__ label) {
    const int64_t i = (int64_t)blk_x() * bdim_x() + tid_x();
    if (i >= n) return;
    const int o = __float_as_int(pts[i].w);
    int base = 0;
    if (nsets > 1) {
        int lo_s = 0, hi_s = nsets - 1;
        while (lo_s < hi_s) {
            const int m = (lo_s + hi_s + 1) >> 1;
            if (set_off[m] <= o) lo_s = m; else hi_s = m - 1;
        }
        base = (int)set_off[lo_s];
    }
    label[o] = minidx[uf[i]] - base;
}

}  // namespace

jz_status run_fof(jz_tree *t, const float *b2_set_host, int32_t *label, hipStream_t s,
                  jz_stats *st_out) {
    CallScope scope(t);
    jz_stats &st = st_out ? *st_out : t->st;
    const AllocCtx *ac = &t->ac;
    const int P = t->P;
    const int64_t n = t->n;
    for (int p = 0; p <= JZ_MAX_PLANES; ++p) st.list_entries[p] = 0;
    st.leaf_pairs = st.leaf_pairs_visited = 0;
    st.evaluations = 0;
    st.leaf_ms = st.total_ms = 0;
    st.reruns = 0;
    st.insert_rounds = st.tile_steps = 0;
    st.lists_sorted_long = st.lists_unordered = 0;
    for (int p = 0; p <= JZ_MAX_PLANES; ++p) st.lists_presorted[p][0] = st.lists_presorted[p][1] = 0;
    if (n == 0) return scope.done();
    JZ_TRY(check_top(t->fof_top_last));

    const bool sets = t->nsets > 1;
    const float b2 = b2_set_host[0];
    // periodic cube of side L (L = 0: open)
    const float L = t->opts.period;
    const bool per = L > 0.0f;
    DBuf d_ctr, d_uf, d_min, d_b2set;
    // counters: one leaf statistic (evaluations)
    const size_t nctr = ctr_words(1);
    JZ_TRY(d_ctr.get(ac, nctr * sizeof(unsigned long long), s));
    JZ_TRY(d_uf.get(ac, n * sizeof(int), s));
    JZ_TRY(d_min.get(ac, n * sizeof(int), s));
    unsigned long long *ctr = d_ctr.as<unsigned long long>();
    DBuf whole[JZ_MAX_PLANES], b2n[JZ_MAX_PLANES], segs[JZ_MAX_PLANES], lists[JZ_MAX_PLANES];
    int64_t cap[JZ_MAX_PLANES];
    for (int p = 0; p < P; ++p) {
        JZ_TRY(whole[p].get(ac, t->L[p] * sizeof(int), s));
        JZ_TRY(segs[p].get(ac, t->L[p] * sizeof(int2), s));
        cap[p] = initial_cap(t, CAP_FOF, 0, p);
    }
    if (sets) {
        JZ_TRY(d_b2set.get(ac, t->nsets * sizeof(float), s));
        JZ_HIP(hipMemcpyAsync(d_b2set.p, b2_set_host, t->nsets * sizeof(float),
                              hipMemcpyHostToDevice, s));
        for (int p = 0; p < P; ++p) {
            JZ_TRY(b2n[p].get(ac, t->L[p] * sizeof(float), s));
            k_node_b2<<<blocks_for(t->L[p], 256), 256, 0, s>>>(t->node_set[p].as<int>(), t->L[p],
                                                               d_b2set.as<float>(),
                                                               b2n[p].as<float>());
        }
    }
    EventSet ev(jz_profiling());
    HostCopy host;  // the counters

    // Groups only ever merge, so an overflowing run is simply rerun from the
    // start with larger lists.
    for (;;) {
        for (int p = 0; p < P; ++p) JZ_TRY(lists[p].ensure(ac, cap[p] * sizeof(int2), s));
        if (ev.on) JZ_HIP(hipEventRecord(ev[0], s));
        (per ? k_fof_init<true> : k_fof_init<false>)<<<blocks_for(t->L[0], WPB), 64 * WPB, 0, s>>>(
            t->nodes[0].as<Node>(), t->pts4.as<float4>(), (int)t->L[0], b2,
            sets ? b2n[0].as<float>() : nullptr, whole[0].as<int>(), d_uf.as<int>(),
            d_min.as<int>(), ctr, (int)nctr, L);
        if (ev.on) JZ_HIP(hipEventRecord(ev[4], s));
        for (int p = P - 1; p >= 0; --p) {
            const bool top = p == P - 1;
            const int2 *seg_in = top ? t->fof_top_seg.as<int2>() : segs[p + 1].as<int2>();
            const int2 *list_in = top ? t->fof_top_list.as<int2>() : lists[p + 1].as<int2>();
            const int *par_spl = top ? t->super_spl.as<int>() : t->spl[p + 1].as<int>();
            const int *whole_par = top ? nullptr : whole[p + 1].as<int>();
            const int64_t n_par = top ? t->S : t->L[p + 1];
            const float *bn = sets ? b2n[p].as<float>() : nullptr;
            (per ? k_fof_p2n<true> : k_fof_p2n<false>)<<<blocks_for(n_par, WPB), 64 * WPB, 0, s>>>(
                par_spl, t->nodes[p].as<Node>(), (int)n_par, whole_par, whole[p].as<int>(),
                d_uf.as<int>(), b2, bn, L, p == 0);
            // a top parent has up to ngr children, others a few: enough items
            // for one pass over most parents' children
            const bool many = n_par >= FOF_MANY;
            const int nsub = many ? 1 : (top ? (t->opts.ngr + 3) / 4 : 2);
            const auto step = many ? (per ? k_fof_step<true, 8> : k_fof_step<false, 8>)
                                   : (per ? k_fof_step<true, 4> : k_fof_step<false, 4>);
            step<<<blocks_for(n_par * nsub, WPB), 64 * WPB, 0, s>>>(
                seg_in, list_in, par_spl, t->nodes[p].as<Node>(), (int)n_par, nsub, b2, bn,
                whole[p].as<int>(), d_uf.as<int>(), segs[p].as<int2>(), lists[p].as<int2>(),
                ctr + (size_t)p * LIST_ARENAS, cap[p] / LIST_ARENAS, ctr + CTR_FLAG, L);
        }
        JZ_HIP(hipGetLastError());
        if (ev.on) JZ_HIP(hipEventRecord(ev[1], s));
        (per ? k_leaf_fof<true> : k_leaf_fof<false>)<<<blocks_for(t->L[0], WPB), 64 * WPB, 0, s>>>(
            segs[0].as<int2>(), lists[0].as<int2>(), t->nodes[0].as<Node>(), t->pts4.as<float4>(),
            (int)t->L[0], b2, sets ? b2n[0].as<float>() : nullptr, whole[0].as<int>(),
            d_uf.as<int>(), ctr + CTR_STATS, ctr + CTR_FLAG, L);
        if (ev.on) JZ_HIP(hipEventRecord(ev[2], s));
        k_flatten_min<<<blocks_for(n, 256), 256, 0, s>>>(d_uf.as<int>(), t->pts4.as<float4>(), n,
                                                          d_min.as<int>());
        k_labels<<<blocks_for(n, 256), 256, 0, s>>>(d_uf.as<int>(), t->pts4.as<float4>(), n,
                                                     d_min.as<int>(), t->d_set_off.as<int64_t>(),
                                                     t->nsets, label);
        JZ_HIP(hipGetLastError());
        if (ev.on) JZ_HIP(hipEventRecord(ev[3], s));
        JZ_TRY(host.read(ctr, nctr * sizeof(unsigned long long), s));
        const unsigned long long *hc = host.as<unsigned long long>();
        bool overflow = false;
        double sum[JZ_MAX_PLANES], need[JZ_MAX_PLANES];
        for (int p = 0; p < P; ++p) {
            arena_need(hc, p, sum[p], need[p]);
            if (need[p] <= (double)(cap[p] / LIST_ARENAS * LIST_ARENAS)) continue;
            overflow = true;
            if (need[p] > (double)INT32_MAX)
                return jz_fail(JZ_E_CAPACITY, "FoF list at plane %d needs %.0f entries "
                               "(more than 2^31-1)", p, need[p]);
            const double want = need[p] * 1.15 + 1024.0;
            cap[p] = want > (double)INT32_MAX ? (int64_t)INT32_MAX : (int64_t)want;
        }
        if (overflow) {
            if (!t->opts.auto_regrow)
                return jz_fail(JZ_E_CAPACITY, "FoF interaction list overflow; raise list_per_node");
            st.reruns++;
            continue;
        }
        for (int p = 0; p < P; ++p) {
            st.list_entries[p] = (int64_t)sum[p];
            cap_learn(CAP_FOF, 0, p, need[p] / (double)std::max<int64_t>(1, t->L[p]));
        }
        st.leaf_pairs = st.list_entries[0];
        st.evaluations = stat_sum(hc, 0);
        if (ev.on) {
            float ms = 0;
            JZ_HIP(hipEventElapsedTime(&ms, ev[1], ev[2]));
            st.leaf_ms = ms;
            JZ_HIP(hipEventElapsedTime(&ms, ev[0], ev[4]));
            st.leaf_ms += ms;
            JZ_HIP(hipEventElapsedTime(&ms, ev[0], ev[3]));
            st.total_ms = ms;
        }
        return scope.done();
    }
}
