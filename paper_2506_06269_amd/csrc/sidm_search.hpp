// sidm_search.hpp -- the candidates of a bucket's search: which particles of the
// halo can lie within reach of some lane of the wave.
//
// One wave per block.  What its lanes can reach is bounded by groups of lanes
// close to each other on the Morton curve: the box of a group's searching lanes
// and their largest reach.  Nodes of the tree, 64 at a time, and
// then the particles of the buckets that pass, 64 at a time, are tested against
// the groups, one per lane; the particles that pass are compacted into LDS.
// Only those are read by every lane.
//
// Every test holds for all lanes at once, so its cost is that of one lane; a
// search that took one node, sub-range and chunk of 16 particles after the
// other, with every lane testing its own sphere, waited for each load in turn
// and evaluated 1750 candidates per bucket where this one evaluates 1016
// (N = 2^20, k = 64).
#pragma once

#include "sidm_plan.hpp"
#include "sidm_wave.hpp"

namespace sidm {

constexpr int kSearchPop = 8;   // pending nodes taken per round: 64 children
// Popping at most kSearchPop nodes per round and pushing their inner children, the
// stack holds at most (kFanout - 1) kSearchPop nodes per level above the
// lowest inner one, plus a round's pushes; halos of at most 2^24 particles have
// six levels above their buckets.
constexpr int kSearchLevels = 6;
constexpr int kSearchStack = (kFanout - 1) * kSearchPop * kSearchLevels + kFanout * kSearchPop;
// Groups: each searching lane its own where they are few; the octets of
// lanes, cut in two where the compact sub-range of an octet's first searching
// lane ends (a jump of the Morton curve), for up to a quarter of a wave; else
// the compact sub-ranges.  Fewer lanes have fewer candidates over which to spread
// the tests, and a lane's worth of them each: kernel sizes of 8192 particles
// (4 lanes a wave) 0.25 ms with sub-ranges, 0.15 with single lanes; of 2^20
// (whole waves) 1.72 ms with sub-ranges, 2.0 with octets.
constexpr int kSearchGroups = 16;
constexpr int kSearchSingles = 8;
constexpr int kSearchOctets = 16;
constexpr int kSearchList = 128;   // buckets that passed, 64 of them pending at most

struct SearchLds {
    uint32_t stack[kSearchStack];
    uint32_t list[kSearchList];
    double group[kSearchGroups][8];   // box (lo xyz, hi xyz), reach
};

// v moved by a DPP control that stays within octets of lanes
template <int CTRL>
__device__ inline double oct_min(double v)
{
    return fmin(v, dpp_f64<CTRL>(v));
}
template <int CTRL>
__device__ inline double oct_max(double v)
{
    return fmax(v, dpp_f64<CTRL>(v));
}

// Box of the octet's lanes with `in` set, and their largest reach.
__device__ inline void octet_group(bool in, double x, double y, double z, double reach, double* o)
{
    const double p[3] = {x, y, z};
#pragma unroll
    for (int c = 0; c < 7; ++c) {
        if (c < 3) {
            double v = in ? p[c] : INFINITY;
            v = oct_min<0xB1>(v);           // quad_perm [1, 0, 3, 2]
            v = oct_min<0x4E>(v);           // quad_perm [2, 3, 0, 1]
            o[c] = oct_min<0x141>(v);       // row_half_mirror
        } else {
            double v = in ? (c < 6 ? p[c - 3] : reach) : -INFINITY;
            v = oct_max<0xB1>(v);
            v = oct_max<0x4E>(v);
            o[c] = oct_max<0x141>(v);
        }
    }
}

// The compact sub-range of a bucket that holds its lane-th particle.
__device__ inline int lane_sub(const SubRange* __restrict__ sub, int ns, int lane)
{
    int f = 0;
    while (f + 1 < ns && lane >= sub[f + 1].off) ++f;
    return f;
}

// The groups of the lanes with `on` set (uniform call); returns their number.
// sid: the lane's compact sub-range.  reach: what the caller's tests take (a
// distance or its square).
__device__ inline int search_groups(SearchLds& L, int lane, int sid, bool on, double x, double y,
                                    double z, double reach)
{
    __syncthreads();
    const unsigned long long m = __ballot(on), below = (1ull << lane) - 1ull;
    int nq = __popcll(m);
    if (nq == 0) return 0;
    if (nq <= kSearchSingles) {
        if (on) {
            double* g = L.group[__popcll(m & below)];
            g[0] = g[3] = x;
            g[1] = g[4] = y;
            g[2] = g[5] = z;
            g[6] = reach;
        }
    } else if (nq > kSearchOctets) {
        unsigned long long todo = m;
        nq = 0;
        while (todo) {
            const int s0 = __shfl(sid, __ffsll((long long)todo) - 1, 64);
            const bool in = on && sid == s0;
            double o[6];
            lanes_box(in, x, y, z, o);
            const double r = rows_max(row_max(in ? reach : -INFINITY));
            if (lane == 0) {
#pragma unroll
                for (int c = 0; c < 6; ++c) L.group[nq][c] = o[c];
                L.group[nq][6] = r;
            }
            ++nq;
            todo &= ~__ballot(in);
        }
    } else {
        // the sub-range of the octet's first searching lane
        const unsigned oct = (unsigned)(m >> (lane & 56)) & 0xFFu;
        const int s0 = __shfl(sid, (lane & 56) + (oct ? __ffs((int)oct) - 1 : 0), 64);
        const bool one = on && sid == s0, two = on && sid != s0;
        nq = 0;
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            const unsigned long long mp = __ballot(part ? two : one);
            if (!mp) continue;
            double o[7];
            octet_group(part ? two : one, x, y, z, reach, o);
            const bool lead = (lane & 7) == 0 && ((mp >> lane) & 0xFFull);
            const unsigned long long ml = __ballot(lead);
            if (lead)
#pragma unroll
                for (int c = 0; c < 7; ++c) L.group[nq + __popcll(ml & below)][c] = o[c];
            nq += __popcll(ml);
        }
    }
    __syncthreads();
    return nq;
}

// Squared distance from group q's box to the box (lo, hi) / the point p.
__device__ inline double group_box_dist2(const double* g, const double* __restrict__ b)
{
    const double gx = fmax(fmax(b[0] - g[3], g[0] - b[3]), 0.0);
    const double gy = fmax(fmax(b[1] - g[4], g[1] - b[4]), 0.0);
    const double gz = fmax(fmax(b[2] - g[5], g[2] - b[5]), 0.0);
    return gx * gx + gy * gy + gz * gz;
}

// Squared distance from point p to an axis-aligned box (lo xyz, hi xyz).
__device__ inline double point_box_dist2(double px, double py, double pz,
                                         const double* __restrict__ b)
{
    const double gx = fmax(fmax(b[0] - px, px - b[3]), 0.0);
    const double gy = fmax(fmax(b[1] - py, py - b[4]), 0.0);
    const double gz = fmax(fmax(b[2] - pz, pz - b[5]), 0.0);
    return gx * gx + gy * gy + gz * gz;
}

__device__ inline double group_point_dist2(const double* g, double px, double py, double pz)
{
    const double gx = fmax(fmax(g[0] - px, px - g[3]), 0.0);
    const double gy = fmax(fmax(g[1] - py, py - g[4]), 0.0);
    const double gz = fmax(fmax(g[2] - pz, pz - g[5]), 0.0);
    return gx * gx + gy * gy + gz * gz;
}

// The buckets of the halo for which test(node) holds; internal nodes are entered
// on the same condition (it must be monotone).  test runs on lanes with a
// different node each.  drain(n, last) takes the first n entries of L.list (uniform); the call
// with `last` set ends the walk (n may be 0).
template <class Test, class Drain>
__device__ inline void search_walk(const HaloDev& H, const NodeChild* __restrict__ nodes,
                                   int64_t n_buckets, SearchLds& L, Test test, Drain drain)
{
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (1ull << lane) - 1ull;
    const uint32_t root = (uint32_t)H.level_off[H.n_levels - 1];
    __syncthreads();
    if (lane == 0) L.stack[0] = L.list[0] = root;
    __syncthreads();
    const bool one = H.n_levels == 1;   // one bucket
    int sp = one ? 0 : 1, ln = one ? 1 : 0;
    for (;;) {
        const int npop = sp < kSearchPop ? sp : kSearchPop;
        const int slot = lane / kFanout;
        bool hit = false, leaf = false;
        uint32_t c = 0;
        if (slot < npop) {
            const NodeChild N = nodes[L.stack[sp - 1 - slot]];
            const int ci = lane % kFanout;
            if (ci < N.nchild) {
                c = (uint32_t)N.child0 + ci;
                leaf = N.child0 < n_buckets;
                hit = test((int64_t)c);
            }
        }
        sp -= npop;
        __syncthreads();   // the popped entries are read before pushes reuse them
        const unsigned long long ml = __ballot(hit && leaf), mi = __ballot(hit && !leaf);
        if (hit && leaf) L.list[ln + __popcll(ml & below)] = c;
        if (hit && !leaf) L.stack[sp + __popcll(mi & below)] = c;
        ln += __popcll(ml);
        sp += __popcll(mi);
        __syncthreads();
        if (sp == 0 || ln > kSearchList - 64) {
            drain(ln, sp == 0);
            ln = 0;
            __syncthreads();
            if (sp == 0) return;
        }
    }
}

// First particle (sorted position) and number of particles of bucket c.
__device__ inline int64_t bucket_start(const HaloDev& H, uint32_t c, int& count)
{
    const int64_t j0 = ((int64_t)c - H.level_off[0]) * kBucket, left = H.n - j0;
    count = (int)(left < kBucket ? left : kBucket);
    return H.sbase + j0;
}

}  // namespace sidm
