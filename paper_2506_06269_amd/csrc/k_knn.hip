// k_knn.hip -- the SIDM kernel size h_i = distance to the k-th nearest other
// particle of the halo (Sec. 2: the kernel size is set by the next N_ngb
// neighbours).
//
// One wavefront per bucket of 64 Morton-consecutive particles, one particle
// per lane, all lanes resolved together (each with its own search sphere).  A
// visit collects the particles that can lie within some lane's sphere
// (sidm_search.hpp); every lane then evaluates each of them.
// Selection works on values only.  When the particle's kernel size before
// the call is a usable value h0 (a warm start: the result does not depend on
// it), one visit of the sphere of radius (1 + d) h0 counts the candidates
// closer than (1 - d) h0 and lists those in between (the band) in an LDS column
// of the lane; if the k-th distance lies in the band and among its kKnnBand
// smallest, it is read off the listed ones.
// In a step h changes by a few tenths of a per cent (a few per cent at the
// tail), so almost every lane ends here.  The other lanes, and lanes without
// a usable h0, take the general search, with a private 32-bin histogram per
// lane (an LDS column, written with LDS atomics that return nothing):
//   1. a histogram of the distances within a starting radius: 1.15 times h0
//      when it is usable, else an estimate out of the nearest of the particles
//      up to a bucket before and after in sorted order; the radius grows until
//      the sphere holds k others;
//   2. a visit restricted to the shell of the bin that holds the k-th
//      collects that bin's members (at most 16, kept sorted in registers) or,
//      if it holds more, records their min..max, whose histogram (step 1 over
//      that range) refines the choice; equal values end the refinement.
// Typical cost: one visit when warm; three for the general search.
//
// Bound by vector issue and the waits between (a warm call of 2^20: vector units
// busy 51 % of the cycles, waves waiting 38 %; 200003 without previous sizes,
// one round of waves of which the slowest last three times the mean: 27 and 41
// %): about 75 cycles per candidate and wave (eight FP64
// operations of four cycles, three comparisons, four LDS reads shared by four
// candidates), most of the rest the tests that select them.  A call of 2^20
// particles (k 64) takes 1.73 ms warm and 5.6 ms without previous sizes, the
// neighbour lists 2.8 ms more (2.6, 9.6 and 18 ms with the lane-by-lane search,
// single row stores and a distance per band slot); 8192 particles (k 32) 0.14
// and 0.27 ms (0.25 and 2.4).
// Distances d2 = (dx*dx + dy*dy) + dz*dz are evaluated in FP64 without fused
// multiply-add, the same expression the oracle uses, so h matches bit for bit.
#include "sidm_search.hpp"

namespace sidm {

constexpr int kKnnBins = 32;
constexpr int kKnnSurv = 16;
constexpr int kKnnLevels = 4;
constexpr int kKnnGrow = 80;
constexpr double kKnnWarm = 1.15 * 1.15;   // squared margin on the previous kernel size
// squared margin on the estimate without one (calls without previous sizes at
// N = 2^20 with 0.35, 0.5, 0.7, 1 and 2: 5.5, 5.3, 5.5, 5.9 and 8.5 ms; 8192: 0.29,
// 0.29, 0.28, 0.27)
constexpr double kKnnCold = 0.7;
constexpr int kKnnBand = 16;               // smallest distances of the band kept per lane
constexpr int kKnnGroup = 4;               // candidates evaluated at once
constexpr int kKnnSplitMax = 16;           // waves per bucket for calls with few buckets

// The band pass and the general search never run at once: the band's
// candidates (sorted indices) are listed in the lane's histogram column (a
// barrier separates the two uses).
struct KnnLds {
    uint32_t hist[kKnnBins][kBucket];
    SearchLds S;
    // candidates within reach of some lane: position and sorted index
    double x[2 * kBucket + kKnnGroup], y[2 * kBucket + kKnnGroup], z[2 * kBucket + kKnnGroup];
    uint32_t p[2 * kBucket + kKnnGroup];
};

__device__ inline double dist2_exact(double ax, double ay, double az, double bx, double by,
                                     double bz)
{
#pragma clang fp contract(off)
    const double dx = bx - ax, dy = by - ay, dz = bz - az;
    return (dx * dx + dy * dy) + dz * dz;
}

__device__ inline double box_diag2_k(const double* b)
{
    const double ex = b[3] - b[0], ey = b[4] - b[1], ez = b[5] - b[2];
    return ex * ex + ey * ey + ez * ez;
}

// Bin of d2 among kKnnBins equal bins starting at lo (monotone in d2; NaN
// products, from an infinite inv, fall in bin 0).
__device__ inline int bin_of(double d2, double lo, double inv)
{
    const double t = (d2 - lo) * inv;
    return t >= (double)(kKnnBins - 1) ? kKnnBins - 1 : (t > 0.0 ? (int)t : 0);
}

// Insertion of v into the ascending list best[0..M) (registers).
template <int M>
__device__ inline void insert_sorted(double (&best)[M], double v)
{
#pragma unroll
    for (int q = 0; q < M; ++q) {
        const double lo = fmin(best[q], v);
        v = fmax(best[q], v);
        best[q] = lo;
    }
}

template <bool LIST>
__global__ __launch_bounds__(kBucket) void k_knn(
    const HaloDev* __restrict__ halos, const BucketInfo* __restrict__ buckets,
    const NodeChild* __restrict__ nodes, const double* __restrict__ box,
    const SubRange* __restrict__ sub, const int* __restrict__ sub_n, int64_t n_buckets,
    const double* __restrict__ sx, const double* __restrict__ sy, const double* __restrict__ sz,
    const uint32_t* __restrict__ perm,
    double* __restrict__ sh, double* __restrict__ h_out, int* __restrict__ status,
    const uint32_t* __restrict__ sid, uint32_t* __restrict__ nbr, int k_max, int split)
{
    __shared__ KnnLds L;
    // split waves per bucket: wave `part` resolves the bucket's lanes
    // [part, part + 1) * 64 / split (a call with few buckets still fills the
    // device, and each wave's candidates are those of its own lanes' spheres)
    const int64_t bw = xcd_contiguous(blockIdx.x, gridDim.x);
    const int64_t b = bw / split;
    const int part = (int)(bw % split);
    const int lane = threadIdx.x;
    const BucketInfo B = buckets[b];
    const HaloDev& H = halos[B.halo];
    const int k = H.k;
    const bool in_bucket = lane < B.count && lane / (kBucket / split) == part;
    const uint32_t mypos = (uint32_t)(B.start + (in_bucket ? lane : 0));
    const double xi = sx[mypos], yi = sy[mypos], zi = sz[mypos];
    const double hint = sh[mypos];   // the kernel size before the call
    const double diag2 = box_diag2_k(box + 6 * H.level_off[H.n_levels - 1]);
    const int sid_l = lane_sub(sub + kSubMax * b, sub_n[b], lane);

    // every candidate within reach of a lane's sphere (radius^2 r2 of the lane;
    // lanes with `off` set do not search); body(p, d2) runs on every lane for
    // kKnnGroup candidates p at once and their squared distances d2 (NaN, and p
    // of no meaning, past the last one): their LDS reads and arithmetic overlap,
    // and one branch serves them all
    auto visit = [&](double r2, bool off, auto body) __attribute__((always_inline)) {
        const int nq = search_groups(L.S, lane, sid_l, !off, xi, yi, zi, r2);
        if (nq == 0) return;
        const bool singles = nq == __popcll(__ballot(!off));   // every group one lane
        int bn = 0;   // candidates in LDS
        auto process = [&](int n) {
            // at most 2 kBucket - 1 entries are in use; the distance of the
            // others is NaN, in no range (an infinite one lies in a range that
            // ends at infinity, and its index ~0 would be read)
            if (lane < kKnnGroup) L.x[n + lane] = NAN;
            __syncthreads();
            for (int j = 0; j < n; j += kKnnGroup) {
                uint32_t p[kKnnGroup];
                double d2[kKnnGroup];
#pragma unroll
                for (int u = 0; u < kKnnGroup; ++u) {
                    p[u] = L.p[j + u];
                    d2[u] = dist2_exact(xi, yi, zi, L.x[j + u], L.y[j + u], L.z[j + u]);
                }
                body(p, d2);
            }
            __syncthreads();
        };
        auto drain = [&](int ln, bool last) __attribute__((always_inline)) {
            // the buckets whose box some lane reaches (the groups' boxes can
            // hold the dense centre without any lane near it)
            int kept = singles ? ln : 0;
            for (int i = 0; i < ln && !singles; i += 4) {
                uint32_t c[4];
                unsigned long long m[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    c[u] = __builtin_amdgcn_readfirstlane(L.S.list[min(i + u, ln - 1)]);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    m[u] = __ballot(!off &&
                                    point_box_dist2(xi, yi, zi, box + 6 * (int64_t)c[u]) <= r2);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (m[u] && i + u < ln) {
                        if (lane == 0) L.S.list[kept] = c[u];
                        ++kept;
                    }
            }
            __syncthreads();
            if (kept == 0) return;
            // the next bucket's particles are in flight while one is tested
            int cnt;
            int64_t p0 = bucket_start(H, __builtin_amdgcn_readfirstlane(L.S.list[0]), cnt);
            bool on = lane < cnt;
            int64_t p = p0 + (on ? lane : 0);
            double x = sx[p], y = sy[p], z = sz[p];
            for (int i = 0; i < kept; ++i) {
                const double cx = x, cy = y, cz = z;
                const uint32_t cp = (uint32_t)p;
                const bool con = on;
                if (i + 1 < kept) {
                    p0 = bucket_start(H, __builtin_amdgcn_readfirstlane(L.S.list[i + 1]), cnt);
                    on = lane < cnt;
                    p = p0 + (on ? lane : 0);
                    x = sx[p]; y = sy[p]; z = sz[p];
                }
                bool keep = false;
                for (int q = 0; q < nq; ++q)
                    keep |= group_point_dist2(L.S.group[q], cx, cy, cz) <= L.S.group[q][6];
                const unsigned long long m = __ballot(con && keep);
                if (con && keep) {
                    const int at = bn + __popcll(m & ((1ull << lane) - 1ull));
                    L.x[at] = cx;
                    L.y[at] = cy;
                    L.z[at] = cz;
                    L.p[at] = cp;
                }
                bn += __popcll(m);
                if (bn >= kBucket) {
                    process(bn);
                    bn = 0;
                }
            }
        };
        search_walk(H, nodes, n_buckets, L.S,
                    [&](int64_t c) {
                        bool in = false;
                        for (int q = 0; q < nq; ++q)
                            in |= group_box_dist2(L.S.group[q], box + 6 * c) <= L.S.group[q][6];
                        return in;
                    },
                    drain);
        if (bn > 0) process(bn);
    };
    // histogram of the distances in [a, z] over kKnnBins bins from lo
    auto histogram = [&](bool on, double a, double z, double lo, double inv)
        __attribute__((always_inline)) {
        if (on)
            for (int q = 0; q < kKnnBins; ++q) L.hist[q][lane] = 0u;
        visit(z * (1.0 + 1e-9), !on, [&](const uint32_t (&p)[kKnnGroup],
                                         const double (&d2)[kKnnGroup]) {
#pragma unroll
            for (int u = 0; u < kKnnGroup; ++u)
                if (on && p[u] != mypos && d2[u] >= a && d2[u] <= z)
                    atomicAdd(&L.hist[bin_of(d2[u], lo, inv)][lane], 1u);
        });
        __syncthreads();
    };

    // h^2 of the lanes with act set, from a starting radius^2 u2 (NaN for the
    // others); a uniform call: every lane of the wave takes part
    auto resolve = [&](bool act, double u2) __attribute__((always_inline)) {
        // ---- 1. histogram of [0, u2]; grow until the sphere holds k others
        bool need = act, failed = false;
        int grow = 0;
        while (__ballot(need)) {
            histogram(need, 0.0, u2, 0.0, (double)kKnnBins / u2);
            if (need) {
                int tot = 0;
                for (int q = 0; q < kKnnBins; ++q) tot += (int)L.hist[q][lane];
                if (tot >= k) {
                    need = false;
                } else if (++grow > kKnnGrow) {
                    need = false;
                    failed = true;
                    atomicOr(&status[B.halo], SIDM_DEV_KNN_OVERFLOW);
                } else {
                    double f = tot > 0 ? 1.44 * pow((double)k / (double)tot, 2.0 / 3.0) : 4.0;
                    u2 *= fmin(fmax(f, 1.44), 4.0);
                }
            }
        }

        // ---- 2. select the bin of the k-th, collect its members or refine.
        // Members of the current set lie in [a, z]; its histogram uses bins
        // (lo, inv); `below` counts the candidates under the selected bin.
        bool done = !act || failed;
        double a = 0.0, z = u2, lo = 0.0, inv = (double)kKnnBins / u2;
        int below = 0, level = 0;
        double d2k = NAN;
        while (__ballot(!done)) {
            int sel = -1, inb = 0;
            double shell2 = 0.0;
            if (!done) {
                int cum = below;
                for (int q = 0; q < kKnnBins; ++q) {
                    const int hq = (int)L.hist[q][lane];
                    if (cum + hq >= k) { sel = q; inb = hq; break; }
                    cum += hq;
                }
                if (sel < 0) {   // cannot happen: the set holds the k-th
                    done = true;
                    atomicOr(&status[B.halo], SIDM_DEV_KNN_OVERFLOW);
                } else {
                    below = cum;
                    shell2 = inv > 0.0 && isfinite(inv) ? fmin(z, lo + (double)(sel + 1) / inv) : z;
                }
            }
            double best[kKnnSurv];
#pragma unroll
            for (int q = 0; q < kKnnSurv; ++q) best[q] = INFINITY;
            double mn = INFINITY, mxv = -INFINITY;
            const bool collect = !done && inb <= kKnnSurv;
            visit(shell2 * (1.0 + 1e-9), done, [&](const uint32_t (&p)[kKnnGroup],
                                                   const double (&d2)[kKnnGroup]) {
                bool hit[kKnnGroup], any = false;
#pragma unroll
                for (int u = 0; u < kKnnGroup; ++u) {
                    hit[u] = !done & (p[u] != mypos) & (d2[u] >= a) & (d2[u] <= z) &
                             (bin_of(d2[u], lo, inv) == sel);
                    any |= hit[u];
                }
                if (!__ballot(any)) return;
                for (int u = 0; u < kKnnGroup; ++u) {
                    if (!__ballot(hit[u])) continue;
                    if (hit[u]) {
                        mn = fmin(mn, d2[u]);
                        mxv = fmax(mxv, d2[u]);
                        if (collect) insert_sorted(best, d2[u]);
                    }
                }
            });
            bool refine = false;
            if (!done) {
                if (collect) {
                    const int r = k - below - 1;
#pragma unroll
                    for (int q = 0; q < kKnnSurv; ++q)
                        if (q == r) d2k = best[q];
                    done = true;
                } else if (mn == mxv) {
                    d2k = mn;        // all members tie at the k-th distance
                    done = true;
                } else if (++level >= kKnnLevels) {
                    done = true;
                    atomicOr(&status[B.halo], SIDM_DEV_KNN_OVERFLOW);
                } else {
                    a = mn;
                    z = mxv;
                    lo = mn;
                    inv = (double)kKnnBins / (mxv - mn);
                    refine = true;
                }
            }
            if (__ballot(refine)) histogram(refine, a, z, lo, inv);
        }
        return act ? d2k : NAN;
    };

    // h^2 of the lanes with act set from one visit of the band around their
    // previous kernel size h0 (NaN for lanes whose k-th distance is not
    // among the kept band values); a uniform call
    auto band_pass = [&](bool act, double h0) __attribute__((always_inline)) {
        // half-width relative to h0: about 12 band members expected (a
        // spherical shell of relative width 2d holds about 6 d k
        // neighbours), at least 1 %, at most 6 %
        const double d = fmin(fmax(2.0 / (double)k, 0.01), 0.06);
        const double rlo = h0 * (1.0 - d), rhi = h0 * (1.0 + d);
        const double blo = rlo * rlo, bhi = rhi * rhi;
        // below the band; candidates in the band, listed in the lane's column
        int nlo = 0, kept = 0;
        visit(bhi * (1.0 + 1e-9), !act, [&](const uint32_t (&p)[kKnnGroup],
                                            const double (&d2)[kKnnGroup]) {
#pragma unroll
            for (int u = 0; u < kKnnGroup; ++u) {
                const bool other = act & (p[u] != mypos), lo = d2[u] < blo;
                nlo += other & lo;
                if (other & !lo & (d2[u] <= bhi)) {
                    L.hist[min(kept, kKnnBins - 1)][lane] = p[u];
                    ++kept;
                }
            }
        });
        // the k-th distance has rank r (0-based) in the band: the r-th of the
        // listed candidates' distances (evaluated again) when the list holds
        // the whole band
        const int r = k - nlo - 1;
        const bool ok = act && r >= 0 && r < kept && r < kKnnBand && kept <= kKnnBins;
        if (!ok) kept = 0;
        __syncthreads();
        double best[kKnnBand];
#pragma unroll
        for (int q = 0; q < kKnnBand; ++q) best[q] = INFINITY;
        for (int q = 0; __ballot(q < kept); q += kKnnGroup) {
            double v[kKnnGroup];
#pragma unroll
            for (int u = 0; u < kKnnGroup; ++u) {
                const uint32_t p = q + u < kept ? L.hist[q + u][lane] : mypos;
                v[u] = dist2_exact(xi, yi, zi, sx[p], sy[p], sz[p]);
            }
#pragma unroll
            for (int u = 0; u < kKnnGroup; ++u)
                insert_sorted(best, q + u < kept ? v[u] : INFINITY);
        }
        double d2k = NAN;
#pragma unroll
        for (int q = 0; q < kKnnBand; ++q)
            if (ok && q == r) d2k = best[q];
        __syncthreads();   // the band columns are read before the histograms reuse them
        return d2k;
    };

    // ---- starting radius
    const bool warm = isfinite(hint) && hint > 0.0 && hint * hint <= diag2;
    double u2 = kKnnWarm * hint * hint;
    if (__ballot(in_bucket && !warm)) {
        // an estimate: the m-th nearest (m <= 8) of the particles up to a bucket
        // before and after this one in sorted order, scaled to k neighbours
        constexpr int kM = 8;
        double best[kM];
#pragma unroll
        for (int q = 0; q < kM; ++q) best[q] = INFINITY;
        const int64_t q0 = max(B.start - kBucket, H.sbase);
        const int64_t q1 = min(B.start + 2 * kBucket, H.sbase + H.n);
        for (int64_t q = q0; q < q1; ++q) {
            const double v = dist2_exact(xi, yi, zi, sx[q], sy[q], sz[q]);
            const bool nearer = (uint32_t)q != mypos && v < best[kM - 1];
            if (!__ballot(nearer)) continue;
            insert_sorted(best, nearer ? v : INFINITY);
        }
        const int m = min(min(kM, k), (int)(q1 - q0) - 1);
        double rm2 = 0.0;
#pragma unroll
        for (int q = 0; q < kM; ++q)
            if (q == m - 1) rm2 = best[q];
        // (from the halo's diagonal / N, far below any neighbour distance, where
        // there are too few to go by)
        double e2 = m >= 1 && rm2 > 0.0 && rm2 < INFINITY
                        ? kKnnCold * rm2 * pow((double)k / (double)m, 2.0 / 3.0)
                        : diag2 / ((double)H.n * (double)H.n);
        if (!(e2 > 0.0)) e2 = 1.0;
        if (!warm) u2 = e2;
    }
    double d2k = NAN;
    bool todo = in_bucket;
    if (__ballot(in_bucket && warm)) {
        d2k = band_pass(in_bucket && warm, hint);
        todo = in_bucket && !(d2k >= 0.0);
    }
    const double d2g = resolve(todo, u2);
    if (todo) d2k = d2g;
    if (in_bucket) {
        const double h = sqrt(d2k);
        sh[mypos] = h;
        h_out[perm[mypos]] = h;
    }
    if (!LIST) return;

    // Neighbour lists: the members of the sphere of the k-th distance, as
    // sorted positions in the particle's row (k_knn_list_order puts them in
    // (d2, id) order and turns them into ids).  The candidates strictly closer
    // than the k-th (fewer than k) are staged in the lane's LDS column, entry q
    // in column (lane + q) mod 64, and written out row by row (stores of
    // single entries, each lane to a row of its own, took 18 of the 21 ms of a
    // warm call at N = 2^20).  Candidates at exactly the k-th distance fill
    // the rest: one as a rule; when they are more than the rest, those with the
    // smallest ids, in a visit of their own.
    const uint32_t my_row = in_bucket ? perm[mypos] : 0u;
    const bool on = in_bucket && isfinite(d2k);
    int cnt = 0, staged = 0, ties = 0;
    uint32_t tie = 0u;
    auto flush = [&]() {
        __syncthreads();
        unsigned long long act = __ballot(staged > 0);
        while (act) {
            const int r = __ffsll((long long)act) - 1;
            act &= act - 1ull;
            const int n = __shfl(staged, r, 64), base = __shfl(cnt, r, 64);
            const uint32_t row = __shfl(my_row, r, 64);
            if (lane < n)
                nbr[(int64_t)row * k_max + base + lane] = L.hist[lane][(r + lane) & 63];
        }
        cnt += staged;
        staged = 0;
        __syncthreads();
    };
    visit(d2k * (1.0 + 1e-9), !on, [&](const uint32_t (&p)[kKnnGroup],
                                       const double (&d2)[kKnnGroup]) {
#pragma unroll
        for (int u = 0; u < kKnnGroup; ++u) {
            const bool other = on & (p[u] != mypos);
            if (other & (d2[u] < d2k)) {
                L.hist[staged][(lane + staged) & 63] = p[u];
                ++staged;
            }
            const bool same = other & (d2[u] == d2k);
            tie = same ? p[u] : tie;
            ties += same;
        }
        if (__ballot(staged > kKnnBins - kKnnGroup)) flush();
    });
    flush();
    const int need = on ? k - cnt : 0;
    if (on && ties == 1 && need == 1) nbr[(int64_t)my_row * k_max + cnt] = tie;
    const bool more = on && !(ties == 1 && need == 1);
    if (!__ballot(more)) return;
    uint32_t* row = nbr + (int64_t)my_row * k_max;
    int nt = 0;
    visit(d2k * (1.0 + 1e-9), !more, [&](const uint32_t (&p)[kKnnGroup],
                                         const double (&d2)[kKnnGroup]) {
        for (int u = 0; u < kKnnGroup; ++u) {
            if (!(more && p[u] != mypos && d2[u] == d2k && need > 0)) continue;
            if (nt < need) {
                row[cnt + nt++] = p[u];
                continue;
            }
            int worst = 0;
            uint32_t wid = 0;
            for (int q = 0; q < need; ++q) {
                const uint32_t iq = sid[row[cnt + q]];
                if (iq >= wid) {
                    wid = iq;
                    worst = q;
                }
            }
            if (sid[p[u]] < wid) row[cnt + worst] = p[u];
        }
    });
}

// The rows k_knn collected, in (d2, id) order, as ids: one wave per particle,
// two entries per lane, each entry's place the number of entries before it (the
// distances recomputed with the same expression).  One thread per particle
// with an insertion sort in scratch memory took 0.80 ms for 200003 rows of 32.
constexpr int kListWaves = 4;
static_assert(SIDM_MAX_K <= 128, "two entries per lane");
__global__ __launch_bounds__(64 * kListWaves) void k_knn_list_order(
    const uint32_t* __restrict__ perm, const BucketInfo* __restrict__ buckets,
    const HaloDev* __restrict__ halos, const double* __restrict__ sx,
    const double* __restrict__ sy, const double* __restrict__ sz, const double* __restrict__ sh,
    const uint32_t* __restrict__ sid, int k_max, uint32_t* __restrict__ nbr)
{
    __shared__ double d2s[kListWaves][SIDM_MAX_K];
    __shared__ uint32_t ids[kListWaves][SIDM_MAX_K];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const BucketInfo B = buckets[blockIdx.x];
    const int k = halos[B.halo].k;
    for (int i = wv; i < B.count; i += kListWaves) {
        const int64_t me = B.start + i;
        if (!isfinite(sh[me])) continue;   // a failed search has no row
        uint32_t* row = nbr + (int64_t)perm[me] * k_max;
        const double xi = sx[me], yi = sy[me], zi = sz[me];
        double d[2];
        uint32_t id[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int q = lane + 64 * u;
            d[u] = INFINITY;
            id[u] = 0u;
            if (q < k) {
                const uint32_t p = row[q];
                d[u] = dist2_exact(xi, yi, zi, sx[p], sy[p], sz[p]);
                id[u] = sid[p];
                d2s[wv][q] = d[u];
                ids[wv][q] = id[u];
            }
        }
        // a wave's own LDS rows, read back in program order
        __builtin_amdgcn_wave_barrier();
        int at[2] = {0, 0};
        for (int q = 0; q < k; ++q) {
            const double dq = d2s[wv][q];
            const uint32_t iq = ids[wv][q];
#pragma unroll
            for (int u = 0; u < 2; ++u)
                at[u] += dq < d[u] || (dq == d[u] && iq < id[u]);
        }
        // Entries equal in both (the state should not hold equal ids) have one
        // place between them, and the sum of the places is short: they follow
        // the row's order.  (Told apart in the loop above: 190 us for 158.)
        const int sum = lanes_scan((lane < k ? at[0] : 0) + (lane + 64 < k ? at[1] : 0));
        if (__builtin_amdgcn_readlane(sum, 63) != k * (k - 1) / 2)
            for (int q = 0; q < k; ++q)
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    at[u] += d2s[wv][q] == d[u] && ids[wv][q] == id[u] && q < lane + 64 * u;
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (lane + 64 * u < k) row[at[u]] = id[u];
        __builtin_amdgcn_wave_barrier();
    }
}

hipError_t launch_knn(const Plan& P, const sidm_state* s, Scratch& w, uint32_t* nbr, int k_max,
                      hipStream_t st)
{
    const int split = search_split(P.n_buckets, kKnnSplitMax);
    auto search = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)(P.n_buckets * split)), dim3(kBucket), 0, st,
                           w.halos, w.buckets, w.nodes, w.box, w.sub, w.sub_n, P.n_buckets, w.sx,
                           w.sy, w.sz, w.perm, w.sh, s->h, w.status, w.sid, nbr, k_max, split);
    };
    if (!nbr) {
        search(k_knn<false>);
        return hipGetLastError();
    }
    search(k_knn<true>);
    hipLaunchKernelGGL(k_knn_list_order, dim3((unsigned)P.n_buckets), dim3(64 * kListWaves), 0,
                       st, w.perm, w.buckets, w.halos, w.sx, w.sy, w.sz, w.sh, w.sid, k_max,
                       nbr);
    return hipGetLastError();
}

}  // namespace sidm
