// k_scatter.hip -- SIDM scattering pass (Sec. 2: rare pairwise scatterings
// through the spline kernel, explicitly conserving energy and momentum;
// Sec. 3.5: the geometric factor Lambda of the interaction probability).
//
// k_pairs: one wavefront per bucket, one i per lane.  The candidates j are the
// particles closer than h_i + h_j to the box of a group of its lanes, h_i the
// group's largest (sidm_search.hpp); every lane tests each of them.
// A bucket takes only candidate buckets of higher index, after the pairs inside
// it, so each pair is tested once, when d2 < (h_i + h_j)^2: first on the matrix
// cores, 32 i by 32 j at once, to within a rounding bound; the pairs that pass
// go through an LDS queue (prefix count) so that the exact test and the
// expensive per-pair work -- Philox4x32-10, |dv|, and Lambda when the draw falls
// below a cheap upper bound of P -- run on full wavefronts.  A pair whose draw
// falls below the bound is appended to a candidate buffer; k_decide evaluates
// Lambda for those and appends the events (u < P) to the event buffer (when the
// candidate buffer is full, the pair pass decides the rest itself).
//
// What bounds it: vector issue (N = 500009: busy 69 % of the cycles, waves
// waiting 30 %; 2^20 74 %).  Half of the time is per-pair work, a chain of LDS
// reads, gathered velocities and ten dependent rounds of the generator at three
// waves per SIMD (145 registers), so each lane takes two pairs at once (64
// halos: 5.4 -> 4.9 ms; four waves with fewer registers: 6.0); a quarter is the
// search, a quarter the screen and the queue.  One in six screened pairs is
// accepted; in double precision on the vector unit they took half of the pass.
//            N = 500009 (126 M pairs)   2^20 (265 M)   64 halos (571 M)   8192
//   bucket after bucket, chunk boxes   2.10 ms   3.7   7.4   0.110
//   candidates a lane each             1.42      2.65  5.9   0.074
//   and the screen                     1.17      2.2   4.9   0.058
//
// k_rounds: the events of a step are applied in (a, b) order as elastic,
// isotropic kicks in the pair's centre-of-mass frame.  Events that share no
// particle commute, so the order is realised by rounds: in each round every
// particle elects the smallest pending event key it belongs to (atomicMin),
// and an event fires when it is the elected one for both of its particles.
// This is exactly the dependency order of one-after-the-other application.
#include "sidm_math.hpp"
#include "sidm_search.hpp"

namespace sidm {

__device__ inline double dist2_pair(double ax, double ay, double az, double bx, double by,
                                    double bz)
{
#pragma clang fp contract(off)
    const double dx = bx - ax, dy = by - ay, dz = bz - az;
    return (dx * dx + dy * dy) + dz * dz;
}

__device__ inline double norm3(double x, double y, double z)
{
#pragma clang fp contract(off)
    return sqrt((x * x + y * y) + z * z);
}

__global__ void k_scatter_reset(DevCounters* __restrict__ counters,
                                unsigned long long* __restrict__ ev_counts, int* __restrict__ status,
                                int n_halos)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t == 0) {
        counters->n_events_total = 0ull;
        counters->n_cands = 0ull;
        counters->ticket = 0ull;
    }
    if (t < kEvCounts * n_halos) ev_counts[t] = 0ull;
    if (t < n_halos) status[t] = 0;
}

// ---------------------------------------------------------------- contract checks
// Ids key the random draws and order the kicks, so they must be unique per
// halo.  Every particle inserts its key (halo << 32 | id) into an open-
// addressing hash table of cap >= 2 n slots (linear probing, the empty slot
// ~0, which no key equals: halo indices stay below 2^31); finding its own key
// already there flags the halo.  A table at most half full always has an
// empty slot, so every probe sequence ends.
constexpr unsigned long long kEmptySlot = ~0ull;

__global__ __launch_bounds__(256) void k_fill_u64(unsigned long long* __restrict__ a, int64_t n,
                                                   unsigned long long v)
{
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < n; p += (int64_t)gridDim.x * 256)
        a[p] = v;
}

__device__ inline unsigned long long mix64(unsigned long long z)
{
    // the finaliser of SplitMix64 (Steele, Lea and Flood 2014)
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

__global__ __launch_bounds__(kStreamBlock) void k_id_insert(
    const StreamBlock* __restrict__ blocks, const uint32_t* __restrict__ id,
    unsigned long long* __restrict__ table, unsigned long long cap, int* __restrict__ status)
{
    const StreamBlock B = blocks[blockIdx.x];
    const int t = threadIdx.x;
    if (t >= B.count) return;
    const unsigned long long key = ((unsigned long long)(uint32_t)B.halo << 32) | id[B.start + t];
    unsigned long long slot = __umul64hi(mix64(key), cap);
    for (unsigned long long probe = 0; probe < cap; ++probe) {
        const unsigned long long prev = atomicCAS(&table[slot], kEmptySlot, key);
        if (prev == kEmptySlot) return;
        if (prev == key) {
            atomicOr(&status[B.halo], SIDM_DEV_DUPLICATE_ID);
            return;
        }
        slot = slot + 1 == cap ? 0 : slot + 1;
    }
}

// OR of the halos' status words into the context's sticky word, which keeps
// them until the host has read it.
__global__ __launch_bounds__(256) void k_publish_status(const int* __restrict__ status,
                                                         int n_halos, int* __restrict__ sticky)
{
    for (int h = threadIdx.x; h < n_halos; h += 256) {
        const int v = status[h];
        if (v) atomicOr(sticky, v);
    }
}

// The fingerprint (halos, state pointers, scratch generation) of the last call
// made outside stream capture.
__global__ void k_set_fingerprint(unsigned long long* __restrict__ fp_dev,
                                  unsigned long long fp)
{
    if (threadIdx.x == 0) *fp_dev = fp;
}

// First kernel of a captured call: a replay after a call outside capture
// changed the fingerprint is flagged in every halo and in the sticky word.
__global__ __launch_bounds__(256) void k_guard(const unsigned long long* __restrict__ fp_dev,
                                               unsigned long long fp, int* __restrict__ status,
                                               int n_halos, int* __restrict__ sticky)
{
    if (*fp_dev == fp) return;
    for (int h = threadIdx.x; h < n_halos; h += 256) atomicOr(&status[h], SIDM_DEV_STALE_GRAPH);
    if (threadIdx.x == 0) atomicOr(sticky, SIDM_DEV_STALE_GRAPH);
}

// The events of the last scattering pass as sidm_event records (nothing when
// they overflowed the context's buffer; at most cap).
__global__ __launch_bounds__(256) void k_copy_events(const DevCounters* __restrict__ counters,
                                                     const EventRec* __restrict__ ev,
                                                     int64_t max_events, int64_t cap,
                                                     sidm_event* __restrict__ out)
{
    const int64_t total = (int64_t)counters->n_events_total;
    if (total > max_events) return;
    const int64_t n = total < cap ? total : cap;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * 256) {
        sidm_event o;
        o.a = (uint32_t)(ev[e].key >> 32);
        o.b = (uint32_t)ev[e].key;
        o.halo = ev[e].halo;
        o.round = ev[e].round;
        out[e] = o;
    }
}

// The exact decision of a candidate: P = (sigma/m) m_b g Lambda dt with the
// overlap integral, an event iff u < P (and a count of P > 1).  One function
// for both callers, so that a decision never depends on which kernel took it.
__device__ __forceinline__ void decide_pair(const CandRec& r, double dt,
                                         DevCounters* __restrict__ counters,
                                         EventRec* __restrict__ events, int64_t max_events,
                                         unsigned long long* __restrict__ ev_counts)
{
    const double lam = kernel_overlap(r.d, r.ha, r.hb);
    const double P = r.sg * r.mb * r.g * lam * dt;
    if (P > 1.0) atomicAdd(&ev_counts[kEvCounts * r.halo + 3], 1ull);
    if (r.u < P) {
        const unsigned long long slot = atomicAdd(&counters->n_events_total, 1ull);
        if ((int64_t)slot < max_events) {
            EventRec e;
            e.key = ((unsigned long long)r.a << 32) | r.b;
            e.ia = r.ia;
            e.ib = r.ib;
            e.halo = r.halo;
            e.round = 0u;
            events[slot] = e;
        }
    }
}

// The pair test runs on the matrix cores first.  With positions from the
// bucket's centre, d2 - (h_i + h_j)^2 = q_i + q_j - 2 (r_i . r_j + h_i h_j),
// q = r^2 - h^2: a product over 16 terms when every factor is the sum of two
// halves, one 32x32x16 instruction for 1024 pairs.  Lengths are scaled by a
// power of two to at most 1 over the lanes and 64 candidates.  A factor is then
// good to 2^-23 (FP32 difference, two halves), a product without the term of
// two low halves to 2^-21, the four of them doubled to 2^-18, both q to 2^-19
// (at most 4, FP32 from FP32, two halves), and the sum of 16 terms of at most
// 16 in all to 2^-17: less than 2^-16 in total.  Pairs with a value below
// kScreenTol are tested exactly, as they were before; no others can be pairs.
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
constexpr float kScreenTol = 0x1p-15f;
constexpr int kScreen = 32;   // rows (i) and columns (j) of one instruction

// the factors of i (left operand) and j (right operand), halves of 8 terms
__device__ inline void screen_factors(float x, float y, float z, float h, bool left, half8* f)
{
    float q = ((x * x + y * y) + z * z) - h * h;
    if (left) q -= kScreenTol;   // the sign of the sum is the test
    // q as rounded to FP32, for both halves: an FMA that rounds to FP16 at once
    // in the place of one of its uses gives a high half that the low one does
    // not belong to
    asm("" : "+v"(q));
    const _Float16 xh = (_Float16)x, yh = (_Float16)y, zh = (_Float16)z, hh = (_Float16)h;
    const _Float16 xl = (_Float16)(x - (float)xh), yl = (_Float16)(y - (float)yh),
                   zl = (_Float16)(z - (float)zh), hl = (_Float16)(h - (float)hh);
    const _Float16 qh = (_Float16)q, ql = (_Float16)(q - (float)qh), one = (_Float16)1.0f,
                   m2 = (_Float16)-2.0f;
    if (left) {
        f[0] = half8{m2 * xh, m2 * yh, m2 * zh, m2 * hh, m2 * xh, m2 * yh, m2 * zh, m2 * hh};
        f[1] = half8{m2 * xl, m2 * yl, m2 * zl, m2 * hl, qh, ql, one, one};
    } else {
        f[0] = half8{xh, yh, zh, hh, xl, yl, zl, hl};
        f[1] = half8{xh, yh, zh, hh, one, one, qh, ql};
    }
}

// row of accumulator register r, 32 lanes `half`
__device__ inline int screen_row(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }

// bucket lane of a queue entry: register 15 - (bits 0-3), tile of 32 rows (bit
// 4), 32 lanes (bit 5); the rest is the candidate
__device__ inline int screen_entry(int e)
{
    return kScreen * ((e >> 4) & 1) + screen_row(15 - (e & 15), (e >> 5) & 1);
}
constexpr int kPairEach = 2;   // queue entries per lane and round of the per-pair work

// LDS of the pair pass: the candidates (position, kernel size, id, sorted
// index), the factors of 64 of them, and the queue of pairs (place in the
// accumulators, slot of j).  What the per-pair work reads of the bucket's own
// particles, and the velocities of j, come from memory, in flight during its
// Philox rounds; the mass is the halo's common one.
struct PairLds {
    SearchLds S;
    double jx[2 * kBucket], jy[2 * kBucket], jz[2 * kBucket], jh[2 * kBucket];
    uint32_t jid[2 * kBucket], jp[2 * kBucket];
    half8 factor[2][kBucket];
    uint16_t queue[kScreen * kScreen + kPairEach * kBucket];
};

// Cross-section per unit mass at relative speed g: sigma_m, or with a velocity
// scale w > 0 the form of Sec. 3.8 (Eq. vel_dep), sigma_m [1 + (g/w)^2]^-2.
__device__ inline double sigma_at(const HaloDev& H, double g)
{
#pragma clang fp contract(off)
    if (!(H.sigma_w > 0.0)) return H.sigma_m;
    const double t = g / H.sigma_w;
    const double q = 1.0 + t * t;
    return H.sigma_m / (q * q);
}

// INLINE: the pass after an overflow of the candidate buffer.  It runs only
// then (it returns at once otherwise), repeats the search and decides every
// candidate itself; k_decide then decides none, and the counts of pairs and
// candidates are those of the first pass.
template <bool INLINE>
__global__ __launch_bounds__(kBucket) void k_pairs(
    const HaloDev* __restrict__ halos, const BucketInfo* __restrict__ buckets,
    const NodeChild* __restrict__ nodes, const double* __restrict__ box,
    const double* __restrict__ hmax, const SubRange* __restrict__ sub,
    const int* __restrict__ sub_n, int64_t n_buckets,
    const double* __restrict__ sx,
    const double* __restrict__ sy, const double* __restrict__ sz, const double* __restrict__ svx,
    const double* __restrict__ svy, const double* __restrict__ svz, const double* __restrict__ sh,
    const double* __restrict__ cmass, const uint32_t* __restrict__ sid,
    const uint32_t* __restrict__ perm, uint32_t step, DevCounters* __restrict__ counters,
    CandRec* __restrict__ cands, int64_t max_cands, EventRec* __restrict__ events,
    int64_t max_events, unsigned long long* __restrict__ ev_counts, const int* __restrict__ status,
    int split)
{
    __shared__ PairLds L;
    // split waves per bucket: wave `part` takes every split-th candidate
    // bucket of the bucket's visit, the first the pairs inside it too (a call
    // with few buckets still fills the device; every pair is still tested by
    // exactly one wave)
    const int64_t b = blockIdx.x / split;
    const int part = (int)(blockIdx.x % split);
    const int lane = threadIdx.x;
    if (INLINE && (int64_t)counters->n_cands <= max_cands) return;
    const BucketInfo B = buckets[b];
    const HaloDev& H = halos[B.halo];
    if (!(H.sigma_m > 0.0)) return;   // uniform over the block
    // a halo with unequal masses or repeated ids is not scattered (flagged)
    if (status[B.halo] & (SIDM_DEV_UNEQUAL_MASS | SIDM_DEV_DUPLICATE_ID)) return;
    const bool act = lane < B.count;
    const double mb = cmass[B.halo];   // the masses of a halo that scatters are equal
    const int64_t pl = B.start + (act ? lane : 0);
    const double xi = sx[pl], yi = sy[pl], zi = sz[pl], hi = act ? sh[pl] : 0.0;
    const uint32_t idi = sid[pl];
    // the lane's particle from the centre of the bucket's box, in FP32
    const double* bb = box + 6 * b;
    const double ctr[3] = {0.5 * (bb[0] + bb[3]), 0.5 * (bb[1] + bb[4]), 0.5 * (bb[2] + bb[5])};
    const float fx = act ? (float)(xi - ctr[0]) : 0.0f, fy = act ? (float)(yi - ctr[1]) : 0.0f,
                fz = act ? (float)(zi - ctr[2]) : 0.0f, fh = (float)hi;
    // the rows of the accumulators that hold a particle (bit 15 - r)
    uint32_t rows[2] = {0, 0};
    for (int r = 0; r < 16; ++r)
        for (int t = 0; t < 2; ++t)
            if (kScreen * t + screen_row(r, lane >> 5) < B.count) rows[t] |= 1u << (15 - r);
    const uint32_t k0 = (uint32_t)(H.seed & 0xffffffffull), k1 = (uint32_t)(H.seed >> 32);
    const double kInvPi8 = 8.0 / 3.14159265358979323846;
    const double cbound = H.sigma_m * mb * kInvPi8 * H.dt;
    const double cbound2 = cbound * cbound * (1.0 + 1e-12);
    const bool sw = H.sigma_w > 0.0;
    const double inv_w2 = sw ? 1.0 / (H.sigma_w * H.sigma_w) : 0.0;
    const unsigned long long lt = (1ull << lane) - 1ull;
    long long my_cands = 0;
    unsigned long long wave_pairs = 0;   // wave-uniform: the ballots' counts
    int qn = 0;

    // the exact test and the per-pair work for queue entries [from, from + cnt):
    // lane l takes entries l and l + 64, two chains of loads and draws at once.
    // Entries past the last one are the pair of lane 0 and slot 0, not counted.
    auto process = [&](int from, int cnt) __attribute__((always_inline)) {
        __syncthreads();
        int e[kPairEach];
        double u[kPairEach];
        unsigned hit = 0;   // entries below the bound
#pragma unroll
        for (int k = 0; k < kPairEach; ++k)
            e[k] = lane + k * kBucket < cnt ? L.queue[from + lane + k * kBucket] : 15;
#pragma unroll
        for (int k = 0; k < kPairEach; ++k) {
            const int il = screen_entry(e[k]), jl = e[k] >> 6;
            const double ha = __shfl(hi, il, 64), hbb = L.jh[jl];
            const double d2 = dist2_pair(__shfl(xi, il, 64), __shfl(yi, il, 64),
                                         __shfl(zi, il, 64), L.jx[jl], L.jy[jl], L.jz[jl]);
            const double hs = ha + hbb;
            const bool pair = lane + k * kBucket < cnt && d2 < hs * hs;
            wave_pairs += (unsigned long long)__popcll(__ballot(pair));
            const int64_t pi = B.start + il;
            const uint32_t pj = L.jp[jl];
            const double dvx = svx[pi] - svx[pj], dvy = svy[pi] - svy[pj],
                         dvz = svz[pi] - svz[pj];
            // the draw of the pair: smaller id first
            const uint32_t ii = __shfl(idi, il, 64), ij = L.jid[jl];
            const Philox4 w = philox4x32_10(min(ii, ij), max(ii, ij), step, 0u, k0, k1);
            u[k] = unit53(w.w[0], w.w[1]);
            const double g2 = (dvx * dvx + dvy * dvy) + dvz * dvz;
            const double hm = fmax(ha, hbb);

            // Lambda <= min(W_a(0), W_b(0)) = 8 / (pi max(h)^3) bounds P by
            // sigma(g) m g 8 / (pi max(h)^3) dt.  The test u < bound, with
            // sigma(g) = sigma_m / q^2, reads u max(h)^3 q^2 < cbound g;
            // both sides are non-negative, so it is taken squared (no square
            // root, no division), with a relative slack of 1e-12 so that the
            // candidates include every pair whose rounded P exceeds u.
            double lhs = u[k] * (hm * hm * hm);
            if (sw) {
                const double q = 1.0 + g2 * inv_w2;
                lhs *= q * q;
            }
            hit |= (unsigned)(pair && lhs * lhs < cbound2 * g2) << k;
        }
        while (hit) {
            // the exact decision needs Lambda: k_decide takes it from here
            // (after an overflow of its buffer, the INLINE pass)
            const int k = __ffs(hit) - 1;
            hit &= hit - 1;
            ++my_cands;
            const int ek = k == 0 ? e[0] : e[1];
            const int jl = ek >> 6;
            const int64_t pi = B.start + screen_entry(ek);
            const uint32_t pj = L.jp[jl], ii = sid[pi], ij = L.jid[jl];
            const bool iswap = ii > ij;   // canonical order of the pair: a = smaller id
            const double ha = sh[pi], hbb = L.jh[jl];
            const double g =
                norm3(svx[pi] - svx[pj], svy[pi] - svy[pj], svz[pi] - svz[pj]);
            CandRec r;
            r.sg = sigma_at(H, g);
            r.mb = mb;
            r.g = g;
            r.d = sqrt(dist2_pair(sx[pi], sy[pi], sz[pi], L.jx[jl], L.jy[jl], L.jz[jl]));
            r.ha = iswap ? hbb : ha;
            r.hb = iswap ? ha : hbb;
            r.u = k == 0 ? u[0] : u[1];
            r.a = iswap ? ij : ii;
            r.b = iswap ? ii : ij;
            const uint32_t oi = perm[pi], oj = perm[pj];
            r.ia = iswap ? oj : oi;
            r.ib = iswap ? oi : oj;
            r.halo = B.halo;
            r.pad = 0;
            if (INLINE) {
                decide_pair(r, H.dt, counters, events, max_events, ev_counts);
            } else {
                const unsigned long long slot = atomicAdd(&counters->n_cands, 1ull);
                if ((int64_t)slot < max_cands) cands[slot] = r;
            }
        }
        __syncthreads();
    };

    // the bucket against the first n candidates in LDS (same: its own
    // particles, a pair taken by the earlier one), and the per-pair work of
    // what passes, whose entries refer to these candidates
    auto test = [&](int n, bool same) __attribute__((always_inline)) {
        half8 fi[2];
        bool wide = false;
        const int steps = 2 * ((n + kScreen - 1) / kScreen);
        __syncthreads();
        for (int u = 0; u < steps; ++u) {
            const int j0 = kScreen * (u >> 1), jc = j0 + (lane & (kScreen - 1));
            if ((u & 3) == 0) {   // the factors for the next 64 candidates
                const int j = j0 + lane;
                const bool in = j < n;
                const float gx = in ? (float)(L.jx[j] - ctr[0]) : 0.0f,
                            gy = in ? (float)(L.jy[j] - ctr[1]) : 0.0f,
                            gz = in ? (float)(L.jz[j] - ctr[2]) : 0.0f,
                            gh = in ? (float)L.jh[j] : 0.0f;
                float m = fmaxf(fmaxf(fabsf(fx), fabsf(fy)), fmaxf(fabsf(fz), fabsf(fh)));
                m = fmaxf(m, fmaxf(fmaxf(fabsf(gx), fabsf(gy)), fmaxf(fabsf(gz), fabsf(gh))));
                m = lanes_max(m);
                // lengths that FP32 does not hold: every pair is tested exactly
                const float sum = ((fx + fy) + (fz + fh)) + ((gx + gy) + (gz + gh));
                wide = !(m > 0x1p-100f && m < 0x1p100f) || __any(!(fabsf(sum) < INFINITY));
                const float s = ldexpf(1.0f, -__builtin_amdgcn_frexp_expf(m));
                half8 f[2];
                screen_factors(fx * s, fy * s, fz * s, fh * s, true, f);
                L.factor[0][lane] = f[0];
                L.factor[1][lane] = f[1];
                __syncthreads();
                fi[0] = L.factor[lane >> 5][lane & (kScreen - 1)];
                fi[1] = L.factor[lane >> 5][kScreen + (lane & (kScreen - 1))];
                __syncthreads();
                screen_factors(gx * s, gy * s, gz * s, gh * s, false, f);
                L.factor[0][lane] = f[0];
                L.factor[1][lane] = f[1];
                __syncthreads();
            }
            const half8 fj = L.factor[lane >> 5][jc & (kBucket - 1)];
            const float16v acc = __builtin_amdgcn_mfma_f32_32x32x16_f16((u & 1) ? fi[1] : fi[0], fj,
                                                                        float16v{}, 0, 0, 0);
            uint32_t m = 0;   // the lane's pairs: signs, register r in bit 15 - r
#pragma unroll
            for (int r = 0; r < 16; ++r)
                m = __builtin_amdgcn_alignbit(m, __float_as_uint(acc[r]), 31);
            if (wide) m = 0xffffu;
            m &= jc < n ? ((u & 1) ? rows[1] : rows[0]) : 0u;
            if (same)
                for (int r = 0; r < 16; ++r)
                    if (kScreen * (u & 1) + screen_row(r, lane >> 5) >= jc) m &= ~(1u << (15 - r));
            const int cnt = __popc(m), upto = lanes_scan(cnt);
            int at = qn + upto - cnt;
            const uint32_t tag = (uint32_t)((u & 1) << 4 | (lane >> 5) << 5 | jc << 6);
            while (m) {
                L.queue[at++] = (uint16_t)(tag | (31 - __clz(m)));
                m &= ~(1u << (31 - __clz(m)));
            }
            qn += __builtin_amdgcn_readlane(upto, 63);
            const int rest = u + 1 < steps ? kPairEach * kBucket - 1 : 0;   // may stay queued
            while (qn > rest) {
                const int c = min(qn, kPairEach * kBucket);
                qn -= c;
                process(qn, c);
            }
        }
        __syncthreads();
    };

    // the first candidates are the bucket's own particles
    bool own = part == 0;
    int jn = own ? B.count : 0;   // candidates in LDS
    if (own) {
        L.jx[lane] = xi;
        L.jy[lane] = yi;
        L.jz[lane] = zi;
        L.jh[lane] = hi;
        L.jid[lane] = idi;
        L.jp[lane] = (uint32_t)pl;
    }
    // A node can hold a partner of lane i only if its box is closer than h_i +
    // max h over it; the later buckets' pairs with this one are taken here.
    const int nq = search_groups(L.S, lane, lane_sub(sub + kSubMax * b, sub_n[b], lane), act, xi,
                                 yi, zi, hi);
    unsigned seen = 0;   // buckets of the walk so far
    auto drain = [&](int ln, bool last) __attribute__((always_inline)) {
        // this part's buckets, and of them those that some lane reaches
        const unsigned first = (unsigned)(part + split - (int)(seen % split)) % split;
        seen += ln;
        int kept = 0;
        for (int i = first; i < ln; i += 4 * split) {
            uint32_t c[4];
            unsigned long long m[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                c[u] = __builtin_amdgcn_readfirstlane(L.S.list[min(i + u * split, ln - 1)]);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double r = hi + hmax[c[u]];
                m[u] = __ballot(act && point_box_dist2(xi, yi, zi, box + 6 * (int64_t)c[u]) <
                                           r * r * (1.0 + 1e-9));
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (m[u] && i + u * split < ln) {
                    if (lane == 0) L.S.list[kept] = c[u];
                    ++kept;
                }
        }
        __syncthreads();
        if (kept == 0 && !last) return;
        // the next bucket's particles are in flight while one is tested
        int cnt;
        int64_t p0 = kept > 0
                         ? bucket_start(H, __builtin_amdgcn_readfirstlane(L.S.list[0]), cnt)
                         : (cnt = 0, B.start);
        bool on = lane < cnt;
        int64_t p = p0 + (on ? lane : 0);
        double x = sx[p], y = sy[p], z = sz[p], h = sh[p];
        uint32_t idj = sid[p];
        for (int i = 0; i <= kept; ++i) {
            if (jn >= kBucket || (jn > 0 && (own || (last && i == kept)))) {
                test(jn, own);
                jn = 0;
                own = false;
            }
            if (i == kept) break;
            const double cx = x, cy = y, cz = z, ch = h;
            const uint32_t cid = idj, cp = (uint32_t)p;
            const bool con = on;
            if (i + 1 < kept) {
                p0 = bucket_start(H, __builtin_amdgcn_readfirstlane(L.S.list[i + 1]), cnt);
                on = lane < cnt;
                p = p0 + (on ? lane : 0);
                x = sx[p]; y = sy[p]; z = sz[p]; h = sh[p];
                idj = sid[p];
            }
            bool keep = false;
            for (int q = 0; q < nq; ++q) {
                const double r = L.S.group[q][6] + ch;
                keep |= group_point_dist2(L.S.group[q], cx, cy, cz) < r * r * (1.0 + 1e-9);
            }
            const unsigned long long m = __ballot(con && keep);
            if (con && keep) {
                const int at = jn + __popcll(m & lt);
                L.jx[at] = cx;
                L.jy[at] = cy;
                L.jz[at] = cz;
                L.jh[at] = ch;
                L.jid[at] = cid;
                L.jp[at] = cp;
            }
            jn += __popcll(m);
        }
    };
    search_walk(H, nodes, n_buckets, L.S,
                [&](int64_t c) {
                    if (nodes[c].last <= b) return false;
                    const double hc = hmax[c];
                    bool in = false;
                    for (int q = 0; q < nq; ++q) {
                        const double r = L.S.group[q][6] + hc;
                        in |= group_box_dist2(L.S.group[q], box + 6 * c) < r * r * (1.0 + 1e-9);
                    }
                    return in;
                },
                [&](int ln, bool last) __attribute__((always_inline)) {
                    // a halo of one bucket has no other pairs than its own
                    drain(H.n_levels > 1 ? ln : 0, last);
                });
    // pairs tested and candidates of the exact decision found by this bucket
    if (INLINE) return;
    long long vc = my_cands;
    for (int o = 32; o > 0; o >>= 1) vc += __shfl_xor(vc, o, 64);
    if (lane == 0 && wave_pairs > 0) atomicAdd(&ev_counts[kEvCounts * B.halo + 2], wave_pairs);
    if (lane == 0 && vc > 0) atomicAdd(&ev_counts[kEvCounts * B.halo + 4], (unsigned long long)vc);
}

// The exact decisions of the candidates the pair pass stored; none after an
// overflow of their buffer (the INLINE pair pass decides them all).
__global__ __launch_bounds__(256) void k_decide(const HaloDev* __restrict__ halos,
                                                const CandRec* __restrict__ cands,
                                                int64_t max_cands,
                                                DevCounters* __restrict__ counters,
                                                EventRec* __restrict__ events, int64_t max_events,
                                                unsigned long long* __restrict__ ev_counts)
{
    const int64_t total = (int64_t)counters->n_cands;
    if (total > max_cands) return;
    for (int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x; c < total;
         c += (int64_t)gridDim.x * 256) {
        const CandRec r = cands[c];
        decide_pair(r, halos[r.halo].dt, counters, events, max_events, ev_counts);
    }
}

// Elastic isotropic scattering in the centre-of-mass frame: the relative speed
// is kept and its direction redrawn uniformly on the sphere from the draw at
// counter (a, b, step, 1).
__device__ inline void kick_pair(uint64_t seed, uint32_t step, uint32_t a, uint32_t b, double ma,
                                 double mb, double* va, double* vb)
{
#pragma clang fp contract(off)
    const Philox4 w = philox4x32_10(a, b, step, 1u, (uint32_t)(seed & 0xffffffffull),
                                    (uint32_t)(seed >> 32));
    const double uc = unit53(w.w[0], w.w[1]);
    const double uphi = unit53(w.w[2], w.w[3]);
    const double M = ma + mb;
    const double dvx = va[0] - vb[0], dvy = va[1] - vb[1], dvz = va[2] - vb[2];
    const double g = sqrt((dvx * dvx + dvy * dvy) + dvz * dvz);
    const double cth = 1.0 - 2.0 * uc;
    const double s2 = 1.0 - cth * cth;
    const double sth = sqrt(s2 > 0.0 ? s2 : 0.0);
    const double ph = 2.0 * 3.14159265358979323846 * uphi;
    double sp, cp;
    sincos(ph, &sp, &cp);
    const double n[3] = {sth * cp, sth * sp, cth};
    const double fa = mb / M * g, fb = ma / M * g;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double vcm = (ma * va[c] + mb * vb[c]) / M;
        va[c] = vcm + fa * n[c];
        vb[c] = vcm - fb * n[c];
    }
}

__device__ inline unsigned long long owner_load(unsigned long long* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline void owner_free(unsigned long long* p)
{
    __hip_atomic_store(p, ~0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kRoundThreads = 1024;
// Halos are independent: workgroup g of kRoundGroups takes the events of the
// halos h with h % groups == g, listed (as event indices) in its own segment
// of max_events words of the candidate buffer, which holds nothing once the
// pair decisions are taken.
constexpr int kRoundGroups = 64;
static_assert(4 * sizeof(CandRec) >= kRoundGroups * sizeof(uint32_t),
              "the candidate buffer holds every workgroup's event list");

// Each workgroup applies the events of its halos; all of its waves leave the
// loop in the same round (the pending count is reduced through LDS).
__global__ __launch_bounds__(kRoundThreads) void k_rounds(
    const HaloDev* __restrict__ halos, int n_halos, const DevCounters* __restrict__ counters,
    EventRec* __restrict__ ev, int64_t max_events, unsigned long long* __restrict__ owner,
    double* __restrict__ vx, double* __restrict__ vy, double* __restrict__ vz,
    const double* __restrict__ m, unsigned long long* __restrict__ ev_counts,
    int* __restrict__ status, uint32_t step, int64_t out_cap, sidm_event* __restrict__ out,
    uint32_t* __restrict__ lists)
{
    __shared__ int pending, n_mine;
    const int t = threadIdx.x;
    const int groups = (int)gridDim.x, g = (int)blockIdx.x;
    const unsigned long long total = counters->n_events_total;
    if ((int64_t)total > max_events) {
        for (int h = g + groups * t; h < n_halos; h += groups * kRoundThreads)
            atomicOr(&status[h], SIDM_DEV_EVENT_OVERFLOW);
        return;
    }
    const int64_t n_all = (int64_t)total;
    uint32_t* __restrict__ mine_e = lists + (int64_t)g * max_events;
    if (t == 0) n_mine = 0;
    __syncthreads();
    for (int64_t e = t; e < n_all; e += kRoundThreads)
        if (ev[e].halo % groups == g) mine_e[atomicAdd(&n_mine, 1)] = (uint32_t)e;
    __syncthreads();
    const int64_t n = n_mine;
    for (int64_t q = t; q < n; q += kRoundThreads) {
        const int64_t e = mine_e[q];
        ev[e].round = 0u;
        owner_free(&owner[ev[e].ia]);
        owner_free(&owner[ev[e].ib]);
    }
    __syncthreads();
    for (uint32_t r = 1; n > 0; ++r) {
        for (int64_t q = t; q < n; q += kRoundThreads) {
            const int64_t e = mine_e[q];
            if (ev[e].round == 0u) {
                atomicMin(&owner[ev[e].ia], ev[e].key);
                atomicMin(&owner[ev[e].ib], ev[e].key);
            }
        }
        __syncthreads();
        for (int64_t q = t; q < n; q += kRoundThreads) {
            const int64_t e = mine_e[q];
            if (ev[e].round == 0u) {
                const unsigned long long key = ev[e].key;
                if (owner_load(&owner[ev[e].ia]) == key && owner_load(&owner[ev[e].ib]) == key)
                    ev[e].round = r;
            }
        }
        __syncthreads();
        if (t == 0) pending = 0;
        for (int64_t q = t; q < n; q += kRoundThreads) {
            const int64_t e = mine_e[q];
            const uint32_t er = ev[e].round;
            if (er == 0u || er == r) {
                owner_free(&owner[ev[e].ia]);
                owner_free(&owner[ev[e].ib]);
            }
        }
        __syncthreads();
        int mine = 0;
        for (int64_t q = t; q < n; q += kRoundThreads) {
            const int64_t e = mine_e[q];
            const EventRec E = ev[e];
            if (E.round == r) {
                const HaloDev& H = halos[E.halo];
                double va[3] = {vx[E.ia], vy[E.ia], vz[E.ia]};
                double vb[3] = {vx[E.ib], vy[E.ib], vz[E.ib]};
                kick_pair(H.seed, step, (uint32_t)(E.key >> 32), (uint32_t)E.key, m[E.ia], m[E.ib],
                          va, vb);
                vx[E.ia] = va[0]; vy[E.ia] = va[1]; vz[E.ia] = va[2];
                vx[E.ib] = vb[0]; vy[E.ib] = vb[1]; vz[E.ib] = vb[2];
                atomicAdd(&ev_counts[kEvCounts * E.halo + 0], 1ull);
                atomicMax(&ev_counts[kEvCounts * E.halo + 1], (unsigned long long)r);
            } else if (E.round == 0u) {
                ++mine;
            }
        }
        if (mine) atomicAdd(&pending, mine);
        __syncthreads();
        const int left = pending;
        __syncthreads();
        if (left == 0) break;
    }
    if (out) {
        for (int64_t q = t; q < n; q += kRoundThreads) {
            const int64_t e = mine_e[q];
            if (e >= out_cap) continue;
            sidm_event o;
            o.a = (uint32_t)(ev[e].key >> 32);
            o.b = (uint32_t)ev[e].key;
            o.halo = ev[e].halo;
            o.round = ev[e].round;
            out[e] = o;
        }
    }
}

hipError_t launch_reset(const Plan& P, Scratch& w, hipStream_t st)
{
    const int nt = kEvCounts * P.n_halos + 1;
    hipLaunchKernelGGL(k_scatter_reset, dim3((nt + 255) / 256), dim3(256), 0, st, w.counters,
                       (unsigned long long*)w.ev_counts, w.status, P.n_halos);
    return hipGetLastError();
}

// The scattering pass's check that ids are unique within each halo (it reuses
// the cell list's sort buffers, which hold nothing the later passes read; that
// a halo that scatters has one common mass is checked with the cell list).
hipError_t launch_id_check(const Plan& P, const sidm_state* s, Scratch& w, hipStream_t st)
{
    if (!P.any_scatter) return hipSuccess;
    // the hash table: the radix sort's two key buffers, 2 max_particles words
    const unsigned long long cap = 2ull * (unsigned long long)w.max_particles;
    if ((int64_t)cap < 2 * P.n_sorted) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_fill_u64, dim3(1024), dim3(256), 0, st, w.keys[0], (int64_t)cap,
                       kEmptySlot);
    hipLaunchKernelGGL(k_id_insert, dim3((unsigned)P.n_blocks), dim3(kStreamBlock), 0, st,
                       w.blocks, s->id, w.keys[0], cap, w.status);
    return hipGetLastError();
}

hipError_t launch_publish_status(const Plan& P, Scratch& w, hipStream_t st)
{
    hipLaunchKernelGGL(k_publish_status, dim3(1), dim3(256), 0, st, w.status, P.n_halos, w.sticky);
    return hipGetLastError();
}

hipError_t launch_fingerprint(const Plan& P, Scratch& w, unsigned long long fp, bool captured,
                              hipStream_t st)
{
    if (captured)
        hipLaunchKernelGGL(k_guard, dim3(1), dim3(256), 0, st, w.fp_dev, fp, w.status, P.n_halos,
                           w.sticky);
    else
        hipLaunchKernelGGL(k_set_fingerprint, dim3(1), dim3(64), 0, st, w.fp_dev, fp);
    return hipGetLastError();
}

__global__ void k_clear_word(int* __restrict__ w)
{
    if (threadIdx.x == 0) *w = 0;
}

hipError_t launch_clear_sticky(Scratch& w, hipStream_t st)
{
    hipLaunchKernelGGL(k_clear_word, dim3(1), dim3(64), 0, st, w.sticky);
    return hipGetLastError();
}

hipError_t launch_copy_events(Scratch& w, sidm_event* out, int64_t cap, hipStream_t st)
{
    hipLaunchKernelGGL(k_copy_events, dim3(64), dim3(256), 0, st, w.counters, w.events,
                       w.max_events, cap, out);
    return hipGetLastError();
}

hipError_t launch_scatter(const Plan& P, const sidm_state* s, Scratch& w, uint32_t step,
                          sidm_event* out_events, int64_t out_cap, hipStream_t st,
                          hipEvent_t after_pairs)
{
    hipError_t e = launch_id_check(P, s, w, st);
    if (e != hipSuccess) return e;
    const int split = search_split(P.n_buckets, kPairSplitMax);
    auto pairs = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)(P.n_buckets * split)), dim3(kBucket), 0, st, w.halos,
                           w.buckets, w.nodes, w.box, w.hmax, w.sub, w.sub_n, P.n_buckets, w.sx,
                           w.sy, w.sz, w.svx, w.svy, w.svz, w.sh, w.cref, w.sid, w.perm, step,
                           w.counters, w.cands, w.max_cands, w.events, w.max_events,
                           (unsigned long long*)w.ev_counts, w.status, split);
    };
    pairs(k_pairs<false>);
    hipLaunchKernelGGL(k_decide, dim3(256), dim3(256), 0, st, w.halos, w.cands, w.max_cands,
                       w.counters, w.events, w.max_events, (unsigned long long*)w.ev_counts);
    pairs(k_pairs<true>);
    if (after_pairs) (void)hipEventRecord(after_pairs, st);
    const int groups = P.n_halos < kRoundGroups ? P.n_halos : kRoundGroups;
    hipLaunchKernelGGL(k_rounds, dim3((unsigned)groups), dim3(kRoundThreads), 0, st, w.halos,
                       P.n_halos, w.counters, w.events, w.max_events, w.owner, s->vx, s->vy,
                       s->vz, s->m, (unsigned long long*)w.ev_counts, w.status, step, out_cap,
                       out_events, (uint32_t*)w.cands);
    return hipGetLastError();
}

}  // namespace sidm
