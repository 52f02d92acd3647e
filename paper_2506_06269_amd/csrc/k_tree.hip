// k_tree.hip -- cell list for the neighbour and pair searches: particles of
// each halo are ordered along a Morton curve (48-bit keys over the halo's
// bounding box, halo rank in the high bits) by a stable LSD radix sort, cut
// into buckets of kBucket consecutive particles, and the bucket bounding boxes
// are merged kFanout at a time into a search tree per halo.
//
// A launch that only waits for the previous one costs 3 to 5 us, whatever it
// does, so up to a few 10^5 particles the list is bound by its number of
// launches: calls whose halos all have at most kSmallN particles sort each
// halo in one workgroup's LDS (k_cell_small), larger ones take one launch per
// radix digit (k_sort_pass).
#include "sidm_plan.hpp"
#include "sidm_steps.hpp"
#include "sidm_wave.hpp"

namespace sidm {

// ---------------------------------------------------------------- bounding boxes
// Box and mass range of a workgroup's particles: per-thread extrema e (min x,
// y, z, m, max x, y, z, m, and whether any value is not finite; with C = kRange
// also the sum of the masses' magnitudes) reduced over NW waves; every thread
// returns the result.  red: C * NW words of LDS.
template <int NW, int C>
__device__ inline void block_range(double (&e)[C], double* red)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        e[c] = c < 4          ? rows_min(row_min(e[c]))
               : c < kExtrema ? rows_max(row_max(e[c]))
                              : rows_sum(row_sum(e[c]));
        if (lane == 0) red[c * NW + wv] = e[c];
    }
    __syncthreads();
    static_assert(16 % NW == 0, "the waves' results repeat in a row of lanes");
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const double v = red[c * NW + lane % NW];
        e[c] = c < 4 ? row_min(v) : c < kExtrema ? row_max(v) : row_sum(v) * (NW / 16.0);
    }
}

// The common mass of a halo (cmass[h], 0 when its masses differ), the largest
// magnitude of its masses (cmass[n_halos + h]), and whether the FP64 symmetric
// tiles can sum it (cmass[2 n_halos + h]): their fixed-point totals need finite
// values and scales, and hold a sum to 2^-104 of its bound n m 0.385 / eps^2
// with m the largest magnitude.  The least force scale of a box of side R is
// M / R^2, M the sum of the magnitudes; the unit is below 2^-63 of it for
// (n m / M) (R / eps)^2 up to 2^40 (equal masses: R up to 2^20 eps; workloads:
// 10^3 to 10^4).  sum: M, or 0 for a halo too small for those tiles.  With a
// status array, a halo that scatters (sigma_m > 0) without a common mass is
// flagged: the probability of a pair takes the mass of one member, which is
// only symmetric when the masses are equal (each run of the paper's Table 1 has
// one particle mass), so such a halo is not scattered.
__device__ inline void put_mass(const HaloDev& H, int h, int n_halos, const double* e, double sum,
                                double* __restrict__ cmass, int* __restrict__ status)
{
    const double lo = e[3], hi = e[7], top = fmax(fabs(lo), fabs(hi));
    const bool equal = lo == hi;
    cmass[h] = equal ? lo : 0.0;
    cmass[n_halos + h] = top;
    const double side = fmax(fmax(e[4] - e[0], e[5] - e[1]), e[6] - e[2]) / H.eps;
    const double mref = equal && lo > 0.0 ? 1.0 : top;
    const double ratio = equal ? 1.0 : (double)H.n * top / sum;
    cmass[2 * n_halos + h] = e[8] == 0.0 && sum > 0.0 && ratio * (side * side) <= 0x1p40 &&
                                     H.eps2 > 0x1p-400 && H.eps2 < 0x1p400 &&
                                     mref > 0x1p-400 && mref < 0x1p400
                                 ? 1.0
                                 : 0.0;
    if (status && !equal && H.sigma_m > 0.0) atomicOr(&status[h], SIDM_DEV_UNEQUAL_MASS);
}

// Per streaming block: its range.  The launch also clears the work space of
// the sort that follows (n_zero words).
__global__ __launch_bounds__(kStreamBlock) void k_block_range(
    const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    const double* __restrict__ m, const StreamBlock* __restrict__ blocks,
    double* __restrict__ brange, uint32_t* __restrict__ zero, int64_t n_zero,
    const int* __restrict__ active, int tick)
{
    if (tick_idle(active, tick)) return;
    __shared__ double red[kRange * (kStreamBlock / 64)];
    const StreamBlock B = blocks[blockIdx.x];
    const int t = threadIdx.x;
    for (int64_t i = (int64_t)blockIdx.x * kStreamBlock + t; i < n_zero;
         i += (int64_t)gridDim.x * kStreamBlock)
        zero[i] = 0u;
    const int64_t i = B.start + (t < B.count ? t : 0);
    const double px = x[i], py = y[i], pz = z[i], mi = m[i];
    const double nf = (px - px) + (py - py) + (pz - pz) + (mi - mi) == 0.0 ? 0.0 : 1.0;
    double e[kRange] = {px, py, pz, mi, px, py, pz, mi, nf, t < B.count ? fabs(mi) : 0.0};
    block_range<kStreamBlock / 64>(e, red);
    if (t == 0)
        for (int c = 0; c < kRange; ++c) brange[kRange * (int64_t)blockIdx.x + c] = e[c];
}

// Per halo, from halo h0 on: its box and masses.
constexpr int kRangeThreads = 1024;
__global__ __launch_bounds__(kRangeThreads) void k_halo_range(
    const HaloDev* __restrict__ halos, int h0, int n_halos, const double* __restrict__ brange,
    double* __restrict__ bbox, double* __restrict__ cmass, int* __restrict__ status,
    const int* __restrict__ active, int tick)
{
    if (tick_idle(active, tick)) return;
    __shared__ double red[kRange * (kRangeThreads / 64)];
    const int h = h0 + (int)blockIdx.x, t = threadIdx.x;
    const HaloDev& H = halos[h];
    const int64_t nb = (H.n + kStreamBlock - 1) / kStreamBlock;
    double e[kRange] = {INFINITY,  INFINITY,  INFINITY,  INFINITY, -INFINITY,
                        -INFINITY, -INFINITY, -INFINITY, 0.0,      0.0};
    for (int64_t b = t; b < nb; b += kRangeThreads)
        for (int c = 0; c < kRange; ++c) {
            const double v = brange[kRange * (H.stream_block0 + b) + c];
            e[c] = c < 4 ? fmin(e[c], v) : c < kExtrema ? fmax(e[c], v) : e[c] + v;
        }
    block_range<kRangeThreads / 64>(e, red);
    if (t == 0) {
        for (int c = 0; c < 3; ++c) {
            bbox[6 * (int64_t)h + c] = e[c];
            bbox[6 * (int64_t)h + 3 + c] = e[4 + c];
        }
        put_mass(H, h, n_halos, e, e[kExtrema], cmass, status);
    }
}

// ---------------------------------------------------------------- Morton keys
__device__ inline unsigned long long spread3(unsigned v)   // bit k -> bit 3k
{
    unsigned long long x = v & 0xFFFFull;
    x = (x | (x << 32)) & 0x001F00000000FFFFull;
    x = (x | (x << 16)) & 0x001F0000FF0000FFull;
    x = (x | (x << 8)) & 0x100F00F00F00F00Full;
    x = (x | (x << 4)) & 0x10C30C30C30C30C3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

__device__ inline unsigned quant16(double v, double lo, double inv)
{
    double q = (v - lo) * inv;
    q = fmin(fmax(q, 0.0), 65535.0);
    return (unsigned)q;
}

// Sort key of particle i (without the halo's rank): the Morton code over the
// halo's box (lo, and 65535 / its largest side).  In a tick of block steps the
// inactive particles of a direct-sum halo sort after its active ones (bit 48),
// so the active ones fill whole i-blocks.
__device__ inline unsigned long long morton_key(const HaloDev& H, double px, double py, double pz,
                                                const double* lo, double inv,
                                                const int8_t* __restrict__ bin, int64_t i,
                                                int tick, int bmax, int rank_shift)
{
    unsigned long long key = spread3(quant16(px, lo[0], inv)) |
                             (spread3(quant16(py, lo[1], inv)) << 1) |
                             (spread3(quant16(pz, lo[2], inv)) << 2);
    if (rank_shift > 48 && tick > 0 && !(H.tree_alpha > 0.0) &&
        !bin_active(H, bin[i], local_tick(H, tick, bmax)))
        key |= 1ull << 48;
    return key;
}

__device__ inline double key_scale(const double* lo, const double* hi)
{
    const double ext = fmax(fmax(hi[0] - lo[0], hi[1] - lo[1]), hi[2] - lo[2]);
    return ext > 0.0 ? 65535.0 / ext : 0.0;
}

// ---------------------------------------------------------------- radix sort
constexpr int kDigits = 1 << kSortBits;
constexpr int kSortWaves = kSortBlock / 64;

// Keys and indices of `group` streaming blocks per workgroup, and the number
// of keys with each value of each digit (hist: kDigits words per pass).
__global__ __launch_bounds__(kStreamBlock) void k_morton_keys(
    const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    const StreamBlock* __restrict__ blocks, int64_t n_blocks, int group,
    const HaloDev* __restrict__ halos, const double* __restrict__ bbox,
    unsigned long long* __restrict__ keys, uint32_t* __restrict__ vals,
    const int8_t* __restrict__ bin, int tick, int bmax, int rank_shift, int passes,
    uint32_t* __restrict__ hist, const int* __restrict__ active)
{
    if (tick_idle(active, tick)) return;
    __shared__ uint32_t cnt[kSortMaxPasses][kDigits];
    const int t = threadIdx.x;
    for (int p = 0; p < passes; ++p) cnt[p][t] = 0u;
    __syncthreads();
    const int64_t b0 = (int64_t)blockIdx.x * group;
    const int64_t b1 = b0 + group < n_blocks ? b0 + group : n_blocks;
    for (int64_t b = b0; b < b1; ++b) {
        const StreamBlock B = blocks[b];
        if (t >= B.count) continue;
        const HaloDev& H = halos[B.halo];
        const int64_t i = B.start + t;
        const double* bb = bbox + 6 * B.halo;
        const unsigned long long key =
            ((unsigned long long)H.rank << rank_shift) |
            morton_key(H, x[i], y[i], z[i], bb, key_scale(bb, bb + 3), bin, i, tick, bmax,
                       rank_shift);
        const int64_t pos = H.sbase + (i - H.offset);
        keys[pos] = key;
        vals[pos] = (uint32_t)i;
        for (int p = 0; p < passes; ++p)
            atomicAdd(&cnt[p][(key >> (kSortBits * p)) & (kDigits - 1)], 1u);
    }
    __syncthreads();
    for (int p = 0; p < passes; ++p)
        if (cnt[p][t]) atomicAdd(&hist[p * kDigits + t], cnt[p][t]);
}

// Lanes of the wave whose digit equals this lane's.
__device__ inline unsigned long long match_digit(uint32_t d)
{
    unsigned long long peers = ~0ull;
#pragma unroll
    for (int bit = 0; bit < kSortBits; ++bit) {
        const bool set = (d >> bit) & 1u;
        const unsigned long long m = __ballot(set);
        peers &= set ? m : ~m;
    }
    return peers;
}

// Ranks of a wave's items among its earlier ones with the same digit: item r
// of lane l is the wave's (64 r + l)-th.  cnt: the wave's count per digit
// (zero on entry, its totals on return).
template <int IPT, class K>
__device__ inline void wave_rank(const K (&key)[IPT], int shift, uint32_t* cnt, uint32_t (&rank)[IPT],
                                 uint32_t (&dig)[IPT])
{
    const unsigned long long below = (1ull << (threadIdx.x & 63)) - 1ull;
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const uint32_t d = (uint32_t)(key[r] >> shift) & (kDigits - 1);
        const unsigned long long peers = match_digit(d);
        const uint32_t before = cnt[d];
        const uint32_t in = (uint32_t)__popcll(peers & below);
        // the wave's lanes run together: every lane has read the count before
        // the last of its peers moves it on
        __builtin_amdgcn_wave_barrier();
        if ((peers & ~below) >> (threadIdx.x & 63) == 1ull)
            cnt[d] = before + in + 1u;
        __builtin_amdgcn_wave_barrier();
        rank[r] = before + in;
        dig[r] = d;
    }
}

// Exclusive prefix over kDigits values, value d on thread d < kDigits of the
// block (others pass 0 and ignore the result); every thread of the block must
// call it.  sw: kDigits / 64 words of LDS.
__device__ inline uint32_t digit_scan(uint32_t v, uint32_t* sw)
{
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    uint32_t inc = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(inc, o, 64);
        if (lane >= o) inc += u;
    }
    if (t < kDigits && lane == 63) sw[wv] = inc;
    __syncthreads();
    uint32_t off = 0;
    for (int w = 0; w < kDigits / 64; ++w)
        if (w < wv) off += sw[w];
    return off + inc - v;
}

// One digit of the stable LSD sort in one launch.  Workgroups take tiles of
// kSortBlock * IPT keys in the order of a ticket, so a tile's predecessors are
// held by workgroups that run or have run; each publishes its count of every
// digit in one word (state in the top two bits, so a word is either whole or
// absent), then adds up its predecessors' words, newest first, back to the
// first one that already holds a running total (Merrill and Garland's
// decoupled look-back).  A workgroup waits only for lower tickets, which never
// wait for higher ones, so every wait ends.
//
// Bound by latency, not by the 24 bytes per key that it moves: 8.4 us per
// digit at 65536 keys, 15.7 at 500009, 22.7 at 2^20, 45 at 2.4 million.  The
// five launches it replaced (tile counts, three for their scan, a scatter that
// took a tile's keys 256 at a time between barriers) took 37, 39, 41 and 68.
constexpr uint32_t kTileSum = 1u << 30, kTileTotal = 2u << 30, kTileValue = kTileSum - 1u;
constexpr int kLookBack = 8;   // words read at once

template <int IPT>
__global__ __launch_bounds__(kSortBlock) void k_sort_pass(
    const unsigned long long* __restrict__ kin, const uint32_t* __restrict__ vin,
    unsigned long long* __restrict__ kout, uint32_t* __restrict__ vout, int64_t n, int shift,
    const uint32_t* __restrict__ hist, uint32_t* __restrict__ ticket, uint32_t* __restrict__ tiles,
    const int* __restrict__ active, int tick)
{
    if (tick_idle(active, tick)) return;
    __shared__ uint32_t cnt[kSortWaves][kDigits];
    __shared__ uint32_t sw[kDigits / 64];
    __shared__ uint32_t tile_s;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    if (t == 0) tile_s = atomicAdd(ticket, 1u);
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) cnt[q][t] = 0u;
    const uint32_t first = digit_scan(hist[t], sw);   // keys with a smaller digit
    const int64_t tile = tile_s;
    const int64_t base = tile * (kSortBlock * IPT) + wv * (64 * IPT) + lane;
    unsigned long long key[IPT];
    uint32_t val[IPT], rank[IPT], dig[IPT];
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const int64_t i = base + 64 * r;
        // past the end: the last keys of the last tile, digit kDigits - 1 in
        // every pass, behind every real key
        key[r] = i < n ? kin[i] : ~0ull;
        val[r] = i < n ? vin[i] : 0u;
    }
    wave_rank<IPT>(key, shift, cnt[wv], rank, dig);
    __syncthreads();
    uint32_t sum = 0u;
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) sum += cnt[q][t];
    uint32_t* mine = tiles + tile * kDigits + t;
    __hip_atomic_store(mine, sum | (tile == 0 ? kTileTotal : kTileSum), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    uint32_t before = 0u;
    for (int64_t j = tile - 1; j >= 0;) {
        uint32_t w[kLookBack];
#pragma unroll
        for (int q = 0; q < kLookBack; ++q)
            w[q] = j >= q ? __hip_atomic_load(tiles + (j - q) * kDigits + t, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT)
                          : kTileTotal;
        bool go = true;
#pragma unroll
        for (int q = 0; q < kLookBack; ++q) {
            go = go && w[q] != 0u;
            if (go) {
                before += w[q] & kTileValue;
                --j;
                if (w[q] & kTileTotal) {
                    j = -1;
                    go = false;
                }
            }
        }
    }
    if (tile > 0)
        __hip_atomic_store(mine, (before + sum) | kTileTotal, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    uint32_t acc = first + before;
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) {
        const uint32_t c = cnt[q][t];
        cnt[q][t] = acc;
        acc += c;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        if (base + 64 * r >= n) continue;
        const uint32_t pos = cnt[wv][dig[r]] + rank[r];
        kout[pos] = key[r];
        vout[pos] = val[r];
    }
}

// ---------------------------------------------------------------- small halos
// Box, masses, keys and the whole sort of one halo of at most 1024 * IPT
// particles in one workgroup: the keys stay in registers, each digit's
// exchange goes through LDS.  Bound by one CU's vector issue (the ballots of
// the ranks): 51 us for 8192 keys, 19 us for 1500, where the general path takes
// ten launches and about 85 us (and took 33 launches and 230 us).
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;
static_assert(kSmallN == 8 * kSmallThreads, "the largest instantiation below");

template <int IPT>
__global__ __launch_bounds__(kSmallThreads) void k_cell_small(
    const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    const double* __restrict__ m, const HaloDev* __restrict__ halos, int h0, int n_halos,
    double* __restrict__ cmass, int* __restrict__ status, unsigned long long* __restrict__ keys,
    uint32_t* __restrict__ vals,
    const int8_t* __restrict__ bin, int tick, int bmax, int rank_shift,
    const int* __restrict__ active)
{
    if (tick_idle(active, tick)) return;
    __shared__ unsigned long long skey[kSmallThreads * IPT];
    __shared__ uint16_t sidx[kSmallThreads * IPT];
    __shared__ uint32_t cnt[kSmallWaves][kDigits];
    __shared__ double red[kExtrema * kSmallWaves];
    __shared__ uint32_t sw[kDigits / 64];
    const int h = h0 + (int)blockIdx.x;
    const HaloDev& H = halos[h];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int n = (int)H.n, q0 = wv * (64 * IPT) + lane;
    double px[IPT], py[IPT], pz[IPT];
    double e[kExtrema] = {INFINITY,  INFINITY,  INFINITY,  INFINITY, -INFINITY,
                        -INFINITY, -INFINITY, -INFINITY, 0.0};
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const int q = q0 + 64 * r;
        px[r] = py[r] = pz[r] = 0.0;
        if (q < n) {
            const int64_t i = H.offset + q;
            px[r] = x[i]; py[r] = y[i]; pz[r] = z[i];
            const double v[4] = {px[r], py[r], pz[r], m[i]};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                e[c] = fmin(e[c], v[c]);
                e[4 + c] = fmax(e[4 + c], v[c]);
                if (!(v[c] - v[c] == 0.0)) e[8] = 1.0;
            }
        }
    }
    block_range<kSmallWaves>(e, red);
    if (t == 0) put_mass(H, h, n_halos, e, 0.0, cmass, status);
    const double inv = key_scale(e, e + 4);
    unsigned long long key[IPT];
    uint32_t id[IPT], rank[IPT], dig[IPT];
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const int q = q0 + 64 * r;
        // past the end: behind every real key in every pass
        key[r] = q < n ? morton_key(H, px[r], py[r], pz[r], e, inv, bin, H.offset + q, tick, bmax,
                                    rank_shift)
                       : ~0ull;
        id[r] = (uint32_t)q;
    }
    const int bits = rank_shift > 48 && tick > 0 ? 49 : 48;
    for (int shift = 0; shift < bits; shift += kSortBits) {
#pragma unroll
        for (int q = 0; q < kDigits / 64; ++q) cnt[wv][64 * q + lane] = 0u;
        __builtin_amdgcn_wave_barrier();
        wave_rank<IPT>(key, shift, cnt[wv], rank, dig);
        __syncthreads();
        uint32_t sum = 0u;
        if (t < kDigits)
            for (int w = 0; w < kSmallWaves; ++w) sum += cnt[w][t];
        uint32_t acc = digit_scan(sum, sw);
        if (t < kDigits)
            for (int w = 0; w < kSmallWaves; ++w) {
                const uint32_t c = cnt[w][t];
                cnt[w][t] = acc;
                acc += c;
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            const uint32_t pos = cnt[wv][dig[r]] + rank[r];
            skey[pos] = key[r];
            sidx[pos] = (uint16_t)id[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            key[r] = skey[q0 + 64 * r];
            id[r] = sidx[q0 + 64 * r];
        }
    }
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const int q = q0 + 64 * r;
        if (q >= n) continue;
        keys[H.sbase + q] = key[r] | ((unsigned long long)H.rank << rank_shift);
        vals[H.sbase + q] = (uint32_t)(H.offset + id[r]);
    }
}

// ---------------------------------------------------------------- permute and boxes
__device__ inline double box_diag2(const double* b)
{
    const double ex = b[3] - b[0], ey = b[4] - b[1], ez = b[5] - b[2];
    return ex * ex + ey * ey + ez * ez;
}

// Split point of the lanes [lo, hi), whose box is `full`, at their coarsest
// internal Morton boundary, kept only if it at least halves the count-weighted
// extent (count x box diagonal summed over the pieces, whose boxes are ba and
// bb): a dense group is then separated from a few far members even when the
// far piece stays large.  -1 if not kept.
__device__ inline int split_range(int lo, int hi, int lane, unsigned long long key, double px,
                                  double py, double pz, const double* full, double* ba, double* bb)
{
    if (hi - lo < 2) return -1;
    const unsigned long long kf = __shfl(key, lo, 64), kl = __shfl(key, hi - 1, 64);
    if (kf == kl) return -1;
    const int hb = 63 - __clzll((long long)(kf ^ kl));
    const bool low = lane >= lo && lane < hi && !(((key ^ kf) >> hb) & 1ull);
    const int s = lo + __popcll(__ballot(low));
    if (s <= lo || s >= hi) return -1;
    lanes_box(lane >= lo && lane < s, px, py, pz, ba);
    lanes_box(lane >= s && lane < hi, px, py, pz, bb);
    const double before = (hi - lo) * sqrt(box_diag2(full));
    const double after = (s - lo) * sqrt(box_diag2(ba)) + (hi - s) * sqrt(box_diag2(bb));
    return after < 0.5 * before ? s : -1;
}

// One wave per bucket: gathers its particles into the sorted arrays, and
// writes its box and up to kSubMax compact sub-ranges (two levels of splits).
__global__ __launch_bounds__(256) void k_bucket_fill(
    const BucketInfo* __restrict__ buckets, int64_t nb, const uint32_t* __restrict__ order,
    const unsigned long long* __restrict__ skeys, const double* __restrict__ x,
    const double* __restrict__ y, const double* __restrict__ z, const double* __restrict__ vx,
    const double* __restrict__ vy, const double* __restrict__ vz, const double* __restrict__ m,
    const uint32_t* __restrict__ id, const double* __restrict__ h, double* __restrict__ sx,
    double* __restrict__ sy, double* __restrict__ sz, double* __restrict__ svx, double* __restrict__ svy, double* __restrict__ svz,
    double* __restrict__ sm, uint32_t* __restrict__ sid, double* __restrict__ sh,
    uint32_t* __restrict__ perm, double* __restrict__ box, SubRange* __restrict__ sub,
    int* __restrict__ sub_n, const int* __restrict__ active, int tick)
{
    if (tick_idle(active, tick)) return;
    const int64_t b = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (b >= nb) return;
    const int lane = threadIdx.x & 63;
    const BucketInfo B = buckets[b];
    const bool live = lane < B.count;
    const int64_t p = B.start + (live ? lane : 0);
    const uint32_t o = order[p];
    const unsigned long long key = skeys[p];
    const double px = x[o], py = y[o], pz = z[o];
    if (live) {
        sx[p] = px; sy[p] = py; sz[p] = pz;
        if (vx) { svx[p] = vx[o]; svy[p] = vy[o]; svz[p] = vz[o]; }
        sm[p] = m[o];
        if (id) sid[p] = id[o];
        sh[p] = h ? h[o] : 0.0;
        perm[p] = o;
    }
    double e[6];
    lanes_box(live, px, py, pz, e);
    if (lane == 0)
        for (int q = 0; q < 6; ++q) box[6 * b + q] = e[q];
    int n = 0;
    auto emit = [&](int lo, int hi, const double* bx) {
        if (lane == 0) {
            SubRange R;
            R.off = lo;
            R.cnt = hi - lo;
            for (int q = 0; q < 6; ++q) R.box[q] = bx[q];
            sub[kSubMax * b + n] = R;
        }
        ++n;
    };
    auto half = [&](int lo, int hi, const double* bx) {
        double ba[6], bb[6];
        const int s = split_range(lo, hi, lane, key, px, py, pz, bx, ba, bb);
        if (s > 0) {
            emit(lo, s, ba);
            emit(s, hi, bb);
        } else {
            emit(lo, hi, bx);
        }
    };
    double ba[6], bb[6];
    const int s = split_range(0, B.count, lane, key, px, py, pz, e, ba, bb);
    if (s > 0) {
        half(0, s, ba);
        half(s, B.count, bb);
    } else {
        emit(0, B.count, e);
    }
    if (lane == 0) sub_n[b] = n;
}

// The largest kernel size of every bucket.
__global__ __launch_bounds__(256) void k_bucket_hmax(
    const BucketInfo* __restrict__ buckets, int64_t nb, const double* __restrict__ sh,
    double* __restrict__ hmax)
{
    const int64_t b = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (b >= nb) return;
    const int lane = threadIdx.x & 63;
    const BucketInfo B = buckets[b];
    const double h = sh[B.start + (lane < B.count ? lane : 0)];
    const double v = rows_max(row_max(h));
    if (lane == 0) hmax[b] = v;
}

// ---------------------------------------------------------------- tree nodes
__device__ inline void node_box(const NodeTask T, double* __restrict__ box)
{
    double o[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int c = 0; c < T.nchild; ++c) {
        const double* b = box + 6 * (T.child0 + c);
        for (int q = 0; q < 3; ++q) {
            o[q] = fmin(o[q], b[q]);
            o[3 + q] = fmax(o[3 + q], b[3 + q]);
        }
    }
    for (int q = 0; q < 6; ++q) box[6 * T.node + q] = o[q];
}

__device__ inline void node_hmax(const NodeTask T, double* __restrict__ hmax)
{
    double v = 0.0;
    for (int c = 0; c < T.nchild; ++c) v = fmax(v, hmax[T.child0 + c]);
    hmax[T.node] = v;
}

// One wide level of nodes: their boxes, or (HMAX) their largest kernel sizes.
template <bool HMAX>
__global__ __launch_bounds__(256) void k_node_level(const NodeTask* __restrict__ tasks, int64_t nt,
                                                    double* __restrict__ a,
                                                    const int* __restrict__ active, int tick)
{
    if (tick_idle(active, tick)) return;
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= nt) return;
    if (HMAX) node_hmax(tasks[k], a);
    else node_box(tasks[k], a);
}

// The levels above: one workgroup, one level after the other (a launch each
// cost more than the work).
template <bool HMAX>
__global__ __launch_bounds__(kTopThreads) void k_node_top(const NodeTask* __restrict__ tasks,
                                                          TopLevels L, double* a,
                                                          const int* __restrict__ active, int tick)
{
    if (tick_idle(active, tick)) return;
    for (int l = L.first; l < L.n_levels; ++l) {
        for (int64_t k = L.off[l - 1] + threadIdx.x; k < L.off[l]; k += kTopThreads) {
            if (HMAX) node_hmax(tasks[k], a);
            else node_box(tasks[k], a);
        }
        __syncthreads();
    }
}


// ---------------------------------------------------------------- launchers
static unsigned grid_of(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

// Stable LSD radix sort of keys[0] (with vals[0]) over their low key_bits bits,
// n keys (digit counts in w.sort_ws); returns the index of the buffer pair
// that holds the result.
static int launch_sort(Scratch& w, int64_t n, int passes, hipStream_t st, const int* active,
                       int tick)
{
    int cur = 0;
    const int ipt = sort_items(n);
    const int64_t ntile = sort_tiles(n);
    for (int p = 0; p < passes; ++p) {
        uint32_t* hist = w.sort_ws + p * kDigits;
        uint32_t* ticket = w.sort_ws + kSortMaxPasses * kDigits + p;
        uint32_t* tiles = w.sort_ws + kSortHead + p * ntile * kDigits;
        auto pass = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3((unsigned)ntile), dim3(kSortBlock), 0, st, w.keys[cur],
                               w.vals[cur], w.keys[cur ^ 1], w.vals[cur ^ 1], n, p * kSortBits,
                               hist, ticket, tiles, active, tick);
        };
        if (ipt == 4) pass(k_sort_pass<4>);
        else if (ipt == 8) pass(k_sort_pass<8>);
        else pass(k_sort_pass<16>);
        cur ^= 1;
    }
    return cur;
}

template <bool HMAX>
static void launch_nodes(const Plan& P, Scratch& w, double* a, hipStream_t st,
                         const int* active = nullptr, int tick = 0)
{
    const TopLevels T = top_levels(P);
    for (int l = 1; l < T.first; ++l) {
        const int64_t t0 = P.level_task_off[l - 1], nt = P.level_task_off[l] - t0;
        hipLaunchKernelGGL(k_node_level<HMAX>, dim3(grid_of(nt, 256)), dim3(256), 0, st,
                           w.node_tasks + t0, nt, a, active, tick);
    }
    if (T.first < T.n_levels)
        hipLaunchKernelGGL(k_node_top<HMAX>, dim3(1), dim3(kTopThreads), 0, st, w.node_tasks, T, a,
                           active, tick);
}

// The cell list of the current positions, the halos' bounding boxes and their
// common masses (w.cref).  status: the halos' status words, where a halo that
// scatters with unequal masses is flagged (null: not checked).
hipError_t launch_cell_list(const Plan& P, const sidm_state* s, Scratch& w, hipStream_t st,
                            int* status, int tick, int bmax)
{
    const int64_t n = P.n_sorted;
    const int* active = idle_word(P, w, tick, bmax);
    int cur = 0;
    if (P.n_max <= kSmallN) {
        auto small = [&](auto kern) {
            launch_chunks(P.n_halos, kSmallThreads, [&](int64_t h0, int64_t count) {
                hipLaunchKernelGGL(kern, dim3((unsigned)count), dim3(kSmallThreads), 0, st, s->x,
                                   s->y, s->z, s->m, w.halos, (int)h0, P.n_halos, w.cref, status,
                                   w.keys[0], w.vals[0], w.bin, tick, bmax, P.rank_shift, active);
            });
        };
        if (P.n_max <= kSmallThreads) small(k_cell_small<1>);
        else if (P.n_max <= 2 * kSmallThreads) small(k_cell_small<2>);
        else if (P.n_max <= 4 * kSmallThreads) small(k_cell_small<4>);
        else small(k_cell_small<8>);
    } else {
        const int passes = (P.key_bits + kSortBits - 1) / kSortBits;
        const int64_t n_zero = kSortHead + passes * sort_tiles(n) * kDigits;
        if (passes > kSortMaxPasses || n > (int64_t)kTileValue || n_zero > w.sort_ws_n)
            return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_block_range, dim3((unsigned)P.n_blocks), dim3(kStreamBlock), 0, st,
                           s->x, s->y, s->z, s->m, w.blocks, w.brange, w.sort_ws, n_zero, active,
                           tick);
        launch_chunks(P.n_halos, kRangeThreads, [&](int64_t h0, int64_t count) {
            hipLaunchKernelGGL(k_halo_range, dim3((unsigned)count), dim3(kRangeThreads), 0, st,
                               w.halos, (int)h0, P.n_halos, w.brange, w.bbox, w.cref, status,
                               active, tick);
        });
        // at most 16 blocks per workgroup; from 64 workgroups on, fewer of them
        // are better: each adds up to kDigits words per pass to the same counts
        // (65536 particles: 10.3 us with 256 workgroups, 7.5 us with 64)
        const int group = (int)std::max<int64_t>(1, std::min<int64_t>(16, P.n_blocks / 64));
        hipLaunchKernelGGL(k_morton_keys, dim3(grid_of(P.n_blocks, group)), dim3(kStreamBlock), 0,
                           st, s->x, s->y, s->z, w.blocks, P.n_blocks, group, w.halos, w.bbox,
                           w.keys[0], w.vals[0], w.bin, tick, bmax, P.rank_shift, passes,
                           w.sort_ws, active);
        cur = launch_sort(w, n, passes, st, active, tick);
    }
    hipLaunchKernelGGL(k_bucket_fill, dim3(grid_of(P.n_buckets, 4)), dim3(256), 0, st, w.buckets,
                       P.n_buckets, w.vals[cur], w.keys[cur], s->x, s->y, s->z, s->vx, s->vy,
                       s->vz, s->m, s->id, s->h, w.sx, w.sy, w.sz, w.svx, w.svy, w.svz,
                       w.sm, w.sid, w.sh, w.perm, w.box, w.sub, w.sub_n, active, tick);
    launch_nodes<false>(P, w, w.box, st, active, tick);
    return hipGetLastError();
}

hipError_t launch_tree_hmax(const Plan& P, Scratch& w, hipStream_t st)
{
    hipLaunchKernelGGL(k_bucket_hmax, dim3(grid_of(P.n_buckets, 4)), dim3(256), 0, st, w.buckets,
                       P.n_buckets, w.sh, w.hmax);
    launch_nodes<true>(P, w, w.hmax, st);
    return hipGetLastError();
}

}  // namespace sidm
