// k_stream.hip -- streaming FP64 passes of the leapfrog and the energy and
// momentum reductions (kick-drift-kick with a fixed step or block steps; the
// paper's energy error is measured relative to the absolute initial energy,
// App. B).
#include "sidm_host.hpp"
#include "sidm_steps.hpp"

namespace sidm {

// Reflecting sphere (Sec. 2): at the drifted position p, outward motion beyond
// the radius is turned inward, v -> v - 2 (v.d) d / |d|^2 (|v| kept).
__device__ inline void reflect(const HaloDev& H, double px, double py, double pz, double& ux,
                               double& uy, double& uz)
{
#pragma clang fp contract(off)
    if (!(H.bnd_r > 0.0)) return;
    const double dx = px - H.bnd_c[0], dy = py - H.bnd_c[1], dz = pz - H.bnd_c[2];
    const double d2 = (dx * dx + dy * dy) + dz * dz;
    const double vd = (ux * dx + uy * dy) + uz * dz;
    if (d2 > H.bnd_r * H.bnd_r && vd > 0.0) {
        const double f = 2.0 * vd / d2;
        ux = ux - f * dx; uy = uy - f * dy; uz = uz - f * dz;
    }
}

// v += a dt/2 ; x += v dt   (opening half kick fused with the drift)
__global__ __launch_bounds__(kStreamBlock) void k_kick_drift(
    const StreamBlock* __restrict__ blocks, const HaloDev* __restrict__ halos,
    double* __restrict__ x, double* __restrict__ y, double* __restrict__ z,
    double* __restrict__ vx, double* __restrict__ vy, double* __restrict__ vz,
    const double* __restrict__ ax, const double* __restrict__ ay, const double* __restrict__ az)
{
#pragma clang fp contract(off)
    const StreamBlock B = blocks[blockIdx.x];
    const int t = threadIdx.x;
    if (t >= B.count) return;
    const HaloDev& H = halos[B.halo];
    const int64_t i = B.start + t;
    const double hdt = 0.5 * H.dt;
    double ux = vx[i] + ax[i] * hdt;
    double uy = vy[i] + ay[i] * hdt;
    double uz = vz[i] + az[i] * hdt;
    const double px = x[i] + ux * H.dt, py = y[i] + uy * H.dt, pz = z[i] + uz * H.dt;
    x[i] = px; y[i] = py; z[i] = pz;
    reflect(H, px, py, pz, ux, uy, uz);
    vx[i] = ux; vy[i] = uy; vz[i] = uz;
}

// Start of a cycle of block steps: the bin of every particle from its
// acceleration, and its opening half kick v += a s/2.
__global__ __launch_bounds__(kStreamBlock) void k_open_kick(
    const StreamBlock* __restrict__ blocks, const HaloDev* __restrict__ halos,
    double* __restrict__ vx, double* __restrict__ vy, double* __restrict__ vz,
    const double* __restrict__ ax, const double* __restrict__ ay, const double* __restrict__ az,
    int8_t* __restrict__ bin)
{
#pragma clang fp contract(off)
    const StreamBlock B = blocks[blockIdx.x];
    const int t = threadIdx.x;
    if (t >= B.count) return;
    const HaloDev& H = halos[B.halo];
    const int64_t i = B.start + t;
    const double gx = ax[i], gy = ay[i], gz = az[i];
    const int b = time_bin(H, gx, gy, gz);
    bin[i] = (int8_t)b;
    const double h = half_step(H, b);
    vx[i] = vx[i] + gx * h;
    vy[i] = vy[i] + gy * h;
    vz[i] = vz[i] + gz * h;
}

// One tick of a cycle: x += v dt / 2^max_bin for every particle of the halos
// that step at this tick, then the reflecting sphere.  active: set to the tick if
// some particle's step ends at it.  Between the ends of the smallest steps taken
// nothing reads a cell list or forces, so the kernels of a tick return at once
// when it is idle (65536 particles, 64 ticks of which 8 end a step: 103 us per
// idle tick with all of its work).
__global__ __launch_bounds__(kStreamBlock) void k_tick_drift(
    const StreamBlock* __restrict__ blocks, const HaloDev* __restrict__ halos,
    double* __restrict__ x, double* __restrict__ y, double* __restrict__ z,
    double* __restrict__ vx, double* __restrict__ vy, double* __restrict__ vz,
    const int8_t* __restrict__ bin, int* __restrict__ active, int tick, int bmax)
{
#pragma clang fp contract(off)
    const StreamBlock B = blocks[blockIdx.x];
    const int t = threadIdx.x;
    if (t >= B.count) return;
    const HaloDev& H = halos[B.halo];
    const int kl = local_tick(H, tick, bmax);
    if (kl == 0) return;
    const int64_t i = B.start + t;
    if (bin_active(H, bin[i], kl)) *active = tick;
    const double tau = ldexp(H.dt, -H.max_bin);
    double ux = vx[i], uy = vy[i], uz = vz[i];
    const double px = x[i] + ux * tau, py = y[i] + uy * tau, pz = z[i] + uz * tau;
    x[i] = px; y[i] = py; z[i] = pz;
    if (H.bnd_r > 0.0) {
        reflect(H, px, py, pz, ux, uy, uz);
        vx[i] = ux; vy[i] = uy; vz[i] = uz;
    }
}

// Per-block partial sums of K, W, Eext, px, py, pz and a non-finite flag.
__global__ __launch_bounds__(kStreamBlock) void k_diag_block(
    const StreamBlock* __restrict__ blocks, const HaloDev* __restrict__ halos,
    const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    const double* __restrict__ vx, const double* __restrict__ vy, const double* __restrict__ vz,
    const double* __restrict__ m, const double* __restrict__ pot, double* __restrict__ bsum)
{
    __shared__ double red[7][kStreamBlock];
    const StreamBlock B = blocks[blockIdx.x];
    const HaloDev& H = halos[B.halo];
    const int t = threadIdx.x;
    double v[7] = {0, 0, 0, 0, 0, 0, 0};
    if (t < B.count) {
        const int64_t i = B.start + t;
        const double mi = m[i];
        const double ux = vx[i], uy = vy[i], uz = vz[i];
        double pe = 0.0;
        if (H.host_kind != 0) pe = host_potential(H, x[i], y[i], z[i]);
        v[0] = 0.5 * mi * ((ux * ux + uy * uy) + uz * uz);
        v[1] = 0.5 * mi * (pot[i] - pe);
        v[2] = mi * pe;
        v[3] = mi * ux; v[4] = mi * uy; v[5] = mi * uz;
        const double chk = x[i] + y[i] + z[i] + ux + uy + uz;
        v[6] = isfinite(chk) ? 0.0 : 1.0;
    }
    for (int c = 0; c < 7; ++c) red[c][t] = v[c];
    __syncthreads();
    for (int s = kStreamBlock / 2; s > 0; s >>= 1) {
        if (t < s)
            for (int c = 0; c < 7; ++c) red[c][t] += red[c][t + s];
        __syncthreads();
    }
    if (t < 7) bsum[7 * (int64_t)blockIdx.x + t] = red[t][0];
}

// One block per halo: fixed-order sum of the block partials into sidm_diag.
__global__ __launch_bounds__(kStreamBlock) void k_diag_halo(
    const HaloDev* __restrict__ halos, const double* __restrict__ bsum,
    const long long* __restrict__ ev_counts, const unsigned long long* __restrict__ tree_terms,
    const int* __restrict__ status, sidm_diag* __restrict__ diag)
{
    __shared__ double red[7][kStreamBlock];
    const HaloDev& H = halos[blockIdx.x];
    const int t = threadIdx.x;
    const int64_t nb = (H.n + kStreamBlock - 1) / kStreamBlock;
    double s[7] = {0, 0, 0, 0, 0, 0, 0};
    for (int64_t b = t; b < nb; b += kStreamBlock)
        for (int c = 0; c < 7; ++c) s[c] += bsum[7 * (H.stream_block0 + b) + c];
    for (int c = 0; c < 7; ++c) red[c][t] = s[c];
    __syncthreads();
    for (int st = kStreamBlock / 2; st > 0; st >>= 1) {
        if (t < st)
            for (int c = 0; c < 7; ++c) red[c][t] += red[c][t + st];
        __syncthreads();
    }
    if (t == 0) {
        sidm_diag d;
        d.K = red[0][0]; d.W = red[1][0]; d.Eext = red[2][0];
        d.px = red[3][0]; d.py = red[4][0]; d.pz = red[5][0];
        const int h = blockIdx.x;
        d.n_events = ev_counts ? ev_counts[kEvCounts * h + 0] : 0;
        d.n_rounds = ev_counts ? ev_counts[kEvCounts * h + 1] : 0;
        d.n_pairs = ev_counts ? ev_counts[kEvCounts * h + 2] : 0;
        d.n_p_gt1 = ev_counts ? ev_counts[kEvCounts * h + 3] : 0;
        d.n_candidates = ev_counts ? ev_counts[kEvCounts * h + 4] : 0;
        d.status = (status ? status[h] : 0) | (red[6][0] > 0.0 ? SIDM_DEV_NONFINITE : 0);
        d.reserved = 0;
        d.n_grav_terms = tree_terms ? (int64_t)tree_terms[h] : 0;
        diag[h] = d;
    }
}

hipError_t launch_kick_drift(const StreamBlock* d_blocks, int64_t n_blocks, const HaloDev* d_halos,
                             double* x, double* y, double* z, double* vx, double* vy, double* vz,
                             const double* ax, const double* ay, const double* az, hipStream_t st)
{
    hipLaunchKernelGGL(k_kick_drift, dim3((unsigned)n_blocks), dim3(kStreamBlock), 0, st, d_blocks,
                       d_halos, x, y, z, vx, vy, vz, ax, ay, az);
    return hipGetLastError();
}

hipError_t launch_open_kick(const StreamBlock* d_blocks, int64_t n_blocks, const HaloDev* d_halos,
                            double* vx, double* vy, double* vz, const double* ax, const double* ay,
                            const double* az, int8_t* bin, hipStream_t st)
{
    hipLaunchKernelGGL(k_open_kick, dim3((unsigned)n_blocks), dim3(kStreamBlock), 0, st, d_blocks,
                       d_halos, vx, vy, vz, ax, ay, az, bin);
    return hipGetLastError();
}

hipError_t launch_tick_drift(const StreamBlock* d_blocks, int64_t n_blocks, const HaloDev* d_halos,
                             double* x, double* y, double* z, double* vx, double* vy, double* vz,
                             const int8_t* bin, int* active, int tick, int bmax, hipStream_t st)
{
    hipLaunchKernelGGL(k_tick_drift, dim3((unsigned)n_blocks), dim3(kStreamBlock), 0, st, d_blocks,
                       d_halos, x, y, z, vx, vy, vz, bin, active, tick, bmax);
    return hipGetLastError();
}

hipError_t launch_diag(const StreamBlock* d_blocks, int64_t n_blocks, const HaloDev* d_halos,
                       int n_halos, const double* x, const double* y, const double* z,
                       const double* vx, const double* vy, const double* vz, const double* m,
                       const double* pot, double* bsum, const long long* ev_counts,
                       const unsigned long long* tree_terms, const int* status, sidm_diag* diag,
                       hipStream_t st)
{
    hipLaunchKernelGGL(k_diag_block, dim3((unsigned)n_blocks), dim3(kStreamBlock), 0, st, d_blocks,
                       d_halos, x, y, z, vx, vy, vz, m, pot, bsum);
    hipLaunchKernelGGL(k_diag_halo, dim3(n_halos), dim3(kStreamBlock), 0, st, d_halos, bsum,
                       ev_counts, tree_terms, status, diag);
    return hipGetLastError();
}

// ---------------------------------------------------------------- central density
// Sec. 3 takes the minimum of the gravitational potential as the halo centre:
// the centre is the particle with the lowest self-potential pot - Phi_host
// (first index on ties, NaN never), and the central density counts the
// particles of the halo within a radius of it.

// Per streaming block: lowest self-potential and its index (as a double).
__global__ __launch_bounds__(kStreamBlock) void k_center_block(
    const StreamBlock* __restrict__ blocks, const HaloDev* __restrict__ halos,
    const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    const double* __restrict__ pot, double* __restrict__ bsum)
{
    __shared__ double val[kStreamBlock];
    __shared__ int64_t idx[kStreamBlock];
    const StreamBlock B = blocks[blockIdx.x];
    const HaloDev& H = halos[B.halo];
    const int t = threadIdx.x;
    double v = INFINITY;
    int64_t i = -1;
    if (t < B.count) {
        const int64_t p = B.start + t;
        double pe = 0.0;
        if (H.host_kind != 0) pe = host_potential(H, x[p], y[p], z[p]);
        const double ps = pot[p] - pe;
        if (ps == ps) { v = ps; i = p; }
    }
    val[t] = v;
    idx[t] = i;
    __syncthreads();
    for (int s = kStreamBlock / 2; s > 0; s >>= 1) {
        if (t < s) {
            const double vo = val[t + s];
            const int64_t io = idx[t + s];
            if (io >= 0 && (idx[t] < 0 || vo < val[t] || (vo == val[t] && io < idx[t]))) {
                val[t] = vo;
                idx[t] = io;
            }
        }
        __syncthreads();
    }
    if (t == 0) {
        bsum[7 * blockIdx.x + 0] = val[0];
        bsum[7 * blockIdx.x + 1] = (double)idx[0];
    }
}

// Per halo: the centre over its blocks; writes index and position.
__global__ __launch_bounds__(kStreamBlock) void k_center_halo(
    const HaloDev* __restrict__ halos, const double* __restrict__ bsum,
    const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    sidm_center* __restrict__ out)
{
    __shared__ double val[kStreamBlock];
    __shared__ int64_t idx[kStreamBlock];
    const HaloDev& H = halos[blockIdx.x];
    const int t = threadIdx.x;
    const int64_t nb = (H.n + kStreamBlock - 1) / kStreamBlock;
    double v = INFINITY;
    int64_t i = -1;
    for (int64_t b = t; b < nb; b += kStreamBlock) {
        const double vo = bsum[7 * (H.stream_block0 + b) + 0];
        const int64_t io = (int64_t)bsum[7 * (H.stream_block0 + b) + 1];
        if (io >= 0 && (i < 0 || vo < v || (vo == v && io < i))) { v = vo; i = io; }
    }
    val[t] = v;
    idx[t] = i;
    __syncthreads();
    for (int s = kStreamBlock / 2; s > 0; s >>= 1) {
        if (t < s) {
            const double vo = val[t + s];
            const int64_t io = idx[t + s];
            if (io >= 0 && (idx[t] < 0 || vo < val[t] || (vo == val[t] && io < idx[t]))) {
                val[t] = vo;
                idx[t] = io;
            }
        }
        __syncthreads();
    }
    if (t == 0) {
        sidm_center c;
        c.index = idx[0];
        c.x = c.index >= 0 ? x[c.index] : NAN;
        c.y = c.index >= 0 ? y[c.index] : NAN;
        c.z = c.index >= 0 ? z[c.index] : NAN;
        c.mass = 0.0;
        c.count = 0;
        out[blockIdx.x] = c;
    }
}

// Per streaming block: number and mass of the particles within the radius.
__global__ __launch_bounds__(kStreamBlock) void k_center_count_block(
    const StreamBlock* __restrict__ blocks, const double* __restrict__ radius,
    const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    const double* __restrict__ m, const sidm_center* __restrict__ out, double* __restrict__ bsum)
{
    __shared__ double cnt[kStreamBlock], mass[kStreamBlock];
    const StreamBlock B = blocks[blockIdx.x];
    const sidm_center C = out[B.halo];
    const int t = threadIdx.x;
    double c = 0.0, w = 0.0;
    if (t < B.count && C.index >= 0) {
#pragma clang fp contract(off)
        const int64_t p = B.start + t;
        const double r = radius[B.halo];
        const double dx = x[p] - C.x, dy = y[p] - C.y, dz = z[p] - C.z;
        const double d2 = (dx * dx + dy * dy) + dz * dz;
        if (d2 <= r * r) { c = 1.0; w = m[p]; }
    }
    cnt[t] = c;
    mass[t] = w;
    __syncthreads();
    for (int s = kStreamBlock / 2; s > 0; s >>= 1) {
        if (t < s) { cnt[t] += cnt[t + s]; mass[t] += mass[t + s]; }
        __syncthreads();
    }
    if (t == 0) {
        bsum[7 * blockIdx.x + 2] = cnt[0];
        bsum[7 * blockIdx.x + 3] = mass[0];
    }
}

__global__ __launch_bounds__(kStreamBlock) void k_center_count_halo(
    const HaloDev* __restrict__ halos, const double* __restrict__ bsum,
    sidm_center* __restrict__ out)
{
    __shared__ double cnt[kStreamBlock], mass[kStreamBlock];
    const HaloDev& H = halos[blockIdx.x];
    const int t = threadIdx.x;
    const int64_t nb = (H.n + kStreamBlock - 1) / kStreamBlock;
    double c = 0.0, w = 0.0;
    for (int64_t b = t; b < nb; b += kStreamBlock) {
        c += bsum[7 * (H.stream_block0 + b) + 2];
        w += bsum[7 * (H.stream_block0 + b) + 3];
    }
    cnt[t] = c;
    mass[t] = w;
    __syncthreads();
    for (int s = kStreamBlock / 2; s > 0; s >>= 1) {
        if (t < s) { cnt[t] += cnt[t + s]; mass[t] += mass[t + s]; }
        __syncthreads();
    }
    if (t == 0) {
        out[blockIdx.x].count = (int64_t)cnt[0];
        out[blockIdx.x].mass = mass[0];
    }
}

hipError_t launch_center(const StreamBlock* d_blocks, int64_t n_blocks, const HaloDev* d_halos,
                         int n_halos, const double* radius, const double* x, const double* y,
                         const double* z, const double* m, const double* pot, double* bsum,
                         sidm_center* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_center_block, dim3((unsigned)n_blocks), dim3(kStreamBlock), 0, st,
                       d_blocks, d_halos, x, y, z, pot, bsum);
    hipLaunchKernelGGL(k_center_halo, dim3(n_halos), dim3(kStreamBlock), 0, st, d_halos, bsum, x,
                       y, z, out);
    hipLaunchKernelGGL(k_center_count_block, dim3((unsigned)n_blocks), dim3(kStreamBlock), 0, st,
                       d_blocks, radius, x, y, z, m, out, bsum);
    hipLaunchKernelGGL(k_center_count_halo, dim3(n_halos), dim3(kStreamBlock), 0, st, d_halos,
                       bsum, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------- tidal radius
// Eq. tidal_radius: G M(<= r) / r^2 = |grad Phi_host(c + r n) - grad Phi_host(c - r n)|,
// bisection in log r.  Per-halo state in `tid` (8 doubles): n (3), lo, hi,
// the initial hi, the mass within hi, whether that is known.

// Per streaming block: the largest squared distance from the halo's centre.
__global__ __launch_bounds__(kStreamBlock) void k_tidal_extent(
    const StreamBlock* __restrict__ blocks, const double* __restrict__ x,
    const double* __restrict__ y, const double* __restrict__ z,
    const sidm_center* __restrict__ cen, double* __restrict__ bsum)
{
    __shared__ double red[kStreamBlock];
    const StreamBlock B = blocks[blockIdx.x];
    const sidm_center C = cen[B.halo];
    const int t = threadIdx.x;
    double v = 0.0;
    if (t < B.count && C.index >= 0) {
#pragma clang fp contract(off)
        const int64_t p = B.start + t;
        const double dx = x[p] - C.x, dy = y[p] - C.y, dz = z[p] - C.z;
        v = (dx * dx + dy * dy) + dz * dz;
    }
    red[t] = v;
    __syncthreads();
    for (int s = kStreamBlock / 2; s > 0; s >>= 1) {
        if (t < s) red[t] = fmax(red[t], red[t + s]);
        __syncthreads();
    }
    if (t == 0) bsum[7 * blockIdx.x + 4] = red[0];
}

// Per halo: the direction from the host centre and the initial bracket.
__global__ __launch_bounds__(kStreamBlock) void k_tidal_init(
    const HaloDev* __restrict__ halos, const double* __restrict__ bsum,
    const sidm_center* __restrict__ cen, double* __restrict__ tid)
{
    __shared__ double red[kStreamBlock];
    const HaloDev& H = halos[blockIdx.x];
    const int t = threadIdx.x;
    const int64_t nb = (H.n + kStreamBlock - 1) / kStreamBlock;
    double v = 0.0;
    for (int64_t b = t; b < nb; b += kStreamBlock) v = fmax(v, bsum[7 * (H.stream_block0 + b) + 4]);
    red[t] = v;
    __syncthreads();
    for (int s = kStreamBlock / 2; s > 0; s >>= 1) {
        if (t < s) red[t] = fmax(red[t], red[t + s]);
        __syncthreads();
    }
    if (t == 0) {
#pragma clang fp contract(off)
        const sidm_center C = cen[blockIdx.x];
        double* T = tid + 8 * blockIdx.x;
        const double ux = C.x - H.host_c[0], uy = C.y - H.host_c[1], uz = C.z - H.host_c[2];
        const double u = sqrt((ux * ux + uy * uy) + uz * uz);
        T[0] = u > 0.0 ? ux / u : 1.0;
        T[1] = u > 0.0 ? uy / u : 0.0;
        T[2] = u > 0.0 ? uz / u : 0.0;
        const double hi = 2.0 * sqrt(red[0]);
        T[4] = hi;
        T[3] = ldexp(hi, -40);
        T[5] = hi;
        T[6] = 0.0;
        T[7] = 0.0;
    }
}

// The bisection takes kTidalLevels steps per launch.  The midpoints that those
// steps can reach are known before any of them is taken (a tree of 2^levels - 1
// radii below the bracket, node q's children 2q and 2q + 1), so one pass over
// the particles sums the mass within each of them and within the upper
// bracket; the next launch adds the workgroups' sums, decides every node at
// once and follows the decisions down.  Every workgroup of a halo does that for
// itself, in the same order, so nothing is exchanged within a launch.  60
// launches of a mass pass and 60 of a one-workgroup sum and decision, 6 and 11
// us each at 2^20 particles, became 13 of 15 us (a chain of loads, square roots
// and fields; the sums themselves take 3).
//
// That chain is every workgroup's, and a compute unit holds one workgroup of
// 512 threads (168 registers), so a call takes about one workgroup per compute
// unit, dealt out to the halos by their sizes in the plan (HaloDev::tidal_wg;
// a division here would add 0.4 us to each pass): with up to 256 for each of them 40
// halos of 50000 took 3.27 ms (1.10 with the 120 launches), now 0.31.  Beyond
// kTidalFew halos, all of them small, a wave per halo is enough and a compute
// unit holds twelve: 20000 halos of 70 take 1.45 ms (9.53 in workgroups of 512,
// 3.42 with the 120 launches).
constexpr int kTidalLevels = 5;
constexpr int kTidalSums = 1 << kTidalLevels;   // 31 nodes (entry q - 1) and the upper bracket
constexpr int kTidalSteps = 60;
constexpr int kTidalFew = 256;                  // more halos than this, of at most
constexpr int64_t kTidalWaveN = 4096;           // this many particles: a wave per halo
static_assert(kTidalSteps % kTidalLevels == 0, "whole launches");

struct Bracket {
    double lo, hi;
};

// The bracket of node q of the tree below b, whose midpoint is the node's
// radius: the steps of the bisection on the way down.
__device__ inline Bracket tidal_node(Bracket b, int q)
{
#pragma clang fp contract(off)
    for (int l = 30 - __clz(q); l >= 0; --l) {
        const double r = sqrt(b.lo * b.hi);
        if ((q >> l) & 1) b.lo = r;
        else b.hi = r;
    }
    return b;
}

// The acceleration of one component of the host at the node's radius on either
// side of the centre (the wave's index: the component; lanes 0 to 31 outwards,
// 32 to 63 inwards).  The fields' square roots, divisions and logarithms are a
// serial chain of 10 us when one lane evaluates all components of both sides.
__device__ inline void tidal_part(const HaloDev& H, const sidm_center& C, const double* T,
                                  const Bracket& b, int part, int lane, double (*field)[64][3])
{
#pragma clang fp contract(off)
    const int q = lane % kTidalSums + 1;
    if (q == kTidalSums) return;
    const Bracket n = tidal_node(b, q);
    const double r = sqrt(n.lo * n.hi), s = lane < kTidalSums ? r : -r;
    const double px = C.x + s * T[0], py = C.y + s * T[1], pz = C.z + s * T[2];
    double phi;
    double* a = field[part][lane];
    host_part(H, part, px - H.host_c[0], py - H.host_c[1], pz - H.host_c[2], a[0], a[1], a[2],
              phi);
}

// Whether the halo's own gravity at r wins over the host's tide there, for the
// node of thread t (the components of its two sides added as host_field does).
__device__ inline bool tidal_inside(const HaloDev& H, const double (*field)[64][3], int t,
                                    double r, double M)
{
#pragma clang fp contract(off)
    double g[3];
    for (int c = 0; c < 3; ++c) {
        double out = field[0][t][c], in = field[0][t + kTidalSums][c];
        for (int k = 1; k < kHostParts; ++k) {
            out += field[k][t][c];
            in += field[k][t + kTidalSums][c];
        }
        g[c] = out - in;
    }
    const double tide = sqrt((g[0] * g[0] + g[1] * g[1]) + g[2] * g[2]);
    return H.G * M / (r * r) > tide;
}

// Workgroup w0 + blockIdx.x: per_halo of them for each halo (those past its own
// leave), or with `blocks` one for each streaming block (of which a halo keeps
// the first ones).  tid_in / tid_out: the state before and after the
// decisions on sums_in (none in the first launch); sums_out: this launch's sums
// (kTidalSums per workgroup).  The last launch writes the record instead.  NT
// threads, at most MOST workgroups per halo.
template <int NT, int MOST>
__global__ __launch_bounds__(NT) void k_tidal_pass(
    const HaloDev* __restrict__ halos, const StreamBlock* __restrict__ blocks, int64_t w0,
    const double* __restrict__ x, const double* __restrict__ y,
    const double* __restrict__ z, const double* __restrict__ m,
    const sidm_center* __restrict__ cen, const double* __restrict__ tid_in,
    double* __restrict__ tid_out, const double* __restrict__ sums_in,
    double* __restrict__ sums_out, int per_halo, int first, int last,
    sidm_tidal* __restrict__ out)
{
    constexpr int NW = NT / 64, NG = NT / kTidalSums;
    __shared__ double red[NG][kTidalSums];
    __shared__ double rad2[kTidalSums];
    __shared__ int inside[kTidalSums];
    __shared__ double field[kHostParts][64][3];
    static_assert(2 * kTidalSums == 64, "a lane per side");
    const int t = threadIdx.x;
    const int64_t wg = w0 + blockIdx.x;
    // (without blocks there are fewer workgroups than streaming blocks or halos)
    const int h = blocks ? blocks[wg].halo : (int)((uint32_t)wg / (uint32_t)per_halo);
    const HaloDev& H = halos[h];
    const int64_t g = blocks ? wg - H.stream_block0 : (uint32_t)wg % (uint32_t)per_halo;
    const int groups = MOST == 1 ? 1 : H.tidal_wg;
    if (g >= (last ? 1 : groups)) return;
    const sidm_center C = cen[h];
    double T[8];
    for (int q = 0; q < 8; ++q) T[q] = tid_in[8 * (int64_t)h + q];
    Bracket b{T[3], T[4]};
    double M_hi = T[6];   // mass within the upper bracket
    if (!first) {
        // the sums of the previous pass, in workgroup order
        const int c = t % kTidalSums, part = t / kTidalSums;
        constexpr int kRows = (MOST + NG - 1) / NG;
        double w[kRows], v = 0.0;
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            const int q = part + u * NG;
            w[u] = q < groups ? sums_in[(H.stream_block0 + q) * kTidalSums + c] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kRows; ++u) v += w[u];
        red[part][c] = v;
        if (NW >= kHostParts) {
            if (t / 64 < kHostParts) tidal_part(H, C, T, b, t / 64, t & 63, field);
        } else {
            for (int k = t / 64; k < kHostParts; k += NW) tidal_part(H, C, T, b, k, t & 63, field);
        }
        __syncthreads();
        if (t < kTidalSums) {
            double M = 0.0;
            for (int q = 0; q < NG; ++q) M += red[q][t];
            red[0][t] = M;
            if (t + 1 < kTidalSums) {
                const Bracket n = tidal_node(b, t + 1);
                inside[t] = tidal_inside(H, field, t, sqrt(n.lo * n.hi), M);
            }
        }
        __syncthreads();
        if (T[7] == 0.0) M_hi = red[0][kTidalSums - 1];   // the initial bracket's
        for (int l = 0, q = 1; l < kTidalLevels; ++l) {
#pragma clang fp contract(off)
            const double r = sqrt(b.lo * b.hi);
            const bool in = inside[q - 1];
            if (in) {
                b.lo = r;
            } else {
                b.hi = r;
                M_hi = red[0][q - 1];
            }
            q = 2 * q + (in ? 1 : 0);
        }
    }
    if (last) {
        if (t == 0) {
            sidm_tidal o;
            o.r_tidal = b.hi;
            o.mass = M_hi;
            o.x = C.x; o.y = C.y; o.z = C.z;
            o.index = C.index;
            o.status = b.hi == T[5] ? 1 : 0;
            o.reserved = 0;
            out[h] = o;
        }
        return;
    }
    if (g == 0 && t < 8)
        tid_out[8 * (int64_t)h + t] = t == 3   ? b.lo
                                      : t == 4 ? b.hi
                                      : t == 6 ? M_hi
                                      : t == 7 ? (first ? 0.0 : 1.0)
                                               : T[t];
    __syncthreads();   // the previous sums are read before red is reused
    if (t < kTidalSums) {
#pragma clang fp contract(off)
        double r = b.hi;
        if (t + 1 < kTidalSums) {
            const Bracket n = tidal_node(b, t + 1);
            r = sqrt(n.lo * n.hi);
        }
        rad2[t] = r * r;
    }
    __syncthreads();
    double v[kTidalSums];
#pragma unroll
    for (int c = 0; c < kTidalSums; ++c) v[c] = 0.0;
    if (C.index >= 0) {
        // four particles' loads in flight
        constexpr int kLoads = 4;
        const int64_t step = (int64_t)groups * NT;
        for (int64_t i = g * NT + t; i < H.n; i += kLoads * step) {
#pragma clang fp contract(off)
            double d2[kLoads], mp[kLoads];
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                const bool on = i + u * step < H.n;
                const int64_t p = H.offset + (on ? i + u * step : i);
                const double dx = x[p] - C.x, dy = y[p] - C.y, dz = z[p] - C.z;
                d2[u] = (dx * dx + dy * dy) + dz * dz;
                mp[u] = on ? m[p] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < kLoads; ++u)
#pragma unroll
                for (int c = 0; c < kTidalSums; ++c) v[c] += d2[u] <= rad2[c] ? mp[u] : 0.0;
        }
    }
    // over the wave: every exchange halves the sums a lane holds; lane l ends
    // with sum l / 2
    const int lane = t & 63;
#pragma unroll
    for (int k = kTidalSums / 2; k > 0; k /= 2) {
        const int o = 2 * k;
        const bool up = lane & o;
#pragma unroll
        for (int c = 0; c < k; ++c) {
            const double keep = up ? v[c + k] : v[c], give = up ? v[c] : v[c + k];
            v[c] = keep + __shfl_xor(give, o, 64);
        }
    }
    v[0] += __shfl_xor(v[0], 1, 64);
    if (!(lane & 1)) red[t >> 6][lane >> 1] = v[0];
    __syncthreads();
    if (t < kTidalSums) {
        double M = 0.0;
        for (int w = 0; w < NW; ++w) M += red[w][t];
        sums_out[(H.stream_block0 + g) * kTidalSums + t] = M;
    }
}

hipError_t launch_tidal(const StreamBlock* d_blocks, int64_t n_blocks, const HaloDev* d_halos,
                        int n_halos, int64_t n_max, int wg_max, const double* x,
                        const double* y, const double* z, const double* m, const double* pot, double* bsum, sidm_center* cen,
                        double* tid, double* sums, sidm_tidal* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_center_block, dim3((unsigned)n_blocks), dim3(kStreamBlock), 0, st,
                       d_blocks, d_halos, x, y, z, pot, bsum);
    hipLaunchKernelGGL(k_center_halo, dim3(n_halos), dim3(kStreamBlock), 0, st, d_halos, bsum, x,
                       y, z, cen);
    hipLaunchKernelGGL(k_tidal_extent, dim3((unsigned)n_blocks), dim3(kStreamBlock), 0, st,
                       d_blocks, x, y, z, cen, bsum);
    hipLaunchKernelGGL(k_tidal_init, dim3(n_halos), dim3(kStreamBlock), 0, st, d_halos, bsum, cen,
                       tid);
    constexpr int kPasses = kTidalSteps / kTidalLevels;
    double* state[2] = {tid, tid + 8 * (int64_t)n_halos};
    double* sum[2] = {sums, sums + n_blocks * kTidalSums};
    const bool waves = n_halos > kTidalFew && n_max <= kTidalWaveN;
    const int groups = waves ? 1 : wg_max;
    // one halo much larger than the others: a workgroup per streaming block
    // instead of the largest halo's number for each
    const bool by_block = n_blocks < (int64_t)groups * n_halos;
    auto passes = [&](auto kern, int threads) {
        for (int it = 0; it <= kPasses; ++it) {
            const bool last = it == kPasses;
            const int per_halo = last ? 1 : groups;
            const StreamBlock* blk = by_block && !last ? d_blocks : nullptr;
            launch_chunks(blk ? n_blocks : (int64_t)per_halo * n_halos, threads,
                          [&](int64_t w0, int64_t count) {
                              hipLaunchKernelGGL(kern, dim3((unsigned)count), dim3(threads), 0, st,
                                                 d_halos, blk, w0, x, y, z, m, cen, state[it & 1],
                                                 state[(it & 1) ^ 1], sum[(it & 1) ^ 1],
                                                 sum[it & 1], per_halo, it == 0, last, out);
                          });
        }
    };
    if (waves) passes(k_tidal_pass<64, 1>, 64);
    else passes(k_tidal_pass<512, kTidalWg>, 512);
    return hipGetLastError();
}

}  // namespace sidm
