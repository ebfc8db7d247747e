// Metropolis Monte Carlo with an adaptive trial cone and simulated annealing
// (Sec. 2.1, Sec. 4.3) on the Hamiltonian of Eq. (1), on gfx950.
//
// Sites are split into colour classes that share no bond (greedy colouring
// on the host), so one class is updated in parallel, one thread per site.
// The state is FP64 and stored colour-major: slot k holds site site_of[k],
// the slots of one class are contiguous and the bond tables are in slot
// order with neighbours given as slots, so a class's own states, bond
// tables and its neighbours' states are read as contiguous runs.  Every random number is a Philox4x32-10 draw of the
// (site, sweep) counter, so a sweep's result does not depend on the order in
// which threads run; the cone and the acceptance counters live in device
// memory and are updated by the last workgroup of a sweep, so a whole
// schedule is queued without host round trips.  Small samples run whole
// stretches of the schedule in one workgroup with the state in LDS.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "sdc_internal.h"

namespace sdc {

namespace {

constexpr double kPi = 3.14159265358979323846;
// The accepted moves of a sweep are counted in kMcCounters counters, one per
// 128-byte line (workgroup b adds to counter b mod kMcCounters), so that the
// workgroups' atomics do not all queue on one address.  The workgroups of a
// sweep's last class also count themselves in the bits from kMcTicketBit on
// (a sweep accepts at most 2^26 moves); the one that completes its counter
// adds what it counted, and a ticket, to the line after the counters.  The
// counts thus travel in the values of the atomics alone, and no order between
// different addresses is assumed (a fence per workgroup would write back its
// L2: 280 us against 22 where the energy sum did it).
constexpr int kMcCounters = 64;
constexpr int kMcCounterStride = 16;  // u64 words between counters
constexpr int kMcTicketBit = 40;
constexpr int kMcSmallThreads = 512;  // two waves per SIMD: the update's 180 registers fit
constexpr int kMcTickets = kMcCounters * kMcCounterStride;  // word of the ticket

// a / l with r = 1 / l: the quotient's rounding error is corrected once, as a
// division does, so that several quotients share one reciprocal.
__device__ inline double quotient(double a, double l, double r) {
    const double q = a * r;
    return fma(fma(-q, l, a), r, q);
}

// Box coordinates of slot t of a class of the stencil's checkerboard: with
// L2 even the t-th site of class c is 2t or 2t + 1.  floor((2t + 1/2) / L) by
// one multiplication: the quotient is at least 1 / (2 L) away from the next
// integer and its error below 2^-26 (n <= 2^26, L <= 2^24).
struct McCell {
    int x, y, z, row, site;
};
__device__ inline McCell mc_cell(const McArgs& a, int cls, uint32_t t) {
    McCell c;
    c.row = (int)(((double)(2 * t) + 0.5) * a.inv_L2);
    c.x = (int)(((double)c.row + 0.5) * a.inv_L1);
    c.y = c.row - c.x * a.L1;
    const int dl = cls ^ ((c.x + c.y) & 1);
    c.z = (int)(2 * t) - c.row * a.L2 + dl;
    c.site = (int)(2 * t) + dl;
    return c;
}

// Bonds of one site: neighbour slots (-1 = none), couplings, DMI vectors.
template <int Z>
struct McBonds {
    int32_t j[Z];
    float J[Z], d[Z][3];
};

// STENCIL: the neighbours' slots follow from the slot by lattice arithmetic
// (McArgs::stencil), so the bond tables are not read; the bonds are the
// table's, in the table's order, so both forms give the same bits.
template <int STENCIL, int Z>
__device__ inline void mc_bonds(const McArgs& a, int cls, const McCell& c, int64_t k, McBonds<Z>& b) {
    if constexpr (STENCIL) {
        const int other = cls ? 0 : (int)(a.n / 2);  // first slot of the neighbours' class
        const int xp = c.x + 1 < a.L0 ? c.x + 1 : 0, xm = c.x > 0 ? c.x - 1 : a.L0 - 1;
        const int yp = c.y + 1 < a.L1 ? c.y + 1 : 0, ym = c.y > 0 ? c.y - 1 : a.L1 - 1;
        const int zp = c.z + 1 < a.L2 ? c.z + 1 : 0, zm = c.z > 0 ? c.z - 1 : a.L2 - 1;
        const int rxy = c.row * a.L2;  // (x L1 + y) L2
        const int sj[6] = {(xp * a.L1 + c.y) * a.L2 + c.z, (xm * a.L1 + c.y) * a.L2 + c.z,
                           (c.x * a.L1 + yp) * a.L2 + c.z, (c.x * a.L1 + ym) * a.L2 + c.z, rxy + zp, rxy + zm};
#pragma unroll
        for (int e = 0; e < 6; ++e) {
            b.j[e] = other + (sj[e] >> 1);
            b.J[e] = a.st_j;
#pragma unroll
            for (int m = 0; m < 3; ++m) b.d[e][m] = m != e / 2 ? a.st_dz : (e & 1) ? a.st_dn : a.st_dp;
        }
    } else {
#pragma unroll
        for (int e = 0; e < Z; ++e) {
            b.j[e] = a.nbr[k * Z + e];
            b.J[e] = a.jval[k * Z + e];
        }
        if (a.dvec) {
#pragma unroll
            for (int e = 0; e < Z; ++e)
#pragma unroll
                for (int m = 0; m < 3; ++m) b.d[e][m] = a.dvec[3 * (k * Z + e) + m];
        }
    }
}

// Field of a site's neighbours, sum_j (J_ij S_j + D_ij x S_j), the bonds in
// table order.  All neighbours are loaded before the first is used (read
// bond by bond, the loads of sc 128^3 waited for one another six times: see
// mc_colour_kernel).
template <int Z, class State>
__device__ inline void mc_field(const McArgs& a, const State& S, const McBonds<Z>& b, double (&w)[3]) {
    double y[Z][3];
#pragma unroll
    for (int e = 0; e < Z; ++e) {
        const int64_t j = 3 * (int64_t)(b.j[e] < 0 ? 0 : b.j[e]);
#pragma unroll
        for (int m = 0; m < 3; ++m) y[e][m] = S[j + m];
    }
    w[0] = w[1] = w[2] = 0.0;
    if (a.dvec) {
#pragma unroll
        for (int e = 0; e < Z; ++e) {
            if (b.j[e] < 0) continue;
            const double J = b.J[e], d0 = b.d[e][0], d1 = b.d[e][1], d2 = b.d[e][2];
            w[0] += J * y[e][0];
            w[1] += J * y[e][1];
            w[2] += J * y[e][2];
            w[0] += d1 * y[e][2] - d2 * y[e][1];
            w[1] += d2 * y[e][0] - d0 * y[e][2];
            w[2] += d0 * y[e][1] - d1 * y[e][0];
        }
    } else {
#pragma unroll
        for (int e = 0; e < Z; ++e) {
            if (b.j[e] < 0) continue;
            const double J = b.J[e];
            w[0] += J * y[e][0];
            w[1] += J * y[e][1];
            w[2] += J * y[e][2];
        }
    }
}

// The same for any number of bonds, one after another.
template <class State>
__device__ inline void mc_field_any(const McArgs& a, const State& S, int64_t k, double (&w)[3]) {
    w[0] = w[1] = w[2] = 0.0;
    for (int e = 0; e < a.z_max; ++e) {
        const int32_t j = a.nbr[k * a.z_max + e];
        if (j < 0) continue;
        const double J = a.jval[k * a.z_max + e];
        const double y0 = S[3 * (int64_t)j], y1 = S[3 * (int64_t)j + 1], y2 = S[3 * (int64_t)j + 2];
        w[0] += J * y0;
        w[1] += J * y1;
        w[2] += J * y2;
        if (a.dvec) {
            const float* d = a.dvec + 3 * (k * a.z_max + e);
            w[0] += (double)d[1] * y2 - (double)d[2] * y1;
            w[1] += (double)d[2] * y0 - (double)d[0] * y2;
            w[2] += (double)d[0] * y1 - (double)d[1] * y0;
        }
    }
}

template <int STENCIL, int Z, class State>
__device__ inline void mc_field_of(const McArgs& a, const State& S, int cls, const McCell& c, int64_t k,
                                   double (&w)[3]) {
    if constexpr (Z > 0) {
        McBonds<Z> b;
        mc_bonds<STENCIL, Z>(a, cls, c, k, b);
        mc_field<Z>(a, S, b, w);
    } else {
        mc_field_any(a, S, k, w);
    }
}

// One Metropolis move of site i in the field w: trial spin in a cone about s
// (cos a uniform in [cos cone, 1], azimuth uniform), acceptance at temperature
// T.  Counter = (i low, sweep low, i high, 2^31 | sweep high), key = seed:
// u_k = (w_k + 1/2) 2^-32.  Returns whether the trial spin replaced s.
__device__ inline bool mc_move(const McArgs& a, int64_t i, int64_t sweep, double T, double cos_cone,
                               const double (&w)[3], double (&s)[3]) {
    uint32_t c[4] = {(uint32_t)i, (uint32_t)sweep, (uint32_t)((uint64_t)i >> 32),
                     0x80000000u | (uint32_t)((uint64_t)sweep >> 32)};
    philox4x32_10(c, (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
    const double u0 = ((double)c[0] + 0.5) * (1.0 / 4294967296.0);
    const double u1 = ((double)c[1] + 0.5) * (1.0 / 4294967296.0);
    const double u2 = ((double)c[2] + 0.5) * (1.0 / 4294967296.0);
    const double cosa = 1.0 - u0 * (1.0 - cos_cone);
    const double sina = sqrt(fmax(0.0, 1.0 - cosa * cosa));
    double sb, cb;
    sincospi(2.0 * u1, &sb, &cb);
    // frame about s: e1 from z (x when s is near z), e2 = s x e1
    const bool near_z = fabs(s[2]) >= 0.9;
    const double ax = near_z ? 1.0 : 0.0, az = near_z ? 0.0 : 1.0;
    const double as = ax * s[0] + az * s[2];
    double e10 = ax - as * s[0], e11 = -as * s[1], e12 = az - as * s[2];
    const double l1 = sqrt(e10 * e10 + e11 * e11 + e12 * e12), r1 = 1.0 / l1;
    e10 = quotient(e10, l1, r1);
    e11 = quotient(e11, l1, r1);
    e12 = quotient(e12, l1, r1);
    const double e20 = s[1] * e12 - s[2] * e11, e21 = s[2] * e10 - s[0] * e12, e22 = s[0] * e11 - s[1] * e10;
    double t0 = cosa * s[0] + sina * (cb * e10 + sb * e20);
    double t1 = cosa * s[1] + sina * (cb * e11 + sb * e21);
    double t2 = cosa * s[2] + sina * (cb * e12 + sb * e22);
    const double lt = sqrt(t0 * t0 + t1 * t1 + t2 * t2), rt = 1.0 / lt;
    t0 = quotient(t0, lt, rt);
    t1 = quotient(t1, lt, rt);
    t2 = quotient(t2, lt, rt);
    const double dE = ((t0 - s[0]) * w[0] + (t1 - s[1]) * w[1] + (t2 - s[2]) * w[2]) -
                      a.A * (t2 * t2 - s[2] * s[2]) - a.Hz * (t2 - s[2]);
    if (!(dE <= 0.0 || u2 < exp(-dE / T))) return false;
    s[0] = t0;
    s[1] = t1;
    s[2] = t2;
    return true;
}

// Cone half-angle and its cosine before a sweep.
__device__ inline double* mc_cone(const McArgs& a, int64_t sweep) { return a.cone + 2 * (sweep & 1); }

// The cone after a sweep with the given number of accepted moves.
__device__ inline double next_cone(const McArgs& a, double c, unsigned long long acc) {
    const double rate = (double)acc / (double)a.n;
    if (rate < a.acc_target) return fmax(1e-3, 0.9 * c);
    if (rate > 2.0 * a.acc_target) return fmin(kPi, 1.1 * c);
    return c;
}

// End of the sweep's last class for one workgroup, by its first wave: `sum` (of
// lane 0) accepted moves.  The workgroup that takes the last ticket records
// the sweep's moves and adapts the cone.  The cone before sweep v is in pair
// v mod 2, so the update is to words that this sweep's workgroups do not read.
__device__ inline void mc_end_sweep(const McArgs& a, unsigned long long sum, long long* history, int64_t sweep) {
    constexpr unsigned long long kOne = 1ull << kMcTicketBit;
    const uint32_t nb = gridDim.x, line = blockIdx.x % kMcCounters;
    if (nb < kMcCounters) {
        // counters past this class's workgroups, from the launches before:
        // every workgroup completes a counter and takes its share of them
        unsigned long long rest = 0ull;
        if (threadIdx.x >= nb && threadIdx.x % nb == blockIdx.x) {
            rest = a.accepted[threadIdx.x * kMcCounterStride];
            a.accepted[threadIdx.x * kMcCounterStride] = 0ull;
        }
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) rest += __shfl_down(rest, w);
        sum += rest;
    }
    if (threadIdx.x != 0) return;
    // adds to a word (after its `total` adds cleared) and tells whether all are in
    auto add = [](unsigned long long* word, unsigned long long& v, uint32_t total) {
        v = atomicAdd(word, v + kOne) + v + kOne;
        if ((v >> kMcTicketBit) != total) return false;
        v &= kOne - 1;
        __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    };
    if (!add(a.accepted + line * kMcCounterStride, sum, (nb - line + kMcCounters - 1) / kMcCounters)) return;
    if (!add(a.accepted + kMcTickets, sum, nb < kMcCounters ? nb : kMcCounters)) return;
    if (history) history[sweep] = (long long)sum;
    const double c = next_cone(a, mc_cone(a, sweep)[0], sum);
    mc_cone(a, sweep + 1)[0] = c;
    mc_cone(a, sweep + 1)[1] = cos(c);
}

// One colour class of one sweep, one thread per site.  Bound: FP64 vector
// arithmetic (Philox, a sine and cosine, three square roots, three
// divisions, one exponential per site: about 650 vector instructions, 18 us of
// issue for the 1 048 576 sites of a class at sc 128^3), beside it the gathers.
// That class takes 20.1 us; 23.0 us when the neighbours were read bond by bond,
// with 64-bit divisions in the stencil's index arithmetic and a division per
// component.
// Workgroups go to the 8 XCDs in turn; workgroup b takes block
// x q + min(x, r) + b / 8 of the class (x = b mod 8, nb = 8 q + r blocks), so
// each XCD sweeps one contiguous stretch of slots in order and its L2 keeps
// the neighbour planes that the following slots read again.
// `last`: this is the sweep's last class, whose last workgroup adapts the cone
// (a launch of its own for that took 4.8 us per sweep).
template <int STENCIL, int Z>
__global__ __launch_bounds__(256) void mc_colour_kernel(McArgs a, int64_t k0, int64_t count, double T, int64_t sweep,
                                                        int last, long long* history) {
    const uint32_t nb = gridDim.x, q = nb / 8, r = nb % 8, x = blockIdx.x % 8;
    const uint32_t lb = x * q + (x < r ? x : r) + blockIdx.x / 8;
    const uint32_t t = lb * 256 + threadIdx.x;
    bool accepted = false;
    if (t < (uint64_t)count) {
        const int64_t k = k0 + t;  // slot
        const int cls = k0 > 0;    // of the stencil
        McCell cell{};
        if constexpr (STENCIL) cell = mc_cell(a, cls, t);
        double* si = a.S + 3 * k;
        double s[3] = {si[0], si[1], si[2]}, w[3];
        mc_field_of<STENCIL, Z>(a, a.S, cls, cell, k, w);
        accepted = mc_move(a, STENCIL ? cell.site : a.site_of[k], sweep, T, mc_cone(a, sweep)[1], w, s);
        if (accepted) {
            si[0] = s[0];
            si[1] = s[1];
            si[2] = s[2];
        }
    }
    __shared__ unsigned int wave_acc[4];
    const unsigned long long ball = __ballot(accepted);
    if ((threadIdx.x & 63) == 0) wave_acc[threadIdx.x >> 6] = (unsigned int)__popcll(ball);
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const unsigned long long sum = (unsigned long long)wave_acc[0] + wave_acc[1] + wave_acc[2] + wave_acc[3];
    if (last)
        mc_end_sweep(a, sum, history, sweep);
    else if (threadIdx.x == 0 && sum)
        atomicAdd(a.accepted + (blockIdx.x % kMcCounters) * kMcCounterStride, sum);
}

// `count` sweeps of a small sample by one workgroup, the state in LDS.  Bound:
// issue on its one CU.  A class of a 32 x 32 lattice is eight waves, two per
// SIMD, of about 700 instructions each, most of them FP64 at four cycles: 5600
// cycles, 2.3 of the 2.4 us that a class takes.  A launch per class and sweep
// end is mostly launch and memory latency: 14.4 us per sweep, 9.1 without the
// launch of the sweep's end, 4.9 in one workgroup (a whole annealing of 310
// sweeps 4.5 -> 1.5 ms).
// T and `done` (sweeps made at T) follow the schedule of the host:
// T_k = T_start cool^k while T_k > T_end, sweeps_per_T each, then T_end.
template <int STENCIL, int Z>
__global__ __launch_bounds__(kMcSmallThreads) void mc_small_kernel(McArgs a, McSmall m, long long* history) {
    extern __shared__ double S[];
    __shared__ unsigned int acc[2];
    const int tid = threadIdx.x;
    for (int x = tid; x < 3 * (int)a.n; x += kMcSmallThreads) S[x] = a.S[x];
    double T = m.T, cone = mc_cone(a, m.sweep)[0], cos_cone = mc_cone(a, m.sweep)[1];
    int64_t done = m.done;
    if (tid < 2) acc[tid] = 0;
    __syncthreads();
    for (int64_t v = 0; v < m.count; ++v) {
        const int64_t sweep = m.sweep + v;
        const double Ts = T > m.T_end ? T : m.T_end;
        for (int c = 0; c < m.n_classes; ++c) {
            const int k1 = m.class_start[c + 1];
            for (int k = m.class_start[c] + tid; k < k1; k += kMcSmallThreads) {
                double s[3] = {S[3 * k], S[3 * k + 1], S[3 * k + 2]}, w[3];
                McCell cell{};
                if constexpr (STENCIL) cell = mc_cell(a, c, (uint32_t)(k - m.class_start[c]));
                mc_field_of<STENCIL, Z>(a, S, c, cell, k, w);
                if (mc_move(a, STENCIL ? cell.site : a.site_of[k], sweep, Ts, cos_cone, w, s)) {
                    S[3 * k] = s[0];
                    S[3 * k + 1] = s[1];
                    S[3 * k + 2] = s[2];
                    atomicAdd(&acc[v & 1], 1u);
                }
            }
            __syncthreads();
        }
        // every thread follows the cone; the counter of the next sweep was
        // last read before this sweep's barriers
        const unsigned int n_acc = acc[v & 1];
        if (tid == 0) {
            if (history) history[sweep] = (long long)n_acc;
            acc[(v + 1) & 1] = 0;
        }
        cone = next_cone(a, cone, n_acc);
        cos_cone = cos(cone);
        if (T > m.T_end && ++done == m.per_T) {
            T *= m.cool;
            done = 0;
        }
        __syncthreads();
    }
    for (int x = tid; x < 3 * (int)a.n; x += kMcSmallThreads) a.S[x] = S[x];
    if (tid == 0) {
        mc_cone(a, m.sweep + m.count)[0] = cone;
        mc_cone(a, m.sweep + m.count)[1] = cos_cone;
    }
}

// The state from init (fp32, unless null), counters cleared, cone set.
__global__ __launch_bounds__(256) void mc_setup_kernel(McArgs a, const float* __restrict__ init, double cone0) {
    if (blockIdx.x == 0) {
        if (threadIdx.x < kMcCounters) a.accepted[threadIdx.x * kMcCounterStride] = 0ull;
        if (threadIdx.x == 0) {
            a.accepted[kMcTickets] = 0ull;
            mc_cone(a, 0)[0] = cone0;
            mc_cone(a, 0)[1] = cos(cone0);
        }
    }
    if (!init) return;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < a.n; k += (int64_t)gridDim.x * 256) {
        const float* x = init + 3 * (int64_t)a.site_of[k];
#pragma unroll
        for (int c = 0; c < 3; ++c) a.S[3 * k + c] = (double)x[c];
    }
}

__device__ inline double mc_block_sum(double v, double* red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    return red[0];
}

// Final state as fp32 and the energy of Eq. (1) per block: half of each site's
// bond energies, S . field (each bond is seen from both ends), plus its
// single-site terms.
template <int STENCIL, int Z>
__global__ __launch_bounds__(256) void mc_finish_kernel(McArgs a, double* __restrict__ partial,
                                                        float* __restrict__ out) {
    __shared__ double red[256];
    double e = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < a.n; k += (int64_t)gridDim.x * 256) {
        const int cls = STENCIL && k >= a.n / 2;
        McCell cell{};
        if constexpr (STENCIL) cell = mc_cell(a, cls, (uint32_t)(k - (cls ? a.n / 2 : 0)));
        const double* si = a.S + 3 * k;
        const double s[3] = {si[0], si[1], si[2]};
        double w[3];
        mc_field_of<STENCIL, Z>(a, a.S, cls, cell, k, w);
        e += 0.5 * (s[0] * w[0] + s[1] * w[1] + s[2] * w[2]) - a.A * s[2] * s[2] - a.Hz * s[2];
        float* o = out + 3 * (int64_t)(STENCIL ? cell.site : a.site_of[k]);
#pragma unroll
        for (int c = 0; c < 3; ++c) o[c] = (float)s[c];
    }
    e = mc_block_sum(e, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = e;
}

// The info block: energy per site (one workgroup: thread t sums partials t,
// t + 256, ... in order, then a fixed tree, the same result on every run),
// cone, last temperature.
__global__ __launch_bounds__(256) void mc_info_kernel(McArgs a, const double* __restrict__ partial, int n_partial,
                                                      int64_t n_sweeps, double T_last, double* __restrict__ info) {
    __shared__ double red[256];
    double e = 0.0;
    for (int b = threadIdx.x; b < n_partial; b += 256) e += partial[b];
    e = mc_block_sum(e, red);
    if (threadIdx.x != 0) return;
    info[0] = e / (double)a.n;
    info[1] = mc_cone(a, n_sweeps)[0];
    info[2] = T_last;
}

unsigned grid_of(int64_t n) {
    int64_t b = (n + 255) / 256;
    return (unsigned)(b > 4096 ? 4096 : (b < 1 ? 1 : b));
}

// Calls f(STENCIL, Z) with the constants of the sample.
template <class F>
void mc_dispatch(const McArgs& a, F f) {
    if (a.stencil) f(std::integral_constant<int, 1>{}, std::integral_constant<int, 6>{});
    else if (a.z_max == 6) f(std::integral_constant<int, 0>{}, std::integral_constant<int, 6>{});
    else if (a.z_max == 8) f(std::integral_constant<int, 0>{}, std::integral_constant<int, 8>{});
    else f(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
}

}  // namespace

int mc_energy_blocks(int64_t n) { return (int)grid_of(n); }

size_t mc_counter_bytes() { return (size_t)(kMcCounters + 1) * kMcCounterStride * sizeof(unsigned long long); }

int launch_mc_setup(const McArgs& a, const float* init, double cone0, void* stream) {
    hipLaunchKernelGGL(mc_setup_kernel, dim3(init ? grid_of(a.n) : 1), dim3(256), 0, (hipStream_t)stream, a, init,
                       cone0);
    return (int)hipGetLastError();
}

int launch_mc_sweep(const McArgs& a, const int64_t* class_start, int n_classes, double T, int64_t sweep,
                    long long* history, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    mc_dispatch(a, [&](auto stencil, auto z) {
        for (int c = 0; c < n_classes; ++c) {
            const int64_t count = class_start[c + 1] - class_start[c];  // at least one site
            const unsigned grid = (unsigned)((count + 255) / 256);
            hipLaunchKernelGGL((mc_colour_kernel<decltype(stencil)::value, decltype(z)::value>), dim3(grid), dim3(256),
                               0, s, a, class_start[c], count, T, sweep, c == n_classes - 1 ? 1 : 0, history);
        }
    });
    return (int)hipGetLastError();
}

bool mc_is_small(int64_t n, const int64_t* class_start, int n_classes) {
    if (n > kMcSmallSites || n_classes > kMcSmallClasses) return false;
    for (int c = 0; c < n_classes; ++c)
        if (class_start[c + 1] - class_start[c] > kMcSmallClassSites) return false;
    return true;
}

int prepare_mc_small(const McArgs& a) {
    int e = 0;
    mc_dispatch(a, [&](auto stencil, auto z) {
        e = (int)hipFuncSetAttribute(
            (const void*)mc_small_kernel<decltype(stencil)::value, decltype(z)::value>,
            hipFuncAttributeMaxDynamicSharedMemorySize, kMcSmallSites * 3 * (int)sizeof(double));
    });
    return e;
}

int launch_mc_small(const McArgs& a, const McSmall& m, long long* history, void* stream) {
    const size_t lds = (size_t)a.n * 3 * sizeof(double);
    mc_dispatch(a, [&](auto stencil, auto z) {
        hipLaunchKernelGGL((mc_small_kernel<decltype(stencil)::value, decltype(z)::value>), dim3(1),
                           dim3(kMcSmallThreads), lds, (hipStream_t)stream, a, m, history);
    });
    return (int)hipGetLastError();
}

int launch_mc_finish(const McArgs& a, double* partial, int64_t n_sweeps, double T_last, float* out, double* info,
                     void* stream) {
    mc_dispatch(a, [&](auto stencil, auto z) {
        hipLaunchKernelGGL((mc_finish_kernel<decltype(stencil)::value, decltype(z)::value>), dim3(grid_of(a.n)),
                           dim3(256), 0, (hipStream_t)stream, a, partial, out);
    });
    hipLaunchKernelGGL(mc_info_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream, a, (const double*)partial,
                       (int)grid_of(a.n), n_sweeps, T_last, info);
    return (int)hipGetLastError();
}

}  // namespace sdc
