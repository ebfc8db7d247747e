// Landau-Lifshitz RK4 (Eq. (2), Sec. 3.1) with Philox4x32-10 starts, on gfx950.
#include <hip/hip_runtime.h>

#include "sdc_internal.h"

namespace sdc {

namespace {

__global__ __launch_bounds__(256) void traj_init_kernel(TrajArgs a) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n) return;
    double x, y, z;
    if (a.init == SDC_INIT_GIVEN) {
        x = a.init_dev[3 * i];
        y = a.init_dev[3 * i + 1];
        z = a.init_dev[3 * i + 2];
    } else {
        uint32_t c[4] = {(uint32_t)i, 0u, (uint32_t)((uint64_t)i >> 32), 0u};
        philox4x32_10(c, (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
        const double u0 = (double)(c[0] >> 8) * (1.0 / 16777216.0);
        const double u1 = (double)(c[1] >> 8) * (1.0 / 16777216.0);
        if (a.init == SDC_INIT_UNIFORM) {
            z = 2.0 * u0 - 1.0;
            const double r = sqrt(fmax(0.0, 1.0 - z * z));
            double sn, cs;
            sincospi(2.0 * u1, &sn, &cs);
            x = r * cs;
            y = r * sn;
        } else {
            const double rr = sqrt(-2.0 * log(1.0 - u0));
            double sn, cs;
            sincospi(2.0 * u1, &sn, &cs);
            const double v0 = a.sigma * rr * cs, v1 = a.sigma * rr * sn;
            const double ang = sqrt(v0 * v0 + v1 * v1);
            const double f = ang > 0.0 ? sin(ang) / ang : 1.0;
            x = f * v0;
            y = f * v1;
            z = cos(ang);
        }
    }
    a.frames[3 * i] = (float)x;
    a.frames[3 * i + 1] = (float)y;
    a.frames[3 * i + 2] = (float)z;
}

// Adds bond (J, d) to the neighbour spin y into the field h.
__device__ inline void add_bond(float (&h)[3], float J, const float (&d)[3], bool dmi, float y0, float y1, float y2) {
    h[0] += J * y0;
    h[1] += J * y1;
    h[2] += J * y2;
    if (dmi) {
        h[0] += d[1] * y2 - d[2] * y1;
        h[1] += d[2] * y0 - d[0] * y2;
        h[2] += d[0] * y1 - d[1] * y0;
    }
}

// k = h x x with the field h of the bonds and the single-site terms of Eq. (1).
__device__ inline void rate(const TrajArgs& a, float (&h)[3], const float (&x)[3], float (&k)[3]) {
    h[2] += -a.aniso2 * x[2] - a.hz;
    k[0] = h[1] * x[2] - h[2] * x[1];
    k[1] = h[2] * x[0] - h[0] * x[2];
    k[2] = h[0] * x[1] - h[1] * x[0];
}

// One RK4 stage with bond tables: k = h_i x X_i with the effective field of
// Eq. (1), h_i = sum_j (J_ij X_j + D_ij x X_j) - 2 A X_i^z z - H_z z.
//  stage 0: acc = k;      Tout = S + dt/2 k
//  stage 1: acc += 2k;    Tout = S + dt/2 k
//  stage 2: acc += 2k;    Tout = S + dt k
//  stage 3: frame = S + dt/6 (acc + k)
// Bound: latency (a launch, the table entries, then the neighbours).  Z: bonds
// per site (0: any number).  The entries of Z bonds, or of four at a time, are
// loaded together, then their neighbours, before the first use (20 011 points
// with about 160 bonds each: 370 us per step, 421 bond by bond; 3001 points
// with about 10: 44.8 and 51.8).
template <int Z>
__global__ __launch_bounds__(256) void traj_stage_kernel(TrajArgs a, int stage, const float* __restrict__ S,
                                                         const float* __restrict__ X, float* __restrict__ Tout,
                                                         float* __restrict__ acc, float* __restrict__ frame) {
    constexpr int B = Z > 0 ? Z : 4;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= a.n) return;
    float h[3] = {0.f, 0.f, 0.f};
    const float x[3] = {X[3 * i], X[3 * i + 1], X[3 * i + 2]};
    const int z = Z > 0 ? Z : a.z_max;
    for (int e0 = 0; e0 < z; e0 += B) {
        int32_t j[B];
        float J[B], y[B][3], d[B][3];
#pragma unroll
        for (int e = 0; e < B; ++e) {
            const bool in = Z > 0 || e0 + e < z;
            const int64_t b = i * z + (in ? e0 + e : z - 1);
            j[e] = a.nbr[b];
            J[e] = a.jval[b];
            d[e][0] = d[e][1] = d[e][2] = 0.f;
            if (!in) j[e] = -1;
        }
        if (a.dvec) {
#pragma unroll
            for (int e = 0; e < B; ++e)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    d[e][c] = a.dvec[3 * (i * z + (Z > 0 || e0 + e < z ? e0 + e : z - 1)) + c];
        }
#pragma unroll
        for (int e = 0; e < B; ++e) {
            const int64_t k = 3 * (int64_t)(j[e] < 0 ? 0 : j[e]);
#pragma unroll
            for (int c = 0; c < 3; ++c) y[e][c] = X[k + c];
        }
#pragma unroll
        for (int e = 0; e < B; ++e)
            if (j[e] >= 0) add_bond(h, J[e], d[e], a.dvec != nullptr, y[e][0], y[e][1], y[e][2]);
    }
    float k[3];
    rate(a, h, x, k);
    const float c = stage == 3 ? a.dt / 6.0f : stage == 2 ? a.dt : 0.5f * a.dt;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const float s = S[3 * i + m];
        if (stage == 0) acc[3 * i + m] = k[m];
        else if (stage < 3) acc[3 * i + m] += 2.f * k[m];
        if (stage < 3) Tout[3 * i + m] = s + c * k[m];
        else frame[3 * i + m] = s + c * (acc[3 * i + m] + k[m]);
    }
}

// One whole RK4 step of a periodic sc box with one uniform coupling, sites in
// the order (x L1 + y) L2 + z: a workgroup takes a brick of b0 x b1 x b2 cells,
// loads it with a halo of four cells and runs the four stages in LDS, each on
// one layer less, so the steps of all bricks are independent and a frame is one
// launch that reads the previous frame.  An axis that the brick spans needs no
// halo: its bonds wrap inside the tile (WRAP; of an axis of one cell they close
// on the site itself and are dropped).  With a halo there, 40 000 x 2 x 2 cells
// took 64.8 us per step (the table launches 25.3) and 3 x 300 x 300 31.7 (36.7),
// now 8.2 and 13.1.  Every halo cell computes what its owner computes, in the
// same order.  Bound: latency (the
// launch, the load of the tile, four short stages); the redundant stages (10x
// the sites' own for bricks of 4^3, 12 for 8^3) are what the idle chip is
// there for.  The four table launches of a frame took 23.5 us at 20 x 22 x 24
// cells with DMI, this one 7.2 (256 threads 9.9, 512 threads 7.8); without DMI
// at 36^3 9.5 us.
constexpr int kStepThreads = 1024;
constexpr int kStepHalo = 4;

// q = floor(i / d) for 0 <= i < 2^20 with inv = 1 / d: (i + 1/2) / d is at least
// 1 / (2 d) away from an integer, far more than the product's rounding.
__device__ inline int div_small(int i, float inv) { return (int)(((float)i + 0.5f) * inv); }

template <int DMI, int WRAP>
__global__ __launch_bounds__(kStepThreads) void traj_step_kernel(TrajArgs a, TrajBrick b, const float* __restrict__ prev,
                                                                 float* __restrict__ frame) {
    extern __shared__ float tile[];  // S, two stage buffers: [3][cells] each; acc [3][brick cells]
    const int cells = b.t[0] * b.t[1] * b.t[2];
    float* const S = tile;
    float* const acc = tile + 9 * cells;
    const int own = b.b[0] * b.b[1] * b.b[2];
    int start[3];
    {
        const int k2 = blockIdx.x % b.nb[2], k01 = blockIdx.x / b.nb[2];
        const int k1 = k01 % b.nb[1], k0 = k01 / b.nb[1];
        start[0] = k0 * b.b[0];
        start[1] = k1 * b.b[1];
        start[2] = k2 * b.b[2];
    }
    const float it1 = 1.0f / (float)b.t[1], it2 = 1.0f / (float)b.t[2];
    const float iL[3] = {1.0f / (float)b.L[0], 1.0f / (float)b.L[1], 1.0f / (float)b.L[2]};
#pragma unroll 4
    for (int x = threadIdx.x; x < cells; x += kStepThreads) {
        const int row = div_small(x, it2), i2 = x - row * b.t[2];
        const int i0 = div_small(row, it1), i1 = row - i0 * b.t[1];
        const int i[3] = {i0, i1, i2};
        int g[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            // the box coordinate of the tile's cell, wrapped (the shift by 4 L
            // keeps it positive for every edge)
            const int v = start[c] + i[c] - b.halo[c] + kStepHalo * b.L[c];
            g[c] = v - div_small(v, iL[c]) * b.L[c];
        }
        const float* p = prev + 3 * (((int64_t)g[0] * b.L[1] + g[1]) * b.L[2] + g[2]);
#pragma unroll
        for (int c = 0; c < 3; ++c) S[c * cells + x] = p[c];
    }
    __syncthreads();
    const int step[3] = {b.t[1] * b.t[2], b.t[2], 1};
#pragma unroll
    for (int stage = 0; stage < 4; ++stage) {
        const float* X = stage == 0 ? S : tile + (stage == 2 ? 6 : 3) * cells;  // stage 1: first, 2: second, 3: first
        float* Tout = tile + (stage == 1 ? 6 : 3) * cells;
        int lo[3], e[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            lo[c] = b.halo[c] ? stage + 1 : 0;
            e[c] = b.t[c] - 2 * lo[c];
        }
        const float ie1 = 1.0f / (float)e[1], ie2 = 1.0f / (float)e[2];
        const int n = e[0] * e[1] * e[2];
        for (int x = threadIdx.x; x < n; x += kStepThreads) {
            const int row = div_small(x, ie2), i2 = x - row * e[2] + lo[2];
            const int r0 = div_small(row, ie1), i0 = r0 + lo[0], i1 = row - r0 * e[1] + lo[1];
            const int at = (i0 * b.t[1] + i1) * b.t[2] + i2;
            float h[3] = {0.f, 0.f, 0.f}, k[3];
            const float v[3] = {X[at], X[cells + at], X[2 * cells + at]};
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                if (b.L[ax] == 1) continue;
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    int j = s == 0 ? at + step[ax] : at - step[ax];
                    if (WRAP && !b.halo[ax]) {
                        const int i = ax == 0 ? i0 : ax == 1 ? i1 : i2, around = b.L[ax] * step[ax];
                        if (s == 0 && i == b.L[ax] - 1) j -= around;
                        if (s == 1 && i == 0) j += around;
                    }
                    float d[3] = {b.dz, b.dz, b.dz};
                    d[ax] = s == 0 ? b.dp : b.dn;
                    add_bond(h, b.J, d, DMI != 0, X[j], X[cells + j], X[2 * cells + j]);
                }
            }
            rate(a, h, v, k);
            const int o[3] = {i0 - b.halo[0], i1 - b.halo[1], i2 - b.halo[2]};
            const bool mine = (unsigned)o[0] < (unsigned)b.b[0] && (unsigned)o[1] < (unsigned)b.b[1] &&
                              (unsigned)o[2] < (unsigned)b.b[2];
            const int q = (o[0] * b.b[1] + o[1]) * b.b[2] + o[2];
            const float c = stage == 3 ? a.dt / 6.0f : stage == 2 ? a.dt : 0.5f * a.dt;
            if (stage < 3) {
#pragma unroll
                for (int m = 0; m < 3; ++m) {
                    if (mine) acc[m * own + q] = stage == 0 ? k[m] : acc[m * own + q] + 2.f * k[m];
                    Tout[m * cells + at] = S[m * cells + at] + c * k[m];
                }
            } else {
                const int g[3] = {start[0] + o[0], start[1] + o[1], start[2] + o[2]};
                if (g[0] < b.L[0] && g[1] < b.L[1] && g[2] < b.L[2]) {  // the last brick of an axis may reach past it
                    float* f = frame + 3 * (((int64_t)g[0] * b.L[1] + g[1]) * b.L[2] + g[2]);
#pragma unroll
                    for (int m = 0; m < 3; ++m) f[m] = S[m * cells + at] + c * (acc[m * own + q] + k[m]);
                }
            }
        }
        __syncthreads();
    }
}

int64_t step_lds(const TrajBrick& b) {
    return (9 * (int64_t)b.t[0] * b.t[1] * b.t[2] + 3 * (int64_t)b.b[0] * b.b[1] * b.b[2]) * (int64_t)sizeof(float);
}

constexpr int64_t kStepMaxLds = 156 * 1024;
// Longest axis that a brick may span beside longer ones (16^3 cells fit LDS).
constexpr int kStepShort = 16;

// Brick of the box: the smallest number of stage evaluations (and half that
// for a tile cell loaded) that a compute unit works through, its rounds over
// `n_cu` of them counted.
TrajBrick choose_brick(const TrajArgs& a, int n_cu) {
    TrajBrick best{}, b{};
    double best_cost = -1.0;
    int axes = 0;
    for (int c = 0; c < 3; ++c) axes += a.L[c] > kStepShort;
    const int most = axes >= 3 ? kStepShort : axes == 2 ? 64 : 512;
    b.J = a.st_j;
    b.dp = a.st_dp;
    b.dn = a.st_dn;
    b.dz = a.st_dz;
    for (int c = 0; c < 3; ++c) b.L[c] = a.L[c];
    auto set = [&](int c, int cells) {
        b.b[c] = cells;
        b.nb[c] = (a.L[c] + cells - 1) / cells;
        b.halo[c] = cells < a.L[c] ? kStepHalo : 0;
        b.t[c] = cells + 2 * b.halo[c];
    };
    // a long axis takes 1 .. `most` cells; a short one beside long ones is
    // spanned, and otherwise takes any number
    auto first = [&](int c) { return axes > 0 && a.L[c] <= kStepShort ? a.L[c] : 1; };
    auto last = [&](int c) { return a.L[c] < most ? a.L[c] : most; };
    for (int b0 = first(0); b0 <= last(0); ++b0) {
        set(0, b0);
        for (int b1 = first(1); b1 <= last(1); ++b1) {
            set(1, b1);
            for (int b2 = first(2); b2 <= last(2); ++b2) {
                set(2, b2);
                if (step_lds(b) > kStepMaxLds) continue;  // a spanned axis needs less than one nearly spanned
                double groups = 1.0, cells = 1.0, evals = 0.0;
                for (int c = 0; c < 3; ++c) {
                    groups *= b.nb[c];
                    cells *= b.t[c];
                }
                for (int s = 1; s <= 4; ++s) {
                    double e = 1.0;
                    for (int c = 0; c < 3; ++c) e *= b.halo[c] ? b.t[c] - 2 * s : b.t[c];
                    evals += e;
                }
                const double rounds = (double)((int64_t)((groups + n_cu - 1) / n_cu));
                const double cost = rounds * (evals + 0.5 * cells + 500.0);
                if (best_cost < 0.0 || cost < best_cost) {
                    best_cost = cost;
                    best = b;
                }
            }
        }
    }
    return best;
}

template <int Z>
void launch_stages(const TrajArgs& a, hipStream_t s) {
    const unsigned grid = (unsigned)((a.n + 255) / 256);
    float* T1 = a.work;
    float* T2 = a.work + 3 * a.n;
    float* acc = a.work + 6 * a.n;
    for (int64_t f = 1; f < a.n_frames; ++f) {
        const float* S = a.frames + (f - 1) * a.n * 3;
        float* frame = a.frames + f * a.n * 3;
        const float* X[4] = {S, T1, T2, T1};
        float* T[4] = {T1, T2, T1, T2};
        for (int stage = 0; stage < 4; ++stage)
            hipLaunchKernelGGL(traj_stage_kernel<Z>, dim3(grid), dim3(256), 0, s, a, stage, S, X[stage], T[stage], acc,
                               frame);
    }
}

}  // namespace

int launch_traj(const TrajArgs& a, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(traj_init_kernel, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, s, a);
    if (a.n_frames > 1 && a.stencil) {
        int dev = 0, n_cu = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1)
            n_cu = 256;
        const TrajBrick b = choose_brick(a, n_cu);
        bool wrap = false;
        for (int c = 0; c < 3; ++c) wrap |= b.L[c] > 1 && !b.halo[c];
        const void* fn = wrap ? (a.st_dmi ? (const void*)traj_step_kernel<1, 1> : (const void*)traj_step_kernel<0, 1>)
                              : (a.st_dmi ? (const void*)traj_step_kernel<1, 0> : (const void*)traj_step_kernel<0, 0>);
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kStepMaxLds);
        if (e != hipSuccess) return (int)e;
        for (int64_t f = 1; f < a.n_frames; ++f) {
            const float* prev = a.frames + (f - 1) * a.n * 3;
            float* frame = a.frames + f * a.n * 3;
            void* params[] = {(void*)&a, (void*)&b, (void*)&prev, (void*)&frame};
            e = hipLaunchKernel(fn, dim3((unsigned)(b.nb[0] * b.nb[1] * b.nb[2])), dim3(kStepThreads), params,
                                (size_t)step_lds(b), s);
            if (e != hipSuccess) return (int)e;
        }
    } else if (a.n_frames > 1) {
        if (a.z_max == 6) launch_stages<6>(a, s);
        else if (a.z_max == 8) launch_stages<8>(a, s);
        else launch_stages<0>(a, s);
    }
    return (int)hipGetLastError();
}

}  // namespace sdc
