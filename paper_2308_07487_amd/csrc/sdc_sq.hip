// q-resolved dynamic structure factor, Eq. (3), at arbitrary wave vectors for
// any point set (lattice or not), on gfx950.
//
// The phase of a pair factorises, exp(-i q.(r_j - r_i)) = conj(e_i) e_j with
// e_j(q) = exp(-i q.r_j), so the double sum over pairs in Eq. (3) becomes
//     S(q, t) = (1 / (N n_o)) sum_o sum_a conj(F_a(q, o s)) F_a(q, o s + t),
//     F_a(q, f) = sum_j e_j(q) S_j^a(f),
// the dense contraction of the phase matrix [n_q x N] with the spin matrix
// [N x 3T] (FP64 MFMA, phases computed on the fly as in the on-the-fly Q of
// Sec. 3.4 but per site instead of per pair), followed by a short
// correlation over the origins.  The connected form (Eq. (4) with its second
// term, i.e. Eq. (5)) centres the origin side: F_a(q, o s) minus its average
// over the origins, which is the transform of the per-site averages.
#include <hip/hip_runtime.h>

#include "sdc_internal.h"

namespace sdc {

typedef double f64x4 __attribute__((ext_vector_type(4)));

namespace {

// sin and cos of x in FP64 for |x| < 2^20, without branches: Cody-Waite
// reduction x = k pi/2 + r with pi/2 in two parts (FMA), Taylor polynomials
// of sin r and cos r on |r| <= pi/4 (terms to r^15 and r^16; the first left
// out is below 1e-16), and the quadrant k mod 4 choosing and signing them.
// Absolute error a few 1e-16, a quarter of the library routine's work.
__device__ inline void sincos_small(double x, double* s, double* c) {
    const double two_over_pi = 0x1.45f306dc9c883p-1;
    const double pio2_hi = 0x1.921fb54442d18p+0;   // pi/2 rounded to double
    const double pio2_lo = 0x1.1a62633145c07p-54;  // pi/2 - pio2_hi, rounded
    const double k = rint(x * two_over_pi);
    const double r = fma(-k, pio2_lo, fma(-k, pio2_hi, x));
    const double r2 = r * r;
    double ps = -1.0 / 1307674368000.0;            // -1/15!
    ps = fma(ps, r2, 1.0 / 6227020800.0);          //  1/13!
    ps = fma(ps, r2, -1.0 / 39916800.0);           // -1/11!
    ps = fma(ps, r2, 1.0 / 362880.0);              //  1/9!
    ps = fma(ps, r2, -1.0 / 5040.0);               // -1/7!
    ps = fma(ps, r2, 1.0 / 120.0);                 //  1/5!
    ps = fma(ps, r2, -1.0 / 6.0);                  // -1/3!
    const double sn = fma(ps * r2, r, r);
    double pc = 1.0 / 20922789888000.0;            //  1/16!
    pc = fma(pc, r2, -1.0 / 87178291200.0);        // -1/14!
    pc = fma(pc, r2, 1.0 / 479001600.0);           //  1/12!
    pc = fma(pc, r2, -1.0 / 3628800.0);            // -1/10!
    pc = fma(pc, r2, 1.0 / 40320.0);               //  1/8!
    pc = fma(pc, r2, -1.0 / 720.0);                // -1/6!
    pc = fma(pc, r2, 1.0 / 24.0);                  //  1/4!
    pc = fma(pc, r2, -0.5);                        // -1/2!
    const double cs = fma(pc, r2, 1.0);
    // quadrant: (sin, cos)(k pi/2 + r) = (sn, cs), (cs, -sn), (-sn, -cs), (-cs, sn)
    const int q = (int)((long long)k & 3);
    const double s0 = (q & 1) ? cs : sn;
    const double c0 = (q & 1) ? sn : cs;
    *s = (q & 2) ? -s0 : s0;
    *c = ((q + 1) & 2) ? -c0 : c0;
}

constexpr int kSqQBlocks = 4;               // 16-row wave-vector blocks per workgroup
constexpr int kSqColParts = 3;              // column ranges per wave-vector block
constexpr int kSqWaves = kSqQBlocks * kSqColParts;  // consumer waves (MFMA), three per SIMD
constexpr int kSqProdWaves = 4;             // producer waves, one per SIMD
constexpr int kSqThreads = 64 * (kSqWaves + kSqProdWaves);
constexpr int kSqQ = 16 * kSqQBlocks;       // wave vectors per workgroup
constexpr int kSqSites = 24;                // sites per chunk (6 MFMA K-steps of 4)
constexpr int kSqCB = 12;                   // 16-column blocks per workgroup
constexpr int kSqCBW = kSqCB / kSqColParts;   // 16-column blocks per consumer wave
constexpr int kSqCols = kSqCB * 16;         // 192 spin-matrix columns = 64 whole frames
constexpr int kSqFrames = kSqCols / 3;
constexpr int kSqPitch = 3 * kSqSites + 4;  // LDS doubles per staged frame (padded against bank conflicts)
constexpr int kSqPhBuf = 2 * kSqSites * kSqQ;    // doubles of one phase buffer (cos, -sin)
constexpr int kSqSbBuf = kSqFrames * kSqPitch;   // doubles of one spin buffer
constexpr int kSqLdsBytes = 2 * (kSqPhBuf + kSqSbBuf) * (int)sizeof(double);
static_assert(kSqCols % 3 == 0, "a column range must cover whole frames");
static_assert(kSqCB % kSqColParts == 0 && kSqSites % 4 == 0, "consumer split");
static_assert(kSqLdsBytes <= 160 * 1024, "two chunk buffers must fit in LDS");

constexpr int kSqProducers = 64 * kSqProdWaves;
constexpr int kSqRow = 3 * kSqSites;                      // spin values of a frame in a chunk
constexpr int kSqPhPer = kSqSites * kSqQ / kSqProducers;  // phases per producer thread
constexpr int kSqQuads = kSqFrames * kSqRow / 4;          // 4-value groups of a block's chunk
constexpr int kSqSbPer = (kSqQuads + kSqProducers - 1) / kSqProducers;  // of them per producer thread
static_assert(kSqPhPer * kSqProducers == kSqSites * kSqQ && kSqProducers % 64 == 0 && kSqQ == 64, "phase split");
static_assert(kSqRow % 4 == 0 && kSqPitch % 2 == 0, "16-byte rows");

// Producer side.  Producer wave w keeps a wave vector per lane (qv, zero past
// n_q) and takes the sites w + 4 i of a chunk, whose positions are then one
// scalar load for the wave; the chunk's spins of 64 frames are one contiguous
// block of the packed spins.  The inputs of a chunk are loaded into registers
// one chunk ahead (sq_load) and turned into an LDS buffer (sq_store) while the
// next ones are on their way.  No load is conditional: indices are clamped
// and the phases masked (loads under a condition became branches with a wait
// each, twelve in a row for the positions alone).
struct SqInputs {
    float pos[kSqPhPer][3];
    float4 spin[kSqSbPer];
};

__device__ __forceinline__ void sq_load(const SqTransformArgs& a, int ptid, int64_t f_first, int64_t j0, int64_t je,
                                        SqInputs& in) {
    const int w = __builtin_amdgcn_readfirstlane(ptid >> 6);
#pragma unroll
    for (int i = 0; i < kSqPhPer; ++i) {
        int64_t j = j0 + w + kSqProdWaves * i;
        j = j < je ? j : je - 1;
#pragma unroll
        for (int c = 0; c < 3; ++c) in.pos[i][c] = a.pos[3 * j + c];
    }
    const float4* src = (const float4*)(a.packed + ((j0 / kSqSites) * a.t_pad + f_first) * kSqRow);
#pragma unroll
    for (int i = 0; i < kSqSbPer; ++i) {
        int e = ptid + kSqProducers * i;
        if (kSqProducers * (i + 1) > kSqQuads) e = e < kSqQuads ? e : kSqQuads - 1;
        in.spin[i] = src[e];
    }
}

__device__ __forceinline__ void sq_store(int ptid, const double (&qv)[3], int64_t j0, int64_t je, const SqInputs& in,
                                         double* __restrict__ ph, double* __restrict__ sb) {
#pragma unroll
    for (int i = 0; i < kSqPhPer; ++i) {
        const bool valid = j0 + (ptid >> 6) + kSqProdWaves * i < je;
        const double th = qv[0] * (double)in.pos[i][0] + qv[1] * (double)in.pos[i][1] + qv[2] * (double)in.pos[i][2];
        double sn, cs;
        sincos_small(th, &sn, &cs);
        const int e = ptid + kSqProducers * i;  // = site * 64 + wave vector
        ph[e] = valid ? cs : 0.0;                    // Re exp(-i q.r), [site][q]
        ph[kSqSites * kSqQ + e] = valid ? -sn : 0.0;  // Im exp(-i q.r)
    }
#pragma unroll
    for (int i = 0; i < kSqSbPer; ++i) {
        const int e = ptid + kSqProducers * i;
        if (kSqProducers * (i + 1) > kSqQuads && e >= kSqQuads) continue;
        const int fl = e / (kSqRow / 4), r = 4 * (e - fl * (kSqRow / 4));
        double2* dst = (double2*)(sb + fl * kSqPitch + r);
        dst[0] = make_double2((double)in.spin[i].x, (double)in.spin[i].y);
        dst[1] = make_double2((double)in.spin[i].z, (double)in.spin[i].w);
    }
}

// Packed spins for the contraction: P[c][f][s][a] = S_j^a(f), j = 24 c + s,
// fp32 as they come, zero for sites past N and frames past n_frames_used
// (t_pad frames per chunk, a multiple of 64), so that a block's 64 frames are
// one contiguous block.  Bound: HBM, 12 B read and 12 B written per site and
// frame.  A thread takes one value of 8 frames.
constexpr int kSqPackFrames = 8;
__global__ __launch_bounds__(256) void sq_pack_kernel(SqTransformArgs a) {
    const int64_t n_chunks = (a.n + kSqSites - 1) / kSqSites, per_frame = n_chunks * kSqRow;
    const int64_t f0 = (int64_t)blockIdx.y * kSqPackFrames;
    for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x < per_frame; x += (int64_t)gridDim.x * 256) {
        const int64_t ch = x / kSqRow;
        const int r = (int)(x - ch * kSqRow);
        const bool in = x < 3 * a.n;  // value x of a frame is component x % 3 of site x / 3
        float v[kSqPackFrames];
#pragma unroll
        for (int k = 0; k < kSqPackFrames; ++k) {
            const int64_t f = f0 + k < a.n_frames_used ? f0 + k : a.n_frames_used - 1;
            v[k] = a.frames[f * a.n * 3 + (in ? x : 0)];
        }
#pragma unroll
        for (int k = 0; k < kSqPackFrames; ++k)
            a.packed[(ch * a.t_pad + f0 + k) * kSqRow + r] = in && f0 + k < a.n_frames_used ? v[k] : 0.0f;
    }
}

// One workgroup: 64 wave vectors x 192 columns (64 frames x 3 components) x
// one range of sites, in chunks of 24 sites with two LDS buffers.  Four
// producer waves fill the next chunk's buffer (64 x 24 phases, cos and -sin
// of q.r in FP64, and the spins) while twelve consumer waves, three per SIMD so
// that one issues MFMAs while the others wait, run the current chunk:
// consumer w takes wave vectors 16 (w % 4) .. +15 and column blocks
// 4 (w / 4) .. +3 through 6 K-steps of 4 sites, two FP64 MFMAs (real and
// imaginary phase rows) per 16-column block sharing the spin operand.  One
// barrier per chunk.  Spins are read from memory once per 64 wave vectors and
// each phase is computed once per 192 columns (the FP64 vector work of the
// phases takes issue cycles from the FP64 MFMAs).  Bound: FP64 MFMA; 1024
// wave vectors x 65 536 points x 573 columns (1.54e11 flops) take 2.9 ms
// against 2.0 at the matrix cores' 77.8 TFLOP/s, 3.5 when the producers waited
// for each of their loads; without producers the consumers alone take 2.3.  The
// partial transform of the site range goes to its own slice of `part` (no
// atomics; the slices are summed in a fixed order).
__global__ __launch_bounds__(kSqThreads, 1) void sq_transform_kernel(SqTransformArgs a) {
    extern __shared__ double lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool producer = wave >= kSqWaves;
    const int q0 = blockIdx.x * kSqQ;
    const int64_t f_first = (int64_t)blockIdx.y * kSqFrames;
    const int64_t c0 = 3 * f_first;
    const int64_t n_cols = 3 * (int64_t)a.n_frames_used;
    const int64_t jb = (int64_t)blockIdx.z * a.sites_per_split;
    const int64_t je = jb + a.sites_per_split < a.n ? jb + a.sites_per_split : a.n;
    // Producer and consumer waves run separate loops with the same barrier
    // count (one before the first chunk, one per chunk), so the consumers'
    // accumulators are not live in the producers' code.
    if (producer) {
        // ahead of the consumers, whose matrix instructions keep the SIMD busy
        // anyway (3.20 against 3.29 ms for 1024 wave vectors x 65 536 points)
        __builtin_amdgcn_s_setprio(3);
        const int ptid = tid - 64 * kSqWaves;
        double qv[3] = {0.0, 0.0, 0.0};  // zero past n_q: rows nobody stores
        if (q0 + ptid % kSqQ < a.n_q) {
            qv[0] = a.q[3 * (q0 + ptid % kSqQ)];
            qv[1] = a.q[3 * (q0 + ptid % kSqQ) + 1];
            qv[2] = a.q[3 * (q0 + ptid % kSqQ) + 2];
        }
        SqInputs in;
        sq_load(a, ptid, f_first, jb, je, in);
        sq_store(ptid, qv, jb, je, in, lds, lds + 2 * kSqPhBuf);
        sq_load(a, ptid, f_first, jb + kSqSites < je ? jb + kSqSites : jb, je, in);
        __syncthreads();
        int nxt = 1;
        for (int64_t j0 = jb; j0 < je; j0 += kSqSites) {
            const int64_t j1 = j0 + kSqSites, j2 = j1 + kSqSites;
            if (j1 < je) {
                sq_store(ptid, qv, j1, je, in, lds + nxt * kSqPhBuf, lds + 2 * kSqPhBuf + nxt * kSqSbBuf);
                sq_load(a, ptid, f_first, j2 < je ? j2 : j1, je, in);
            }
            __syncthreads();  // the consumers are done with the other buffer
            nxt ^= 1;
        }
        return;
    }
    const int qb = wave % kSqQBlocks, cb0 = (wave / kSqQBlocks) * kSqCBW;
    const bool active = q0 + 16 * qb < a.n_q;  // wave-uniform
    // LDS offset of this lane's column in each block (frame row, component)
    int boff[kSqCBW];
#pragma unroll
    for (int b = 0; b < kSqCBW; ++b) {
        const int c = (cb0 + b) * 16 + (lane & 15);
        boff[b] = (c / 3) * kSqPitch + c % 3;
    }
    f64x4 acc_re[kSqCBW], acc_im[kSqCBW];
#pragma unroll
    for (int b = 0; b < kSqCBW; ++b) {
        acc_re[b] = f64x4{0.0, 0.0, 0.0, 0.0};
        acc_im[b] = f64x4{0.0, 0.0, 0.0, 0.0};
    }
    // this lane's first phase and spin in a buffer: A[i][k] = phase of wave
    // vector i at site k sits in lane i + 16 k, B[k][c] = spin column c at
    // site k in lane c + 16 k
    const int a_off = (lane >> 4) * kSqQ + 16 * qb + (lane & 15);
#pragma unroll
    for (int b = 0; b < kSqCBW; ++b) boff[b] += 3 * (lane >> 4);
    __syncthreads();  // the first chunk is staged
    int cur = 0;
    for (int64_t j0 = jb; j0 < je; j0 += kSqSites) {
        if (active) {
            const double* ph = lds + cur * kSqPhBuf + a_off;
            const double* sb = lds + 2 * kSqPhBuf + cur * kSqSbBuf;
            // Two register sets: the operands of K-step k + 1 are read from
            // LDS while the MFMAs of step k run.
            double are[2], aim[2], bv[2][kSqCBW];
            auto fetch = [&](int k, int r) {
                are[r] = ph[4 * k * kSqQ];
                aim[r] = ph[kSqSites * kSqQ + 4 * k * kSqQ];
#pragma unroll
                for (int b = 0; b < kSqCBW; ++b) bv[r][b] = sb[boff[b] + 12 * k];
            };
            fetch(0, 0);
#pragma unroll
            for (int k = 0; k < kSqSites / 4; ++k) {
                const int r = k & 1;
                if (k + 1 < kSqSites / 4) fetch(k + 1, r ^ 1);
#pragma unroll
                for (int b = 0; b < kSqCBW; ++b) {
                    acc_re[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(are[r], bv[r][b], acc_re[b], 0, 0, 0);
                    acc_im[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(aim[r], bv[r][b], acc_im[b], 0, 0, 0);
                }
            }
        }
        __syncthreads();  // done with `cur`; the producers have filled the other buffer
        cur ^= 1;
    }
    if (!active) return;
    // D[i][c] of the FP64 16x16x4 form: lane l, item v holds row 4 v + l / 16
    // of column l % 16 (rows interleave across the lane groups, unlike the
    // FP32 forms)
    double* out = a.part + (int64_t)blockIdx.z * a.n_q * 2 * n_cols;
#pragma unroll
    for (int b = 0; b < kSqCBW; ++b) {
        const int64_t c = c0 + (cb0 + b) * 16 + (lane & 15);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int qq = q0 + 16 * qb + 4 * v + (lane >> 4);
            if (qq < a.n_q && c < n_cols) {
                out[(int64_t)qq * 2 * n_cols + c] = acc_re[b][v];
                out[((int64_t)qq * 2 + 1) * n_cols + c] = acc_im[b][v];
            }
        }
    }
}

// F[q][f][a] = sum over the site ranges of the partial transforms, in range
// order (deterministic), as interleaved (re, im).
__global__ __launch_bounds__(256) void sq_reduce_kernel(SqTransformArgs a, double* __restrict__ F) {
    const int64_t n_cols = 3 * (int64_t)a.n_frames_used;
    const int64_t per = (int64_t)a.n_q * 2 * n_cols;
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < per; x += (int64_t)gridDim.x * blockDim.x) {
        double sum = 0.0;
#pragma unroll 8
        for (int sp = 0; sp < a.n_split; ++sp) sum += a.part[sp * per + x];
        const int64_t c = x % n_cols, qr = x / n_cols;
        F[((qr >> 1) * n_cols + c) * 2 + (qr & 1)] = sum;
    }
}

// One workgroup per wave vector, one thread per lag:
// raw[q][t] += sum_o sum_a conj(F_a(q, o s) - <F_a>) F_a(q, o s + t), FP64,
// <F_a> the average over the origins in the connected form (else 0).
// LDS: the wave vector's transform staged first (12 loads per origin and lag
// come from LDS instead of the cache); otherwise, for long series, read where
// it is, one origin at a time (100 wave vectors x 1000 lags x 1000 origins
// take 750 us, two origins at a time 822; staged 931: one workgroup fills LDS).
template <int LDS>
__global__ __launch_bounds__(256) void sq_corr_kernel(SqCorrArgs a) {
    extern __shared__ double staged[];
    const int qq = blockIdx.x;
    const double* F = a.F + (int64_t)qq * a.n_cols * 2;
    if constexpr (LDS) {
        for (int x = threadIdx.x; x < (int)a.n_cols * 2; x += 256) staged[x] = F[x];
        __syncthreads();
        F = staged;
    }
    double mre[3] = {0.0, 0.0, 0.0}, mim[3] = {0.0, 0.0, 0.0};
    if (a.connected) {
        for (int o = 0; o < a.n_origins; ++o)
            for (int al = 0; al < 3; ++al) {
                const int64_t x = ((int64_t)o * a.stride * 3 + al) * 2;
                mre[al] += F[x];
                mim[al] += F[x + 1];
            }
        for (int al = 0; al < 3; ++al) {
            mre[al] /= a.n_origins;
            mim[al] /= a.n_origins;
        }
    }
    for (int t = threadIdx.x; t < a.n_lags; t += 256) {
        double re = 0.0, im = 0.0;
        constexpr int kTurn = LDS ? 2 : 1;  // origins per turn
#pragma unroll kTurn
        for (int o = 0; o < a.n_origins; ++o) {
            const int64_t f0 = (int64_t)o * a.stride, f1 = f0 + t;
#pragma unroll
            for (int al = 0; al < 3; ++al) {
                const double ar = F[(f0 * 3 + al) * 2] - mre[al], ai = F[(f0 * 3 + al) * 2 + 1] - mim[al];
                const double br = F[(f1 * 3 + al) * 2], bi = F[(f1 * 3 + al) * 2 + 1];
                re += ar * br + ai * bi;
                im += ar * bi - ai * br;
            }
        }
        double* r = a.raw + ((int64_t)qq * a.n_lags + t) * 2;
        r[0] += re;
        r[1] += im;
    }
    if (qq == 0 && threadIdx.x == 0) a.n_org[0] += (double)a.n_origins;
}

dim3 sq_transform_grid(int n_q, int n_frames_used, int n_split) {
    return dim3((unsigned)((n_q + kSqQ - 1) / kSqQ), (unsigned)((n_frames_used + kSqFrames - 1) / kSqFrames),
                (unsigned)n_split);
}

int64_t blocks_for(int64_t n) {
    int64_t b = (n + 255) / 256;
    return b > 8192 ? 8192 : (b < 1 ? 1 : b);
}

}  // namespace

int64_t sq_tiles_per_split(int n_q, int n_frames_used) {
    const dim3 g = sq_transform_grid(n_q, n_frames_used, 1);
    return (int64_t)g.x * g.y;
}

int sq_site_chunk() { return kSqSites; }

int prepare_sq_kernels() {
    return (int)hipFuncSetAttribute((const void*)sq_transform_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    kSqLdsBytes);
}

int sq_frames_per_block() { return kSqFrames; }

int launch_sq_pack(const SqTransformArgs& a, void* stream) {
    const int64_t per_frame = (a.n + kSqSites - 1) / kSqSites * kSqRow;
    hipLaunchKernelGGL(sq_pack_kernel, dim3((unsigned)blocks_for(per_frame), (unsigned)(a.t_pad / kSqPackFrames)),
                       dim3(256), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

int launch_sq_transform(const SqTransformArgs& a, void* stream) {
    hipLaunchKernelGGL(sq_transform_kernel, sq_transform_grid(a.n_q, a.n_frames_used, a.n_split), dim3(kSqThreads),
                       kSqLdsBytes, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

int launch_sq_corr(const SqTransformArgs& t, const SqCorrArgs& a, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    const int64_t per = (int64_t)t.n_q * 2 * 3 * (int64_t)t.n_frames_used;
    hipLaunchKernelGGL(sq_reduce_kernel, dim3((unsigned)blocks_for(per)), dim3(256), 0, s, t, a.F);
    const int64_t lds = a.n_cols * 2 * (int64_t)sizeof(double);
    if (lds <= 64 * 1024)
        hipLaunchKernelGGL(sq_corr_kernel<1>, dim3((unsigned)a.n_q), dim3(256), (size_t)lds, s, a);
    else
        hipLaunchKernelGGL(sq_corr_kernel<0>, dim3((unsigned)a.n_q), dim3(256), 0, s, a);
    return (int)hipGetLastError();
}

int launch_sq_finalize(const double* raw, const double* n_org, int64_t n_sites, int n_q, int n_lags, double* sqt,
                       double* sqw, void* stream) {
    return launch_sqw(raw, n_org, n_sites, sqt, sqw, n_q, n_lags, stream);
}

}  // namespace sdc
