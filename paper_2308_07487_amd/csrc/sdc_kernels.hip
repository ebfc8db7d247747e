// gfx950 kernels of the sdc library.
//
//  pack    : [T][N][3] fp32 trajectory -> component-major, site-permuted,
//            K-contiguous blocks of 8 time samples (Sec. 3.2: the N x 3M
//            rearrangement; Sec. 3.1: realization-major storage for
//            coalescing), split into hi + lo halves for reduced precision.
//  fused   : launches of the product with the fused epilogue (sdc_fused.h).
//  count   : exact integer pair counts per bin with the same tile walk.
//  self    : the i = j term per lag in FP64.
//  final   : normalisation, site sum and the windowed time DFT (Sec. 2.2).
#include "sdc_device.h"

namespace sdc {

// ---------------------------------------------------------------------------
// pack
// ---------------------------------------------------------------------------

template <int PREC>
__device__ inline PackElem<PREC> make_chunk(const float v[8]) {
    PackElem<PREC> c;
    if constexpr (PREC == SDC_PREC_BF16X3) {
        // x = hi + mid + lo exactly: each difference has at most 16 (then 8)
        // significant bits and is exact in fp32
        uint32_t hi[8], mi[8], lo[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            hi[e] = bf16_bits(v[e]);
            const float r1 = v[e] - bf16_val(hi[e]);
            mi[e] = bf16_bits(r1);
            lo[e] = bf16_bits(r1 - bf16_val(mi[e]));
        }
        c.x = make_uint4(hi[0] | hi[1] << 16, hi[2] | hi[3] << 16, hi[4] | hi[5] << 16, hi[6] | hi[7] << 16);
        c.y = make_uint4(mi[0] | mi[1] << 16, mi[2] | mi[3] << 16, mi[4] | mi[5] << 16, mi[6] | mi[7] << 16);
        c.z = make_uint4(lo[0] | lo[1] << 16, lo[2] | lo[3] << 16, lo[4] | lo[5] << 16, lo[6] | lo[7] << 16);
    } else if constexpr (PREC == SDC_PREC_FP32) {
        c.x = make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]),
                         __float_as_uint(v[3]));
        c.y = make_uint4(__float_as_uint(v[4]), __float_as_uint(v[5]), __float_as_uint(v[6]),
                         __float_as_uint(v[7]));
    } else {
        uint32_t hi[8], lo[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if constexpr (PREC == SDC_PREC_SPLIT_BF16) {
                hi[e] = bf16_bits(v[e]);
                lo[e] = bf16_bits(v[e] - bf16_val(hi[e]));  // v - hi is exact in fp32
            } else {
                hi[e] = f16_bits(v[e]);
                lo[e] = f16_bits(v[e] - f16_val(hi[e]));
            }
        }
        c.x = make_uint4(hi[0] | hi[1] << 16, hi[2] | hi[3] << 16, hi[4] | hi[5] << 16,
                         hi[6] | hi[7] << 16);
        c.y = make_uint4(lo[0] | lo[1] << 16, lo[2] | lo[3] << 16, lo[4] | lo[5] << 16,
                         lo[6] | lo[7] << 16);
    }
    return c;
}

// Site-summed spin M(f) = sum_i S_i(f) of one frame in FP64, by one workgroup.
__device__ inline void frame_sum(const float* __restrict__ frames, int64_t n, int64_t f, double* __restrict__ M) {
    __shared__ double red[3][4];
    const float* x = frames + f * n * 3;
    double s[3] = {0.0, 0.0, 0.0};
    for (int64_t i = threadIdx.x; i < n; i += 256)
#pragma unroll
        for (int c = 0; c < 3; ++c) s[c] += (double)x[3 * i + c];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) s[c] += __shfl_down(s[c], w);
        if ((threadIdx.x & 63) == 0) red[c][threadIdx.x >> 6] = s[c];
    }
    __syncthreads();
    if (threadIdx.x < 3)
        M[f * 3 + threadIdx.x] =
            (red[threadIdx.x][0] + red[threadIdx.x][1]) + (red[threadIdx.x][2] + red[threadIdx.x][3]);
    __syncthreads();  // the next frame reuses the partial sums
}

// Grid rows of a pack launch that sum frames, gx workgroups each.
__host__ __device__ inline int sum_rows(int64_t n_sums, int64_t gx) {
    const int64_t r = (n_sums + gx - 1) / gx;
    return (int)(r < 4096 ? r : 4096);  // a grid has at most 65535 rows; the sums then take several frames each
}

// One thread per (block of 8 samples, packed site); writes the three
// components.  Rows 0..3*O8 of the work index the A pack (origins o*s),
// the rest the B packs (phase copies: sample g of phase ph is frame s*g + ph).
// The first rows of the grid sum the frames that the site sums read, one
// frame per workgroup (independent work that would be a launch of its own:
// at sc 8^3 each launch costs about as much as its kernel).
template <int PREC>
__global__ __launch_bounds__(256) void pack_kernel(PackArgs a) {
    const int n_sum = sum_rows(a.n_sums, gridDim.x);
    const int row = (int)blockIdx.y - n_sum;  // 0..O8 + n_phase*F8 - 1 after the frame sums
    if (row < 0) {
        for (int64_t f = (int64_t)blockIdx.y * gridDim.x + blockIdx.x; f < a.n_sums; f += (int64_t)n_sum * gridDim.x)
            frame_sum(a.frames, a.n, f, a.mframe);
        return;
    }
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.n_pad) return;
    const int32_t orig = a.perm[p];
    float v[3][8];
    const bool isA = row < a.O8;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        int64_t f;
        bool ok;
        if (isA) {
            const int o = row * 8 + e;
            f = (int64_t)o * a.stride;
            ok = o < a.n_origins;
        } else {
            const int r = row - a.O8;
            const int ph = r / a.F8;
            const int g = (r % a.F8) * 8 + e;
            f = (int64_t)g * a.stride + ph;
            ok = true;
        }
        ok = ok && orig >= 0 && f < a.frames_valid;
        const float* src = a.frames + (f * a.n + (ok ? orig : 0)) * 3;
        v[0][e] = ok ? src[0] : 0.0f;
        v[1][e] = ok ? src[1] : 0.0f;
        v[2][e] = ok ? src[2] : 0.0f;
        // connected form: the origin side is centred on its average over the
        // origins (Eq. (5)); since the centred values sum to zero over the
        // origins, the later side needs no centring
        if (isA && ok && a.mean) {
            v[0][e] -= a.mean[4 * orig];
            v[1][e] -= a.mean[4 * orig + 1];
            v[2][e] -= a.mean[4 * orig + 2];
        }
    }
    PackUnit<PREC>* dst;
    int64_t comp_stride, plane;
    if (isA) {
        dst = (PackUnit<PREC>*)a.A + (int64_t)row * a.n_pad + p;
        comp_stride = (int64_t)a.O8 * a.n_pad;
        plane = pack_plane_a(a);
    } else {
        const int r = row - a.O8;
        const int ph = r / a.F8;
        dst = (PackUnit<PREC>*)a.B + ((int64_t)ph * 3 * a.F8 + (r % a.F8)) * a.n_pad + p;
        comp_stride = (int64_t)a.F8 * a.n_pad;
        plane = pack_plane_b(a);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const PackElem<PREC> e = make_chunk<PREC>(v[c]);
        if constexpr (pack_planes(PREC)) {
            dst[c * comp_stride] = e.x;
            dst[c * comp_stride + plane] = e.y;
        } else {
            dst[c * comp_stride] = e;
        }
    }
}

int launch_pack(const PackArgs& a, void* stream) {
    dim3 block(256);
    const int64_t gx = (a.n_pad + 255) / 256;
    dim3 grid((unsigned)gx, (unsigned)(a.O8 + a.n_phase * a.F8 + sum_rows(a.n_sums, gx)));
    hipStream_t s = (hipStream_t)stream;
    switch (a.precision) {
        case SDC_PREC_FP32: hipLaunchKernelGGL(pack_kernel<SDC_PREC_FP32>, grid, block, 0, s, a); break;
        case SDC_PREC_SPLIT_BF16: hipLaunchKernelGGL(pack_kernel<SDC_PREC_SPLIT_BF16>, grid, block, 0, s, a); break;
        case SDC_PREC_SPLIT_FP16: hipLaunchKernelGGL(pack_kernel<SDC_PREC_SPLIT_FP16>, grid, block, 0, s, a); break;
        case SDC_PREC_BF16X3: hipLaunchKernelGGL(pack_kernel<SDC_PREC_BF16X3>, grid, block, 0, s, a); break;
        default: return (int)hipErrorInvalidValue;
    }
    return (int)hipGetLastError();
}

// ---------------------------------------------------------------------------
// launches of the fused kernels
// ---------------------------------------------------------------------------

int fused_lds_bytes(int win, int precision) {
    return hist_pitch(precision) * win * (int)sizeof(double) + 1024 * (int)sizeof(float);
}

// The fused kernels of each precision (sdc_fused_*.hip).
const void* fused_kernel_fp32(int sched, int radial, int paired, bool batch);
const void* fused_kernel_bf16(int sched, int radial, int paired, bool batch);
const void* fused_kernel_fp16(int sched, int radial, int paired, bool batch);
const void* fused_kernel_x3(int sched, int radial, int paired, bool batch);

// Kernel of a fused launch, or null for a (precision, schedule) pair that
// does not exist.
static const void* fused_kernel_of(int precision, int sched, int radial, int paired, bool batch) {
    switch (precision) {
        case SDC_PREC_FP32: return fused_kernel_fp32(sched, radial, paired, batch);
        case SDC_PREC_BF16X3: return fused_kernel_x3(sched, radial, paired, batch);
        case SDC_PREC_SPLIT_BF16: return fused_kernel_bf16(sched, radial, paired, batch);
        case SDC_PREC_SPLIT_FP16: return fused_kernel_fp16(sched, radial, paired, batch);
        default: return nullptr;
    }
}

int launch_fused(const FusedArgs& a, void* stream) {
    if (a.n_groups * a.n_streams == 0) return 0;
    if (!sched_valid(a.precision, a.sched)) return (int)hipErrorInvalidValue;
    const void* fn = fused_kernel_of(a.precision, a.sched, a.map.kind == SDC_BINS_RADIAL, a.O8 % 2 == 0, false);
    if (!fn) return (int)hipErrorInvalidValue;
    const int lds = fused_lds_bytes(a.win, a.precision);
    const int n_tasks = a.n_groups * a.n_streams;
    const int grid = 8 * ((n_tasks + 7) / 8);
    void* params[] = {(void*)&a};
    return (int)hipLaunchKernel(fn, dim3(grid), dim3(threads_per_wg(a.sched)), params, lds, (hipStream_t)stream);
}

int batch_grid(int precision, int sched, int radial, int lds, int device, int64_t total, int* grid) {
    const void* fn = fused_kernel_of(precision, sched, radial, 0, true);
    if (!fn) return (int)hipErrorInvalidValue;
    int per_cu = 0, n_cu = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads_per_wg(sched), lds);
    if (e != hipSuccess) return (int)e;
    e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return (int)e;
    if (per_cu < 1) per_cu = 1;
    int64_t g = (int64_t)per_cu * n_cu;
    if (g > total) g = total;
    g = 8 * ((g + 7) / 8);
    *grid = (int)(g < 8 ? 8 : g);
    return 0;
}

int launch_fused_batch(const BatchLaunch& b, void* stream) {
    if (b.total == 0) return 0;
    const void* fn = fused_kernel_of(b.precision, b.sched, b.radial, 0, true);
    if (!fn) return (int)hipErrorInvalidValue;
    int e = launch_zero(b.queue, 8 * sizeof(unsigned), stream);
    if (e != 0) return e;
    const FusedArgs* args = b.args;
    const int64_t* task_start = b.task_start;
    int n_plans = b.n_plans;
    unsigned* queue = b.queue;
    const int64_t* ranges = b.ranges;
    int64_t total = b.total;
    void* params[] = {(void*)&args, (void*)&task_start, (void*)&n_plans, (void*)&queue, (void*)&ranges,
                      (void*)&total};
    return (int)hipLaunchKernel(fn, dim3(b.grid), dim3(threads_per_wg(b.sched)), params, b.lds,
                                (hipStream_t)stream);
}

// ---------------------------------------------------------------------------
// exact pair counts
// ---------------------------------------------------------------------------

template <int RADIAL>
__global__ __launch_bounds__(256) void count_kernel(CountArgs a) {
    extern __shared__ unsigned int hcount[];  // [win], then radial edges
    float* e2s = (float*)(hcount + a.win);
    const int tid = threadIdx.x;
    const KStream st = a.streams[blockIdx.x];
    for (int x = tid; x < a.win; x += 256) hcount[x] = 0u;
    if constexpr (RADIAL) {
        for (int x = tid; x < a.n_shells; x += 256) e2s[x] = a.e2[x];
    }
    __syncthreads();
    for (int p = st.p0; p < st.p1; ++p) {
        const KPair pr = a.pairs[p];
        for (int e = tid; e < kTile * kTile; e += 256) {
            const int64_t pi = (int64_t)pr.ti * kTile + (e >> 6);
            const int64_t pj = (int64_t)pr.tj * kTile + (e & 63);
            if (a.perm[pi] < 0 || a.perm[pj] < 0) continue;
            int w;
            if constexpr (RADIAL) {
                const float4 ri = *(const float4*)(a.pos4 + 4 * pi);
                const float4 rj = *(const float4*)(a.pos4 + 4 * pj);
                w = shell_of(dist2_f32(ri.x, ri.y, ri.z, rj.x, rj.y, rj.z), e2s, a.n_shells, a.inv_w);
            } else {
                w = a.map.linear ? linear_window(e >> 6, a.gtab[pi], e & 63, a.gtab[pj], pr.shift)
                                 : a.gtab[pj] - a.gtab[pi] + pr.shift;
            }
            atomicAdd(&hcount[w], 1u);
        }
    }
    __syncthreads();
    for (int w = tid; w < a.win; w += 256) {
        const unsigned int v = hcount[w];
        if (v == 0u) continue;
        int64_t b;
        if constexpr (RADIAL) {
            b = w;
        } else {
            b = window_bin(a.map, st, w);
        }
        atomicAdd(&a.counts[b], (unsigned long long)v);
    }
}

// One workgroup per tile pair; thread (wave, lane) writes the 16 shells its
// accumulator registers hold in the fused kernel (same row/column mapping).
__global__ __launch_bounds__(256) void radial_keys_kernel(CountArgs a, int64_t n_pairs, uint16_t* __restrict__ keys) {
    __shared__ float e2s[1024];
    const int tid = threadIdx.x;
    for (int x = tid; x < a.n_shells; x += 256) e2s[x] = a.e2[x];
    __syncthreads();
    const int wave = tid >> 6, lane = tid & 63;
    const int wi = wave >> 1, wj = wave & 1, h = lane >> 5, l32 = lane & 31;
    for (int64_t p = blockIdx.x; p < n_pairs; p += gridDim.x) {
        const KPair pr = a.pairs[p];
        const int64_t sj = (int64_t)pr.tj * kTile + wj * 32 + l32;
        const int64_t rowbase = (int64_t)pr.ti * kTile + wi * 32 + 4 * h;
        const float4 pj = *(const float4*)(a.pos4 + 4 * sj);
        uint32_t kw[8];
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            const float4 p0 = *(const float4*)(a.pos4 + 4 * (rowbase + 8 * (r / 4) + (r % 4)));
            const float4 p1 = *(const float4*)(a.pos4 + 4 * (rowbase + 8 * ((r + 1) / 4) + ((r + 1) % 4)));
            const uint32_t k0 = (uint32_t)shell_of(dist2_f32(p0.x, p0.y, p0.z, pj.x, pj.y, pj.z), e2s, a.n_shells, a.inv_w);
            const uint32_t k1 = (uint32_t)shell_of(dist2_f32(p1.x, p1.y, p1.z, pj.x, pj.y, pj.z), e2s, a.n_shells, a.inv_w);
            kw[r / 2] = k0 | (k1 << 16);
        }
        uint4* dst = (uint4*)(keys + ((p * 4 + wave) * 64 + lane) * 16);
        dst[0] = make_uint4(kw[0], kw[1], kw[2], kw[3]);
        dst[1] = make_uint4(kw[4], kw[5], kw[6], kw[7]);
    }
}

int launch_radial_keys(const CountArgs& a, int64_t n_pairs, uint16_t* keys, void* stream) {
    if (n_pairs == 0) return 0;
    if (a.n_shells > 1024) return (int)hipErrorInvalidValue;
    const int64_t grid = n_pairs < 65536 ? n_pairs : 65536;
    hipLaunchKernelGGL(radial_keys_kernel, dim3((unsigned)grid), dim3(256), 0, (hipStream_t)stream, a, n_pairs,
                       keys);
    return (int)hipGetLastError();
}

int launch_count(const CountArgs& a, void* stream) {
    if (a.n_streams == 0) return 0;
    hipStream_t s = (hipStream_t)stream;
    const int lds = a.win * 4 + (a.map.kind == SDC_BINS_RADIAL ? a.n_shells * 4 : 0);
    hipError_t e;
    if (a.map.kind == SDC_BINS_RADIAL) {
        e = hipFuncSetAttribute((const void*)count_kernel<1>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return (int)e;
        hipLaunchKernelGGL(count_kernel<1>, dim3(a.n_streams), dim3(256), lds, s, a);
    } else {
        e = hipFuncSetAttribute((const void*)count_kernel<0>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return (int)e;
        hipLaunchKernelGGL(count_kernel<0>, dim3(a.n_streams), dim3(256), lds, s, a);
    }
    return (int)hipGetLastError();
}

// ---------------------------------------------------------------------------
// self term: sum_o sum_i S_i(o s) . S_i(o s + t) in FP64
// ---------------------------------------------------------------------------

// Small pieces of v exactly as the pack kernel forms them: lo of the hi/lo
// splits; mid and lo of the three-piece form.
template <int PREC>
__device__ inline void small_pieces(float v, float (&p)[2]) {
    if constexpr (PREC == SDC_PREC_SPLIT_BF16) {
        p[0] = bf16_val(bf16_bits(v - bf16_val(bf16_bits(v))));
    } else if constexpr (PREC == SDC_PREC_SPLIT_FP16) {
        p[0] = f16_val(f16_bits(v - f16_val(f16_bits(v))));
    } else if constexpr (PREC == SDC_PREC_BF16X3) {
        const float r = v - bf16_val(bf16_bits(v));
        p[0] = bf16_val(bf16_bits(r));
        p[1] = bf16_val(bf16_bits(r - p[0]));
    }
}
// Pieces kept per value: the number of small ones.
template <int PREC>
constexpr int n_small() {
    return PREC == SDC_PREC_FP32 ? 0 : PREC == SDC_PREC_BF16X3 ? 2 : 1;
}
// The part of x*y that the reduced-precision contraction leaves out, from
// the small pieces (FP64, exact): lo*lo for the hi/lo splits; mid*lo +
// lo*mid + lo*lo for the three-piece form.
template <int PREC>
__device__ inline double dropped_product(const float (&x)[2], const float (&y)[2]) {
    if constexpr (PREC == SDC_PREC_BF16X3)
        return (double)x[0] * (double)y[1] + (double)x[1] * (double)y[0] + (double)x[1] * (double)y[1];
    else
        return (double)x[0] * (double)y[0];
}

// Site-summed correlation of selected lag l: the sum over all ordered pairs
// of S_i(o s) . S_j(o s + t) equals M(o s) . M(o s + t), summed over the
// origins in FP64 (one thread per lag).  For the connected form the origin
// side is centred: the sum over all pairs of (S_i(o s) - <S_i>) . S_j(o s + t)
// is (M(o s) - <M>) . M(o s + t).
__device__ inline void site_sum(const SelfArgs& a, int l) {
    const int t = a.lags[l];
    double mb[3] = {0.0, 0.0, 0.0};
    if (a.mean) {
        for (int o = 0; o < a.n_origins; ++o)
            for (int c = 0; c < 3; ++c) mb[c] += a.mframe[(int64_t)o * a.stride * 3 + c];
        for (int c = 0; c < 3; ++c) mb[c] /= (double)a.n_origins;
    }
    double s = 0.0;
#pragma unroll 4
    for (int o = 0; o < a.n_origins; ++o) {
        const double* m0 = a.mframe + (int64_t)o * a.stride * 3;
        const double* m1 = m0 + (int64_t)t * 3;
        s += (m0[0] - mb[0]) * m1[0] + (m0[1] - mb[1]) * m1[1] + (m0[2] - mb[2]) * m1[2];
    }
    a.msum[t] += s;
}

// Where the self kernel finds the samples of its sites: in global memory, as
// whole series in LDS, or in LDS with their small pieces and the centred
// origin side beside them (kSelfPieces; when all of it fits the budget).
constexpr int kSelfGlobal = 0, kSelfSeries = 1, kSelfPieces = 2;

// LDS floats per site.
static int64_t self_floats(int mode, int pieces, int64_t t_need, int n_origins) {
    if (mode == kSelfSeries) return 3 * t_need;
    if (mode == kSelfPieces) return 3 * (1 + pieces) * (t_need + n_origins);
    return 0;
}

// Self sums.  A workgroup takes groups of `spb` consecutive sites (a power of
// two, 256 / spb threads each, every thread the lags r, r + 256 / spb, ...) and
// adds its lag sums to the global ones once at the end.  Bound: FP64 vector
// arithmetic, 3 n_o multiply-adds per site and lag, twice that with the
// dropped products.  The pieces are split once per sample and origin (split
// again in every product the kernel took 3.8 ms at sc 36^3 x 256 lags and 25 us
// at sc 8^3 x 64), and spb shrinks until the chip is filled (16 sites per
// workgroup left sc 8^3 with 32 workgroups, and larger samples with one
// workgroup per compute unit).
// Besides the exact self sum it forms, for split precisions, the lo*lo
// product that the three-product contraction leaves out, restricted to the
// i = j pairs, and adds it to bin 0 (the bin of zero displacement for every
// bin kind).  On the diagonal that term has a fixed sign, so dropping it
// would bias C(0, 0); off the diagonal it is unbiased rounding noise.
// The blocks from n_blocks on form the site sums (the frame sums were queued
// before).
template <int MODE, int PREC>
__global__ __launch_bounds__(256) void self_kernel(SelfArgs a, int spb, int n_blocks) {
    // sums per lag, then (except kSelfGlobal) the series [t_need][spb][3], per
    // small piece the same, and the origin side
    extern __shared__ double part[];
    double* const part_lo = part + a.n_sel;
    float* const ser = (float*)(part + 2 * a.n_sel);
    constexpr int P = n_small<PREC>();
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= n_blocks) {
        const int l = ((int)blockIdx.x - n_blocks) * 256 + tid;
        if (l < a.n_sel) site_sum(a, l);
        return;
    }
    const int w = spb * 3;  // values per frame
    float* const lo = ser + a.t_need * w;                    // [P][t_need][spb][3]
    float* const org = lo + P * a.t_need * w;                // [n_origins][spb][3] (kSelfPieces)
    float* const org_lo = org + (int64_t)a.n_origins * w;    // [P][n_origins][spb][3]
    const int tps = 256 / spb, q = tid / tps, r = tid % tps;
    for (int x = tid; x < a.n_sel; x += 256) {
        part[x] = 0.0;
        part_lo[x] = 0.0;
    }
    for (int64_t i0 = (int64_t)blockIdx.x * spb; i0 < a.n; i0 += (int64_t)n_blocks * spb) {
        const int nsb = (int)((a.n - i0) < spb ? (a.n - i0) : spb);
        __syncthreads();
        if constexpr (MODE != kSelfGlobal) {
#pragma unroll 4
            for (int x = tid; x < (int)a.t_need * w; x += 256) {
                const int f = x / w, rem = x - f * w;
                const float v = rem < nsb * 3 ? a.frames[((int64_t)f * a.n + i0) * 3 + rem] : 0.0f;
                ser[x] = v;
                if constexpr (MODE == kSelfPieces && P > 0) {
                    float p[2];
                    small_pieces<PREC>(v, p);
#pragma unroll
                    for (int k = 0; k < P; ++k) lo[k * a.t_need * w + x] = p[k];
                }
            }
            __syncthreads();
        }
        if constexpr (MODE == kSelfPieces) {
            for (int x = tid; x < a.n_origins * w; x += 256) {
                const int o = x / w, rem = x - o * w;
                if (rem >= nsb * 3) continue;
                const int64_t y = (int64_t)o * a.stride * w + rem;
                if (a.mean) {  // as the pack kernel forms it
                    const float u = ser[y] - a.mean[4 * (i0 + rem / 3) + rem % 3];
                    org[x] = u;
                    float p[2];
                    small_pieces<PREC>(u, p);
#pragma unroll
                    for (int k = 0; k < P; ++k) org_lo[k * a.n_origins * w + x] = p[k];
                } else {
                    org[x] = ser[y];
#pragma unroll
                    for (int k = 0; k < P; ++k) org_lo[k * a.n_origins * w + x] = lo[k * a.t_need * w + y];
                }
            }
            __syncthreads();
        }
        if (q >= nsb) continue;
        float mu[3] = {0.0f, 0.0f, 0.0f};  // origin-side average (connected form)
        if (MODE != kSelfPieces && a.mean)
            for (int c = 0; c < 3; ++c) mu[c] = a.mean[4 * (i0 + q) + c];
        // lags l, l + tps, ... of the site, L at a time: L lags share the
        // reads and conversions of the origin side
        auto lags = [&](auto count, int l) {
            constexpr int L = decltype(count)::value;
            double s[L] = {}, sl[L] = {};
            if constexpr (MODE == kSelfPieces) {
                const float* x0 = org + 3 * q;
                const float* l0 = org_lo + 3 * q;
                const int step = a.stride * w, pa = a.n_origins * w, pb = (int)a.t_need * w;
                int at[L];
#pragma unroll
                for (int j = 0; j < L; ++j) at[j] = a.lags[l + j * tps] * w + 3 * q;
#pragma unroll 2
                for (int o = 0; o < a.n_origins; ++o) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const double x = (double)x0[o * w + c];
                        float u[2];
#pragma unroll
                        for (int k = 0; k < P; ++k) u[k] = l0[k * pa + o * w + c];
#pragma unroll
                        for (int j = 0; j < L; ++j) {
                            const int y = at[j] + o * step + c;
                            s[j] += x * (double)ser[y];
                            if constexpr (P > 0) {
                                float v[2];
#pragma unroll
                                for (int k = 0; k < P; ++k) v[k] = lo[k * pb + y];
                                sl[j] += dropped_product<PREC>(u, v);
                            }
                        }
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < L; ++j) {
                    const int t = a.lags[l + j * tps];
                    for (int o = 0; o < a.n_origins; ++o) {
                        const int64_t f0 = (int64_t)o * a.stride, f1 = f0 + t;
                        const float* x0 = MODE == kSelfSeries ? ser + f0 * w + 3 * q : a.frames + (f0 * a.n + i0 + q) * 3;
                        const float* x1 = MODE == kSelfSeries ? ser + f1 * w + 3 * q : a.frames + (f1 * a.n + i0 + q) * 3;
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            const float u = x0[c] - mu[c];  // as the pack kernel forms it
                            s[j] += (double)u * (double)x1[c];
                            if constexpr (P > 0) {
                                float pu[2], pv[2];
                                small_pieces<PREC>(u, pu);
                                small_pieces<PREC>(x1[c], pv);
                                sl[j] += dropped_product<PREC>(pu, pv);
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < L; ++j) {
                const int k = l + j * tps;
                if (a.det) {
                    atomicAdd(reinterpret_cast<unsigned long long*>(part) + k, to_fixed(s[j]));
                    if constexpr (P > 0) atomicAdd(reinterpret_cast<unsigned long long*>(part_lo) + k, to_fixed(sl[j]));
                } else {
                    atomicAdd(&part[k], s[j]);
                    if constexpr (P > 0) atomicAdd(&part_lo[k], sl[j]);
                }
            }
        };
        int l = r;
        if constexpr (MODE == kSelfPieces)
            for (; l + 3 * tps < a.n_sel; l += 4 * tps) lags(std::integral_constant<int, 4>{}, l);
        for (; l < a.n_sel; l += tps) lags(std::integral_constant<int, 1>{}, l);
    }
    __syncthreads();
    // origin totals live on the device so that replays of a captured
    // accumulate count their origins too
    if (blockIdx.x == 0)
        for (int l = tid; l < a.n_sel; l += 256) a.norg[a.lags[l]] += (double)a.n_origins;
    for (int l = tid; l < a.n_sel; l += 256) {
        if (a.det) {
            atomicAdd(&a.selfq[a.lags[l]], reinterpret_cast<const unsigned long long*>(part)[l]);
            if constexpr (P > 0)
                atomicAdd(&a.Hq[(int64_t)a.lags[l] * a.n_bins], reinterpret_cast<const unsigned long long*>(part_lo)[l]);
        } else {
            unsafeAtomicAdd(&a.self[a.lags[l]], part[l]);
            if constexpr (P > 0) unsafeAtomicAdd(&a.H[(int64_t)a.lags[l] * a.n_bins], part_lo[l]);
        }
    }
}

template <int MODE>
static const void* self_fn(int precision) {
    switch (precision) {
        case SDC_PREC_SPLIT_BF16: return (const void*)self_kernel<MODE, SDC_PREC_SPLIT_BF16>;
        case SDC_PREC_SPLIT_FP16: return (const void*)self_kernel<MODE, SDC_PREC_SPLIT_FP16>;
        case SDC_PREC_BF16X3: return (const void*)self_kernel<MODE, SDC_PREC_BF16X3>;
        default: return (const void*)self_kernel<MODE, SDC_PREC_FP32>;
    }
}
static const void* self_kernel_of(int mode, int precision) {
    return mode == kSelfPieces   ? self_fn<kSelfPieces>(precision)
           : mode == kSelfSeries ? self_fn<kSelfSeries>(precision)
                                 : self_fn<kSelfGlobal>(precision);
}

__global__ __launch_bounds__(256) void mean_kernel(const float* __restrict__ frames, int64_t n, int n_origins,
                                                   int stride, float* __restrict__ mean) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    for (int o = 0; o < n_origins; ++o) {
        const float* x = frames + ((int64_t)o * stride * n + i) * 3;
        s0 += (double)x[0];
        s1 += (double)x[1];
        s2 += (double)x[2];
    }
    const double inv = 1.0 / (double)n_origins;
    mean[4 * i] = (float)(s0 * inv);
    mean[4 * i + 1] = (float)(s1 * inv);
    mean[4 * i + 2] = (float)(s2 * inv);
    mean[4 * i + 3] = 0.0f;
}

int launch_mean(const float* frames, int64_t n, int n_origins, int stride, float* mean, void* stream) {
    hipLaunchKernelGGL(mean_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       frames, n, n_origins, stride, mean);
    return (int)hipGetLastError();
}

int launch_self(const SelfArgs& a, void* stream) {
    if (a.n_sel == 0) return 0;
    if (a.n_sel > 1024) return (int)hipErrorInvalidValue;
    const int pieces = a.precision == SDC_PREC_FP32 ? 0 : a.precision == SDC_PREC_BF16X3 ? 2 : 1;
    int mode = kSelfPieces;
    while (mode != kSelfGlobal && self_floats(mode, pieces, a.t_need, a.n_origins) * 4 > kSelfLdsBudget) --mode;
    // sites per workgroup: at most 16, few enough for four workgroups per
    // compute unit (256 of them) both by their number and by their LDS, but
    // enough to give every thread a lag (more workgroups than that only queue
    // their atomics on the sums: sc 8^3 x 64 lags took 16 us with one site per
    // workgroup)
    const int64_t per_site = self_floats(mode, pieces, a.t_need, a.n_origins) * 4, sums = (int64_t)16 * a.n_sel;
    int spb = 16;
    while (spb > 1 && (spb * per_site + sums > 40 * 1024 || (a.n < (int64_t)1024 * spb && a.n_sel * spb > 256)))
        spb /= 2;
    // 1024 workgroups share the sites: each adds 2 n_sel sums to global memory
    const int64_t groups = (a.n + spb - 1) / spb;
    int n_blocks = (int)(groups < 1024 ? groups : 1024);
    SelfArgs args = a;
    void* params[] = {(void*)&args, (void*)&spb, (void*)&n_blocks};
    return (int)hipLaunchKernel(self_kernel_of(mode, a.precision), dim3((unsigned)(n_blocks + (a.n_sel + 255) / 256)),
                                dim3(256), params, (size_t)(spb * per_site + sums), (hipStream_t)stream);
}

// Dynamic-LDS limits of every kernel that takes more than the default, set
// once per device at plan creation so that the launch paths make no attribute
// calls (they stay legal under stream capture).
int prepare_kernels() {
    for (int prec = SDC_PREC_FP32; prec <= SDC_PREC_BF16X3; ++prec)
        for (int sched = kSchedOnePass; sched <= kSchedFold; ++sched)
            for (int k = 0; k < 6; ++k) {  // (radial, paired) of the single-plan kernels, then the batch ones
                const bool batch = k >= 4;
                const int radial = batch ? (k & 1) : ((k >> 1) & 1), paired = batch ? 0 : (k & 1);
                const void* f = fused_kernel_of(prec, sched, radial, paired, batch);
                if (!f) continue;
                hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxFusedLds);
                if (e != hipSuccess) return (int)e;
            }
    for (int prec = SDC_PREC_FP32; prec <= SDC_PREC_BF16X3; ++prec)
        for (int mode = kSelfSeries; mode <= kSelfPieces; ++mode) {
            const hipError_t e = hipFuncSetAttribute(self_kernel_of(mode, prec),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     (int)kSelfLdsBudget + 16 * 1024);
            if (e != hipSuccess) return (int)e;
        }
    return 0;
}

// ---------------------------------------------------------------------------
// finalize: normalisation, site sums, windowed DFT (all FP64)
// ---------------------------------------------------------------------------

// Windowed DFT over the lags of NS complex series x of length m:
// out[k] = sum_t w_t x_t exp(-2 pi i k t / m), w_t = (1 + cos(pi t / m)) / 2, for 64 k per
// workgroup (k0 + tid % 64), a quarter of the t per thread group.  lds holds
// the m phases and then the windowed series (2 + 2 NS doubles per t), filled
// here; value(s, t, re, im) gives x.  The phases come from one table of m
// sines and cosines instead of one pair per (k, t): with those the kernel of
// 256 lags took 56 us.
template <int NS, class Value, class Store>
__device__ inline void lag_dft(int m, int k0, double* lds, const Value& value, const Store& store) {
    double* const cs = lds;
    double* const sn = lds + m;
    double* const x = lds + 2 * m;  // [NS][2][m]
    for (int t = threadIdx.x; t < m; t += 256) {
        sincospi(-2.0 * (double)t / (double)m, &sn[t], &cs[t]);
        const double w = 0.5 * (1.0 + cospi((double)t / (double)m));
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            double re, im;
            value(s, t, re, im);
            x[2 * s * m + t] = w * re;
            x[(2 * s + 1) * m + t] = w * im;
        }
    }
    __syncthreads();
    const int k = k0 + (int)(threadIdx.x & 63), g = threadIdx.x >> 6;
    const int t0 = g * m / 4, t1 = (g + 1) * m / 4;
    double re[NS] = {}, im[NS] = {};
    if (k < m) {
        int kt = (int)(((int64_t)k * t0) % m);
        for (int t = t0; t < t1; ++t) {
            const double c = cs[kt], d = sn[kt];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const double xr = x[2 * s * m + t], xi = x[(2 * s + 1) * m + t];
                re[s] += xr * c - xi * d;
                im[s] += xr * d + xi * c;
            }
            kt += k;
            if (kt >= m) kt -= m;
        }
    }
    __syncthreads();
    double* const red = lds;  // [4][64][2 NS] in the space of the tables
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        red[(threadIdx.x * NS + s) * 2] = re[s];
        red[(threadIdx.x * NS + s) * 2 + 1] = im[s];
    }
    __syncthreads();
    if (g == 0 && k < m) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            double r = 0.0, i = 0.0;
            for (int h = 0; h < 4; ++h) {
                r += red[((threadIdx.x + 64 * h) * NS + s) * 2];
                i += red[((threadIdx.x + 64 * h) * NS + s) * 2 + 1];
            }
            store(s, k, r, i);
        }
    }
}
template <int NS>
static int lag_dft_lds(int m) {
    const int tables = (2 + 2 * NS) * m, red = 256 * 2 * NS;
    return (tables > red ? tables : red) * (int)sizeof(double);
}

// Rows 0 .. n_lags - 1 of the grid normalise H (when C is asked for); the
// blocks of the rows after them form the site-summed and self correlations
// and their spectra, 64 frequencies each.  The site sum comes from the
// magnetisation products (an exact identity for the sum of H over all bins),
// which keeps the per-bin rounding of the reduced-precision products from
// adding up over N^2 pairs.
__global__ __launch_bounds__(256) void finalize_kernel(FinalArgs a) {
    extern __shared__ double lds[];
    const int rows = a.C ? a.n_lags : 0;
    if ((int)blockIdx.y < rows) {
        const int t = blockIdx.y;
        const double no = a.n_org[t];
        for (int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x; b < a.n_bins; b += (int64_t)gridDim.x * 256) {
            const double den = no * (double)a.counts[b];
            a.C[t * a.n_bins + b] = den > 0.0 ? a.H[t * a.n_bins + b] / den : 0.0;
            if (t == 0 && a.counts_out) a.counts_out[b] = a.counts[b];
        }
        return;
    }
    const int k0 = (((int)blockIdx.y - rows) * (int)gridDim.x + (int)blockIdx.x) * 64;
    if (k0 >= a.n_lags) return;
    lag_dft<2>(
        a.n_lags, k0, lds,
        [&](int s, int t, double& re, double& im) {
            const double d = (double)a.n_sites * a.n_org[t];
            re = d > 0.0 ? (s == 0 ? a.msum[t] : a.self[t]) / d : 0.0;
            im = 0.0;
            if (k0 == 0) (s == 0 ? a.csum : a.cself)[t] = re;
        },
        [&](int s, int k, double re, double im) {
            double* out = (s == 0 ? a.ssum : a.sself) + 2 * k;
            out[0] = re;
            out[1] = im;
        });
}

// S(q, t) = sum_b exp(-i q.d_b) H(b, t) / (N n_org), d_b the displacement of
// bin b (bcc: the parity adds half a cell on every axis).  One workgroup per q
// and kSqtLags lags: a bin's phase is computed once and applied to all of
// them (one FP64 sine, cosine and three remainders per bin; per bin and lag
// they took 233 of the 240 us of 40 wave vectors x 100 lags x 7980 bins).
// FP64 throughout; the phase is reduced exactly in integers first.
constexpr int kSqtLags = 8;
__global__ __launch_bounds__(256) void sqt_kernel(SqtArgs a) {
    __shared__ double red[4][2 * kSqtLags];
    const int qi = blockIdx.x, t0 = (int)blockIdx.y * kSqtLags;
    const int L[3] = {a.L0, a.L1, a.L2};
    // q.d / pi = sum_a 2 m_a (k_a + p/2) / L_a = sum_a m_a (2 k_a + p) / L_a, taken mod 2
    // per axis in integers: m_a (2 k_a + p) mod 2 L_a, with m_a reduced first
    // (edges are at most 4096, so the products stay below 2^27)
    int m[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) m[c] = pmod_dev(a.m[3 * qi + c], 2 * L[c]);
    const bool bcc = a.kind == SDC_BINS_PERIODIC_BCC;
    double re[kSqtLags] = {}, im[kSqtLags] = {};
    for (int64_t b = threadIdx.x; b < a.n_bins; b += 256) {
        const uint32_t c = (uint32_t)(bcc ? b >> 1 : b);
        const int par = bcc ? (int)(b & 1) : 0;
        const uint32_t row = c / (uint32_t)a.L2;
        const int k2 = (int)(c - row * (uint32_t)a.L2), k0 = (int)(row / (uint32_t)a.L1);
        const int k1 = (int)(row - (uint32_t)k0 * (uint32_t)a.L1);
        const int n0 = (m[0] * (2 * k0 + par)) % (2 * L[0]);
        const int n1 = (m[1] * (2 * k1 + par)) % (2 * L[1]);
        const int n2 = (m[2] * (2 * k2 + par)) % (2 * L[2]);
        const double x = (double)n0 / a.L0 + (double)n1 / a.L1 + (double)n2 / a.L2;
        double sn, cs;
        sincospi(-x, &sn, &cs);
#pragma unroll
        for (int j = 0; j < kSqtLags; ++j) {
            const double h = t0 + j < a.n_lags ? a.H[(int64_t)(t0 + j) * a.n_bins + b] : 0.0;
            re[j] += cs * h;
            im[j] += sn * h;
        }
    }
#pragma unroll
    for (int j = 0; j < kSqtLags; ++j) {
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) {
            re[j] += __shfl_down(re[j], w);
            im[j] += __shfl_down(im[j], w);
        }
        if ((threadIdx.x & 63) == 0) {
            red[threadIdx.x >> 6][2 * j] = re[j];
            red[threadIdx.x >> 6][2 * j + 1] = im[j];
        }
    }
    __syncthreads();
    if (threadIdx.x < 2 * kSqtLags) {
        const int j = threadIdx.x / 2, t = t0 + j;
        if (t < a.n_lags) {
            const double d = (double)a.n_sites * a.n_org[t], s = (red[0][threadIdx.x] + red[1][threadIdx.x]) +
                                                                 (red[2][threadIdx.x] + red[3][threadIdx.x]);
            a.sqt[((int64_t)qi * a.n_lags + t) * 2 + (threadIdx.x & 1)] = d > 0.0 ? s / d : 0.0;
        }
    }
}

// Windowed DFT over the lags of each q (same window as the site sums).  With
// n_org, x holds raw sums: they are divided by n_sites n_org[0] first, and the
// quotients stored in sqt.
__global__ __launch_bounds__(256) void sqw_kernel(const double* __restrict__ in, const double* __restrict__ n_org,
                                                  int64_t n_sites, double* __restrict__ sqt,
                                                  double* __restrict__ sqw, int m) {
    extern __shared__ double lds[];
    const int64_t at = (int64_t)blockIdx.y * m * 2;
    const double* x = in + at;
    const double d = n_org ? (double)n_sites * n_org[0] : 1.0;
    lag_dft<1>(
        m, (int)blockIdx.x * 64, lds,
        [&](int, int t, double& re, double& im) {
            re = x[2 * t];
            im = x[2 * t + 1];
            if (n_org) {
                re = d > 0.0 ? re / d : 0.0;
                im = d > 0.0 ? im / d : 0.0;
                if (blockIdx.x == 0) {
                    sqt[at + 2 * t] = re;
                    sqt[at + 2 * t + 1] = im;
                }
            }
        },
        [&](int, int k, double re, double im) {
            sqw[at + 2 * k] = re;
            sqw[at + 2 * k + 1] = im;
        });
}

int launch_sqw(const double* in, const double* n_org, int64_t n_sites, double* sqt, double* sqw, int n_q, int n_lags,
               void* stream) {
    for (int q = 0; q < n_q; q += 65535) {  // rows of one grid
        const int nq = n_q - q < 65535 ? n_q - q : 65535;
        const int64_t at = (int64_t)q * n_lags * 2;
        hipLaunchKernelGGL(sqw_kernel, dim3((unsigned)((n_lags + 63) / 64), (unsigned)nq), dim3(256),
                           lag_dft_lds<1>(n_lags), (hipStream_t)stream, in + at, n_org, n_sites,
                           sqt ? sqt + at : nullptr, sqw + at, n_lags);
    }
    return (int)hipGetLastError();
}

int launch_sqt(const SqtArgs& a, void* stream) {
    if (a.n_q == 0) return 0;
    hipLaunchKernelGGL(sqt_kernel, dim3((unsigned)a.n_q, (unsigned)((a.n_lags + kSqtLags - 1) / kSqtLags)), dim3(256),
                       0, (hipStream_t)stream, a);
    const int e = (int)hipGetLastError();
    return e != 0 ? e : launch_sqw(a.sqt, nullptr, 0, nullptr, a.sqw, a.n_q, a.n_lags, stream);
}

int launch_finalize(const FinalArgs& a, void* stream) {
    int64_t gx = a.C ? (a.n_bins + 255) / 256 : 1;
    if (gx > 256) gx = 256;
    const int64_t n_dft = (a.n_lags + 63) / 64;
    const int64_t gy = (a.C ? a.n_lags : 0) + (n_dft + gx - 1) / gx;
    hipLaunchKernelGGL(finalize_kernel, dim3((unsigned)gx, (unsigned)gy), dim3(256), lag_dft_lds<2>(a.n_lags),
                       (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

__global__ __launch_bounds__(256) void zero_kernel(ZeroRanges z) {
    for (int k = 0; k < z.n; ++k) {
        uint32_t* p = (uint32_t*)z.ptr[k];
        const int64_t words = z.bytes[k] / 4;
        for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < words;
             x += (int64_t)gridDim.x * blockDim.x)
            p[x] = 0u;
    }
}

__global__ void fixed_to_double_kernel(const unsigned long long* __restrict__ q, double* __restrict__ d, int64_t n) {
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x)
        d[x] = (double)(long long)q[x] / kFixedScale;
}

__global__ void double_to_fixed_kernel(const double* __restrict__ d, unsigned long long* __restrict__ q, int64_t n) {
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x)
        q[x] = to_fixed(d[x]);
}

static int64_t grid_for(int64_t n) {
    int64_t blocks = (n + 255) / 256;
    return blocks > 8192 ? 8192 : (blocks < 1 ? 1 : blocks);
}

int launch_fixed_to_double(const unsigned long long* q, double* d, int64_t n, void* stream) {
    if (n <= 0) return 0;
    hipLaunchKernelGGL(fixed_to_double_kernel, dim3((unsigned)grid_for(n)), dim3(256), 0, (hipStream_t)stream, q, d, n);
    return (int)hipGetLastError();
}

int launch_double_to_fixed(const double* d, unsigned long long* q, int64_t n, void* stream) {
    if (n <= 0) return 0;
    hipLaunchKernelGGL(double_to_fixed_kernel, dim3((unsigned)grid_for(n)), dim3(256), 0, (hipStream_t)stream, d, q, n);
    return (int)hipGetLastError();
}

int launch_zero_ranges(const ZeroRanges& z, void* stream) {
    int64_t words = 0;
    for (int k = 0; k < z.n; ++k) words = z.bytes[k] / 4 > words ? z.bytes[k] / 4 : words;
    if (words <= 0) return 0;
    int64_t blocks = (words + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, z);
    return (int)hipGetLastError();
}

int launch_zero(void* ptr, int64_t bytes, void* stream) {
    ZeroRanges z{};
    z.add(ptr, bytes);
    return launch_zero_ranges(z, stream);
}

// ---------------------------------------------------------------------------
// seeded spins (Philox)
// ---------------------------------------------------------------------------

// Independent uniform unit vectors for every (frame, site): Philox4x32-10,
// key = seed, counter = (site low, frame, site high, 7); z = 2u0 - 1,
// phi = 2 pi u1 (the autotuner's input; any spins time the same).
__global__ void unit_spins_kernel(float* __restrict__ out, int64_t n, int64_t n_frames, uint64_t seed) {
    const int64_t total = n * n_frames;
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < total;
         x += (int64_t)gridDim.x * blockDim.x) {
        const int64_t f = x / n, i = x - f * n;
        uint32_t c[4] = {(uint32_t)i, (uint32_t)f, (uint32_t)((uint64_t)i >> 32), 7u};
        philox4x32_10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
        const double z = 2.0 * ((double)(c[0] >> 8) * (1.0 / 16777216.0)) - 1.0;
        const double r = sqrt(fmax(0.0, 1.0 - z * z));
        double sn, cs;
        sincospi(2.0 * ((double)(c[1] >> 8) * (1.0 / 16777216.0)), &sn, &cs);
        out[3 * x] = (float)(r * cs);
        out[3 * x + 1] = (float)(r * sn);
        out[3 * x + 2] = (float)z;
    }
}

int launch_unit_spins(float* out, int64_t n, int64_t n_frames, uint64_t seed, void* stream) {
    const int64_t total = n * n_frames;
    if (total <= 0) return 0;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(unit_spins_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, out, n,
                       n_frames, seed);
    return (int)hipGetLastError();
}

}  // namespace sdc
