// Internal declarations of the sdc library: tile layout, kernel arguments and
// launch wrappers.  Not part of the public ABI (include/sdc.h).
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "sdc.h"

namespace sdc {

// Sites are grouped in tiles of 64.  Periodic lattices: a tile is a brick of
// at most 64 cells of one sublattice, slot (o0 s1 + o1) s2 + o2, or, where
// bricks would leave clearly more tiles, 64 consecutive cells in box order (see
// build_periodic).  Radial: 64 consecutive points in Morton order.  Unused
// slots are padding (zero spins, no counts).
constexpr int kTile = 64;
// Lags handled together by one fused task (consecutive lag indices u): 8
// for the reduced-precision forms (128 accumulator registers per wave for
// one set of sums), 16 for FP32: its MFMAs cover one workgroup's loads by
// themselves, and 8-lag groups in two workgroups per CU, which hide the
// epilogue, read three times the operands (fused ms with 16 / 8: sc 30^3 x 64
// origins x 128 lags 290 / 404, sq 100x100 31.7 / 35.1, sc 21x20x19 with
// stride 2, where 16 pads more, 21.0 / 19.4).
constexpr int lag_group(int precision) { return precision == SDC_PREC_FP32 ? 16 : 8; }
// Doubles between the LDS histogram rows of two bins: the group's lags side
// by side, so that the adds of an element's lags take constant offsets from
// one address (with a row per lag each add needs an address of its own), and
// an odd pitch, so that neighbouring bins lie in different banks.  A window
// has at most 512 bins (2 s_a per axis for bricks of s_0 s_1 s_2 <= 64
// cells, 508 for tiles in box order), a radial one 1024: 78 KB for 8-lag
// groups, two of which fit in a CU's LDS, and 143 KB for FP32's 16.  Together with the separate loop of
// the deterministic mode (one basic block of adds instead of one block per
// element) this took the fused launch from 1093 to 1081 ms at sc 36^3
// split-BF16, 58.8 to 57.3 ms on 20 011 points in 1024 shells, 30.8 to 28.2
// ms for FP32 at sc 21x20x19 and 9.0 to 8.5 ms for BF16x3 at 90x90 (each
// before the box-order tiles and the plane-wise packs).
constexpr int hist_pitch(int precision) { return lag_group(precision) + 1; }
// Schedules of the fused product (a tuning choice per plan and batch; the
// results differ only by rounding).  The small products of the reduced forms
// always get sums of their own (see the pass constants of the kernel).
//  kSchedOnePass: every product in one K loop per tile pair; the reduced
//    forms keep a second accumulator set for the small products (256
//    registers), so one workgroup fits on a CU; three-stage register
//    prefetch.  Every precision has it.
//  kSchedTwoPass: hi/lo splits only: per tile pair one K loop for hi*lo +
//    lo*hi from zero, then one for hi*hi on top of those sums, in the same
//    128 registers, then the histogram adds; two workgroups per CU, so one
//    workgroup's epilogue and memory waits overlap the other's MFMAs.
//  kSchedLagSplit: one K loop as in kSchedOnePass, but workgroups of eight
//    waves in which two waves share each 32x32 quadrant and take half of the
//    lag group each: 2 x 64 accumulator registers for the reduced forms (128
//    for FP32), two waves per SIMD.  Every precision.
//  kSchedFold: reduced forms only: one K loop; per K-step and lag the
//    small products are summed from zero in a transient 32x32 tile and added
//    to the large sums with FP32 vector adds (round to nearest, no bias),
//    beside the hi*hi MFMA; 128 accumulator registers, two workgroups per
//    CU.
constexpr int kSchedOnePass = 0, kSchedTwoPass = 1, kSchedLagSplit = 2, kSchedFold = 3;
constexpr int threads_per_wg(int sched) { return sched == kSchedLagSplit ? 512 : 256; }
// Register buffers of the K loops (loads of NS - 1 K-steps ahead in flight).
// At two workgroups per CU the other workgroup covers the rest of the load
// latency: two to six buffers in either loop of the two-pass schedule time
// the same (1085-1102 ms at sc 36^3), so the fewest registers win.
constexpr int kStagesOnePass = 3, kStagesTwoPassSmall = 2, kStagesTwoPassLarge = 2, kStagesFold = 2;
// Kernel schedule of a public sdc_schedule (ONE_PASS or TWO_PASS).
constexpr int sched_index(int schedule) {
    return schedule == SDC_SCHED_TWO_PASS  ? kSchedTwoPass
           : schedule == SDC_SCHED_LAG_SPLIT ? kSchedLagSplit
           : schedule == SDC_SCHED_FOLD      ? kSchedFold
                                             : kSchedOnePass;
}
constexpr int wg_per_cu(int sched) { return sched == kSchedTwoPass || sched == kSchedFold ? 2 : 1; }
// Waves per SIMD at that occupancy: the launch-bounds minimum that sets the
// register budget (four SIMDs per CU, 64-lane waves).
constexpr int waves_per_simd(int sched) { return wg_per_cu(sched) * threads_per_wg(sched) / 256; }
// The schedule a plan takes when nothing is asked for.
constexpr int default_sched(int precision) {
    return precision == SDC_PREC_SPLIT_BF16 || precision == SDC_PREC_SPLIT_FP16 ? kSchedTwoPass : kSchedOnePass;
}
constexpr bool sched_valid(int precision, int sched) {
    return sched == kSchedOnePass || sched == kSchedLagSplit ||
           (sched == kSchedTwoPass && (precision == SDC_PREC_SPLIT_BF16 || precision == SDC_PREC_SPLIT_FP16)) ||
           (sched == kSchedFold && precision != SDC_PREC_FP32);
}
// Pack elements (8 samples each) in one lane's B window: LG - 1 + 8 samples.
constexpr int win_blocks(int lg) { return (lg + 14) / 8; }
// Origins per pack block; a K-step of the fused product takes two blocks
// (one per lane half of the 32x32 MFMA), running over the blocks of all three
// components in turn.
constexpr int kOriginBlock = 8;

// One tile pair of a stream: i-tile, j-tile and the window shift of this pair.
struct KPair {
    int32_t ti, tj, shift, pad;
};

// A stream is a run of tile pairs whose epilogue shares one LDS histogram.
// Periodic: all pairs (I, I + db) for a fixed brick offset db and fixed
// sublattices; the histogram is indexed by the window coordinate and maps to
// global bins through base/parity.  Tiles in box order: all pairs of a fixed
// tile offset d and sublattices, those that wrap around the end apart; base[0]
// is the bin cell of window 0.  Radial: all pairs (I, J) of one I; the
// histogram is indexed by shell.
struct KStream {
    int32_t p0, p1;
    int32_t base[3];
    int32_t parity;
    int32_t pad[2];
};

// Lag group: lags t = s*(u0 + m) + phase for m in [0, 16) with bit m of mask.
struct KGroup {
    int32_t phase, u0, mask, pad;
};

struct Layout {
    int kind = 0;
    int L[3] = {0, 0, 0};
    int64_t n = 0;
    int64_t n_bins = 0;
    int64_t n_pad = 0;
    int32_t n_tiles = 0;
    int W[3] = {1, 1, 1};   // periodic window extents (bricks)
    bool linear = false;    // tiles in box order
    int win = 0;            // histogram bins per lag (window size or n_shells)
    int n_shells = 0;
    std::vector<int32_t> perm;   // [n_pad] original site index, -1 = padding
    std::vector<int32_t> gtab;   // [n_pad] window coordinate of the slot (box order: y << 16 | z of its cell)
    std::vector<float> pos4;     // [n_pad][4] radial positions, packed order
    std::vector<float> e2;       // [n_shells] radial squared edges
    std::vector<KPair> pairs;
    std::vector<KStream> streams;
};

// Records the thread-local error text returned by sdc_last_error(); returns s.
sdc_status set_error(sdc_status s, const std::string& msg);

// Builds the tile layout of a sample, streams cut into segments of at most
// segment_pairs tile pairs.  precision: the product's, which weighs the tile
// shapes against each other (-1: the fewest tiles).  Returns SDC_OK or an error
// with text.
sdc_status build_layout(const float* pos, int64_t n, const sdc_bin_spec* spec, int precision, int segment_pairs,
                        Layout* out, std::string* err);

// What the default segment length is called (sdc_tuning::segment_pairs): plans
// and tuning files hold these values, and the length is fitted_segment()'s.
constexpr int kDefaultSegmentPeriodic = 96;
constexpr int kMaxSegmentPairs = 1 << 20;
constexpr int default_segment_pairs(int kind) {
    return kind == SDC_BINS_RADIAL ? kMaxSegmentPairs : kDefaultSegmentPeriodic;
}

// Tuning a plan runs with (sdc_tune.cpp): the caller's fields where set,
// else the entry of the tuning file named by SDC_TUNING_FILE for the plan's
// size class, else the defaults.  Every field of *out is set (no zeros).
// *default_segment (may be null): the segment length is the default one, for
// fitted_segment() to choose.
sdc_status resolve_tuning(const sdc_tuning* given, int64_t n_sites, const sdc_bin_spec* bins,
                          const sdc_corr_spec* corr, int device, sdc_tuning* out, bool* default_segment = nullptr);

// Cuts every stream into consecutive, about equal segments of at most seg
// tile pairs.
std::vector<KStream> split_streams(const std::vector<KStream>& streams, int seg);
// Tile pairs per task that suit the whole streams of a layout run with
// n_groups lag groups by `slots` workgroups of a schedule at a time, as many as
// fit one launch where segments of up to kLongestSegmentPeriodic pairs
// (radial: whole streams) allow that.  alone: nothing else fills the slots.
constexpr int kFittedSegmentPeriodic = 32, kFittedSegmentRadial = 64, kLongestSegmentPeriodic = 128;
int fitted_segment(const Layout& lay, const std::vector<KStream>& whole, int n_groups, int64_t slots, int sched,
                   bool alone);
// Tasks of one fused launch: 2^32 - 1 threads in whole rows of 8 workgroups.
constexpr int64_t max_fused_tasks(int sched) { return (int64_t)UINT32_MAX / threads_per_wg(sched) / 8 * 8; }

#if defined(__HIPCC__)
#define SDC_HD __host__ __device__
#else
#define SDC_HD
#endif

// Tiles in box order.  Cell (x, y, z) is number (x L1 + y) L2 + z of its
// sublattice; a displacement's bin cell b = (kx L1 + ky) L2 + kz, k = (c_j - c_i
// - s) mod L (s = 1 from the second sublattice to the first, else 0), is
//   b = (j - i) - s (1 + L2 + L1 L2) + cz L2 + cy L1 L2  (mod the cells),
// j - i the difference of the cell numbers, cz = [z_j - s < z_i] and cy =
// [y_j - s < y_i] the borrows.  For a fixed tile offset j - i takes 127 values,
// so the window is 4 x 127: w = (slot_j - slot_i + 63) + 127 cz + 254 cy.
constexpr int kLinearSpan = 2 * kTile - 1, kLinearWin = 4 * kLinearSpan;
SDC_HD inline int linear_window(int slot_i, int gi, int slot_j, int gj, int s) {
    const int cz = ((gj & 0xFFFF) - s - (gi & 0xFFFF)) >> 31, cy = ((gj >> 16) - s - (gi >> 16)) >> 31;  // -1 or 0
    return slot_j - slot_i + (kTile - 1) - kLinearSpan * cz - 2 * kLinearSpan * cy;
}

// What maps a stream's window coordinates to global bins (periodic kinds).
struct WindowMap {
    int kind, linear, L0, L1, L2, W1, W2;
};

// Global bin of window coordinate w of stream s.
SDC_HD inline int64_t window_bin(const WindowMap& m, const KStream& s, int w) {
    int64_t b;
    if (m.linear) {
        const int q = w / kLinearSpan, r = w - q * kLinearSpan;
        const int64_t plane = (int64_t)m.L1 * m.L2;
        b = (s.base[0] + r + (int64_t)(q & 1) * m.L2 + (q >> 1) * plane) % (m.L0 * plane);
    } else {
        const int w0 = w / (m.W1 * m.W2), w1 = (w / m.W2) % m.W1, w2 = w % m.W2;
        int k0 = (s.base[0] + w0) % m.L0, k1 = (s.base[1] + w1) % m.L1, k2 = (s.base[2] + w2) % m.L2;
        if (k0 < 0) k0 += m.L0;
        if (k1 < 0) k1 += m.L1;
        if (k2 < 0) k2 += m.L2;
        b = ((int64_t)k0 * m.L1 + k1) * m.L2 + k2;
    }
    return m.kind == SDC_BINS_PERIODIC_BCC ? 2 * b + s.parity : b;
}
WindowMap window_map(const Layout& lay);

// Radial shell of a squared distance: the largest k with e2[k] <= d2.
#if defined(__HIPCC__)
__host__ __device__
#endif
inline int shell_of(float d2, const float* e2, int n_shells, float inv_w) {
    // first guess from the square root, then move to the exact rule
    float r = __builtin_sqrtf(d2);
    int k = (int)(r * inv_w);
    if (k < 0) k = 0;
    if (k > n_shells - 1) k = n_shells - 1;
    while (k > 0 && e2[k] > d2) --k;
    while (k + 1 < n_shells && e2[k + 1] <= d2) ++k;
    return k;
}

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of the
// multiply-xor bijection with Weyl key increments.  c is updated in place.
#if defined(__HIPCC__)
__host__ __device__
#endif
inline void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c[1] ^ k0;
        const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c[3] ^ k1;
        c[1] = (uint32_t)p1;
        c[3] = (uint32_t)p0;
        c[0] = n0;
        c[2] = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// FP32 squared distance in the fixed order ((dx*dx + dy*dy) + dz*dz), no
// contraction.
#if defined(__HIPCC__)
__host__ __device__
#endif
inline float dist2_f32(float xi, float yi, float zi, float xj, float yj, float zj) {
#pragma clang fp contract(off)
    float dx = xj - xi;
    float dy = yj - yi;
    float dz = zj - zi;
    float a = dx * dx;
    float b = dy * dy;
    float c = dz * dz;
    return (a + b) + c;
}

// ---------------------------------------------------------------------------
// Kernel launch wrappers (sdc_kernels.hip).  All return hipError_t as int.
// ---------------------------------------------------------------------------

struct PackArgs {
    const float* frames;  // [n_frames][n][3]
    int64_t n, n_frames, n_pad;
    const int32_t* perm;  // [n_pad]
    int n_origins, stride, precision;
    int O8;               // origin blocks of 8 in the A pack (per component)
    int F8;               // frame blocks of 8 in each B phase pack
    int n_phase;          // = stride
    int64_t frames_valid; // frames usable: min(n_frames, required)
    const float* mean;    // [n][4] per-site origin averages subtracted from A, or null
    void* A;              // [3 O8 + 1][n_pad] elements, or as many pieces per plane
    void* B;              // [n_phase][3][F8][n_pad], likewise
    double* mframe;       // [n_sums][3]: site-summed spin of the first n_sums frames
    int64_t n_sums;
};
int launch_pack(const PackArgs& a, void* stream);

struct FusedArgs {
    const void* A;
    const void* B;
    int64_t n_pad;
    int O8, F8;                    // origin blocks per component (A), window blocks (B)
    int nk;                        // K-steps: ceil(3 O8 / 2)
    int n_phase;                   // B phases (the origin stride)
    int64_t phase_stride;          // pieces (of a plane) or elements per B phase
    const KPair* pairs;
    const KStream* streams;
    int n_streams;
    const KGroup* groups;
    int n_groups;
    const int32_t* gtab;
    const float* pos4;
    const uint16_t* keys;          // radial: per-pair key tiles, or null (computed in the epilogue)
    const float* e2;
    int n_shells;
    float inv_w;
    WindowMap map;                 // periodic kinds
    int win;
    double* H;
    int det;                       // deterministic mode: fixed-point bins in Hq
    unsigned long long* Hq;
    int64_t n_bins;
    int stride;
    int precision;
    int sched;                     // kSchedOnePass / kSchedTwoPass
    int tail;                      // samples of the last K-step with an origin in either lane half
};
int launch_fused(const FusedArgs& a, void* stream);

// Most tasks of a batch: the claims of a queue, one too many per workgroup,
// stay within its 32-bit counter.
constexpr int64_t kMaxBatchTasks = 4000000000;
// One persistent launch over the tasks of several plans (same precision and
// bin class): args[n_plans] and task_start[n_plans + 1] in device memory,
// queue = 8 device counters (zeroed by the launch itself).
struct BatchLaunch {
    const FusedArgs* args;
    const int64_t* task_start;
    int n_plans;
    unsigned* queue;
    const int64_t* ranges;  // [9]: XCD queue x holds tasks [ranges[x], ranges[x + 1])
    int64_t total;          // at most kMaxBatchTasks
    int precision, radial, sched;
    int lds, grid;
};
int launch_fused_batch(const BatchLaunch& b, void* stream);
// Workgroups that fit on the device at once (a multiple of 8, at most `total`
// rounded up to 8).
int batch_grid(int precision, int sched, int radial, int lds, int device, int64_t total, int* grid);

struct CountArgs {
    const KPair* pairs;
    const KStream* streams;
    int n_streams;
    const int32_t* perm;
    const int32_t* gtab;
    const float* pos4;
    const float* e2;
    int n_shells;
    float inv_w;
    WindowMap map;
    int win;
    unsigned long long* counts;
};
int launch_count(const CountArgs& a, void* stream);
// Radial key table: keys[((p*4 + wave)*64 + lane)*16 + r] = shell of the pair
// element that accumulator register r of that lane holds for tile pair p.
int launch_radial_keys(const CountArgs& a, int64_t n_pairs, uint16_t* keys, void* stream);

struct SelfArgs {
    const float* frames;
    int64_t n, n_frames;
    int n_origins, stride;
    const int32_t* lags;  // device [n_sel]
    int n_sel;
    int64_t t_need;       // frames read: (n_origins - 1) * stride + max lag + 1
    double* self;         // [n_lags] indexed by lag value
    int precision;        // split precisions: add the diagonal lo*lo term to H
    double* H;            // [n_lags][n_bins]; the i = j pairs all fall in bin 0
    int64_t n_bins;
    double* norg;         // [n_lags] origin totals, += n_origins per selected lag
    const double* mframe; // [t_need][3] site-summed spin of each frame (from the pack launch)
    double* msum;         // [n_lags] += sum_o M(o s) . M(o s + t)
    const float* mean;    // [n][4] origin averages (connected form), or null
    int det;              // deterministic mode: fixed-point self sums and bins
    unsigned long long* selfq;
    unsigned long long* Hq;
};
int launch_self(const SelfArgs& a, void* stream);
// Per-site averages over the origins of one accumulate (connected form):
// mean[4 i + c] = fp32((1/n_o) sum_o S_i^c(o s)), summed in FP64.
int launch_mean(const float* frames, int64_t n, int n_origins, int stride, float* mean, void* stream);

struct FinalArgs {
    const double* H;
    const unsigned long long* counts;
    const double* n_org;   // device [n_lags]
    const double* self;    // device [n_lags]
    const double* msum;    // device [n_lags] site-summed raw correlation
    int64_t n_bins, n_sites;
    int n_lags;
    double* C;             // [n_lags][n_bins] or null
    unsigned long long* counts_out;  // [n_bins] or null: a copy of the counts beside C
    double* csum;          // [n_lags]
    double* cself;         // [n_lags]
    double* ssum;          // [n_lags][2]
    double* sself;         // [n_lags][2]
};
int launch_finalize(const FinalArgs& a, void* stream);

// S(q, t) of Eq. (3) from the bins of a periodic plan, for wave vectors
// q_a = 2 pi m_a / L_a (integer m), and its windowed time transform.
struct SqtArgs {
    const double* H;       // [n_lags][n_bins]
    const double* n_org;   // [n_lags]
    int64_t n_bins, n_sites;
    int n_lags;
    int kind, L0, L1, L2;  // periodic bin enumeration (sc / bcc)
    const int32_t* m;      // [n_q][3]
    int n_q;
    double* sqt;           // [n_q][n_lags][2]
    double* sqw;           // [n_q][n_lags][2]
};
int launch_sqt(const SqtArgs& a, void* stream);
// Windowed time transform over the lags of every q (the window of the site
// sums), (re, im) pairs: sqw[q][k] = sum_t w_t x[q][t] exp(-2 pi i k t / n_lags),
// x = in, or with n_org (device [1]) x = in / (n_sites n_org), stored in sqt.
int launch_sqw(const double* in, const double* n_org, int64_t n_sites, double* sqt, double* sqw, int n_q, int n_lags,
               void* stream);

// q-resolved S(q, t) of Eq. (3) at arbitrary wave vectors (sdc_sq.hip).
struct SqTransformArgs {
    const float* frames;      // [>= n_frames_used][n][3] fp32, caller's site order (pack input)
    float* packed;            // [ceil(n / chunk)][t_pad][chunk][3], chunk = sq_site_chunk() (pack output, contraction input)
    int t_pad;                // n_frames_used rounded up to whole 64-frame column blocks
    const float* pos;         // [n][3] fp32
    const double* q;          // [n_q][3]
    int64_t n;
    int n_q;
    int n_frames_used;        // (n_origins - 1) * stride + n_lags
    int n_split;              // site ranges, one partial transform each
    int64_t sites_per_split;
    double* part;             // [n_split][n_q][2][3 n_frames_used]
};
struct SqCorrArgs {
    double* F;                // [n_q][n_frames_used][3][2], written by the range sum
    int n_q;
    int64_t n_cols;           // 3 n_frames_used
    int n_origins, stride, n_lags;
    int connected;
    double* raw;              // [n_q][n_lags][2], accumulated
    double* n_org;            // [1] origins accumulated
};
// Workgroups of the transform per site range, and the sites one workgroup
// stages per step (site ranges are multiples of it).
int64_t sq_tiles_per_split(int n_q, int n_frames_used);
// Set the contraction kernel's dynamic-LDS limit on the current device.
int prepare_sq_kernels();
int sq_site_chunk();
int sq_frames_per_block();
// Packs the frames site-chunk-major (a.frames -> a.packed).
int launch_sq_pack(const SqTransformArgs& a, void* stream);
// The phase contraction alone (partial transforms of the site ranges).
int launch_sq_transform(const SqTransformArgs& a, void* stream);
// Sum of the site ranges into a.F, then the origin correlation.
int launch_sq_corr(const SqTransformArgs& t, const SqCorrArgs& a, void* stream);
int launch_sq_finalize(const double* raw, const double* n_org, int64_t n_sites, int n_q, int n_lags, double* sqt,
                       double* sqw, void* stream);

int launch_zero(void* ptr, int64_t bytes, void* stream);
// Several ranges (whole 32-bit words) cleared in one launch.
struct ZeroRanges {
    void* ptr[6];
    int64_t bytes[6];
    int n;
    void add(void* p, int64_t b) {
        ptr[n] = p;
        bytes[n++] = b;
    }
};
int launch_zero_ranges(const ZeroRanges& z, void* stream);

// Fixed device scratch of the entry points that allocate nothing
// (sdc_static.hip): kStaticScratchBytes per device, shared by every call on
// that device.  static_scratch() returns the device address of `device`'s
// copy, looked up on the first call for that device (with it current).
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
int static_scratch(int device, void** ptr);

// Deterministic mode: every sum that several threads add into is kept as a
// two's-complement 64-bit fixed-point number with 2^-20 resolution, so
// integer atomics make the result independent of the order of the adds.
constexpr double kFixedScale = 1048576.0;
int launch_fixed_to_double(const unsigned long long* q, double* d, int64_t n, void* stream);
int launch_double_to_fixed(const double* d, unsigned long long* q, int64_t n, void* stream);

struct TrajArgs {
    int64_t n;
    int z_max;                 // neighbours per site (ELL width)
    const int32_t* nbr;        // [n][z_max], -1 = none
    const float* jval;         // [n][z_max]
    const float* dvec;         // [n][z_max][3] DMI vectors D_ij, or null
    float aniso2, hz;          // 2 A and H_z of Eq. (1)
    float dt;
    int init, pad;
    double sigma;
    uint64_t seed;
    const float* init_dev;
    float* frames;             // [n_frames][n][3]
    int64_t n_frames;
    float* work;               // [3][n][3] fp32 scratch of the bond tables' stages: two stage states, acc
    // Periodic sc box L0 x L1 x L2 with one uniform coupling, sites in the order
    // (x L1 + y) L2 + z: a whole step per launch, no tables (nbr, jval, dvec and
    // work null).  DMI vectors (st_dp, st_dz, st_dz) rotated onto each axis,
    // st_dn for the negative directions.
    int stencil, st_dmi;
    int L[3];
    float st_j, st_dp, st_dn, st_dz;
};
// Bricks of the one-launch step: b cells per axis (nb of them), tile t with halo.
struct TrajBrick {
    int L[3], b[3], t[3], nb[3], halo[3];
    float J, dp, dn, dz;
};
int launch_traj(const TrajArgs& a, void* stream);
// Seeded independent uniform unit vectors, [n_frames][n][3] fp32.
int launch_unit_spins(float* out, int64_t n, int64_t n_frames, uint64_t seed, void* stream);

// Metropolis sweeps (sdc_mc.hip).
struct McArgs {
    int64_t n;
    int z_max;
    const int32_t* site_of;    // [n] site of each slot (slots colour-major)
    const int32_t* nbr;        // [n slots][z_max] neighbour slots, -1 = none
    const float* jval;         // [n slots][z_max]
    const float* dvec;         // [n slots][z_max][3] DMI vectors, or null
    double A, Hz;              // anisotropy and field of Eq. (1)
    uint64_t seed;             // Philox key of the moves
    double acc_target;         // acceptance-rate target of the cone adaptation
    double* S;                 // [n slots][3] FP64 state
    double* cone;              // [2][2]: cone half-angle and its cosine before even and odd sweeps
    unsigned long long* accepted;  // accepted moves of the current sweep (mc_counter_bytes())
    // Lattice stencil (set only when the host has checked that it reproduces
    // the tables above slot for slot): periodic sc box L0 x L1 x L2, every edge
    // even, site (x L1 + y) L2 + z, two colour classes (the checkerboard),
    // class c in slots c n/2 .. (c + 1) n/2 in site order, bonds +x, -x, +y,
    // -y, +z, -z with coupling st_j and DMI vectors (st_dp, st_dz, st_dz)
    // rotated onto each axis, st_dn for the negative directions.
    int stencil;
    int L0, L1, L2;
    double inv_L1, inv_L2;     // 1 / L1, 1 / L2
    float st_j, st_dp, st_dn, st_dz;
};
int mc_energy_blocks(int64_t n);
size_t mc_counter_bytes();
// Samples whose sweeps one workgroup of 512 threads runs with the state in
// LDS.  Per sweep of two classes, one workgroup against one launch per class:
// 512 sites per class 5.0 / 9.1 us, 648: 6.5 / 9.2, 800: 8.7 / 9.1, 1024:
// 8.5 / 9.1, 1408: 12.4 / 9.0; the line leaves room for couplings that cost
// more per site (with DMI 800 sites take 10.1 / 9.5).  Open samples with more
// bonds, read one by one, gain as well, also where a class takes two turns:
// sc 13^3 within 1.5 (18 bonds, four classes of about 550 sites) 38.6 / 43.1, 14^3
// (690 sites) 40.8 / 44.5, sc 15^3 within 2.5 (80 bonds, 31 classes) 625 / 983.
constexpr int kMcSmallSites = 4096, kMcSmallClassSites = 768, kMcSmallClasses = 32;
// A stretch of the annealing schedule: `count` sweeps from number `sweep` on,
// the first at temperature T after `done` of its per_T sweeps.
struct McSmall {
    double T, T_end, cool;
    int64_t per_T, done, sweep, count;
    int n_classes;
    int class_start[kMcSmallClasses + 1];
};
bool mc_is_small(int64_t n, const int64_t* class_start, int n_classes);
int launch_mc_small(const McArgs& a, const McSmall& m, long long* history, void* stream);
// Set the dynamic-LDS limit of the sample's kernel on the current device.
int prepare_mc_small(const McArgs& a);
// Loads init (fp32, or keeps the FP64 state when init is null), sets the cone.
int launch_mc_setup(const McArgs& a, const float* init, double cone0, void* stream);
// One sweep: every colour class in order (class c = slots class_start[c] ..
// class_start[c + 1]), the last one ending with the cone update
// (history[sweep] receives the accepted moves when history is not null).
int launch_mc_sweep(const McArgs& a, const int64_t* class_start, int n_classes, double T, int64_t sweep,
                    long long* history, void* stream);
// Energy per site, cone after n_sweeps sweeps and temperature into
// info[0..2]; state as fp32.
int launch_mc_finish(const McArgs& a, double* partial, int64_t n_sweeps, double T_last, float* out, double* info,
                     void* stream);

int fused_lds_bytes(int win, int precision);
// Largest dynamic LDS of a fused launch (the CU's 160 KB less room for the
// batch kernel's few static words) and the self kernel's budget for the
// samples of one site (beside at most 16 KB of lag sums).
constexpr int kMaxFusedLds = 160 * 1024 - 256;
constexpr int64_t kSelfLdsBudget = 96 * 1024;
// Set the kernels' dynamic-LDS limits on the current device.
int prepare_kernels();

}  // namespace sdc
