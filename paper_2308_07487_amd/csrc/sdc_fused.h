// The fused product and its binning epilogue (Sec. 3.3-3.4, Fig. 2, Eq. (6)).
// Each precision is compiled in a file of its own (sdc_fused_*.hip).
#pragma once

#include "sdc_device.h"

namespace sdc {

// ---------------------------------------------------------------------------
// fused product + binning epilogue
// ---------------------------------------------------------------------------
//
// Work: task = (lag group, stream).  A workgroup of 4 waves takes one task
// and walks the stream's tile pairs (64 i-sites x 64 j-sites).  Wave w owns
// the 32x32 quadrant (w >> 1, w & 1) for all LG lags of the group: LG MFMA
// accumulator tiles.  The K loop runs over the 3 components and over
// K-steps of 16 origins; in a K-step, lane (i, h) holds origins
// 16c + 8h + [0, 8) of its site and lane (j, h) holds the 8*NB samples
// 16c + 8h + u0 + [0, 8*NB) of its site, from which the operand of lag
// u0 + m is the 8-sample slice starting at m (a register select for even m,
// a byte align for odd m).  No operand goes through LDS; LDS holds the
// histogram.  Two workgroups share a CU, so one workgroup's epilogue and
// memory waits overlap the other's MFMA work.

__device__ inline uint32_t align2(uint32_t hi, uint32_t lo) {
    return __builtin_amdgcn_alignbyte(hi, lo, 2);
}

// Operand of lag u0 + M: the 8 halves starting at window element M.
template <int M, int NW>
__device__ inline uint4 slice8(const uint32_t (&w)[NW]) {
    constexpr int e = M / 2;
    static_assert(e + 4 + (M & 1) <= NW, "window too short");
    if constexpr ((M & 1) == 0) {
        return make_uint4(w[e], w[e + 1], w[e + 2], w[e + 3]);
    } else {
        return make_uint4(align2(w[e + 1], w[e]), align2(w[e + 2], w[e + 1]),
                          align2(w[e + 3], w[e + 2]), align2(w[e + 4], w[e + 3]));
    }
}

template <int PREC>
__device__ inline f32x16 mfma16(uint4 a, uint4 b, f32x16 c) {
    if constexpr (PREC == SDC_PREC_SPLIT_BF16 || PREC == SDC_PREC_BF16X3) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    } else {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
}

// Products one K loop forms (PASS):
//  kPassAll   : every product of the form; the large ones into acc.v, the
//               small ones into acc.s (one-pass and lag-split schedules);
//  kPassSmall : hi*lo + lo*hi into acc.v (first loop of the two-pass
//               schedule, from zero);
//  kPassLarge : hi*hi into acc.v (second loop, on top of the small sums).
// The small products are never added to a sum that already holds the large
// ones: the BF16/FP16 matrix cores align every addend of an instruction to
// the largest one and drop the bits that fall below a fixed window, always
// downwards, so the low bits of small products added to a large sum would
// bias each element by a fraction of its last place per K-step.  Added to a
// sum of their own size they keep every bit, and the large products added
// afterwards (16 significant bits each) lose none either.
//  kPassFold  : every product of the form; per K-step and lag the small
//               products are summed from zero in a transient tile, which FP32
//               vector adds (round to nearest) then add to acc.v, next to
//               the hi*hi MFMA (fold schedule).
constexpr int kPassAll = 0, kPassLarge = 1, kPassSmall = 2, kPassFold = 3;

__device__ inline void add16(f32x16& acc, const f32x16& t) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] += t[r];
}

// Three-product split for the wave's lag M (its window slice OFF + M):
// hi*hi + hi*lo + lo*hi.
template <int PREC, int PASS, int OFF, int M, int NW, int LW>
__device__ inline void split_step(const Chunk& av, const uint32_t (&wh)[NW],
                                  const uint32_t (&wl)[NW], f32x16 (&acc)[LW], f32x16 (&acc_s)[LW]) {
    const uint4 bh = slice8<OFF + M, NW>(wh);
    if constexpr (PASS == kPassLarge) {
        acc[M] = mfma16<PREC>(av.x, bh, acc[M]);
    } else {
        const uint4 bl = slice8<OFF + M, NW>(wl);
        if constexpr (PASS == kPassAll) {
            acc[M] = mfma16<PREC>(av.x, bh, acc[M]);
            acc_s[M] = mfma16<PREC>(av.x, bl, acc_s[M]);
            acc_s[M] = mfma16<PREC>(av.y, bh, acc_s[M]);
        } else if constexpr (PASS == kPassFold) {
            f32x16 t = {};
            t = mfma16<PREC>(av.x, bl, t);
            t = mfma16<PREC>(av.y, bh, t);
            acc[M] = mfma16<PREC>(av.x, bh, acc[M]);
            add16(acc[M], t);
        } else {
            acc[M] = mfma16<PREC>(av.x, bl, acc[M]);
            acc[M] = mfma16<PREC>(av.y, bh, acc[M]);
        }
    }
}

// Three-piece BF16 for the wave's lag M: the six products hh, hm, mh, mm,
// hl, lh (the dropped ml, lm, ll are below 2^-24 of the product); hh goes to
// the main accumulator, the other five (2^-8 and smaller) to the second one.
template <int OFF, int M, int NW, int LW>
__device__ inline void x3_step(const Chunk3& av, const uint32_t (&wh)[NW], const uint32_t (&wm)[NW],
                               const uint32_t (&wl)[NW], f32x16 (&acc)[LW], f32x16 (&acc_s)[LW]) {
    const uint4 bh = slice8<OFF + M, NW>(wh);
    const uint4 bm = slice8<OFF + M, NW>(wm);
    const uint4 bl = slice8<OFF + M, NW>(wl);
    acc[M] = mfma16<SDC_PREC_BF16X3>(av.x, bh, acc[M]);
    acc_s[M] = mfma16<SDC_PREC_BF16X3>(av.x, bm, acc_s[M]);
    acc_s[M] = mfma16<SDC_PREC_BF16X3>(av.y, bh, acc_s[M]);
    acc_s[M] = mfma16<SDC_PREC_BF16X3>(av.y, bm, acc_s[M]);
    acc_s[M] = mfma16<SDC_PREC_BF16X3>(av.x, bl, acc_s[M]);
    acc_s[M] = mfma16<SDC_PREC_BF16X3>(av.z, bh, acc_s[M]);
}

// The same with the small products folded into the main sums per K-step.
template <int OFF, int M, int NW, int LW>
__device__ inline void x3_fold_step(const Chunk3& av, const uint32_t (&wh)[NW], const uint32_t (&wm)[NW],
                                    const uint32_t (&wl)[NW], f32x16 (&acc)[LW]) {
    const uint4 bh = slice8<OFF + M, NW>(wh);
    const uint4 bm = slice8<OFF + M, NW>(wm);
    const uint4 bl = slice8<OFF + M, NW>(wl);
    f32x16 t = {};
    t = mfma16<SDC_PREC_BF16X3>(av.x, bm, t);
    t = mfma16<SDC_PREC_BF16X3>(av.y, bh, t);
    t = mfma16<SDC_PREC_BF16X3>(av.y, bm, t);
    t = mfma16<SDC_PREC_BF16X3>(av.x, bl, t);
    t = mfma16<SDC_PREC_BF16X3>(av.z, bh, t);
    acc[M] = mfma16<SDC_PREC_BF16X3>(av.x, bh, acc[M]);
    add16(acc[M], t);
}

template <int OFF, int NW, int LW, int... Ms>
__device__ inline void x3_all(const Chunk3& av, const uint32_t (&wh)[NW], const uint32_t (&wm)[NW],
                              const uint32_t (&wl)[NW], f32x16 (&acc)[LW], f32x16 (&acc_s)[LW],
                              std::integer_sequence<int, Ms...>) {
    (x3_step<OFF, Ms, NW, LW>(av, wh, wm, wl, acc, acc_s), ...);
}

template <int OFF, int NW, int LW, int... Ms>
__device__ inline void x3_fold_all(const Chunk3& av, const uint32_t (&wh)[NW], const uint32_t (&wm)[NW],
                                   const uint32_t (&wl)[NW], f32x16 (&acc)[LW], std::integer_sequence<int, Ms...>) {
    (x3_fold_step<OFF, Ms, NW, LW>(av, wh, wm, wl, acc), ...);
}

template <int PREC, int PASS, int OFF, int NW, int LW, int... Ms>
__device__ inline void split_all(const Chunk& av, const uint32_t (&wh)[NW], const uint32_t (&wl)[NW],
                                 f32x16 (&acc)[LW], f32x16 (&acc_s)[LW], std::integer_sequence<int, Ms...>) {
    (split_step<PREC, PASS, OFF, Ms, NW, LW>(av, wh, wl, acc, acc_s), ...);
}

// FP32: MFMA q of the K-step takes origin 16c + 8h + q on both sides.
template <int Q, int OFF, int M, int NF, int LW>
__device__ inline void f32_step(const float (&a)[8], const float (&w)[NF], f32x16 (&acc)[LW]) {
    acc[M] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[Q], w[Q + OFF + M], acc[M], 0, 0, 0);
}
template <int Q, int OFF, int NF, int LW, int... Ms>
__device__ inline void f32_q(const float (&a)[8], const float (&w)[NF], f32x16 (&acc)[LW],
                             std::integer_sequence<int, Ms...>) {
    (f32_step<Q, OFF, Ms, NF, LW>(a, w, acc), ...);
}
template <int OFF, int NF, int LW, int... Qs>
__device__ inline void f32_all(const float (&a)[8], const float (&w)[NF], f32x16 (&acc)[LW],
                               std::integer_sequence<int, Qs...>) {
    (f32_q<Qs, OFF, NF, LW>(a, w, acc, std::make_integer_sequence<int, LW>{}), ...);
}
// The first nq (uniform) of them; the operands move down a register per turn.
template <int OFF, int NF, int LW>
__device__ inline void f32_first(int nq, float (&a)[8], float (&w)[NF], f32x16 (&acc)[LW]) {
    for (int q = 0; q < nq; ++q) {
        f32_q<0, OFF, NF, LW>(a, w, acc, std::make_integer_sequence<int, LW>{});
#pragma unroll
        for (int e = 0; e < 7; ++e) a[e] = a[e + 1];
#pragma unroll
        for (int e = 0; e < NF - 1; ++e) w[e] = w[e + 1];
    }
}

// Accumulators of one wave: LW 32x32 tiles, and for the schedules that
// keep them apart a second set for the small products of the reduced forms.
template <int PREC, int SCHED, int LW>
struct Acc {
    f32x16 v[LW];
    f32x16 s[(PREC == SDC_PREC_FP32 || SCHED == kSchedTwoPass || SCHED == kSchedFold) ? 1 : LW];
};

// Operands of one K-step for one lane: A (8 origins, hi/lo or fp32) and the
// B window of NB pack elements.
template <int PREC, int NB>
struct Stage {
    PackElem<PREC> a;
    PackElem<PREC> b[NB];
};

template <int PREC, int PASS, int SCHED, int NB, int LW, int OFF>
__device__ inline void stage_mma(const Stage<PREC, NB>& s, Acc<PREC, SCHED, LW>& ac, int nq = 8) {
    f32x16 (&acc)[LW] = ac.v;
    constexpr int NW = 4 * NB;
    if constexpr (PREC == SDC_PREC_BF16X3) {
        uint32_t wh[NW], wm[NW], wl[NW];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const uint32_t h4[4] = {s.b[k].x.x, s.b[k].x.y, s.b[k].x.z, s.b[k].x.w};
            const uint32_t m4[4] = {s.b[k].y.x, s.b[k].y.y, s.b[k].y.z, s.b[k].y.w};
            const uint32_t l4[4] = {s.b[k].z.x, s.b[k].z.y, s.b[k].z.z, s.b[k].z.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                wh[4 * k + e] = h4[e];
                wm[4 * k + e] = m4[e];
                wl[4 * k + e] = l4[e];
            }
        }
        if constexpr (PASS == kPassFold)
            x3_fold_all<OFF, NW, LW>(s.a, wh, wm, wl, acc, std::make_integer_sequence<int, LW>{});
        else
            x3_all<OFF, NW, LW>(s.a, wh, wm, wl, acc, ac.s, std::make_integer_sequence<int, LW>{});
    } else if constexpr (PREC == SDC_PREC_FP32) {
        float af[8], w[8 * NB];
        const uint32_t ar[8] = {s.a.x.x, s.a.x.y, s.a.x.z, s.a.x.w, s.a.y.x, s.a.y.y, s.a.y.z, s.a.y.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) af[e] = __uint_as_float(ar[e]);
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const uint32_t r[8] = {s.b[k].x.x, s.b[k].x.y, s.b[k].x.z, s.b[k].x.w,
                                   s.b[k].y.x, s.b[k].y.y, s.b[k].y.z, s.b[k].y.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) w[8 * k + e] = __uint_as_float(r[e]);
        }
        if (__builtin_constant_p(nq) && nq == 8)
            f32_all<OFF, 8 * NB, LW>(af, w, acc, std::make_integer_sequence<int, 8>{});
        else
            f32_first<OFF, 8 * NB, LW>(nq, af, w, acc);
    } else {
        uint32_t wh[NW], wl[NW];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            wh[4 * k] = s.b[k].x.x;
            wh[4 * k + 1] = s.b[k].x.y;
            wh[4 * k + 2] = s.b[k].x.z;
            wh[4 * k + 3] = s.b[k].x.w;
            wl[4 * k] = s.b[k].y.x;
            wl[4 * k + 1] = s.b[k].y.y;
            wl[4 * k + 2] = s.b[k].y.z;
            wl[4 * k + 3] = s.b[k].y.w;
        }
        // the two-pass schedule has no second accumulator set (its passes
        // never write one)
        if constexpr (SCHED == kSchedTwoPass || SCHED == kSchedFold)
            split_all<PREC, PASS, OFF, NW, LW>(s.a, wh, wl, acc, acc, std::make_integer_sequence<int, LW>{});
        else
            split_all<PREC, PASS, OFF, NW, LW>(s.a, wh, wl, acc, ac.s, std::make_integer_sequence<int, LW>{});
    }
}

// MFMA instructions one stage_mma call issues per wave.
template <int PREC, int PASS, int LW>
constexpr int mfma_per_stage() {
    if constexpr (PREC == SDC_PREC_FP32) return 8 * LW;
    else if constexpr (PREC == SDC_PREC_BF16X3) return 6 * LW;
    else if constexpr (PASS == kPassLarge) return LW;
    else if constexpr (PASS == kPassSmall) return 2 * LW;
    else return 3 * LW;
}

// Instruction order of one K-step for the schedules with a second
// accumulator set (one-pass, lag-split): the next stage's loads first, then
// each MFMA followed by up to NV vector instructions (the operand shuffles of
// the following lags), so that the shuffles issue while the matrix core works
// instead of in a burst in front of it (about 5% at the 36^3 workload).  The
// two-pass and fold loops keep the compiler's order with the loads fenced
// off from the MFMAs: there the interleave gains nothing (two-pass) or costs
// register spills (fold, and the batch kernel).
template <int NMF, int NV>
__device__ __forceinline__ void interleave() {
    __builtin_amdgcn_sched_group_barrier(0x020, 16, 0);  // vector memory reads
#pragma unroll
    for (int i = 0; i < NMF; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, NV, 0);  // vector ALU
    }
}

// One K loop over all K-steps of a tile pair with NS register buffers: the
// loads of the next NS - 1 K-steps are in flight while one step's MFMAs run
// (load indices clamp to the last step, so the last round's extra loads are
// harmless re-reads).  For the interleaved schedules the main loop takes NS
// steps per trip without a branch, so loads and MFMAs of a step share one
// scheduling region, and the fewer than NS steps left after it (loaded
// already) follow; the others skip the steps past the end inside the loop
// and fence the loads off from the MFMAs.
// FP32, one-pass: the samples of the last step past `tail` are zero in both
// lane halves (a component's last origins and the zero block) and are left
// out: a sum is the same without a zero product.  The steps after the loop
// share one short body for it.  Fused ms before / after: sc 21x20x19 x 100
// lags, 50 origins (2 of the last step's 8) 21.0 / 19.9; 64 origins, where it
// is the short body alone, sc 30^3 x 128 lags 290 / 283, 24^3 x 40 25.4 / 24.7
// (lag-split had it cost 4% at the first of these and keeps its own steps).
template <int PREC, int PASS, int SCHED, int NB, int LW, int OFF, int NS, class Load>
__device__ __forceinline__ void k_loop(int nk, int tail, const Load& load, Acc<PREC, SCHED, LW>& acc) {
    Stage<PREC, NB> s[NS];
#pragma unroll
    for (int j = 0; j < NS - 1; ++j) load(s[j], j);
    if constexpr (SCHED == kSchedOnePass || SCHED == kSchedLagSplit) {
        constexpr int NMF = mfma_per_stage<PREC, PASS, LW>();
        constexpr bool TAIL = PREC == SDC_PREC_FP32 && SCHED == kSchedOnePass;  // the loop leaves the last step
        int kk = 0;
        for (; kk + NS + TAIL <= nk; kk += NS) {
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                load(s[(j + NS - 1) % NS], kk + j + NS - 1);
                stage_mma<PREC, PASS, SCHED, NB, LW, OFF>(s[j], acc);
                interleave<NMF, 4>();
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (TAIL) {
            load(s[NS - 1], kk + NS - 1);
#pragma unroll
            for (int j = 0; j < NS; ++j)
                if (kk + j < nk) stage_mma<PREC, PASS, SCHED, NB, LW, OFF>(s[j], acc, kk + j + 1 < nk ? 8 : tail);
        } else {
#pragma unroll
            for (int j = 0; j < NS - 1; ++j)
                if (kk + j < nk) stage_mma<PREC, PASS, SCHED, NB, LW, OFF>(s[j], acc);
        }
    } else {
        for (int kk = 0; kk < nk; kk += NS) {
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                load(s[(j + NS - 1) % NS], kk + j + NS - 1);
                __builtin_amdgcn_sched_barrier(0);
                if (j == 0 || kk + j < nk) stage_mma<PREC, PASS, SCHED, NB, LW, OFF>(s[j], acc);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

// What the tile-pair loop of one wave needs of its task.
struct TaskCtx {
    const FusedArgs* a;
    KGroup grp;
    KStream st;
    double* hist;
    const float* e2s;
    int quadrant;  // 32x32 quadrant of the 64x64 tile pair (wave index mod 4)
};

// The tile pairs of a task for one wave: its quadrant, its LW lags starting
// at lag OFF of the group (all LG of them unless the lag-split schedule
// gives the group's two halves to two waves).
template <int PREC, int RADIAL, int PAIRED, int SCHED, int LW, int OFF>
__device__ __forceinline__ void pair_loop(const TaskCtx& c) {
    constexpr int LG = lag_group(PREC);
    constexpr int NB = win_blocks(LG);
    constexpr int PITCH = hist_pitch(PREC);
    constexpr bool TWO = SCHED == kSchedTwoPass;
    constexpr bool FOLD = SCHED == kSchedFold;
    const FusedArgs& a = *c.a;
    const KGroup grp = c.grp;
    double* hist = c.hist;
    const int lane = threadIdx.x & 63;
    const int wi = c.quadrant >> 1, wj = c.quadrant & 1, h = lane >> 5, l32 = lane & 31;

    using Elem = PackUnit<PREC>;
    const Elem* Ab = (const Elem*)a.A;
    const Elem* Bb = (const Elem*)a.B + (int64_t)grp.phase * a.phase_stride;
    // K-steps run over the 3 O8 origin blocks of all components, two blocks
    // per step (one per lane half); a half past the last block reads the A
    // pack's zero block 3 O8
    const int nk = a.nk;
    const int nblk = 3 * a.O8;
    const int ublk = grp.u0 / 8;
    const int dF = a.F8 - a.O8;  // B block of A block k (component c): k + c dF + ublk
    const int n_c = a.O8 / 2;    // PAIRED: K-steps per component

    // lane byte offsets from a block's tile base: the site within the tile
    // and, for the upper lane half, the next block (the plan keeps two pack
    // blocks within 4 GiB)
    const uint32_t offA = (uint32_t)(((int64_t)h * a.n_pad + wi * 32 + l32) * (int64_t)sizeof(Elem));
    const uint32_t offB = (uint32_t)(((int64_t)h * a.n_pad + wj * 32 + l32) * (int64_t)sizeof(Elem));

    for (int p = c.st.p0; p < c.st.p1; ++p) {
        const KPair pr = a.pairs[p];
        const int64_t sj = (int64_t)pr.tj * kTile + wj * 32 + l32;
        Acc<PREC, SCHED, LW> acc;
#pragma unroll
        for (int m = 0; m < LW; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc.v[m][r] = 0.0f;
        if constexpr (PREC != SDC_PREC_FP32 && !TWO && !FOLD) {
#pragma unroll
            for (int m = 0; m < LW; ++m)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc.s[m][r] = 0.0f;
        }

        // Register buffers: while K-step kk is multiplied the loads of later
        // steps are in flight (indices clamp to the last block).  Parts of
        // an element a pass does not use are not loaded (dead loads).  Each
        // load is a uniform block address plus the lane's fixed byte offset.
        const Elem* At = Ab + (int64_t)pr.ti * kTile;
        const Elem* Bt = Bb + (int64_t)pr.tj * kTile;
        auto load = [&](Stage<PREC, NB>& b, int kk) {
            kk = kk < nk ? kk : nk - 1;
            const int64_t np = a.n_pad;
            // A block of lane half h: 2 kk + h (the zero block for the half
            // past the last block)
            const Elem* pa = At + (int64_t)(2 * kk) * np;
            const Elem* pb;
            uint32_t ob = offB;
            if constexpr (PAIRED) {
                // both halves in component alpha: B block 2 kk + h + alpha dF + ublk
                const int alpha = (kk >= n_c) + (kk >= 2 * n_c);
                pb = Bt + (int64_t)(2 * kk + alpha * dF + ublk) * np;
            } else {
                // block indices of both lane halves from the step index
                // (uniform); A: [3][O8] blocks flattened, then the zero block
                const int k0 = 2 * kk;
                const int k1 = k0 + 1 < nblk ? k0 + 1 : nblk - 1;
                const int b0 = k0 + ((k0 >= a.O8) + (k0 >= 2 * a.O8)) * dF + ublk;
                const int b1 = k1 + ((k1 >= a.O8) + (k1 >= 2 * a.O8)) * dF + ublk;
                pb = Bt + (int64_t)b0 * np;
                // offB holds one block for the upper half; it needs b1 - b0
                ob += h ? (uint32_t)((int64_t)(b1 - b0 - 1) * np * (int64_t)sizeof(Elem)) : 0u;
            }
            if constexpr (pack_planes(PREC)) {
                b.a.x = *(const Elem*)((const char*)pa + offA);
                b.a.y = *(const Elem*)((const char*)(pa + pack_plane_a(a)) + offA);
#pragma unroll
                for (int q = 0; q < NB; ++q) {
                    b.b[q].x = *(const Elem*)((const char*)(pb + q * np) + ob);
                    b.b[q].y = *(const Elem*)((const char*)(pb + q * np + pack_plane_b(a)) + ob);
                }
            } else {
                b.a = *(const PackElem<PREC>*)((const char*)pa + offA);
#pragma unroll
                for (int q = 0; q < NB; ++q) b.b[q] = *(const PackElem<PREC>*)((const char*)(pb + q * np) + ob);
            }
        };

        // Epilogue: bin of each accumulator element, LDS FP64 add per lag.
        // Accumulator register r of lane (l32, h) holds row 8(r/4) + 4h + r%4,
        // column l32 of the wave's 32x32 quadrant.
        int bin[16];
        auto bins = [&]() {
            const int64_t rowbase = (int64_t)pr.ti * kTile + wi * 32 + 4 * h;
            if constexpr (RADIAL) {
                if (a.keys) {
                    // the pair's shells, computed once per plan for all lag groups
                    const uint4* kp =
                        (const uint4*)(a.keys + (((int64_t)p * 4 + c.quadrant) * 64 + lane) * 16);
                    const uint4 k0 = kp[0], k1 = kp[1];
                    const uint32_t kw[8] = {k0.x, k0.y, k0.z, k0.w, k1.x, k1.y, k1.z, k1.w};
#pragma unroll
                    for (int r = 0; r < 16; ++r) bin[r] = (int)((kw[r / 2] >> (16 * (r & 1))) & 0xFFFFu);
                } else {
                    const float4 pj = *(const float4*)(a.pos4 + 4 * sj);
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float4 pi = *(const float4*)(a.pos4 + 4 * (rowbase + 8 * (r / 4) + (r % 4)));
                        const float d2 = dist2_f32(pi.x, pi.y, pi.z, pj.x, pj.y, pj.z);
                        bin[r] = shell_of(d2, c.e2s, a.n_shells, a.inv_w);
                    }
                }
            } else if (a.map.linear) {
                const int gj = a.gtab[sj];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = 8 * (r / 4) + (r % 4);
                    bin[r] = linear_window(wi * 32 + 4 * h + row, a.gtab[rowbase + row], wj * 32 + l32, gj, pr.shift);
                }
            } else {
                const int gj = a.gtab[sj] + pr.shift;
#pragma unroll
                for (int r = 0; r < 16; ++r) bin[r] = gj - a.gtab[rowbase + 8 * (r / 4) + (r % 4)];
            }
        };
        // One LDS add per element, at its bin's row plus the lag's constant
        // offset (see hist_pitch).  The deterministic mode is a loop of its
        // own: a test per element would cut the adds into basic blocks of one.
        auto add_hist = [&](auto with_small, auto det) {
#pragma unroll
            for (int m = 0; m < LW; ++m) {
                if ((grp.mask >> (OFF + m)) & 1) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        double v = (double)acc.v[m][r];
                        if constexpr (decltype(with_small)::value) v += (double)acc.s[m][r];
                        double* cell = hist + bin[r] * PITCH + (OFF + m);
                        if constexpr (decltype(det)::value)
                            atomicAdd(reinterpret_cast<unsigned long long*>(cell), to_fixed(v));
                        else
                            atomicAdd(cell, v);
                    }
                }
            }
        };
        auto epilogue = [&](auto with_small) {
            bins();
            if (a.det)
                add_hist(with_small, std::true_type{});
            else
                add_hist(with_small, std::false_type{});
        };

        if constexpr (TWO) {
            // small products first, while the sums are still small, then the
            // large ones on top (see the pass constants)
            k_loop<PREC, kPassSmall, SCHED, NB, LW, OFF, kStagesTwoPassSmall>(nk, a.tail, load, acc);
            k_loop<PREC, kPassLarge, SCHED, NB, LW, OFF, kStagesTwoPassLarge>(nk, a.tail, load, acc);
            epilogue(std::false_type{});
        } else if constexpr (FOLD) {
            k_loop<PREC, kPassFold, SCHED, NB, LW, OFF, kStagesFold>(nk, a.tail, load, acc);
            epilogue(std::false_type{});
        } else {
            k_loop<PREC, kPassAll, SCHED, NB, LW, OFF, kStagesOnePass>(nk, a.tail, load, acc);
            epilogue(std::integral_constant<bool, PREC != SDC_PREC_FP32>{});
        }
    }
}

// One task of a plan: the stream's tile pairs for one lag group, histogram
// in LDS (`hist`: [win][hist_pitch] FP64, then the radial edge table), merged into
// the plan's global bins at the end.  Called by the whole workgroup.
// PAIRED: O8 is even, so a K-step's two origin blocks always lie in one
// component and the block offsets follow from the step with one scalar
// division; otherwise the blocks of all components are taken in turn and a
// step may straddle two components.
// SCHED: kSchedOnePass, kSchedTwoPass (hi/lo splits only) or kSchedLagSplit
// (eight waves: wave w takes quadrant w mod 4 and the lag half w / 4).
// The last lag group of a phase may hold few lags: in the default schedules a
// group with none in its upper half, or upper three quarters, multiplies only
// the rest (50 lags of a phase in 16-lag groups cost 52 instead of 64).
template <int PREC, int RADIAL, int PAIRED, int SCHED>
__device__ __forceinline__ void fused_task(const FusedArgs& a, int task, double* hist) {
    constexpr int LG = lag_group(PREC);
    constexpr int NT = threads_per_wg(SCHED);
    constexpr int PITCH = hist_pitch(PREC);
    float* e2s = (float*)(hist + PITCH * a.win);
    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    TaskCtx c;
    c.a = &a;
    // an even number of lag groups is taken in an order that turns with the
    // segment: workgroups go to the shader engines in turn, and a short last
    // group that always met the same engine would leave it idle (FP32 sc
    // 21x20x19 with 2 x 50 lags: 21.2 instead of 25.0 ms)
    const int segment = task / a.n_groups;
    c.grp = a.groups[(task - segment * a.n_groups + (a.n_groups % 2 == 0 ? segment : 0)) % a.n_groups];
    c.st = a.streams[segment];
    c.hist = hist;
    c.e2s = e2s;
    c.quadrant = wave & 3;

    for (int x = tid; x < PITCH * a.win; x += NT) hist[x] = 0.0;
    if constexpr (RADIAL) {
        for (int x = tid; x < a.n_shells; x += NT) e2s[x] = a.e2[x];
    }
    __syncthreads();

    if constexpr (SCHED == kSchedLagSplit) {
        if (wave < 4)
            pair_loop<PREC, RADIAL, PAIRED, SCHED, LG / 2, 0>(c);
        else
            pair_loop<PREC, RADIAL, PAIRED, SCHED, LG / 2, LG / 2>(c);
    } else if (SCHED == default_sched(PREC) && c.grp.mask < (1 << LG / 4)) {
        pair_loop<PREC, RADIAL, PAIRED, SCHED, SCHED == default_sched(PREC) ? LG / 4 : LG, 0>(c);
    } else if (SCHED == default_sched(PREC) && c.grp.mask < (1 << LG / 2)) {
        pair_loop<PREC, RADIAL, PAIRED, SCHED, SCHED == default_sched(PREC) ? LG / 2 : LG, 0>(c);
    } else {
        pair_loop<PREC, RADIAL, PAIRED, SCHED, LG, 0>(c);
    }
    __syncthreads();

    // Merge the stream's histogram into the global bins.  With short segments
    // the merges of a small sample cost as much as its products.
    const KGroup grp = c.grp;
    const KStream st = c.st;
    if constexpr (RADIAL) {
        for (int x = tid; x < LG * a.win; x += NT) {
            const int m = x / a.win;
            const int w = x - m * a.win;
            const double v = hist[w * PITCH + m];
            const unsigned long long vq = reinterpret_cast<const unsigned long long*>(hist)[w * PITCH + m];
            if (vq != 0ull && ((grp.mask >> m) & 1)) {
                const int64_t b = w;
                const int64_t t = (int64_t)a.stride * (grp.u0 + m) + grp.phase;
                // the address per branch: taken before them, the compiler's
                // schedule of the whole kernel changes (6 FP32 samples of 5000
                // points, 64 lags: 19.6 -> 20.3 ms)
                if (a.det)
                    atomicAdd(&a.Hq[t * a.n_bins + b], vq);
                else
                    unsafeAtomicAdd(&a.H[t * a.n_bins + b], v);
            }
        }
    } else {
        // a lane takes one displacement with all lags, so that its bin is
        // worked out once and not once a lag: 200 samples of sc 6^3, 64 lags,
        // 1292 -> 1245 us, 48 of 8^3 694 -> 656 us (FP32 1737 -> 1642), 4 FP32
        // samples of 20^3 30.6 -> 29.2 ms.  A rolled loop: unrolled, the larger
        // body cost BF16x3 2% (4 samples of 20^3 18.75 -> 19.3 ms, rolled 18.8).
        // Radial windows need no bin and keep the lags side by side.
        for (int w = tid; w < a.win; w += NT) {
            const int64_t b = window_bin(a.map, st, w);
#pragma unroll 1
            for (int m = 0; m < LG; ++m) {
                if (!((grp.mask >> m) & 1)) continue;
                const int64_t at = ((int64_t)a.stride * (grp.u0 + m) + grp.phase) * a.n_bins + b;
                const double v = hist[w * PITCH + m];
                const unsigned long long vq = reinterpret_cast<const unsigned long long*>(hist)[w * PITCH + m];
                if (vq == 0ull) continue;
                if (a.det)
                    atomicAdd(&a.Hq[at], vq);
                else
                    unsafeAtomicAdd(&a.H[at], v);
            }
        }
    }
}

template <int PREC, int RADIAL, int PAIRED, int SCHED>
__global__ __launch_bounds__(threads_per_wg(SCHED), waves_per_simd(SCHED)) void fused_kernel(FusedArgs a) {
    extern __shared__ double hist[];
    // XCD-aware task order: consecutive tasks land on the same XCD (work-
    // groups are dealt to the 8 XCDs round-robin), and consecutive tasks are
    // the lag groups of one stream.  The workgroups running together on an
    // XCD then walk the same tile pairs in step: they share the i-tile
    // operand and overlapping time windows of the j-tile operand in L2.
    const int n_tasks = a.n_groups * a.n_streams;
    const int per = (n_tasks + 7) / 8;
    const int task = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if (task >= n_tasks) return;
    fused_task<PREC, RADIAL, PAIRED, SCHED>(a, task, hist);
}

// Persistent kernel over the tasks of several plans (one launch for a
// batch of samples).  The global task list (plan-major, then stream, then
// lag group) is cut into 8 contiguous ranges of about equal work, at stream
// boundaries, one queue per XCD; a workgroup takes tasks from its own XCD's
// queue with an atomic counter and, once that queue is empty, from the
// following queues in turn.  Equal work keeps the XCDs on their own queues
// until the end, so the lag groups of a stream segment run on one XCD and
// share its operands in L2 (ranges of equal task counts let the XCDs with
// the small samples' short tasks steal the large samples' tasks for most of
// the launch, and the operand fetches grew 8x).  Every counter only grows
// and each queue is visited until it is found empty, so every workgroup
// leaves the loop after at most total + 8 claims.  The K-step addressing
// follows each plan's origin-block count (per component when it is even).
template <int PREC, int RADIAL, int SCHED>
__global__ __launch_bounds__(threads_per_wg(SCHED), waves_per_simd(SCHED)) void fused_batch_kernel(
    const FusedArgs* __restrict__ args, const int64_t* __restrict__ task_start, int n_plans,
    unsigned* __restrict__ queue, const int64_t* __restrict__ ranges, int64_t total) {
    extern __shared__ double hist[];
    __shared__ int s_task, s_plan, s_queue, s_exhausted;
    if (threadIdx.x == 0) {
        s_queue = (int)(blockIdx.x % 8);
        s_exhausted = 0;
    }
    for (;;) {
        if (threadIdx.x == 0) {
            // queue state in LDS: no registers stay live across a task
            int x = s_queue, exhausted = s_exhausted;
            int64_t t = -1;
            while (exhausted < 8) {
                const int64_t lo = ranges[x];
                const int64_t hi = ranges[x + 1] < total ? ranges[x + 1] : total;
                if (lo < hi) {
                    const unsigned k = atomicAdd(&queue[x], 1u);
                    if ((int64_t)k < hi - lo) {
                        t = lo + k;
                        break;
                    }
                }
                x = (x + 1) % 8;
                ++exhausted;
            }
            int pl = 0;
            if (t >= 0) {  // last plan whose first task is <= t
                int lo = 0, hi = n_plans - 1;
                while (lo < hi) {
                    const int mid = (lo + hi + 1) / 2;
                    if (task_start[mid] <= t) lo = mid;
                    else hi = mid - 1;
                }
                pl = lo;
                t -= task_start[pl];
            }
            s_task = (int)t;
            s_plan = pl;
            s_queue = x;
            s_exhausted = exhausted;
        }
        __syncthreads();
        const int task = __builtin_amdgcn_readfirstlane(s_task);
        const int pl = __builtin_amdgcn_readfirstlane(s_plan);
        __syncthreads();
        if (task < 0) break;
        const int paired = __builtin_amdgcn_readfirstlane(args[pl].O8 % 2 == 0);
        if (paired)
            fused_task<PREC, RADIAL, 1, SCHED>(args[pl], task, hist);
        else
            fused_task<PREC, RADIAL, 0, SCHED>(args[pl], task, hist);
        __syncthreads();  // the histogram is reused by the next task
    }
}

// Instantiated kernels: (precision, schedule) pairs the library runs.
template <int PREC, int SCHED, int RADIAL, int PAIRED>
static const void* fused_fn() {
    return (const void*)fused_kernel<PREC, RADIAL, PAIRED, SCHED>;
}
template <int PREC, int SCHED, int RADIAL>
static const void* batch_fn() {
    return (const void*)fused_batch_kernel<PREC, RADIAL, SCHED>;
}

template <int PREC, int SCHED>
static const void* pick_fused(int radial, int paired, bool batch) {
    if (batch) return radial ? batch_fn<PREC, SCHED, 1>() : batch_fn<PREC, SCHED, 0>();
    if (radial) return paired ? fused_fn<PREC, SCHED, 1, 1>() : fused_fn<PREC, SCHED, 1, 0>();
    return paired ? fused_fn<PREC, SCHED, 0, 1>() : fused_fn<PREC, SCHED, 0, 0>();
}

template <int PREC>
static const void* pick_sched(int sched, int radial, int paired, bool batch) {
    switch (sched) {
        case kSchedOnePass: return pick_fused<PREC, kSchedOnePass>(radial, paired, batch);
        case kSchedLagSplit: return pick_fused<PREC, kSchedLagSplit>(radial, paired, batch);
        case kSchedTwoPass:
            if constexpr (PREC == SDC_PREC_SPLIT_BF16 || PREC == SDC_PREC_SPLIT_FP16)
                return pick_fused<PREC, kSchedTwoPass>(radial, paired, batch);
            return nullptr;
        case kSchedFold:
            if constexpr (PREC != SDC_PREC_FP32) return pick_fused<PREC, kSchedFold>(radial, paired, batch);
            return nullptr;
        default: return nullptr;
    }
}

}  // namespace sdc
