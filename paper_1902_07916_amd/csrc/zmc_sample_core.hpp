// zmc_sample_core.hpp -- the body of the sampling kernel, shared by the
// precompiled integrand registry (zmc_sample.hip) and the run-time compiled
// user integrands (zmc_rtc.cpp): direct Monte Carlo over (cube, trial,
// chunk) units with random numbers produced at the time of use (ZMCintegral,
// Sec. 2.1 and Sec. 2.2).
//
// Work decomposition (gfx950, wave64): every wave takes one (cube, trial,
// chunk) unit at a time, independently of the other waves of its block (no
// LDS, no barrier).  A chunk is 4 * 64 * G points and lane l evaluates the
// 4-point groups g = chunk*G*64 + l + 64*j, j < G.  One group of 4 points uses
// D Philox blocks (4*D words, point q dimension i = word q*D + i), so counter
// word 0 of block k is g*D + k; the other three counter words and the key are
// wave-uniform.  Each lane sums f (and f^2 on traced levels) in FP64 and the
// wave reduces with a fixed butterfly, so a unit's partial sums depend only on the
// unit and G.  The grid is persistent: wave w takes a contiguous range of
// units; only the first unit's segment is found by binary search and only
// its position decoded by division, later units follow by increments, and
// a cube's corner and integrand constants are formed once for all of its
// units.
//
// What bounds it: VALU issue.  Measured cycles per wave64 instruction and SIMD
// with 8 waves: v_mad_u64_u32 and FP64 4.2; v_alignbit, v_bfi, v_min_f32,
// v_rndne_f32 4.1; v_bitop3, v_xor, v_fma_f32 2.2-2.4 with vector operands
// (two waves issue at once), 4.1-4.4 with a scalar one.  A v_mad issues beside
// another wave's v_fma_f32 (2.9 each) but hardly beside a v_bitop3, nor does
// FP64 (3.8 each).  A lone wave issues one instruction in 4.6 cycles, chained or not.
// The 6-D sine in FP32 takes 338 instructions a group of 256 points: 5.75e11
// points/s, 0.92 of the rate of its integer and FP64 instructions at one a
// quad-cycle.
//
// An integrand class I provides P64 / P32 parameter blocks, prep64 / prep32
// (per cube, from the slot descriptor and the cube corner), f64 / f32, the
// FP64 scale P32::scale that multiplies each FP32 unit sum, kRangeCheck
// (whether its FP32 values can fall below FP32's normal range) and kProduct
// (whether the last step of its FP32 value can be a product).
#pragma once

#include "zmc_device.hpp"

namespace zmc {

template <int D>
__device__ __forceinline__ void corner(const SlotDesc& sd, int level, uint64_t uid, uint32_t uid_hi, double* lo,
                                       double* h)
{
    uint64_t K[D];
    const uint32_t d = (uint32_t)sd.divisions;
    if (sd.split == 2) {
        // uid = root << (D * level) | path, D bits per split
        uint64_t root = shr_id(uid, uid_hi, D * level);
        if (root < (1ull << 32)) {
            uint32_t r32 = (uint32_t)root;
#pragma unroll
            for (int i = D - 1; i >= 0; --i) {
                K[i] = r32 % d;
                r32 /= d;
            }
        } else {
#pragma unroll
            for (int i = D - 1; i >= 0; --i) {
                K[i] = root % d;
                root /= d;
            }
        }
        for (int j = 1; j <= level; ++j) {
            const uint64_t c = shr_id(uid, uid_hi, D * (level - j));
#pragma unroll
            for (int i = 0; i < D; ++i) K[i] = 2u * K[i] + ((c >> (uint64_t)(D - 1 - i)) & 1u);
        }
#pragma unroll
        for (int i = 0; i < D; ++i) {
            h[i] = ldexp(sd.h0[i], -level);
            lo[i] = fma((double)K[i], h[i], sd.lower[i]);
        }
    } else {
        // b-way splits: uid = root * kids^level + path, one base-kids digit
        // per split (kids = b^D <= 2^24).  The digits come off the low end,
        // the last split's first, and each adds its base-b digit for axis i
        // at the place value b^(splits after it): K_i = root_i b^level +
        // sum over splits j of digit_{j,i} b^(level - j).
        const uint64_t b = (uint64_t)sd.split, kids = (uint64_t)sd.kids;
        uint64_t rest = uid;
        uint32_t rest_hi = uid_hi;
        uint64_t mult = 1;
#pragma unroll
        for (int i = 0; i < D; ++i) K[i] = 0;
        for (int j = 0; j < level; ++j) {
            uint64_t c = divmod_id(rest, rest_hi, kids);
#pragma unroll
            for (int i = D - 1; i >= 0; --i) {
                K[i] += (c % b) * mult;
                c /= b;
            }
            mult *= b;
        }
        uint64_t root = rest; // < d^D < 2^64
#pragma unroll
        for (int i = D - 1; i >= 0; --i) {
            K[i] += (root % d) * mult;
            root /= d;
        }
        const uint64_t parts = mult;
#pragma unroll
        for (int i = 0; i < D; ++i) {
            h[i] = sd.h0[i] / (double)parts;
            lo[i] = fma((double)K[i], h[i], sd.lower[i]);
        }
    }
}

// The 4 samples of a thread's group take words s*D + i, s = 0..3, i < D:
// Philox blocks cb .. cb + D - 1 (4 words each), generated in lockstep in the
// source; the registry's kernels leave the order to a scheduler that goes by
// register need (see build.py).  Run-time compiled kernels take the compiler's
// own schedule, which keeps all of a lockstep's words live: with many
// dimensions they generate the blocks in two halves (HALVES = 1), those holding
// samples 0-1, whose samples are evaluated, and then the rest; HALVES = 2 also
// bars the scheduler from moving instructions between the two.
// eval(q, w) gets sample q's D words in order.
template <int D, int HALVES, class Eval>
__device__ __forceinline__ void group_samples(uint32_t cb, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                              uint32_t k1, Eval&& eval)
{
    constexpr int A = HALVES ? (D + 1) / 2 : D, B = D - A; // blocks of the first half (or all), of the second
    constexpr int QA = HALVES ? 2 : 4;                     // samples that lie in the first alone
    uint32_t ca[A], wa[4 * A];
#pragma unroll
    for (int k = 0; k < A; ++k) ca[k] = cb + (uint32_t)k;
    philox4x32_10_lockstep<A>(ca, c1, c2, c3, k0, k1, wa);
#pragma unroll
    for (int q = 0; q < QA; ++q) {
        uint32_t ws[D];
#pragma unroll
        for (int i = 0; i < D; ++i) ws[i] = wa[q * D + i];
        eval(q, ws);
    }
    if constexpr (HALVES) {
        if constexpr (HALVES == 2) __builtin_amdgcn_sched_barrier(0);
        uint32_t cc[B], wb[4 * B];
#pragma unroll
        for (int k = 0; k < B; ++k) cc[k] = cb + (uint32_t)(A + k);
        philox4x32_10_lockstep<B>(cc, c1, c2, c3, k0, k1, wb);
#pragma unroll
        for (int q = QA; q < 4; ++q) {
            uint32_t ws[D];
#pragma unroll
            for (int i = 0; i < D; ++i) {
                const int n = q * D + i;
                ws[i] = n < 4 * A ? wa[n] : wb[n - 4 * A];
            }
            eval(q, ws);
        }
    }
}

// a + b; unless FUSED, a product that one of them is rounds before it.
template <bool FUSED>
__device__ __forceinline__ float group_add(float a, float b)
{
    if constexpr (FUSED) {
        return a + b;
    } else {
#pragma clang fp contract(off)
        return a + b;
    }
}

template <bool B>
struct BoolTag {
    static constexpr bool value = B;
};

// Per-cube state of the sampling loop: FP32 evaluation keeps the integrand's
// cube-relative constants (formed in FP64 from the corner), FP64 evaluation
// the corner and the edge lengths scaled by 2^-32 with the integrand's
// constants.  Computed once per cube, for all of its (trial, chunk) units.
template <class I, int D, bool FP32>
struct CubeState;

template <class I, int D>
struct CubeState<I, D, true> {
    typename I::P32 p;
    __device__ __forceinline__ void set(const SlotDesc& sd, int level, uint64_t uid, uint32_t uid_hi)
    {
        double lo[D], h[D];
        corner<D>(sd, level, uid, uid_hi, lo, h);
        I::prep32(sd, lo, h, p);
    }
};

template <class I, int D>
struct CubeState<I, D, false> {
    typename I::P64 p;
    double lo[D], h32[D];
    __device__ __forceinline__ void set(const SlotDesc& sd, int level, uint64_t uid, uint32_t uid_hi)
    {
        double h[D];
        corner<D>(sd, level, uid, uid_hi, lo, h);
#pragma unroll
        for (int i = 0; i < D; ++i) h32[i] = ldexp(h[i], -32);
        I::prep64(sd, p);
    }
};

// KEEP_S2: also accumulate the sum of squares (only the per-(cube, trial)
// trace reads it; the estimator uses the sums alone).  Without it the
// partial's second member is 0.
// HALVES: see group_samples.
template <class I, int D, bool FP32, bool KEEP_S2, int HALVES = 0>
__device__ __forceinline__ void sample_units(const SampleArgs& a)
{
    // blocks of 64, 128 or 256 threads (the tile table's block shape)
    const int waves_per_block = (int)(blockDim.x >> 6);
    const int lane = threadIdx.x & 63;
    // the wave index is uniform over the wave: keep it (and all unit
    // bookkeeping derived from it) in scalar registers
    const int64_t wave = (int64_t)blockIdx.x * waves_per_block + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t n_waves = (int64_t)gridDim.x * waves_per_block;
    if (a.clock && wave == 0 && lane == 0) *a.clock = device_clock();
    const int64_t U = a.total_units;
    // contiguous ranges that differ by one unit at most: rounding every range
    // up to the same length leaves waves without work when a wave's share is
    // small (14.07 units of 8192 waves rounded to 15 cost the 4-D oscillatory
    // bucket at N = 4096 over 14^4 cubes 5%)
    const int64_t per = U / n_waves, extra = U - per * n_waves;
    int64_t u = a.unit0 + wave * per + min(wave, extra);
    const int64_t uend = u + per + (wave < extra ? 1 : 0);
    if (u >= uend) return;

    int bs = 0;
    {
        int hi = a.n_bsegs - 1;
        while (bs < hi) {
            const int mid = (bs + hi + 1) >> 1;
            if (a.bsegs[mid].unit_base <= u) bs = mid;
            else hi = mid - 1;
        }
    }

    // The wave's first unit is decoded by division; every later one follows
    // by increments (chunk, then trial, then cube), and a new bucket segment
    // is decoded afresh.  Units are [cube][trial][chunk] within a segment.
    const Segment* sg = nullptr;
    const SlotDesc* sd = nullptr;
    int64_t local = 0, cl = 0;
    int trial = 0, chunk = 0;
    auto decode = [&]() {
        sg = &a.segs[a.bsegs[bs].seg];
        sd = &a.slots[sg->slot];
        local = u - a.bsegs[bs].unit_base;
        const int nch = sd->nch;
        const int64_t upc = (int64_t)sd->trials * nch;
        cl = local / upc;
        const int rem = (int)(local - cl * upc);
        trial = rem / nch;
        chunk = rem - trial * nch;
    };
    decode();
    CubeState<I, D, FP32> cs;
    uint64_t uid = 0;
    uint32_t uid_hi = 0;
    bool fresh = true; // the cube's state is to be (re)computed

    for (; u < uend; ++u) {
        if (bs + 1 < a.n_bsegs && a.bsegs[bs + 1].unit_base <= u) {
            while (bs + 1 < a.n_bsegs && a.bsegs[bs + 1].unit_base <= u) ++bs;
            decode();
            fresh = true;
        }
        const int level = sg->level;
        if (fresh) {
            uid = a.uid[sg->cube_base + cl];
            uid_hi = a.uid_hi ? a.uid_hi[sg->cube_base + cl] : 0u;
            cs.set(*sd, level, uid, uid_hi);
            fresh = false;
        }

        const uint32_t k0 = (uint32_t)sd->seed, k1 = (uint32_t)(sd->seed >> 32);
        const uint32_t c1 = ctr_word1(trial, level, uid_hi);
        const uint32_t c2 = (uint32_t)uid, c3 = (uint32_t)(uid >> 32);
        // This chunk's points: whole groups of all 64 lanes, then at most one
        // group in which lanes stop short.  The counts are wave-uniform and
        // kept in scalar registers (the loads they come from are vector
        // loads), so that the loop's control takes no vector instruction.
        const int G = __builtin_amdgcn_readfirstlane(sd->groups);
        const int64_t left = sd->samples - (int64_t)chunk * G * 256;
        const int pts = __builtin_amdgcn_readfirstlane((int)min((int64_t)G * 256, left));
        const int n_whole = pts >> 8;
        uint32_t cb = (uint32_t)((int64_t)chunk * G * 64 + lane) * (uint32_t)D; // the lane's next Philox block

        double S1 = 0.0, S2 = 0.0;
        // FP64 evaluation: the cell bits of a word and its mid-cell bit, in
        // vector registers (an instruction with a scalar operand issues at
        // half the rate of the same one without)
        [[maybe_unused]] uint32_t cell_mask = 0xFFFFFE00u, cell_mid = 0x100u;
        if constexpr (!FP32) asm("" : "+v"(cell_mask), "+v"(cell_mid));
        // Groups of 4 points.  FP32 evaluation adds a group's 4 values in
        // FP32 and the group's sum in FP64: one conversion and one FP64 add
        // per group instead of per point.  The 4 values are added in point
        // order, except at D = 6 and 7, where (v0 + v1) + (v2 + v3) ran
        // 1-2.4% faster than both the point-order sum and per-value FP64 adds
        // in a same-box A/B (and 0.5-3.7% slower at the other D).
        constexpr bool kPairSum = D == 6 || D == 7;
        // nvalid: the lane's points of a ragged group that count; rounded:
        // the FP32 value is rounded before it is added (below)
        auto group = [&](auto ragged, auto rounded, int nvalid) {
            constexpr bool kRagged = decltype(ragged)::value;
            [[maybe_unused]] float gs = 0.0f, gb = 0.0f;
            group_samples<D, HALVES>(cb, c1, c2, c3, k0, k1, [&](int q, const uint32_t* w) {
                if constexpr (FP32) {
                    float v[D];
#pragma unroll
                    for (int i = 0; i < D; ++i) v[i] = unit_interval_f32(w[i]);
                    float f = I::f32(cs.p, v);
                    // rounded by an opaque move, or (HALVES = 2) by sums that may not be fused
                    constexpr bool kFree = !(decltype(rounded)::value && HALVES == 2);
                    auto add = [](float a, float b) { return group_add<kFree>(a, b); };
                    if constexpr (decltype(rounded)::value && HALVES != 2) asm("" : "+v"(f));
                    if constexpr (kRagged) f = (q < nvalid) ? f : 0.0f;
                    if constexpr (kPairSum) {
                        if (q == 0) gs = f;
                        else if (q == 1) gs = add(gs, f);
                        else if (q == 2) gb = f;
                        else gb = add(gb, f);
                    } else {
                        gs = q == 0 ? f : add(gs, f);
                    }
                    if constexpr (KEEP_S2) {
                        const double fd = (double)f;
                        S2 = fma(fd, fd, S2);
                    }
                } else {
                    double x[D];
                    // x = fma(h, (2*(w>>9)+1) 2^-24, lo) computed as
                    // fma(h 2^-32, (w & ~511) | 256, lo): the same exact
                    // product, the word placed by one three-input
                    // instruction instead of a shift and an OR (FP64
                    // evaluation is bound by VALU issue: 3.6-5% faster,
                    // the 6-D sine over 6^6 cubes of 16384 points 2.56e11
                    // -> 2.66e11 points/s, the 9-D Gaussian 2.22e11 ->
                    // 2.34e11)
#pragma unroll
                    for (int i = 0; i < D; ++i)
                        x[i] = fma(cs.h32[i], (double)bits_or(w[i], cell_mask, cell_mid), cs.lo[i]);
                    double f = I::f64(cs.p, x);
                    if constexpr (kRagged) f = (q < nvalid) ? f : 0.0;
                    S1 += f;
                    if constexpr (KEEP_S2) S2 = fma(f, f, S2);
                }
            });
            if constexpr (FP32) S1 += (double)(kPairSum ? gs + gb : gs);
            cb += 64u * (uint32_t)D;
        };
        // An FP32 value that ends in a product can be fused into the group's
        // sum, which then rounds once less (a sum of 256 points moves by some
        // 1e-9).  Whether it may be depends on the request alone: in full
        // chunks up to D = 3, with a multiple of 4 points up to D = 9, never
        // above.  The lines lie where separate copies of this loop once had
        // them, for the sake of the same bits.  Where it may be, the compiler's
        // contraction does it: a body's last operation is not known here.
        constexpr bool kProduct = FP32 && I::kProduct;
        bool fused = false;
        if constexpr (kProduct && D <= 3) fused = pts == G * 256;
        else if constexpr (kProduct && D <= 9) fused = (sd->samples & 3) == 0;
        if (fused) {
            // whole groups of 4 points only, the last for some lanes
            const int n_lane = n_whole + ((pts & 255) > 4 * lane ? 1 : 0);
            for (int j = 0; j < n_lane; ++j) group(BoolTag<false>{}, BoolTag<false>{}, 4);
        } else {
            for (int j = 0; j < n_whole; ++j) group(BoolTag<false>{}, BoolTag<kProduct>{}, 4);
            if (pts & 255) group(BoolTag<true>{}, BoolTag<kProduct>{}, (pts & 255) - 4 * lane);
        }

        S1 = wave_sum(S1);
        if constexpr (KEEP_S2) S2 = wave_sum(S2);
        if constexpr (FP32) {
            if constexpr (I::kRangeCheck) {
                // values below FP32's normal range: report it for the segment
                if (lane == 0 && fabs(S1) < (double)pts * 0x1p-126)
                    atomicOr(a.seg_flags + a.bsegs[bs].seg, kRangeLost);
            }
            S1 *= cs.p.scale;
            if constexpr (KEEP_S2) S2 *= cs.p.scale * cs.p.scale;
        }
        // partial sums in unit order, [cube][trial * nch + chunk]: a wave's
        // consecutive units fill whole cache lines
        if (lane == 0) a.partial[sg->part_base + local] = make_double2(S1, S2);

        // the next unit: chunk, then trial, then cube
        ++local;
        if (++chunk == sd->nch) {
            chunk = 0;
            if (++trial == sd->trials) {
                trial = 0;
                ++cl;
                fresh = true;
            }
        }
    }
}

} // namespace zmc
