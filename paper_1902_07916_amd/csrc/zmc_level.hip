// zmc_level.hip -- per-cube and per-integral kernels of one tree level
// (ZMCintegral, Sec. 2.1): trial mean / standard deviation per sub-domain,
// the threshold from the mean and standard deviation of the level's standard
// deviations, selection, acceptance, and the split of the selected cubes.
//
// All of these are HBM-bound and small next to the sampling kernel.  The
// per-cube kernels work on tiles of 1024 consecutive cubes of one segment
// (512 threads, 2 cubes each, strided so that loads coalesce).  The
// per-integral step that follows each of them (the mean of s, the threshold,
// the decision) runs, for small levels, in the same launch: the last tile
// block of a segment to finish, found with a per-segment counter, reduces
// that segment's tile records in tile order, so a level costs three short
// launches after sampling.  Publishing a tile record to the other XCDs takes
// an L2 write-back per block, which outweighs a launch once a level has a few
// hundred tiles; large levels therefore run the per-segment steps as their own
// one-block-per-segment launches.  Every reduction has a fixed shape (thread-serial over its
// elements, then a butterfly in each wave, then one over the waves), so results
// are bitwise reproducible and independent of which block finishes last or
// of what else is resident.
#include <float.h>

#include <algorithm>

#include "zmc_kernels.hpp"

namespace zmc {

namespace {

constexpr int kWaves = kLevelThreads / 64;
constexpr int kPerThread = kTileCubes / kLevelThreads;

// Block-wide reductions in a fixed order, every thread getting the result: a
// butterfly in each wave, then one over the waves' values.
template <class T, class Op>
__device__ __forceinline__ T over_waves(const T* sh, Op op)
{
    static_assert(kWaves == 4 || kWaves == 8 || kWaves == 16, "the waves' values repeat within a row of lanes");
    return row_reduce<kWaves>(sh[threadIdx.x & (kWaves - 1)], op);
}

template <class T, class Op>
__device__ __forceinline__ T block_reduce(T v, T* sh, Op op)
{
    v = wave_reduce(v, op);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return over_waves(sh, op);
}

__device__ __forceinline__ double block_sum(double v, double* sh) { return block_reduce(v, sh, OpAdd{}); }
__device__ __forceinline__ double block_min(double v, double* sh) { return block_reduce(v, sh, OpMin{}); }
__device__ __forceinline__ double block_max(double v, double* sh) { return block_reduce(v, sh, OpMax{}); }

// The selection totals of a tile or a segment, reduced over the block in one
// exchange: four sums, a minimum and a count, each combined in the same
// fixed order as block_sum / block_min / block_sum_i.
struct SelTotals {
    double accM, accS2, selM, selS2, margin;
    int64_t nsel;
};

__device__ SelTotals block_reduce_sel(SelTotals v)
{
    __shared__ double shd[5][kWaves];
    __shared__ int64_t shn[kWaves];
    v.accM = wave_sum(v.accM);
    v.accS2 = wave_sum(v.accS2);
    v.selM = wave_sum(v.selM);
    v.selS2 = wave_sum(v.selS2);
    v.margin = wave_reduce(v.margin, OpMin{});
    v.nsel = wave_reduce(v.nsel, OpAdd{});
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        const int w = threadIdx.x >> 6;
        shd[0][w] = v.accM;
        shd[1][w] = v.accS2;
        shd[2][w] = v.selM;
        shd[3][w] = v.selS2;
        shd[4][w] = v.margin;
        shn[w] = v.nsel;
    }
    __syncthreads();
    return SelTotals{over_waves(shd[0], OpAdd{}), over_waves(shd[1], OpAdd{}), over_waves(shd[2], OpAdd{}),
                     over_waves(shd[3], OpAdd{}), over_waves(shd[4], OpMin{}), over_waves(shn, OpAdd{})};
}

// Exclusive prefix of a 0/1 flag over the block in thread order; *total gets
// the block's count.
__device__ int block_excl_scan_flag(int flag, int* sh, int* total)
{
    const unsigned long long mask = __ballot(flag);
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int in_wave = __popcll(mask & ((1ull << lane) - 1ull));
    __syncthreads();
    if (lane == 0) sh[wv] = __popcll(mask);
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        if (w < wv) base += sh[w];
        tot += sh[w];
    }
    *total = tot;
    return base + in_wave;
}

// Segment that owns tile t (segments are in list order, tile_base ascending).
__device__ __forceinline__ int seg_of_tile(const Segment* segs, int n, int64_t t)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (segs[mid].tile_base <= t) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Called by every tile block of segment si once its tile record is written:
// true in the block that completes the segment, which then sees every other
// block's records.  The counter is back at 0 when the launch ends.
__device__ bool last_tile_of_segment(int32_t* count, int si, int64_t n_tiles)
{
    __shared__ int last;
    stores_done();
    __syncthreads();
    // a one-tile segment has no other block to wait for: its own record is
    // visible to the block after the barrier, and no device-scope fence (an
    // L2 write-back on this chip) is needed
    if (n_tiles == 1) return true;
    if (threadIdx.x == 0) {
        __threadfence(); // release this block's tile record
        const int old = atomicAdd(&count[si], 1);
        last = (old == (int)n_tiles - 1);
        if (last) atomicExch(&count[si], 0);
    }
    __syncthreads();
    if (last) __threadfence(); // acquire the other blocks' records
    return last != 0;
}

// ---- per-segment steps (one block) ------------------------------------------
__device__ void seg_mean(const LevelArgs& a, int si)
{
    __shared__ double sh[kWaves];
    const Segment& sg = a.segs[si];
    double v = 0.0, lo = DBL_MAX, hi = -DBL_MAX;
    for (int64_t t = threadIdx.x; t < sg.n_tiles; t += kLevelThreads) {
        const TileRec& T = a.tiles[sg.tile_base + t];
        v += T.sum_s;
        lo = fmin(lo, T.s_min);
        hi = fmax(hi, T.s_max);
    }
    const double tot = block_sum(v, sh);
    lo = block_min(lo, sh);
    hi = block_max(hi, sh);
    if (threadIdx.x == 0) {
        a.stats[si].mu = tot / (double)sg.n_cubes;
        a.stats[si].s_min = lo;
        a.stats[si].s_max = hi;
    }
}

// The scale exponent of the threshold's std: the largest |s - mu| is at the
// smallest or the largest s (rounding is monotonic).
__device__ __forceinline__ int thr_scale_exp(double mu, double lo, double hi)
{
    return std_scale_exp(fmax(fabs(hi - mu), fabs(lo - mu)));
}

__device__ void seg_thr(const LevelArgs& a, int si)
{
    __shared__ double sh[kWaves];
    const Segment& sg = a.segs[si];
    double v = 0.0;
    for (int64_t t = threadIdx.x; t < sg.n_tiles; t += kLevelThreads) v += a.tiles[sg.tile_base + t].sum_sq;
    const double tot = block_sum(v, sh);
    if (threadIdx.x == 0) {
        const SegStats& S = a.stats[si];
        const double sd = ldexp(sqrt(tot / (double)sg.n_cubes), thr_scale_exp(S.mu, S.s_min, S.s_max));
        a.stats[si].sd = sd;
        a.stats[si].thr = a.stats[si].mu + a.slots[sg.slot].sigma_mult * sd;
    }
}

// What the decision reads besides the totals.  Loaded before the reductions:
// the last step of a level is one thread's, and each of these would be a
// memory latency of its own there.
struct DecideIn {
    double2 prev;
    double rtol;
    int64_t max_cubes;
    int32_t trials, kids, range_lost;
};

__device__ __forceinline__ DecideIn decide_in(const LevelArgs& a, int si)
{
    const SlotDesc& sd = a.slots[a.segs[si].slot];
    return DecideIn{a.prev_tot[si], sd.rtol, sd.max_cubes, sd.trials, sd.kids, a.seg_flags ? a.seg_flags[si] : 0};
}

__device__ void seg_decide(const LevelArgs& a, int si);
__device__ Decision decide_write(const LevelArgs& a, int si, const DecideIn& in, double accM, double accS2,
                                 double selM, double selS2, double margin, int64_t nsel, int bad);

// ---- finalize: per cube I_t = V * S1_t / N, m = mean I_t, s = std I_t ------
// The partial sums of a pass's cubes are contiguous ([cube][trial *
// nch + chunk]); when their S1 members fit kStage values, the block first
// copies those to LDS with coalesced loads, and each thread then reads its own
// cube's row there.  The row then takes the trial values I_t, so that the
// division and the product of each are done once and not again for the
// deviations.  Wider rows (many trials or chunks) are read from memory, only
// their trial values kept in LDS, or formed again for each of the three sums
// where those do not fit either.

// KEEP: also leave each thread's cubes' m and s in m_r / s_r (pass j at
// index j), for the one-block level path.
// KEEP also returns the tile's sum of s, non-finite flag and extremes of s
// (every thread).
template <bool KEEP = false>
__device__ void finalize_tile(const LevelArgs& a, int64_t tile, int si, double* m_r = nullptr,
                              double* s_r = nullptr, double* tot_s = nullptr, int* any_bad_out = nullptr,
                              double* s_ext = nullptr)
{
    __shared__ double sh[kWaves];
    __shared__ double stage[kStage];
    const Segment& sg = a.segs[si];
    const SlotDesc& sd = a.slots[sg.slot];
    const int D = sd.dim, n1 = sd.trials, nch = sd.nch;
    const int64_t per = (int64_t)n1 * nch; // partials per cube
    const bool staged = row_fits(per);
    const bool rows = row_fits(n1); // the trial values fit LDS
    const double V = cube_volume(sd, D, sg.level);
    const double N = (double)sd.samples;
    const int64_t first = (tile - sg.tile_base) * kTileCubes;
    double sum_s = 0.0, s_lo = DBL_MAX, s_hi = -DBL_MAX;
    int bad = 0;
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) {
        const int64_t c0 = first + (int64_t)j * kLevelThreads; // first cube of this pass
        if (c0 >= sg.n_cubes) break;                            // uniform over the block
        const int cnt = (int)min<int64_t>(kLevelThreads, sg.n_cubes - c0);
        const double2* src = a.partial + sg.part_base + c0 * per;
        if (staged) {
            __syncthreads(); // the previous pass is done with the stage
            for (int e = threadIdx.x; e < cnt * (int)per; e += kLevelThreads) stage[e] = src[e].x;
            __syncthreads();
        }
        if ((int)threadIdx.x >= cnt) continue;
        const int64_t cl = c0 + threadIdx.x;
        const int64_t c = sg.cube_base + cl;
        const double2* P = src + (int64_t)threadIdx.x * per;
        double* row = stage + threadIdx.x * (staged ? (int)per : n1); // this thread's alone from here on
        auto S1_mem = [&](int t) {
            double S1 = 0.0;
            for (int ch = 0; ch < nch; ++ch) S1 += P[(int64_t)t * nch + ch].x;
            return S1;
        };
        if (a.tr_S1) {
            for (int t = 0; t < n1; ++t) {
                double S2 = 0.0;
                for (int ch = 0; ch < nch; ++ch) S2 += P[(int64_t)t * nch + ch].y;
                a.tr_S1[c * n1 + t] = S1_mem(t);
                a.tr_S2[c * n1 + t] = S2;
            }
        }
        double sum = 0.0;
        for (int t = 0; t < n1; ++t) {
            double S1 = 0.0;
            if (staged) {
                for (int ch = 0; ch < nch; ++ch) S1 += row[t * nch + ch];
            } else {
                S1 = S1_mem(t);
            }
            const double I = V * (S1 / N);
            if (rows) row[t] = I; // among the row's partials already read
            sum += I;
        }
        auto value = [&](int t) { return rows ? row[t] : V * (S1_mem(t) / N); };
        const double m = sum / (double)n1;
        double dmax = 0.0;
        for (int t = 0; t < n1; ++t) {
            const double d = fabs(value(t) - m);
            if (d > dmax) dmax = d;
        }
        const int e = std_scale_exp(dmax);
        double ss = 0.0;
        for (int t = 0; t < n1; ++t) {
            const double d = ldexp(value(t) - m, -e);
            ss += d * d;
        }
        const double s = ldexp(sqrt(ss / (double)n1), e);
        a.m[c] = m;
        a.s[c] = s;
        if constexpr (KEEP) {
            m_r[j] = m;
            s_r[j] = s;
        }
        sum_s += s;
        s_lo = fmin(s_lo, s);
        s_hi = fmax(s_hi, s);
        bad |= !(isfinite(m) && isfinite(s));
    }
    const double tot = block_sum(sum_s, sh);
    const double lo = block_min(s_lo, sh);
    const double hi = block_max(s_hi, sh);
    const int any_bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) {
        a.tiles[tile].sum_s = tot;
        a.tiles[tile].s_min = lo;
        a.tiles[tile].s_max = hi;
        a.tiles[tile].nonfinite = any_bad;
    }
    if constexpr (KEEP) {
        *tot_s = tot;
        *any_bad_out = any_bad;
        s_ext[0] = lo;
        s_ext[1] = hi;
    }
}

__global__ __launch_bounds__(kLevelThreads) void finalize_kernel(const LevelArgs a)
{
    if (a.clock && blockIdx.x == 0 && threadIdx.x == 0) *a.clock = device_clock();
    const int64_t tile = blockIdx.x;
    const int si = seg_of_tile(a.segs, a.n_segs, tile);
    const Segment& sg = a.segs[si];
    finalize_tile(a, tile, si);
    if (a.fused && sg.need_thr && !sg.group_size && last_tile_of_segment(a.seg_count, si, sg.n_tiles))
        seg_mean(a, si);
}

// ---- threshold: std of s around the mean, per segment ----------------------
__device__ void sqdev_tile(const LevelArgs& a, int64_t tile, int si)
{
    __shared__ double sh[kWaves];
    const Segment& sg = a.segs[si];
    const double mu = a.stats[si].mu;
    const int e = thr_scale_exp(mu, a.stats[si].s_min, a.stats[si].s_max);
    const int64_t first = (tile - sg.tile_base) * kTileCubes;
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) {
        const int64_t cl = first + threadIdx.x + (int64_t)j * kLevelThreads;
        const double d = cl < sg.n_cubes ? ldexp(a.s[sg.cube_base + cl] - mu, -e) : 0.0;
        acc += d * d;
    }
    const double tot = block_sum(acc, sh);
    if (threadIdx.x == 0) a.tiles[tile].sum_sq = tot;
}

__global__ __launch_bounds__(kLevelThreads) void tile_sqdev_kernel(const LevelArgs a)
{
    const int64_t tile = blockIdx.x;
    const int si = seg_of_tile(a.segs, a.n_segs, tile);
    const Segment& sg = a.segs[si];
    if (!sg.need_thr || sg.group_size) return;
    sqdev_tile(a, tile, si);
    if (a.fused && last_tile_of_segment(a.seg_count, si, sg.n_tiles)) seg_thr(a, si);
}

// ---- per-segment steps as their own launches (large levels) -----------------
__global__ __launch_bounds__(kLevelThreads) void seg_mean_kernel(const LevelArgs a)
{
    const Segment& sg = a.segs[blockIdx.x];
    if (!sg.need_thr || sg.group_size) return;
    seg_mean(a, blockIdx.x);
}

__global__ __launch_bounds__(kLevelThreads) void seg_thr_kernel(const LevelArgs a)
{
    const Segment& sg = a.segs[blockIdx.x];
    if (!sg.need_thr || sg.group_size) return;
    seg_thr(a, blockIdx.x);
}

// ---- per-parent thresholds: one per group of siblings -----------------------
// One wave per group (groups of the segments with group_size > 0, in list
// order): mean of the group's s, then the population std, in a fixed order.
__device__ __forceinline__ int seg_of_group(const Segment* segs, int n, int64_t g)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (segs[mid].group_base <= g) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__global__ __launch_bounds__(kLevelThreads) void group_thr_kernel(const LevelArgs a)
{
    const int lane = threadIdx.x & 63;
    const int64_t n_waves = (int64_t)gridDim.x * kWaves;
    for (int64_t g = (int64_t)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
         g < a.n_groups; g += n_waves) {
        const int si = seg_of_group(a.segs, a.n_segs, g);
        const Segment& sg = a.segs[si];
        const int64_t gs = sg.group_size;
        const double* s = a.s + sg.cube_base + (g - sg.group_base) * gs;
        double v = 0.0;
        for (int64_t j = lane; j < gs; j += 64) v += s[j];
        const double mu = wave_sum(v) / (double)gs;
        double dmax = 0.0;
        for (int64_t j = lane; j < gs; j += 64) dmax = fmax(dmax, fabs(s[j] - mu));
        const int e = std_scale_exp(wave_reduce(dmax, OpMax{}));
        double q = 0.0;
        for (int64_t j = lane; j < gs; j += 64) {
            const double d = ldexp(s[j] - mu, -e);
            q += d * d;
        }
        const double sd = ldexp(sqrt(wave_sum(q) / (double)gs), e);
        if (lane == 0) a.gthr[g] = mu + a.slots[sg.slot].sigma_mult * sd;
    }
}

// ---- selection: split = s > thr; accepted and selected sums per tile -------
__device__ void select_tile(const LevelArgs& a, int64_t tile, int si)
{
    const Segment& sg = a.segs[si];
    const bool thr_on = sg.need_thr != 0;
    const double level_thr = (thr_on && !sg.group_size) ? a.stats[si].thr : 0.0;
    const int64_t first = (tile - sg.tile_base) * kTileCubes;
    double accM = 0.0, accS2 = 0.0, selM = 0.0, selS2 = 0.0, margin = DBL_MAX;
    int64_t nsel = 0;
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) {
        const int64_t cl = first + threadIdx.x + (int64_t)j * kLevelThreads;
        if (cl >= sg.n_cubes) break;
        const int64_t c = sg.cube_base + cl;
        const double m = a.m[c], s = a.s[c];
        const double thr = (thr_on && sg.group_size) ? a.gthr[sg.group_base + cl / sg.group_size] : level_thr;
        const bool sel = thr_on && (s > thr);
        a.sel[c] = sel ? 1 : 0;
        if (sel) {
            selM += m;
            selS2 += s * s;
            ++nsel;
        } else {
            accM += m;
            accS2 += s * s;
        }
        if (thr_on && thr > 0.0) margin = fmin(margin, fabs(s - thr) / thr);
    }
    const SelTotals tot = block_reduce_sel(SelTotals{accM, accS2, selM, selS2, margin, nsel});
    if (threadIdx.x == 0) {
        TileRec& T = a.tiles[tile];
        T.accM = tot.accM;
        T.accS2 = tot.accS2;
        T.selM = tot.selM;
        T.selS2 = tot.selS2;
        T.min_margin = tot.margin;
        T.n_sel = tot.nsel;
    }
}

__global__ __launch_bounds__(kLevelThreads) void tile_select_kernel(const LevelArgs a)
{
    const int64_t tile = blockIdx.x;
    const int si = seg_of_tile(a.segs, a.n_segs, tile);
    const Segment& sg = a.segs[si];
    select_tile(a, tile, si);
    if (a.fused && last_tile_of_segment(a.seg_count, si, sg.n_tiles)) seg_decide(a, si);
}

// ---- per segment: totals, stop rules, rank base of every tile --------------
__device__ void seg_decide(const LevelArgs& a, int si)
{
    __shared__ int64_t shi[kWaves];
    const Segment& sg = a.segs[si];
    const DecideIn in = decide_in(a, si);
    double accM = 0.0, accS2 = 0.0, selM = 0.0, selS2 = 0.0, margin = DBL_MAX;
    int64_t nsel = 0;
    int bad = 0;
    for (int64_t t = threadIdx.x; t < sg.n_tiles; t += kLevelThreads) {
        const TileRec& T = a.tiles[sg.tile_base + t];
        accM += T.accM;
        accS2 += T.accS2;
        selM += T.selM;
        selS2 += T.selS2;
        margin = fmin(margin, T.min_margin);
        nsel += T.n_sel;
        bad |= T.nonfinite;
    }
    {
        const SelTotals tot = block_reduce_sel(SelTotals{accM, accS2, selM, selS2, margin, nsel});
        accM = tot.accM;
        accS2 = tot.accS2;
        selM = tot.selM;
        selS2 = tot.selS2;
        margin = tot.margin;
        nsel = tot.nsel;
    }
    bad = __syncthreads_or(bad);

    // exclusive prefix of the tiles' selection counts (rank base for spawn)
    int64_t carry = 0;
    for (int64_t t0 = 0; t0 < sg.n_tiles; t0 += kLevelThreads) {
        const int64_t t = t0 + threadIdx.x;
        const int64_t v = t < sg.n_tiles ? a.tiles[sg.tile_base + t].n_sel : 0;
        // inclusive wave scan
        int64_t x = v;
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int64_t y = __shfl_up(x, off, 64);
            if (lane >= off) x += y;
        }
        __syncthreads();
        if (lane == 63) shi[threadIdx.x >> 6] = x;
        __syncthreads();
        int64_t base = carry;
        int64_t chunk = 0;
        for (int w = 0; w < kWaves; ++w) {
            if (w < (threadIdx.x >> 6)) base += shi[w];
            chunk += shi[w];
        }
        if (t < sg.n_tiles) a.tiles[sg.tile_base + t].sel_prefix = base + x - v;
        carry += chunk;
    }

    // the record is the last a segment's block writes: behind every wave's prefixes
    stores_done();
    __syncthreads();
    if (threadIdx.x == 0) decide_write(a, si, in, accM, accS2, selM, selS2, margin, nsel, bad);
}

// The segment's outcome from its totals (thread 0): stop rules, running
// totals, the record in device memory and in the mapped host buffer, then the
// level's number there.  The host goes on once it sees the number, and a call
// may end there, so what the segment's blocks store they store before it (the
// caller waits for its waves' stores; the fence here writes them back).  The
// one exception is the next level laid out ahead, see level_small_kernel.
__device__ Decision decide_write(const LevelArgs& a, int si, const DecideIn& in, double accM, double accS2,
                                 double selM, double selS2, double margin, int64_t nsel, int bad)
{
    const Segment& sg = a.segs[si];
    {
        SegStats& S = a.stats[si];
        if (!sg.need_thr || sg.group_size) {
            S.mu = S.sd = S.thr = __builtin_nan("");
        }
        S.min_margin = margin;
        S.accM = accM;
        S.accS2 = accS2;
        S.selM = selM;
        S.selS2 = selS2;
        S.n_sel = nsel;
        S.nonfinite = bad;
        S.range_lost = in.range_lost;
        Decision dec;
        double totM = in.prev.x + accM, totS2 = in.prev.y + accS2;
        if (!sg.need_thr || nsel == 0) {
            dec = kDone;
        } else {
            const double runM = totM + selM, runS2 = totS2 + selS2;
            if (in.rtol > 0.0 && sqrt(runS2 / (double)(in.trials - 1)) <= in.rtol * fabs(runM)) {
                dec = kRtolMet;
            } else if ((uint64_t)nsel * (uint64_t)in.kids > (uint64_t)in.max_cubes) {
                dec = kTruncated;
            } else {
                dec = kSplit;
            }
            if (dec != kSplit) {
                totM = runM;
                totS2 = runS2;
            }
        }
        S.decision = dec;
        S.totM = totM;
        S.totS2 = totS2;
        if (a.host_stats) {
            a.host_stats[si] = S;
            __threadfence_system(); // the record is in host memory before its number is
            __hip_atomic_store(a.host_seq + si, a.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        return dec;
    }
}

__global__ __launch_bounds__(kLevelThreads) void seg_decide_kernel(const LevelArgs a) { seg_decide(a, blockIdx.x); }

// The children of n_parents cubes (ids list, list_hi in LDS) in order, by the
// whole block: child c of (hi:lo) is (hi:lo) * kids + c; with bisection
// (hi:lo) << D | c.
__device__ __forceinline__ void write_children(const uint64_t* list, const uint32_t* list_hi, int n_parents, int split,
                                               int D, int64_t kids, uint64_t* out, uint32_t* out_hi)
{
    const int64_t n_writes = (int64_t)n_parents * kids;
    if (split == 2) {
        const uint64_t mask = (1ull << D) - 1ull;
        for (int64_t w = threadIdx.x; w < n_writes; w += kLevelThreads) {
            const uint64_t parent = list[w >> D];
            out[w] = (parent << D) | ((uint64_t)w & mask);
            if (out_hi) out_hi[w] = (list_hi[w >> D] << D) | (uint32_t)(parent >> (64 - D));
        }
    } else {
        for (int64_t w = threadIdx.x; w < n_writes; w += kLevelThreads) {
            const int64_t i = w / kids;
            const uint64_t plo = list[i] * (uint64_t)kids;
            const uint64_t lo = plo + (uint64_t)(w - i * kids);
            out[w] = lo;
            if (out_hi)
                out_hi[w] = (uint32_t)((uint64_t)list_hi[i] * (uint64_t)kids + __umul64hi(list[i], (uint64_t)kids) +
                                       (lo < plo ? 1u : 0u));
        }
    }
}

// ---- a whole small level in one launch ----------------------------------------
// When every segment of the level is one tile (at most 1024 cubes) and no
// segment forms per-parent thresholds, one block per segment runs finalize,
// the mean of s, the threshold, the selection and the decision, with each
// thread's m and s kept in registers between the steps and the reductions in
// LDS.  With one tile per segment each per-segment reduction of the
// multi-launch path reduces a single tile record (the other threads add
// zeros), so this is the same arithmetic in the same order and the results
// are bitwise those of the multi-launch path.
//
// The level of a single integral also lays out the next one if it splits:
// the children's ids and the table the host would send, so that the next
// level starts with its sampling launch and not with a next-list kernel
// before it (3.5 us and a gap, of 24 us for a level of a hundred cubes).
__global__ __launch_bounds__(kLevelThreads) void level_small_kernel(const LevelArgs a)
{
    __shared__ double sh[kWaves];
    __shared__ uint64_t list[kTileCubes];
    __shared__ uint32_t list_hi[kTileCubes];
    __shared__ int shf[kWaves];
    __shared__ int go_on;
    if (a.clock && blockIdx.x == 0 && threadIdx.x == 0) *a.clock = device_clock();
    const int si = blockIdx.x;
    const Segment& sg = a.segs[si];
    const int slot = sg.slot, level = sg.level;
    const int64_t tile = sg.tile_base;
    const bool thr_on = sg.need_thr != 0;
    const DecideIn in = decide_in(a, si);
    const double sigma_mult = a.slots[sg.slot].sigma_mult;
    double m_r[kPerThread], s_r[kPerThread];
    double tot_s = 0.0, s_ext[2] = {0.0, 0.0};
    int bad = 0;
    finalize_tile<true>(a, tile, si, m_r, s_r, &tot_s, &bad, s_ext);
    const int64_t n = sg.n_cubes;
    double mu = 0.0, sdv = 0.0, thr = 0.0, tot_sq = 0.0;
    if (thr_on) {
        mu = tot_s / (double)n;
        const int e = thr_scale_exp(mu, s_ext[0], s_ext[1]);
        double acc = 0.0;
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) {
            const double d = (int64_t)threadIdx.x + j * kLevelThreads < n ? ldexp(s_r[j] - mu, -e) : 0.0;
            acc += d * d;
        }
        tot_sq = block_sum(acc, sh);
        sdv = ldexp(sqrt(tot_sq / (double)n), e);
        thr = mu + sigma_mult * sdv;
    }
    double accM = 0.0, accS2 = 0.0, selM = 0.0, selS2 = 0.0, margin = DBL_MAX;
    int64_t nsel = 0;
    int sel_r[kPerThread] = {};
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) {
        const int64_t cl = threadIdx.x + (int64_t)j * kLevelThreads;
        if (cl >= n) break;
        const int64_t c = sg.cube_base + cl;
        const double m = m_r[j], s = s_r[j];
        const bool sel = thr_on && (s > thr);
        sel_r[j] = sel;
        a.sel[c] = sel ? 1 : 0;
        if (sel) {
            selM += m;
            selS2 += s * s;
            ++nsel;
        } else {
            accM += m;
            accS2 += s * s;
        }
        if (thr_on && thr > 0.0) margin = fmin(margin, fabs(s - thr) / thr);
    }
    stores_done(); // ahead of the reduction's barriers: the record goes out behind every wave's stores
    const SelTotals tot = block_reduce_sel(SelTotals{accM, accS2, selM, selS2, margin, nsel});
    if (threadIdx.x == 0) {
        TileRec& T = a.tiles[tile];
        T.sum_sq = tot_sq;
        T.accM = tot.accM;
        T.accS2 = tot.accS2;
        T.selM = tot.selM;
        T.selS2 = tot.selS2;
        T.min_margin = tot.margin;
        T.n_sel = tot.nsel;
        T.sel_prefix = 0;
        if (thr_on) {
            a.stats[si].mu = mu;
            a.stats[si].s_min = s_ext[0];
            a.stats[si].s_max = s_ext[1];
            a.stats[si].sd = sdv;
            a.stats[si].thr = thr;
        }
        const Decision dec =
            decide_write(a, si, in, tot.accM, tot.accS2, tot.selM, tot.selS2, tot.margin, tot.nsel, bad);
        // a non-finite integral ends here whatever its decision
        go_on = dec == kSplit && !bad && tot.nsel * (int64_t)in.kids <= a.ahead_cap;
    }
    if (!a.ahead) return;
    __syncthreads();
    if (!go_on) return;
    const SlotDesc& sd = a.slots[slot];
    int base = 0;
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) {
        int total;
        const int pos = block_excl_scan_flag(sel_r[j], shf, &total);
        if (sel_r[j]) {
            const int64_t c = sg.cube_base + threadIdx.x + (int64_t)j * kLevelThreads;
            list[base + pos] = a.uid[c];
            list_hi[base + pos] = a.uid_hi ? a.uid_hi[c] : 0u;
        }
        base += total;
    }
    __syncthreads();
    const int64_t nn = (int64_t)base * sd.kids;
    const AheadList at = AheadList::place(nn, a.ahead_cap, a.ahead_wide != 0, a.ahead_side);
    write_children(list, list_hi, base, sd.split, sd.dim, sd.kids, (uint64_t*)(a.ahead + at.uid),
                   a.ahead_wide ? (uint32_t*)(a.ahead + at.hi) : nullptr);
    __syncthreads(); // every thread is past its reads of this level's segment
    if (threadIdx.x == 0) {
        Segment g{};
        g.slot = slot;
        g.level = level + 1;
        g.n_cubes = nn;
        g.n_tiles = (nn + kTileCubes - 1) / kTileCubes;
        g.need_thr = g.level < sd.max_depth ? 1 : 0;
        if (g.need_thr && sd.scope == 1 && nn > sd.kids) g.group_size = sd.kids;
        *a.ahead_seg = g;
        *a.ahead_bseg = BSeg{0, 0, 0};
        *a.ahead_prev = make_double2(in.prev.x + tot.accM, in.prev.y + tot.accS2);
        *a.ahead_flags = 0;
    }
}

// ---- spawn: children of the selected cubes, in list order ------------------
// One block per tile of the finished level.
__device__ void spawn_tile(const LevelArgs& a, int64_t tile)
{
    __shared__ uint64_t list[kTileCubes];
    __shared__ uint32_t list_hi[kTileCubes];
    __shared__ int shf[kWaves];
    const int si = seg_of_tile(a.segs, a.n_segs, tile);
    const Segment& sg = a.segs[si];
    if (!sg.do_split) return;
    const SlotDesc& sd = a.slots[sg.slot];
    const int D = sd.dim;
    const int64_t kids = sd.kids;
    const int64_t first = (tile - sg.tile_base) * kTileCubes;
    int flags[kPerThread];
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) {
        const int64_t cl = first + threadIdx.x + (int64_t)j * kLevelThreads;
        flags[j] = (cl < sg.n_cubes) ? a.sel[sg.cube_base + cl] : 0;
    }
    int base = 0;
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) {
        int total;
        const int pos = block_excl_scan_flag(flags[j], shf, &total);
        if (flags[j]) {
            const int64_t c = sg.cube_base + first + threadIdx.x + (int64_t)j * kLevelThreads;
            list[base + pos] = a.uid[c];
            list_hi[base + pos] = a.uid_hi ? a.uid_hi[c] : 0u;
        }
        base += total;
    }
    __syncthreads();
    const int64_t first_out = sg.child_base + a.tiles[tile].sel_prefix * kids;
    write_children(list, list_hi, base, sd.split, D, kids, a.next_uid + first_out,
                   a.next_uid_hi ? a.next_uid_hi + first_out : nullptr);
}

// ---- roots: uid = r for the d^D cubes of a newly admitted integral ----------
__device__ void roots_block(const RootArgs& a, int blk)
{
    const int si = blk / a.blocks_per_seg;
    const int part = blk % a.blocks_per_seg;
    const Segment& sg = a.segs[si];
    for (int64_t r = (int64_t)part * kLevelThreads + threadIdx.x; r < sg.n_cubes;
         r += (int64_t)a.blocks_per_seg * kLevelThreads) {
        a.uid[sg.cube_base + r] = (uint64_t)r;
        if (a.uid_hi) a.uid_hi[sg.cube_base + r] = 0u;
    }
}

// The next list in one launch: the first n_spawn blocks spawn children (one
// per tile of the finished level), the next n_roots write roots of new
// integrals, and the rest copy a small level's table and the new integrals'
// descriptors from mapped host memory.
__global__ __launch_bounds__(kLevelThreads) void next_list_kernel(const LevelArgs a, const RootArgs ra,
                                                                  const CopyArgs ca, int64_t n_spawn, int64_t n_roots)
{
    const int64_t b = blockIdx.x;
    if (b < n_spawn) {
        spawn_tile(a, b);
    } else if (b < n_spawn + n_roots) {
        roots_block(ra, (int)(b - n_spawn));
    } else if (b == n_spawn + n_roots) {
        for (int i = threadIdx.x; i < ca.n; i += kLevelThreads) ca.dst[i] = ca.src[i];
    } else {
        constexpr int kWords = sizeof(SlotDesc) / sizeof(uint4);
        static_assert(kWords * sizeof(uint4) == sizeof(SlotDesc) && kWords <= kLevelThreads, "one word a thread");
        const int slot = ca.slots[b - n_spawn - n_roots - 1];
        if (threadIdx.x < kWords)
            ((uint4*)(ca.slot_dst + slot))[threadIdx.x] = ((const uint4*)(ca.slot_src + slot))[threadIdx.x];
    }
}

// ---- debug entry points ------------------------------------------------------
__global__ void debug_philox_kernel(uint32_t k0, uint32_t k1, const uint32_t* ctr, uint32_t* out, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const U4 r = philox4x32_10(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3], k0, k1);
    out[4 * i] = r.x;
    out[4 * i + 1] = r.y;
    out[4 * i + 2] = r.z;
    out[4 * i + 3] = r.w;
}

__global__ void debug_points_kernel(const SlotDesc* sdp, int level, uint64_t uid, int trial, int64_t s0, int64_t n,
                                    double* x)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const SlotDesc& sd = *sdp;
    const int D = sd.dim;
    double lo[kMaxDim], h[kMaxDim];
    cube_corner(sd, D, level, uid, lo, h);
    const int64_t s = s0 + k;
    for (int i = 0; i < D; ++i) {
        const uint64_t nw = (uint64_t)s * (uint64_t)D + (uint64_t)i;
        const U4 r = philox4x32_10((uint32_t)(nw >> 2), ctr_word1(trial, level, 0u), (uint32_t)uid,
                                   (uint32_t)(uid >> 32), (uint32_t)sd.seed, (uint32_t)(sd.seed >> 32));
        const uint32_t words[4] = {r.x, r.y, r.z, r.w};
        const uint32_t w = words[nw & 3u];
        x[k * D + i] = fma(ldexp(h[i], -24), (double)((w >> 8) | 1u), lo[i]);
    }
}

} // namespace

hipError_t launch_finalize(const LevelArgs& a, hipStream_t st)
{
    if (a.n_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(finalize_kernel, dim3((unsigned)a.n_tiles), dim3(kLevelThreads), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_level_small(const LevelArgs& a, hipStream_t st)
{
    if (a.n_segs <= 0) return hipSuccess;
    hipLaunchKernelGGL(level_small_kernel, dim3((unsigned)a.n_segs), dim3(kLevelThreads), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_threshold(const LevelArgs& a, hipStream_t st)
{
    if (a.n_tiles <= 0) return hipSuccess;
    if (!a.fused) hipLaunchKernelGGL(seg_mean_kernel, dim3(a.n_segs), dim3(kLevelThreads), 0, st, a);
    hipLaunchKernelGGL(tile_sqdev_kernel, dim3((unsigned)a.n_tiles), dim3(kLevelThreads), 0, st, a);
    if (!a.fused) hipLaunchKernelGGL(seg_thr_kernel, dim3(a.n_segs), dim3(kLevelThreads), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_group_threshold(const LevelArgs& a, hipStream_t st)
{
    if (a.n_groups <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((a.n_groups + kWaves - 1) / kWaves, 65536);
    hipLaunchKernelGGL(group_thr_kernel, dim3((unsigned)blocks), dim3(kLevelThreads), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_select(const LevelArgs& a, hipStream_t st)
{
    if (a.n_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(tile_select_kernel, dim3((unsigned)a.n_tiles), dim3(kLevelThreads), 0, st, a);
    if (!a.fused) hipLaunchKernelGGL(seg_decide_kernel, dim3(a.n_segs), dim3(kLevelThreads), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_next_list(const LevelArgs& a, const RootArgs& ra, const CopyArgs& ca, hipStream_t st)
{
    const int64_t n_spawn = a.n_tiles > 0 ? a.n_tiles : 0;
    const int64_t n_roots = ra.n_segs > 0 ? (int64_t)ra.n_segs * ra.blocks_per_seg : 0;
    const int64_t n_copy = ca.n > 0 ? 1 + ca.n_slots : 0;
    if (n_spawn + n_roots + n_copy <= 0) return hipSuccess;
    hipLaunchKernelGGL(next_list_kernel, dim3((unsigned)(n_spawn + n_roots + n_copy)), dim3(kLevelThreads), 0, st, a,
                       ra, ca, n_spawn, n_roots);
    return hipGetLastError();
}

hipError_t launch_debug_philox(uint32_t k0, uint32_t k1, const uint32_t* ctr, uint32_t* out, int64_t n,
                               hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(debug_philox_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, k0, k1, ctr, out,
                       n);
    return hipGetLastError();
}

hipError_t launch_debug_points(const SlotDesc* sd, int level, uint64_t uid, int trial, int64_t s0, int64_t n,
                               double* x, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(debug_points_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, sd, level, uid,
                       trial, s0, n, x);
    return hipGetLastError();
}

hipError_t launch_sample(int integrand, int dim, int eval, int hint, int grid, int block, hipStream_t st,
                         const SampleArgs& a)
{
    switch (integrand) {
    case 0: return launch_sample_0(dim, eval, hint, grid, block, st, a);
    case 1: return launch_sample_1(dim, eval, hint, grid, block, st, a);
    case 2: return launch_sample_2(dim, eval, hint, grid, block, st, a);
    case 3: return launch_sample_3(dim, eval, hint, grid, block, st, a);
    case 4: return launch_sample_4(dim, eval, hint, grid, block, st, a);
    case 5: return launch_sample_5(dim, eval, hint, grid, block, st, a);
    case 6: return launch_sample_6(dim, eval, hint, grid, block, st, a);
    case 7: return launch_sample_7(dim, eval, hint, grid, block, st, a);
    default: return hipErrorInvalidValue;
    }
}

const void* sample_kernel_ptr(int integrand, int dim, int eval, int hint)
{
    switch (integrand) {
    case 0: return sample_kernel_ptr_0(dim, eval, hint);
    case 1: return sample_kernel_ptr_1(dim, eval, hint);
    case 2: return sample_kernel_ptr_2(dim, eval, hint);
    case 3: return sample_kernel_ptr_3(dim, eval, hint);
    case 4: return sample_kernel_ptr_4(dim, eval, hint);
    case 5: return sample_kernel_ptr_5(dim, eval, hint);
    case 6: return sample_kernel_ptr_6(dim, eval, hint);
    case 7: return sample_kernel_ptr_7(dim, eval, hint);
    default: return nullptr;
    }
}

} // namespace zmc
