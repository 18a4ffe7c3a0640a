// zmc_kernels.hpp -- argument blocks and host-side launchers of the device
// pipeline that runs one level of the tree search over every resident
// integral:
//
//   sample      (cube, trial, chunk) units -> FP64 partial sums S1 = sum f,
//               S2 = sum f^2 over the chunk's points (one kernel per
//               (integrand, D, eval) bucket, persistent over its units)
//   finalize    per cube: I_t = V * S1_t / N, m = mean_t I_t, s = std_t I_t
//   seg_mean / tile_sqdev / seg_thr
//               per integral: thr = mean(s) + sigma_mult * std(s)
//   tile_select per cube: split = s > thr; accepted / selected sums per tile
//   seg_decide  per integral: totals, stop rules, rank base of every tile
//   spawn       2^D children of every split cube, in list order
//   roots       level-0 list of a newly admitted integral
//   level_small finalize .. seg_decide in one launch when every segment of
//               the level is a single tile
#pragma once

#include <hip/hip_runtime.h>

#include "zmc_device.hpp"

namespace zmc {

struct LevelArgs {
    const SlotDesc* slots;
    const Segment* segs;
    int32_t n_segs;
    int32_t fused;           // per-segment steps in the tile kernels' last blocks
    int64_t n_tiles;
    const uint64_t* uid;
    const uint32_t* uid_hi;  // id bits 64..83, or NULL (all zero)
    const double2* partial;
    double* m;
    double* s;
    uint8_t* sel;
    TileRec* tiles;
    SegStats* stats;
    const double2* prev_tot; // per segment: running (M, S2) before this level
    double* tr_S1;           // optional per (cube, trial) sums (trace)
    double* tr_S2;
    uint64_t* next_uid;      // spawn output
    uint32_t* next_uid_hi;   // spawn output: id bits 64..83, or NULL
    double* gthr;            // per-parent thresholds, one per sibling group
    int64_t n_groups;
    int32_t* seg_count;      // per segment: tile blocks done (0 between kernels)
    SegStats* host_stats;    // optional mapped host copy of the decisions
    const int32_t* seg_flags; // per segment: flags the sampling launches raised
    uint64_t* clock;          // mapped host memory: when the per-cube kernels began (device clock)
    uint32_t* host_seq;       // per segment, mapped host memory: set to seq once host_stats holds the decision
    uint32_t seq;             // number of this level, unlike any that came before
    // the one-block level of a single integral lays out the next level itself
    // (ahead NULL: it does not): the children's ids into this block, where
    // the host would have allocated lists of their number (AheadList), and the
    // table in place of this level's own
    char* ahead;
    int32_t ahead_side;       // end of the arena that the block was taken from
    int32_t ahead_wide;       // the ids take a second array
    Segment* ahead_seg;
    BSeg* ahead_bseg;
    double2* ahead_prev;
    int32_t* ahead_flags;
    int64_t ahead_cap;        // children the block holds; with more the host lays the list out
};

// The lists of n children within a block for `cap` of them: at its lower end
// for side 0 of the arena, at its upper end for side 1, the upper id words
// after (before, for side 1) the lower ones, each in whole 256 bytes.  So the
// host can give the block back and take the n children's bytes alone, and the
// next level leaves as much of the arena as with a list that the host laid out.
struct AheadList {
    int64_t uid, hi; // byte offsets
    __host__ __device__ static constexpr int64_t padded(int64_t bytes) { return (bytes + 255) & ~(int64_t)255; }
    __host__ __device__ static constexpr int64_t bytes(int64_t n, bool wide)
    {
        return padded(n * (int64_t)sizeof(uint64_t)) + (wide ? padded(n * (int64_t)sizeof(uint32_t)) : 0);
    }
    __host__ __device__ static constexpr AheadList place(int64_t n, int64_t cap, bool wide, int side)
    {
        const int64_t u = padded(n * (int64_t)sizeof(uint64_t));
        return side == 0 ? AheadList{0, u} : AheadList{bytes(cap, wide) - u, bytes(cap, wide) - bytes(n, wide)};
    }
};

// What next_list_kernel copies from mapped host memory into device memory for
// the kernels that follow it: a small level's table and the descriptors of
// newly admitted integrals.
struct CopyArgs {
    static constexpr int kMaxSlots = 8;
    const uint4* src; // the table
    uint4* dst;
    int32_t n;        // 16-byte words; 0: nothing is copied
    int32_t n_slots;
    const SlotDesc* slot_src;
    SlotDesc* slot_dst;
    int32_t slots[kMaxSlots];
};

struct RootArgs {
    const Segment* segs; // segments whose roots are written (cube_base, n_cubes)
    int32_t n_segs;
    int32_t blocks_per_seg;
    uint64_t* uid;
    uint32_t* uid_hi; // written 0 when not NULL
};

// Threads per block of the per-cube kernels, two cubes of a tile each.  A small
// level has few tiles and waits for each block's chain of loads, divisions and
// reductions: finalize over 8 tiles takes 18.0 us with 256 threads, 13.5 with
// 512 and 13.5 with 1024, the selection 8.7, 9.8 and 13.2 (its barriers wait
// for more waves); over 464 tiles finalize takes 35, 27 and 48.
constexpr int kLevelThreads = 512;

// The doubles (40 KiB) that finalize stages in LDS: a row for each thread's
// cube where a row of n values fits.  Compared by division: trials times
// chunks reaches 2^29 and more.
constexpr int kStage = 5120;
__host__ __device__ constexpr bool row_fits(int64_t n) { return n <= kStage / kLevelThreads; }

// Launchers; each returns the hipError_t of its launch.
// Occupancy variants of every sampling kernel: the waves per SIMD the
// register allocator and the scheduler aim at (1 = no constraint).  Most
// buckets run within 2% of their best in the first; where more registers or
// more waves pay, which variant wins depends on the bucket and is measured.
constexpr int kWaveHints[] = {1, 4, 5, 6};
constexpr int kNumWaveHints = 4;
// hint value that selects the sampling kernel that also keeps the sums of
// squares (traced levels); it runs at the compiler's default occupancy
constexpr int kSumsVariant = kNumWaveHints;
// hint value of the FP64 sine and cosine kernels whose arguments may exceed
// kTrigMax (every other bucket takes its unconstrained variant for it)
constexpr int kAnyArgVariant = kNumWaveHints + 1;

// block: threads per sampling block, 64, 128 or 256 (whole waves; results
// do not depend on it: every unit is one wave's work)
hipError_t launch_sample(int integrand, int dim, int eval, int hint, int grid, int block, hipStream_t st,
                         const SampleArgs& a);
const void* sample_kernel_ptr(int integrand, int dim, int eval, int hint);
hipError_t launch_finalize(const LevelArgs& a, hipStream_t st);
// finalize + threshold + selection + decision of a level whose segments are
// all one tile without per-parent thresholds, one block per segment
hipError_t launch_level_small(const LevelArgs& a, hipStream_t st);
hipError_t launch_threshold(const LevelArgs& a, hipStream_t st);
hipError_t launch_group_threshold(const LevelArgs& a, hipStream_t st);
hipError_t launch_select(const LevelArgs& a, hipStream_t st);
// Spawn (a.n_tiles blocks, none when 0), roots (ra.n_segs segments, none when
// 0) and the copies of ca in one launch.
hipError_t launch_next_list(const LevelArgs& a, const RootArgs& ra, const CopyArgs& ca, hipStream_t st);
hipError_t launch_debug_philox(uint32_t k0, uint32_t k1, const uint32_t* ctr, uint32_t* out, int64_t n,
                               hipStream_t st);
hipError_t launch_debug_points(const SlotDesc* sd, int level, uint64_t uid, int trial, int64_t s0, int64_t n,
                               double* x, hipStream_t st);

// Per-integrand launch tables (one translation unit per integrand).
#define ZMC_DECLARE_SAMPLE(F)                                                                              \
    hipError_t launch_sample_##F(int dim, int eval, int hint, int grid, int block, hipStream_t st,               \
                                 const SampleArgs& a);                                                             \
    const void* sample_kernel_ptr_##F(int dim, int eval, int hint);
ZMC_DECLARE_SAMPLE(0)
ZMC_DECLARE_SAMPLE(1)
ZMC_DECLARE_SAMPLE(2)
ZMC_DECLARE_SAMPLE(3)
ZMC_DECLARE_SAMPLE(4)
ZMC_DECLARE_SAMPLE(5)
ZMC_DECLARE_SAMPLE(6)
ZMC_DECLARE_SAMPLE(7)
#undef ZMC_DECLARE_SAMPLE

} // namespace zmc
