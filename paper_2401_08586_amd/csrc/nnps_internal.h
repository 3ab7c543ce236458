// Internal definitions shared by the HIP kernels and the C-ABI host code.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nnps {

// Targets per work block: one wavefront, one target per lane.
constexpr int kWave = 64;
// Candidate positions staged in LDS per chunk in the count pass (even).
constexpr int kStage = 512;
// Largest candidate union of a block (ranked by original index in the count pass, staged
// whole in the fill); blocks above it send their rows to the long-row path.
constexpr int kUnion2 = 512;
constexpr int kUnion3 = 1024;
// Accepted-candidate bits the count pass keeps per target, indexed by the candidate's
// position in the block's union (32 positions per word), stored word-major so a
// wavefront's stores coalesce. Blocks with a larger union take the long-row path.
constexpr int kCandWords2 = kUnion2 / 32;
constexpr int kCandWords3 = kUnion3 / 32;
// Rows of cells are walked in segments of this many cells, so that is also a work block's
// largest x-span. (Where the matrix cores test in FP16 or FP32 the recheck band grows with the
// square of the span, 2^-18 of twice the squared half widths, to 0.016 squared cell widths there.)
constexpr int kRowSegment = 64;
// 3D sets are counted by small blocks, a wavefront each for unions up to kSmallUnion (k_count_small),
// where a block's union is expected to be below kSparseUnion candidates, unless the last
// synchronising call found more than kSparseTargets targets in the average block: a clump in a large
// box is sparse by the first measure only. Steps of a million uniform points in 3D (random numbering,
// FP16 / FP64, us): 0.1 points a cell 1156 / 1486 against 1850 / 2578 with four wavefronts a block,
// 0.25 (a union of 148, 16 targets) 640 / 787 and 905 / 1215, 0.5 (297, 32) 565 / 700 and 527 / 684,
// 1.0 548 / 683 and 504 / 644. (Before the unions were ranked in the count: 2090 / 1945, 1080 / 1025,
// 650 / 660, 589 / 625.)
constexpr int kSmallUnion = 256;
constexpr double kSparseUnion = 220.0;
constexpr int kSparseTargets = 20;
// Dense-cell path: candidates staged per chunk, targets per work unit (a workgroup of
// four wavefronts, 64 targets each) and the default thresholds.
constexpr int kDenseChunk = 1024;
// The FP16 fill that tests stages fewer candidates per chunk, so that its tables (test records,
// positions and the per-wavefront queues of accepted candidates) fit five workgroups per CU (a
// multiple of 128).
constexpr int kDenseChunkF16 = 896;
// Default bound on the device scratch for the count's kept bits (MiB).
constexpr int kDenseBitsMiB = 16384;
constexpr int kDenseQueue = 512;  // per-wavefront queue of a row's accepted candidates in a chunk
constexpr int kDenseThreads = 256;
constexpr int kDenseFillThreads = 1024;  // the dense fill that takes the count's kept bits
constexpr int kDenseFillQueue = 448;     // and its per-wavefront queue
// Targets of one dense cell that share staged candidates: 256 in the count and the testing
// fill, 64, a work unit, in the fill that takes the kept bits, whose output decides the time
// (a core cell's 256 rows can be 18 MB, as much as a workgroup's share of a whole batch: units
// of 256 left half of the chip idle at the end, 3000 us for a clustered batch alone against
// 2260 with 64 and 2200 with 32; several batches in flight 1956, 1945 and 1956).
constexpr int kDenseSlice = 256;
constexpr int kDenseUnit = 64;
constexpr int kDenseUnion3 = 512;
constexpr int kDenseUnion2 = 160;
constexpr int kDenseGrid = 1280;  // five workgroups on each of the 256 compute units
constexpr int64_t kDenseMaxEntries = int64_t(1) << 28;
constexpr int kDenseStats = 6;  // candidates, band, false pos, false neg, outside disagree, rows

// Per-block descriptors the count pass leaves for the fill (ints per block), and the
// spare descriptors of the last round over the XCDs.
constexpr int kBlockDescInts = 24;
constexpr int kXcdPad = 8;
// Where the count pass leaves the ranks of the blocks' unions, in pieces of kRankPiece entries. A
// place for a full union per block while that is at most kRankRoom entries a particle (a million
// lattice points in 3D: 34, and 142 while it isn't known whether there are dense cells) or
// kRankSmall in all; else, and where many blocks are expected to be small
// (a grid of few particles: up to a block, so 2 KB, per particle), kRankPool entries a particle and
// a full union more in each of kRankPools pools from which the blocks take what they need (a
// particle is in the unions of the blocks of 27 cells, 14 of them in a lattice). A block that finds
// its pool empty sends its rows to the long-row path.
constexpr int kRankPiece = 16;
constexpr int64_t kRankRoom = 160;
constexpr int64_t kRankSmall = int64_t(1) << 24;
constexpr int64_t kRankPool = 48;
constexpr int kRankPools = 256;
constexpr int kRankPoolStride = 16;  // ints between two pools' counters: a cache line each

// Device error flags.
constexpr int kErrDomain = 1;
constexpr int kErrCapacity = 2;
constexpr int kErrLongRow = 4;

// A structure's flags and counters (int32 on the device). A build or an update starts
// them at zero; a pass leaves the counters it used as it found them, so a count or a
// fill may follow another, or be replayed, without a launch that clears them.
enum Flag {
    kFlagErr = 0,    // device error flags
    kFlagSeen,       // 1: some cell is dense
    kFlagHeavy,      // long rows listed by the running fill
    kFlagLong,       // long rows of the last fill
    kFlagLongDone,   // workgroups of the long-row kernel that are through with the list
    kFlagUnit,       // next work unit of the running dense pass
    kFlagBad,        // the assignment's error flags (the cell starts' scan moves them on)
    kFlagBlocks,     // work blocks of the last count
    kFlags           // an even number: 64-bit counts follow
};
static_assert(kFlags % 2 == 0, "64-bit counts follow the flags");

// Statistic slots (int64 on the device).
enum StatSlot {
    kStCandidates = 0,
    kStBand,
    kStFalsePos,
    kStFalseNeg,
    kStOutsideDisagree,
    kStHeavy,
    kStDenseRows,
    kStCount
};

// Everything a kernel needs to know about one particle set's grid and thresholds.
struct Frame {
    int dim;
    int mode;
    int n;
    int F;              // fixed-point fraction bits per cell width
    int nc[3];          // cells per axis (1 for unused axes)
    int ncell;
    double lo[3], hi[3];
    double w;           // cell width
    double s;           // 2^F / w
    double R2;          // fl(R*R)
    int xwin;           // largest x-span of a work block, in cells
    uint16_t t_lo, t_hi, t_mid;  // FP16 thresholds on r2 = 4|delta|^2 (bit patterns)
    float t32_lo, t32_hi, t32_mid;  // FP32 thresholds on the same r2
    // FP32 distances of the fill: positions in units of quantum = 2^-k, a power of two; pairs
    // nearer than near2 (squared, in quanta) are taken in binary64
    double inv_quantum;
    float quantum, near2;
};

// One particle set of a launch. All sets of a launch share one global particle index
// space (set s owns [poff, poff + n)) and one global cell index space ([coff, coff +
// ncell)), so one sort and one kernel launch per pass cover every set.
struct SetDesc {
    Frame fr;                // fr.n = this set's particle count
    int poff, coff;          // first global particle / cell index
    const double* pos;       // caller's positions [n][dim] (float64)
    const double* disp;      // incremental update: displacements [n][dim] added to pos, or null
    int64_t* row_ptr;        // caller's CSR row pointers [n + 1]
    int32_t* col;            // caller's CSR column indices (set-local)
    float* dist;             // caller's CSR distances
    int64_t capacity;        // entries available in col and dist
};

// Index of the set owning global index v, given offs[0..nsets] ascending.
__device__ __forceinline__ int find_set(const int* __restrict__ offs, int nsets, int v)
{
    int lo = 0, hi = nsets - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (offs[mid] <= v) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

}  // namespace nnps
