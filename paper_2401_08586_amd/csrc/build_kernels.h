// Launchers for the cell-build and search kernels (internal to the library).
#pragma once

#include "nnps_internal.h"

namespace nnps {

// What every kernel of one launch shares: the set table and the global index spaces.
struct Launch {
    int dim, mode;             // shared by all sets of a launch
    int nsets;
    int ntot;                  // total particles (sum of the sets' n)
    int ncell_tot;             // total cells
    const SetDesc* sets;       // [nsets] (device)
    const int* poffs;          // [nsets + 1] particle offsets (device)
    const int* coffs;          // [nsets + 1] cell offsets (device)
    const int* roffs;          // [nsets + 1] offsets of the sets' row segments (device)
    int nrows_tot;             // total row segments (x-lines cut into pieces of 64 cells)
};

hipError_t launch_fill_i32(int* p, int64_t m, int v, hipStream_t st);
int row_segments(int ncx);  // pieces a row of ncx cells is walked in
// hot: cells of thousands of particles are expected.
hipError_t launch_assign(const Launch& L, bool hot, uint32_t* key, int* slot, int* cell_count, int* err, hipStream_t st);
// Cell starts from the cells' counts; also starts the structure's flags for this build.
hipError_t launch_cell_scan(const Launch& L, const int* cell_count, int* cell_start, int64_t* partial, int* flags,
                            hipStream_t st);
int64_t scan_partials_needed(int64_t m);
int radix_tiles(int n);
size_t radix_table_entries(int n);
// Incremental update of a built structure (see k_upd_move): device tables of one update.
struct Update {
    uint32_t* knew;           // [ntot] new cell key by particle
    uint32_t* mig;            // [ceil(ntot / 32)] bit s: the particle at old position s changed cell
    int* leave;               // [ncell_tot + 1] migrants out of each cell
    int* arrive;              // [ncell_tot + 1] migrants into each cell
                              // (leave, arrive and mig are one block, zero between updates: see update_of)
    int* aslot;               // [ntot] by particle: a migrant's arrival slot in its new cell
    int* cs_old;              // [ncell_tot + 1] cell starts before the update
    uint32_t* skey2;          // [ntot] new order: cell keys
    int* perm2;               // [ntot] new order: particle indices
};
// U1: move (when the set has displacements), cells, migrant flags and counts.
hipError_t launch_update_move(const Launch& L, const uint32_t* skey, const int* inv, const Update& u, int* err,
                              hipStream_t st);
// U2: new cell occupancies and starts (cell_start is rewritten; the old one goes to cs_old).
hipError_t launch_update_cells(const Launch& L, int* cell_start, int* cnt, const Update& u, int64_t* partial,
                               int* flags, hipStream_t st);
// Dense-cell path: device tables of one build. A cell is "dense" when its stencil holds
// more than `thresh` particles; runs of dense cells get no work blocks. Each dense cell g owns the list ulist[uoff[g] ..
// uoff[g] + usz[g]) of the sorted positions of the particles in its 3^d stencil, in
// ascending original index, and ceil(occupancy / kDenseUnit) work units.
struct DenseBuild {
    int thresh;             // stencil size above which a window is dense
    int64_t cap;            // capacity of the union lists (entries)
    int* usz;               // [ncell_tot] stencil size of dense cells, else 0
    int* wdense;            // [ncell_tot] 1 for every cell of a dense window
    int64_t* uoff;          // [ncell_tot + 1] exclusive scan of usz
    int* nsl;               // [ncell_tot] work units per cell
    int* unit_off;          // [ncell_tot + 1] exclusive scan of nsl
    int* ucell;             // [ntot] cell of each work unit
    int* dn;                // [1] entries in use; 0 when the dense path is off for the build
    int* ecnt;              // [ntot] dense stencils each particle belongs to
    int* epos;              // [ntot + 1] exclusive scan of ecnt
    uint32_t *uk0, *uk1;    // [cap] sort keys (dense cell)
    int *uv0, *uv1;         // [cap] sort values (sorted position)
    uint32_t* table;        // radix scratch
    int64_t* partial;       // scan scratch
    int* seen;              // [1] set to 1 when any cell is dense
    uint32_t* dbn;          // [ncell_tot] (target, chunk) pairs of each dense cell (saturated)
    int64_t* dboff;         // [ncell_tot + 1] exclusive scan of dbn
};

// The sort by cell: of a build (key and slot of every particle), or of an update (moved: the
// old order skey / perm and u, every particle's new sorted position going to u.skey2, u.perm2).
struct PlaceArgs {
    bool moved;
    const uint32_t* key;
    const int* slot;
    uint32_t* skey_out;
    int* perm_out;
    const uint32_t* skey;
    const int* perm;
    Update u;
};

// The pack of the sorted particles (see pack_particle); skey_out / perm_out: a copy of the
// order, or null; clear0, clear1: counters to leave zero for the next build or update.
struct PackArgs {
    const uint32_t* skey;
    const int* perm;
    double* spos;
    float4* rq;
    int* inv;
    uint32_t* skey_out;
    int* perm_out;
    int* clear0;
    int64_t nclear0;
    int* clear1;
    int64_t nclear1;
};

// The work-block table (see row_blocks).
struct BlockTable {
    const int* wdense;      // null: no dense cells
    int* boff;              // [nrows_tot + 1] blocks of each segment, then the total
    int* bstart;            // [total + 1]
    int* bset;              // [total]
    const int* cell_start;  // set by the launchers
    int fold;
};

// After the cell starts: the sort (place), the stencil sizes with the dense flag (dense) and
// the segments' block counts (blocks), each if given.
hipError_t launch_sort(const Launch& L, const PlaceArgs* place, const DenseBuild* dense, const BlockTable* blocks,
                       const int* cell_start, hipStream_t st);
// After that: the pack and the block table, each if given.
hipError_t launch_pack(const Launch& L, const PackArgs* pack, const BlockTable* blocks, const int* cell_start,
                       int64_t* partial, hipStream_t st);
// After the stencil sizes, before the block table: dense windows, union offsets, work units.
hipError_t launch_dense_cells(const Launch& L, const int* cell_start, const DenseBuild& d, hipStream_t st);
// After the sort and pack: the union lists. *ulist receives the list array. `nmax` is the
// largest set's size; above a bound (dense_unions_sorted) the lists are made by a sort, which
// needs ecnt, epos, uk0, uk1, uv1 and table, else they are ranked in place.
bool dense_unions_sorted(int64_t nmax);
hipError_t launch_dense_unions(const Launch& L, int64_t nmax, const int* cell_start, const uint32_t* skey, const int* perm,
                               const int* inv, const DenseBuild& d, hipStream_t st, int** ulist);
// What the row pointer kernel does beside them: what a caller that waits for the count wants on
// the host, written there (the structure's flags, then each set's nnz, and `pairs`, if given, in
// the last word), and the count's own counters cleared.
struct RowptrExtras {
    int64_t* host = nullptr;  // kHostWords words that the host reads after the stream; null: none
    int* flags = nullptr;
    const int64_t* pairs = nullptr;
    const int* nblk = nullptr;  // the number of blocks, to go with the flags
    int* rpool = nullptr;     // the rank pools' counters, to leave zero for the next count; or null
};
constexpr int kHostWords = 64;
constexpr int kHostSets = kHostWords - 1 - kFlags / 2;  // sets that fit
// Row pointers of every set from the counts; also each particle's row start by sorted
// position (rsort[inv[i]]).
hipError_t launch_rowptr(const Launch& L, const int* counts, int64_t* partial, int64_t* nnz, const int* inv,
                         int64_t* rsort, const RowptrExtras& rep, hipStream_t st);

// Search passes over every block of every set. `nblk_max` bounds the number of blocks
// (the exact count is on the device).
struct SearchArgs {
    Launch L;
    const uint32_t* skey;     // sorted global cell keys
    const int* perm;          // sorted position -> global particle index
    const int* cell_start;    // [ncell_tot + 1]
    const double* spos;       // sorted FP64 positions [ntot][4], the fourth the particle index (int64 bits)
    const float4* rq;         // sorted FP32 relative coordinates + packed cell bits
    const int* bstart;        // block starts [nblk + 1]
    const int* bset;          // set of each block [nblk]
    const int* nblk;          // device pointer to the block count
    int* counts;              // per global particle (count pass)
    int* counts_s;            // the same by sorted position (the fill reads them in block order)
    int64_t* rsort;           // each particle's row start in its set's output, by sorted position
    int* bdesc;               // [nblk_max][24] per-block descriptors the count pass leaves for the fill
    uint16_t* branks;         // ranks of each block's union by original index (the order of its
                              // candidate bits), a place per block or, with rpool, taken from pools
    int* rpool;               // [kRankPools] entries taken of each pool, zero between counts; or null
    int rpool_cap;            // entries of a pool (a multiple of kRankPiece)
    int* heavy;               // sorted positions of long rows
    int* flags;               // the structure's flags and counters (kFlag*)
    unsigned long long* stats;      // [kStCount] totals
    unsigned long long* blk_stats;  // [nblk_max][5] per-block partial statistics
    uint32_t* cbits;                // accepted-candidate bits, word-major [words][ntot]
    int sparse;                     // 1: the count by small blocks (3D, see kSparseUnion)
    int lr_keys;                    // keys a long-row workgroup sorts in LDS
    int half;                       // 1: rows keep only neighbours of larger original index
    // dense-cell path (wdense == nullptr: off)
    const int* wdense;
    const int* usz;
    const int64_t* uoff;
    const int* ulist;
    const int* unit_off;
    const int* ucell;
    const int* dn;
    unsigned long long* dstats;     // [dgrid][kDenseStats] per-workgroup statistics
    int dgrid;
    // the dense count keeps each target's accepted bits per chunk of kDenseChunk candidates,
    // in candidate order (64 x 16 bits), at dbits[(dboff[cell] + target_in_cell * chunks +
    // chunk) * 64] when dboff[ncell_tot] * 64 <= dbits_cap, and the fill then reads them
    // instead of testing
    const int64_t* dboff;
    uint16_t* dbits;
    int64_t dbits_cap;
};

hipError_t launch_count(const SearchArgs& a, int nblk_max, hipStream_t st);
hipError_t launch_fill(const SearchArgs& a, int nblk_max, hipStream_t st);
hipError_t launch_long_rows(const SearchArgs& a, int grid, hipStream_t st);
// The dense-cell path's passes over its work units.
enum class DensePass { kCount, kFill, kStats };
hipError_t launch_dense(const SearchArgs& a, DensePass pass, hipStream_t st);
// The last count's statistics, summed into a.stats: the count passes decide on the matrix
// cores and tally nothing, so they are made here.
hipError_t launch_stats(const SearchArgs& a, int nblk_max, hipStream_t st);

}  // namespace nnps
