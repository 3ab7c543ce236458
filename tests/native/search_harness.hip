// Launches the count, fill and statistics kernels on arrays that a test makes, so that their behaviour
// on bits, counts, row pointers and coordinates that do not match each other can be tested: the
// library's own passes never leave such arrays. One set, one grid cell of width 1.
#include <cstdint>

#include "build_kernels.h"

extern "C" {

// Device arrays unless a plain number; unused ones may be null.
struct HarnessArgs {
    int32_t dim, mode, n, half;
    int64_t capacity, dbits_cap;
    const double* pos;
    int64_t* row_ptr;
    int32_t* col;
    float* dist;
    unsigned char* set_room;  // room for a SetDesc
    int32_t* offs;            // [2]: 0, n
    int32_t* cell_offs;       // [2]: 0, 1
    uint32_t* skey;
    int32_t *perm, *cell_start;
    double* spos;
    float* rq;  // [n][4]
    int32_t *bstart, *bset, *nblk, *counts, *counts_s;
    int64_t* rsort;
    int32_t* bdesc;
    uint16_t* branks;
    int32_t *heavy, *flags;
    uint32_t* cbits;
    int32_t *wdense, *usz;
    int64_t* uoff;
    int32_t *ulist, *unit_off, *ucell, *dn;
    int64_t* dboff;
    uint16_t* dbits;
    uint64_t *blk_stats, *dstats, *stats;
    int32_t* rpool;
    double radius;
    int32_t t_lo, t_hi, t_mid, nblk_max;  // FP16 thresholds as bits
    int32_t rpool_cap, sparse;
};

int harness_set_bytes() { return static_cast<int>(sizeof(nnps::SetDesc)); }

static hipError_t search_args(const HarnessArgs* h, int dense, nnps::SearchArgs& a)
{
    using namespace nnps;
    SetDesc sd{};
    Frame& fr = sd.fr;
    fr.dim = h->dim;
    fr.mode = h->mode;
    fr.n = h->n;
    fr.F = 40;
    fr.ncell = 1;
    for (int k = 0; k < 3; ++k) {
        fr.nc[k] = 1;
        fr.hi[k] = 1.0;
    }
    fr.w = 1.0;
    fr.s = 0x1p40;
    fr.R2 = h->radius * h->radius;
    fr.xwin = 1;
    fr.inv_quantum = 0x1p30;
    fr.quantum = 0x1p-30f;
    fr.near2 = 3.0f * 0x1p46f;
    fr.t_lo = static_cast<uint16_t>(h->t_lo);
    fr.t_hi = static_cast<uint16_t>(h->t_hi);
    fr.t_mid = static_cast<uint16_t>(h->t_mid);
    fr.t32_mid = static_cast<float>(4.0 * fr.R2);
    sd.pos = h->pos;
    sd.row_ptr = h->row_ptr;
    sd.col = h->col;
    sd.dist = h->dist;
    sd.capacity = h->capacity;
    a = SearchArgs{};
    a.L.dim = h->dim;
    a.L.mode = h->mode;
    a.L.nsets = 1;
    a.L.ntot = h->n;
    a.L.ncell_tot = 1;
    a.L.sets = reinterpret_cast<const SetDesc*>(h->set_room);
    a.L.poffs = h->offs;
    a.L.coffs = h->cell_offs;
    a.L.nrows_tot = 1;
    a.skey = h->skey;
    a.perm = h->perm;
    a.cell_start = h->cell_start;
    a.spos = h->spos;
    a.rq = reinterpret_cast<const float4*>(h->rq);
    a.bstart = h->bstart;
    a.bset = h->bset;
    a.nblk = h->nblk;
    a.counts = h->counts;
    a.counts_s = h->counts_s;
    a.rsort = h->rsort;
    a.bdesc = h->bdesc;
    a.branks = h->branks;
    a.heavy = h->heavy;
    a.flags = h->flags;
    a.cbits = h->cbits;
    a.half = h->half;
    if (dense) {
        a.wdense = h->wdense;
        a.usz = h->usz;
        a.uoff = h->uoff;
        a.ulist = h->ulist;
        a.unit_off = h->unit_off;
        a.ucell = h->ucell;
        a.dn = h->dn;
        a.dgrid = 2;
        a.dboff = h->dboff;
        a.dbits = h->dbits;
        a.dbits_cap = h->dbits_cap;
        a.dstats = reinterpret_cast<unsigned long long*>(h->dstats);
    }
    a.blk_stats = reinterpret_cast<unsigned long long*>(h->blk_stats);
    a.stats = reinterpret_cast<unsigned long long*>(h->stats);
    a.rpool = h->rpool;
    a.rpool_cap = h->rpool_cap;
    a.sparse = h->sparse;
    return hipMemcpy(h->set_room, &sd, sizeof(sd), hipMemcpyHostToDevice);
}

// dense 0: the block fill; 1: the dense fills. Waits for the device; returns a hipError_t.
int harness_fill(const HarnessArgs* h, int dense)
{
    using namespace nnps;
    SearchArgs a;
    hipError_t e = search_args(h, dense, a);
    if (e == hipSuccess) e = dense ? launch_dense(a, DensePass::kFill, nullptr) : launch_fill(a, h->nblk_max, nullptr);
    return e != hipSuccess ? e : hipDeviceSynchronize();
}

// The block count. Waits for the device.
int harness_count(const HarnessArgs* h)
{
    using namespace nnps;
    SearchArgs a;
    hipError_t e = search_args(h, 0, a);
    if (e == hipSuccess) e = launch_count(a, h->nblk_max, nullptr);
    return e != hipSuccess ? e : hipDeviceSynchronize();
}

// The statistics of blocks (and dense cells). Waits for the device.
int harness_stats(const HarnessArgs* h, int dense)
{
    using namespace nnps;
    SearchArgs a;
    hipError_t e = search_args(h, dense, a);
    if (e == hipSuccess) e = launch_stats(a, h->nblk_max, nullptr);
    return e != hipSuccess ? e : hipDeviceSynchronize();
}

}  // extern "C"
