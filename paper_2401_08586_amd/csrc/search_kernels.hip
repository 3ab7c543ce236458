// Neighbour search over the sorted cell structure: the 3^d-cell stencil test (relative
// coordinates, Eq. 6-7 with the factor 1/2 Eq. 7 drops) on the matrix cores, with a binary64
// recheck near the cutoff, the count pass and the fill pass with per-row ascending order and
// wave-cooperative CSR writes; the dense-cell and long-row paths; the statistics.
//
// Work decomposition: a block is up to 64 consecutive sorted targets inside one (y, z) row of
// cells. Cells along x are contiguous in sorted order, so a block's candidates are 3^(d-1)
// contiguous runs ("row segments"), one per (dy, dz): its union.
#include <algorithm>
#include <type_traits>

#include "build_kernels.h"

namespace nnps {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ h2 as_h2(uint32_t u) { return __builtin_bit_cast(h2, u); }
__device__ __forceinline__ uint32_t as_u32(h2 v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ _Float16 as_f16(uint16_t u) { return __builtin_bit_cast(_Float16, u); }
__device__ __forceinline__ h2 splat(_Float16 v) { return h2{v, v}; }

// The binary64 predicate, in the fixed order and with no contraction.
template <int DIM>
__device__ __forceinline__ double r2_fp64(const double* pi, const double* pj)
{
    const double d0 = __dsub_rn(pj[0], pi[0]);
    const double d1 = __dsub_rn(pj[1], pi[1]);
    double r2 = __dmul_rn(d0, d0);
    r2 = __dadd_rn(r2, __dmul_rn(d1, d1));
    if (DIM == 3) {
        const double d2 = __dsub_rn(pj[2], pi[2]);
        r2 = __dadd_rn(r2, __dmul_rn(d2, d2));
    }
    return r2;
}

// The same against the particle at sorted position j.
template <int DIM>
__device__ __forceinline__ bool recheck_sorted(const double* __restrict__ spos, const double* pi, int j, double R2)
{
    return r2_fp64<DIM>(pi, spos + static_cast<size_t>(j) * 4) <= R2;
}

// Square root, within 0.51 units in the last place (the hardware's own is off by up to one, and
// low on average): its reciprocal root (relative error below 2^-22) and one Heron step. For
// normal numbers whose square root's square does not overflow.
__device__ __forceinline__ float root(float s2)
{
    const float r = __builtin_amdgcn_rsqf(s2);
    const float y = s2 * r;
    return __builtin_fmaf(__builtin_fmaf(-y, y, s2), 0.5f * r, y);
}

// FP32 distance from binary64 positions: the displacement in quanta (a power of two, so no
// rounding, and no overflow of the squares), rounded once to FP32 per axis.
template <int DIM>
__device__ __forceinline__ float dist_near(const double* pi, const double* pj, double inv_quantum, float quantum)
{
    float s2 = 0.0f;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        const float f = static_cast<float>((pj[k] - pi[k]) * inv_quantum);
        s2 = __builtin_fmaf(f, f, s2);
    }
    return __fsqrt_rn(s2) * quantum;  // rare: any s2, 0 and infinity among them
}

// A coordinate in quanta (Frame::quantum), the low 32 bits: rounded to an integer in the low
// bits of 1.5 2^52 + x.
__device__ __forceinline__ int in_quanta(double x, double lo, double inv_quantum)
{
    const double q = __dadd_rn(__dmul_rn(__dsub_rn(x, lo), inv_quantum), 0x1.8p52);
    return static_cast<int>(static_cast<uint32_t>(__builtin_bit_cast(uint64_t, q)));
}

// Squared distance in quanta of two positions in quanta, neighbours (fewer than 2^31 apart):
// the difference mod 2^32 is exact, and is rounded once to FP32.
template <int DIM>
__device__ __forceinline__ float quanta2(const int4& i, const int4& j)
{
    auto diff = [](int x, int y) {
        return static_cast<float>(static_cast<int>(static_cast<uint32_t>(x) - static_cast<uint32_t>(y)));
    };
    const float dx = diff(j.x, i.x), dy = diff(j.y, i.y);
    float s2 = __builtin_fmaf(dy, dy, dx * dx);
    if (DIM == 3) {
        const float dz = diff(j.z, i.z);
        s2 = __builtin_fmaf(dz, dz, s2);
    }
    return s2;
}

// The FP32 distance of the FP16 RCLL mode, the same on every path: in quanta, pairs nearer
// than near2 from the binary64 displacement.
template <int DIM>
__device__ __forceinline__ float dist_quanta(const Frame& fr, const double* pi, const double* pj)
{
    auto fixed = [&](const double* x) {
        return make_int4(in_quanta(x[0], fr.lo[0], fr.inv_quantum), in_quanta(x[1], fr.lo[1], fr.inv_quantum),
                         DIM == 3 ? in_quanta(x[2], fr.lo[2], fr.inv_quantum) : 0, 0);
    };
    const float s2 = quanta2<DIM>(fixed(pi), fixed(pj));
    return s2 >= fr.near2 ? root(s2) * fr.quantum  // exact: a power of two
                          : dist_near<DIM>(pi, pj, fr.inv_quantum, fr.quantum);
}

template <int DIM>
__device__ __forceinline__ float dist_fp64(const double* pi, const double* pj)
{
    return static_cast<float>(__dsqrt_rn(r2_fp64<DIM>(pi, pj)));
}

// Data-parallel-primitive step: lane i receives v of the lane that `CTRL` names, or `old`
// where there is none (rows of 16 lanes outside `ROWS` keep `old`).
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ int dpp(int old, int v)
{
    return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xF, false);
}
// Folds v over the wavefront's lanes (all active) in lane order with op and its identity:
// lane i ends with the fold of lanes 0..i, in six steps that use no LDS.
template <typename Op>
__device__ __forceinline__ int wave_fold_i32(int v, int identity, Op&& op)
{
    v = op(v, dpp<0x111>(identity, v));       // row_shr:1
    v = op(v, dpp<0x112>(identity, v));       // row_shr:2
    v = op(v, dpp<0x114>(identity, v));       // row_shr:4
    v = op(v, dpp<0x118>(identity, v));       // row_shr:8
    v = op(v, dpp<0x142, 0xA>(identity, v));  // row_bcast:15 into rows 1 and 3
    v = op(v, dpp<0x143, 0xC>(identity, v));  // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ int wave_excl_scan_i32(int v, int* total)
{
    const int inc = wave_fold_i32(v, 0, [](int x, int y) { return x + y; });
    *total = __builtin_amdgcn_readlane(inc, 63);
    return inc - v;
}

__device__ __forceinline__ int wave_sum_i32(int v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Geometry of one block and of one lane's row segments.
template <int DIM>
struct Geom {
    static constexpr int NSEG = DIM == 3 ? 9 : 3;
    static constexpr int SELF = DIM == 3 ? 4 : 1;  // segment with dy = dz = 0
    int p0, p1, p;
    bool active;
    int x, sx0;
    int U;
    int seg_g0[NSEG], seg_base[NSEG], la[NSEG], lb[NSEG];
    int pself;
    const SetDesc* sd;  // the block's set
    Frame fr;

    __device__ __forceinline__ void init(const SearchArgs& a, int b)
    {
        sd = a.L.sets + a.bset[b];
        fr = sd->fr;
        const uint32_t coff = static_cast<uint32_t>(sd->coff);
        const int* cs = a.cell_start + coff;
        const int lane = threadIdx.x & 63;
        p0 = a.bstart[b];
        p1 = a.bstart[b + 1];
        p = p0 + lane;
        active = p < p1;
        const uint32_t ncx = static_cast<uint32_t>(fr.nc[0]);
        const int ncy = fr.nc[1], ncz = fr.nc[2];
        const uint32_t k0 = a.skey[p0] - coff;
        const uint32_t row0 = k0 / ncx;
        const int xa = static_cast<int>(k0 - row0 * ncx);
        const int y0 = static_cast<int>(row0 % static_cast<uint32_t>(ncy));
        const int z0 = static_cast<int>(row0 / static_cast<uint32_t>(ncy));
        const uint32_t kl = a.skey[p1 - 1] - coff;
        const int xb = static_cast<int>(kl - (kl / ncx) * ncx);
        const uint32_t mk = a.skey[active ? p : p1 - 1] - coff;
        x = static_cast<int>(mk - (mk / ncx) * ncx);
        sx0 = xa > 0 ? xa - 1 : 0;
        const int sx1 = xb + 1 < static_cast<int>(ncx) ? xb + 1 : static_cast<int>(ncx) - 1;
        const int lx0 = x > 0 ? x - 1 : 0;
        const int lx1 = x + 1 < static_cast<int>(ncx) ? x + 1 : static_cast<int>(ncx) - 1;
        U = 0;
#pragma unroll
        for (int r = 0; r < NSEG; ++r) {
            const int dy = r % 3 - 1;
            const int dz = DIM == 3 ? r / 3 - 1 : 0;
            const int yy = y0 + dy, zz = z0 + dz;
            int g0 = 0, g1 = 0, ga = 0, gb = 0;
            if (yy >= 0 && yy < ncy && zz >= 0 && zz < ncz) {
                const int rb = (zz * ncy + yy) * static_cast<int>(ncx);
                g0 = cs[rb + sx0];
                g1 = cs[rb + sx1 + 1];
                ga = cs[rb + lx0];
                gb = cs[rb + lx1 + 1];
            }
            seg_g0[r] = g0;
            seg_base[r] = U;
            la[r] = U + (ga - g0);
            lb[r] = U + (gb - g0);
            U += g1 - g0;
        }
        pself = seg_base[SELF] + (p - seg_g0[SELF]);
    }

    // global sorted index of a logical (staged) position
    __device__ __forceinline__ int global_of(int r, int posl) const { return posl - seg_base[r] + seg_g0[r]; }

    __device__ __forceinline__ int global_of_any(int posl) const
    {
        // static indices only, so the segment tables stay in registers
        int gi = posl - seg_base[0] + seg_g0[0];
#pragma unroll
        for (int k = 1; k < NSEG; ++k)
            if (posl >= seg_base[k]) gi = posl - seg_base[k] + seg_g0[k];
        return gi;
    }
};

// Per-block descriptor the count pass leaves for the fill, so the fill's set-up reads the
// block's geometry with one load instead of re-deriving it through the block table, the
// sorted cell keys and the cell starts: [0] first particle, [1] end, [2] set, [3] union
// size (above the union limit for a block without ranks), [4] 1 for a block of the dense-cell
// path (2: not counted yet), then the NSEG segment first-particle indices and the NSEG segment union offsets, and
// last the place of its ranks in pieces of kRankPiece.
constexpr int kDescInts = kBlockDescInts;
constexpr int kDescRanks = kDescInts - 1;
static_assert(5 + 2 * 9 <= kDescRanks, "the segments of 3D fit");

template <int DIM, typename G>
__device__ __forceinline__ void write_desc(const SearchArgs& a, const G& g, int b, int U, uint32_t ranks, int state = 0)
{
    const int lane = threadIdx.x & 63;
    int v = 0;
    if (lane == 0) v = g.p0;
    if (lane == 1) v = g.p1;
    if (lane == 2) v = a.bset[b];
    if (lane == 3) v = U;
    if (lane == 4) v = state;
    if (lane == kDescRanks) v = static_cast<int>(ranks);
#pragma unroll
    for (int r = 0; r < Geom<DIM>::NSEG; ++r) {
        if (lane == 5 + r) v = g.seg_g0[r];
        if (lane == 5 + Geom<DIM>::NSEG + r) v = g.seg_base[r];
    }
    if (lane < kDescInts) a.bdesc[static_cast<size_t>(b) * kDescInts + lane] = v;
}

// The place of block b's ranks, in pieces: its own, or for U of them from the pools (kNoRanks
// where its pool has no room).
constexpr uint32_t kNoRanks = ~0u;
template <int DIM>
__device__ __forceinline__ uint32_t block_ranks(int b)
{
    constexpr int UCAP = DIM == 3 ? kUnion3 : kUnion2;
    static_assert(UCAP % kRankPiece == 0, "whole pieces");
    return static_cast<uint32_t>(b) * (UCAP / kRankPiece);
}
__device__ __forceinline__ uint32_t take_ranks(const SearchArgs& a, int b, int U)
{
    const int pool = b % kRankPools, need = (U + kRankPiece - 1) / kRankPiece * kRankPiece;
    const int at = atomicAdd(a.rpool + pool * kRankPoolStride, need);
    if (at + need > a.rpool_cap) return kNoRanks;
    return static_cast<uint32_t>((static_cast<int64_t>(pool) * a.rpool_cap + at) / kRankPiece);
}

// A dense-cell block: only its flag is written.
__device__ __forceinline__ void write_desc_dense(const SearchArgs& a, int b)
{
    if ((threadIdx.x & 63) == 4) a.bdesc[static_cast<size_t>(b) * kDescInts + 4] = 1;
}

// The fields of a set a kernel uses in its loops, read once into registers. Read through
// the set table instead, they would be loaded again after every store (the compiler
// cannot tell the stores from the table), each time waiting on memory. The outputs are
// global-address-space pointers, so their stores are plain global stores.
#define NNPS_GLOBAL __attribute__((address_space(1)))
// Memory that no kernel of the launch writes: uniform reads become scalar loads wherever
// they stand.
#define NNPS_CONST __attribute__((address_space(4)))
struct SetView {
    const NNPS_GLOBAL double* pos;
    const NNPS_GLOBAL int64_t* row_ptr;
    NNPS_GLOBAL int32_t* col;
    NNPS_GLOBAL float* dist;
    int64_t capacity;
    int poff;
    __device__ __forceinline__ explicit SetView(const SetDesc& sd)
        : pos((const NNPS_GLOBAL double*)sd.pos),
          row_ptr((const NNPS_GLOBAL int64_t*)sd.row_ptr),
          col((NNPS_GLOBAL int32_t*)sd.col),
          dist((NNPS_GLOBAL float*)sd.dist),
          capacity(sd.capacity),
          poff(sd.poff)
    {
    }
};

// The work block a workgroup takes. Workgroups are dealt to the eight XCDs in turn (the
// i-th to XCD i mod 8), each XCD with its own L2, while neighbouring blocks share most of
// their candidate unions. So XCD k is given the k-th contiguous eighth of the blocks,
// walked in order: block = (i mod 8) * ceil(nblk / 8) + i / 8. Returns -1 for workgroups
// with no block (the grid is sized for an upper bound of the count).
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_block(int nblk)
{
    const int i = blockIdx.x;
    const int per = (nblk + kXcds - 1) / kXcds;
    const int b = (i % kXcds) * per + i / kXcds;
    return (i / kXcds < per && b < nblk) ? b : -1;
}

// Blocks of the dense-cell path's windows are left to that path.
__device__ __forceinline__ bool dense_block(const SearchArgs& a, int b)
{
    return a.wdense && a.wdense[a.skey[a.bstart[b]]];
}

// A particle's FP16 relative coordinates (Eq. 6) from its f32 record: x, y, z, and its cell
// index along x mod 2^10.
__device__ __forceinline__ ushort4 q16_of(const float4& v)
{
    auto h = [](float f) { return __builtin_bit_cast(uint16_t, static_cast<_Float16>(f)); };
    return make_ushort4(h(v.x), h(v.y), h(v.z), static_cast<uint16_t>(__builtin_bit_cast(uint32_t, v.w) & 1023u));
}

// Stage logical positions [cb, ce) as pair records.
template <int DIM>
__device__ __forceinline__ void stage(const SearchArgs& a, const Geom<DIM>& g, int cb, int ce, uint4* srec)
{
    const int lane = threadIdx.x & 63;
    const int m0 = cb >> 1, m1 = (ce + 1) >> 1;
    // a chunk is at most kStage / 128 records per lane: every gather is issued before
    // the first record is built
    constexpr int RPL = kStage / 128;
    ushort4 v[RPL][2];
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
        const int m = m0 + lane + 64 * i;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int posl = 2 * m + h;
            v[i][h] = make_ushort4(0, 0, 0, 0);
            if (m < m1 && posl < ce) {
                const int gi = g.global_of_any(posl);
                v[i][h] = q16_of(a.rq[gi]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
        const int m = m0 + lane + 64 * i;
        if (m >= m1) continue;
        uint32_t w0 = 0, w1 = 0, w2 = 0, w3 = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int posl = 2 * m + h;
            if (posl < ce) {
                // the union spans fewer than 2^10 cells in x
                const int rel = (static_cast<int>(v[i][h].w) - g.sx0) & 1023;
                const _Float16 cx2 = static_cast<_Float16>(2 * rel);
                const uint32_t sh = 16u * h;
                w0 |= static_cast<uint32_t>(v[i][h].x) << sh;
                w1 |= static_cast<uint32_t>(v[i][h].y) << sh;
                w2 |= static_cast<uint32_t>(v[i][h].z) << sh;
                w3 |= static_cast<uint32_t>(__builtin_bit_cast(uint16_t, cx2)) << sh;
            }
        }
        srec[m - m0] = make_uint4(w0, w1, w2, w3);
    }
}

// Per-lane constants of the FP16 test for row segment r.
template <int DIM>
struct Target16 {
    h2 qix, cx2i;
    _Float16 qiy, qiz;
    __device__ __forceinline__ void init(const ushort4& qi, int x, int sx0)
    {
        qix = splat(as_f16(qi.x));
        qiy = as_f16(qi.y);
        qiz = as_f16(qi.z);
        cx2i = splat(static_cast<_Float16>(2 * (x - sx0)));
    }
};

// The packed FP16 r2 for the pair record `rec` (two candidates); ay, az are
// RN16(q_i,y + 2dc_y), RN16(q_i,z + 2dc_z) for the segment.
template <int DIM>
__device__ __forceinline__ uint32_t r2_pair(const Target16<DIM>& t, h2 ay, h2 az, const uint4& rec)
{
    const h2 s = t.qix - as_h2(rec.x);
    const h2 dcx2 = t.cx2i - as_h2(rec.w);
    const h2 tx = s + dcx2;
    const h2 ty = ay - as_h2(rec.y);
    h2 r2;
    if (DIM == 3) {
        const h2 tz = az - as_h2(rec.z);
        r2 = tz * tz;
        r2 = __builtin_elementwise_fma(ty, ty, r2);
    } else {
        r2 = ty * ty;
    }
    r2 = __builtin_elementwise_fma(tx, tx, r2);
    return as_u32(r2);
}

struct Tally {
    unsigned long long cand = 0, band = 0, fpos = 0, fneg = 0, odis = 0;
};

// Tallies one candidate (FP16 bits r2h at union position posl). MODE 0: band pairs against
// the FP64 predicate; MODE 2: every candidate.
template <int DIM, int MODE>
__device__ __forceinline__ void classify(const SearchArgs& a, const Geom<DIM>& g, const double* pi, int posl,
                                         uint32_t r2h, Tally& t)
{
    const Frame& fr = g.fr;
    const bool in16 = r2h < fr.t_lo;
    const bool band = !in16 && r2h <= fr.t_hi;
    if (MODE == 2 || band) {
        const bool truth = recheck_sorted<DIM>(a.spos, pi, g.global_of_any(posl), fr.R2);
        const bool naive = r2h <= fr.t_mid;
        t.band += band;
        t.fpos += naive && !truth;
        t.fneg += !naive && truth;
        if (MODE == 2) t.odis += !band && (in16 != truth);
    }
}

// ---------------------------------------------------------------------------
// Branch-free classification of a pair of FP16 r2 values. Non-negative FP16 bit
// patterns order like unsigned integers, so with d = r2 - T_lo per 16-bit half
// (wrapping): the sign bit of d is set exactly when r2 < T_lo ("in"), and
// sat16(d + 0xFFFE - (T_hi - T_lo)) is 0xFFFF exactly when r2 lies outside
// [T_lo, T_hi] (not in the band). Halves to ignore get r2 bits >= 0x7C00 (+inf),
// which land in neither class.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 as_u16x2(uint32_t u) { return __builtin_bit_cast(u16x2, u); }
__device__ __forceinline__ uint32_t u16x2_bits(u16x2 v) { return __builtin_bit_cast(uint32_t, v); }

struct Thresh {
    u16x2 tlo2, bias2, w12;
    __device__ __forceinline__ void init(const Frame& fr)
    {
        tlo2 = u16x2{fr.t_lo, fr.t_lo};
        const uint16_t b = static_cast<uint16_t>(0xFFFE - (fr.t_hi - fr.t_lo));
        bias2 = u16x2{b, b};
        const uint16_t w1 = static_cast<uint16_t>(fr.t_hi - fr.t_lo + 1);
        w12 = u16x2{w1, w1};
    }
};

// Bits j (j < 8) and 16 + j of x moved to bits 2j and 2j + 1.
__device__ __forceinline__ uint32_t interleave8(uint32_t x)
{
    x &= 0x00FF00FFu;
    x = (x | (x << 4)) & 0x0F0F0F0Fu;
    x = (x | (x << 2)) & 0x33333333u;
    x = (x | (x << 1)) & 0x55555555u;
    return (x & 0xFFFFu) | ((x >> 15) & 0x1FFFEu);
}

// Bits [a, b) of an 8-bit field (a, b clamped to [0, 8]).
__device__ __forceinline__ uint32_t span8(int a, int b)
{
    a = min(max(a, 0), 8);
    b = min(max(b, 0), 8);
    return ((1u << b) - 1u) & ~((1u << a) - 1u);
}

constexpr int kGroup = 8;  // pair records per group in the FP16 count loop

// ---------------------------------------------------------------------------
// Statistics of the last count pass, made when they are asked for (the count pass decides on
// the matrix cores and tallies nothing): one wavefront per block, lane = target, over the
// target's own stencil ranges, from the structure's arrays only. Each writes its block's five
// sums.
template <int DIM>
__device__ __forceinline__ void write_stats(const SearchArgs& a, const Geom<DIM>& g, int b, Tally& t)
{
    if (g.active) {  // candidates: the lane's ranges minus itself
        int total = 0;
#pragma unroll
        for (int r = 0; r < Geom<DIM>::NSEG; ++r) total += g.lb[r] - g.la[r];
        t.cand += total - 1;
    }
    unsigned long long v[5] = {t.cand, t.band, t.fpos, t.fneg, t.odis};
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const unsigned long long sum = wave_sum_u64(v[k]);
        if ((threadIdx.x & 63) == 0) a.blk_stats[static_cast<size_t>(b) * 5 + k] = sum;
    }
}

// The block of a statistics kernel, or -1 (no block, or one of the dense-cell path, whose
// sums are cleared).
__device__ __forceinline__ int stats_block(const SearchArgs& a)
{
    const int b = xcd_block(*a.nblk);
    if (b < 0 || !dense_block(a, b)) return b;
    if ((threadIdx.x & 63) < 5) a.blk_stats[static_cast<size_t>(b) * 5 + (threadIdx.x & 63)] = 0;
    return -1;
}

// The packed-FP16 test (MODE 0: band pairs against the FP64 predicate; MODE 2, recheck-all:
// every candidate).
template <int DIM, int MODE>
__global__ void __launch_bounds__(64)
k_stats16(SearchArgs a)
{
    // pair records of the staged chunk, and kGroup more that the last group of a range may
    // read past the chunk (their bits are masked)
    __shared__ uint4 srec[kStage / 2 + kGroup];
    const int b = stats_block(a);
    if (b < 0) return;
    Geom<DIM> g;
    g.init(a, b);
    const int pp = g.active ? g.p : g.p1 - 1;
    double pi[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < DIM; ++k) pi[k] = a.spos[static_cast<size_t>(pp) * 4 + k];
    Target16<DIM> tg;
    tg.init(q16_of(a.rq[pp]), g.x, g.sx0);
    Thresh th;
    th.init(g.fr);
    Tally t;
    for (int cb = 0; cb < g.U; cb += kStage) {
        const int ce = min(g.U, cb + kStage);
        __syncthreads();
        stage<DIM>(a, g, cb, ce, srec);
        __syncthreads();
        if (!g.active) continue;
        const uint4* rec = srec - (cb >> 1);
#pragma unroll
        for (int r = 0; r < Geom<DIM>::NSEG; ++r) {
            const int lo = max(g.la[r], cb), hi = min(g.lb[r], ce);
            if (lo >= hi) continue;
            const int dy = r % 3 - 1, dz = DIM == 3 ? r / 3 - 1 : 0;
            const h2 ay = splat(tg.qiy + static_cast<_Float16>(-2 * dy));
            const h2 az = splat(tg.qiz + static_cast<_Float16>(-2 * dz));
            // kGroup pair records (2 kGroup positions) at a time: bit j for position
            // 2(mg + j), bit 16 + j for position 2(mg + j) + 1
            const int m0 = lo >> 1, mend = (hi + 1) >> 1;
            for (int mg = m0; mg < mend; mg += kGroup) {
                uint32_t acc = 0, ebits = 0;
                if (MODE == 0) {
#pragma unroll
                    for (int j = 0; j < kGroup; ++j) {
                        const uint32_t rb = r2_pair<DIM>(tg, ay, az, rec[mg + j]);
                        const u16x2 d = as_u16x2(rb) - th.tlo2;
                        const u16x2 e = d - th.w12;
                        acc |= (u16x2_bits(d) >> (15 - j)) & (0x10001u << j);
                        ebits |= (u16x2_bits(e) >> (15 - j)) & (0x10001u << j);
                    }
                }
                // the group's positions inside [lo, hi)
                const int a0 = lo - 2 * mg, b0 = hi - 2 * mg;
                const uint32_t valid = span8((a0 + 1) >> 1, (b0 + 1) >> 1) | (span8(a0 >> 1, b0 >> 1) << 16);
                for (uint32_t q = MODE == 0 ? ebits & ~acc & valid : valid; q; q &= q - 1u) {
                    const int k = __builtin_ctz(q);
                    const int posl = 2 * (mg + (k & 15)) + (k >> 4);
                    if (posl == g.pself) continue;
                    const uint32_t rb = r2_pair<DIM>(tg, ay, az, rec[posl >> 1]);
                    classify<DIM, MODE>(a, g, pi, posl, (rb >> (16 * (posl & 1))) & 0xFFFFu, t);
                }
            }
        }
    }
    write_stats<DIM>(a, g, b, t);
}

// FP32 r2 of Eq. 7 on twice the displacement in cell widths: per axis
// t = (q_i - q_j) + 2 dc, then the squares summed left to right, every operation rounded
// once to f32 (no contraction). 2 dc_x = w_i - w_j, where w is twice the cell's x offset
// from the block's first stencil cell (small integers: exact); 2 dc_y and 2 dc_z are the
// row segment's constants.
template <int DIM>
__device__ __forceinline__ float r2_fp32(const float4& qi, float wi, float cy, float cz, const float4& s)
{
#pragma clang fp contract(off)
    const float tx = (qi.x - s.x) + (wi - s.w);
    const float ty = (qi.y - s.y) + cy;
    float r2 = tx * tx + ty * ty;
    if (DIM == 3) {
        const float tz = (qi.z - s.z) + cz;
        r2 = r2 + tz * tz;
    }
    return r2;
}

// The FP32 test of the relative coordinates (the paper's FP32 variant), band pairs against
// the FP64 predicate.
template <int DIM>
__global__ void __launch_bounds__(64)
k_stats32(SearchArgs a)
{
    const int b = stats_block(a);
    if (b < 0) return;
    Geom<DIM> g;
    g.init(a, b);
    const int pp = g.active ? g.p : g.p1 - 1;
    const double* pi = a.spos + static_cast<size_t>(pp) * 4;
    const float4 qi = a.rq[pp];
    const float wi = static_cast<float>(2 * (g.x - g.sx0));
    Tally t;
    if (g.active) {
#pragma unroll
        for (int r = 0; r < Geom<DIM>::NSEG; ++r) {
            const float cy = static_cast<float>(2 - 2 * (r % 3));                 // -2 dy
            const float cz = DIM == 3 ? static_cast<float>(2 - 2 * (r / 3)) : 0.0f;  // -2 dz
            for (int posl = g.la[r]; posl < g.lb[r]; ++posl) {
                const int gj = g.global_of(r, posl);
                float4 v = a.rq[gj];
                // the union spans fewer than 2^10 cells in x, so the offset mod 2^10 is exact
                v.w = static_cast<float>(2 * ((__builtin_bit_cast(int, v.w) - g.sx0) & 1023));
                const float r2 = r2_fp32<DIM>(qi, wi, cy, cz, v);
                if (posl == g.pself || r2 < g.fr.t32_lo || !(r2 <= g.fr.t32_hi)) continue;
                const bool truth = recheck_sorted<DIM>(a.spos, pi, gj, g.fr.R2);
                const bool naive = r2 <= g.fr.t32_mid;
                t.band++;
                t.fpos += naive && !truth;
                t.fneg += !naive && truth;
            }
        }
    }
    write_stats<DIM>(a, g, b, t);
}

// FP64: the candidates only.
template <int DIM>
__global__ void __launch_bounds__(64)
k_stats64(SearchArgs a)
{
    const int b = stats_block(a);
    if (b < 0) return;
    Geom<DIM> g;
    g.init(a, b);
    Tally t;
    write_stats<DIM>(a, g, b, t);
}

// Sum of the per-block statistics and of the dense path's per-workgroup statistics
// (one workgroup; no contended atomics).
__global__ void __launch_bounds__(1024)
k_reduce_stats(const unsigned long long* __restrict__ blk, const int* __restrict__ nblk,
               const unsigned long long* __restrict__ dst, int ndst, unsigned long long* __restrict__ out)
{
    __shared__ unsigned long long sh[16][kDenseStats];
    const int nb = *nblk;
    unsigned long long acc[kDenseStats] = {0, 0, 0, 0, 0, 0};
    for (int b = threadIdx.x; b < nb; b += blockDim.x)
#pragma unroll
        for (int k = 0; k < 5; ++k) acc[k] += blk[static_cast<size_t>(b) * 5 + k];
    for (int w = threadIdx.x; w < ndst; w += blockDim.x)
#pragma unroll
        for (int k = 0; k < kDenseStats; ++k) acc[k] += dst[static_cast<size_t>(w) * kDenseStats + k];
#pragma unroll
    for (int k = 0; k < kDenseStats; ++k) {
        const unsigned long long s = wave_sum_u64(acc[k]);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][k] = s;
    }
    __syncthreads();
    if (threadIdx.x < kDenseStats) {
        unsigned long long s = 0;
        for (int w = 0; w < static_cast<int>(blockDim.x >> 6); ++w) s += sh[w][threadIdx.x];
        // slots 0..4 as in StatSlot; the sixth (rows of the dense path) goes to kStDenseRows
        out[threadIdx.x < 5 ? threadIdx.x : kStDenseRows] = s;
    }
}

// ---------------------------------------------------------------------------
// Limits of the block path: candidates of a block's union.
template <int DIM>
struct FillCfg {
    static constexpr int UCAP = DIM == 3 ? kUnion3 : kUnion2;
    static constexpr int MW = UCAP / 32;    // mask words per lane
    static constexpr int FLAT = DIM == 3 ? 1024 : 512;  // entries a wavefront of the fill compacts at a time
    static constexpr int SHIFT = DIM == 3 ? 10 : 9;  // log2(UCAP)
};

// Bitonic sort of 64*EPL keys held blocked across the wavefront (element e = lane*EPL + i).
template <int EPL>
__device__ __forceinline__ void wave_bitonic(uint32_t (&v)[EPL])
{
    const int lane = threadIdx.x & 63;
    constexpr int P = 64 * EPL;
#pragma unroll
    for (int k = 2; k <= P; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
            if (j >= EPL) {
                const int lx = j / EPL;
                const bool lower = (lane & lx) == 0;
                const bool asc = ((lane * EPL) & k) == 0;
#pragma unroll
                for (int i = 0; i < EPL; ++i) {
                    const uint32_t w = static_cast<uint32_t>(__shfl_xor(static_cast<int>(v[i]), lx, 64));
                    const uint32_t mn = min(v[i], w), mx = max(v[i], w);
                    v[i] = (lower == asc) ? mn : mx;
                }
            } else {
#pragma unroll
                for (int i = 0; i < EPL; ++i) {
                    if (i & j) continue;
                    const bool asc = ((lane * EPL + i) & k) == 0;
                    const uint32_t x = v[i], y = v[i | j];
                    const uint32_t mn = min(x, y), mx = max(x, y);
                    v[i] = asc ? mn : mx;
                    v[i | j] = asc ? mx : mn;
                }
            }
        }
    }
}

// One wavefront sorts n <= 64 EPL column indices of a row in place (registers, element
// e = lane EPL + i; padding sorts last and is not written back).
template <int EPL>
__device__ __forceinline__ void wave_sort_row(NNPS_GLOBAL int32_t* col, int n)
{
    const int lane = threadIdx.x & 63;
    uint32_t v[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        const int e = lane * EPL + i;
        v[i] = e < n ? static_cast<uint32_t>(col[e]) : 0xFFFFFFFFu;
    }
    wave_bitonic<EPL>(v);
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        const int e = lane * EPL + i;
        if (e < n) col[e] = static_cast<int32_t>(v[i]);
    }
}

// Number of keys below `key` in a sorted run of P keys (P a power of two, the run padded
// with all-ones keys): fixed-step binary lifting, every read inside the run.
template <int P>
__device__ __forceinline__ int count_below(const uint32_t* run, uint32_t key)
{
    int c = 0;
#pragma unroll
    for (int s = P >> 1; s > 0; s >>= 1) c += run[c + s - 1] < key ? s : 0;
    return c + (run[c] < key ? 1 : 0);
}

// Ranks of the U union keys (key_of(e), e < U) across NW wavefronts: wavefront wv sorts
// keys [wv Q, wv Q + Q) in registers and stores them padded to 64 EPL entries; a key's
// rank is the number of keys below it in the NW sorted quarters. rk[i] receives the rank of
// element tid + i 64 NW. Keys that carry their position (packed) are ranked straight from
// the registers of whichever thread sorted them and handed over through rank_of; otherwise
// every thread looks its own elements' keys up in all quarters.
template <int UCAP, int SHIFT, int NW, int EPL, typename K>
__device__ __forceinline__ void rank_union(int U, int Q, bool packed, K&& key_of, uint32_t* skeys, uint16_t* rank_of,
                                           int (&out)[UCAP / (64 * NW)])
{
    constexpr int EPT = UCAP / (64 * NW);
    constexpr int QP = 64 * EPL;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int e0 = wv * Q, n = max(0, min(Q, U - e0));
    uint32_t v[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        const int k = lane * EPL + i;
        v[i] = k < n ? key_of(e0 + k) : 0xFFFFFFFFu;
    }
    wave_bitonic<EPL>(v);
#pragma unroll
    for (int i = 0; i < EPL; ++i) skeys[wv * QP + lane * EPL + i] = v[i];
    __syncthreads();
    if (packed) {
        int rk[EPL];
#pragma unroll
        for (int i = 0; i < EPL; ++i) rk[i] = lane * EPL + i;
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            if (q == wv) continue;
#pragma unroll
            for (int i = 0; i < EPL; ++i) rk[i] += count_below<QP>(skeys + q * QP, v[i]);
        }
#pragma unroll
        for (int i = 0; i < EPL; ++i)
            if (v[i] != 0xFFFFFFFFu) rank_of[v[i] & (UCAP - 1)] = static_cast<uint16_t>(rk[i]);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < EPT; ++i) out[i] = tid + i * 64 * NW < U ? rank_of[tid + i * 64 * NW] : 0;
    } else {
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            const int e = tid + i * 64 * NW;
            if (e < U) {
                const uint32_t key = key_of(e);
                int r = 0;
#pragma unroll
                for (int q = 0; q < NW; ++q) r += count_below<QP>(skeys + q * QP, key);
                out[i] = r;
            }
        }
    }
}

// Ranks by bitmap, for unions whose original indices span at most 32 BW values (the
// common case when particles are numbered in space): one bit per index in [omin, omin +
// range), an exclusive scan of the word popcounts, and a key's rank is the number of set
// bits below it. og[i] is the original index of element tid + i 64 NW (below U), rk[i] its
// rank. bw (BW words) and pc (BW 16-bit prefixes) are scratch.
template <int UCAP, int NW, int BW>
__device__ __forceinline__ void rank_bitmap(int U, int omin, int range, const int (&og)[UCAP / (64 * NW)], uint32_t* bw,
                                            uint16_t* pc, int* wsum, int (&rk)[UCAP / (64 * NW)])
{
    constexpr int NT = 64 * NW;
    constexpr int EPT = UCAP / NT;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int W = (range + 31) >> 5;
    for (int w = tid; w < W; w += NT) bw[w] = 0u;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
        const int e = tid + i * NT;
        if (e < U) {
            const int o = og[i] - omin;
            atomicOr(&bw[o >> 5], 1u << (o & 31));
        }
    }
    __syncthreads();
    // thread t takes words [t per, t per + per): their popcounts, scanned across the block
    const int per = (W + NT - 1) / NT;
    const int w0 = min(W, tid * per), w1 = min(W, w0 + per);
    int cnt = 0;
    for (int w = w0; w < w1; ++w) cnt += __builtin_popcount(bw[w]);
    int wtot;
    const int ex = wave_excl_scan_i32(cnt, &wtot);
    if (lane == 0) wsum[wv] = wtot;
    __syncthreads();
    int run = ex;
    for (int q = 0; q < wv; ++q) run += wsum[q];
    for (int w = w0; w < w1; ++w) {
        pc[w] = static_cast<uint16_t>(run);
        run += __builtin_popcount(bw[w]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
        const int e = tid + i * NT;
        if (e < U) {
            const int o = og[i] - omin;
            const int w = o >> 5;
            rk[i] = pc[w] + __builtin_popcount(bw[w] & ((1u << (o & 31)) - 1u));
        }
    }
}

// Ranks by a two-level bitmap, for unions whose original indices span fewer than 2^17
// values but too many for one bit per index (3D lattices numbered row by row: a union
// covers a few planes of indices, sparsely). Level 1 marks which 32-index chunks of
// [omin, omin + 2^17) hold a union index (4096 bits); the occupied chunks are numbered in
// order by a scan of the level-1 word popcounts; level 2 keeps one 32-bit word of index
// bits per occupied chunk; a key's rank is the set level-2 bits before it (a block scan of
// the level-2 word popcounts, plus the bits below it in its own word). Input and output as
// rank_bitmap. l1 (128 words), l1pre (128), l2 (UCAP words) and l2pre (UCAP) are scratch.
template <int UCAP, int NW>
__device__ __forceinline__ void rank_bitmap2(int U, int omin, const int (&og)[UCAP / (64 * NW)], uint32_t* l1,
                                             uint16_t* l1pre, uint32_t* l2, uint16_t* l2pre, int* wsum,
                                             int (&rk)[UCAP / (64 * NW)])
{
    constexpr int NT = 64 * NW;
    constexpr int EPT = UCAP / NT;
    static_assert(NT >= 128 && UCAP % NT == 0, "the level-1 words fit one pass of the block");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (tid < 128) l1[tid] = 0u;
#pragma unroll
    for (int i = 0; i < EPT; ++i) l2[tid * EPT + i] = 0u;
    __syncthreads();
    int ch[EPT];
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
        const int e = tid + i * NT;
        ch[i] = e < U ? (og[i] - omin) >> 5 : 0;
        if (e < U) atomicOr(&l1[ch[i] >> 5], 1u << (ch[i] & 31));
    }
    __syncthreads();
    // number the occupied chunks: exclusive scan of the 128 level-1 popcounts (waves 0, 1)
    {
        const int c = tid < 128 ? __builtin_popcount(l1[tid]) : 0;
        int tot;
        const int ex = wave_excl_scan_i32(c, &tot);
        if (lane == 0 && wv < 2) wsum[wv] = tot;
        __syncthreads();
        if (tid < 128) l1pre[tid] = static_cast<uint16_t>(ex + (wv == 1 ? wsum[0] : 0));
    }
    __syncthreads();
    int slot[EPT];
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
        const int e = tid + i * NT;
        const int w1 = ch[i] >> 5;
        slot[i] = l1pre[w1] + __builtin_popcount(l1[w1] & ((1u << (ch[i] & 31)) - 1u));
        if (e < U) atomicOr(&l2[slot[i]], 1u << ((og[i] - omin) & 31));
    }
    __syncthreads();
    // exclusive scan of the level-2 popcounts: thread t takes slots [t EPT, t EPT + EPT)
    {
        int c[EPT], sum = 0;
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            c[i] = __builtin_popcount(l2[tid * EPT + i]);
            sum += c[i];
        }
        int tot;
        int run = wave_excl_scan_i32(sum, &tot);
        if (lane == 0) wsum[wv] = tot;
        __syncthreads();
        for (int q = 0; q < wv; ++q) run += wsum[q];
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            l2pre[tid * EPT + i] = static_cast<uint16_t>(run);
            run += c[i];
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
        const int e = tid + i * NT;
        if (e < U)
            rk[i] = l2pre[slot[i]] + __builtin_popcount(l2[slot[i]] & ((1u << ((og[i] - omin) & 31)) - 1u));
    }
}

__device__ __forceinline__ int wave_min_i32(int v)
{
    return __builtin_amdgcn_readlane(wave_fold_i32(v, 0x7FFFFFFF, [](int x, int y) { return min(x, y); }), 63);
}

__device__ __forceinline__ int wave_max_i32(int v)
{
    return __builtin_amdgcn_readlane(wave_fold_i32(v, -0x7FFFFFFF - 1, [](int x, int y) { return max(x, y); }), 63);
}

// Scratch of rank_originals (bytes): the two-level bitmap's tables (level 1 and its prefixes
// 768, level 2 and its prefixes 6 UCAP), or the sorted quarters and the keys (8 UCAP).
template <int UCAP>
constexpr int kRankScratch = 8 * UCAP > 6 * UCAP + 768 ? 8 * UCAP : 6 * UCAP + 768;

// The rank rk[i] of union element tid + i 64 NW (below U) by original index, og[i] its index.
// Unions spanning few indices are ranked by a bitmap, up to 2^17 by a two-level bitmap, the
// others (an unordered numbering) by sorting: keys (orig - omin) << SHIFT | position when the
// range allows, else the original index itself, distinct either way and below the all-ones key
// that pads the sorted quarters.
// rank_of (UCAP entries) is scratch too; both are free again on return.
template <int UCAP, int SHIFT, int NW>
__device__ __forceinline__ void rank_originals(int U, const int (&og)[UCAP / (64 * NW)], unsigned char* scratch,
                                               int (*sred)[NW], int* wsum, uint16_t* rank_of,
                                               int (&rk)[UCAP / (64 * NW)])
{
    constexpr int NT = 64 * NW, EPT = UCAP / NT;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int omin = 0x7FFFFFFF, omax = 0;
#pragma unroll
    for (int i = 0; i < EPT; ++i)
        if (tid + i * NT < U) {
            omin = min(omin, og[i]);
            omax = max(omax, og[i]);
        }
    omin = wave_min_i32(omin);
    omax = wave_max_i32(omax);
    if (lane == 0) {
        sred[0][wv] = omin;
        sred[1][wv] = omax;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        omin = min(omin, sred[0][w]);
        omax = max(omax, sred[1][w]);
    }
    constexpr int BW = kRankScratch<UCAP> / 6;
    uint32_t* s32 = reinterpret_cast<uint32_t*>(scratch);
    if (static_cast<unsigned>(omax - omin) < 32u * BW) {
        rank_bitmap<UCAP, NW, BW>(U, omin, omax - omin + 1, og, s32, reinterpret_cast<uint16_t*>(s32 + BW), wsum, rk);
    } else if (static_cast<unsigned>(omax - omin) < (1u << 17)) {
        rank_bitmap2<UCAP, NW>(U, omin, og, s32, reinterpret_cast<uint16_t*>(s32 + 128), s32 + 192,
                               reinterpret_cast<uint16_t*>(s32 + 192 + UCAP), wsum, rk);
    } else {
        const bool packed = static_cast<uint32_t>(omax - omin) < (1u << (32 - SHIFT)) - 1u;
        uint32_t* keys = s32 + UCAP;
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            const int e = tid + i * NT;
            if (e < U)
                keys[e] = packed ? (static_cast<uint32_t>(og[i] - omin) << SHIFT) | static_cast<uint32_t>(e)
                                 : static_cast<uint32_t>(og[i]);
        }
        __syncthreads();
        auto key_of = [&](int e) { return keys[e]; };
        const int Q = (U + NW - 1) / NW;
        if (Q <= 64) rank_union<UCAP, SHIFT, NW, 1>(U, Q, packed, key_of, s32, rank_of, rk);
        else if (UCAP / NW <= 128 || Q <= 128) rank_union<UCAP, SHIFT, NW, 2>(U, Q, packed, key_of, s32, rank_of, rk);
        else rank_union<UCAP, SHIFT, NW, UCAP / NW <= 128 ? 2 : 4>(U, Q, packed, key_of, s32, rank_of, rk);
    }
    __syncthreads();
}

// The same by one wavefront, for up to 256 candidates: og[i] is element lane + 64 i. Sorted in
// registers with the position in the key where the index range allows (24 bits), else the indices
// alone and looked up. scratch: 256 words.
template <int EPL>
__device__ __forceinline__ void rank_wave_of(int U, const int (&og)[4], int omin, bool packed, uint32_t* scratch,
                                             uint16_t* rank_of, int (&rk)[4])
{
    const int lane = threadIdx.x & 63;
    uint32_t v[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        const int e = lane + 64 * i;
        const uint32_t key = packed ? (static_cast<uint32_t>(og[i] - omin) << 8) | static_cast<uint32_t>(e)
                                    : static_cast<uint32_t>(og[i]);
        v[i] = e < U ? key : 0xFFFFFFFFu;
    }
    wave_bitonic<EPL>(v);
    if (packed) {
#pragma unroll
        for (int i = 0; i < EPL; ++i)
            if (v[i] != 0xFFFFFFFFu) rank_of[v[i] & 255u] = static_cast<uint16_t>(lane * EPL + i);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < EPL; ++i) rk[i] = lane + 64 * i < U ? rank_of[lane + 64 * i] : 0;
    } else {
#pragma unroll
        for (int i = 0; i < EPL; ++i) scratch[lane * EPL + i] = v[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < EPL; ++i) rk[i] = count_below<64 * EPL>(scratch, static_cast<uint32_t>(og[i]));
    }
}

template <int UC>
__device__ __forceinline__ void rank_wave(int U, const int (&og)[UC / 64], uint32_t* scratch, uint16_t* rank_of,
                                          int (&rk)[UC / 64])
{
    static_assert(UC == 256, "positions take 8 bits of a key");
    const int lane = threadIdx.x & 63;
    int omin = 0x7FFFFFFF, omax = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (lane + 64 * i < U) {
            omin = min(omin, og[i]);
            omax = max(omax, og[i]);
        }
    omin = wave_min_i32(omin);
    omax = wave_max_i32(omax);
    const bool packed = omax - omin < (1 << 24) - 1;
    if (U <= 64) rank_wave_of<1>(U, og, omin, packed, scratch, rank_of, rk);
    else if (U <= 128) rank_wave_of<2>(U, og, omin, packed, scratch, rank_of, rk);
    else rank_wave_of<4>(U, og, omin, packed, scratch, rank_of, rk);
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Count pass, on the matrix cores. Four wavefronts per block: the block's union is ranked by
// original index first, so the candidate bits come out in row order and the fill only has to
// compact them.
//
// The test is the contraction r2 = |c|^2 - 2 c.t + |t|^2 over candidates c and targets t
// about the block's centre, with the cutoff on the target side (|t|^2 - R^2), so the result D
// is negative for "in"; |D| below an error bound is decided by the binary64 predicate.
//   P = 16 (FP16 RCLL): coordinates in half cell widths (Eq. 6 plus twice the cell offset),
//     each and the squares split into two FP16 parts, the dominant products of which take
//     the 16 slots of one 32x32x16 FP16 MFMA with FP32 sums: 1024 pairs per 8 passes.
//   P = 32 (FP32 RCLL): the same coordinates in FP32, three 32x32x2 FP32 MFMAs.
//   P = 64: binary64 positions less the first target's, one 16x16x4 FP64 MFMA per 256 pairs
//     with |t|^2 - R^2 as its accumulator.
// One funnel shift per 64 pairs moves D's sign bits into a lane's row bits (lane = target;
// candidates are dealt to operand rows so that a lane's 16 results are consecutive ranks),
// and half a three-way minimum watches |D|.
//
// Error of D against M, the sum of the magnitudes of its terms, M <= 2 (|c|^2 + |t|^2) + R^2,
// bounded from the block's x-span: the products are exact (P = 16) or rounded once, the sum
// of at most 16 errs by 2^-19 M (P = 16 and 32; any order, truncating; 2^-21.9 M measured
// for the FP16 instruction) and 2^-49 M (P = 64), the FP16 splits by 2^-21 M, the
// coordinates by 2^-22 M (2^-51 M). The bounds taken are 2^-18 M and 2^-46 M. The instructions'
// order and rounding of a sum are assumed, not documented: recheck-all compares every decision
// outside the FP16 bound with binary64 (k_check_tiles; of 2.2e9 candidates of lattices, uniform,
// sparse and clustered sets in 2D and 3D none was wrong), the equal lists of the tests check all
// three.
//
// What bounds it: VALU issue, about half of it the ranking. At 1M particles in 3D (64 targets
// against 870 candidates per block, 28 tiles) packed-FP16 tests of each target's own 348
// candidates, with bits in union order, took 251 us per launch, this 162; FP64 486 -> 280 us.
// (Skipping the rounds of a thread's candidates that lie past a small union spoils the loads
// that are issued together: 53 us in 2D either way, the 3D step 437 instead of 414.)
// Wavefronts per block: in 2D a union has a few hundred candidates and the work that every
// wavefront repeats (geometry, target operands) weighs more.
template <int DIM>
constexpr int kCountThreads = DIM == 3 ? 256 : 128;
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Geometry of a block, the same in every lane (scalar registers).
template <int DIM>
struct BlockGeom {
    static constexpr int NSEG = Geom<DIM>::NSEG;
    static constexpr int SELF = Geom<DIM>::SELF;
    int p0, p1, U, xa, xb, y0, z0;  // xa, xb: the targets' first and last cell along x
    int seg_g0[NSEG], seg_base[NSEG];
    const SetDesc* sd;
    __device__ __forceinline__ void init(const SearchArgs& a, int b)
    {
        auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
        sd = a.L.sets + uni(a.bset[b]);
        const int coff = sd->coff;
        const int* cs = a.cell_start + coff;
        p0 = uni(a.bstart[b]);
        p1 = uni(a.bstart[b + 1]);
        const uint32_t ncx = static_cast<uint32_t>(sd->fr.nc[0]);
        const int ncy = sd->fr.nc[1], ncz = sd->fr.nc[2];
        const uint32_t k0 = static_cast<uint32_t>(uni(static_cast<int>(a.skey[p0])) - coff);
        const uint32_t k1 = static_cast<uint32_t>(uni(static_cast<int>(a.skey[p1 - 1])) - coff);
        const uint32_t row0 = k0 / ncx;
        xa = static_cast<int>(k0 - row0 * ncx);
        xb = static_cast<int>(k1 - row0 * ncx);  // the block lies in one row of cells
        y0 = static_cast<int>(row0 % static_cast<uint32_t>(ncy));
        z0 = static_cast<int>(row0 / static_cast<uint32_t>(ncy));
        const int sx0 = max(xa - 1, 0), sx1 = min(xb + 1, static_cast<int>(ncx) - 1);
        U = 0;
#pragma unroll
        for (int r = 0; r < NSEG; ++r) {
            const int yy = y0 + r % 3 - 1, zz = DIM == 3 ? z0 + r / 3 - 1 : 0;
            const bool in = yy >= 0 && yy < ncy && zz >= 0 && zz < ncz;
            const int rb = in ? (zz * ncy + yy) * static_cast<int>(ncx) : 0;
            const int g0 = uni(cs[rb + sx0]), g1 = uni(cs[rb + sx1 + 1]);
            seg_g0[r] = in ? g0 : 0;
            seg_base[r] = U;
            U += in ? g1 - g0 : 0;
        }
    }
    __device__ __forceinline__ int global_of_any(int posl) const
    {
        int delta = seg_g0[0] - seg_base[0];
#pragma unroll
        for (int k = 1; k < NSEG; ++k)
            if (posl >= seg_base[k]) delta = seg_g0[k] - seg_base[k];
        return posl + delta;
    }
};

// The FP16 parts v = h + l + (a residual of 2^-22 |v|), and two halves in a word.
struct Split16 {
    _Float16 h, l;
    __device__ __forceinline__ explicit Split16(float v)
        : h(static_cast<_Float16>(v)), l(static_cast<_Float16>(v - static_cast<float>(h)))
    {
    }
};
__device__ __forceinline__ uint32_t halves(_Float16 lo, _Float16 hi) { return as_u32(h2{lo, hi}); }

// MFMA operands of one item per lane: words 0-3 hold slots 0-7, words 4-7 slots 8-15.
// Candidates: xh xh xl xl yh yh yl zh | zh zl s0 s1 0 1 1 1, with s the squared norm;
// targets (x = -2 x and so on): xh xl xh xl yh yl yh zh | zl zh 1 1 1 u0 u1 0, with u the
// squared norm less 4 rho^2.
__device__ __forceinline__ void candidate_words(float x, float y, float z, uint32_t (&w)[8])
{
    const Split16 X(x), Y(y), Z(z), S(x * x + y * y + z * z);
    w[0] = halves(X.h, X.h);
    w[1] = halves(X.l, X.l);
    w[2] = halves(Y.h, Y.h);
    w[3] = halves(Y.l, Z.h);
    w[4] = halves(Z.h, Z.l);
    w[5] = halves(S.h, S.l);
    w[6] = 0x3C000000u;
    w[7] = 0x3C003C00u;
}
__device__ __forceinline__ void target_words(float x, float y, float z, float rho4, uint32_t (&w)[8])
{
    const Split16 X(-2.0f * x), Y(-2.0f * y), Z(-2.0f * z), Uu(x * x + y * y + z * z - rho4);
    w[0] = halves(X.h, X.l);
    w[1] = w[0];
    w[2] = halves(Y.h, Y.l);
    w[3] = halves(Y.h, Z.h);
    w[4] = halves(Z.l, Z.h);
    w[5] = 0x3C003C00u;
    w[6] = halves(static_cast<_Float16>(1.0f), Uu.h);
    w[7] = halves(Uu.l, static_cast<_Float16>(0.0f));
}
// 4x4 transposes over the wavefront's quarters: out[i] of quarter q = in[q] of quarter i.
__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b)
{
    const u32x2 v = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = v[0];
    b = v[1];
}
__device__ __forceinline__ void swap16(uint32_t& a, uint32_t& b)
{
    const u32x2 v = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = v[0];
    b = v[1];
}
__device__ __forceinline__ void quarter_transpose(uint32_t (&v)[4])
{
    swap32(v[0], v[2]);
    swap32(v[1], v[3]);
    swap16(v[0], v[1]);
    swap16(v[2], v[3]);
}

// The lowest n bits of a word.
__device__ __forceinline__ uint32_t first_bits(int n)
{
    return n >= 32 ? ~0u : (n <= 0 ? 0u : (1u << n) - 1u);
}

// The MFMA operands of 64 items, one prepared per lane, and 64 x 64 tests. prepare: the
// fragments of 64 candidates (lane l prepares candidate item(l); `past`: none, so far away that
// every result is out, or, where the bound sends all results to decide, decided there as out);
// words: the two row words (candidates 0-31 and 32-63 of the step) of target `lane`, with
// `decide(bnd, acc, e, t)` settling the results bnd (bits) of a lane whose 16 results are the
// step's candidates e.. against target t.
template <int DIM, int P>
struct Tiles;

// P = 16: words 0-3 of an item hold slots 0-7, words 4-7 slots 8-15; an operand lane l holds
// item l mod 32, slots 8 (l / 32) onwards. Operand row rho = 8 (r / 4) + 4 h + r mod 4 gives
// result r of the lanes 32 h ..., and holds candidate 16 h + r.
template <int DIM>
struct Tiles<DIM, 16> {
    using Rec = float4;  // a union record in LDS
    struct Coord { float x, y, z; };
    h8 t0, t1;
    float beta;
    static __device__ __forceinline__ int item(int lane)
    {
        return 16 * ((lane >> 2) & 1) + 4 * ((lane >> 3) & 3) + (lane & 3) + (lane & 32);
    }
    static __device__ __forceinline__ Rec fetch(const SearchArgs& a, int j) { return a.rq[j]; }
    // coordinates about the block's centre, in half cell widths
    static __device__ __forceinline__ Coord coords(const Rec& rec, const BlockGeom<DIM>& g)
    {
        // the low ten bits as a signed number: cell indices are kept mod 2^10
        auto sbits10 = [](int v) { return static_cast<int>(static_cast<uint32_t>(v) << 22) >> 22; };
        const int cb = __builtin_bit_cast(int, rec.w);
        Coord c;
        c.x = rec.x + static_cast<float>(2 * sbits10(cb - g.xa) + g.xa - g.xb);
        c.y = rec.y + static_cast<float>(2 * sbits10((cb >> 10) - g.y0));
        c.z = DIM == 3 ? rec.z + static_cast<float>(2 * sbits10((cb >> 20) - g.z0)) : 0.0f;
        return c;
    }
    static __device__ __forceinline__ float bound(const BlockGeom<DIM>& g)
    {
        const float ht = static_cast<float>(g.xb - g.xa + 1);
        return 0x1p-18f * (2.0f * (ht * ht + 2.0f + (ht + 2.0f) * (ht + 2.0f) + 18.0f) + 4.0f);
    }
    static __device__ __forceinline__ void fragments(uint32_t (&w)[8], h8& f0, h8& f1)
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) swap32(w[k], w[k + 4]);
        f0 = __builtin_bit_cast(h8, make_uint4(w[0], w[1], w[2], w[3]));
        f1 = __builtin_bit_cast(h8, make_uint4(w[4], w[5], w[6], w[7]));
    }
    __device__ __forceinline__ void targets(const Rec& rec, const BlockGeom<DIM>& g)
    {
        const Coord c = coords(rec, g);
        uint32_t w[8];
        target_words(c.x, c.y, c.z, g.sd->fr.t32_mid, w);
        fragments(w, t0, t1);
        beta = bound(g);
    }
    // the sign bits of D's 16 results, result r at bit r; decide settles those with |D| below
    // the bound, if the wavefront has any
    template <typename F>
    static __device__ __forceinline__ uint32_t row_bits(const f32x16& D, float beta, F&& decide)
    {
        uint32_t acc = 0;
        float m = fabsf(D[15]);
#pragma unroll
        for (int r = 15; r >= 0; --r) {
            const float d = D[r];
            acc = __builtin_amdgcn_alignbit(acc, __builtin_bit_cast(uint32_t, d), 31);
        }
#pragma unroll
        for (int r = 0; r < 14; r += 2) m = fminf(fminf(m, fabsf(D[r])), fabsf(D[r + 1]));
        m = fminf(m, fabsf(D[14]));
        if (__builtin_amdgcn_ballot_w64(m < beta)) {
            uint32_t bnd = 0;
#pragma unroll
            for (int r = 15; r >= 0; --r) {
                const float d = fabsf(D[r]) - beta;
                bnd = __builtin_amdgcn_alignbit(bnd, __builtin_bit_cast(uint32_t, d), 31);
            }
            acc = decide(bnd, acc);
        }
        return acc;
    }
    struct Frag { h8 c[2]; };
    __device__ __forceinline__ Frag prepare(const Rec& rec, const BlockGeom<DIM>& g, bool past) const
    {
        const Coord x = coords(rec, g);
        uint32_t w[8];
        candidate_words(x.x, x.y, x.z, w);
        if (past) {
            w[0] = w[1] = w[2] = w[3] = w[4] = 0u;
            w[5] = 0x7800u;  // 32768
        }
        Frag f;
        fragments(w, f.c[0], f.c[1]);
        return f;
    }
    template <typename F>
    __device__ __forceinline__ u32x2 words(const Frag& f, const BlockGeom<DIM>&, F&& decide) const
    {
        const int lane = threadIdx.x & 63, e = 16 * (lane >> 5), tl = lane & 31;
        const f32x16 zero = {};
        u32x2 out;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const f32x16 D0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.c[t], t0, zero, 0, 0, 0);
            const f32x16 D1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.c[t], t1, zero, 0, 0, 0);
            uint32_t b0 = row_bits(D0, beta, [&](uint32_t n, uint32_t q) { return decide(n, q, 32 * t + e, tl); });
            uint32_t b1 = row_bits(D1, beta, [&](uint32_t n, uint32_t q) { return decide(n, q, 32 * t + e, 32 + tl); });
            swap32(b0, b1);
            out[t] = b0 | (b1 << 16);
        }
        return out;
    }
};

// P = 32: slots x y | z s | 1 0 (targets -2x -2y | -2z 1 | u 0), two per instruction; an
// operand lane l holds item l mod 32, slot l / 32 of each pair.
template <int DIM>
struct Tiles<DIM, 32> : Tiles<DIM, 16> {
    using B = Tiles<DIM, 16>;
    using typename B::Coord;
    using typename B::Rec;
    float t[2][3];
    static __device__ __forceinline__ void pair(float a, float b, float& f0, float& f1)
    {
        uint32_t x = __builtin_bit_cast(uint32_t, a), y = __builtin_bit_cast(uint32_t, b);
        swap32(x, y);
        f0 = __builtin_bit_cast(float, x);
        f1 = __builtin_bit_cast(float, y);
    }
    __device__ __forceinline__ void targets(const Rec& rec, const BlockGeom<DIM>& g)
    {
        const Coord c = B::coords(rec, g);
        pair(-2.0f * c.x, -2.0f * c.y, t[0][0], t[1][0]);
        pair(-2.0f * c.z, 1.0f, t[0][1], t[1][1]);
        pair(c.x * c.x + c.y * c.y + c.z * c.z - g.sd->fr.t32_mid, 0.0f, t[0][2], t[1][2]);
        this->beta = B::bound(g);
    }
    struct Frag { float c[2][2]; };
    __device__ __forceinline__ Frag prepare(const Rec& rec, const BlockGeom<DIM>& g, bool past) const
    {
        Coord x = B::coords(rec, g);
        float s = x.x * x.x + x.y * x.y + x.z * x.z;
        if (past) {
            x.x = x.y = x.z = 0.0f;
            s = 0x1p60f;
        }
        Frag f;
        pair(x.x, x.y, f.c[0][0], f.c[1][0]);
        pair(x.z, s, f.c[0][1], f.c[1][1]);
        return f;
    }
    template <typename F>
    __device__ __forceinline__ u32x2 words(const Frag& f, const BlockGeom<DIM>&, F&& decide) const
    {
        const int lane = threadIdx.x & 63, e = 16 * (lane >> 5), tl = lane & 31;
        const float one = lane < 32 ? 1.0f : 0.0f;
        u32x2 out;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            uint32_t b[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                f32x16 D = {};
                D = __builtin_amdgcn_mfma_f32_32x32x2f32(one, t[h][2], D, 0, 0, 0);
                D = __builtin_amdgcn_mfma_f32_32x32x2f32(f.c[k][0], t[h][0], D, 0, 0, 0);
                D = __builtin_amdgcn_mfma_f32_32x32x2f32(f.c[k][1], t[h][1], D, 0, 0, 0);
                b[h] = B::row_bits(D, this->beta,
                                   [&](uint32_t n, uint32_t q) { return decide(n, q, 32 * k + e, 32 * h + tl); });
            }
            swap32(b[0], b[1]);
            out[k] = b[0] | (b[1] << 16);
        }
        return out;
    }
};

// P = 64: slots x y z s (targets -2x -2y -2z 1, accumulator |t|^2 - R^2); an operand lane l
// holds item l mod 16, slot l / 16. Operand row rho = 4 r + q of tile i gives result r of the
// wavefront's quarter q, and holds candidate 16 q + 4 i + r of the step's 64.
template <int DIM>
struct Tiles<DIM, 64> {
    struct Rec { double x, y, z; };  // a union record in LDS
    double t[4], u[4], ox, oy, oz;
    int bhi;  // the high word of the bound, rounded up
    static __device__ __forceinline__ int item(int lane)
    {
        return 16 * (lane & 3) + 4 * (lane >> 4) + ((lane >> 2) & 3);
    }
    static __device__ __forceinline__ Rec fetch(const SearchArgs& a, int j)
    {
        const double2* s = reinterpret_cast<const double2*>(a.spos + static_cast<size_t>(j) * 4);
        const double2 xy = s[0];
        return Rec{xy.x, xy.y, DIM == 3 ? s[1].x : 0.0};
    }
    // out[i]: component l / 16 of item 16 i + l mod 16
    static __device__ __forceinline__ void fragments(const double (&v)[4], double (&out)[4])
    {
        uint32_t lo[4], hi[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint64_t q = __builtin_bit_cast(uint64_t, v[k]);
            lo[k] = static_cast<uint32_t>(q);
            hi[k] = static_cast<uint32_t>(q >> 32);
        }
        quarter_transpose(lo);
        quarter_transpose(hi);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            out[k] = __builtin_bit_cast(double, static_cast<uint64_t>(hi[k]) << 32 | lo[k]);
    }
    // about the wavefront's first target
    __device__ __forceinline__ void targets(const Rec& rec, const BlockGeom<DIM>& g)
    {
        auto first = [](double v) {
            const uint64_t q = __builtin_bit_cast(uint64_t, v);
            const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(q));
            const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(q >> 32));
            return __builtin_bit_cast(double, static_cast<uint64_t>(hi) << 32 | lo);
        };
        targets_about(rec, Rec{first(rec.x), first(rec.y), first(rec.z)}, g);
    }
    __device__ __forceinline__ void targets_about(const Rec& rec, const Rec& origin, const BlockGeom<DIM>& g)
    {
        ox = origin.x;
        oy = origin.y;
        oz = origin.z;
        const double x = rec.x - ox, y = rec.y - oy, z = rec.z - oz;
        const double v[4] = {-2.0 * x, -2.0 * y, -2.0 * z, 1.0};
        fragments(v, t);
        const double uu = x * x + y * y + z * z - g.sd->fr.R2;
        // the accumulator of target tile k: u of target 16 k + l mod 16
#pragma unroll
        for (int k = 0; k < 4; ++k) u[k] = __shfl(uu, 16 * k + static_cast<int>(threadIdx.x & 15), 64);
        const double xs = static_cast<double>(g.xb - g.xa + 2), w = g.sd->fr.w;
        const double beta = 0x1p-46 * w * w * (4.0 * (xs * xs + 8.0) + 1.0);
        // cells so wide or so narrow that a square or the bound could leave the exponent range
        // (and a NaN pass the minimum below unseen): no result is below a NaN, all are decided
        bhi = w > 0x1p-450 && w < 0x1p450 ? static_cast<int>(__builtin_bit_cast(uint64_t, beta) >> 32) + 1 : 0x7FFFFFFF;
    }
    struct Frag { double c[4]; };
    __device__ __forceinline__ Frag prepare(const Rec& rec, const BlockGeom<DIM>&, bool past) const
    {
        const double x = past ? 0.0 : rec.x - ox, y = past ? 0.0 : rec.y - oy, z = past ? 0.0 : rec.z - oz;
        // past: |t|^2 - R^2 stays below 2^917 in the range where signs decide (see targets_about)
        const double v[4] = {x, y, z, past ? 0x1p1000 : x * x + y * y + z * z};
        Frag f;
        fragments(v, f.c);
        return f;
    }
    template <typename F>
    __device__ __forceinline__ u32x2 words(const Frag& f, const BlockGeom<DIM>& g, F&& decide) const
    {
        const int lane = threadIdx.x & 63, nt = g.p1 - g.p0;
        uint32_t b[4] = {0, 0, 0, 0};
        // non-negative doubles order like their high words read as floats
        const float below = __builtin_bit_cast(float, bhi);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (16 * k >= nt) break;
            const f64x4 acc0 = {u[k], u[k], u[k], u[k]};
            float hi[16];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f64x4 D = __builtin_amdgcn_mfma_f64_16x16x4f64(f.c[i], t[k], acc0, 0, 0, 0);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const double d = D[r];
                    const uint32_t top = static_cast<uint32_t>(__builtin_bit_cast(uint64_t, d) >> 32);
                    hi[4 * i + r] = __builtin_bit_cast(float, top);
                }
            }
            uint32_t acc = 0;
            float m = fabsf(hi[15]);
#pragma unroll
            for (int r = 15; r >= 0; --r)
                acc = __builtin_amdgcn_alignbit(acc, __builtin_bit_cast(uint32_t, hi[r]), 31);
#pragma unroll
            for (int r = 0; r < 14; r += 2) m = fminf(fminf(m, fabsf(hi[r])), fabsf(hi[r + 1]));
            m = fminf(m, fabsf(hi[14]));
            if (__builtin_amdgcn_ballot_w64(!(m >= below))) {
                uint32_t bnd = 0;
#pragma unroll
                for (int r = 15; r >= 0; --r) bnd = (bnd << 1) | (fabsf(hi[r]) >= below ? 0u : 1u);
                acc = decide(bnd, acc, 16 * (lane >> 4), 16 * k + (lane & 15));
            }
            b[k] = acc;
        }
        quarter_transpose(b);
        return u32x2{b[0] | (b[1] << 16), b[2] | (b[3] << 16)};
    }
};

// LDS of a block's count by NW wavefronts, unions of up to UC candidates ranked.
template <int DIM, int P, int NW, int UC>
struct CountShared {
    using Rec = typename Tiles<DIM, P>::Rec;
    // the ranking's scratch, then the union's records by rank
    static constexpr int kRecs = UC * static_cast<int>(sizeof(Rec));
    static constexpr int kBytes = NW > 1 && kRankScratch<UC> > kRecs ? kRankScratch<UC> : kRecs;
    alignas(16) unsigned char scratch[kBytes];
    int slist[UC];  // sorted positions by rank (the ranking's ranks before)
    int srself[64];  // the targets' own ranks
    int sred[2][NW];
    int swsum[NW];
    int spart[NW][64];
    uint32_t splace;
};

// Counts block b and writes its descriptor. Unions above UC are counted in union order, unranked;
// they, and blocks whose pool is empty, keep no bits (their rows take the long-row path).
// POOL: the ranks' places come from the pools.
template <int DIM, int P, bool HALF, bool POOL, int NW, int UC>
__device__ __forceinline__ void count_block(const SearchArgs& a, const BlockGeom<DIM>& g, int b,
                                            CountShared<DIM, P, NW, UC>& sh)
{
    constexpr int NT = 64 * NW, EPT = UC / NT;
    using T = Tiles<DIM, P>;
    using Rec = typename T::Rec;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int U = g.U, nt = g.p1 - g.p0;
    const bool ranked = NW == 1 || U <= UC;
    Rec* const srec = reinterpret_cast<Rec*>(sh.scratch);
    int* const slist = sh.slist;
    const Rec trec = T::fetch(a, g.p0 + min(lane, nt - 1));
    int rself = g.seg_base[g.SELF] + (g.p0 + lane - g.seg_g0[g.SELF]);
    uint32_t place = !POOL && ranked ? block_ranks<DIM>(b) : kNoRanks;
    if (!POOL && wv == 0) write_desc<DIM>(a, g, b, U, place);
    if (ranked) {
        // a pool's counter is asked before the loads and read after the ranking
        uint32_t mine = 0;
        if (POOL && tid == 0) mine = take_ranks(a, b, U);
        // the union's indices and records, in union order (contiguous along x); one wavefront
        // loads no more than the union has, several issue their loads together
        int gi[EPT], og[EPT] = {}, rk[EPT];
        Rec rec[EPT];
#pragma unroll
        for (int i = 0; i < EPT; ++i) gi[i] = g.global_of_any(min(tid + i * NT, U - 1));
#pragma unroll
        for (int i = 0; i < EPT; ++i)
            if (NW > 1 || i * NT < U) og[i] = a.perm[gi[i]];
#pragma unroll
        for (int i = 0; i < EPT; ++i)
            if (NW > 1 || i * NT < U) rec[i] = T::fetch(a, gi[i]);
        if (POOL && tid == 0) sh.splace = mine;
        if constexpr (NW == 1)
            rank_wave<UC>(U, og, reinterpret_cast<uint32_t*>(sh.scratch), reinterpret_cast<uint16_t*>(slist), rk);
        else
            rank_originals<UC, FillCfg<DIM>::SHIFT, NW>(U, og, sh.scratch, sh.sred, sh.swsum,
                                                        reinterpret_cast<uint16_t*>(slist), rk);
        const int self0 = g.seg_base[g.SELF] + (g.p0 - g.seg_g0[g.SELF]);  // the first target's union position
        if (POOL) place = __builtin_amdgcn_readfirstlane(sh.splace);
        uint16_t* ranks = a.branks + static_cast<size_t>(place) * kRankPiece;
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            const int e = tid + i * NT;
            if (e < U) {
                srec[rk[i]] = rec[i];
                slist[rk[i]] = gi[i];
                if (!POOL || place != kNoRanks) ranks[e] = static_cast<uint16_t>(rk[i]);
                if (static_cast<unsigned>(e - self0) < static_cast<unsigned>(nt)) sh.srself[e - self0] = rk[i];
            }
        }
        __syncthreads();
        rself = lane < nt ? sh.srself[lane] : 0;
    }
    const bool kept = POOL ? place != kNoRanks : ranked;
    if (POOL && wv == 0) write_desc<DIM>(a, g, b, kept ? U : max(U, FillCfg<DIM>::UCAP + 1), place);
    T tiles;
    tiles.targets(trec, g);
    const double R2 = g.sd->fr.R2;
    const int mi = T::item(lane);
    int cnt = 0;
    for (int c0 = 0; c0 < U; c0 += UC) {  // one pass when ranked
        const int m = min(UC, U - c0);
        if (!ranked) {
            __syncthreads();
            for (int e = tid; e < m; e += NT) {
                slist[e] = g.global_of_any(c0 + e);
                srec[e] = T::fetch(a, slist[e]);
            }
            __syncthreads();
        }
        // 64 list entries a step, steps dealt to the wavefronts
#pragma unroll 1
        for (int s = wv; 64 * s < m; s += NW) {
            const Rec rec = srec[min(64 * s + mi, m - 1)];
            auto decide = [&](uint32_t bnd, uint32_t acc, int e0, int t) -> uint32_t {
                const double* pi = a.spos + static_cast<size_t>(g.p0 + min(t, nt - 1)) * 4;
                while (bnd) {
                    const int r = __builtin_ctz(bnd);
                    bnd &= bnd - 1u;
                    const int e = 64 * s + e0 + r;
                    const bool in = e < m && recheck_sorted<DIM>(a.spos, pi, slist[e], R2);
                    acc = (acc & ~(1u << r)) | (static_cast<uint32_t>(in) << r);
                }
                return acc;
            };
            const u32x2 ww = tiles.words(tiles.prepare(rec, g, 64 * s + mi >= m), g, decide);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int tile = 2 * s + k;
                uint32_t word = ww[k];
                // the target itself is no neighbour; half lists keep larger original indices
                const int d = rself - c0 - 32 * tile;
                if (HALF && ranked) word &= d < 0 ? ~0u : (d >= 31 ? 0u : 0xFFFFFFFEu << d);
                else word &= (d >= 0 && d < 32) ? ~(1u << d) : ~0u;
                if (HALF && !ranked && lane < nt) {
                    const int oi = a.perm[g.p0 + lane];
                    for (uint32_t q = word; q; q &= q - 1u) {
                        const int j = __builtin_ctz(q);
                        if (a.perm[slist[32 * tile + j]] < oi) word &= ~(1u << j);
                    }
                }
                cnt += __builtin_popcount(word);
                if (kept && lane < nt && 32 * tile < m)
                    a.cbits[static_cast<size_t>(tile) * a.L.ntot + g.p0 + lane] = word;
            }
        }
    }
    if (NW > 1) {
        sh.spart[wv][lane] = cnt;
        __syncthreads();
    }
    if (tid < nt) {
        int c = NW > 1 ? 0 : cnt;
#pragma unroll
        for (int q = 0; NW > 1 && q < NW; ++q) c += sh.spart[q][tid];
        a.counts[a.perm[g.p0 + tid]] = c;
        a.counts_s[g.p0 + tid] = c;
    }
}

template <int DIM, int P, bool HALF, bool POOL>
__global__ void __launch_bounds__(kCountThreads<DIM>) __attribute__((amdgpu_waves_per_eu(P == 64 ? 4 : 5)))
k_count(SearchArgs a)
{
    constexpr int UCAP = FillCfg<DIM>::UCAP;
    __shared__ CountShared<DIM, P, kCountThreads<DIM> / 64, UCAP> sh;
    if (a.wdense && blockIdx.x == 0 && threadIdx.x == 0) a.flags[kFlagUnit] = 0;  // for the dense count behind this
    const int b = xcd_block(*a.nblk);
    if (b < 0) return;
    if (dense_block(a, b)) {
        if (threadIdx.x < 64) write_desc_dense(a, b);
        return;
    }
    BlockGeom<DIM> g;
    g.init(a, b);
    count_block<DIM, P, HALF, POOL>(a, g, b, sh);
}

// Sparse sets in 3D (see kSparseUnion): most blocks have a few targets and unions of tens of
// candidates, and what bounds the count is the chain of dependent loads and the ranking per block, so
// one wavefront takes a block and the chip holds four times as many at once. Unions above
// kSmallUnion are left to k_count_rest, marked in their descriptor.
template <int P, bool HALF>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4)))
k_count_small(SearchArgs a)
{
    __shared__ CountShared<3, P, 1, kSmallUnion> sh;
    if (a.wdense && blockIdx.x == 0 && threadIdx.x == 0) a.flags[kFlagUnit] = 0;  // for the dense count behind this
    const int b = xcd_block(*a.nblk);
    if (b < 0) return;
    if (dense_block(a, b)) {
        write_desc_dense(a, b);
        return;
    }
    BlockGeom<3> g;
    g.init(a, b);
    if (g.U <= kSmallUnion) count_block<3, P, HALF, true>(a, g, b, sh);
    else write_desc<3>(a, g, b, g.U, kNoRanks, 2);
}

// The blocks that k_count_small left, found by their descriptors: workgroup i takes those of the
// blocks i, i + gridDim, ... (dealt out one by one, as they may all lie in a small part of the box).
template <int P, bool HALF>
__global__ void __launch_bounds__(kCountThreads<3>) __attribute__((amdgpu_waves_per_eu(P == 64 ? 4 : 5)))
k_count_rest(SearchArgs a)
{
    constexpr int NT = kCountThreads<3>;
    __shared__ CountShared<3, P, NT / 64, kUnion3> sh;
    __shared__ int sfound[NT];
    __shared__ int snfound;
    const int nblk = *a.nblk, step = gridDim.x;
    for (int64_t i0 = blockIdx.x; i0 < nblk; i0 += static_cast<int64_t>(NT) * step) {
        if (threadIdx.x == 0) snfound = 0;
        __syncthreads();
        const int64_t i = i0 + static_cast<int64_t>(threadIdx.x) * step;
        if (i < nblk && a.bdesc[static_cast<size_t>(i) * kDescInts + 4] == 2)
            sfound[atomicAdd(&snfound, 1)] = static_cast<int>(i);
        __syncthreads();
        const int nfound = __builtin_amdgcn_readfirstlane(snfound);
        for (int k = 0; k < nfound; ++k) {
            const int b = __builtin_amdgcn_readfirstlane(sfound[k]);
            BlockGeom<3> g;
            g.init(a, b);
            count_block<3, P, HALF, true>(a, g, b, sh);
            __syncthreads();  // the next block writes the shared tables
        }
        __syncthreads();
    }
}

constexpr int kFillThreads = 256;  // four wavefronts share one block's union

// Fill pass. The union's positions and set-local indices are staged in LDS in rank order;
// then each wavefront works alone on sixteen of the block's targets: their accepted
// candidates (the count pass's bits, in rank order; lane = target and quarter of the row's
// words) are compacted into its flat list of 16-bit entries (target << 10 | rank), as many
// quarter rows at a time as the list holds, and written 64 entries per store, the entries'
// gathers being LDS reads. One workgroup barrier per block and 26 KB of LDS, so that
// memory, LDS and vector work overlap over six workgroups per compute unit (lists of 512 entries
// fit seven, but walk the words twice: 222 against 213 us).
// F64: positions in binary64, distances (float)sqrt(r2) in binary64. Otherwise the low 32 bits
// of the positions in units of 2^-30 or so of a cell width (Frame::quantum), one 16-byte
// record per candidate: neighbours lie fewer than 2^31 units apart, so the difference mod
// 2^32 is exact, and is rounded once to FP32; pairs so near that the unit would show are
// recomputed from the binary64 positions. (Non-temporal stores were slower in 2D and at 64,000
// points, two entries a store no faster: 412 against 414 us for the step in 3D, 172 against 169 in 2D.)
// What bounds it: vector issue and HBM about evenly. At 1M particles in 3D (60 M entries, 728 MB
// of DRAM traffic, 78 M vector instructions): 322 us with the ranking and gathers from global
// memory here, 213 now; 2D 93 -> 60, binary64 321 -> 244 us.
// POOL: the ranks' places come from the pools (else a block's is known without its descriptor).
template <int DIM, bool F64, bool POOL>
__global__ void __launch_bounds__(kFillThreads) __attribute__((amdgpu_waves_per_eu(F64 ? 4 : 6)))
k_fill(SearchArgs a)
{
    using C = FillCfg<DIM>;
    constexpr int NW = kFillThreads / 64;
    constexpr int EPT = C::UCAP / kFillThreads;
    constexpr int KW = C::MW / 4;  // bit words per lane
    constexpr int TW = 64 / NW;    // targets per wavefront
    static_assert(TW == 16, "a lane's target is its place in a row of 16 lanes");
    constexpr int FW = C::FLAT;
    static_assert(FW >= 32 * KW, "a quarter row fits the list");
    __shared__ uint16_t sflat[NW][FW];
    __shared__ int4 srec[F64 ? 1 : C::UCAP];          // position, set-local index, by rank
    __shared__ double spos[F64 ? DIM * C::UCAP : 1];  // axis-major, by rank
    __shared__ int sorig[F64 ? C::UCAP : 1];          // set-local index by rank
    __shared__ int4 strec[F64 ? 1 : 64];              // the targets' positions
    __shared__ double sxi[F64 ? 64 * DIM : 1];
    __shared__ long long sbase[64];  // row start in the output minus the row's flat offset

    const int b = xcd_block(*a.nblk);
    if (b < 0) return;
    // the block's geometry from the count pass's descriptor (wave-uniform), and each
    // target's row start and length in sorted order: no chain of dependent loads
    const NNPS_CONST int* dsc = (const NNPS_CONST int*)(a.bdesc + static_cast<size_t>(b) * kDescInts);
    if (dsc[4]) return;  // a block of the dense-cell path
    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront index, uniform
    const int p0 = dsc[0], nt = dsc[1] - p0, U = dsc[3];
    if (U > C::UCAP) {
        // too big for this path: every row of the block goes to the long-row path
        if (tid < nt) a.heavy[atomicAdd(a.flags + kFlagHeavy, 1)] = p0 + tid;
        return;
    }
    const NNPS_CONST SetDesc& sd = ((const NNPS_CONST SetDesc*)a.L.sets)[dsc[2]];
    // this lane's target and quarter of its row's words
    const int tg = wv * TW + (lane & 15), quarter = lane >> 4;
    const bool active = tg < nt;
    const int pt = p0 + min(tg, nt - 1);
    const int nw = (U + 31) >> 5, qw = (nw + 3) >> 2, wa = quarter * qw;
    // union position -> sorted position, from the segments' first particles and union offsets
    auto global_of = [&](int posl) {
        constexpr int NSEG = Geom<DIM>::NSEG;
        int delta = dsc[5] - dsc[5 + NSEG];
#pragma unroll
        for (int k = 1; k < NSEG; ++k)
            if (posl >= dsc[5 + NSEG + k]) delta = dsc[5 + k] - dsc[5 + NSEG + k];
        return posl + delta;
    };
    int rank[EPT];
#pragma unroll
    for (int i = 0; i < EPT; ++i)
        rank[i] = a.branks[static_cast<size_t>(POOL ? static_cast<uint32_t>(dsc[kDescRanks]) : block_ranks<DIM>(b)) *
                               kRankPiece + min(tid + i * kFillThreads, U - 1)];
    uint32_t wbits[KW];
#pragma unroll
    for (int k = 0; k < KW; ++k) wbits[k] = a.cbits[static_cast<size_t>(min(wa + k, nw - 1)) * a.L.ntot + pt];
    const long long rs = a.rsort[pt];
    int rlen = a.counts_s[pt];
    struct Raw {
        double2 lo, hi;
    };
    auto raw = [&](int j) {
        const double2* s = reinterpret_cast<const double2*>(a.spos + static_cast<size_t>(j) * 4);
        return Raw{s[0], s[1]};
    };
    const double inv_quantum = sd.fr.inv_quantum;
    const double lo[3] = {sd.fr.lo[0], sd.fr.lo[1], sd.fr.lo[2]};
    auto fixed = [&](double x, int k) { return in_quanta(x, lo[k], inv_quantum); };
    auto packed = [&](const Raw& r, int w) {
        return make_int4(fixed(r.lo.x, 0), fixed(r.lo.y, 1), DIM == 3 ? fixed(r.hi.x, 2) : 0, w);
    };
    // 1. the union and the targets to LDS, a thread's gathers issued together
    {
        const int poff = sd.poff;
        Raw r[EPT];
#pragma unroll
        for (int i = 0; i < EPT; ++i) r[i] = raw(global_of(min(tid + i * kFillThreads, U - 1)));
        const Raw t = raw(p0 + min(tid, nt - 1));
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            const int e = tid + i * kFillThreads;
            const int oj = static_cast<int>(__builtin_bit_cast(int64_t, r[i].hi.y)) - poff;
            if (e >= U) continue;
            if (F64) {
                spos[rank[i]] = r[i].lo.x;
                spos[C::UCAP + rank[i]] = r[i].lo.y;
                if (DIM == 3) spos[2 * C::UCAP + rank[i]] = r[i].hi.x;
                sorig[rank[i]] = oj;
            } else {
                srec[rank[i]] = packed(r[i], oj);
            }
        }
        if (tid < 64) {
            if (F64) {
                sxi[tid * DIM] = t.lo.x;
                sxi[tid * DIM + 1] = t.lo.y;
                if (DIM == 3) sxi[tid * DIM + 2] = t.hi.x;
            } else {
                strec[tid] = packed(t, 0);
            }
        }
    }
    // the rows' places: off among the wavefront's sixteen rows, before among the row's quarters
    int cnt = 0;
#pragma unroll
    for (int k = 0; k < KW; ++k) {
        if (!(active && k < qw && wa + k < nw)) wbits[k] = 0u;
        cnt += __builtin_popcount(wbits[k]);
    }
    if (!active) rlen = 0;
    int before = 0, have = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int c = __shfl(cnt, 16 * q + (lane & 15), 64);
        if (q < quarter) before += c;
        have += c;
    }
    // a row whose bits do not match its count writes nothing: it takes no place in the list
    if (have != rlen) {
        atomicOr(a.flags + kFlagErr, kErrLongRow);
        cnt = before = rlen = 0;
#pragma unroll
        for (int k = 0; k < KW; ++k) wbits[k] = 0u;
    }
    int incl = rlen;  // inclusive over the 16 lanes of a row
    incl += dpp<0x111>(0, incl);
    incl += dpp<0x112>(0, incl);
    incl += dpp<0x114>(0, incl);
    incl += dpp<0x118>(0, incl);
    const int off = incl - rlen;
    if (lane < TW) sbase[tg] = rs - off;
    __syncthreads();
    NNPS_GLOBAL int32_t* const col = (NNPS_GLOBAL int32_t*)sd.col;
    NNPS_GLOBAL float* const dist = (NNPS_GLOBAL float*)sd.dist;
    const int64_t cap = sd.capacity;
    const long long rend = active ? rs + rlen : 0;  // the row's end in the output
    const bool room = __builtin_amdgcn_ballot_w64(rend > cap) == 0;
    if (!room && rend > cap) atomicOr(a.flags + kFlagErr, kErrCapacity);
    const float quantum = sd.fr.quantum, near2 = sd.fr.near2;
    uint16_t* const flat = sflat[wv];
    // the lane's quarter row among the wavefront's entries
    const int u0 = off + before, u1 = u0 + cnt;
    for (int o0 = 0;;) {
        // the quarter rows from o0 up to the list's capacity
        const bool mine = u0 >= o0 && u1 - o0 <= FW;
        const int o1 = wave_max_i32(mine ? u1 : o0);
        if (o1 == o0) break;
        // 2. compaction: each row's bits walked in rank order
        if (mine) {
            uint16_t* f = flat + (u0 - o0);
            const uint32_t tag0 = static_cast<uint32_t>((lane & 15) << 10);
#pragma unroll
            for (int k = 0; k < KW; ++k) {
                uint32_t bits = wbits[k];
                const uint32_t tag = tag0 | static_cast<uint32_t>((wa + k) * 32);
                while (bits) {
                    *f++ = static_cast<uint16_t>(tag | __builtin_ctz(bits));
                    bits &= bits - 1u;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        // 3. emission: consecutive lanes write consecutive entries, two entries of a lane in
        // flight (entries past the list repeat its last one)
        const int n = o1 - o0;
        constexpr int Q = 2;
        for (int e0 = lane; e0 < n; e0 += Q * 64) {
            int t[Q], rk[Q], oj[Q];
            long long idx[Q];
            float d[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const uint32_t f = flat[min(e0 + q * 64, n - 1)];
                t[q] = wv * TW + static_cast<int>(f >> 10);
                rk[q] = static_cast<int>(f & 1023u);
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                idx[q] = sbase[t[q]] + (o0 + min(e0 + q * 64, n - 1));
                if constexpr (F64) {
                    double xi[3], xj[3];
#pragma unroll
                    for (int k = 0; k < DIM; ++k) {
                        xj[k] = spos[k * C::UCAP + rk[q]];
                        xi[k] = sxi[t[q] * DIM + k];
                    }
                    oj[q] = sorig[rk[q]];
                    d[q] = dist_fp64<DIM>(xi, xj);
                } else {
                    const int4 j = srec[rk[q]];
                    oj[q] = j.w;
                    d[q] = quanta2<DIM>(strec[t[q]], j);
                }
            }
            if constexpr (!F64) {
                float least = d[0];
#pragma unroll
                for (int q = 1; q < Q; ++q) least = fminf(least, d[q]);
                const bool near = !(least >= near2);
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const float s2 = d[q];
                    d[q] = root(s2) * quantum;  // exact: a power of two
                    if (near && !(s2 >= near2))
                        d[q] = dist_near<DIM>(a.spos + static_cast<size_t>(p0 + t[q]) * 4,
                                              (const double*)sd.pos + static_cast<size_t>(oj[q]) * DIM, inv_quantum,
                                              quantum);
                }
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if (room || idx[q] < cap) {
                    col[idx[q]] = oj[q];
                    dist[idx[q]] = d[q];
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        o0 = o1;
    }
}

// ---------------------------------------------------------------------------
// Long rows (blocks whose union exceeds the fill's limit or that have no ranks): one workgroup per
// target. Its candidates are tested in binary64 across the workgroup and the accepted original
// indices appended to the row in any order; the row is then sorted
// in place (LDS bitonic network for up to lr_keys entries, in which every comparator puts
// the smaller key first so padding at +inf never moves; longer rows are sorted in chunks
// and merged pairwise by rank, using the row's distance slots as scratch), and finally
// the distances are computed from the sorted column indices.
constexpr int kLongThreads = 256;

template <int DIM, int MODE>
__global__ void __launch_bounds__(kLongThreads)
k_long(SearchArgs a)
{
    extern __shared__ uint32_t keys[];  // a.lr_keys entries
    __shared__ int fill;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.flags[kFlagUnit] = 0;  // for the dense fill behind this
    const int nh = a.flags[kFlagHeavy];
    if (nh == 0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) a.flags[kFlagLong] = 0;
        return;
    }
    const int T = kLongThreads;
    for (int h = blockIdx.x; h < nh; h += gridDim.x) {
        const int p = a.heavy[h];
        const uint32_t gkey = a.skey[p];
        const SetDesc& sdesc = a.L.sets[find_set(a.L.coffs, a.L.nsets, static_cast<int>(gkey))];
        const Frame fr = sdesc.fr;
        const int* cs = a.cell_start + sdesc.coff;
        const uint32_t scoff = static_cast<uint32_t>(sdesc.coff);
        const SetView sd(sdesc);
        const uint32_t ncx = static_cast<uint32_t>(fr.nc[0]);
        const int ncy = fr.nc[1], ncz = fr.nc[2];
        const uint32_t key = gkey - scoff;
        const uint32_t row = key / ncx;
        const int x = static_cast<int>(key - row * ncx);
        const int y0 = static_cast<int>(row % static_cast<uint32_t>(ncy));
        const int z0 = static_cast<int>(row / static_cast<uint32_t>(ncy));
        const int oi = a.perm[p];
        const int li = oi - sd.poff;
        const long long rs = sd.row_ptr[li];
        const int rlen = static_cast<int>(sd.row_ptr[li + 1] - rs);
        double pi[3] = {0, 0, 0};
#pragma unroll
        for (int k = 0; k < DIM; ++k) pi[k] = a.spos[static_cast<size_t>(p) * 4 + k];
        if (threadIdx.x == 0) fill = 0;
        __syncthreads();
        const bool room = rs + rlen <= sd.capacity;
        NNPS_GLOBAL int32_t* col = sd.col + rs;
        // 1. test every candidate; append accepted set-local indices in any order
        constexpr int NSEG = DIM == 3 ? 9 : 3;
        const int lx0 = x > 0 ? x - 1 : 0;
        const int lx1 = x + 1 < static_cast<int>(ncx) ? x + 1 : static_cast<int>(ncx) - 1;
        for (int r = 0; r < NSEG; ++r) {
            const int dy = r % 3 - 1, dz = DIM == 3 ? r / 3 - 1 : 0;
            const int yy = y0 + dy, zz = z0 + dz;
            if (yy < 0 || yy >= ncy || zz < 0 || zz >= ncz) continue;
            const int rb = (zz * ncy + yy) * static_cast<int>(ncx);
            const int ga = cs[rb + lx0], gb = cs[rb + lx1 + 1];
            for (int j = ga + static_cast<int>(threadIdx.x); j < gb; j += T) {
                if (j == p) continue;
                const bool nb = recheck_sorted<DIM>(a.spos, pi, j, fr.R2);
                const int oj = a.perm[j];
                if (nb && (!a.half || oj > oi)) {
                    const int slot = atomicAdd(&fill, 1);
                    if (slot < rlen && room) col[slot] = oj - sd.poff;
                }
            }
        }
        __syncthreads();
        const int L = fill;
        if (L != rlen || !room) {
            if (threadIdx.x == 0) atomicOr(a.flags + kFlagErr, !room ? kErrCapacity : kErrLongRow);
            __syncthreads();
            continue;
        }
        // 2. sort the row's column indices (distinct keys): rows of up to 512 entries in the
        // registers of the first wavefront (no workgroup barrier inside the network), longer
        // ones in LDS chunks merged pairwise below
        const int K = L <= 512 ? 512 : a.lr_keys;
        if (L <= 512) {
            if (threadIdx.x < 64) {
                if (L <= 64) wave_sort_row<1>(col, L);
                else if (L <= 128) wave_sort_row<2>(col, L);
                else if (L <= 256) wave_sort_row<4>(col, L);
                else wave_sort_row<8>(col, L);
            }
            __syncthreads();
        }
        for (int c0 = 0; L > 512 && c0 < L; c0 += K) {
            const int len = min(K, L - c0);
            int P = 1;
            while (P < len) P <<= 1;
            for (int i = threadIdx.x; i < P; i += T) keys[i] = i < len ? static_cast<uint32_t>(col[c0 + i]) : 0xFFFFFFFFu;
            __syncthreads();
            for (int k = 2; k <= P; k <<= 1) {
                for (int j = k >> 1; j > 0; j >>= 1) {
                    for (int t = threadIdx.x; t < P / 2; t += T) {
                        int i0, i1;
                        if (j == (k >> 1)) {
                            i0 = (t / j) * k + (t % j);
                            i1 = (t / j) * k + (k - 1 - (t % j));
                        } else {
                            i0 = (t / j) * 2 * j + (t % j);
                            i1 = i0 + j;
                        }
                        const uint32_t u = keys[i0], v = keys[i1];
                        if (u > v) {
                            keys[i0] = v;
                            keys[i1] = u;
                        }
                    }
                    __syncthreads();
                }
            }
            for (int i = threadIdx.x; i < len; i += T) col[c0 + i] = static_cast<int32_t>(keys[i]);
            __syncthreads();
        }
        // merge sorted runs of width K, 2K, ... between the column slots and the
        // distance slots (reinterpreted as 32-bit keys)
        NNPS_GLOBAL uint32_t* src = (NNPS_GLOBAL uint32_t*)col;
        NNPS_GLOBAL uint32_t* dst = (NNPS_GLOBAL uint32_t*)(sd.dist + rs);
        for (int width = K; width < L; width <<= 1) {
            for (int e = threadIdx.x; e < L; e += T) {
                const int run = e / width;
                const int base = (run & ~1) * width;           // start of the pair of runs
                const int mid = min(base + width, L), end = min(base + 2 * width, L);
                const uint32_t v = src[e];
                // position among the other run: keys are distinct
                int lo, hi, own;
                if (e < mid) { lo = mid; hi = end; own = e - base; }
                else { lo = base; hi = mid; own = e - mid; }
                int cnt = 0, l = lo, r = hi;
                while (l < r) {
                    const int m = (l + r) >> 1;
                    if (src[m] < v) l = m + 1;
                    else r = m;
                }
                cnt = l - lo;
                dst[base + own + cnt] = v;
            }
            __syncthreads();
            NNPS_GLOBAL uint32_t* tmp = src;
            src = dst;
            dst = tmp;
        }
        if (src != (NNPS_GLOBAL uint32_t*)col) {
            for (int e = threadIdx.x; e < L; e += T) col[e] = static_cast<int32_t>(src[e]);
            __syncthreads();
        }
        // 3. distances of the sorted row
        for (int e = threadIdx.x; e < L; e += T) {
            double pj[3] = {0, 0, 0};
#pragma unroll
            for (int k = 0; k < DIM; ++k) pj[k] = sd.pos[static_cast<size_t>(col[e]) * DIM + k];
            float d;
            if (MODE == 1) {
                d = dist_fp64<DIM>(pi, pj);
            } else {  // as the block path's fill: which rows come here depends on the block table
                d = dist_quanta<DIM>(fr, pi, pj);
            }
            sd.dist[rs + e] = d;
        }
        __syncthreads();
    }
    // the last workgroup hands the list back empty, once every thread has read its length
    __syncthreads();
    if (threadIdx.x == 0 && atomicAdd(a.flags + kFlagLongDone, 1) == static_cast<int>(gridDim.x) - 1) {
        a.flags[kFlagLong] = nh;
        a.flags[kFlagLongDone] = 0;
        a.flags[kFlagHeavy] = 0;
    }
}

// ---------------------------------------------------------------------------
// Grid of the block kernels: a whole number of rounds over the XCDs, so xcd_block reaches
// every block of any count up to nblk_max.
static dim3 block_grid(int nblk_max) { return dim3((nblk_max + kXcds - 1) / kXcds * kXcds); }

// Workgroups of k_count_rest: as many as the 256 compute units can hold.
constexpr int kRestGrid = 2048;

template <int P, bool HALF>
void launch_count_sparse(const SearchArgs& a, const dim3& g, hipStream_t st)
{
    hipLaunchKernelGGL((k_count_small<P, HALF>), g, dim3(64), 0, st, a);
    hipLaunchKernelGGL((k_count_rest<P, HALF>), dim3(kRestGrid), dim3(kCountThreads<3>), 0, st, a);
}

template <int DIM, int P, bool HALF>
void launch_count_of(const SearchArgs& a, const dim3& g, hipStream_t st)
{
    if (DIM == 3 && a.sparse && a.rpool) launch_count_sparse<P, HALF>(a, g, st);
    else if (a.rpool) hipLaunchKernelGGL((k_count<DIM, P, HALF, true>), g, dim3(kCountThreads<DIM>), 0, st, a);
    else hipLaunchKernelGGL((k_count<DIM, P, HALF, false>), g, dim3(kCountThreads<DIM>), 0, st, a);
}

template <int DIM, bool HALF>
void launch_count_mode(const SearchArgs& a, int mode, const dim3& g, hipStream_t st)
{
    if (mode == 0) launch_count_of<DIM, 16, HALF>(a, g, st);
    else if (mode == 3) launch_count_of<DIM, 32, HALF>(a, g, st);
    else launch_count_of<DIM, 64, HALF>(a, g, st);
}

hipError_t launch_count(const SearchArgs& a, int nblk_max, hipStream_t st)
{
    if (a.L.ntot == 0 || nblk_max == 0) return hipSuccess;
    const dim3 g = block_grid(nblk_max);
    const int d = a.L.dim, m = a.L.mode;
    if (a.half) {
        if (d == 2) launch_count_mode<2, true>(a, m, g, st);
        else launch_count_mode<3, true>(a, m, g, st);
    } else {
        if (d == 2) launch_count_mode<2, false>(a, m, g, st);
        else launch_count_mode<3, false>(a, m, g, st);
    }
    return hipGetLastError();
}

hipError_t launch_fill(const SearchArgs& a, int nblk_max, hipStream_t st)
{
    if (a.L.ntot == 0 || nblk_max == 0) return hipSuccess;
    const int d = a.L.dim;
    const bool f64 = a.L.mode == 1 || a.L.mode == 3;  // FP64 and FP32 modes: binary64 distances
    const dim3 g = block_grid(nblk_max), b(kFillThreads);
    auto k = [&](auto pool) {
        constexpr bool POOL = decltype(pool)::value;
        return d == 2 ? (f64 ? k_fill<2, true, POOL> : k_fill<2, false, POOL>)
                      : (f64 ? k_fill<3, true, POOL> : k_fill<3, false, POOL>);
    };
    hipLaunchKernelGGL(a.rpool ? k(std::true_type{}) : k(std::false_type{}), g, b, 0, st, a);
    return hipGetLastError();
}

hipError_t launch_long_rows(const SearchArgs& a, int grid, hipStream_t st)
{
    if (a.L.ntot == 0) return hipSuccess;
    const int d = a.L.dim, m = a.L.mode == 3 ? 1 : a.L.mode;  // FP32 mode: long rows in FP64
    const dim3 gh(grid), bh(kLongThreads);
    const size_t lds = static_cast<size_t>(a.lr_keys) * 4;
    if (d == 2 && m != 1) hipLaunchKernelGGL((k_long<2, 0>), gh, bh, lds, st, a);
    else if (d == 3 && m != 1) hipLaunchKernelGGL((k_long<3, 0>), gh, bh, lds, st, a);
    else if (d == 2) hipLaunchKernelGGL((k_long<2, 1>), gh, bh, lds, st, a);
    else hipLaunchKernelGGL((k_long<3, 1>), gh, bh, lds, st, a);
    return hipGetLastError();
}

__device__ __forceinline__ int rl32(int v, int k) { return __builtin_amdgcn_readlane(v, k); }
// A pointer every lane holds, marked wave-uniform (scalar registers), so that stores through
// it can take a 32-bit per-lane offset.
template <typename T>
__device__ __forceinline__ NNPS_GLOBAL T* uniform_ptr(NNPS_GLOBAL T* p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
    return (NNPS_GLOBAL T*)((static_cast<uint64_t>(hi) << 32) | lo);
}
__device__ __forceinline__ long long rl64(long long v, int k)
{
    const int lo = __builtin_amdgcn_readlane(static_cast<int>(v & 0xFFFFFFFF), k);
    const int hi = __builtin_amdgcn_readlane(static_cast<int>(v >> 32), k);
    return (static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo);
}
__device__ __forceinline__ double rlf64(double v, int k)
{
    return __builtin_bit_cast(double, rl64(__builtin_bit_cast(long long, v), k));
}

// ---------------------------------------------------------------------------
// Dense-cell path. A work unit is up to kDenseUnit targets of one dense cell (the count and
// the testing fill take kDenseSlice at a time, with the first of their units), all with
// the same stencil union (the cell's list, ascending original index); persistent workgroups
// take units from a counter.
//
// Count: four wavefronts of 64 targets each against the list in chunks of kDenseChunk, whose
// MFMA operands the wavefronts prepare once and share through LDS (see k_count: the same
// contraction, about the cell's centre; binary64 outside the FP16 RCLL mode). The accepted
// bits of every (target, chunk) are kept when the buffer holds them. What bounds it: vector
// issue, 1.7 instructions per 64 pairs (the packed-FP16 count took 2.36 ms per
// launch on 422 thousand clustered particles, 2.2 G candidates; this 0.41).
//
// Fill: it takes the kept bits, or (no room for them) tests again with packed FP16 (or in
// binary64) and an FP64 recheck. For each chunk the workgroup stages the candidates' indices and
// positions (in quanta, or binary64) in LDS, then each wavefront runs its targets one at a time
// over the chunk. Lane L holds a contiguous run of the chunk's candidates, so a target's accepted
// ones come out lane by lane in row order: one wavefront prefix sum of the lanes' counts
// places them, they are queued per lane and written 64 at a time, so consecutive lanes store
// consecutive CSR entries and the row comes out ascending.
// Wavefront w of a unit's W holds targets w, w + W, ...: lane k keeps target w + W k's data
// in registers, read by the whole wavefront with readlane when its turn comes.
constexpr int kNotSeen = 1 << 30;  // a target whose own place in the union has not come yet

__device__ __forceinline__ bool dense_bits_fit(const SearchArgs& a, int nunits)
{
    return a.dbits && nunits > 0 && a.dboff[a.L.ncell_tot] * 64 <= a.dbits_cap;
}

template <int DIM, int P, bool HALF>
__global__ void __launch_bounds__(kDenseThreads) __attribute__((amdgpu_waves_per_eu(4)))
k_dense_count(SearchArgs a)
{
    using T = Tiles<DIM, P>;
    using Frag = typename T::Frag;
    constexpr int K = kDenseChunk, NW = kDenseThreads / 64, NS = K / 64;
    static_assert(kDenseSlice == 64 * NW && sizeof(Frag) == 32, "a wavefront per 64 targets; operands of 32 bytes");
    __shared__ uint4 sfrag[NS][2][64];  // the chunk's operands, 64 candidates a step
    __shared__ int slist[K];            // its sorted positions
    __shared__ int sself[kDenseSlice];  // the targets' own places in the union
    __shared__ int s_unit;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nunits = *a.dn > 0 ? a.unit_off[a.L.ncell_tot] : 0;
    const bool bits = dense_bits_fit(a, nunits);
    const int mi = T::item(lane);
    for (;;) {
        __syncthreads();  // the previous unit is done with the shared tables
        if (tid == 0) s_unit = atomicAdd(a.flags + kFlagUnit, 1);
        __syncthreads();
        const int u = __builtin_amdgcn_readfirstlane(s_unit);
        if (u >= nunits) break;
        const int c = __builtin_amdgcn_readfirstlane(a.ucell[u]);
        const int slice = u - __builtin_amdgcn_readfirstlane(a.unit_off[c]);
        if (slice % (kDenseSlice / kDenseUnit)) continue;  // with the unit that starts its 256 targets
        const SetDesc& sd = a.L.sets[__builtin_amdgcn_readfirstlane(find_set(a.L.coffs, a.L.nsets, c))];
        const int ncx = sd.fr.nc[0], ncy = sd.fr.nc[1];
        const int lk = c - sd.coff, row = lk / ncx;
        const int u0 = __builtin_amdgcn_readfirstlane(a.cell_start[c]) + slice * kDenseUnit;
        const int u1 = min(__builtin_amdgcn_readfirstlane(a.cell_start[c + 1]), u0 + kDenseSlice);
        const int U = __builtin_amdgcn_readfirstlane(a.usz[c]);
        const int* list = a.ulist + a.uoff[c];
        const int nchunk = (U + K - 1) / K;
        // the wavefront's targets, tests about the cell's centre
        BlockGeom<DIM> g;
        g.sd = &sd;
        g.xa = g.xb = lk - row * ncx;
        g.y0 = row % ncy;
        g.z0 = row / ncy;
        g.p0 = min(u0 + 64 * wv, u1);
        g.p1 = min(u0 + 64 * wv + 64, u1);
        const int nt = g.p1 - g.p0;
        const int pt = nt > 0 ? g.p0 + min(lane, nt - 1) : u0;
        const double R2 = sd.fr.R2;
        T tiles;
        if constexpr (P == 64) {
            // one origin for the workgroup, whose wavefronts share the candidates' operands
            tiles.targets_about(T::fetch(a, pt), T::fetch(a, u0), g);
        } else {
            tiles.targets(T::fetch(a, pt), g);
        }
        for (int t = tid; t < kDenseSlice; t += kDenseThreads) sself[t] = kNotSeen;
        int cnt = 0;
        for (int c0 = 0; c0 < U; c0 += K) {
            const int nc = min(K, U - c0), ns = (nc + 63) >> 6;
            __syncthreads();
            for (int s = wv; s < ns; s += NW) {
                const int e = 64 * s + mi;
                const int j = list[c0 + min(e, nc - 1)];
                const Frag f = tiles.prepare(T::fetch(a, j), g, e >= nc);
                uint4 q[2];
                __builtin_memcpy(q, &f, sizeof(f));
                sfrag[s][0][lane] = q[0];
                sfrag[s][1][lane] = q[1];
                if (e < nc) {
                    slist[e] = j;
                    if (j >= u0 && j < u1) sself[j - u0] = c0 + e;
                }
            }
            __syncthreads();
            if (nt == 0) continue;
            const int self = sself[64 * wv + lane] - c0;
            uint4* out = nullptr;
            if (bits)
                out = reinterpret_cast<uint4*>(a.dbits + (a.dboff[c] + static_cast<int64_t>(pt - a.cell_start[c]) * nchunk +
                                                          c0 / K) * 64);
            // four steps' words go out together (32 bytes a target)
#pragma unroll 1
            for (int sb = 0; sb < ns; sb += 4) {
                uint32_t w[8];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int s = sb + k;
                    w[2 * k] = w[2 * k + 1] = 0u;
                    if (s >= ns) continue;
                    auto decide = [&](uint32_t bnd, uint32_t acc, int e0, int t) -> uint32_t {
                        const double* pi = a.spos + static_cast<size_t>(g.p0 + min(t, nt - 1)) * 4;
                        while (bnd) {
                            const int r = __builtin_ctz(bnd);
                            bnd &= bnd - 1u;
                            const int e = 64 * s + e0 + r;
                            const bool in = e < nc && recheck_sorted<DIM>(a.spos, pi, slist[e], R2);
                            acc = (acc & ~(1u << r)) | (static_cast<uint32_t>(in) << r);
                        }
                        return acc;
                    };
                    const uint4 q[2] = {sfrag[s][0][lane], sfrag[s][1][lane]};
                    Frag f;
                    __builtin_memcpy(&f, q, sizeof(f));
                    const u32x2 ww = tiles.words(f, g, decide);
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        // the target itself is no neighbour; half lists keep larger original indices
                        const int d = self - 64 * s - 32 * h;
                        uint32_t word = ww[h];
                        if (HALF) word &= d < 0 ? ~0u : (d >= 31 ? 0u : 0xFFFFFFFEu << d);
                        else word &= (d >= 0 && d < 32) ? ~(1u << d) : ~0u;
                        cnt += __builtin_popcount(word);
                        w[2 * k + h] = word;
                    }
                }
                if (bits && lane < nt) {
                    out[sb >> 1] = make_uint4(w[0], w[1], w[2], w[3]);
                    out[(sb >> 1) + 1] = make_uint4(w[4], w[5], w[6], w[7]);
                }
            }
        }
        if (lane < nt) a.counts[a.perm[g.p0 + lane]] = cnt;
    }
}

// The fill that takes the count's bits. Sixteen wavefronts share the staged candidates, as many
// as two workgroups per compute unit have room for: 4096 as 16-byte records in quanta (see
// k_fill), 2048 in binary64. A wavefront takes a target's bits 1024 candidates at a time, one
// after the other, so that several KB of a row go out at once: rows lie far apart in the
// output, and with 1024 candidates staged at a time the pieces of about 0.8 KB cost DRAM
// efficiency (2.9 ms per launch for 4.6 GB of lists against 2.2; 1.4 with units of 64 targets).
template <int DIM, bool F64>
__global__ void __launch_bounds__(kDenseFillThreads) __attribute__((amdgpu_waves_per_eu(8)))
k_dense_fill(SearchArgs a)
{
    constexpr int NW = kDenseFillThreads / 64, QCAP = kDenseFillQueue;
    constexpr int NSUB = F64 ? 2 : 4, K = NSUB * kDenseChunk;
    constexpr int GT = 8 / NSUB;  // targets whose bits are loaded together
    __shared__ int4 srec[F64 ? 1 : K];            // position, set-local index
    __shared__ double sdbl[F64 ? K * DIM : 1];    // [K][DIM]
    __shared__ int sorig[F64 ? K : 1];
    __shared__ uint16_t squeue[NW * QCAP];        // per wavefront: accepted candidates, in row order
    __shared__ int s_unit;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nunits = *a.dn > 0 ? a.unit_off[a.L.ncell_tot] : 0;
    if (!dense_bits_fit(a, nunits)) return;
    uint16_t* const queue = squeue + wv * QCAP;
    for (;;) {
        __syncthreads();  // the previous unit is done with the shared tables
        if (tid == 0) s_unit = atomicAdd(a.flags + kFlagUnit, 1);
        __syncthreads();
        const int u = __builtin_amdgcn_readfirstlane(s_unit);
        if (u >= nunits) break;
        const int c = __builtin_amdgcn_readfirstlane(a.ucell[u]);
        const int slice = u - __builtin_amdgcn_readfirstlane(a.unit_off[c]);
        const NNPS_CONST SetDesc& sd =
            ((const NNPS_CONST SetDesc*)a.L.sets)[__builtin_amdgcn_readfirstlane(find_set(a.L.coffs, a.L.nsets, c))];
        const int poff = sd.poff;
        const double inv_quantum = sd.fr.inv_quantum;
        const float quantum = sd.fr.quantum, near2 = sd.fr.near2;
        const double lo[3] = {sd.fr.lo[0], sd.fr.lo[1], sd.fr.lo[2]};
        const int64_t cap = sd.capacity;
        const int u0 = __builtin_amdgcn_readfirstlane(a.cell_start[c]) + slice * kDenseUnit;
        const int u1 = min(__builtin_amdgcn_readfirstlane(a.cell_start[c + 1]), u0 + kDenseUnit);
        const int U = __builtin_amdgcn_readfirstlane(a.usz[c]);
        const int* list = a.ulist + a.uoff[c];
        const int nchunk = (U + kDenseChunk - 1) / kDenseChunk;
        const uint16_t* rows = a.dbits + (a.dboff[c] + static_cast<int64_t>(slice * kDenseUnit + wv) * nchunk) * 64 + lane;
        auto packed = [&](const double2& xy, const double2& zw, int w) {
            return make_int4(in_quanta(xy.x, lo[0], inv_quantum), in_quanta(xy.y, lo[1], inv_quantum),
                             DIM == 3 ? in_quanta(zw.x, lo[2], inv_quantum) : 0, w);
        };
        // this lane's target (held for the wavefront): targets wv, wv + NW, ... of the unit
        const int pk = u0 + wv + NW * lane;
        const int nt = u1 - u0 > wv ? (u1 - u0 - wv + NW - 1) / NW : 0;
        int rl_k = 0, acc_k = 0;
        long long rs_k = 0;
        int4 t_k = make_int4(0, 0, 0, 0);
        double pi_k[3] = {0, 0, 0};
        if (pk < u1) {
            const double2* r = reinterpret_cast<const double2*>(a.spos + static_cast<size_t>(pk) * 4);
            const double2 xy = r[0], zw = r[1];
            const int li = static_cast<int>(__builtin_bit_cast(int64_t, zw.y)) - poff;
            rs_k = sd.row_ptr[li];
            rl_k = static_cast<int>(sd.row_ptr[li + 1] - rs_k);
            if (F64) {
                pi_k[0] = xy.x;
                pi_k[1] = xy.y;
                pi_k[2] = zw.x;
            } else {
                t_k = packed(xy, zw, 0);
            }
        }
        for (int c0 = 0; c0 < U; c0 += K) {
            const int nc = min(K, U - c0), nsub = (nc + kDenseChunk - 1) / kDenseChunk;
            uint32_t inside[NSUB];  // this lane's candidates of each 1024 that the list has
#pragma unroll
            for (int q = 0; q < NSUB; ++q) inside[q] = first_bits(nc - q * kDenseChunk - 16 * lane);
            __syncthreads();
            for (int e = tid; e < nc; e += kDenseFillThreads) {
                const double2* r = reinterpret_cast<const double2*>(a.spos + static_cast<size_t>(list[c0 + e]) * 4);
                const double2 xy = r[0], zw = r[1];
                const int oj = static_cast<int>(__builtin_bit_cast(int64_t, zw.y)) - poff;
                if (F64) {
                    sdbl[e * DIM] = xy.x;
                    sdbl[e * DIM + 1] = xy.y;
                    if (DIM == 3) sdbl[e * DIM + 2] = zw.x;
                    sorig[e] = oj;
                } else {
                    srec[e] = packed(xy, zw, oj);
                }
            }
            __syncthreads();
            for (int k0 = 0; k0 < nt; k0 += GT) {
                // the bits of GT targets, loaded together (waiting for a load also waits for
                // every store issued before it); lane L takes candidates 16 L ... of each 1024
                uint32_t wb[GT * NSUB];
#pragma unroll
                for (int t = 0; t < GT; ++t)
#pragma unroll
                    for (int q = 0; q < NSUB; ++q)
                        wb[t * NSUB + q] = rows[(static_cast<int64_t>(NW * min(k0 + t, nt - 1)) * nchunk +
                                                 min(c0 / kDenseChunk + q, nchunk - 1)) * 64];
#pragma unroll
                for (int t = 0; t < GT; ++t) {
                    const int k = k0 + t;
                    if (k >= nt) break;
                    const long long rs = rl64(rs_k, k);
                    const int rl = rl32(rl_k, k);
                    int done = rl32(acc_k, k);
                    const bool room = rs + rl <= cap;
                    const int4 ti = make_int4(rl32(t_k.x, k), rl32(t_k.y, k), rl32(t_k.z, k), 0);
                    double pi[3];
                    if (F64) {
#pragma unroll
                        for (int d = 0; d < 3; ++d) pi[d] = rlf64(pi_k[d], k);
                    }
                    // the row's output, wave-uniform: entries are addressed by a 32-bit slot
                    NNPS_GLOBAL int32_t* const rcol = uniform_ptr((NNPS_GLOBAL int32_t*)sd.col + rs);
                    NNPS_GLOBAL float* const rdist = uniform_ptr((NNPS_GLOBAL float*)sd.dist + rs);
#pragma unroll
                    for (int q = 0; q < NSUB; ++q) {
                        if (q >= nsub) break;
                        const int lb = q * kDenseChunk + 16 * lane;  // the lane's first candidate
                        const uint32_t M = wb[t * NSUB + q] & inside[q];
                        int tot;
                        const int base = wave_excl_scan_i32(__builtin_popcount(M), &tot);
                        // accepted candidates queued per lane, as many as the queue holds at a
                        // time, then written 64 at a time with all lanes active
                        for (int w0 = 0; w0 < tot; w0 += QCAP) {
                            int pos = base - w0;
                            for (uint32_t mm = M; mm; mm &= mm - 1, ++pos)
                                if (static_cast<unsigned>(pos) < static_cast<unsigned>(QCAP))
                                    queue[pos] = static_cast<uint16_t>(lb + __builtin_ctz(mm));
                            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                            const int n = min(QCAP, tot - w0);
                            for (int i = lane; i < n; i += 64) {
                                const int e = queue[i], slot = done + w0 + i;  // a staged candidate (see inside)
                                float dv;
                                int oj;
                                if constexpr (F64) {
                                    oj = sorig[e];
                                    dv = dist_fp64<DIM>(pi, sdbl + e * DIM);
                                } else {
                                    const int4 r = srec[e];
                                    oj = r.w;
                                    const float s2 = quanta2<DIM>(ti, r);
                                    dv = root(s2) * quantum;
                                    if (!(s2 >= near2))
                                        dv = dist_near<DIM>(a.spos + static_cast<size_t>(u0 + wv + NW * k) * 4,
                                                            (const double*)sd.pos + static_cast<size_t>(oj) * DIM,
                                                            inv_quantum, quantum);
                                }
                                if (slot < rl && room) {
                                    if (rl <= (1 << 30)) {  // byte offsets within the row fit 32 bits
                                        const uint32_t off = static_cast<uint32_t>(slot) * 4u;
                                        *(NNPS_GLOBAL int32_t*)((NNPS_GLOBAL char*)rcol + off) = oj;
                                        *(NNPS_GLOBAL float*)((NNPS_GLOBAL char*)rdist + off) = dv;
                                    } else {
                                        rcol[slot] = oj;
                                        rdist[slot] = dv;
                                    }
                                }
                            }
                            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                        }
                        done += tot;
                    }
                    if (!room && lane == 0 && rl > 0) atomicOr(a.flags + kFlagErr, kErrCapacity);
                    if (lane == k) acc_k = done;
                }
            }
        }
        if (pk < u1 && acc_k != rl_k) atomicOr(a.flags + kFlagErr, kErrLongRow);
    }
}

// Statistics of the dense cells decided in binary64: candidates and rows.
__global__ void __launch_bounds__(kDenseThreads)
k_dense_stats64(SearchArgs a)
{
    __shared__ unsigned long long sh[2][kDenseThreads / 64];
    unsigned long long cand = 0, rows = 0;
    const bool on = *a.dn > 0;
    for (int c = blockIdx.x * kDenseThreads + threadIdx.x; on && c < a.L.ncell_tot; c += gridDim.x * kDenseThreads) {
        const int U = a.usz[c];
        if (U == 0) continue;
        const unsigned long long occ = static_cast<unsigned long long>(a.cell_start[c + 1] - a.cell_start[c]);
        rows += occ;
        cand += occ * static_cast<unsigned long long>(U - 1);
    }
    cand = wave_sum_u64(cand);
    rows = wave_sum_u64(rows);
    if ((threadIdx.x & 63) == 0) {
        sh[0][threadIdx.x >> 6] = cand;
        sh[1][threadIdx.x >> 6] = rows;
    }
    __syncthreads();
    if (threadIdx.x < kDenseStats) {
        unsigned long long v = 0;
        if (threadIdx.x == 0 || threadIdx.x == 5)
            for (int w = 0; w < kDenseThreads / 64; ++w) v += sh[threadIdx.x == 5 ? 1 : 0][w];
        a.dstats[static_cast<size_t>(blockIdx.x) * kDenseStats + threadIdx.x] = v;
    }
}

// The fill that tests the candidates itself, and the packed-FP16 statistics (FILL false:
// nothing but dstats is written).
template <int DIM, int MODE, bool FILL>
__global__ void __launch_bounds__(kDenseThreads) __attribute__((amdgpu_waves_per_eu(4))) k_dense(SearchArgs a)
{
    constexpr int NTH = kDenseThreads;  // threads per workgroup
    constexpr int NWV = NTH / 64;       // wavefronts per workgroup
    constexpr bool F16 = MODE != 1;
    static_assert(FILL || F16, "the statistics are the FP16 test's");
    constexpr int K = F16 ? kDenseChunkF16 : kDenseChunk;
    constexpr int QCAP = kDenseQueue;
    static_assert(K % 128 == 0 && K <= 2048, "whole 128-candidate groups, chunk positions fit 16 bits");
    static_assert(QCAP >= 64 && K <= 65536, "a queue holds a full store; chunk positions fit 16 bits");
    static_assert(K / 64 <= 16, "a lane's accepted bits of a chunk fit 16 bits");
    __shared__ uint4 recA[F16 ? K / 2 : 1];             // qx, qy, qz, 2(c_x - c_jx) pairs
    __shared__ uint2 recB[F16 ? K / 2 : 1];             // 2(c_y - c_jy), 2(c_z - c_jz) pairs
    constexpr bool QUANTA = F16 && FILL;  // candidates as k_dense_fill stages them
    __shared__ int4 srec[QUANTA ? K : 1];               // position in quanta, set-local index
    __shared__ __attribute__((aligned(16))) int sorig[QUANTA ? 1 : K];
    __shared__ double spj[F16 ? 1 : K * DIM];           // FP64 positions, [K][DIM]
    __shared__ unsigned long long s_red[FILL ? 1 : kDenseThreads / 64][kDenseStats];  // count pass only
    // fill: per-wavefront queues of a row's accepted candidates in a chunk (chunk positions,
    // in row order)
    __shared__ uint16_t squeue[FILL ? NWV * QCAP : 1];
    // fill: each target's position in the union (found while staging; kNotSeen before)
    __shared__ int sself[FILL ? kDenseSlice : 1];
    // the unit counter's broadcast slot: the first record word, free between the last use of
    // one unit's staged chunk and the staging of the next unit's first chunk
    int* const s_unit = reinterpret_cast<int*>(recA);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int nunits = *a.dn > 0 ? a.unit_off[a.L.ncell_tot] : 0;
    // the count keeps the accepted bits of every (target, chunk) when they fit, and the fill
    // then takes them instead of testing again. The host launches both fills; the one that
    // does not apply returns here.
    if (FILL && dense_bits_fit(a, nunits)) return;
    unsigned long long tc[kDenseStats] = {0, 0, 0, 0, 0, 0};
    for (;;) {
        __syncthreads();  // the previous unit is done with s_unit and the staged chunk
        if (threadIdx.x == 0) *s_unit = atomicAdd(a.flags + kFlagUnit, 1);
        __syncthreads();
        const int u = *s_unit;
        if (u >= nunits) break;
        const int g = a.ucell[u];
        const int slice = u - a.unit_off[g];
        if (slice % (kDenseSlice / kDenseUnit)) continue;  // with the unit that starts its 256 targets
        const SetDesc& sdesc = a.L.sets[find_set(a.L.coffs, a.L.nsets, g)];
        const SetView sd(sdesc);
        const int poff = sd.poff;
        const double R2 = sdesc.fr.R2;
        const int ncx = sdesc.fr.nc[0], ncy = sdesc.fr.nc[1];
        const uint32_t coff = static_cast<uint32_t>(sdesc.coff);
        const int lk = g - sdesc.coff;
        const int cx = lk % ncx, crow = lk / ncx, cy = crow % ncy, cz = crow / ncy;
        const int t0 = a.cell_start[g] + slice * kDenseUnit;
        const int t1 = min(a.cell_start[g + 1], t0 + kDenseSlice);
        const int U = a.usz[g];
        const int64_t ub = a.uoff[g];
        Thresh th;
        th.init(sdesc.fr);
        const uint16_t tmid = sdesc.fr.t_mid;
        // this lane's target (held for the wavefront)
        const int pk = t0 + wv + NWV * lane;
        const bool vk = pk < t1;
        const int nt = (t1 - t0 > wv) ? (t1 - t0 - wv + NWV - 1) / NWV : 0;
        int oi_k = 0, q01_k = 0, q2_k = 0, acc_k = 0, rl_k = 0;
        long long rs_k = 0;
        double pi_k[3] = {0, 0, 0};
        int4 t_k = make_int4(0, 0, 0, 0);
        const double inv_quantum = sdesc.fr.inv_quantum;
        const float quantum = sdesc.fr.quantum, near2 = sdesc.fr.near2;
        const double lo[3] = {sdesc.fr.lo[0], sdesc.fr.lo[1], sdesc.fr.lo[2]};
        auto packed = [&](const double* x, int w) {
            return make_int4(in_quanta(x[0], lo[0], inv_quantum), in_quanta(x[1], lo[1], inv_quantum),
                             DIM == 3 ? in_quanta(x[2], lo[2], inv_quantum) : 0, w);
        };
        if (vk) {
            oi_k = a.perm[pk];
            const int li = oi_k - poff;
#pragma unroll
            for (int k = 0; k < DIM; ++k) pi_k[k] = a.spos[static_cast<size_t>(pk) * 4 + k];
            if (QUANTA) t_k = packed(pi_k, 0);
            if (F16) {
                const ushort4 q = q16_of(a.rq[pk]);
                q01_k = static_cast<int>(static_cast<uint32_t>(q.x) | (static_cast<uint32_t>(q.y) << 16));
                q2_k = static_cast<int>(q.z);
            }
            if (FILL) {
                rs_k = sd.row_ptr[li];
                rl_k = static_cast<int>(sd.row_ptr[li + 1] - rs_k);
            } else {
                tc[0] += static_cast<unsigned long long>(U - 1);
                tc[5] += 1;
            }
        }
        if (FILL) {
            for (int t = threadIdx.x; t < kDenseSlice; t += NTH) sself[t] = kNotSeen;
        }
        for (int c0 = 0; c0 < U; c0 += K) {
            const int nc = min(K, U - c0);
            // lane L tests the chunk's candidates 2 L nit ... 2 (L + 1) nit - 1, pair by pair
            // (pair L nit + it at iteration it), so a target's accepted candidates come out
            // in order lane by lane
            const int nit = (nc + 127) >> 7;
            __syncthreads();
            // stage the chunk (padding tests as +inf / far away: never a neighbour)
            if constexpr (F16) {
                // pair m goes to record slot (m mod nit) 64 + m / nit: the test reads slot
                // it 64 + lane, consecutive lanes, at iteration it
                for (int m = threadIdx.x; m < 64 * nit; m += NTH) {
                    uint32_t w0 = 0, w1 = 0, w2 = 0, w3 = 0, w4 = 0, w5 = 0;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int e = 2 * m + h;
                        const uint32_t sh = 16u * h;
                        if (e < nc) {
                            const int j = a.ulist[ub + c0 + e];
                            const ushort4 v = q16_of(a.rq[j]);
                            const uint32_t kj = a.skey[j] - coff;
                            const int xj = static_cast<int>(kj % static_cast<uint32_t>(ncx));
                            const uint32_t rj = kj / static_cast<uint32_t>(ncx);
                            const int yj = static_cast<int>(rj % static_cast<uint32_t>(ncy));
                            const int zj = static_cast<int>(rj / static_cast<uint32_t>(ncy));
                            const _Float16 c2x = static_cast<_Float16>(2 * (cx - xj));
                            const _Float16 c2y = static_cast<_Float16>(2 * (cy - yj));
                            const _Float16 c2z = static_cast<_Float16>(2 * (cz - zj));
                            w0 |= static_cast<uint32_t>(v.x) << sh;
                            w1 |= static_cast<uint32_t>(v.y) << sh;
                            w2 |= static_cast<uint32_t>(v.z) << sh;
                            w3 |= static_cast<uint32_t>(__builtin_bit_cast(uint16_t, c2x)) << sh;
                            w4 |= static_cast<uint32_t>(__builtin_bit_cast(uint16_t, c2y)) << sh;
                            w5 |= static_cast<uint32_t>(__builtin_bit_cast(uint16_t, c2z)) << sh;
                            const int oj = a.perm[j];
                            if constexpr (QUANTA) {
                                srec[e] = packed(a.spos + static_cast<size_t>(j) * 4, oj - poff);
                                if (j >= t0 && j < t1) sself[j - t0] = c0 + e;  // a target of this unit
                            } else {
                                sorig[e] = oj;
                            }
                        } else {
                            w0 |= 0x7C00u << sh;  // qx = +inf: r2 = +inf
                            if (QUANTA) srec[e].w = -1 - poff;
                            else sorig[e] = -1;
                        }
                    }
                    const int slot = (m % nit) * 64 + m / nit;
                    recA[slot] = make_uint4(w0, w1, w2, w3);
                    recB[slot] = make_uint2(w4, w5);
                }
            } else {
                for (int e = threadIdx.x; e < K; e += NTH) {
                    if (e < nc) {
                        const int j = a.ulist[ub + c0 + e];
                        sorig[e] = a.perm[j];
                        if (FILL && j >= t0 && j < t1) sself[j - t0] = c0 + e;  // a target of this unit
#pragma unroll
                        for (int k = 0; k < DIM; ++k) spj[e * DIM + k] = a.spos[static_cast<size_t>(j) * 4 + k];
                    } else {
                        sorig[e] = -1;
#pragma unroll
                        for (int k = 0; k < DIM; ++k) spj[e * DIM + k] = __builtin_nan("");  // never a neighbour
                    }
                }
            }
            __syncthreads();
            // original index of candidate e
            auto orig_of = [&](int e) { return QUANTA ? srec[e].w + poff : sorig[e]; };
            // the fill's emission of target k's accepted candidates in this chunk: bit j of
            // M is the lane's candidate 2 lane nit + j
            auto fill_row = [&](int k, uint32_t M, const double* pi) {
                // ascending emission: candidate order is original-index order and a lane
                // holds a contiguous run of it, so a lane's accepted candidates go to the row's
                // slots after those of the lanes below it (a wave prefix of the lanes' counts).
                // They pass through the wavefront's queue in LDS, where each lane writes its
                // own in order; then lane i takes entries i, i + 64, ..., computes their
                // distances and writes them, so every store covers 64 consecutive slots with
                // all lanes active
                const long long rs = rl64(rs_k, k);
                const int rl = rl32(rl_k, k);
                const int done = rl32(acc_k, k);
                const bool room = rs + rl <= sd.capacity;
                const int4 ti = make_int4(rl32(t_k.x, k), rl32(t_k.y, k), rl32(t_k.z, k), 0);
                // the row's output, wave-uniform: entries are addressed by a 32-bit slot
                NNPS_GLOBAL int32_t* const rcol = uniform_ptr(sd.col + rs);
                NNPS_GLOBAL float* const rdist = uniform_ptr(sd.dist + rs);
                auto emit = [&](int e, int slot) {
                    int lj;
                    float dv;
                    if constexpr (QUANTA) {  // as k_dense_fill
                        const int4 r = srec[e];
                        lj = r.w;
                        const float s2 = quanta2<DIM>(ti, r);
                        dv = root(s2) * quantum;
                        if (!(s2 >= near2))
                            dv = dist_near<DIM>(a.spos + static_cast<size_t>(t0 + wv + NWV * k) * 4,
                                                a.spos + static_cast<size_t>(a.ulist[ub + c0 + e]) * 4, inv_quantum, quantum);
                    } else {
                        lj = sorig[e] - poff;
                        dv = dist_fp64<DIM>(pi, spj + e * DIM);
                    }
                    if (slot < rl && room) {
                        if (rl <= (1 << 30)) {  // byte offsets within the row fit 32 bits
                            const uint32_t off = static_cast<uint32_t>(slot) * 4u;
                            *(NNPS_GLOBAL int32_t*)((NNPS_GLOBAL char*)rcol + off) = lj;
                            *(NNPS_GLOBAL float*)((NNPS_GLOBAL char*)rdist + off) = dv;
                        } else {
                            rcol[slot] = lj;
                            rdist[slot] = dv;
                        }
                    }
                };
                const int lb = 2 * lane * nit;  // the lane's first candidate
                // the target itself is never its own neighbour and half lists keep only
                // larger original indices: the union is in original-index order, so both
                // are a condition on the chunk position against the target's own, p
                const int p = sself[wv + NWV * k] - c0;
                const int d = p - lb;
                if (a.half) M &= d < 0 ? 0xFFFFu : (d >= 15 ? 0u : (0xFFFEu << d) & 0xFFFFu);
                else if (p >= 0 && p < nc && d >= 0 && d < 2 * nit) M &= ~(1u << d);
                int tot;
                const int base = wave_excl_scan_i32(__builtin_popcount(M), &tot);
                if (tot <= QCAP) {
                    uint16_t* const q = squeue + wv * QCAP;
                    int pos = base;
                    for (uint32_t mm = M; mm; mm &= mm - 1) q[pos++] = static_cast<uint16_t>(lb + __builtin_ctz(mm));
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                    for (int q0 = 0; q0 < tot; q0 += 64) {
                        if (q0 + lane < tot) emit(q[q0 + lane], done + q0 + lane);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                } else {
                    // more than the queue holds (a chunk with most candidates accepted): each
                    // lane writes its own entries
                    int pos = done + base;
                    for (uint32_t mm = M; mm; mm &= mm - 1) emit(lb + __builtin_ctz(mm), pos++);
                }
                const int w = done + tot;
                if (!room && lane == 0 && w > done) atomicOr(a.flags + kFlagErr, kErrCapacity);
                if (lane == k) acc_k = w;
            };
            {
                for (int k = 0; k < nt; ++k) {
                    const int oi = rl32(oi_k, k);
                    double pi[3] = {0.0, 0.0, 0.0};
                    // the FP16 test needs the target's FP64 position only for a band recheck
                    if (!F16) {
#pragma unroll
                        for (int d = 0; d < 3; ++d) pi[d] = rlf64(pi_k[d], k);
                    }
                    uint32_t inb = 0, bnd = 0;
                    {
                        h2 qix2, qiy2, qiz2;
                        if (F16) {
                            const uint32_t q01 = static_cast<uint32_t>(rl32(q01_k, k));
                            const uint32_t q2 = static_cast<uint32_t>(rl32(q2_k, k));
                            qix2 = splat(as_f16(static_cast<uint16_t>(q01 & 0xFFFF)));
                            qiy2 = splat(as_f16(static_cast<uint16_t>(q01 >> 16)));
                            qiz2 = splat(as_f16(static_cast<uint16_t>(q2 & 0xFFFF)));
                        }
                        // candidate bits: bit it for candidate 2 (lane nit + it), bit 16 + it for the
                        // one after it; "in" and "in or band" from the sign bits of two 16-bit
                        // subtractions
                        uint32_t ebits = 0;
#pragma unroll
                        for (int it = 0; it < K / 128; ++it) {
                            if (it >= nit) break;
                            const int m = it * 64 + lane;  // record slot of pair lane nit + it
                            const int e0 = 2 * (lane * nit + it);
                            if (F16) {
                                const uint4 A = recA[m];
                                const uint2 B = recB[m];
                                const h2 s = qix2 - as_h2(A.x);
                                const h2 tx = s + as_h2(A.w);
                                const h2 ay = qiy2 + as_h2(B.x);
                                const h2 ty = ay - as_h2(A.y);
                                h2 r2;
                                if (DIM == 3) {
                                    const h2 az = qiz2 + as_h2(B.y);
                                    const h2 tz = az - as_h2(A.z);
                                    r2 = tz * tz;
                                    r2 = __builtin_elementwise_fma(ty, ty, r2);
                                } else {
                                    r2 = ty * ty;
                                }
                                r2 = __builtin_elementwise_fma(tx, tx, r2);
                                const u16x2 dd = as_u16x2(as_u32(r2)) - th.tlo2;
                                const u16x2 ee = dd - th.w12;
                                inb |= (u16x2_bits(dd) >> (15 - it)) & (0x10001u << it);
                                ebits |= (u16x2_bits(ee) >> (15 - it)) & (0x10001u << it);
                            } else {
#pragma unroll
                                for (int h = 0; h < 2; ++h)
                                    if (r2_fp64<DIM>(pi, spj + (e0 + h) * DIM) <= R2) inb |= 1u << (it + 16 * h);
                            }
                        }
                        bnd = ebits & ~inb;
                        // the FP64 recheck of candidate e
                        auto recheck = [&](int e) -> bool {
                            double pt[3];
#pragma unroll
                            for (int d = 0; d < 3; ++d) pt[d] = rlf64(pi_k[d], k);
                            return recheck_sorted<DIM>(a.spos, pt, a.ulist[ub + c0 + e], R2);
                        };
                        if (MODE == 2) {
                            // every candidate decided in FP64; the FP16 classes are only compared
                            uint32_t all = 0;
                            for (int it = 0; it < nit; ++it) {
                                const int e0 = 2 * (lane * nit + it);
                                all |= (e0 < nc ? 1u << it : 0u) | (e0 + 1 < nc ? 1u << (16 + it) : 0u);
                            }
                            uint32_t dec = 0;
                            while (all) {
                                const int bb = __builtin_ctz(all);
                                all &= all - 1;
                                const int e = 2 * (lane * nit + (bb & 15)) + (bb >> 4);
                                const int oj = orig_of(e);
                                if (oj == oi) continue;
                                const bool truth = recheck(e);
                                if (truth) dec |= 1u << bb;
                                if (!FILL) {
                                    const bool band = (bnd >> bb) & 1u;
                                    const bool in16 = (inb >> bb) & 1u;
                                    // naive FP16 test: r2 <= RN16(4 rho^2), from the staged record
                                    const uint4 A = recA[(bb & 15) * 64 + lane];
                                    const uint2 B = recB[(bb & 15) * 64 + lane];
                                    const h2 s = qix2 - as_h2(A.x);
                                    const h2 tx = s + as_h2(A.w);
                                    const h2 ty = (qiy2 + as_h2(B.x)) - as_h2(A.y);
                                    h2 r2;
                                    if (DIM == 3) {
                                        const h2 tz = (qiz2 + as_h2(B.y)) - as_h2(A.z);
                                        r2 = tz * tz;
                                        r2 = __builtin_elementwise_fma(ty, ty, r2);
                                    } else {
                                        r2 = ty * ty;
                                    }
                                    r2 = __builtin_elementwise_fma(tx, tx, r2);
                                    const uint16_t r2h = static_cast<uint16_t>((as_u32(r2) >> (16 * (e & 1))) & 0xFFFF);
                                    const bool naive = r2h <= tmid;
                                    tc[1] += band;
                                    tc[2] += naive && !truth;
                                    tc[3] += !naive && truth;
                                    tc[4] += !band && (in16 != truth);
                                }
                            }
                            inb = dec;
                        } else if (MODE == 0) {
                            uint32_t bb_all = bnd;
                            while (bb_all) {
                                const int bb = __builtin_ctz(bb_all);
                                bb_all &= bb_all - 1;
                                const int e = 2 * (lane * nit + (bb & 15)) + (bb >> 4);
                                const int oj = orig_of(e);
                                if (oj == oi) continue;  // itself (a band pair only when T_lo = 0)
                                const bool truth = recheck(e);
                                if (truth) inb |= 1u << bb;
                                if (!FILL) {
                                    const uint4 A = recA[(bb & 15) * 64 + lane];
                                    const uint2 B = recB[(bb & 15) * 64 + lane];
                                    const h2 s = qix2 - as_h2(A.x);
                                    const h2 tx = s + as_h2(A.w);
                                    const h2 ty = (qiy2 + as_h2(B.x)) - as_h2(A.y);
                                    h2 r2;
                                    if (DIM == 3) {
                                        const h2 tz = (qiz2 + as_h2(B.y)) - as_h2(A.z);
                                        r2 = tz * tz;
                                        r2 = __builtin_elementwise_fma(ty, ty, r2);
                                    } else {
                                        r2 = ty * ty;
                                    }
                                    r2 = __builtin_elementwise_fma(tx, tx, r2);
                                    const uint16_t r2h = static_cast<uint16_t>((as_u32(r2) >> (16 * (e & 1))) & 0xFFFF);
                                    const bool naive = r2h <= tmid;
                                    tc[1] += 1;
                                    tc[2] += naive && !truth;
                                    tc[3] += !naive && truth;
                                }
                            }
                        }
                    }
                    if constexpr (FILL) fill_row(k, interleave8(inb), pi);
                }
            }
        }
        if (FILL && vk && acc_k != rl_k) atomicOr(a.flags + kFlagErr, kErrLongRow);
    }
    if (!FILL) {
#pragma unroll
        for (int k = 0; k < kDenseStats; ++k) {
            const unsigned long long sum = wave_sum_u64(tc[k]);
            if (lane == 0) s_red[wv][k] = sum;
        }
        __syncthreads();
        if (threadIdx.x < kDenseStats) {
            unsigned long long sum = 0;
            for (int w = 0; w < kDenseThreads / 64; ++w) sum += s_red[w][threadIdx.x];
            a.dstats[static_cast<size_t>(blockIdx.x) * kDenseStats + threadIdx.x] = sum;
        }
    }
}

// Recheck-all: the decisions of the FP16 mode's matrix tiles, made over the counted structure and
// each compared with the binary64 predicate. A result within the bound is decided by the predicate
// itself; one outside it that is wrong counts as a disagreement. One wavefront per 64 targets, every
// pair of a target and a candidate (at(e) its sorted position) of the union's U.
template <int DIM, typename At>
__device__ __forceinline__ unsigned long long tile_disagreements(const SearchArgs& a, const BlockGeom<DIM>& g, int U,
                                                                 At&& at)
{
    using T = Tiles<DIM, 16>;
    const int lane = threadIdx.x & 63, nt = g.p1 - g.p0, p = g.p0 + min(lane, nt - 1);
    const double R2 = g.sd->fr.R2;
    const double* pi = a.spos + static_cast<size_t>(p) * 4;
    T tiles;
    tiles.targets(T::fetch(a, p), g);
    unsigned long long wrong = 0;
    for (int c0 = 0; c0 < U; c0 += 64) {
        const int e = c0 + T::item(lane);
        const typename T::Frag f = tiles.prepare(T::fetch(a, at(min(e, U - 1))), g, e >= U);
        // the row words with every result within the bound taken as out, and as in
        const u32x2 low = tiles.words(f, g, [](uint32_t bnd, uint32_t acc, int, int) { return acc & ~bnd; });
        const u32x2 high = tiles.words(f, g, [](uint32_t bnd, uint32_t acc, int, int) { return acc | bnd; });
        for (int j = 0; lane < nt && j < min(64, U - c0); ++j) {
            const int q = at(c0 + j);
            if (q == p) continue;
            const bool in = recheck_sorted<DIM>(a.spos, pi, q, R2);
            wrong += in ? !(high[j >> 5] >> (j & 31) & 1) : low[j >> 5] >> (j & 31) & 1;
        }
    }
    return wave_sum_u64(wrong);
}

// Added to the blocks' sums (after k_stats16).
template <int DIM>
__global__ void __launch_bounds__(64)
k_check_tiles(SearchArgs a)
{
    const int b = xcd_block(*a.nblk);
    if (b < 0 || dense_block(a, b)) return;
    BlockGeom<DIM> g;
    g.init(a, b);
    const unsigned long long wrong = tile_disagreements<DIM>(a, g, g.U, [&](int e) { return g.global_of_any(e); });
    if (threadIdx.x == 0) a.blk_stats[static_cast<size_t>(b) * 5 + 4] += wrong;
}

// Added to the dense path's sums (after k_dense).
template <int DIM>
__global__ void __launch_bounds__(64)
k_check_dense_tiles(SearchArgs a)
{
    const int nunits = *a.dn > 0 ? a.unit_off[a.L.ncell_tot] : 0;
    unsigned long long wrong = 0;
    for (int u = blockIdx.x; u < nunits; u += gridDim.x) {
        const int c = __builtin_amdgcn_readfirstlane(a.ucell[u]);
        const SetDesc& sd = a.L.sets[__builtin_amdgcn_readfirstlane(find_set(a.L.coffs, a.L.nsets, c))];
        const int ncx = sd.fr.nc[0], ncy = sd.fr.nc[1], lk = c - sd.coff, row = lk / ncx;
        BlockGeom<DIM> g;
        g.sd = &sd;
        g.xa = g.xb = lk - row * ncx;
        g.y0 = row % ncy;
        g.z0 = row / ncy;
        g.p0 = __builtin_amdgcn_readfirstlane(a.cell_start[c] + (u - a.unit_off[c]) * kDenseUnit);
        g.p1 = min(__builtin_amdgcn_readfirstlane(a.cell_start[c + 1]), g.p0 + kDenseUnit);
        const int* list = a.ulist + a.uoff[c];
        wrong += tile_disagreements<DIM>(a, g, __builtin_amdgcn_readfirstlane(a.usz[c]), [&](int e) { return list[e]; });
    }
    if (threadIdx.x == 0) a.dstats[static_cast<size_t>(blockIdx.x) * kDenseStats + 4] += wrong;
}

template <int D>
void launch_dense_count(const SearchArgs& a, hipStream_t st)
{
    const dim3 g(a.dgrid), b(kDenseThreads);
    const bool f16 = a.L.mode == 0;  // the others decide dense cells in binary64
    if (f16 && a.half) hipLaunchKernelGGL((k_dense_count<D, 16, true>), g, b, 0, st, a);
    else if (f16) hipLaunchKernelGGL((k_dense_count<D, 16, false>), g, b, 0, st, a);
    else if (a.half) hipLaunchKernelGGL((k_dense_count<D, 64, true>), g, b, 0, st, a);
    else hipLaunchKernelGGL((k_dense_count<D, 64, false>), g, b, 0, st, a);
}

// Both fills run, and the one that does not match whether the count kept its bits returns at
// once.
template <int D>
void launch_dense_fill(const SearchArgs& a, hipStream_t st)
{
    const dim3 g(a.dgrid), b(kDenseThreads), bb(kDenseFillThreads);
    if (a.L.mode == 0 || a.L.mode == 2) {
        if (a.dbits) hipLaunchKernelGGL((k_dense_fill<D, false>), g, bb, 0, st, a);
        if (a.L.mode == 0) hipLaunchKernelGGL((k_dense<D, 0, true>), g, b, 0, st, a);
        else hipLaunchKernelGGL((k_dense<D, 2, true>), g, b, 0, st, a);
    } else {
        if (a.dbits) hipLaunchKernelGGL((k_dense_fill<D, true>), g, bb, 0, st, a);
        hipLaunchKernelGGL((k_dense<D, 1, true>), g, b, 0, st, a);
    }
}

template <int D>
void launch_dense_stats(const SearchArgs& a, hipStream_t st)
{
    const dim3 g(a.dgrid), b(kDenseThreads);
    if (a.L.mode == 0) hipLaunchKernelGGL((k_dense<D, 0, false>), g, b, 0, st, a);
    else if (a.L.mode == 2) hipLaunchKernelGGL((k_dense<D, 2, false>), g, b, 0, st, a);
    else hipLaunchKernelGGL(k_dense_stats64, g, b, 0, st, a);
    if (a.L.mode == 2) hipLaunchKernelGGL(k_check_dense_tiles<D>, g, dim3(64), 0, st, a);
}

hipError_t launch_dense(const SearchArgs& a, DensePass pass, hipStream_t st)
{
    if (a.L.ntot == 0 || !a.wdense) return hipSuccess;
    if (pass == DensePass::kCount) {
        if (a.L.dim == 2) launch_dense_count<2>(a, st);
        else launch_dense_count<3>(a, st);
    } else if (pass == DensePass::kFill) {
        if (a.L.dim == 2) launch_dense_fill<2>(a, st);
        else launch_dense_fill<3>(a, st);
    } else {
        const hipError_t e = launch_fill_i32(a.flags + kFlagUnit, 1, 0, st);
        if (e != hipSuccess) return e;
        if (a.L.dim == 2) launch_dense_stats<2>(a, st);
        else launch_dense_stats<3>(a, st);
    }
    return hipGetLastError();
}

template <int DIM>
void launch_block_stats(const SearchArgs& a, const dim3& g, hipStream_t st)
{
    const int m = a.L.mode;
    if (m == 0) hipLaunchKernelGGL((k_stats16<DIM, 0>), g, dim3(64), 0, st, a);
    else if (m == 1) hipLaunchKernelGGL((k_stats64<DIM>), g, dim3(64), 0, st, a);
    else if (m == 2) hipLaunchKernelGGL((k_stats16<DIM, 2>), g, dim3(64), 0, st, a);
    else hipLaunchKernelGGL((k_stats32<DIM>), g, dim3(64), 0, st, a);
    if (m == 2) hipLaunchKernelGGL(k_check_tiles<DIM>, g, dim3(64), 0, st, a);
}

hipError_t launch_stats(const SearchArgs& a, int nblk_max, hipStream_t st)
{
    if (a.L.ntot == 0) return hipSuccess;
    if (nblk_max > 0) {
        if (a.L.dim == 2) launch_block_stats<2>(a, block_grid(nblk_max), st);
        else launch_block_stats<3>(a, block_grid(nblk_max), st);
    }
    const hipError_t e = launch_dense(a, DensePass::kStats, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_reduce_stats, dim3(1), dim3(1024), 0, st, a.blk_stats, a.nblk,
                       static_cast<const unsigned long long*>(a.dstats), a.dstats ? a.dgrid : 0, a.stats);
    return hipGetLastError();
}

}  // namespace nnps
