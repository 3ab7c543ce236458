// Cell build: FP64 cell assignment with a slot per particle in its cell, cell starts by a
// device-wide scan, a counting sort by cell, the FP16 relative-coordinate pack and the
// work-block table (the LDS radix sort serves the dense-cell lists).
//
// Paper: cell link list with cell size equal to the search radius (SPH method
// section, Fig. 3b); cell-relative coordinates (Eq. 5-6, Fig. 5); spatial sorting
// so that neighbouring threads work on neighbouring particles (Results, memory
// section and Table 6).
#include <algorithm>
#include <utility>

#include "build_kernels.h"

namespace nnps {

// ---------------------------------------------------------------------------
// Exact int64 -> float32 (one rounding) for |v| < 2^44: v = hi*2^20 + lo with
// hi exactly representable, lo < 2^20, and a single fused multiply-add rounds once.
__device__ __forceinline__ float exact_i64_to_f32(int64_t v)
{
    const int32_t hi = static_cast<int32_t>(v >> 20);
    const int32_t lo = static_cast<int32_t>(v & 0xFFFFF);
    return __builtin_fmaf(static_cast<float>(hi), 1048576.0f, static_cast<float>(lo));
}

// ---------------------------------------------------------------------------
// Fixed-point position of a coordinate: X = rint((p - lo) * 2^F / w) (round half to even; an
// integer below 2^52). The assignment takes the cell X >> F from it and the pack the
// relative coordinate; both compute it from the position (three operations) rather than
// pass it through memory.
__device__ __forceinline__ int64_t fixed_point(double p, double lo, double s)
{
    return static_cast<int64_t>(rint(__dmul_rn(__dsub_rn(p, lo), s)));
}

// A1: cell assignment in FP64: cell = X >> F, global key = coff + cx + ncx (cy +
// ncy cz). Positions outside [lo, hi] (or NaN) raise the domain flag and are treated as
// lo so every index stays in range. Each particle also takes a slot in its cell (the
// cell's count before it), which places it in the sort by cell: runs of consecutive lanes
// with the same cell take their slots with one atomic, in lane order.
// TABLE: atomics on one cell's count follow one another at about 15 ns, and a cell at a
// cluster's core holds thousands of particles. So a workgroup adds its runs up by cell in a
// hash table in LDS first and takes the slots of each cell it holds with one atomic: 85 -> 41 us
// on 422,000 clustered particles in random order, but 12 -> 18 on a million of a lattice, so it
// serves the builds that expect dense cells.
constexpr int kAssignThreads = 1024;
constexpr int kAssignTable = 2 * kAssignThreads;  // at most half full, so every probe ends

template <int DIM, bool TABLE>
__global__ void __launch_bounds__(TABLE ? kAssignThreads : 256)
k_assign(const SetDesc* __restrict__ sets, const int* __restrict__ poffs, int nsets, int ntot,
         uint32_t* __restrict__ key, int* __restrict__ slot, int* __restrict__ cell_count, int* __restrict__ err)
{
    __shared__ uint32_t hkey[TABLE ? kAssignTable : 1];
    __shared__ int hcnt[TABLE ? kAssignTable : 1];
    constexpr uint32_t kEmpty = 0xFFFFFFFFu;  // keys are below 2^31
    const int tid = threadIdx.x, i = blockIdx.x * blockDim.x + tid;
    const bool active = i < ntot;
    if (TABLE) {
        for (int e = tid; e < kAssignTable; e += kAssignThreads) {
            hkey[e] = kEmpty;
            hcnt[e] = 0;
        }
        __syncthreads();
    } else if (!active) {
        return;
    }
    bool bad = false;
    auto cell_of = [&](const SetDesc& sd) -> uint32_t {
        const Frame& fr = sd.fr;
        const int li = i - sd.poff;
        int64_t c[3] = {0, 0, 0};
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            double p = sd.pos[static_cast<size_t>(li) * DIM + k];
            if (!(p >= fr.lo[k] && p <= fr.hi[k])) {
                bad = true;
                p = fr.lo[k];
            }
            c[k] = fixed_point(p, fr.lo[k], fr.s) >> fr.F;
        }
        return static_cast<uint32_t>(sd.coff + c[0] + fr.nc[0] * (c[1] + fr.nc[1] * c[2]));
    };
    const int lane = tid & 63;
    int head = 0, h = 0, local = 0;
    if (active) {
        // a wavefront inside one set reads the set's fields with scalar loads
        const int s = find_set(poffs, nsets, i);
        const int s0 = __builtin_amdgcn_readfirstlane(s);
        const uint32_t kk = __all(s == s0) ? cell_of(sets[s0]) : cell_of(sets[s]);
        key[i] = kk;
        // the active lanes are a prefix of the wavefront (i = base + lane)
        const int prev = __shfl_up(static_cast<int>(kk), 1, 64);
        const uint64_t heads = __ballot(lane == 0 || static_cast<uint32_t>(prev) != kk);
        const int nact = __popcll(__ballot(1));
        const uint64_t upto = lane == 63 ? ~0ull : (2ull << lane) - 1ull;
        head = 63 - __clzll(heads & upto);  // first lane of this lane's run
        const uint64_t after = heads & ~upto;
        const int next = after ? __ffsll(static_cast<long long>(after)) - 1 : nact;
        if (!TABLE) {
            if (head == lane) local = atomicAdd(&cell_count[kk], next - lane);
            slot[i] = __shfl(local, head, 64) + (lane - head);
        } else if (head == lane) {
            h = static_cast<int>((kk * 2654435761u) >> (32 - __builtin_ctz(kAssignTable)));
            for (;;) {
                const uint32_t was = atomicCAS(&hkey[h], kEmpty, kk);
                if (was == kEmpty || was == kk) break;
                h = (h + 1) & (kAssignTable - 1);
            }
            local = atomicAdd(&hcnt[h], next - lane);
        }
        if (bad) atomicOr(err, kErrDomain);
    }
    if (!TABLE) return;
    __syncthreads();
    for (int e = tid; e < kAssignTable; e += kAssignThreads) {
        const int c = hcnt[e];
        if (c) hcnt[e] = atomicAdd(&cell_count[hkey[e]], c);
    }
    __syncthreads();
    if (active) slot[i] = __shfl(hcnt[h] + local, head, 64) + (lane - head);
}

// Fill an int32 array with a value (a kernel rather than a memset node, so the sequence
// can be captured in a graph).
__global__ void __launch_bounds__(256)
k_fill_i32(int* __restrict__ p, int64_t m, int v)
{
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < m;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// Device-wide exclusive scan (int32 in, TOut out) over tiles of kScanTile elements, four
// consecutive elements to a thread; out[m] receives the total. What a tile has to add is
// found in one of three ways:
//   kScanSelf    the workgroup sums the input before its tile itself: one launch, for up to
//                kScanSelfTiles tiles and an output apart from the input;
//   kScanFold    a launch before this one leaves the tile sums, the workgroup sums those
//                before its own: for up to kScanFoldTiles tiles;
//   kScanScanned the tile sums are scanned by a launch of their own in between.
// All three are bound by latency, not bandwidth: a launch in a graph takes 4.6 us however
// little it does, and 16 tiles read again are 4 loads in flight per thread.
constexpr int kScanThreads = 1024;
constexpr int kScanTile = kScanThreads * 4;
constexpr int64_t kScanSelfTiles = 16;
constexpr int64_t kScanFoldTiles = 1024;
enum ScanOffset { kScanSelf, kScanFold, kScanScanned };

__device__ __forceinline__ int64_t wave_incl_scan(int64_t v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    return v;
}

// Block-wide exclusive scan of one value per thread (kScanThreads threads); returns the
// exclusive prefix and the block total.
__device__ __forceinline__ int64_t block_excl_scan(int64_t v, int64_t* total, int64_t* sh /*[kScanThreads / 64]*/)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t inc = wave_incl_scan(v);
    if (lane == 63) sh[w] = inc;
    __syncthreads();
    int64_t base = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < kScanThreads / 64; ++k) {
        if (k < w) base += sh[k];
        tot += sh[k];
    }
    __syncthreads();
    *total = tot;
    return base + inc - v;
}

// Block-wide sum of one value per thread.
template <int THREADS>
__device__ __forceinline__ int64_t block_sum(int64_t v, int64_t* sh /*[THREADS / 64]*/)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    int64_t t = 0;
#pragma unroll
    for (int k = 0; k < THREADS / 64; ++k) t += sh[k];
    __syncthreads();
    return t;
}

// Four elements from idx (a multiple of 4; `in` is 16-byte aligned), zeros from m on.
template <typename T>
__device__ __forceinline__ void load4(const T* __restrict__ in, int64_t idx, int64_t m, T (&v)[4])
{
    static_assert(sizeof(T) == 4, "one 16-byte load");
    if (idx + 4 <= m) {
        const uint4 q = *reinterpret_cast<const uint4*>(in + idx);
        v[0] = static_cast<T>(q.x);
        v[1] = static_cast<T>(q.y);
        v[2] = static_cast<T>(q.z);
        v[3] = static_cast<T>(q.w);
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = idx + r < m ? in[idx + r] : T(0);
    }
}

// This thread's part of the sum of in[a, b) (b a multiple of 4).
template <typename T>
__device__ __forceinline__ int64_t range_part(const T* __restrict__ in, int64_t a, int64_t b)
{
    int64_t s = 0;
    const int64_t a4 = min((a + 3) & ~int64_t(3), b);
    if (a + threadIdx.x < a4) s += static_cast<int64_t>(in[a + threadIdx.x]);
#pragma unroll 8
    for (int64_t i = a4 + 4 * static_cast<int64_t>(threadIdx.x); i < b; i += kScanTile) {
        const uint4 q = *reinterpret_cast<const uint4*>(in + i);
        s += static_cast<int64_t>(static_cast<T>(q.x)) + static_cast<int64_t>(static_cast<T>(q.y)) +
             static_cast<int64_t>(static_cast<T>(q.z)) + static_cast<int64_t>(static_cast<T>(q.w));
    }
    return s;
}

// A non-null `gate` pointing at 0 turns a scan kernel into a no-op (work that depends
// on a count known only on the device).
template <typename TIn>
__global__ void __launch_bounds__(kScanThreads)
k_scan_reduce(const TIn* __restrict__ in, int64_t m, int64_t* __restrict__ partial, const int* gate)
{
    if (gate && *gate == 0) return;
    __shared__ int64_t sh[kScanThreads / 64];
    TIn v[4];
    load4(in, static_cast<int64_t>(blockIdx.x) * kScanTile + 4 * threadIdx.x, m, v);
    const int64_t s = static_cast<int64_t>(v[0]) + static_cast<int64_t>(v[1]) + static_cast<int64_t>(v[2]) +
                      static_cast<int64_t>(v[3]);
    const int64_t tot = block_sum<kScanThreads>(s, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

// One workgroup scans the tile sums in place (exclusive); partial[nt] = total.
__global__ void __launch_bounds__(kScanThreads)
k_scan_partials(int64_t* __restrict__ partial, int64_t nt, const int* gate)
{
    if (gate && *gate == 0) return;
    __shared__ int64_t sh[kScanThreads / 64];
    int64_t carry = 0;  // the same in every thread
    for (int64_t b = 0; b < nt; b += kScanThreads) {
        const int64_t idx = b + threadIdx.x;
        const int64_t v = idx < nt ? partial[idx] : 0;
        int64_t tot;
        const int64_t ex = block_excl_scan(v, &tot, sh);
        if (idx < nt) partial[idx] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) partial[nt] = carry;
}

// With `flags` (the cell starts' scan, between the assignment and everything else) it also
// starts the structure's flags for this build: the assignment's finding, and zeros.
template <typename TIn, typename TOut, int OFF>
__global__ void __launch_bounds__(kScanThreads)
k_scan(const TIn* in, int64_t m, const int64_t* __restrict__ partial, TOut* out, const int* gate, int* flags)
{
    if (gate && *gate == 0) return;
    if (flags && blockIdx.x == 0 && threadIdx.x == 0) {
        // an exchange: a uniform load goes through the scalar cache, and nothing keeps it before
        // a later vector store to its address
        flags[kFlagErr] = atomicExch(flags + kFlagBad, 0);
        for (int k = kFlagErr + 1; k < kFlagBad; ++k) flags[k] = 0;
    }
    __shared__ int64_t sh[kScanThreads / 64];
    const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * kScanTile;
    const int64_t base = tile0 + 4 * threadIdx.x;
    TIn v[4];
    load4(in, base, m, v);
    int64_t before = 0;
    if (OFF == kScanSelf) before = range_part(in, 0, tile0);
    if (OFF == kScanFold)
        for (int64_t t = threadIdx.x; t < blockIdx.x; t += kScanThreads) before += partial[t];
    int64_t offset;
    if (OFF == kScanScanned) offset = partial[blockIdx.x];
    else offset = block_sum<kScanThreads>(before, sh);
    const int64_t s = static_cast<int64_t>(v[0]) + static_cast<int64_t>(v[1]) + static_cast<int64_t>(v[2]) +
                      static_cast<int64_t>(v[3]);
    int64_t tot;
    int64_t run = block_excl_scan(s, &tot, sh) + offset;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (base + r < m) out[base + r] = static_cast<TOut>(run);
        run += static_cast<int64_t>(v[r]);
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[m] = static_cast<TOut>(offset + tot);
}

template <typename T>
__global__ void k_zero_one(T* p) { *p = T(0); }

// The tile sums a scan of nt tiles needs (and their own scan), or none.
template <typename TIn>
ScanOffset scan_sums(const TIn* in, int64_t m, int64_t nt, bool apart, int64_t* partial, hipStream_t st, const int* gate)
{
    if (nt == 1 || (apart && nt <= kScanSelfTiles)) return kScanSelf;
    hipLaunchKernelGGL(k_scan_reduce<TIn>, dim3(nt), dim3(kScanThreads), 0, st, in, m, partial, gate);
    if (nt <= kScanFoldTiles) return kScanFold;
    hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(kScanThreads), 0, st, partial, nt, gate);
    return kScanScanned;
}

template <typename TIn, typename TOut>
hipError_t scan_exclusive(const TIn* in, int64_t m, TOut* out, int64_t* partial, hipStream_t st,
                          const int* gate = nullptr, int* flags = nullptr)
{
    const int64_t nt = (m + kScanTile - 1) / kScanTile;
    if (nt == 0) {
        // m == 0: out[0] = 0
        hipLaunchKernelGGL(k_zero_one<TOut>, dim3(1), dim3(1), 0, st, out);
        return hipGetLastError();
    }
    const bool apart = static_cast<const void*>(in) != static_cast<const void*>(out);
    const dim3 g(nt), b(kScanThreads);
    switch (scan_sums(in, m, nt, apart, partial, st, gate)) {
    case kScanSelf:
        hipLaunchKernelGGL((k_scan<TIn, TOut, kScanSelf>), g, b, 0, st, in, m, partial, out, gate, flags);
        break;
    case kScanFold:
        hipLaunchKernelGGL((k_scan<TIn, TOut, kScanFold>), g, b, 0, st, in, m, partial, out, gate, flags);
        break;
    default: hipLaunchKernelGGL((k_scan<TIn, TOut, kScanScanned>), g, b, 0, st, in, m, partial, out, gate, flags);
    }
    return hipGetLastError();
}

int64_t scan_partials_needed(int64_t m) { return (m + kScanTile - 1) / kScanTile + 1; }

// ---------------------------------------------------------------------------
// A2: stable LSD radix sort of (key, index) pairs (the dense cells' union lists), up to
// 8 bits per pass. Tiles of kRsTile keys; each wave of a tile owns 1024 consecutive keys
// and ranks them 64 at a time: lanes holding the same digit find each other with one
// ballot per digit bit, and a per-wave LDS counter per digit keeps the order of rounds.
// Tile order, then wave, then round, then lane equals index order: the sort is stable.
// The tile is put in output order in LDS first, so a digit's run is written by
// consecutive threads.
constexpr int kRsThreads = 256;
constexpr int kRsRounds = 16;
constexpr int kRsTile = kRsThreads * kRsRounds;
constexpr int kRsMaxBits = 11;
// Digit width per pass: at most 8 bits, so a tile's keys fall into runs of 16 or more per
// digit on average and the scatter's stores fill whole cache lines (with 10- or 11-bit
// digits a tile has 2-4 keys per digit and nearly every store writes its own line).
constexpr int kRsPassBits = 8;

__global__ void __launch_bounds__(kRsThreads)
k_radix_hist(const uint32_t* __restrict__ keys, int n, int shift, int bits,
             uint32_t* __restrict__ table, int ntiles, const int* ndev)
{
    // ndev: the number of keys is on the device (at most n; 0 skips the pass)
    if (ndev) {
        if (*ndev == 0) return;
        n = min(n, *ndev);
    }
    __shared__ uint32_t h[1 << kRsMaxBits];
    const int bins = 1 << bits;
    const uint32_t mask = bins - 1;
    for (int i = threadIdx.x; i < bins; i += kRsThreads) h[i] = 0;
    __syncthreads();
    const int base = blockIdx.x * kRsTile;
    for (int r = 0; r < kRsRounds; ++r) {
        const int idx = base + r * kRsThreads + threadIdx.x;
        if (idx < n) atomicAdd(&h[(keys[idx] >> shift) & mask], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < bins; i += kRsThreads) table[static_cast<size_t>(i) * ntiles + blockIdx.x] = h[i];
}

__global__ void __launch_bounds__(kRsThreads)
k_radix_scatter(const uint32_t* __restrict__ kin, const int* __restrict__ vin,
                uint32_t* __restrict__ kout, int* __restrict__ vout, int n, int shift, int bits,
                const uint32_t* __restrict__ offs, int ntiles, const int* ndev)
{
    if (ndev) {
        if (*ndev == 0) return;
        n = min(n, *ndev);
    }
    if (blockIdx.x * kRsTile >= n) return;  // a tile past the keys (the grid is sized for a bound)
    constexpr int MB = 1 << kRsPassBits;
    constexpr int NWV = kRsThreads / 64;
    static_assert(MB <= kRsThreads, "one thread per digit in the tile's digit scan");
    __shared__ uint32_t cw[NWV][MB];
    __shared__ uint32_t tstart[MB];  // the tile's first position of each digit
    __shared__ uint32_t wtot[NWV];
    __shared__ uint32_t sk[kRsTile];  // the tile's keys and values in output order
    __shared__ int sv[kRsTile];
    const int bins = 1 << bits;  // bits <= kRsPassBits
    const uint32_t mask = bins - 1;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < NWV * MB; i += kRsThreads) cw[i / MB][i % MB] = 0;
    __syncthreads();
    const int base = blockIdx.x * kRsTile + w * (kRsRounds * 64);
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t myk[kRsRounds];
    int myv[kRsRounds];
    uint32_t rank[kRsRounds];
#pragma unroll
    for (int r = 0; r < kRsRounds; ++r) {
        const int idx = base + r * 64 + lane;
        const bool valid = idx < n;
        const uint32_t k = valid ? kin[idx] : 0u;
        const int v = valid ? (vin ? vin[idx] : idx) : 0;
        const uint32_t d = (k >> shift) & mask;
        uint64_t m = __ballot(valid);
        for (int b = 0; b < bits; ++b) {
            const bool set = (d >> b) & 1u;
            const uint64_t bb = __ballot(set);
            m &= set ? bb : ~bb;
        }
        const uint32_t rnk = __popcll(m & lt);
        const uint32_t cnt = __popcll(m);
        const uint32_t b0 = cw[w][d];
        __builtin_amdgcn_wave_barrier();
        if (valid && rnk == 0) cw[w][d] = b0 + cnt;
        __builtin_amdgcn_wave_barrier();
        myk[r] = k;
        myv[r] = v;
        rank[r] = b0 + rnk;
    }
    __syncthreads();
    // per digit: each wavefront's offset inside the tile's run of that digit, and the run's
    // length; then the runs' starts (exclusive scan over the digits, one thread per digit)
    uint32_t len = 0;
    if (threadIdx.x < bins) {
#pragma unroll
        for (int k = 0; k < NWV; ++k) {
            const uint32_t t = cw[k][threadIdx.x];
            cw[k][threadIdx.x] = len;
            len += t;
        }
    }
    uint32_t inc = len;  // inclusive scan inside the wavefront
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
    }
    if (lane == 63) wtot[w] = inc;
    __syncthreads();
    uint32_t before = 0;
    for (int k = 0; k < w; ++k) before += wtot[k];
    if (threadIdx.x < bins) tstart[threadIdx.x] = before + inc - len;
    __syncthreads();
    // the tile in output order, in LDS
#pragma unroll
    for (int r = 0; r < kRsRounds; ++r) {
        const int idx = base + r * 64 + lane;
        if (idx < n) {
            const uint32_t d = (myk[r] >> shift) & mask;
            const uint32_t lp = tstart[d] + cw[w][d] + rank[r];
            sk[lp] = myk[r];
            sv[lp] = myv[r];
        }
    }
    __syncthreads();
    // consecutive threads write consecutive positions of a digit's run
    const int nvalid = min(kRsTile, n - static_cast<int>(blockIdx.x) * kRsTile);
    for (int i = threadIdx.x; i < nvalid; i += kRsThreads) {
        const uint32_t k = sk[i];
        const uint32_t d = (k >> shift) & mask;
        const uint32_t p = offs[static_cast<size_t>(d) * ntiles + blockIdx.x] + (static_cast<uint32_t>(i) - tstart[d]);
        kout[p] = k;
        vout[p] = sv[i];
    }
}

// ---------------------------------------------------------------------------
// A4: pack in sorted order. q_k = f32(D_k) 2^(1-F) with D_k = X_k - c_k 2^F - 2^(F-1), the
// Eq. 6 relative coordinate in [-1, 1], in f32 (the passes that compute in FP16 round it to
// FP16 as they load it), with the cell indices mod 2^10 per axis (the cells of a block's
// candidate union lie fewer than 2^10 apart, so differences mod 2^10 recover the offsets).
// Beside it the FP64 position and the particle index, one 32-byte record per particle: the
// FP64 predicates and the distances of every mode read these, contiguous in sorted order.
template <int DIM>
__device__ __forceinline__ void pack_particle(const Launch& L, const PackArgs& a, int p)
{
    if (p >= L.ntot) return;
    const int o = a.perm[p];
    const uint32_t key = a.skey[p];
    auto pack = [&](const SetDesc& sd) {
        const Frame& fr = sd.fr;
        double x[3] = {0.0, 0.0, 0.0};
        float q32[3] = {0.0f, 0.0f, 0.0f};
        uint32_t cbits = 0;
        const float scale = __builtin_ldexpf(1.0f, 1 - fr.F);
#pragma unroll
        for (int k = 0; k < DIM; ++k) x[k] = sd.pos[static_cast<size_t>(o - sd.poff) * DIM + k];
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            // as the assignment: a position outside the box counts as lo
            const double pk = (x[k] >= fr.lo[k] && x[k] <= fr.hi[k]) ? x[k] : fr.lo[k];
            const int64_t X = fixed_point(pk, fr.lo[k], fr.s);
            const int64_t c = X >> fr.F;
            const int64_t D = X - (c << fr.F) - (int64_t(1) << (fr.F - 1));
            q32[k] = exact_i64_to_f32(D) * scale;  // exact power-of-two scaling
            cbits |= static_cast<uint32_t>(c & 1023) << (10 * k);
        }
        double2* sp = reinterpret_cast<double2*>(a.spos + static_cast<size_t>(p) * 4);
        sp[0] = make_double2(x[0], x[1]);
        sp[1] = make_double2(x[2], __builtin_bit_cast(double, static_cast<int64_t>(o)));
        a.rq[p] = make_float4(q32[0], q32[1], q32[2], __builtin_bit_cast(float, cbits));
    };
    // a wavefront inside one set reads the set's fields with scalar loads
    const int s = find_set(L.coffs, L.nsets, static_cast<int>(key));
    const int s0 = __builtin_amdgcn_readfirstlane(s);
    if (__all(s == s0)) pack(L.sets[s0]);
    else pack(L.sets[s]);
    a.inv[o] = p;
    // the incremental update places into a second pair of arrays: copied back here
    if (a.perm_out) {
        a.perm_out[p] = o;
        a.skey_out[p] = key;
    }
}

// ---------------------------------------------------------------------------
// Incremental update after the particles moved (Mixed-precision SPH framework section,
// Eq. 8-9, Fig. 6): a particle's relative coordinate advances by its displacement, and a
// particle leaving its cell migrates to the new one. Here the advance is made on the
// binary64 position (p = p + dp, one rounding, written back when a displacement array is
// given) and the fixed-point position and cell are recomputed from it exactly as the
// assignment computes them, so the relative coordinate carries no error from earlier
// steps and the structure equals a fresh build's up to the order inside cells. Only
// migrants are re-binned: the sorted order is kept, stayers keep their relative order in
// their cell, and each cell's migrants are appended after its stayers.

// U1 (per particle, in the caller's order so positions and displacements stream): move,
// recompute the cell. A displacement component that would
// take the particle out of [lo, hi] is applied with its sign flipped (a reflection at the
// box faces). A particle whose cell changed is a migrant: bit inv[i] of `mig` is set, it
// counts out of its old cell and takes an arrival slot in its new one. Every particle's
// new cell key is kept by particle index (knew).
template <int DIM>
__global__ void __launch_bounds__(256)
k_upd_move(const SetDesc* __restrict__ sets, const int* __restrict__ poffs, int nsets, int ntot,
           const uint32_t* __restrict__ skey, const int* __restrict__ inv, uint32_t* __restrict__ knew,
           uint32_t* __restrict__ mig, int* __restrict__ leave, int* __restrict__ arrive, int* __restrict__ aslot, int* __restrict__ err)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ntot) return;
    bool bad = false;
    auto cell_of = [&](const SetDesc& sd) -> uint32_t {
        // the set's fields in registers: read through the table they would be loaded again
        // after every store below (the compiler cannot tell the stores from the table)
        double lo[DIM], hi[DIM];
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            lo[k] = sd.fr.lo[k];
            hi[k] = sd.fr.hi[k];
        }
        const double scale = sd.fr.s;
        const int F = sd.fr.F, ncx = sd.fr.nc[0], ncy = sd.fr.nc[1], coff = sd.coff;
        const int li = i - sd.poff;
        double* pos = const_cast<double*>(sd.pos);  // the caller lent them for the update
        const double* disp = sd.disp;
        double p[DIM];
#pragma unroll
        for (int k = 0; k < DIM; ++k) p[k] = pos[static_cast<size_t>(li) * DIM + k];
        if (disp) {
#pragma unroll
            for (int k = 0; k < DIM; ++k) {
                const double d = disp[static_cast<size_t>(li) * DIM + k];
                const double q = __dadd_rn(p[k], d);
                p[k] = (q >= lo[k] && q <= hi[k]) ? q : __dadd_rn(p[k], -d);
            }
#pragma unroll
            for (int k = 0; k < DIM; ++k) pos[static_cast<size_t>(li) * DIM + k] = p[k];
        }
        int64_t c[3] = {0, 0, 0};
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            double pk = p[k];
            if (!(pk >= lo[k] && pk <= hi[k])) {
                bad = true;
                pk = lo[k];
            }
            c[k] = fixed_point(pk, lo[k], scale) >> F;
        }
        return static_cast<uint32_t>(coff + c[0] + ncx * (c[1] + ncy * c[2]));
    };
    // a wavefront inside one set reads the set's fields with scalar loads
    const int st = find_set(poffs, nsets, i);
    const int s0 = __builtin_amdgcn_readfirstlane(st);
    const uint32_t kn = __all(st == s0) ? cell_of(sets[s0]) : cell_of(sets[st]);
    knew[i] = kn;
    const int sp = inv[i];
    const uint32_t kold = skey[sp];
    if (kn != kold) {
        atomicOr(&mig[sp >> 5], 1u << (sp & 31));
        atomicAdd(&leave[kold], 1);
        aslot[i] = atomicAdd(&arrive[kn], 1);
    }
    if (bad) atomicOr(err, kErrDomain);
}

// U2 (per cell, and one more thread for the end): the new occupancy, old count - leavers
// + arrivals, as the scan's input, and a copy of the old cell starts (the scan writes the
// new ones in place).
__global__ void __launch_bounds__(256)
k_upd_counts(int ncell, const int* __restrict__ cell_start, const int* __restrict__ leave,
             const int* __restrict__ arrive, int* __restrict__ cnt, int* __restrict__ cs_old)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c > ncell) return;
    const int a = cell_start[c];
    cs_old[c] = a;
    if (c < ncell) cnt[c] = cell_start[c + 1] - a - leave[c] + arrive[c];
}

// Set bits of `mig` at positions [a, b).
__device__ __forceinline__ int mig_bits(const uint32_t* __restrict__ mig, int a, int b)
{
    int n = 0;
    for (int w = a >> 5; (w << 5) < b; ++w) {
        uint32_t m = mig[w];
        const int lo = a - (w << 5), hi = b - (w << 5);  // bit range of this word, clipped below
        if (lo > 0) m &= ~0u << lo;
        if (hi < 32) m &= (1u << hi) - 1u;
        n += __builtin_popcount(m);
    }
    return n;
}

// U3 (per old sorted position s): the particle's new sorted position. A stayer keeps its
// rank among the stayers of its cell (its old offset less the leavers before it); a
// migrant goes after the stayers of its new cell, at its arrival slot.
__device__ __forceinline__ void update_place(const Launch& L, const PlaceArgs& a, const int* cell_start, int s)
{
    if (s >= L.ntot) return;
    const Update& u = a.u;
    const int o = a.perm[s];
    const uint32_t kold = a.skey[s], kn = u.knew[o];
    int at;
    if (kn == kold) {
        const int c0 = u.cs_old[kold];
        const int lb = u.leave[kold] > 0 ? mig_bits(u.mig, c0, s) : 0;
        at = cell_start[kold] + (s - c0) - lb;
    } else {
        at = cell_start[kn] + (u.cs_old[kn + 1] - u.cs_old[kn] - u.leave[kn]) + u.aslot[o];
    }
    u.skey2[at] = kn;
    u.perm2[at] = o;
}

// ---------------------------------------------------------------------------
// Work blocks, one wavefront per segment of 64 cells of a row of cells of a set: walking
// the segment in x, a block is a run of at most kWave consecutive sorted particles whose
// cells span at most fr.xwin cells; it starts where the previous one ended (so blocks are
// full unless the span, the segment or the row ends them). A run of dense cells (the
// dense-cell path's) is one block that the block kernels skip. The walk runs twice: the
// first counts each segment's blocks (nb[r]), the second, after an exclusive scan of the
// counts into boff, writes block boff[r] + j's first particle and set. Blocks come out in
// particle order, so block b ends where block b + 1 starts; bstart[total] = ntot.
// The walk steps from block to block with ballots over the segment's cells, one lane each
// (one cell at a time took 12 us a pass on a 1000 x 1000 lattice).
//
// For up to kRowFold segments the second walk's workgroups sum the counts before theirs
// themselves, and no scan is launched (8192 counts are 32 KB read by each of 2048 workgroups).
constexpr int kRowsPerGroup = 4;
constexpr int kRowFold = 8192;

template <bool WRITE>
__device__ __forceinline__ void row_blocks(const Launch& L, const BlockTable& t, int group)
{
    const int w = static_cast<int>(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int r0 = group * kRowsPerGroup, r = r0 + w;
    const bool valid = r < L.nrows_tot;
    // the cells and the counts before this group are loaded side by side: the kernel is a
    // chain of loads and little else
    int s = 0, span = 0, c0 = 0, c1 = 0, dn = 0, b0 = 0;
    if (valid) {
        s = find_set(L.roffs, L.nsets, r);
        const SetDesc& sd = L.sets[s];
        const int ncx = sd.fr.nc[0];
        span = sd.fr.xwin;
        const int nseg = (ncx + kRowSegment - 1) / kRowSegment;
        const int rs = r - L.roffs[s];
        const int x = (rs % nseg) * kRowSegment + lane, g = sd.coff + (rs / nseg) * ncx + x;
        if (x < ncx) {
            c0 = t.cell_start[g];
            c1 = t.cell_start[g + 1];
            dn = t.wdense ? t.wdense[g] : 0;
        }
    }
    if (WRITE && t.fold) {
        __shared__ int sh[kRowsPerGroup];
        int before = 0;
        static_assert(kRowsPerGroup == 4, "r0 is a multiple of 4");
#pragma unroll 4
        for (int i = 4 * threadIdx.x; i < r0; i += 4 * 64 * kRowsPerGroup) {
            const int4 q = *reinterpret_cast<const int4*>(t.boff + i);
            before += q.x + q.y + q.z + q.w;
        }
        int mine = 0;
        for (int i = r0; i < min(r, L.nrows_tot); ++i) mine += t.boff[i];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
        if (lane == 0) sh[w] = before;
        __syncthreads();
        b0 = mine + sh[0] + sh[1] + sh[2] + sh[3];
    } else if (WRITE && valid) {
        b0 = t.boff[r];
    }
    if (!valid) return;
    const uint64_t filled = __ballot(c1 > c0), dense = __ballot(c1 > c0 && dn);
    // wavefront-uniform walk state: the block starts at particle a in the segment's cell i
    int nb = 0;
    int i = filled ? __builtin_ctzll(filled) : 64;
    int a = __builtin_amdgcn_readlane(c0, i & 63);
    while (i < 64) {
        if (WRITE && lane == 0) {
            t.bstart[b0 + nb] = a;
            t.bset[b0 + nb] = s;
        }
        ++nb;
        const uint64_t from = ~0ull << i, after = from << 1;
        uint64_t next;
        if (dense >> i & 1) {
            next = filled & ~dense & after;
        } else {
            next = filled & after & (dense | (i + span < 64 ? ~0ull << (i + span) : 0ull));
            // the first cell that holds the particle kWave after a
            const uint64_t full = __ballot(c1 - a > kWave) & filled & from;
            if (full && (!next || __builtin_ctzll(full) < __builtin_ctzll(next))) {
                i = __builtin_ctzll(full);
                a += kWave;
                continue;
            }
        }
        if (!next) break;
        i = __builtin_ctzll(next);
        a = __builtin_amdgcn_readlane(c0, i);
    }
    if (lane) return;
    if (!WRITE) {
        t.boff[r] = nb;
    } else if (r == L.nrows_tot - 1) {
        const int total = b0 + nb;
        t.bstart[total] = L.ntot;
        if (t.fold) t.boff[L.nrows_tot] = total;
    }
}

// Row pointers of every set: the exclusive scan of its own counts (row_ptr), each particle's
// row start by sorted position (rsort) and the set's nnz. A tile's first set started before
// it: the workgroup adds up the counts from that set's start (OFF, as the scan); a set that
// starts inside the tile subtracts the tile's prefix there. 1M rows in 9 to 12 us (24 MB
// written); stores of four rows a thread instead of lane by lane took 14 to 16.
template <int OFF>
__global__ void __launch_bounds__(kScanThreads)
k_rowptr(const SetDesc* __restrict__ sets, const int* __restrict__ poffs, int nsets, const int* __restrict__ counts,
         int64_t m, const int64_t* __restrict__ partial, int64_t* __restrict__ nnz, const int* __restrict__ inv,
         int64_t* __restrict__ rsort, RowptrExtras rep)
{
    auto total = [&](int s, int64_t v) {
        nnz[s] = v;
        if (rep.host) rep.host[kFlags / 2 + s] = v;
    };
    __shared__ int64_t sh[kScanThreads / 64];
    __shared__ int64_t local[kScanTile + kScanTile / 16];  // the tile's prefixes, one pad per 16
    const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * kScanTile;
    const int64_t base = tile0 + 4 * threadIdx.x;
    const int s0 = find_set(poffs, nsets, static_cast<int>(tile0));
    const int s1 = find_set(poffs, nsets, static_cast<int>(min(tile0 + kScanTile, m) - 1));
    int v[4];
    load4(counts, base, m, v);
    const int64_t p0 = poffs[s0];
    int64_t before = 0;
    if (OFF == kScanSelf) {
        before = range_part(counts, p0, tile0);
    } else {
        const int64_t tb = (p0 + kScanTile - 1) / kScanTile;
        before = range_part(counts, p0, min(tb * kScanTile, tile0));
        if (OFF == kScanFold)
            for (int64_t t = tb + threadIdx.x; t < blockIdx.x; t += kScanThreads) before += partial[t];
        else if (threadIdx.x == 0 && tb < blockIdx.x) before += partial[blockIdx.x] - partial[tb];
    }
    const int64_t offset = block_sum<kScanThreads>(before, sh);
    const int64_t sum = static_cast<int64_t>(v[0]) + v[1] + v[2] + v[3];
    int64_t tot;
    int64_t run = block_excl_scan(sum, &tot, sh);
    // through LDS, so that the stores below go out lane by lane
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int e = 4 * threadIdx.x + r;
        local[e + (e >> 4)] = run;
        run += v[r];
    }
    __syncthreads();
    auto put = [&](const SetDesc& sd, int s, int64_t shift, int e, int64_t start) {
        const int64_t i = tile0 + e, val = local[e + (e >> 4)] + shift;
        int64_t* rp = sd.row_ptr;
        rp[i - start] = val;
        rsort[inv[i]] = val;
        if (i + 1 == start + sd.fr.n) {
            rp[sd.fr.n] = val + counts[i];
            total(s, val + counts[i]);
        }
    };
    const int len = static_cast<int>(min(m - tile0, static_cast<int64_t>(kScanTile)));
    if (s0 == s1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e = r * kScanThreads + threadIdx.x;
            if (e < len) put(sets[s0], s0, offset, e, p0);
        }
    } else {
        for (int e = threadIdx.x; e < len; e += kScanThreads) {
            const int s = find_set(poffs, nsets, static_cast<int>(tile0) + e);
            const int64_t start = poffs[s];
            const int b = static_cast<int>(start - tile0);
            put(sets[s], s, start <= tile0 ? (s == s0 ? offset : 0) : -local[b + (b >> 4)], e, start);
        }
    }
    if (blockIdx.x) return;
    // sets without particles own no element of the scan
    for (int s = threadIdx.x; s < nsets; s += kScanThreads)
        if (sets[s].fr.n == 0) {
            sets[s].row_ptr[0] = 0;
            total(s, 0);
        }
    // what goes with the row pointers
    const int t = threadIdx.x;
    if (t == kFlagBlocks) rep.flags[t] = *rep.nblk;
    if (rep.host) {
        if (t < kFlags) reinterpret_cast<int*>(rep.host)[t] = t == kFlagBlocks ? *rep.nblk : rep.flags[t];
        if (t == kFlags) rep.host[kHostWords - 1] = rep.pairs ? *rep.pairs : 0;
    }
    if (rep.rpool && t < kRankPools) rep.rpool[t * kRankPoolStride] = 0;
}

// ---------------------------------------------------------------------------
// Dense-cell path tables. Where clustering piles hundreds or thousands of particles
// into a cell, every target of the cell tests the same stencil union, and its rows are
// long. A cell is dense when its stencil holds more than a threshold of particles. For such
// cells the search stages the union once per chunk for all the cell's targets, in ascending
// original index, so each row comes out sorted with no per-row sort. The union lists are ranked
// in a bitmap (k_union_rank), or come from one stable sort: every particle, visited in original
// order, emits (dense cell, sorted position) for each dense cell whose stencil holds it.

// Global cell index -> local coordinates of its set.
struct CellXYZ {
    int x, y, z, ncx, ncy, ncz;
    __device__ __forceinline__ CellXYZ(const Frame& fr, int lk)
    {
        ncx = fr.nc[0];
        ncy = fr.nc[1];
        ncz = fr.nc[2];
        x = lk % ncx;
        const int row = lk / ncx;
        y = row % ncy;
        z = row / ncy;
    }
};

// Stencil size of every occupied cell; a cell is dense when it exceeds the threshold.
template <int DIM>
__device__ __forceinline__ void dense_cell(const Launch& L, const int* cell_start, const DenseBuild& d, int g)
{
    if (g >= L.ncell_tot) return;
    const SetDesc& sd = L.sets[find_set(L.coffs, L.nsets, g)];
    const CellXYZ c(sd.fr, g - sd.coff);
    const int* cs = cell_start + sd.coff;
    int u = 0;
    if (cell_start[g + 1] > cell_start[g]) {
        const int x0 = c.x > 0 ? c.x - 1 : 0;
        const int x1 = c.x + 1 < c.ncx ? c.x + 1 : c.ncx - 1;
        for (int dz = (DIM == 3 ? -1 : 0); dz <= (DIM == 3 ? 1 : 0); ++dz) {
            const int zz = c.z + dz;
            if (zz < 0 || zz >= c.ncz) continue;
            for (int dy = -1; dy <= 1; ++dy) {
                const int yy = c.y + dy;
                if (yy < 0 || yy >= c.ncy) continue;
                const int rb = (zz * c.ncy + yy) * c.ncx;
                u += cs[rb + x1 + 1] - cs[rb + x0];
            }
        }
    }
    const bool dense = u > d.thresh;
    d.usz[g] = dense ? u : 0;
    d.wdense[g] = dense ? 1 : 0;
    if (dense) *d.seen = 1;  // every writer writes the same value
}

// The launch after the cell starts, three pieces of work that need nothing else, a range of
// workgroups each: the segments' block counts (rows), the cells' stencil sizes (dense), and
// the sort by cell, as a counting sort (particle i goes to cell_start[key] + slot) or as the
// update's re-binning. Each alone leaves the chip mostly idle and a launch costs 4.6 us: as
// launches of their own (and the block table and the clearing of the counters too) a step
// took 17 instead of 9 or 10; a search of 10,000 particles 139 instead of 75 us, a step of a
// 1000 x 1000 lattice 188 instead of 169.
template <int DIM, bool MOVED>
__global__ void __launch_bounds__(256)
k_sort(Launch L, PlaceArgs a, DenseBuild d, BlockTable t, int nrows, int ndense)
{
    const int b = blockIdx.x;
    if (b < nrows) {
        row_blocks<false>(L, t, b);
    } else if (b < nrows + ndense) {
        dense_cell<DIM>(L, t.cell_start, d, (b - nrows) * 256 + static_cast<int>(threadIdx.x));
    } else {
        const int i = (b - nrows - ndense) * 256 + static_cast<int>(threadIdx.x);
        if (MOVED) {
            update_place(L, a, t.cell_start, i);
        } else if (i < L.ntot) {
            const uint32_t kk = a.key[i];
            const int at = t.cell_start[kk] + a.slot[i];
            a.skey_out[at] = kk;
            a.perm_out[at] = i;
        }
    }
}

// The launch after that: the block table from the segments' counts, and the pack, which also
// clears the counters that this build is through with for the next one.
template <int DIM>
__global__ void __launch_bounds__(256)
k_pack(Launch L, PackArgs a, BlockTable t, int nrows)
{
    const int b = blockIdx.x;
    if (b < nrows) {
        row_blocks<true>(L, t, b);
        return;
    }
    const int i = (b - nrows) * 256 + static_cast<int>(threadIdx.x), step = (gridDim.x - nrows) * 256;
    for (int64_t k = i; k < a.nclear0; k += step) a.clear0[k] = 0;
    for (int64_t k = i; k < a.nclear1; k += step) a.clear1[k] = 0;
    pack_particle<DIM>(L, a, i);
}

// After the scan of the stencil sizes: if the lists would not fit, the build falls back
// to the block path (every window normal); otherwise each dense cell gets its work
// units. dn receives the number of list entries in use (0 = path off).
__global__ void __launch_bounds__(256)
k_dense_units(int ncell_tot, const int* __restrict__ cell_start, const int64_t* __restrict__ uoff, int64_t cap,
              int* __restrict__ usz, int* __restrict__ wdense, int* __restrict__ nsl, int* __restrict__ dn,
              uint32_t* __restrict__ dbn)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t ue = uoff[ncell_tot];
    const bool over = ue > cap;
    if (g == 0) *dn = over ? 0 : static_cast<int>(ue);
    if (g >= ncell_tot) return;
    if (over) {
        usz[g] = 0;
        wdense[g] = 0;
    }
    const int occ = cell_start[g + 1] - cell_start[g];
    const bool on = !over && usz[g] > 0;
    nsl[g] = on ? (occ + kDenseUnit - 1) / kDenseUnit : 0;
    // 2^32 - 1 pairs would be 512 GiB of kept bits: more than any buffer holds, so none are kept
    const int64_t pairs = on ? static_cast<int64_t>(occ) * ((usz[g] + kDenseChunk - 1) / kDenseChunk) : 0;
    dbn[g] = static_cast<uint32_t>(min(pairs, static_cast<int64_t>(0xFFFFFFFFu)));
}

__global__ void __launch_bounds__(256)
k_dense_unit_cells(int ncell_tot, const int* __restrict__ nsl, const int* __restrict__ unit_off,
                   const int* __restrict__ dn, int* __restrict__ ucell)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= ncell_tot || *dn == 0) return;
    const int k = nsl[g], u0 = unit_off[g];
    for (int s = 0; s < k; ++s) ucell[u0 + s] = g;
}

// Visit the dense cells whose stencil holds the particle at sorted position j. The 3^d
// stencil sizes are loaded together first (cells outside the grid read as 0), then the
// dense ones are visited in x-fastest order.
template <int DIM, typename F>
__device__ __forceinline__ void for_dense_stencils(const SetDesc* __restrict__ sets, const int* __restrict__ coffs,
                                                   int nsets, const uint32_t* __restrict__ skey,
                                                   const int* __restrict__ usz, int j, F&& f)
{
    constexpr int NS = DIM == 3 ? 27 : 9;
    const int gk = static_cast<int>(skey[j]);
    const SetDesc& sd = sets[find_set(coffs, nsets, gk)];
    const CellXYZ c(sd.fr, gk - sd.coff);
    int sz[NS];
#pragma unroll
    for (int t = 0; t < NS; ++t) {
        const int dx = t % 3 - 1, dy = (t / 3) % 3 - 1, dz = DIM == 3 ? t / 9 - 1 : 0;
        const int xx = c.x + dx, yy = c.y + dy, zz = c.z + dz;
        const bool in = xx >= 0 && xx < c.ncx && yy >= 0 && yy < c.ncy && zz >= 0 && zz < c.ncz;
        sz[t] = in ? usz[gk + dx + c.ncx * (dy + c.ncy * dz)] : 0;
    }
#pragma unroll
    for (int t = 0; t < NS; ++t) {
        const int dx = t % 3 - 1, dy = (t / 3) % 3 - 1, dz = DIM == 3 ? t / 9 - 1 : 0;
        if (sz[t] > 0) f(gk + dx + c.ncx * (dy + c.ncy * dz));
    }
}

template <int DIM>
__global__ void __launch_bounds__(256)
k_union_count(const SetDesc* __restrict__ sets, const int* __restrict__ coffs, int nsets, int ntot,
              const uint32_t* __restrict__ skey, const int* __restrict__ inv, const int* __restrict__ usz,
              const int* __restrict__ dn, int* __restrict__ ecnt)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ntot || *dn == 0) return;
    int k = 0;
    for_dense_stencils<DIM>(sets, coffs, nsets, skey, usz, inv[i], [&](int) { ++k; });
    ecnt[i] = k;
}

template <int DIM>
__global__ void __launch_bounds__(256)
k_union_emit(const SetDesc* __restrict__ sets, const int* __restrict__ coffs, int nsets, int ntot,
             const uint32_t* __restrict__ skey, const int* __restrict__ inv, const int* __restrict__ usz,
             const int* __restrict__ dn, const int* __restrict__ epos, uint32_t* __restrict__ ukey,
             int* __restrict__ uval)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ntot || *dn == 0) return;
    const int j = inv[i];
    int m = epos[i];
    for_dense_stencils<DIM>(sets, coffs, nsets, skey, usz, j, [&](int g2) {
        ukey[m] = static_cast<uint32_t>(g2);
        uval[m] = j;
        ++m;
    });
}

// The same lists without a sort: a workgroup per dense cell marks the candidates' set-local
// indices in a bitmap in LDS and places each by its rank there, kUnionWindow indices at a time.
// Two reads of the candidates' indices and one write of the list; the clearing and counting of
// the bitmap, per window, is what grows with the set: ranked against sorted, a clustered set in
// 2D takes 31 and 93 us at 10,000 particles, 51 and 132 at 200,000, 211 and 262 at a million
// (four windows), 639 and 445 at two; in 3D 33 and 100, 91 and 176, 639 and 863, 1329 and 1379.
// So sets of up to four windows are ranked. (256 threads a cell: 167 at 200,000 in 3D, 1024: 125.)
constexpr int kUnionThreads = 512;
constexpr int kUnionWords = 16 * kUnionThreads;  // 16 words a thread
constexpr int kUnionWindow = 32 * kUnionWords;
constexpr int kUnionWindows = 4;                 // larger sets' lists are sorted
constexpr int kUnionGrid = 768;                  // three workgroups a CU: 49 KB of LDS each

template <int DIM>
__global__ void __launch_bounds__(kUnionThreads)
k_union_rank(Launch L, const int* __restrict__ cell_start, const int* __restrict__ perm, DenseBuild d,
             int* __restrict__ ulist)
{
    // 16 words and 4 of padding per thread, so that the 16-byte accesses of a quarter
    // wavefront cover every bank once
    __shared__ uint4 bits[kUnionThreads * 5];
    __shared__ int before4[kUnionThreads * 4];  // marked before each group of 4 words
    __shared__ int wsum[kUnionThreads / 64];
    if (*d.dn == 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int nunits = d.unit_off[L.ncell_tot];
    constexpr int NR = DIM == 3 ? 9 : 3;
    for (int u = blockIdx.x; u < nunits; u += gridDim.x) {
        const int g = d.ucell[u];
        if (d.unit_off[g] != u) continue;  // a cell's first unit stands for the cell
        const SetDesc& sd = L.sets[find_set(L.coffs, L.nsets, g)];
        const CellXYZ c(sd.fr, g - sd.coff);
        const int* cs = cell_start + sd.coff;
        const int n = sd.fr.n, poff = sd.poff;
        // the candidates are NR runs of sorted positions: run r from first[r], shift[r] = its
        // first position less the candidates before it
        int first[NR + 1], shift[NR];
        const int x0 = max(c.x - 1, 0), x1 = min(c.x + 1, c.ncx - 1);
        first[0] = 0;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int yy = c.y + r % 3 - 1, zz = c.z + (DIM == 3 ? r / 3 - 1 : 0);
            const bool in = yy >= 0 && yy < c.ncy && zz >= 0 && zz < c.ncz;
            const int rb = in ? (zz * c.ncy + yy) * c.ncx : 0;
            const int a = in ? cs[rb + x0] : 0, b = in ? cs[rb + x1 + 1] : 0;
            shift[r] = a - first[r];
            first[r + 1] = first[r] + b - a;
        }
        const int total = first[NR];
        auto position = [&](int e) {
            int p = e + shift[0];
#pragma unroll
            for (int r = 1; r < NR; ++r) p = e >= first[r] ? e + shift[r] : p;
            return p;
        };
        int* out = ulist + d.uoff[g];
        int base = 0;
        for (int w0 = 0; w0 < n; w0 += kUnionWindow) {
#pragma unroll
            for (int k = 0; k < 4; ++k) bits[5 * tid + k] = make_uint4(0, 0, 0, 0);
            __syncthreads();
            for (int e = tid; e < total; e += kUnionThreads) {
                const uint32_t o = static_cast<uint32_t>(perm[position(e)] - poff - w0);
                if (o < kUnionWindow) {
                    const uint32_t w = o >> 5;
                    atomicOr(reinterpret_cast<uint32_t*>(bits) + w + (w >> 4) * 4, 1u << (o & 31));
                }
            }
            __syncthreads();
            int sum[4], mine = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint4 q = bits[5 * tid + k];
                sum[k] = mine;
                mine += __builtin_popcount(q.x) + __builtin_popcount(q.y) + __builtin_popcount(q.z) + __builtin_popcount(q.w);
            }
            int inc = mine;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(inc, o, 64);
                if (lane >= o) inc += y;
            }
            if (lane == 63) wsum[wv] = inc;
            __syncthreads();
            int start = base + inc - mine;
#pragma unroll
            for (int k = 0; k < kUnionThreads / 64; ++k) {
                if (k < wv) start += wsum[k];
                base += wsum[k];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) before4[4 * tid + k] = start + sum[k];
            __syncthreads();
            for (int e = tid; e < total; e += kUnionThreads) {
                const int p = position(e);
                const uint32_t o = static_cast<uint32_t>(perm[p] - poff - w0);
                if (o >= kUnionWindow) continue;
                const uint32_t w = o >> 5, in4 = w & 3;
                const uint4 q = bits[(w >> 2) + (w >> 4)];
                const uint32_t below = (1u << (o & 31)) - 1u;
                int rank = before4[w >> 2];
                rank += __builtin_popcount(in4 > 0 ? q.x : q.x & below);
                rank += in4 > 0 ? __builtin_popcount(in4 > 1 ? q.y : q.y & below) : 0;
                rank += in4 > 1 ? __builtin_popcount(in4 > 2 ? q.z : q.z & below) : 0;
                rank += in4 > 2 ? __builtin_popcount(q.w & below) : 0;
                out[rank] = p;
            }
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------
// Host-side launchers.
int row_segments(int ncx) { return (ncx + kRowSegment - 1) / kRowSegment; }

hipError_t launch_fill_i32(int* p, int64_t m, int v, hipStream_t st)
{
    if (m <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((m + 255) / 256, 4096);
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks), dim3(256), 0, st, p, m, v);
    return hipGetLastError();
}

hipError_t launch_assign(const Launch& L, bool hot, uint32_t* key, int* slot, int* cell_count, int* err, hipStream_t st)
{
    if (L.ntot == 0) return hipSuccess;
    const int threads = hot ? kAssignThreads : 256;
    const dim3 g((L.ntot + threads - 1) / threads), b(threads);
    auto k = L.dim == 2 ? (hot ? k_assign<2, true> : k_assign<2, false>) : (hot ? k_assign<3, true> : k_assign<3, false>);
    hipLaunchKernelGGL(k, g, b, 0, st, L.sets, L.poffs, L.nsets, L.ntot, key, slot, cell_count, err);
    return hipGetLastError();
}

hipError_t launch_cell_scan(const Launch& L, const int* cell_count, int* cell_start, int64_t* partial, int* flags,
                            hipStream_t st)
{
    return scan_exclusive<int, int>(cell_count, L.ncell_tot, cell_start, partial, st, nullptr, flags);
}

int radix_tiles(int n) { return (n + kRsTile - 1) / kRsTile; }

// Stable LSD sort of (key, value) pairs held in (k0, v0), with (k1, v1) as the second
// buffers; the number of pairs is read on the device (*ndev <= n; 0 skips the sort).
hipError_t radix_sort_kv_dev(int n, const int* ndev, int keybits, uint32_t* k0, int* v0, uint32_t* k1, int* v1,
                             uint32_t* table, int64_t* partial, hipStream_t st, uint32_t** kfinal, int** vfinal)
{
    const int ntiles = radix_tiles(n);
    const int passes = keybits <= 0 ? 1 : (keybits + kRsPassBits - 1) / kRsPassBits;
    const int bits = keybits <= 0 ? 1 : (keybits + passes - 1) / passes;
    if (bits > kRsPassBits) return hipErrorInvalidValue;  // cannot happen: passes fit the bound
    uint32_t *kin = k0, *kout = k1;
    int *vin = v0, *vout = v1;
    for (int p = 0; p < passes; ++p) {
        const int shift = p * bits;
        hipLaunchKernelGGL(k_radix_hist, dim3(ntiles), dim3(kRsThreads), 0, st, kin, n, shift, bits,
                           table, ntiles, ndev);
        hipError_t e = scan_exclusive<uint32_t, uint32_t>(table, static_cast<int64_t>(ntiles) << bits,
                                                          table, partial, st, ndev);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_radix_scatter, dim3(ntiles), dim3(kRsThreads), 0, st, kin, vin, kout,
                           vout, n, shift, bits, table, ntiles, ndev);
        std::swap(kin, kout);
        std::swap(vin, vout);
    }
    *kfinal = kin;
    *vfinal = vin;
    return hipGetLastError();
}

size_t radix_table_entries(int n) { return static_cast<size_t>(radix_tiles(n)) << kRsMaxBits; }

hipError_t launch_sort(const Launch& L, const PlaceArgs* place, const DenseBuild* dense, const BlockTable* blocks,
                       const int* cell_start, hipStream_t st)
{
    const int nrows = blocks && L.ntot > 0 ? (L.nrows_tot + kRowsPerGroup - 1) / kRowsPerGroup : 0;
    const int ndense = dense ? (L.ncell_tot + 255) / 256 : 0;
    const int nplace = place ? (L.ntot + 255) / 256 : 0;
    const dim3 g(static_cast<unsigned>(nrows) + ndense + nplace), b(256);
    if (g.x == 0) return hipSuccess;
    const PlaceArgs a = place ? *place : PlaceArgs{};
    const DenseBuild d = dense ? *dense : DenseBuild{};
    BlockTable t = blocks ? *blocks : BlockTable{};
    t.cell_start = cell_start;
    if (L.dim == 2 && a.moved) hipLaunchKernelGGL((k_sort<2, true>), g, b, 0, st, L, a, d, t, nrows, ndense);
    else if (a.moved) hipLaunchKernelGGL((k_sort<3, true>), g, b, 0, st, L, a, d, t, nrows, ndense);
    else if (L.dim == 2) hipLaunchKernelGGL((k_sort<2, false>), g, b, 0, st, L, a, d, t, nrows, ndense);
    else hipLaunchKernelGGL((k_sort<3, false>), g, b, 0, st, L, a, d, t, nrows, ndense);
    return hipGetLastError();
}

hipError_t launch_pack(const Launch& L, const PackArgs* pack, const BlockTable* blocks, const int* cell_start,
                       int64_t* partial, hipStream_t st)
{
    if (L.ntot == 0) return blocks ? launch_fill_i32(blocks->boff, static_cast<int64_t>(L.nrows_tot) + 1, 0, st) : hipSuccess;
    BlockTable t = blocks ? *blocks : BlockTable{};
    t.cell_start = cell_start;
    t.fold = L.nrows_tot <= kRowFold;
    if (blocks && !t.fold) {
        const hipError_t e = scan_exclusive<int, int>(t.boff, L.nrows_tot, t.boff, partial, st);
        if (e != hipSuccess) return e;
    }
    const int nrows = blocks ? (L.nrows_tot + kRowsPerGroup - 1) / kRowsPerGroup : 0;
    // workgroups for the particles, and for the counters where a grid has far more cells than
    // particles (16 of them a thread, as many as keep the chip busy)
    const PackArgs a = pack ? *pack : PackArgs{};
    const int64_t clear = std::min<int64_t>((a.nclear0 + a.nclear1) / (256 * 16), 2048);
    const int npack = pack ? static_cast<int>(std::max<int64_t>((static_cast<int64_t>(L.ntot) + 255) / 256, clear)) : 0;
    const dim3 g(static_cast<unsigned>(nrows) + npack), b(256);
    if (L.dim == 2) hipLaunchKernelGGL(k_pack<2>, g, b, 0, st, L, a, t, nrows);
    else hipLaunchKernelGGL(k_pack<3>, g, b, 0, st, L, a, t, nrows);
    return hipGetLastError();
}

hipError_t launch_update_move(const Launch& L, const uint32_t* skey, const int* inv, const Update& u, int* err,
                              hipStream_t st)
{
    if (L.ntot == 0) return hipSuccess;
    const dim3 g((L.ntot + 255) / 256), b(256);
    if (L.dim == 2)
        hipLaunchKernelGGL(k_upd_move<2>, g, b, 0, st, L.sets, L.poffs, L.nsets, L.ntot, skey, inv, u.knew, u.mig,
                           u.leave, u.arrive, u.aslot, err);
    else
        hipLaunchKernelGGL(k_upd_move<3>, g, b, 0, st, L.sets, L.poffs, L.nsets, L.ntot, skey, inv, u.knew, u.mig,
                           u.leave, u.arrive, u.aslot, err);
    return hipGetLastError();
}

hipError_t launch_update_cells(const Launch& L, int* cell_start, int* cnt, const Update& u, int64_t* partial,
                               int* flags, hipStream_t st)
{
    const int nc = L.ncell_tot;
    hipLaunchKernelGGL(k_upd_counts, dim3((nc + 256) / 256), dim3(256), 0, st, nc, cell_start, u.leave, u.arrive,
                       cnt, u.cs_old);
    return launch_cell_scan(L, cnt, cell_start, partial, flags, st);
}

hipError_t launch_dense_cells(const Launch& L, const int* cell_start, const DenseBuild& d, hipStream_t st)
{
    const int nc = L.ncell_tot;
    const dim3 g((nc + 255) / 256), b(256);
    hipError_t e = scan_exclusive<int, int64_t>(d.usz, nc, d.uoff, d.partial, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_dense_units, dim3((nc + 256) / 256), b, 0, st, nc, cell_start, d.uoff, d.cap, d.usz,
                       d.wdense, d.nsl, d.dn, d.dbn);
    e = scan_exclusive<int, int>(d.nsl, nc, d.unit_off, d.partial, st);
    if (e != hipSuccess) return e;
    e = scan_exclusive<uint32_t, int64_t>(d.dbn, nc, d.dboff, d.partial, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_dense_unit_cells, g, b, 0, st, nc, d.nsl, d.unit_off, d.dn, d.ucell);
    return hipGetLastError();
}

bool dense_unions_sorted(int64_t nmax) { return nmax > static_cast<int64_t>(kUnionWindows) * kUnionWindow; }

hipError_t launch_dense_unions(const Launch& L, int64_t nmax, const int* cell_start, const uint32_t* skey, const int* perm,
                               const int* inv, const DenseBuild& d, hipStream_t st, int** ulist)
{
    *ulist = d.uv0;
    if (L.ntot == 0 || d.cap == 0) return hipSuccess;
    if (!dense_unions_sorted(nmax)) {
        if (L.dim == 2)
            hipLaunchKernelGGL(k_union_rank<2>, dim3(kUnionGrid), dim3(kUnionThreads), 0, st, L, cell_start, perm, d, d.uv0);
        else
            hipLaunchKernelGGL(k_union_rank<3>, dim3(kUnionGrid), dim3(kUnionThreads), 0, st, L, cell_start, perm, d, d.uv0);
        return hipGetLastError();
    }
    const dim3 g((L.ntot + 255) / 256), b(256);
    if (L.dim == 2)
        hipLaunchKernelGGL(k_union_count<2>, g, b, 0, st, L.sets, L.coffs, L.nsets, L.ntot, skey, inv, d.usz, d.dn,
                           d.ecnt);
    else
        hipLaunchKernelGGL(k_union_count<3>, g, b, 0, st, L.sets, L.coffs, L.nsets, L.ntot, skey, inv, d.usz, d.dn,
                           d.ecnt);
    hipError_t e = scan_exclusive<int, int>(d.ecnt, L.ntot, d.epos, d.partial, st, d.dn);
    if (e != hipSuccess) return e;
    if (L.dim == 2)
        hipLaunchKernelGGL(k_union_emit<2>, g, b, 0, st, L.sets, L.coffs, L.nsets, L.ntot, skey, inv, d.usz, d.dn,
                           d.epos, d.uk0, d.uv0);
    else
        hipLaunchKernelGGL(k_union_emit<3>, g, b, 0, st, L.sets, L.coffs, L.nsets, L.ntot, skey, inv, d.usz, d.dn,
                           d.epos, d.uk0, d.uv0);
    const int keybits = std::max(1, 32 - __builtin_clz(static_cast<unsigned>(std::max(L.ncell_tot - 1, 1))));
    uint32_t* kf = nullptr;
    e = radix_sort_kv_dev(static_cast<int>(d.cap), d.dn, keybits, d.uk0, d.uv0, d.uk1, d.uv1, d.table, d.partial,
                          st, &kf, ulist);
    if (e != hipSuccess) return e;
    return hipGetLastError();
}

hipError_t launch_rowptr(const Launch& L, const int* counts, int64_t* partial, int64_t* nnz, const int* inv,
                         int64_t* rsort, const RowptrExtras& rep, hipStream_t st)
{
    const int64_t m = L.ntot, nt = std::max<int64_t>(1, (m + kScanTile - 1) / kScanTile);
    const dim3 g(nt), b(kScanThreads);
    switch (scan_sums(counts, m, nt, true, partial, st, nullptr)) {
    case kScanSelf:
        hipLaunchKernelGGL(k_rowptr<kScanSelf>, g, b, 0, st, L.sets, L.poffs, L.nsets, counts, m, partial, nnz, inv, rsort, rep);
        break;
    case kScanFold:
        hipLaunchKernelGGL(k_rowptr<kScanFold>, g, b, 0, st, L.sets, L.poffs, L.nsets, counts, m, partial, nnz, inv, rsort, rep);
        break;
    default:
        hipLaunchKernelGGL(k_rowptr<kScanScanned>, g, b, 0, st, L.sets, L.poffs, L.nsets, counts, m, partial, nnz, inv,
                           rsort, rep);
    }
    return hipGetLastError();
}

}  // namespace nnps
