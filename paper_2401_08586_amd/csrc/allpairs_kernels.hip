// All-list neighbour search for small sets (SPH method section, Fig. 3a: every particle
// tested against every other; the paper finds it faster than cell lists below about 1e4
// particles). Binary64 throughout, with the same predicate as the cell-list paths
// (r2 = ((dx0^2) + dx1^2) + dx2^2 in that order, no contraction, r2 <= R^2), so rows and
// distances are bit-identical to the FP64 cell list.
//
// A wavefront takes one to four rows and walks all candidates, 64 at a time, one a lane: a
// ballot gives a row's accepted candidates of a step, its population the row's count, and
// the lanes before a lane its place in the row, so entries come out in ascending j with no
// sort and neighbouring lanes write neighbouring entries. The small sets this is for are
// bound by latency: 2000 points are 32 steps, of which eight are loaded while the eight
// before are tested; count and fill take 8 and 10 us there (one row a lane against slices of
// the candidates, through LDS, was a chain of 256 tests of four dependent FP64 operations in
// 256 wavefronts: 14 and 41 us, and two more launches and two copies). A search of 2000
// points in 3D takes 32 us instead of 78, of 12,000 150 instead of 186.
#include "allpairs_kernels.h"

#include <type_traits>

namespace nnps {

namespace {

constexpr int kApThreads = 256;
constexpr int kApWaves = kApThreads / 64;

// Visit the candidates of R rows from row i0 on: f(r, j0, r2) for each step, r2 the squared
// distance of row i0 + r to candidate j0 + lane (itself among them; NaN past the last).
template <int DIM, int R, typename F>
__device__ __forceinline__ void walk(int n, int i0, const double* __restrict__ pos, F&& f)
{
    const int lane = threadIdx.x & 63;
    const double nan = __builtin_nan("");
    double p[R][DIM];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int k = 0; k < DIM; ++k) p[r][k] = i0 + r < n ? pos[static_cast<size_t>(i0 + r) * DIM + k] : nan;
    constexpr int AHEAD = R == 1 ? 8 : 4;  // steps loaded together, and while those before are tested
    double q[2][AHEAD][DIM];
    auto load = [&](double (&d)[AHEAD][DIM], int t0) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int j = t0 + 64 * u + lane;
            const double* src = pos + static_cast<size_t>(min(j, n - 1)) * DIM;
#pragma unroll
            for (int k = 0; k < DIM; ++k) d[u][k] = src[k];
            if (j >= n) d[u][0] = nan;  // accepted by no row
        }
    };
    auto test = [&](const double (&d)[AHEAD][DIM], int t0) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const double d0 = __dsub_rn(d[u][0], p[r][0]);
                const double d1 = __dsub_rn(d[u][1], p[r][1]);
                double r2 = __dadd_rn(__dmul_rn(d0, d0), __dmul_rn(d1, d1));
                if (DIM == 3) {
                    const double d2 = __dsub_rn(d[u][DIM - 1], p[r][DIM - 1]);
                    r2 = __dadd_rn(r2, __dmul_rn(d2, d2));
                }
                f(r, t0 + 64 * u, r2);
            }
        }
    };
    constexpr int STEP = 64 * AHEAD;
    load(q[0], 0);
    for (int t0 = 0; t0 < n; t0 += 2 * STEP) {
        load(q[1], t0 + STEP);
        test(q[0], t0);
        if (t0 + STEP >= n) break;
        load(q[0], t0 + 2 * STEP);
        test(q[1], t0 + STEP);
    }
}

// Counts of kApWaves * R rows into row_ptr[i + 1]; bit 0 of *bad: a position outside
// [lo, hi] or not finite.
template <int DIM, int R>
__global__ void __launch_bounds__(kApThreads)
k_allpairs_count(int n, const double* __restrict__ pos, double R2, ApBox box, int64_t* __restrict__ row_ptr,
                 int* __restrict__ flag)
{
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i0 = (static_cast<int>(blockIdx.x) * kApWaves + wv) * R;
    int c[R] = {};
    walk<DIM, R>(n, i0, pos, [&](int r, int, double r2) { c[r] += r2 <= R2 ? 1 : 0; });
    int mine = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) c[r] += __shfl_xor(c[r], o, 64);
        mine = lane == r ? c[r] : mine;
    }
    if (lane < R && i0 + lane < n) {
        bool bad = false, self = true;
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            const double x = pos[static_cast<size_t>(i0 + lane) * DIM + k];
            bad |= !(x >= box.lo[k] && x <= box.hi[k]);
            self &= __dsub_rn(x, x) == 0.0;
        }
        // less the row itself, which is among those counted if its position is finite
        row_ptr[i0 + lane + 1] = mine - (self ? 1 : 0);
        if (bad) atomicOr(flag, 1);
    }
}

// One workgroup: the counts in row_ptr[1..n] replaced by their inclusive prefix sums, row_ptr[0]
// = 0; nnz and the flag to `host`, and the flag zero again. (As the work of the count's last
// workgroup it saved a launch of 4 us, but the fence that every workgroup then needs cost 14.)
constexpr int kApScanThreads = 1024;

__global__ void __launch_bounds__(kApScanThreads)
k_allpairs_scan(int n, int64_t* __restrict__ row_ptr, int* __restrict__ flag, int64_t* __restrict__ host)
{
    constexpr int PER = 4, TILE = kApScanThreads * PER, WAVES = kApScanThreads / 64;
    __shared__ int64_t s_wave[WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int64_t carry = 0;
    for (int t0 = 0; t0 < n; t0 += TILE) {
        const int e0 = t0 + tid * PER;
        int64_t v[PER], sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) v[k] = e0 + k < n ? row_ptr[e0 + k + 1] : 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            sum += v[k];
            v[k] = sum;
        }
        int64_t inc = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t y = __shfl_up(inc, o, 64);
            if (lane >= o) inc += y;
        }
        if (lane == 63) s_wave[wv] = inc;
        __syncthreads();
        int64_t base = carry + inc - sum;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            if (w < wv) base += s_wave[w];
            carry += s_wave[w];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (e0 + k < n) row_ptr[e0 + k + 1] = base + v[k];
    }
    if (tid == 0) {
        row_ptr[0] = 0;
        host[0] = carry;
        host[1] = atomicExch(flag, 0);
    }
}

// Row i's entries at [row_ptr[i], min(row_ptr[i + 1], cap)), never outside; a row that finds
// more or fewer pairs than that (the positions or row pointers changed since the count) sets
// bit kApErrFill of *err. Accepted candidates gather in LDS, 64 are written at a time: the
// square roots are then taken by full wavefronts.
template <int DIM, int R>
__global__ void __launch_bounds__(kApThreads)
k_allpairs_fill(int n, const double* __restrict__ pos, double R2, const int64_t* __restrict__ row_ptr,
                int32_t* __restrict__ col, float* __restrict__ dist, int64_t cap, int* __restrict__ err)
{
    __shared__ double s_r2[kApWaves][R][128];
    __shared__ int s_col[kApWaves][R][128];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i0 = (static_cast<int>(blockIdx.x) * kApWaves + wv) * R;
    int64_t w[R], wend[R];
    int held[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        w[r] = wend[r] = 0;
        held[r] = 0;
        if (i0 + r < n) {
            w[r] = max(row_ptr[i0 + r], int64_t(0));
            wend[r] = min(row_ptr[i0 + r + 1], cap);
        }
    }
    auto put = [&](int r, int m) {  // the first m <= 64 held entries
        const int64_t at = w[r] + lane;
        if (lane < m && at < wend[r]) {
            col[at] = s_col[wv][r][lane];
            dist[at] = static_cast<float>(__dsqrt_rn(s_r2[wv][r][lane]));
        }
        w[r] += m;
    };
    walk<DIM, R>(n, i0, pos, [&](int r, int j0, double r2) {
        uint64_t acc = __ballot(r2 <= R2);
        if (!acc) return;
        const uint32_t self = static_cast<uint32_t>(i0 + r - j0);
        if (self < 64u) acc &= ~(1ull << self);
        const uint32_t before = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(acc >> 32),
                                                          __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(acc), 0));
        if (acc >> lane & 1) {
            s_r2[wv][r][held[r] + before] = r2;
            s_col[wv][r][held[r] + before] = j0 + lane;
        }
        held[r] += __builtin_popcountll(acc);
        if (held[r] >= 64) {
            // the buffers are the wavefront's own: its LDS operations complete in order
            __builtin_amdgcn_wave_barrier();
            put(r, 64);
            const double x = s_r2[wv][r][64 + lane];
            const int y = s_col[wv][r][64 + lane];
            __builtin_amdgcn_wave_barrier();
            s_r2[wv][r][lane] = x;
            s_col[wv][r][lane] = y;
            held[r] -= 64;
        }
        __builtin_amdgcn_wave_barrier();
    });
    bool off = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        put(r, held[r]);
        off |= w[r] != wend[r];
    }
    if (off && lane == 0) atomicOr(err, kApErrFill);
}

// Rows a wavefront takes: one while the rows alone are few for the chip's 1024 SIMDs, more
// for larger sets, where each candidate loaded then serves several. A search in 3D with 1, 2
// and 4 rows: 31.4, 31.4, - us at 2048 points; 40.8, 38.5, - at 3000; 97, 66, 77 at 6000;
// 153, 93, 92 at 8000; 313, 177, 150 at 12,000.
template <typename F>
void by_rows(int n, F&& f)
{
    if (n <= 2048) f(std::integral_constant<int, 1>{});
    else if (n <= 8192) f(std::integral_constant<int, 2>{});
    else f(std::integral_constant<int, 4>{});
}

template <int R>
dim3 grid_of(int n) { return dim3((n + kApWaves * R - 1) / (kApWaves * R)); }

}  // namespace

hipError_t launch_allpairs_count(int dim, int n, const double* pos, double R2, const ApBox& box, int64_t* row_ptr,
                                 int* flag, int64_t* host, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    by_rows(n, [&](auto r) {
        constexpr int R = decltype(r)::value;
        if (dim == 2)
            hipLaunchKernelGGL((k_allpairs_count<2, R>), grid_of<R>(n), dim3(kApThreads), 0, st, n, pos, R2, box, row_ptr,
                               flag);
        else
            hipLaunchKernelGGL((k_allpairs_count<3, R>), grid_of<R>(n), dim3(kApThreads), 0, st, n, pos, R2, box, row_ptr,
                               flag);
    });
    hipLaunchKernelGGL(k_allpairs_scan, dim3(1), dim3(kApScanThreads), 0, st, n, row_ptr, flag, host);
    return hipGetLastError();
}

hipError_t launch_allpairs_fill(int dim, int n, const double* pos, double R2, const int64_t* row_ptr, int32_t* col,
                                float* dist, int64_t cap, int* err, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    by_rows(n, [&](auto r) {
        constexpr int R = decltype(r)::value;
        if (dim == 2)
            hipLaunchKernelGGL((k_allpairs_fill<2, R>), grid_of<R>(n), dim3(kApThreads), 0, st, n, pos, R2, row_ptr, col,
                               dist, cap, err);
        else
            hipLaunchKernelGGL((k_allpairs_fill<3, R>), grid_of<R>(n), dim3(kApThreads), 0, st, n, pos, R2, row_ptr, col,
                               dist, cap, err);
    });
    return hipGetLastError();
}

}  // namespace nnps
