// SPH gradient of a scalar field over the CSR neighbour list, in binary64: the standard
// kernel-gradient sum (SPH method section, Eq. 2) with the cubic B-spline kernel (Eq. 3),
// and the normalised, volume-free first-order operator of the appendix (Eq. A5).
//
// Eight lanes per row: lane k of a row takes the row's entries k, k + 8, ..., the next
// entry's data on the way while one is computed; the partial sums are combined over the
// lanes by DPP. Rows of one wavefront are consecutive particles, so their neighbour lists
// overlap in cache, and where numbering follows position the lanes that are at the same entry
// of their rows read neighbouring particles.
// For each neighbour j of i:
//   dx = x_j - x_i (per axis), r = sqrt(dx0^2 + dx1^2 [+ dx2^2]), q = r / h (as r (1/h)),
//   dW/dq = -2q + 1.5q^2 (q < 1), -0.5(2 - q)^2 (1 <= q < 2), 0 beyond,
//   dW/dx_i = alpha_d / h * dW/dq * (x_i - x_j) / r   (0 when r = 0; as a product with 1/r),
// with alpha_d = 15 / (7 pi h^2) in 2D and 3 / (2 pi h^3) in 3D. Outputs per axis:
//   grad      = sum_j V_j f_j dW/dx_i                                  (Eq. 2)
//   grad_norm = sum_j (f_j - f_i) dW/dx_i / sum_j (x_j - x_i) dW/dx_i   (Eq. A5; 0 when the
//               denominator is 0)
#include "sph_kernels.h"

namespace nnps {

constexpr int kGradThreads = 256;
// Lanes per row. The kernel is bound by the gathers (the address units are busy nine tenths of
// the time), so lanes at neighbouring entries, which often are neighbouring particles, pay:
// with 4, 8 and 16 lanes a 100^3 lattice takes 280, 246 and 280 us, a 500 x 500 lattice 17, 21
// and 32, 300,000 randomly numbered points in 2D 94, 89 and 87. Entries in consecutive shares
// a lane, their indices four at a load, took 391 on the 100^3 lattice. (Sixteen lanes with the
// library's square root and division, no look-ahead and sums through LDS: 365, 44 and 89.)
constexpr int kRowLanes = 8;
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_mov_dpp(static_cast<int>(b), CTRL, 0xF, 0xF, false);
    const uint32_t hi = __builtin_amdgcn_mov_dpp(static_cast<int>(b >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, static_cast<uint64_t>(hi) << 32 | lo);
}

// Sum over a row's eight lanes, in every one of them: within quads, then with the mirror
// image, which holds the other quad's sum.
__device__ __forceinline__ double row_sum_f64(double v)
{
    static_assert(kRowLanes == 8, "three steps");
    v = __dadd_rn(v, dpp_f64<0xB1>(v));  // quad_perm 1,0,3,2
    v = __dadd_rn(v, dpp_f64<0x4E>(v));  // quad_perm 2,3,0,1
    return __dadd_rn(v, dpp_f64<0x141>(v));  // row_half_mirror
}

// r = sqrt(r2) and 1 / r (0 for r2 = 0). Inside 2^-900 .. 2^900 from the hardware's reciprocal
// square root (relative error below 2^-22) with one third-order step, y (1 + e/2 + 3 e^2/8),
// e = 1 - r2 y^2, and one Newton step each for r and 1 / r (Householder's and Heron's
// iterations): both within 0.51 units in the last place, as the library's square root
// followed by a division (which take about 30 operations where these take 12). Outside,
// where those residuals would underflow or overflow, the library's.
__device__ __forceinline__ void root_and_inverse(double r2, double& r, double& inv_r)
{
    const double y = __builtin_amdgcn_rsq(r2);
    const double e = __fma_rn(-__dmul_rn(r2, y), y, 1.0);
    const double y1 = __fma_rn(__dmul_rn(y, e), __fma_rn(0.375, e, 0.5), y);
    const double g = __dmul_rn(r2, y1);
    r = __fma_rn(__fma_rn(-g, g, r2), __dmul_rn(0.5, y1), g);
    inv_r = __fma_rn(y1, __fma_rn(-r, y1, 1.0), y1);
}

__device__ __forceinline__ bool root_in_range(double r2)  // false for 0, infinity and NaN too
{
    const uint32_t hi = static_cast<uint32_t>(__builtin_bit_cast(uint64_t, r2) >> 32);
    return hi - ((1023u - 900u) << 20) < (1800u << 20);
}

// dW/dq of the cubic B-spline without alpha_d (Eq. 3 differentiated in q = r / h), as a
// product: q (1.5 q - 2) inside q = 1, t (-t / 2) with t = max(2 - q, 0) from there on.
__device__ __forceinline__ double bspline_dwdq(double q)
{
    const double t = fmax(__dsub_rn(2.0, q), 0.0);
    const bool inner = q < 1.0;
    return __dmul_rn(inner ? q : t, inner ? __fma_rn(1.5, q, -2.0) : __dmul_rn(-0.5, t));
}

// OFF: unsigned type of a particle's byte offset (32 bits while they reach: one address
// operation per load instead of three).
template <int DIM, bool VOL, typename OFF>
__global__ void __launch_bounds__(kGradThreads)
k_sph_gradient(int n, double inv_h, double alpha_h, const double* __restrict__ pos, const double* __restrict__ f,
               const double* __restrict__ vol, const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
               int64_t ncol, double* __restrict__ grad, double* __restrict__ grad_norm, int* __restrict__ err)
{
    const int64_t i = (static_cast<int64_t>(blockIdx.x) * kGradThreads + threadIdx.x) / kRowLanes;
    const int sub = threadIdx.x & (kRowLanes - 1);
    if (i >= n) return;  // a row's lanes leave together
    double xi[DIM];
#pragma unroll
    for (int a = 0; a < DIM; ++a) xi[a] = pos[i * DIM + a];
    const double fi = f[i];
    // row bounds clamped to the column array, column indices outside [0, n) skipped: a
    // list inconsistent with ncol or n cannot make the kernel read outside its arrays, and
    // it is reported (kErrBadList) instead of passing silently
    const int64_t r0 = row_ptr[i], r1 = row_ptr[i + 1];
    const int64_t rs = min(max(r0, int64_t(0)), ncol);
    const int64_t re = min(max(r1, rs), ncol);
    bool bad = sub == 0 && (rs != r0 || re != r1);
    double s[DIM], num[DIM], den[DIM];  // without alpha_d / h and the sign of x_i - x_j
#pragma unroll
    for (int a = 0; a < DIM; ++a) s[a] = num[a] = den[a] = 0.0;
    struct Entry {
        double x[DIM], f, v;
        bool in;
    };
    // an index outside [0, n) reads particle i itself, and is skipped (its r2 is out of range)
    auto fetch = [&](int j, Entry& e) {
        e.in = static_cast<uint32_t>(j) < static_cast<uint32_t>(n);
        bad |= !e.in;
        const OFF o = e.in ? static_cast<OFF>(j) : static_cast<OFF>(i);
        typedef double pair __attribute__((ext_vector_type(2), aligned(8)));
        const char* p = reinterpret_cast<const char*>(pos) + (DIM == 3 ? (o + (o << 1)) << 3 : o << 4);
        const pair xy = *reinterpret_cast<const pair*>(p);
        e.x[0] = xy.x;
        e.x[1] = xy.y;
        if (DIM == 3) e.x[DIM - 1] = *reinterpret_cast<const double*>(p + 16);
        e.f = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(f) + (o << 3));
        if (VOL) e.v = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(vol) + (o << 3));
    };
    auto add = [&](const Entry& e) {
        double dx[DIM];
#pragma unroll
        for (int a = 0; a < DIM; ++a) dx[a] = __dsub_rn(e.x[a], xi[a]);
        double r2 = __dmul_rn(dx[0], dx[0]);
#pragma unroll
        for (int a = 1; a < DIM; ++a) r2 = __dadd_rn(r2, __dmul_rn(dx[a], dx[a]));
        double r, inv_r;
        root_and_inverse(r2, r, inv_r);
        if (!root_in_range(r2)) {
            if (!e.in) return;
            r = __dsqrt_rn(r2);
            inv_r = r > 0.0 ? __ddiv_rn(1.0, r) : 0.0;
        }
        const double g = __dmul_rn(bspline_dwdq(__dmul_rn(r, inv_h)), inv_r);
        const double vfj = VOL ? __dmul_rn(e.v, e.f) : e.f;
        const double df = __dsub_rn(e.f, fi);
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            const double gx = __dmul_rn(g, dx[a]);
            s[a] = __fma_rn(vfj, gx, s[a]);
            num[a] = __fma_rn(df, gx, num[a]);
            den[a] = __fma_rn(dx[a], gx, den[a]);
        }
    };
    // the row in pieces whose positions fit 32 bits (any list a search makes is one piece);
    // loads past the end read the last entry again
    constexpr int kPiece = 1 << 30;
    for (int64_t at = rs; at < re; at += kPiece) {
        const int len = static_cast<int>(min(re - at, static_cast<int64_t>(kPiece)));
        const int32_t* c = col + at;
        auto index = [&](int k) { return c[min(k, len - 1)]; };
        if (sub >= len) continue;
        Entry e0, e1;
        int k = sub;
        fetch(index(k), e0);
        int j = index(k + kRowLanes);
        for (;;) {
            fetch(j, e1);
            j = index(k + 2 * kRowLanes);
            add(e0);
            k += kRowLanes;
            if (k >= len) break;
            fetch(j, e0);
            j = index(k + 2 * kRowLanes);
            add(e1);
            k += kRowLanes;
            if (k >= len) break;
        }
    }
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        s[a] = row_sum_f64(s[a]);
        num[a] = row_sum_f64(num[a]);
        den[a] = row_sum_f64(den[a]);
    }
    if (bad) atomicOr(err, kErrBadList);
    if (sub < DIM) {  // lane a of a row writes axis a
        double so = s[0], no = num[0], de = den[0];
#pragma unroll
        for (int a = 1; a < DIM; ++a) {
            so = sub == a ? s[a] : so;
            no = sub == a ? num[a] : no;
            de = sub == a ? den[a] : de;
        }
        // a row that adds nothing gives +0, also where alpha_d / h overflows
        if (grad) grad[i * DIM + sub] = so != 0.0 ? -__dmul_rn(alpha_h, so) : 0.0;
        if (grad_norm) grad_norm[i * DIM + sub] = de != 0.0 ? __ddiv_rn(no, de) : 0.0;  // the factor cancels
    }
}

struct GradArgs {
    int n;
    double inv_h, alpha_h;
    const double *pos, *f, *vol;
    const int64_t* row_ptr;
    const int32_t* col;
    int64_t ncol;
    double *grad, *grad_norm;
    int* err;
};

template <int DIM, bool VOL, typename OFF>
void gradient_rows(const GradArgs& a, hipStream_t st)
{
    constexpr int kRows = kGradThreads / kRowLanes;
    hipLaunchKernelGGL((k_sph_gradient<DIM, VOL, OFF>), dim3((static_cast<unsigned>(a.n) + kRows - 1) / kRows),
                       dim3(kGradThreads), 0, st, a.n, a.inv_h, a.alpha_h, a.pos, a.f, a.vol, a.row_ptr, a.col, a.ncol,
                       a.grad, a.grad_norm, a.err);
}

template <int DIM>
void gradient_of(const GradArgs& a, hipStream_t st)
{
    const bool small = static_cast<int64_t>(a.n) * DIM * 8 <= INT32_MAX;
    if (a.vol) small ? gradient_rows<DIM, true, uint32_t>(a, st) : gradient_rows<DIM, true, uint64_t>(a, st);
    else small ? gradient_rows<DIM, false, uint32_t>(a, st) : gradient_rows<DIM, false, uint64_t>(a, st);
}

hipError_t launch_sph_gradient(int dim, int64_t n, double h, const double* pos, const double* f, const double* vol,
                               const int64_t* row_ptr, const int32_t* col, int64_t ncol, double* grad,
                               double* grad_norm, int* err, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    const double pi = 3.14159265358979323846;
    const double alpha = dim == 2 ? 15.0 / (7.0 * pi * h * h) : 3.0 / (2.0 * pi * h * h * h);
    const double alpha_h = alpha / h;
    const GradArgs a{static_cast<int>(n), 1.0 / h, alpha_h, pos, f, vol, row_ptr, col, ncol, grad, grad_norm, err};
    if (dim == 2) gradient_of<2>(a, st);
    else gradient_of<3>(a, st);
    return hipGetLastError();
}

}  // namespace nnps
