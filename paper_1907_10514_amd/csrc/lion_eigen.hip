// Eigenvalues of a dense symmetric FP64 matrix of order up to kEigenMax on the GPU:
// Householder tridiagonalisation, then one wave per eigenvalue bisecting with Sturm
// counts (Golub and Van Loan, Matrix Computations, sections 8.3 and 8.4).
//
// A matrix of order <= 192 is reduced inside one workgroup with every element in a
// register; a larger one first loses a column per launch over the whole chip.  Both
// are bound by the latency of a column (a norm, a product with the matrix and an
// inner product, each waiting for the last), not by the arithmetic.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lion_internal.h"
#include "lion_wave.h"

namespace lion {
namespace {

// Reflector of a column x (entries below the diagonal; x0 the first, sigma the sum of
// squares of the others): (I - beta v v^T) x = alpha e1 with v = x but v0 first.  Others
// whose squares add up to less than kTinySquare are taken as zero: beta could leave the
// range of a double, and against a matrix of norm kNormMin or more, the least that
// k_bisect accepts, what is left out is below 2^-150.
constexpr double kTinySquare = 0x1p-900, kNormMin = 0x1p-300, kNormMax = 0x1p+500;
struct Reflector {
    double beta, alpha, v0;
};

__device__ __forceinline__ Reflector reflector(double x0, double sigma) {
    Reflector h;
    if (sigma < kTinySquare) {
        h.beta = 0.0;
        h.alpha = x0;
        h.v0 = 0.0;
    } else {
        // the hardware's seeds with a cubic step each: every wave runs this chain
        const double s = fma(x0, x0, sigma);
        const double y0 = __builtin_amdgcn_rsq(s);
        const double e = fma(-(s * y0), y0, 1.0);
        const double y = fma(y0 * e, fma(e, 0.375, 0.5), y0);
        const double g = s * y, mu = fma(0.5 * y, fma(-g, g, s), g);
        h.alpha = x0 > 0.0 ? -mu : mu;
        h.v0 = x0 - h.alpha;
        const double q = mu * (mu + fabs(x0));
        const double z = __builtin_amdgcn_rcp(q), r = fma(-q, z, 1.0);
        h.beta = fma(z, fma(r, r, r), z);
    }
    return h;
}

// Arrays of the reduction (m doubles each unless said).
struct TriWork {
    double* d;        // diagonal
    double* e;        // off-diagonal
    double* v[2];     // reflector of a column, alternating
    double* p[2];     // matrix times reflector
    double* col[2];   // the next column before that reflector's update
    double* beta;     // [2]
};

// Column j of an order-m matrix per launch: every workgroup forms the update of
// reflector j - 1 and the reflector of column j for itself, then each wave updates
// one row of the trailing matrix, multiplies it by the new reflector and keeps its
// entry of column j + 1 for the next launch.  About 5.5 us a column at order 384, a
// launch and the chain through its two sums.
constexpr int kStepWaves = 4;
constexpr int kStepCols = kEigenMax / 64;

__global__ __launch_bounds__(64 * kStepWaves) void k_tri_step(double* __restrict__ A, int m,
                                                              int j, TriWork t) {
    __shared__ double v[kEigenMax], w[kEigenMax], x[kEigenMax];
    __shared__ double red[kStepWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cur = j & 1, old = cur ^ 1;
    const int i = j + 1 + (int)blockIdx.x * kStepWaves + wave;
    double a[kStepCols];
#pragma unroll
    for (int b = 0; b < kStepCols; ++b) {
        const int c = lane + 64 * b;
        a[b] = i < m && c < m && c > j ? A[(size_t)i * m + c] : 0.0;
    }
    // w = beta p - (beta / 2) (beta p . v) v of the last reflector
    const double beta0 = j > 0 ? t.beta[old] : 0.0;
    double dot = 0.0;
    for (int r = tid; r < m; r += 64 * kStepWaves) {
        const double vr = j > 0 && r >= j ? t.v[old][r] : 0.0;
        const double pr = j > 0 && r >= j ? beta0 * t.p[old][r] : 0.0;
        v[r] = vr;
        w[r] = pr;
        x[r] = j > 0 ? t.col[cur][r] : A[(size_t)r * m];
        dot = fma(pr, vr, dot);
    }
    dot = wave_sum(dot);
    if (lane == 0) red[wave] = dot;
    __syncthreads();
    dot = 0.0;
    for (int k = 0; k < kStepWaves; ++k) dot += red[k];
    const double half = 0.5 * beta0 * dot;
    const double vj = v[j], wj = fma(-half, vj, w[j]);
    __syncthreads();
    double sigma = 0.0;
    for (int r = tid; r < m; r += 64 * kStepWaves) {
        const double vr = v[r], wr = fma(-half, vr, w[r]);
        const double xr = r >= j ? x[r] - vr * wj - wr * vj : 0.0;
        w[r] = wr;
        x[r] = xr;
        if (r > j + 1) sigma = fma(xr, xr, sigma);
    }
    sigma = wave_sum(sigma);
    if (lane == 0) red[wave] = sigma;
    __syncthreads();
    sigma = 0.0;
    for (int k = 0; k < kStepWaves; ++k) sigma += red[k];
    const Reflector h = reflector(x[j + 1], sigma);
    if (blockIdx.x == 0) {
        for (int r = tid; r < m; r += 64 * kStepWaves)
            t.v[cur][r] = r > j + 1 ? (h.beta != 0.0 ? x[r] : 0.0) : (r == j + 1 ? h.v0 : 0.0);
        if (tid == 0) {
            t.d[j] = x[j];
            t.e[j] = h.alpha;
            t.beta[cur] = h.beta;
        }
    }
    if (i >= m) return;
    const double vi = v[i], wi = w[i];
    double s = 0.0;
#pragma unroll
    for (int b = 0; b < kStepCols; ++b) {
        const int c = lane + 64 * b;
        if (c >= m || c <= j) continue;
        const double n = a[b] - vi * w[c] - wi * v[c];
        if (j > 0) A[(size_t)i * m + c] = n;
        if (c == j + 1) t.col[old][i] = n;
        s = fma(n, c == j + 1 ? h.v0 : x[c], s);
    }
    s = wave_sum(s);
    if (lane == 0) t.p[cur][i] = s;
}

// The last n = m - j0 <= 64 NR columns inside one workgroup of 8 waves: wave g holds
// the columns g, g + 8, ... and lane l the rows l, l + 64, ... of the trailing matrix,
// 8 NR^2 elements a thread.  Per column: its reflector (every wave for itself), the
// product with the matrix (partial sums per wave, added over 8 lanes), and the
// rank-two update.  Three barriers a column.  What every wave does for itself and the
// broadcasts bound it, hence 8 waves, the most columns a wave's registers hold: order
// 192 takes 426 us (16 waves, entries broadcast by v_readlane: 523; the library's
// whole solver 3.6 ms).
constexpr int kTriWaves = 8;

template <int NR>
__global__ __launch_bounds__(64 * kTriWaves) void k_tri_regs(const double* __restrict__ A, int m,
                                                             int j0, TriWork t) {
    constexpr int NC = 64 * NR / kTriWaves, N = 64 * NR, S = N + 8;
    // column c of a vector sits at wave c % 8, entry c / 8: a wave reads its own in pairs
    // (two doubles of padding keep the lanes of a whole vector off one LDS bank)
    constexpr int NP = NC + 2;
    __shared__ __align__(16) double vbuf[2][kTriWaves][NP], pbuf[kTriWaves][NP];
    __shared__ double part[kTriWaves][S];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = m - j0;  // rows and columns below count from j0
    auto at = [](double(&buf)[kTriWaves][NP], int c) -> double& {
        return buf[c % kTriWaves][c / kTriWaves];
    };
    double a[NR][NC];
    // clamped loads, all in flight; outside the matrix zero
#pragma unroll
    for (int b = 0; b < NC; ++b) {
        const int c = wave + kTriWaves * b;
        const double* col = A + (size_t)(j0 + min(c, n - 1)) * m + j0;
#pragma unroll
        for (int q = 0; q < NR; ++q) a[q][b] = col[min(lane + 64 * q, n - 1)];
    }
#pragma unroll
    for (int b = 0; b < NC; ++b)
#pragma unroll
        for (int q = 0; q < NR; ++q)
            if (lane + 64 * q >= n || wave + kTriWaves * b >= n) a[q][b] = 0.0;
    if (j0 > 0) {
        // the update of reflector j0 - 1 is applied on the way in
        const int old = (j0 & 1) ^ 1;
        const double beta0 = t.beta[old];
        double vr[NR], wr[NR], dot = 0.0;
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            const int r = lane + 64 * q;
            vr[q] = r < n ? t.v[old][j0 + r] : 0.0;
            wr[q] = r < n ? beta0 * t.p[old][j0 + r] : 0.0;
            dot = fma(wr[q], vr[q], dot);
        }
        const double half = 0.5 * beta0 * wave_sum(dot);
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            wr[q] = fma(-half, vr[q], wr[q]);
            if (wave == 0) {
                at(vbuf[1], lane + 64 * q) = vr[q];
                at(pbuf, lane + 64 * q) = wr[q];
            }
        }
        __syncthreads();
#pragma unroll
        for (int b = 0; b < NC; ++b) {
            const double vc = vbuf[1][wave][b], wc = pbuf[wave][b];
#pragma unroll
            for (int q = 0; q < NR; ++q) a[q][b] = a[q][b] - vr[q] * wc - wr[q] * vc;
        }
        __syncthreads();
    }
    constexpr int G = 4;  // columns per test for what is left of the matrix
    for (int k = 0; k < n; ++k) {
        auto& vb = vbuf[k & 1];
        if (wave == k % kTriWaves) {
            const int bk = k / kTriWaves;
#pragma unroll
            for (int b0 = 0; b0 < NC; b0 += G) {
                if (b0 / G != bk / G) continue;
#pragma unroll
                for (int b = b0; b < b0 + G; ++b) {
                    if (b != bk) continue;
#pragma unroll
                    for (int q = 0; q < NR; ++q) {
                        const int r = lane + 64 * q;
                        at(vb, r) = r > k ? a[q][b] : 0.0;
                        if (r == k) t.d[j0 + k] = a[q][b];
                    }
                }
            }
        }
        if (k + 1 >= n) break;
        __syncthreads();
        double vr[NR], sigma = 0.0;
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            const int r = lane + 64 * q;
            vr[q] = at(vb, r);
            if (r > k + 1) sigma = fma(vr[q], vr[q], sigma);
        }
        double vc[NC];
#pragma unroll
        for (int b = 0; b < NC; ++b) vc[b] = vb[wave][b];
        const Reflector h = reflector(at(vb, k + 1), wave_sum(sigma));
        if (threadIdx.x == 0) t.e[j0 + k] = h.alpha;
        if (h.beta == 0.0) continue;  // the same in every thread
        if (wave == (k + 1) % kTriWaves) {
#pragma unroll
            for (int b = 0; b < NC; ++b)
                if (b == (k + 1) / kTriWaves) vc[b] = h.v0;
        }
#pragma unroll
        for (int q = 0; q < NR; ++q)
            if (lane + 64 * q == k + 1) vr[q] = h.v0;
        double s[NR];
#pragma unroll
        for (int q = 0; q < NR; ++q) s[q] = 0.0;
#pragma unroll
        for (int b0 = 0; b0 < NC; b0 += G) {
            if (kTriWaves * (b0 + G) <= k) continue;
#pragma unroll
            for (int b = b0; b < b0 + G; ++b)
#pragma unroll
                for (int q = 0; q < NR; ++q) s[q] = fma(a[q][b], vc[b], s[q]);
        }
#pragma unroll
        for (int q = 0; q < NR; ++q) part[wave][lane + 64 * q] = s[q];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            // eight rows a time, their eight partial sums in consecutive lanes
            const int r = (wave * NR + q) * 8 + (lane >> 3);
            const double p = row8_sum(part[lane & 7][r]);
            if ((lane & 7) == 0) at(pbuf, r) = r > k ? h.beta * p : 0.0;
        }
        __syncthreads();
        double wr[NR], dot = 0.0;
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            wr[q] = at(pbuf, lane + 64 * q);
            dot = fma(wr[q], vr[q], dot);
        }
        const double half = 0.5 * h.beta * wave_sum(dot);
#pragma unroll
        for (int q = 0; q < NR; ++q) wr[q] = fma(-half, vr[q], wr[q]);
#pragma unroll
        for (int b0 = 0; b0 < NC; b0 += G) {
            if (kTriWaves * (b0 + G) <= k) continue;
#pragma unroll
            for (int b = b0; b < b0 + G; ++b) {
                const double wc = fma(-half, vc[b], pbuf[wave][b]);
#pragma unroll
                for (int q = 0; q < NR; ++q) a[q][b] = a[q][b] - vr[q] * wc - wr[q] * vc[b];
            }
        }
    }
    if (threadIdx.x == 0) t.e[m - 1] = 0.0;
}

// Eigenvalues below x of T: sign changes of the leading minors p_i of T - x I,
//   p_{i+1} = (d_i - x) p_i - e_{i-1}^2 p_{i-1},
// one multiply-add on the dependent chain (the pivots p_{i+1} / p_i take a division:
// order 192 took 83 us with them, 41 with the minors).  T is scaled to norm 1 and no e^2 is below 2^-200, so
// eight minors neither overflow nor vanish, and then the last two are rescaled.
// de holds {d_i, e_{i-1}^2}, padded to a multiple of 8 by rows that never change sign.
__device__ __forceinline__ int sturm_count(const double2* de, int m8, double x) {
    int count = 0;
    double p0 = 0.0, p1 = 1.0;
    for (int i = 0; i < m8; i += 8) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const double2 r = de[i + k];
            const double p2 = fma(r.x - x, p1, -(r.y * p0));
            count += (int)((uint32_t)(__double2hiint(p1) ^ __double2hiint(p2)) >> 31);
            p0 = p1;
            p1 = p2;
        }
        const int e = max(__builtin_amdgcn_frexp_exp(p0), __builtin_amdgcn_frexp_exp(p1));
        p0 = __builtin_amdgcn_ldexp(p0, -e);
        p1 = __builtin_amdgcn_ldexp(p1, -e);
    }
    return count;
}

// One wave per eigenvalue: 64 points cut its interval into 65 parts a round, until
// the ends are neighbours to rounding.  Bound by the chain of m minors a round: 41 us
// at order 192.  NaN for a matrix that is not finite or (checked: not after k_scale) whose
// norm leaves its reduction's squares out of range.
__global__ __launch_bounds__(64) void k_bisect(TriWork t, int m, bool checked,
                                               double* __restrict__ W) {
    __shared__ double2 de[kEigenMax];
    const int lane = threadIdx.x, m8 = (m + 7) & ~7;
    double lo = __builtin_inf(), hi = -__builtin_inf();
    bool finite = true;
    for (int i = lane; i < m; i += 64) {
        const double di = t.d[i], ei = t.e[i], ep = i > 0 ? t.e[i - 1] : 0.0;
        const double rad = fabs(ei) + fabs(ep);
        lo = fmin(lo, di - rad);
        hi = fmax(hi, di + rad);
        finite = finite && __builtin_isfinite(di) && __builtin_isfinite(ei);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, off));
        hi = fmax(hi, __shfl_xor(hi, off));
    }
    const double norm = fmax(fabs(lo), fabs(hi));
    if (__ballot(!finite) != 0 || (checked && !(norm >= kNormMin && norm <= kNormMax))) {
        if (lane == 0) W[blockIdx.x] = __builtin_nan("");
        return;
    }
    if (norm == 0.0) {  // the zero matrix
        if (lane == 0) W[blockIdx.x] = 0.0;
        return;
    }
    const int ex = __builtin_amdgcn_frexp_exp(norm);
    for (int i = lane; i < m8; i += 64) {
        const double ep = i > 0 && i < m ? __builtin_amdgcn_ldexp(t.e[i - 1], -ex) : 0.0;
        de[i] = i < m ? make_double2(__builtin_amdgcn_ldexp(t.d[i], -ex), fmax(ep * ep, 0x1p-200))
                      : make_double2(4.0, 0.0);
    }
    __syncthreads();
    const int k = blockIdx.x;
    const double eps = 0x1p-52, pad = 4.0 * eps * m;
    lo = __builtin_amdgcn_ldexp(lo, -ex) - pad;
    hi = __builtin_amdgcn_ldexp(hi, -ex) + pad;
    for (int round = 0; round < 24; ++round) {
        const double width = hi - lo;
        if (!(width > fmax(eps * fmax(fabs(lo), fabs(hi)), 0x1p-56))) break;
        const double x = fma(width, (lane + 1) * (1.0 / 65.0), lo);
        // the points at or below the eigenvalue come first
        const int c = __popcll(__ballot(sturm_count(de, m8, x) <= k));
        const double l = __shfl(x, c > 0 ? c - 1 : 0), r = __shfl(x, c < 64 ? c : 63);
        const double nlo = c > 0 ? l : lo, nhi = c < 64 ? r : hi;
        if (nlo == lo && nhi == hi) break;
        lo = nlo;
        hi = nhi;
    }
    if (lane == 0) W[k] = __builtin_amdgcn_ldexp(0.5 * (lo + hi), ex);
}

// One workgroup: A (count entries) times the power of two that brings its largest entry
// into [1/2, 1), and that power's negative exponent; kNotFinite and A as it was if an entry
// is not finite.
__global__ __launch_bounds__(1024) void k_scale(double* __restrict__ A, int count,
                                                int* __restrict__ exponent) {
    __shared__ double top;
    __shared__ double red[16];
    const int tid = threadIdx.x;
    double mx = 0.0;
    for (int i = tid; i < count; i += 1024) {
        const double a = fabs(A[i]);
        mx = a <= 0x1.fffffffffffffp+1023 ? fmax(mx, a) : __builtin_inf();
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
    if ((tid & 63) == 0) red[tid >> 6] = mx;
    __syncthreads();
    if (tid == 0) {
        for (int k = 0; k < 16; ++k) mx = fmax(mx, red[k]);
        top = mx;
    }
    __syncthreads();
    const bool finite = __builtin_isfinite(top);
    const int e = finite ? __builtin_amdgcn_frexp_exp(top) : kNotFinite;
    if (tid == 0) *exponent = e;
    if (!finite) return;  // the same in every thread
    for (int i = tid; i < count; i += 1024) A[i] = __builtin_amdgcn_ldexp(A[i], -e);
}

// *flag = kNotFinite if one of the count entries is not finite.
__global__ __launch_bounds__(256) void k_matrix_finite(const double* __restrict__ A,
                                                       int64_t count, int* __restrict__ flag) {
    bool finite = true;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * 256)
        finite = finite && __builtin_isfinite(A[i]);
    if (!finite) *flag = kNotFinite;
}

}  // namespace

hipError_t launch_scale_matrix(double* A, int m, int* exponent, hipStream_t st) {
    if (m < 1 || m > kEigenMax) return hipErrorInvalidValue;
    k_scale<<<1, 1024, 0, st>>>(A, m * m, exponent);
    return hipGetLastError();
}

hipError_t launch_matrix_finite(const double* A, int64_t count, int* flag, hipStream_t st) {
    const unsigned g = (unsigned)std::min<int64_t>((count + 255) / 256, 4096);
    k_matrix_finite<<<g, 256, 0, st>>>(A, count, flag);
    return hipGetLastError();
}

size_t eigenvalues_scratch_bytes(int m) { return (size_t)(7 * m + 2) * sizeof(double); }

hipError_t launch_eigenvalues(double* A, int m, bool scaled, double* W, double* E,
                              void* scratch, hipStream_t st) {
    if (m < 1 || m > kEigenMax) return hipErrorInvalidValue;
    double* s = (double*)scratch;
    TriWork t{};
    t.d = s;
    t.e = E;
    t.v[0] = s + m;
    t.v[1] = s + 2 * m;
    t.p[0] = s + 3 * m;
    t.p[1] = s + 4 * m;
    t.col[0] = s + 5 * m;
    t.col[1] = s + 6 * m;
    t.beta = s + 7 * m;
    const int j0 = std::max(0, m - 192);
    for (int j = 0; j < j0; ++j)
        k_tri_step<<<(unsigned)((m - j - 1 + kStepWaves - 1) / kStepWaves), 64 * kStepWaves, 0,
                     st>>>(A, m, j, t);
    const int n = m - j0;
    if (n <= 64)
        k_tri_regs<1><<<1, 64 * kTriWaves, 0, st>>>(A, m, j0, t);
    else if (n <= 128)
        k_tri_regs<2><<<1, 64 * kTriWaves, 0, st>>>(A, m, j0, t);
    else
        k_tri_regs<3><<<1, 64 * kTriWaves, 0, st>>>(A, m, j0, t);
    k_bisect<<<m, 64, 0, st>>>(t, m, !scaled, W);
    return hipGetLastError();
}

}  // namespace lion
