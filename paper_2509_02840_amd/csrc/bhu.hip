// bhu.hip -- gfx950 kernels of the Householder bidiagonal update (Section
// 3.3, Theorem 1, Algorithm 1).  Each step of the algorithm needs column k
// (then row k) of Q_i^T (B + b c^T) P_j, never formed: it is reached through
// matrix-vector products with the reflector collections Y (m x i), W (n x j)
// and the explicit inverses S = T^{-1}, Rv = R^{-1} of the unit upper
// triangular matrices of eq. (TR).  Those products stream Y, W, S and Rv and
// are bound by memory bandwidth; the products with Q and P at the end are
// dense contractions and run on the FP64 matrix cores.
#include <hip/hip_runtime.h>

#include "bhu.h"

namespace bdu {

namespace {

typedef double acc4 __attribute__((ext_vector_type(4)));

// The sum of s over 256 threads, in a fixed tree: t += t + 128, t + 64, ...
// (t: the thread among its 256, with 256 places in red).  Every thread of the
// workgroup calls it; the sum is in red[0] and returned to every thread.  The
// last six levels stay in a wavefront.
__device__ __forceinline__ double tree_sum(double *red, int t, double s)
{
    red[t] = s;
    __syncthreads();
    if (t < 64) {
        s = (red[t] + red[t + 128]) + (red[t + 64] + red[t + 192]);
        for (int w = 32; w > 0; w >>= 1) s += __shfl_down(s, w);
        if (t == 0) red[0] = s;
    }
    __syncthreads();
    return red[0];
}

__global__ __launch_bounds__(256) void bhu_gemv_t_kernel(const double *X, int64_t ld, int64_t rows, const double *v,
                                                         double alpha, double *out)
{
    const int64_t c = blockIdx.x;
    const double *col = X + c * ld;
    double s = 0.0;
    for (int64_t r = threadIdx.x; r < rows; r += 256) s = fma(col[r], v[r], s);
    __shared__ double red[256];
    s = tree_sum(red, threadIdx.x, s);
    if (threadIdx.x == 0) out[c] = alpha * s;
}

// out = base + e_unit + alpha X h.  The sum over the columns is in chunks of
// kChunk, added in order; within a chunk four partial sums take every fourth
// column.
//
// Up to kOnePass columns: a workgroup has 64 rows and four wavefronts for each
// chunk (wavefront g of a chunk takes its columns g, g + 4, ...; lane = row,
// so every column read is 512 contiguous bytes, all of them in flight), and
// adds the chunks itself.  The step is a chain of launches that cost their
// latency: n = 256 took 5.2 us in a first pass and 1.9 us in a second over
// the chunks, 4.2 us so (4.7 us with 16 rows a workgroup: more of them fetch
// from memory what a neighbour's L2 cache has).  More columns: those two
// passes, so that a few thousand rows spread over the chip.
constexpr int kChunk = 128;
constexpr int kOnePass = 4 * kChunk;

// Sum over columns c0 + g, c0 + g + 4, ... below c1 (at most kChunk columns
// from c0; past c1 the last one is loaded again).
__device__ __forceinline__ double chunk_sum(const double *X, int64_t ld, const double *h, int64_t hs, int64_t c0,
                                            int64_t c1, int g, int lane)
{
    constexpr int N = kChunk / 4;
    if (c0 >= c1) return 0.0;
    const int64_t hc = c0 + g + 4 * (lane % N);
    const uint64_t hl = __builtin_bit_cast(uint64_t, h[(hc < c1 ? hc : c1 - 1) * hs]);
    double x[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const int64_t c = c0 + g + 4 * q;
        x[q] = X[(c < c1 ? c : c1 - 1) * ld];
    }
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)hl, q);
        const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(hl >> 32), q);
        const double hq = __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
        if (c0 + g + 4 * q < c1) s = fma(x[q], hq, s);
    }
    return s;
}

__global__ __launch_bounds__(1024) void bhu_gemv_n_kernel(const double *X, int64_t ld, int64_t rows, int64_t cols,
                                                          const double *h, int64_t hs, double alpha,
                                                          const double *base, int64_t unit, double *out)
{
    __shared__ double red[kOnePass / kChunk][4][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = wave & 3,
              q = wave >> 2;
    const int64_t r = (int64_t)blockIdx.x * 64 + lane, rl = r < rows ? r : rows - 1;
    const int64_t c0 = (int64_t)q * kChunk, c1 = c0 + kChunk < cols ? c0 + kChunk : cols;
    red[q][g][lane] = chunk_sum(X + rl, ld, h, hs, c0, c1, g, lane);
    __syncthreads();
    if (threadIdx.x >= 64 || r >= rows) return;
    double t = 0.0;
    for (int k = 0; k * kChunk < cols; ++k) t += (red[k][0][lane] + red[k][1][lane]) + (red[k][2][lane] + red[k][3][lane]);
    const double b0 = (base ? base[r] : 0.0) + (r == unit ? 1.0 : 0.0);
    out[r] = fma(alpha, t, b0);
}

__global__ __launch_bounds__(256) void bhu_gemv_n_part_kernel(const double *X, int64_t ld, int64_t rows,
                                                               int64_t cols, const double *h, int64_t hs,
                                                               double *part, int64_t lp)
{
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int64_t r = (int64_t)blockIdx.x * 64 + lane;
    const int64_t c0 = (int64_t)blockIdx.y * kChunk;
    const int64_t c1 = c0 + kChunk < cols ? c0 + kChunk : cols;
    double s = 0.0;
    if (r < rows)
        for (int64_t c = c0 + g; c < c1; c += 4) s = fma(X[r + c * ld], h[c * hs], s);
    __shared__ double red[4][64];
    red[g][lane] = s;
    __syncthreads();
    if (g == 0 && r < rows) part[blockIdx.y * lp + r] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

__global__ __launch_bounds__(256) void bhu_gemv_n_sum_kernel(const double *part, int64_t lp, int64_t nch,
                                                             int64_t rows, double alpha, const double *base,
                                                             int64_t unit, double *out)
{
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r >= rows) return;
    double t = 0.0;
    for (int64_t q = 0; q < nch; ++q) t += part[q * lp + r];
    const double b0 = (base ? base[r] : 0.0) + (r == unit ? 1.0 : 0.0);
    out[r] = fma(alpha, t, b0);
}

// x = B p + bv (cv^T p) (B the m x n upper bidiagonal d, e), and out[c] =
// X(:, c)^T x; or with TR x = B^T p + cv (bv^T p) of n entries.  A workgroup
// per column, each with its own copy of the dot product and of x, which the
// first one stores: one launch where the dot, x and the products took three.
template <bool TR>
__global__ __launch_bounds__(256) void bhu_bmul_gemv_t_kernel(const double *d, const double *e, int64_t m, int64_t n,
                                                              const double *p, const double *bv, const double *cv,
                                                              double *x, const double *X, int64_t ld, int64_t cols,
                                                              double *out)
{
    __shared__ double red[256];
    const int64_t c = blockIdx.x, plen = TR ? m : n, len = TR ? n : m;
    const double *other = TR ? bv : cv, *mine = TR ? cv : bv, *col = X + c * ld;
    double s = 0.0;
    for (int64_t r = threadIdx.x; r < plen; r += 256) s = fma(other[r], p[r], s);
    const double dot = tree_sum(red, threadIdx.x, s);
    __syncthreads();
    s = 0.0;
    for (int64_t r = threadIdx.x; r < len; r += 256) {
        double v = 0.0;
        if constexpr (TR) {
            v = d[r] * p[r];
            if (r > 0) v = fma(e[r - 1], p[r - 1], v);
        } else {
            if (r < n) v = d[r] * p[r];
            if (r + 1 < n) v = fma(e[r], p[r + 1], v);
        }
        v = fma(mine[r], dot, v);
        if (c == 0) x[r] = v;
        if (c < cols) s = fma(col[r], v, s);
    }
    if (c >= cols) return;
    s = tree_sum(red, threadIdx.x, s);
    if (threadIdx.x == 0) out[c] = s;
}

// The reflector of a[off .. len) (alpha and y), and out[c] = beta X(:, c)^T y.
// A workgroup makes the reflector for itself and takes four columns, 256
// threads each; the first one stores it.  One launch for two.
__global__ __launch_bounds__(1024) void bhu_house_gemv_t_kernel(const double *a, int64_t off, int64_t len,
                                                                double *alpha, double *y, const double *X, int64_t ld,
                                                                int64_t cols, double beta, double *out)
{
    __shared__ double ss[1024];
    __shared__ int nz;
    __shared__ double scal[2];  // y[off] and the divisor (0: identity)
    double s = 0.0;
    int f = 0;
    for (int64_t t = off + 1 + threadIdx.x; t < len; t += 1024) {
        const double v = a[t];
        s = fma(v, v, s);
        f |= v != 0.0;
    }
    ss[threadIdx.x] = s;
    if (threadIdx.x == 0) nz = 0;
    __syncthreads();
    if (f) nz = 1;
    for (int w = 512; w > 64; w >>= 1) {
        if ((int)threadIdx.x < w) ss[threadIdx.x] += ss[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 64) {
        s = ss[threadIdx.x] + ss[threadIdx.x + 64];
        for (int w = 32; w > 0; w >>= 1) s += __shfl_down(s, w);
    }
    if (threadIdx.x == 0) {
        const double x0 = a[off], sigma = s;
        double al = x0;
        scal[0] = 0.0;
        scal[1] = 0.0;
        if (nz) {
            const double nrm = sqrt(fma(x0, x0, sigma));
            al = x0 >= 0.0 ? -nrm : nrm;
            const double y0 = x0 - al;
            const double yn = sqrt(fma(y0, y0, sigma));
            scal[0] = y0 / yn;
            scal[1] = yn;
        }
        if (blockIdx.x == 0) *alpha = al;
    }
    __syncthreads();
    const double y0 = scal[0], yn = scal[1];
    auto reflector = [&](int64_t t) { return yn != 0.0 ? (t == off ? y0 : (t > off ? a[t] / yn : 0.0)) : 0.0; };
    if (blockIdx.x == 0)
        for (int64_t t = threadIdx.x; t < len; t += 1024) y[t] = reflector(t);
    const int64_t c = (int64_t)blockIdx.x * 4 + threadIdx.x / 256;
    const int t = threadIdx.x % 256;
    s = 0.0;
    if (c < cols)
        for (int64_t r = t; r < len; r += 256) s = fma(X[r + c * ld], reflector(r), s);
    s = tree_sum(ss + threadIdx.x / 256 * 256, t, s);
    if (c < cols && t == 0) out[c] = beta * s;
}

__global__ __launch_bounds__(256) void bhu_copy_kernel(double *dst, const double *src, int64_t count)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) dst[i] = src ? src[i] : 0.0;
}

// v_mfma_f64_16x16x4f64: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]
// and holds D[l / 16 + 4 q][l % 16] in element q of its accumulator.
// (At least two wavefronts per SIMD are asked for, so that the accumulators
// stay in the vector registers.)
template <bool TB>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void bhu_gemm_kernel(const double *A, int64_t lda, const double *B, int64_t ldb,
                                                      double *C, int64_t ldc, int64_t m, int64_t n, int64_t K,
                                                      double alpha, double beta)
{
    const int l = threadIdx.x, rr = l / 16, cc = l % 16;
    const int64_t R0 = (int64_t)blockIdx.x * 64, J0 = (int64_t)blockIdx.y * 64;
    acc4 acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = acc4{0.0, 0.0, 0.0, 0.0};
    for (int64_t c0 = 0; c0 < K; c0 += 4) {
        const int64_t c = c0 + rr;
        double av[4], bv[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int64_t i = R0 + 16 * t + cc, j = J0 + 16 * t + cc;
            av[t] = (c < K && i < m) ? A[i + c * lda] : 0.0;
            bv[t] = (c < K && j < n) ? (TB ? B[j + c * ldb] : B[c + j * ldb]) : 0.0;
        }
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t i = R0 + 16 * a + rr + 4 * q, j = J0 + 16 * b + cc;
                if (i >= m || j >= n) continue;
                const double v = alpha * acc[a][b][q];
                C[i + j * ldc] = beta == 0.0 ? v : fma(beta, C[i + j * ldc], v);
            }
}

}  // namespace

hipError_t launch_bhu_gemv_t(const double *X, int64_t ld, int64_t rows, int64_t cols, const double *v, double alpha,
                             double *out, hipStream_t st)
{
    if (cols <= 0) return hipSuccess;
    hipLaunchKernelGGL(bhu_gemv_t_kernel, dim3((unsigned)cols), dim3(256), 0, st, X, ld, rows, v, alpha, out);
    return hipGetLastError();
}

hipError_t launch_bhu_gemv_n(const double *X, int64_t ld, int64_t rows, int64_t cols, const double *h, int64_t hs,
                             double alpha, const double *base, int64_t unit, double *out, double *part, int64_t lp,
                             hipStream_t st)
{
    if (rows <= 0) return hipSuccess;
    if (rows > lp) return hipErrorInvalidValue;
    const int64_t nch = (cols + kChunk - 1) / kChunk;
    if (cols <= kOnePass) {
        hipLaunchKernelGGL(bhu_gemv_n_kernel, dim3((unsigned)((rows + 63) / 64)),
                           dim3((unsigned)(256 * (nch > 0 ? nch : 1))), 0, st, X, ld, rows, cols, h, hs, alpha, base,
                           unit, out);
        return hipGetLastError();
    }
    if (nch > 0)
        hipLaunchKernelGGL(bhu_gemv_n_part_kernel, dim3((unsigned)((rows + 63) / 64), (unsigned)nch), dim3(256), 0,
                           st, X, ld, rows, cols, h, hs, part, lp);
    hipLaunchKernelGGL(bhu_gemv_n_sum_kernel, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, st,
                       (const double *)part, lp, nch, rows, alpha, base, unit, out);
    return hipGetLastError();
}

hipError_t launch_bhu_bmul_gemv_t(const double *d, const double *e, int64_t m, int64_t n, const double *p,
                                  const double *bv, const double *cv, bool transb, double *x, const double *X,
                                  int64_t ld, int64_t cols, double *out, hipStream_t st)
{
    const dim3 grid((unsigned)(cols > 0 ? cols : 1));
    if (transb)
        hipLaunchKernelGGL(bhu_bmul_gemv_t_kernel<true>, grid, dim3(256), 0, st, d, e, m, n, p, bv, cv, x, X, ld, cols,
                           out);
    else
        hipLaunchKernelGGL(bhu_bmul_gemv_t_kernel<false>, grid, dim3(256), 0, st, d, e, m, n, p, bv, cv, x, X, ld,
                           cols, out);
    return hipGetLastError();
}

hipError_t launch_bhu_house_gemv_t(const double *a, int64_t off, int64_t len, double *alpha, double *y,
                                   const double *X, int64_t ld, int64_t cols, double beta, double *out, hipStream_t st)
{
    if (off < 0 || off >= len) return hipErrorInvalidValue;
    hipLaunchKernelGGL(bhu_house_gemv_t_kernel, dim3((unsigned)(cols > 0 ? (cols + 3) / 4 : 1)), dim3(1024), 0, st, a,
                       off, len, alpha, y, X, ld, cols, beta, out);
    return hipGetLastError();
}

hipError_t launch_bhu_copy(double *dst, const double *src, int64_t count, hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(bhu_copy_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, dst, src, count);
    return hipGetLastError();
}

hipError_t launch_bhu_gemm(const double *A, int64_t lda, const double *B, int64_t ldb, bool transb, double *C,
                           int64_t ldc, int64_t m, int64_t n, int64_t K, double alpha, double beta, hipStream_t st)
{
    if (m <= 0 || n <= 0) return hipSuccess;
    const dim3 grid((unsigned)((m + 63) / 64), (unsigned)((n + 63) / 64));
    if (transb)
        hipLaunchKernelGGL(bhu_gemm_kernel<true>, grid, dim3(64), 0, st, A, lda, B, ldb, C, ldc, m, n, K, alpha, beta);
    else
        hipLaunchKernelGGL(bhu_gemm_kernel<false>, grid, dim3(64), 0, st, A, lda, B, ldb, C, ldc, m, n, K, alpha,
                           beta);
    return hipGetLastError();
}

}  // namespace bdu
