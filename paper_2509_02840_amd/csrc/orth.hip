// orth.hip -- gfx950 kernels of the orthogonality monitor and correction
// (the paper reorthogonalizes its factors a few times over a stream; this is
// the dense-contraction part of the method, so it runs on the FP64 matrix
// cores: v_mfma_f64_16x16x4f64).
//
// Operand layout of v_mfma_f64_16x16x4f64 (D = A B + C, A 16 x 4, B 4 x 16):
// lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] and holds
// D[l / 16 + 4 q][l % 16] in element q of its 4-double accumulator.
#include <hip/hip_runtime.h>

#include "orth.h"

namespace bdu {

typedef double mfma_acc __attribute__((ext_vector_type(4)));

// E = X^T X - I on the blocks at or above the diagonal, each entry also
// written to its mirror, so E is exactly symmetric.  grid (nb, nb), nb =
// lde / 64; the contraction runs over the ld rows (padding rows are zero).
//
// Bound by the matrix cores: a 64 x 64 block over 2048 rows is 16 x 512
// instructions of 64 cycles, and 2048 columns have 528 blocks for 1024
// SIMDs.  So a block's four 32 x 32 quarters go to the four wavefronts of a
// workgroup (one wavefront per block left half of the SIMDs idle).  The MFMA
// operands run across columns of X, so 16-row x 64-column tiles of X are
// loaded down the columns (16 consecutive doubles per 16 lanes) into LDS,
// double buffered, the next two tiles' loads in flight while one is multiplied.  A tile column is 18 doubles apart: a 32-lane half of an operand
// read (columns c = 0..15, rows r and r+1) then meets 32 distinct bank pairs.
// Columns past k repeat the last one; their entries are not written.
// 2048 x 2048: 473 us with one wavefront per block, 290 us so (112 at the rate
// of the matrix cores if the blocks divided evenly, 164 as they do).
constexpr int kGramRows = 16, kGramPad = kGramRows + 2;

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void orth_gram_kernel(const double *X, int64_t ld, int64_t k, double *E,
                                                        int64_t lde)
{
    __shared__ double tile[2][2][64 * kGramPad];  // buffer, operand
    const int bi = blockIdx.x, bj = blockIdx.y;
    if (bj < bi) return;
    const int w = threadIdx.x / 64, l = threadIdx.x % 64, rr = l / 16, cc = l % 16;
    const int64_t I0 = (int64_t)bi * 64, J0 = (int64_t)bj * 64;
    const int i0 = 32 * (w / 2), j0 = 32 * (w % 2);  // this wavefront's quarter
    mfma_acc acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = mfma_acc{0.0, 0.0, 0.0, 0.0};
    // load q of a tile: row cc, column 16 w + 4 q + rr of the 64-column block
    const double *xi[4], *xj[4];
    int to[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int c = 16 * w + 4 * q + rr;
        xi[q] = X + cc + (I0 + c < k ? I0 + c : k - 1) * ld;
        xj[q] = X + cc + (J0 + c < k ? J0 + c : k - 1) * ld;
        to[q] = c * kGramPad + cc;
    }
    double pi[2][4], pj[2][4];
    auto load = [&](int set, int64_t r0) {
        r0 = r0 < ld ? r0 : 0;  // past the end, for nobody
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            pi[set][q] = xi[q][r0];
            pj[set][q] = xj[q][r0];
        }
    };
    auto store = [&](int set) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            tile[set][0][to[q]] = pi[set][q];
            tile[set][1][to[q]] = pj[set][q];
        }
    };
    auto multiply = [&](int buf) {
        const double *ta = tile[buf][0] + (i0 + cc) * kGramPad + rr, *tb = tile[buf][1] + (j0 + cc) * kGramPad + rr;
#pragma unroll
        for (int s4 = 0; s4 < kGramRows / 4; ++s4) {
            double av[2], bv[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                av[t] = ta[16 * t * kGramPad + 4 * s4];
                bv[t] = tb[16 * t * kGramPad + 4 * s4];
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
        }
    };
    load(0, 0);
    load(1, kGramRows);
    store(0);
    __syncthreads();
    // ld is a whole number of pairs of tiles
    for (int64_t r0 = 0; r0 < ld; r0 += 2 * kGramRows) {
#pragma unroll
        for (int set = 0; set < 2; ++set) {
            load(set, r0 + (2 + set) * kGramRows);
            multiply(set);
            __builtin_amdgcn_sched_barrier(0);  // the other set's loads are waited for here, not earlier
            store(1 - set);
            __syncthreads();
        }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t i = I0 + i0 + 16 * a + rr + 4 * q, j = J0 + j0 + 16 * b + cc;
                if (i >= k || j >= k || (bi == bj && i > j)) continue;
                const double v = acc[a][b][q] - (i == j ? 1.0 : 0.0);
                E[i + j * lde] = v;
                E[j + i * lde] = v;
            }
}

// part[j] = sum_i E(i, j)^2 over the k rows of column j (one block of 256
// lanes per column, a fixed tree), then out[0] = sqrt(sum_j part[j]).
__global__ __launch_bounds__(256) void orth_colsq_kernel(const double *E, int64_t k, int64_t lde, double *part)
{
    __shared__ double red[256];
    const int64_t j = blockIdx.x;
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < k; i += 256) s = fma(E[i + j * lde], E[i + j * lde], s);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[j] = red[0];
}

__global__ __launch_bounds__(256) void orth_sum_kernel(const double *part, int64_t k, double *out)
{
    __shared__ double red[256];
    double s = 0.0;
    for (int64_t j = threadIdx.x; j < k; j += 256) s += part[j];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = sqrt(red[0]);
}

// Y = X - (X E) / 2.  E is symmetric, so the B operand E(c, j) is read as
// E(j, c): both operands then run down columns.  grid (ld / 64, lde / 64),
// two wavefronts of 32 rows each.
//
// Bound by the matrix cores (a wavefront's 32 x 64 block over 2048 columns:
// 8 x 512 instructions of 64 cycles, two wavefronts per SIMD at 2048 x 2048)
// as long as the operands are there in time: they are loaded kAhead steps of
// four columns ahead.  At least two wavefronts per SIMD are asked for, which
// keeps the accumulators in the vector registers: with the whole register
// file the compiler moves them to the accumulation registers and back in
// every turn of the loop.  Rows of E past k only reach entries that are not
// written.  2048 x 2048: 664 us with one wavefront per 64 x 64 block and each
// step's loads waited for at once, 300 us so (218 at the rate of the matrix
// cores); 350 us with the operands of 128 x 64 blocks staged through LDS.
constexpr int kAhead = 4;

__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(2))) void orth_update_kernel(const double *X, int64_t ld, int64_t k, const double *E,
                                                          int64_t lde, double *Y)
{
    const int w = threadIdx.x / 64, l = threadIdx.x % 64, rr = l / 16, cc = l % 16;
    const int64_t R0 = (int64_t)blockIdx.x * 64 + 32 * w, J0 = (int64_t)blockIdx.y * 64;
    mfma_acc acc[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = mfma_acc{0.0, 0.0, 0.0, 0.0};
    auto multiply = [&](const double(&av)[2], const double(&bv)[4]) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
    };
    const int64_t steps = k / 4;  // whole ones
    const double *xp = X + (R0 + cc) + rr * ld, *ep = E + (J0 + cc) + rr * lde;
    double av[kAhead][2], bv[kAhead][4];
    int64_t at = 0;  // the step xp and ep are at
    // the next step's operands (past the last step, that one's again)
    auto load = [&](int slot) {
#pragma unroll
        for (int t = 0; t < 2; ++t) av[slot][t] = xp[16 * t];
#pragma unroll
        for (int t = 0; t < 4; ++t) bv[slot][t] = ep[16 * t];
        const bool more = ++at < steps;
        xp += more ? 4 * ld : 0;
        ep += more ? 4 * lde : 0;
    };
    if (steps > 0) {
#pragma unroll
        for (int s = 0; s < kAhead; ++s) load(s);
        int64_t c = 0;
        for (; c + kAhead <= steps; c += kAhead) {
#pragma unroll
            for (int s = 0; s < kAhead; ++s) {
                multiply(av[s], bv[s]);
                load(s);
            }
        }
#pragma unroll
        for (int s = 0; s < kAhead; ++s)
            if (c + s < steps) multiply(av[s], bv[s]);
    }
    if (k % 4) {  // the last columns
        const int64_t c = 4 * steps + rr;
        double at4[2], bt4[4];
#pragma unroll
        for (int t = 0; t < 2; ++t) at4[t] = c < k ? X[(R0 + 16 * t + cc) + c * ld] : 0.0;
#pragma unroll
        for (int t = 0; t < 4; ++t) bt4[t] = c < k ? E[(J0 + 16 * t + cc) + c * lde] : 0.0;
        multiply(at4, bt4);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t i = R0 + 16 * a + rr + 4 * q, j = J0 + 16 * b + cc;
                if (j >= k) continue;
                Y[i + j * ld] = X[i + j * ld] - 0.5 * acc[a][b][q];
            }
}

hipError_t launch_orth_gram(const double *X, int64_t ld, int64_t k, double *E, int64_t lde, hipStream_t st)
{
    if (ld % 128 || lde % 64 || lde < k || k < 1) return hipErrorInvalidValue;  // ld: whole 16-row tiles
    const unsigned nb = (unsigned)(lde / 64);
    hipLaunchKernelGGL(orth_gram_kernel, dim3(nb, nb), dim3(256), 0, st, X, ld, k, E, lde);
    return hipGetLastError();
}

hipError_t launch_orth_norm(const double *E, int64_t k, int64_t lde, double *part, double *out, hipStream_t st)
{
    hipLaunchKernelGGL(orth_colsq_kernel, dim3((unsigned)k), dim3(256), 0, st, E, k, lde, part);
    hipLaunchKernelGGL(orth_sum_kernel, dim3(1), dim3(256), 0, st, (const double *)part, k, out);
    return hipGetLastError();
}

hipError_t launch_orth_update(const double *X, int64_t ld, int64_t k, const double *E, int64_t lde, double *Y,
                              hipStream_t st)
{
    if (ld % 128 || lde % 64 || lde < k || k < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(orth_update_kernel, dim3((unsigned)(ld / 64), (unsigned)(lde / 64)), dim3(128), 0, st, X, ld,
                       k, E, lde, Y);
    return hipGetLastError();
}

}  // namespace bdu
