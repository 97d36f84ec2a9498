// track.hip -- gfx950 kernels of the subspace-tracking update (Brust &
// Saunders, Section 4, eqs. (lrup)-(bdlrup) and the unaugmented case after
// them): projections of b and c onto the tracked bases and their
// complements, the middle matrix's inputs, the truncation of the updated
// bidiagonal and the thin products.  The middle update itself is an
// ordinary BGU handle.  FP64; every sum is a sequential fma in a stated
// order.
#include <hip/hip_runtime.h>

#include "primitives.h"
#include "track.h"

namespace bdu {

// Row sums over a tracked basis run in chunks of kTrackChunk rows: a
// sequential fma from 0 inside a chunk (rows ascending), then the chunk
// partials added in ascending order from 0.

// part[side][k][j] = sum over the rows i of chunk k of A(i, j) x_i.  grid
// (chunks, ceil(cols / 64), 2 sides), one lane per column j; each lane runs
// down its own column, 32 loads ahead.
__global__ __launch_bounds__(64) void track_partial_kernel(TrackSides s, double *part, int64_t nchunk)
{
    const TrackSide &t = s.side[blockIdx.z];
    const int64_t i0 = (int64_t)blockIdx.x * kTrackChunk;
    const int64_t j = (int64_t)blockIdx.y * 64 + threadIdx.x;
    if (i0 >= t.rows || j >= t.cols) return;
    const int64_t i1 = i0 + kTrackChunk < t.rows ? i0 + kTrackChunk : t.rows;
    const double *a = t.A + j * t.lda;
    double p = 0.0;
    int64_t i = i0;
    for (; i + 32 <= i1; i += 32) {
        double av[32], xv[32];
#pragma unroll
        for (int q = 0; q < 32; ++q) {
            av[q] = a[i + q];
            xv[q] = t.x[i + q];
        }
#pragma unroll
        for (int q = 0; q < 32; ++q) p = fma(av[q], xv[q], p);
    }
    for (; i < i1; ++i) p = fma(a[i], t.x[i], p);
    part[((int64_t)blockIdx.z * nchunk + blockIdx.x) * t.cols + j] = p;
}

// xhat_j = sum over chunks k (ascending) of part[side][k][j], from 0.
// grid (ceil(cols / 64), 2 sides).
__global__ __launch_bounds__(64) void track_combine_kernel(TrackSides s, const double *part, int64_t nchunk)
{
    const TrackSide &t = s.side[blockIdx.y];
    const int64_t j = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (j >= t.cols) return;
    const int64_t nk = (t.rows + kTrackChunk - 1) / kTrackChunk;
    double total = 0.0;
    for (int64_t k = 0; k < nk; ++k) total = total + part[((int64_t)blockIdx.y * nchunk + k) * t.cols + j];
    t.xhat[j] = total;
}

// xperp_i = x_i - s_i, s_i = sum_j A(i, j) xhat_j (fma, j ascending); one
// block per chunk of rows, one lane per row (x may be xperp itself: each
// lane reads its entry before writing it); then the chunk's x_i^2 and
// xperp_i^2 are summed in row order (fma from 0) into npart[side][chunk], one
// chain by a lane of each of two wavefronts.  grid (chunks, 2 sides),
// kTrackChunk lanes.
//
// A has to be read once, and 12000 rows are 188 wavefronts: what counts is
// the loads each has in flight, two groups of 32 columns.  10000 x 2000 and
// 2000 x 2000: 473 us with a load at a time, 160 us so.
__global__ __launch_bounds__(kTrackChunk) void track_residual_kernel(TrackSides s, double *npart, int64_t nchunk)
{
    constexpr int G = 32;
    __shared__ double sq[2][kTrackChunk];  // x, xperp
    const TrackSide &t = s.side[blockIdx.y];
    const int64_t i0 = (int64_t)blockIdx.x * kTrackChunk;
    if (i0 >= t.rows) return;
    const int64_t i = i0 + threadIdx.x, il = i < t.rows ? i : t.rows - 1;
    const double *a = t.A + il;
    double acc = 0.0, u[G], v[G];
    auto load = [&](double(&x)[G], int64_t j) {
#pragma unroll
        for (int q = 0; q < G; ++q) x[q] = a[(j + q < t.cols ? j + q : t.cols - 1) * t.lda];
    };
    auto use = [&](const double(&x)[G], int64_t j) {
#pragma unroll
        for (int q = 0; q < G; ++q) acc = fma(x[q], t.xhat[j + q], acc);
    };
    int64_t j = 0;
    load(u, 0);
    for (; j + 2 * G <= t.cols; j += 2 * G) {
        load(v, j + G);
        use(u, j);
        load(u, j + 2 * G);
        use(v, j + G);
    }
    if (j + G <= t.cols) {
        use(u, j);
        j += G;
    }
    for (; j < t.cols; ++j) acc = fma(a[j * t.lda], t.xhat[j], acc);
    double xv = 0.0, xp = 0.0;
    if (i < t.rows) {
        xv = t.x[i];
        xp = xv - acc;
        t.xperp[i] = xp;
    }
    sq[0][threadIdx.x] = xv;
    sq[1][threadIdx.x] = xp;
    __syncthreads();
    if (threadIdx.x % 64 == 0 && threadIdx.x < 128) {
        const double *z = sq[threadIdx.x / 64];
        const int cnt = t.rows - i0 < kTrackChunk ? (int)(t.rows - i0) : kTrackChunk;
        double p = 0.0;
        int q = 0;
        for (; q + 16 <= cnt; q += 16) {
            double w[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) w[k] = z[q + k];
#pragma unroll
            for (int k = 0; k < 16; ++k) p = fma(w[k], w[k], p);
        }
        for (; q < cnt; ++q) p = fma(z[q], z[q], p);
        npart[2 * ((int64_t)blockIdx.y * nchunk + blockIdx.x) + threadIdx.x / 64] = p;
    }
}

// sums[2 side] = x^T x, sums[2 side + 1] = xperp^T xperp: the chunk
// partials added in ascending order from 0.  Lanes 0 and 1: the two sides.
__global__ __launch_bounds__(64) void track_sums_kernel(TrackSides s, const double *npart, int64_t nchunk,
                                                        double *sums)
{
    const int side = threadIdx.x;
    if (side > 1) return;
    const TrackSide &t = s.side[side];
    const int64_t nk = (t.rows + kTrackChunk - 1) / kTrackChunk;
    double tx = 0.0, tp = 0.0;
    for (int64_t k = 0; k < nk; ++k) {
        tx = tx + npart[2 * ((int64_t)side * nchunk + k)];
        tp = tp + npart[2 * ((int64_t)side * nchunk + k) + 1];
    }
    sums[2 * side] = tx;
    sums[2 * side + 1] = tp;
}

// xhat += add for the sides in mask (bit side).  grid (ceil(cols / 64), 2).
__global__ __launch_bounds__(64) void track_accumulate_kernel(TrackSides s, const double *add, int64_t r, int mask)
{
    const int side = blockIdx.y;
    if (!((mask >> side) & 1)) return;
    const int64_t j = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (j >= r) return;
    s.side[side].xhat[j] = s.side[side].xhat[j] + add[side * r + j];
}

// w_i = xperp_i / norm (in place) for each side with a positive norm.
// grid (ceil(rows / 256), 2 sides).
__global__ __launch_bounds__(256) void track_scale_kernel(TrackSides s, double delta, double gamma)
{
    const TrackSide &t = s.side[blockIdx.y];
    const double nrm = blockIdx.y == 0 ? delta : gamma;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (!(nrm > 0.0) || i >= t.rows) return;
    t.xperp[i] = t.xperp[i] / nrm;
}

// The middle factorization before its pass: Q = I (pm x pm, leading
// dimension ldq), P = I (pn x pn), and
//   not flipped: d = [d; 0], e = [e; 0] (pn and pn - 1 entries),
//                u = [b_hat; delta] (pm), v = [c_hat; gamma] (pn);
//   flipped:     d, e reversed (r, r - 1 entries), u = [J c_hat; gamma],
//                v = J b_hat (J: reversal of r entries).
// grid (pm), up to 1024 lanes.
__global__ void track_setup_kernel(TrackMiddle mid, TrackSides s, const double *d, const double *e, int r,
                                   double delta, double gamma, double *u, double *v)
{
    const int col = blockIdx.x;
    for (int i = threadIdx.x; i < mid.pm; i += blockDim.x) {
        mid.Q[i + (int64_t)col * mid.ldq] = i == col ? 1.0 : 0.0;
        if (col < mid.pn && i < mid.pn) mid.P[i + (int64_t)col * mid.ldp] = i == col ? 1.0 : 0.0;
    }
    if (col != 0) return;
    const double *bh = s.side[0].xhat, *ch = s.side[1].xhat;
    for (int i = threadIdx.x; i < mid.pm; i += blockDim.x) {
        if (!mid.flip) {
            u[i] = i < r ? bh[i] : delta;
            if (i < mid.pn) {
                v[i] = i < r ? ch[i] : gamma;
                mid.d[i] = i < r ? d[i] : 0.0;
                if (i + 1 < mid.pn) mid.e[i] = i + 1 < r ? e[i] : 0.0;
            }
        } else {
            u[i] = i < r ? ch[r - 1 - i] : gamma;
            if (i < r) {
                v[i] = bh[r - 1 - i];
                mid.d[i] = d[r - 1 - i];
                if (i + 1 < r) mid.e[i] = e[r - 2 - i];
            }
        }
    }
}

// The tracked bidiagonal after the pass.  Both sides augmented: drop the
// row and column k of the (r+1) x (r+1) result with the smallest column
// norm (d_k^2 + e_{k-1}^2 as fma(d_k, d_k, e_{k-1} e_{k-1}); ties drop the
// highest k), with 0 joining k-1 and k+1.  Otherwise the r x r result as it
// is (reversed back when flipped) and k = -1.  One block of 256 lanes.
__global__ __launch_bounds__(256) void track_truncate_kernel(TrackMiddle mid, int r, double *d, double *e,
                                                             int *kdrop)
{
    const int t = threadIdx.x;
    if (!(mid.aug[0] && mid.aug[1])) {
        for (int j = t; j < r; j += 256) d[j] = mid.d[mid.flip ? r - 1 - j : j];
        for (int j = t; j + 1 < r; j += 256) e[j] = mid.e[mid.flip ? r - 2 - j : j];
        if (t == 0) *kdrop = -1;
        return;
    }
    // The column of least norm, as a scan from j = R - 1 down that keeps the
    // first strictly smaller value would find it: the smallest value, the
    // highest index among equal ones, NaN norms never chosen, and R - 1 when
    // its own norm is NaN (nothing compares below a NaN).  Each lane scans a
    // strided share, then a tree over the lanes with the same rule.
    __shared__ double bv[256];
    __shared__ int bk[256];
    const int R = r + 1;
    auto norm = [&](int j) {
        return j == 0 ? mid.d[0] * mid.d[0] : fma(mid.d[j], mid.d[j], mid.e[j - 1] * mid.e[j - 1]);
    };
    double best = 0.0;
    int k = -1;
    for (int j = t; j < R; j += 256) {
        const double nj = norm(j);
        if (nj == nj && (k < 0 || nj < best || (nj == best && j > k))) {
            best = nj;
            k = j;
        }
    }
    bv[t] = best;
    bk[t] = k;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) {
            const double ov = bv[t + w];
            const int ok = bk[t + w];
            if (ok >= 0 && (bk[t] < 0 || ov < bv[t] || (ov == bv[t] && ok > bk[t]))) {
                bv[t] = ov;
                bk[t] = ok;
            }
        }
        __syncthreads();
    }
    if (t == 0) {
        const double top = norm(R - 1);
        bk[0] = (top != top || bk[0] < 0) ? R - 1 : bk[0];
        *kdrop = bk[0];
    }
    __syncthreads();
    const int kd = bk[0];
    for (int j = t; j < R - 1; j += 256) d[j] = mid.d[j < kd ? j : j + 1];
    for (int j = t; j + 1 < R - 1; j += 256) {
        const int a = j < kd ? j : j + 1, b = j + 1 < kd ? j + 1 : j + 2;
        e[j] = b == a + 1 ? mid.e[a] : 0.0;
    }
}

// out(i, j) = sum_{l < r} A(i, l) M(rm(l), cm(j)) [+ w_i M(r, cm(j))], each
// term an fma in that order.  Not flipped: M is the middle Q for side 0 and
// P for side 1, rm(l) = l, cm(j) = j, or j + 1 from the dropped index k on,
// and w (the unit complement) only on an augmented side.  Flipped
// (U2 = U J P3 J, V2 = [V, w] diag(J,1) Q3(:, 1:r) J): M is the middle P
// for side 0 and Q for side 1, rm(l) = r - 1 - l, cm(j) = r - 1 - j, and w
// on side 1 only.
//
// Register-tiled outer products, l running in order over the whole sum, so
// every entry is still the sequential fma chain above.  A block of four
// wavefronts has 64 R rows by 64 columns of out; a lane of wavefront w has R
// rows (64 apart) by columns 16 w .. 16 w + 15.  kProdChunk terms of A and M
// at a time are staged in LDS, double buffered, the next ones' loads in
// flight while these are used; a term's operands are read from there a term
// ahead (12 reads for 64 fma at R = 4; M is read as broadcasts).
// 10000 x 2000 and 2000 x 2000 by 2000: 2.81 ms (1.2 ms at the peak of the
// FP64 units; 3.16 without reading ahead, 3.63 with R = 2, 3.16 with 8 rows
// by 8 columns a lane), 4.52 ms with two rows and 32 columns a thread and A's
// loads waited for one by one.  grid (ceil(rows / (64 R)), ceil(r / 64), 2
// sides).
constexpr int kProdChunk = 8;

template <int R>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void track_product_kernel(
    TrackSides s, TrackMiddle mid, const int *kdrop, double *out0, double *out1)
{
    constexpr int ROWS = 64 * R, NA = kProdChunk * ROWS / 256;
    __shared__ double As[2][kProdChunk][ROWS];
    __shared__ __attribute__((aligned(16))) double Ms[2][kProdChunk][64];
    const int side = blockIdx.z;
    const TrackSide &t = s.side[side];
    const int64_t rows = t.rows, i0 = (int64_t)blockIdx.x * ROWS;
    if (i0 >= rows) return;  // the other side has more rows
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int r = (int)t.cols;
    const int j0 = blockIdx.y * 64;
    const int k = *kdrop;
    const bool useQ = mid.flip ? side == 1 : side == 0;
    const double *Mb = useQ ? mid.Q : mid.P;
    const int64_t ldm = useQ ? mid.ldq : mid.ldp;
    const bool with_w = mid.flip ? side == 1 : mid.aug[side] != 0;
    auto colof = [&](int j) { return mid.flip ? r - 1 - j : (k >= 0 && j >= k ? j + 1 : j); };
    double acc[R][16];
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
        for (int c = 0; c < 16; ++c) acc[q][c] = 0.0;
    // loads past the last row, term or column repeat the last one, for nobody
    const int arow = tid % ROWS;
    const double *ap = t.A + (i0 + arow < rows ? i0 + arow : rows - 1);
    const int ml = tid % kProdChunk, mc = tid / kProdChunk;  // and column mc + 32
    const double *mp[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int j = j0 + mc + 32 * q;
        mp[q] = Mb + (int64_t)colof(j < r ? j : r - 1) * ldm;
    }
    double av[NA], mv[2];
    auto load = [&](int l0) {
#pragma unroll
        for (int q = 0; q < NA; ++q) {
            const int l = l0 + tid / ROWS + q * (256 / ROWS);
            av[q] = ap[(int64_t)(l < r ? l : r - 1) * t.lda];
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int l = l0 + ml < r ? l0 + ml : r - 1;
            mv[q] = mp[q][mid.flip ? r - 1 - l : l];
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int q = 0; q < NA; ++q) As[buf][tid / ROWS + q * (256 / ROWS)][arow] = av[q];
#pragma unroll
        for (int q = 0; q < 2; ++q) Ms[buf][ml][mc + 32 * q] = mv[q];
    };
    // a term's operands, read from LDS one term ahead
    double a[2][R], m[2][16];
    auto read = [&](int set, int buf, int ll) {
#pragma unroll
        for (int q = 0; q < R; ++q) a[set][q] = As[buf][ll][64 * q + lane];
#pragma unroll
        for (int c = 0; c < 16; ++c) m[set][c] = Ms[buf][ll][16 * w + c];
    };
    auto use = [&](int set) {
#pragma unroll
        for (int c = 0; c < 16; ++c)
#pragma unroll
            for (int q = 0; q < R; ++q) acc[q][c] = fma(a[set][q], m[set][c], acc[q][c]);
    };
    load(0);
    store(0);
    __syncthreads();
    int buf = 0, l0 = 0;
    for (; l0 + kProdChunk <= r; l0 += kProdChunk) {
        load(l0 + kProdChunk);
        read(0, buf, 0);
#pragma unroll
        for (int ll = 0; ll < kProdChunk; ++ll) {
            if (ll + 1 < kProdChunk) read((ll + 1) % 2, buf, ll + 1);
            __builtin_amdgcn_sched_barrier(0);  // the reads go out before this term's fma
            use(ll % 2);
        }
        store(buf ^ 1);
        __syncthreads();
        buf ^= 1;
    }
    for (int ll = 0; l0 + ll < r; ++ll) {
        read(0, buf, ll);
        use(0);
    }
    double *out = side == 0 ? out0 : out1;
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        const int j = j0 + 16 * w + c;
        if (j >= r) break;
        const double mw = with_w ? Mb[r + (int64_t)colof(j) * ldm] : 0.0;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int64_t i = i0 + 64 * q + lane;
            if (i >= rows) continue;
            double v = acc[q][c];
            if (with_w) v = fma(t.xperp[i], mw, v);
            out[i + (int64_t)j * t.lda] = v;
        }
    }
}

hipError_t launch_track_project(const TrackSides &s, int64_t max_rows, int64_t r, double *part, hipStream_t st)
{
    const int64_t nchunk = (max_rows + kTrackChunk - 1) / kTrackChunk;
    hipLaunchKernelGGL(track_partial_kernel, dim3((unsigned)nchunk, (unsigned)((r + 63) / 64), 2), dim3(64), 0, st, s,
                       part, nchunk);
    hipLaunchKernelGGL(track_combine_kernel, dim3((unsigned)((r + 63) / 64), 2), dim3(64), 0, st, s,
                       (const double *)part, nchunk);
    return hipGetLastError();
}

hipError_t launch_track_complement(const TrackSides &s, int64_t max_rows, double *npart, double *sums,
                                   hipStream_t st)
{
    const int64_t nchunk = (max_rows + kTrackChunk - 1) / kTrackChunk;
    hipLaunchKernelGGL(track_residual_kernel, dim3((unsigned)nchunk, 2), dim3(kTrackChunk), 0, st, s, npart, nchunk);
    hipLaunchKernelGGL(track_sums_kernel, dim3(1), dim3(64), 0, st, s, (const double *)npart, nchunk, sums);
    return hipGetLastError();
}

hipError_t launch_track_accumulate(const TrackSides &s, const double *add, int64_t r, int mask, hipStream_t st)
{
    hipLaunchKernelGGL(track_accumulate_kernel, dim3((unsigned)((r + 63) / 64), 2), dim3(64), 0, st, s, add, r,
                       mask);
    return hipGetLastError();
}

hipError_t launch_track_scale(const TrackSides &s, int64_t max_rows, double delta, double gamma, hipStream_t st)
{
    hipLaunchKernelGGL(track_scale_kernel, dim3((unsigned)((max_rows + 255) / 256), 2), dim3(256), 0, st, s, delta,
                       gamma);
    return hipGetLastError();
}

hipError_t launch_track_setup(const TrackMiddle &mid, const TrackSides &s, const double *d, const double *e,
                              int64_t r, double delta, double gamma, double *u, double *v, hipStream_t st)
{
    hipLaunchKernelGGL(track_setup_kernel, dim3(mid.pm), dim3(mid.pm < 1024 ? ((mid.pm + 63) / 64) * 64 : 1024), 0,
                       st, mid, s, d, e, (int)r, delta, gamma, u, v);
    return hipGetLastError();
}

hipError_t launch_track_finish(const TrackSides &s, const TrackMiddle &mid, double *d, double *e, int *kdrop,
                               int64_t max_rows, int64_t r, double *out0, double *out1, hipStream_t st)
{
    hipLaunchKernelGGL(track_truncate_kernel, dim3(1), dim3(256), 0, st, mid, (int)r, d, e, kdrop);
    // Four rows a lane while that gives every CU a block; else one, for four
    // times as many blocks (10000 x 2000, r = 64: 19 us, 64 us before)
    const int64_t cols = (r + 63) / 64;
    if ((s.side[0].rows + s.side[1].rows) / 256 * cols >= 256)
        hipLaunchKernelGGL(track_product_kernel<4>, dim3((unsigned)((max_rows + 255) / 256), (unsigned)cols, 2),
                           dim3(256), 0, st, s, mid, kdrop, out0, out1);
    else
        hipLaunchKernelGGL(track_product_kernel<1>, dim3((unsigned)((max_rows + 63) / 64), (unsigned)cols, 2),
                           dim3(256), 0, st, s, mid, kdrop, out0, out1);
    return hipGetLastError();
}

}  // namespace bdu
