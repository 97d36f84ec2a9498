// kernels.hip -- gfx950 kernels of the Givens bidiagonal update
// (Brust & Saunders, Section 3.4, Algorithm 2).  FP64 throughout.
//
//  project_kernel  u = Q^T b, v = P^T c (eq. bidiagsubproblem); one lane per
//                  output, sequential fma over the rows, 64x64 tiles staged
//                  through LDS so that global reads stay coalesced.
//  spike_kernel    m > n: the reverse-order rotations that fold u(n+1:m)
//                  into u(n+1); a dependent chain, one lane.
//  (The generation of phases 1 and 2 is in gen.hip.)
//  apply_kernel    accumulates the rotation streams into Q and P
//                  (eq. bidiagplus): lanes own rows, a register window of
//                  columns slides along each block of chains, and the
//                  wavefronts of a workgroup form a pipeline that passes
//                  finished columns through LDS.  (The staged applier, the
//                  one the plain tilings use, is in apply.hip.)
//
// Rounding: every operation is rounded on its own (-ffp-contract=off);
// fma only where written; sqrt and division are IEEE.
#include <hip/hip_runtime.h>

#include "device.h"
#include "kernels.h"
#include "primitives.h"
#include "schedule.h"

namespace bdu {

__device__ __forceinline__ BlockDesc load_block(const BlockDesc *p, int b)
{
    const CONSTANT BlockDesc *q = kptr(p) + b;
    BlockDesc d;
    d.base = q->base;
    d.lmax = q->lmax;
    d.nfront = q->nfront;
    d.phase = q->phase;
    d.off = q->off;
    d.start = q->start;
    d.start2 = q->start2;
    return d;
}

// ---- projection ---------------------------------------------------------------

// grid (tiles, handles), 64 threads.  Tile t < ceil(m/64) projects with Q,
// the rest with P.  Lane l of tile t owns output column 64 t + l.
//
// Q and P have to be read once, by one wavefront per 64 columns: the next 64
// rows are on their way (32 KB a wavefront) while these are summed.
// 10000 x 2000: 357 us (172 us at the rate of a copy), 636 us with each
// tile waited for.
__global__ __launch_bounds__(64) void project_kernel(HandleDev *const *hs, Gate gate)
{
    if (gate.ranks && gate.pass >= gate.ranks[blockIdx.y]) return;
    const int pass = gate.pass;
    const CONSTANT HandleDev *h = kptr(hs[blockIdx.y]);
    const int m = h->m, n = h->n;
    const int qt = (m + 63) / 64, pt = (n + 63) / 64;
    int tile = blockIdx.x;
    if (tile >= qt + pt) return;
    const GLOBAL double *A;
    const GLOBAL double *x;
    GLOBAL double *out;
    int rows, ld;
    if (tile < qt) {
        A = gptr(h->Q); x = gptr(gate.xb ? gate.xb : h->bst) + (int64_t)pass * m; out = gptr(h->u); rows = m;
        ld = h->ldq;
    } else {
        tile -= qt;
        A = gptr(h->P); x = gptr(gate.xc ? gate.xc : h->cst) + (int64_t)pass * n; out = gptr(h->v); rows = n;
        ld = h->ldp;
    }
    const int cols = rows;
    __shared__ double tileA[64 * 65];
    __shared__ double xs[64];
    const int lane = threadIdx.x;
    const int col0 = tile * 64;
    double acc = 0.0, next[64], xn;
    // coalesced: lane reads row j0+lane of each of the tile's 64 columns
    // (rows past the end are padding inside the leading dimension)
    auto load = [&](int j0) {
#pragma unroll
        for (int c = 0; c < 64; ++c) {
            const int col = col0 + c < cols ? col0 + c : cols - 1;
            next[c] = A[(int64_t)col * ld + j0 + lane];
        }
        xn = j0 + lane < rows ? x[j0 + lane] : 0.0;
    };
    load(0);
    for (int j0 = 0; j0 < rows; j0 += 64) {
        const int jn = rows - j0 < 64 ? rows - j0 : 64;
#pragma unroll
        for (int c = 0; c < 64; ++c) tileA[c * 65 + lane] = next[c];
        xs[lane] = xn;
        if (j0 + 64 < rows) load(j0 + 64);
        __syncthreads();
        if (jn == 64) {
#pragma unroll
            for (int j = 0; j < 64; ++j) acc = fma(tileA[lane * 65 + j], xs[j], acc);
        } else {
            for (int j = 0; j < jn; ++j) acc = fma(tileA[lane * 65 + j], xs[j], acc);
        }
        __syncthreads();
    }
    if (col0 + lane < cols) out[col0 + lane] = acc;
}

// ---- spike (m > n) -----------------------------------------------------------------

// grid (handles), 64 threads.  For j = m..n+2 the pair (u_{j-1}, u_j) is
// rotated onto u_{j-1} (mode 2).  Rows n+1.. of the band are zero, so only u
// and the rotation list change.
__global__ __launch_bounds__(64) void spike_kernel(HandleDev *const *hs, Gate gate)
{
    if (gate.ranks && gate.pass >= gate.ranks[blockIdx.x]) return;
    const CONSTANT HandleDev *h = kptr(hs[blockIdx.x]);
    if (h->m <= h->n) return;
    const int m = h->m, n = h->n;
    __shared__ double chunk[64];
    double *u = h->u;
    double surv = u[m - 1];  // u_m
    int j = m;               // next pair is (u_{j-1}, u_j)
    while (j >= n + 2) {
        const int lo = (j - 64 > n + 1) ? j - 64 : n + 1;  // 1-based u indices lo..j-1
        const int cnt = j - lo;
        if ((int)threadIdx.x < cnt) chunk[threadIdx.x] = u[lo - 1 + threadIdx.x];
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int q = cnt - 1; q >= 0; --q) {  // pair (u_{lo+q}, u_{lo+q+1})
                double c, s, r;
                givens(chunk[q], surv, 2, c, s, r);
                h->csSp[m - (lo + q + 1)] = make_double2(c, s);
                chunk[q] = r;
                surv = r;
            }
        }
        __syncthreads();
        j = lo;
    }
    if (threadIdx.x == 0) {
        u[n] = surv;  // u_{n+1}
        for (int i = n + 1; i < m; ++i) u[i] = 0.0;
    }
}

// ---- application ----------------------------------------------------------------

__host__ __device__ constexpr int pmod(int a, int b) { return ((a % b) + b) % b; }

// Columns in the LDS ring between two wavefronts: at most 14 columns are live
// (written but not yet read), and 3 r with r | (K0 + 3) keeps slots static.
__host__ __device__ constexpr int ring_cols(int K0)
{
    int U = K0 + 3, r = 5;
    while (U % r) ++r;
    return 3 * r;
}

// Sweep one block of K = K0*NW chains over this workgroup's 64*R rows (lane l
// owns rows l, l+64, ..., l+64(R-1) of the panel).  Wavefront w holds local
// columns [3(f-K0+1), 3f+9] of its rows in registers (f = its local front),
// applies chains w*K0 .. w*K0+K0-1 at each front, and hands finished columns
// to wavefront w+1 through an LDS ring (the last wavefront writes them back to
// memory).  Every front of the loop has a slot per chain (identity where the
// chain has no rotation), so the body has no data-dependent branches around
// the rotations.  Columns outside the block are loaded from a clamped address
// and never stored: an identity rotation leaves a finite partner unchanged,
// and real rotations never touch them.  Each coefficient pair serves R rows.
template <int K0, int NW, int R, int MODE>
__device__ __forceinline__ void sweep(GLOBAL double *__restrict__ X, int ld, int ncols, int row0,
                                      const CONSTANT double *__restrict__ cs, const BlockDesc bd,
                                      double *ring, int w, int lane)
{
    constexpr int U = K0 + 3, WSZ = 3 * U, S = U, K = K0 * NW;
    constexpr bool DESC = MODE < 2;
    constexpr int DIR = DESC ? -1 : 1;
    const int lmax = bd.lmax;
    if (lmax < 0) return;
    const int nfront = bd.nfront;
    const int base = bd.base;
    // local columns lam in [lam_lo, lam_hi] exist in this block and matrix
    const int lam_hi = lmax + 1;
    const int lam_lo = DESC ? (base - ncols > 0 ? base - ncols : 0) : 0;
    const int col0 = base - 1;  // 0-based matrix column of local column 0
    double buf[R][WSZ];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < WSZ; ++i) buf[r][i] = 0.0;

    // column base address is uniform; the lane adds its row
    auto colptr = [&](int lam) -> const GLOBAL double * {
        int c = col0 + DIR * lam;
        c = c < 0 ? 0 : (c >= ncols ? ncols - 1 : c);
        return X + (int64_t)c * ld;
    };
    // ring slot of local column lam is lam mod RC (RC = ring_cols(K0) divides
    // WSZ, so the slot is a compile-time constant in the unrolled loop)
    constexpr int RC = ring_cols(K0);
    double *rin = ring + (w > 0 ? w - 1 : 0) * RC * 64 * R + lane;
    double *rout = ring + w * RC * 64 * R + lane;

    if (w == 0) {
#pragma unroll
        for (int k = 0; k <= 6; ++k) {
            const GLOBAL double *cp = colptr(k);
#pragma unroll
            for (int r = 0; r < R; ++r) buf[r][k] = cp[row0 + 64 * r];
        }
    }
    // Coefficients come in groups of G rotations.  The address of the group
    // after next (crossing into the next front at a front's end) is made
    // opaque two groups early, so its scalar loads are issued while the
    // current group computes but are never hoisted further (scalar registers
    // are few).
    constexpr int G = K0 % 4 == 0 ? 4 : 3;
    constexpr int NG = K0 / G;
    static_assert(K0 % G == 0 && NG >= 2 && K0 <= 24, "coefficient groups must tile a front");
    constexpr FrontOrder ord = front_order(MODE, K, K0);
    // Chunks of U = S fronts where this wavefront meets only identity
    // rotations (pipeline fill, local fronts f < 0; drain, after its last
    // column has left the window) only keep the workgroup's barriers.
    // Live chunks are F0 = w S + c U, c = 0 .. ceil((flush_end + 1) / U) - 1.
    const int flush_end = lam_hi / 3 + K0 - 1;
    const int nchunk = nfront / U;
    int live_end = w + (flush_end + U) / U;  // one past the last live chunk
    live_end = live_end < nchunk ? live_end : nchunk;
    auto idle = [&](int chunks) {
        if (NW > 1)
            for (int c = 0; c < chunks * U; ++c) __syncthreads();
    };
    idle(w);
    for (int F0 = w * S; F0 < live_end * U; F0 += U) {
        const CONSTANT double *pg = cs + 2 * ((int64_t)F0 * K + w * K0);
        const CONSTANT double *pg1 = pg + 2 * G;  // always two groups in flight
        asm volatile("" : "+s"(pg));
        asm volatile("" : "+s"(pg1));
#pragma unroll
        for (int phi = 0; phi < U; ++phi) {
            const int F = F0 + phi;
            const int f = F - w * S;
            // new columns: from memory (first wavefront, two fronts ahead) or
            // from the previous wavefront's ring
            if (w == 0) {
#pragma unroll
                for (int k = 7; k <= 9; ++k) {
                    const GLOBAL double *cp = colptr(3 * f + k);
#pragma unroll
                    for (int r = 0; r < R; ++r) buf[r][pmod(3 * phi + k, WSZ)] = cp[row0 + 64 * r];
                }
            } else {
                if (phi == 0 && f == 0) {
#pragma unroll
                    for (int r = 0; r < R; ++r) buf[r][0] = rin[64 * r];
                }
#pragma unroll
                for (int k = 1; k <= 3; ++k)
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        buf[r][pmod(3 * phi + k, WSZ)] = rin[(pmod(3 * phi + k, RC) * R + r) * 64];
            }
            // this wavefront's K0 rotations at front F, in front_order (their
            // coefficients are stored in that order)
            const CONSTANT double *csF = cs + 2 * ((int64_t)F * K + w * K0);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                // address of the group after next (crossing into the next front)
                const int gg = g + 2;
                const CONSTANT double *pn = csF + (gg < NG ? 2 * G * gg : 2 * K + 2 * G * (gg - NG));
                asm volatile("" : "+s"(pn));
#pragma unroll
                for (int q = 0; q < G; ++q) {
                    const int t = ord.t[g * G + q];
                    const int l0 = 3 * (phi - t) + rho_of(MODE, K, t);
                    const int sx = pmod(l0 + (DESC ? 1 : 0), WSZ);
                    const int sy = pmod(l0 + (DESC ? 0 : 1), WSZ);
                    const double c = pg[2 * q], sn = pg[2 * q + 1];
#pragma unroll
                    for (int r = 0; r < R; ++r) rot(c, sn, buf[r][sx], buf[r][sy]);
                }
                pg = pg1;
                pg1 = pn;
            }
            // finished columns leave the window
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int lam = 3 * (f - K0 + 1) + k;
                const int sl = pmod(3 * (phi - K0 + 1) + k, WSZ);
                if (w == NW - 1) {
                    if (lam >= lam_lo && lam <= lam_hi) {
                        GLOBAL double *cp = X + (int64_t)(col0 + DIR * lam) * ld;
#pragma unroll
                        for (int r = 0; r < R; ++r) cp[row0 + 64 * r] = buf[r][sl];
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < R; ++r) rout[(pmod(3 * (phi - K0 + 1) + k, RC) * R + r) * 64] = buf[r][sl];
                }
            }
            if (NW > 1) __syncthreads();
            // keep fronts in order: the columns in use (local 3(f-K0+1) ..
            // 3f+3) are materialised here, so the scheduler cannot interleave
            // two fronts (and their coefficients).  Columns loaded ahead are
            // left out: their loads stay in flight until first use.
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int j = -3 * (K0 - 1); j <= 3; ++j) asm volatile("" : "+v"(buf[r][pmod(3 * phi + j, WSZ)]));
        }
    }
    idle(nchunk - (live_end > w ? live_end : w));
}

// Spike rotations on Q columns (j-1, j), j = m..n+2, for one row: a running
// carry keeps column j between consecutive rotations.
__device__ void spike_apply(GLOBAL double *Q, int ld, int m, int n, int row, const CONSTANT double *cs)
{
    double carry = Q[(int64_t)(m - 1) * ld + row];
    for (int t = 0; t < m - n - 1; ++t) {
        const int xc = m - 2 - t;  // 0-based column of the pair's first entry
        double x = Q[(int64_t)xc * ld + row];
        rot(cs[2 * t], cs[2 * t + 1], x, carry);
        Q[(int64_t)(xc + 1) * ld + row] = carry;
        carry = x;
    }
    Q[(int64_t)n * ld + row] = carry;
}

// grid (panels, handles): panels [0, ceil(m/(64R))) update Q, the rest P.  Q
// and P have leading dimensions padded to a multiple of 128 rows.
//
// Occupancy: at one wavefront per SIMD a rotation loop issues at well under
// half the FP64 rate, so the register budget is capped to keep at least two
// wavefronts per SIMD (the (12, *, 2) tilings fit 256 registers without
// spilling; the smaller windows fit three).
template <int K0, int NW, int R>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(K0 * R >= 24 ? 2 : 3))) void apply_kernel(
    HandleDev *const *hs, Gate gate)
{
    // Workgroups are dispatched round-robin over the 8 XCDs.  Renumber them so
    // that the panels of one handle run on the same XCD and share its L2 copy
    // of the handle's rotation streams.
    const int total = gridDim.x * gridDim.y;
    const int lin = blockIdx.y * gridDim.x + blockIdx.x;
    int item = lin;
    if (total % 8 == 0) item = (lin % 8) * (total / 8) + lin / 8;
    const int hidx = item / gridDim.x, pid = item % gridDim.x;
    if (gate.ranks && gate.pass >= gate.ranks[hidx]) return;
    const CONSTANT HandleDev *h = kptr(hs[hidx]);
    const int m = h->m, n = h->n;
    constexpr int PH = 64 * R;
    const int qp = (m + PH - 1) / PH, pp = (n + PH - 1) / PH;
    if (pid >= qp + pp) return;
    constexpr int RING = (NW > 1 ? NW - 1 : 1) * ring_cols(K0) * 64 * R;
    __shared__ double ring[RING];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    // the ring starts finite (stale slots may meet identity rotations)
    for (int i = threadIdx.x; i < RING; i += 64 * NW) ring[i] = 0.0;
    const int nb1 = h->nb1;
    // blocks of this part (phase 1 = [0, nb1), phase 2 = [nb1, nb1 + nb2))
    int bbeg, bend;
    const bool spike_part = part_blocks(h, gate.part, &bbeg, &bend);
    const int b1a = bbeg < nb1 ? bbeg : nb1, b1e = bend < nb1 ? bend : nb1;  // phase-1 blocks [b1a, b1e)
    const int b2a = bbeg > nb1 ? bbeg : nb1, b2e = bend;                     // phase-2 blocks [b2a, b2e)
    if (pid < qp) {
        const int row0 = pid * PH + lane;
        GLOBAL double *Q = gptr(h->Q);
        if (m > n && w == 0 && spike_part) {
#pragma unroll
            for (int r = 0; r < R; ++r) spike_apply(Q, h->ldq, m, n, row0 + 64 * r, kptr((const double *)h->csSp));
        }
        __syncthreads();
        for (int b = b1a; b < b1e; ++b) {
            const BlockDesc bd = load_block(h->blkL, b);
            sweep<K0, NW, R, 0>(Q, h->ldq, m, row0, kptr((const double *)h->csL) + 2 * bd.off, bd, ring, w, lane);
            __syncthreads();
        }
        for (int b = b2a; b < b2e; ++b) {
            const BlockDesc bd = load_block(h->blkL, b);
            sweep<K0, NW, R, 2>(Q, h->ldq, m, row0, kptr((const double *)h->csL) + 2 * bd.off, bd, ring, w, lane);
            __syncthreads();
        }
    } else {
        const int row0 = (pid - qp) * PH + lane;
        GLOBAL double *P = gptr(h->P);
        for (int b = b1a; b < b1e; ++b) {
            const BlockDesc bd = load_block(h->blkR, b);
            sweep<K0, NW, R, 1>(P, h->ldp, n, row0, kptr((const double *)h->csR) + 2 * bd.off, bd, ring, w, lane);
            __syncthreads();
        }
        for (int b = b2a; b < b2e; ++b) {
            const BlockDesc bd = load_block(h->blkR, b);
            sweep<K0, NW, R, 3>(P, h->ldp, n, row0, kptr((const double *)h->csR) + 2 * bd.off, bd, ring, w, lane);
            __syncthreads();
        }
    }
}

// The rotation primitive on arrays (checks the device arithmetic against the
// reference bit for bit).
__global__ void givens_kernel(const double *a, const double *b, int mode, double *c, double *s, double *r,
                              int64_t count)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x) {
        double cc, ss, rr;
        givens(a[i], b[i], mode, cc, ss, rr);
        c[i] = cc;
        s[i] = ss;
        r[i] = rr;
    }
}

hipError_t launch_givens(const double *a, const double *b, int mode, double *c, double *s, double *r,
                         int64_t count, hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(givens_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a, b, mode, c, s, r, count);
    return hipGetLastError();
}

// Fill rotation streams with the identity (c, s) = (1, 0).
__global__ void fill_identity_kernel(double2 *p, int64_t count)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = make_double2(1.0, 0.0);
}

// ---- launchers ---------------------------------------------------------------------

hipError_t launch_project(HandleDev *const *hs, int count, int max_tiles, Gate gate, hipStream_t st)
{
    hipLaunchKernelGGL(project_kernel, dim3(max_tiles, count), dim3(64), 0, st, hs, gate);
    return hipGetLastError();
}

hipError_t launch_spike(HandleDev *const *hs, int count, Gate gate, hipStream_t st)
{
    hipLaunchKernelGGL(spike_kernel, dim3(count), dim3(64), 0, st, hs, gate);
    return hipGetLastError();
}

template <int K0, int NW, int R>
static hipError_t launch_apply_t(HandleDev *const *hs, int count, int max_panels, Gate gate, hipStream_t st)
{
    hipLaunchKernelGGL((apply_kernel<K0, NW, R>), dim3(max_panels, count), dim3(64 * NW), 0, st, hs, gate);
    return hipGetLastError();
}

// nw in {1, 2, 4, 8}: nw wavefronts, each loading or storing what it needs;
// nw in {3, 5, 7, 15}: the staged applier of apply.hip (k0 = 12: nw in {3, 7, 15}, rpl 2 only for nw <= 7; k0 = 18:
// nw in {3, 5, 7}, rpl 1).
static bool staged(int nw) { return nw == 3 || nw == 5 || nw == 7 || nw == 15; }

bool tiling_supported(int k0, int nw, int rpl)
{
    if (staged(nw)) {
        if (k0 == 12) return nw != 5 && (rpl == 1 || (rpl == 2 && nw != 15));
        return k0 == 18 && nw != 15 && rpl == 1;
    }
    if (k0 == 6 && nw == 8 && rpl == 2) return false;  // its LDS ring exceeds 160 KB
    return (k0 == 6 || k0 == 12) && (nw == 1 || nw == 2 || nw == 4 || nw == 8) && (rpl == 1 || rpl == 2);
}

hipError_t launch_apply(HandleDev *const *hs, int count, int max_panels, int k0, int nw, int rpl, bool spike,
                        Gate gate, hipStream_t st)
{
    if (staged(nw)) return launch_apply_staged(hs, count, max_panels, k0, nw, rpl, spike, gate, st);
#define BDU_APPLY_CASE(A, B, C) \
    if (k0 == A && nw == B && rpl == C) return launch_apply_t<A, B, C>(hs, count, max_panels, gate, st);
    BDU_APPLY_CASE(6, 1, 1) BDU_APPLY_CASE(6, 2, 1) BDU_APPLY_CASE(6, 4, 1) BDU_APPLY_CASE(6, 8, 1)
    BDU_APPLY_CASE(12, 1, 1) BDU_APPLY_CASE(12, 2, 1) BDU_APPLY_CASE(12, 4, 1) BDU_APPLY_CASE(12, 8, 1)
    BDU_APPLY_CASE(6, 1, 2) BDU_APPLY_CASE(6, 2, 2) BDU_APPLY_CASE(6, 4, 2)
    BDU_APPLY_CASE(12, 1, 2) BDU_APPLY_CASE(12, 2, 2) BDU_APPLY_CASE(12, 4, 2) BDU_APPLY_CASE(12, 8, 2)
#undef BDU_APPLY_CASE
    return hipErrorInvalidValue;
}

// flag[0] = 1 if any of the count values is NaN or infinite (flag[0] is
// cleared by the caller; every writer stores the same value).
__global__ void nonfinite_kernel(const double *p, int64_t count, int *flag)
{
    bool bad = false;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        bad |= !isfinite(p[i]);
    if (bad) flag[0] = 1;
}

hipError_t launch_nonfinite(const double *p, int64_t count, int *flag, hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(nonfinite_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, count, flag);
    return hipGetLastError();
}

hipError_t launch_fill_identity(double2 *p, int64_t count, hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_identity_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, count);
    return hipGetLastError();
}

}  // namespace bdu
