// apply.hip -- launches of the staged applier (apply_kernel.h): which split of
// the rows and wavefronts a launch takes, and the spike's rotations.
#include "apply_kernel.h"

namespace bdu {

namespace {

// Spike rotations on Q columns (j-1, j), j = m..n+2, one row per lane: a
// running carry keeps column j between consecutive rotations.  The rotations
// of a row are a dependent chain, so the columns come kSpikeCols at a time,
// the next ones on their way while these are rotated: 0.13 us a rotation at
// 10000 rows (0.16 with 16 columns), against 0.55 us when a wavefront of the applier did it, a
// column in flight at a time, before its panel's sweep.
constexpr int kSpikeCols = 32;

__global__ __launch_bounds__(64) void spike_apply_kernel(HandleDev *const *hs, Gate gate)
{
    if (gate.ranks && gate.pass >= gate.ranks[blockIdx.y]) return;
    const CONSTANT HandleDev *h = kptr(hs[blockIdx.y]);
    const int m = h->m, n = h->n, ld = h->ldq;
    if (m <= n || (int)blockIdx.x * 64 >= m) return;
    GLOBAL double *X = gptr(h->Q) + blockIdx.x * 64 + threadIdx.x;  // rows past m are padding
    const CONSTANT double *cs = kptr((const double *)h->csSp);
    const int total = m - n - 1;  // rotation t turns columns m - 2 - t, m - 1 - t (0-based)
    auto col = [&](int t) { return X + (int64_t)(m - 2 - (t < total ? t : total - 1)) * ld; };
    double carry = X[(int64_t)(m - 1) * ld];
    double x[kSpikeCols], y[kSpikeCols];
    if (total > 0) {
#pragma unroll
        for (int q = 0; q < kSpikeCols; ++q) x[q] = *col(q);
    }
    for (int t0 = 0; t0 < total; t0 += kSpikeCols) {
#pragma unroll
        for (int q = 0; q < kSpikeCols; ++q) y[q] = *col(t0 + kSpikeCols + q);
#pragma unroll
        for (int q = 0; q < kSpikeCols; ++q) {
            const int t = t0 + q;
            if (t < total) {
                rot(cs[2 * t], cs[2 * t + 1], x[q], carry);
                X[(int64_t)(m - 1 - t) * ld] = carry;
                carry = x[q];
            }
        }
#pragma unroll
        for (int q = 0; q < kSpikeCols; ++q) x[q] = y[q];
    }
    X[(int64_t)n * ld] = carry;
}

}  // namespace

// Instances in files of their own, compiled beside each other (half a minute each).
hipError_t launch_apply_k84(HandleDev *const *hs, int count, int panels, int G, int P, Gate gate, hipStream_t st);
hipError_t launch_apply_k180(HandleDev *const *hs, int count, int panels, int G, Gate gate, hipStream_t st);

constexpr int kCUs = 256, kFill = 250;

hipError_t launch_apply_staged(HandleDev *const *hs, int count, int max_panels, int k0, int nw, int rpl, bool spike,
                               Gate gate, hipStream_t st)
{
    const int panels = max_panels * rpl;  // of 64 rows
    if (spike && (gate.part <= 1 || gate.part == 3)) {
        hipLaunchKernelGGL(spike_apply_kernel, dim3(panels, count), dim3(64), 0, st, hs, gate);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // Which split, by the launch's 64-row panels (the largest handle's, times the
    // handles: a batch of mixed sizes, or a pass that only some of its handles
    // take, has fewer): kFill workgroups leave a few CUs to the generator, which
    // runs beside this kernel and needs a CU of its own (a launch of 256
    // slowed it from 5.3 to 6.7 ms at n = 2048, and itself with it).
    //   K = 84: G 4 while that leaves at most one workgroup per CU (n = 1024:
    //   2.20 ms with P 2, 2.82 with P 1, against 2.71 for G 1, P 2; n = 2048:
    //   8.7 against 8.3), with P 1 for up to eight panels (few blocks to run
    //   side by side: n = 200 325 us against 337); then G 1, P 2 as long as
    //   its workgroups, one per CU, all run at once (10000 x 2000: 10.3 ms,
    //   12.6 with P 1); then P 1, two workgroups per CU (128 streams of 128 to
    //   2048: 115 against 131 ms).
    //   K = 180: two pipelines of 15 wavefronts do not fit a workgroup.  G 4
    //   (n = 1024: 2.13 ms, 2.54 with G 3, P 2, 2.69 with G 1), then G 3, P 2
    //   (n = 2048: 6.3 ms, 7.0 with P 1, 8.1 with G 1), then G 1.
    const int64_t wgs = (int64_t)count * panels;
    if (k0 == 12 && nw == 7 && rpl == 1) {
        if (wgs * 4 <= kFill) return launch_apply_k84(hs, count, panels, 4, wgs <= 8 ? 1 : 2, gate, st);
        return launch_apply_k84(hs, count, panels, 1, wgs <= kCUs ? 2 : 1, gate, st);
    }
    if (k0 == 12 && nw == 15 && rpl == 1)
        return launch_apply_k180(hs, count, panels, wgs * 4 <= kFill ? 4 : wgs * 3 <= kFill ? 3 : 1, gate, st);
#define BDU_STAGED_CASE(K0, NW, R, W) \
    if (k0 == K0 && nw == NW && rpl == R) return launch_t<K0, NW, R, 1, 1, K0, W>(hs, count, panels, gate, st);
    BDU_STAGED_CASE(12, 3, 1, 4) BDU_STAGED_CASE(12, 3, 2, 2) BDU_STAGED_CASE(12, 7, 2, 2)
    BDU_STAGED_CASE(18, 3, 1, 2) BDU_STAGED_CASE(18, 5, 1, 2) BDU_STAGED_CASE(18, 7, 1, 2)
#undef BDU_STAGED_CASE
    return hipErrorInvalidValue;
}

}  // namespace bdu
