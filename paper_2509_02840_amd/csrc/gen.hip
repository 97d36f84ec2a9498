// gen.hip -- gfx950 kernels generating the rotations of one pass of the
// Givens bidiagonal update (Brust & Saunders, Section 3.4, Algorithm 2):
// phases 1 and 2 on the band of the working matrix, one thread per chain in
// flight, one rotation per tick.  gen_lds_kernel holds the band in LDS and
// orders ticks inside a wavefront by the LDS pipeline, with one barrier for
// every kGenStep ticks; gen_mem_kernel holds it in device memory (n too
// large for LDS) with a barrier for every tick.  FP64 throughout.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device.h"
#include "gen_chains.h"
#include "kernels.h"
#include "primitives.h"
#include "schedule.h"
#include "until_done.h"

namespace bdu {

// ---- generation in LDS ------------------------------------------------------------
//
// What bounds it: a pass is a chain of dependent rotations (8/3 n ticks of
// phase 1, 6 n of phase 2), so the time is the number of ticks times the
// time of one; a tick is bound by the vector instructions of the wavefronts
// that share a SIMD (4 cycles each), then by the latency of one Givens
// rotation.  So the layout makes a tick carry almost nothing but arithmetic:
//
// Coordinates.  Give L(i) the position s = 2 i and R(j) the position
// s = 2 j - 1, and keep the band in two arrays,
//   M1[2r - 1] = (r, r-1), M1[2r] = (r, r),
//   M2[2r + 1] = (r, r+1), M2[2r + 2] = (r, r+2).
// With (A, B) = (M1, M2) for a left and (M2, M1) for a right rotation, the
// five window pairs (device.h) of the rotation at position s are, whatever
// its side,
//   w0 = (A[s-1], *)  w1 = (A[s], A[s+1])  w2 = (B[s+1], A[s+2])
//   w3 = (B[s+2], B[s+3])  w4 = (*, B[s+4])
// where * is the bulge cell: it is zero in memory at every tick boundary, as
// the rotation that fills it and the one that empties it are consecutive in
// one chain, which carries it in registers.  A chain moves s by -3 a tick in
// phase 1 and by +3 in phase 2 and swaps A and B.
//
// Time.  In phase 1 chain c (0-based) starts at position c + 1, one tick
// after chain c - 1; in phase 2 chain c starts at position c + 2, three
// ticks after chain c - 1 (the earliest starts the window overlaps allow).
// So at any tick all chains in flight are on the same side, 4 (phase 1) or 8
// (phase 2) positions apart, and their positions agree modulo 4 or 8.  The
// arrays are stored by residue, M[s] at (s mod R) E + s / R with R = 4 in
// phase 1 and 8 in phase 2: neighbouring lanes then touch neighbouring
// doubles (no bank conflicts), and the cells of the kGenStep = 8 ticks of a
// step are at compile-time offsets from one base per array that moves by a
// constant from step to step.
//
// Wavefronts.  Chain c runs on thread c mod blockDim, so 64 consecutive
// chains share a wavefront, where a tick's LDS reads follow the previous
// tick's LDS writes in order, with no barrier.  The plan starts each chunk
// of 64 chains kGenStep ticks late, so what a rotation needs from another
// wavefront lies in an earlier step, and one barrier a step is enough.
//
// Measured on one stream, a pass generated in one launch: n = 2048 (18 749
// ticks) 13.3 -> 5.2 ms, 0.75 -> 0.28 us a tick; n = 200 (1821 ticks) 1.05 ->
// 0.44 ms.  The earlier kernel kept five band cells of padded rows with an
// address register for each, rotated u and v along and ran a barrier a tick.
// A tick of one wavefront inside its chains takes about 340 cycles (51
// vector instructions, 180 cycles of them one dependent chain), one in which
// chains start about 480.

typedef LOCAL double *LdsPtr;

// LDS image for up to CAP rows, in doubles: u and v, then M1 and M2.
template <int CAP>
struct GenLds {
    static constexpr int UV = CAP + 8;
    static constexpr int M = 2 * CAP + 32;  // positions of M1 (and M2), whole residues of 4 and 8
    static constexpr int BYTES = 8 * 2 * (UV + M);
    static_assert(CAP % 4 == 0 && BYTES <= kMaxGenLds, "the image fits in LDS");
};

// Position s of M1 or M2 in an array stored by residue modulo R.
template <int CAP, int R>
__device__ __forceinline__ int gen_index(int s)
{
    return (s % R) * (GenLds<CAP>::M / R) + s / R;
}

// A lane's chain: its length and start tick, and for each side the byte
// offset of its first rotation's slot in that side's stream.
struct GenLane {
    int len, tau;
    uint32_t sl, sr;
};

__device__ __forceinline__ GenLane gen_lane(const GenChain *chains, int idx)
{
    typedef int int4v __attribute__((ext_vector_type(4)));
    const GLOBAL int4v *p = (const GLOBAL int4v *)gptr(chains) + 2 * (int64_t)idx;
    const int4v a = p[0], b = p[1];
    GenLane l;
    l.len = a[2];
    l.tau = a[3];
    l.sl = 16u * (uint32_t)b[0];  // the plan keeps 16 slot below 2^32
    l.sr = 16u * (uint32_t)b[2];
    return l;
}

// A lane among its wavefront's, as gen_chains.h sees it.
template <typename Place, typename Fetch>
struct GenWave {
    GenCursor<GenLane> &lane;
    Place &at;
    Fetch &load;
    template <typename F>
    __device__ __forceinline__ bool any(F f) const
    {
        return __any(f(lane));
    }
    template <typename F, typename G>
    __device__ __forceinline__ void each(F f, G g)
    {
        if (f(lane)) g(lane);
    }
    __device__ __forceinline__ void place(GenCursor<GenLane> &) { at(); }
    __device__ __forceinline__ void fetch() { load(); }
};

// Byte offset of the cell at position s from a step's base pointer, e = s
// less R times the base's index (which phase 1 lowers by 8 to keep the
// offsets of its eight ticks non-negative).
template <int CAP, bool P1>
__device__ constexpr int gen_offset(int e)
{
    constexpr int R = P1 ? 4 : 8, E = GenLds<CAP>::M / R;
    const int r = ((e % R) + R) % R;
    return 8 * (r * E + (e - r) / R + (P1 ? 8 : 0));
}

typedef double double2v __attribute__((ext_vector_type(2)));

// Writes of the lanes in `mask` (and in the execution mask): by narrowing
// the execution mask around them, with no branch.
template <int O0, int O1, int O2, int O3, int O4>
__device__ __forceinline__ void gen_write(uint64_t mask, LdsPtr p, double x0, double x1, double x2, LdsPtr q,
                                          double x3, LdsPtr r, double x4, GLOBAL char *stream, uint32_t so,
                                          double2v value)
{
    uint64_t all;
    asm volatile(
        "s_and_saveexec_b64 %[all], %[mask]\n\t"
        "global_store_dwordx4 %[so], %[value], %[stream]\n\t"
        "ds_write_b64 %[p], %[x0] offset:%[o0]\n\t"
        "ds_write_b64 %[p], %[x1] offset:%[o1]\n\t"
        "ds_write_b64 %[p], %[x2] offset:%[o2]\n\t"
        "ds_write_b64 %[q], %[x3] offset:%[o3]\n\t"
        "ds_write_b64 %[r], %[x4] offset:%[o4]\n\t"
        "s_mov_b64 exec, %[all]"
        : [all] "=&s"(all)
        : [mask] "s"(mask), [p] "v"(p), [q] "v"(q), [r] "v"(r), [x0] "v"(x0), [x1] "v"(x1), [x2] "v"(x2),
          [x3] "v"(x3), [x4] "v"(x4), [so] "v"(so), [value] "v"(value), [stream] "s"(stream), [o0] "n"(O0),
          [o1] "n"(O1), [o2] "n"(O2), [o3] "n"(O3), [o4] "n"(O4)
        : "memory", "scc");
}

template <int O0, int O1, int O2>
__device__ __forceinline__ void gen_write3(uint64_t mask, LdsPtr p, double x0, double x1, double x2)
{
    uint64_t all;
    asm volatile(
        "s_and_saveexec_b64 %[all], %[mask]\n\t"
        "ds_write_b64 %[p], %[x0] offset:%[o0]\n\t"
        "ds_write_b64 %[p], %[x1] offset:%[o1]\n\t"
        "ds_write_b64 %[p], %[x2] offset:%[o2]\n\t"
        "s_mov_b64 exec, %[all]"
        : [all] "=&s"(all)
        : [mask] "s"(mask), [p] "v"(p), [x0] "v"(x0), [x1] "v"(x1), [x2] "v"(x2), [o0] "n"(O0), [o1] "n"(O1),
          [o2] "n"(O2)
        : "memory", "scc");
}

template <int O0>
__device__ __forceinline__ void gen_write1(uint64_t mask, LdsPtr p, double x0)
{
    uint64_t all;
    asm volatile(
        "s_and_saveexec_b64 %[all], %[mask]\n\t"
        "ds_write_b64 %[p], %[x0] offset:%[o0]\n\t"
        "s_mov_b64 exec, %[all]"
        : [all] "=&s"(all)
        : [mask] "s"(mask), [p] "v"(p), [x0] "v"(x0), [o0] "n"(O0)
        : "memory", "scc");
}

// The lanes in `mask` take the pairs of a chain's first rotation.
__device__ __forceinline__ void gen_enter(uint64_t mask, double &a, double &bg, double &b, double &g, double fa,
                                          double fbg, double fb, double fg)
{
    uint64_t all;
    asm volatile(
        "s_and_saveexec_b64 %[all], %[mask]\n\t"
        "v_mov_b64 %[a], %[fa]\n\t"
        "v_mov_b64 %[bg], %[fbg]\n\t"
        "v_mov_b64 %[b], %[fb]\n\t"
        "v_mov_b64 %[g], %[fg]\n\t"
        "s_mov_b64 exec, %[all]"
        : [all] "=&s"(all), [a] "+v"(a), [bg] "+v"(bg), [b] "+v"(b), [g] "+v"(g)
        : [mask] "s"(mask), [fa] "v"(fa), [fbg] "v"(fbg), [fb] "v"(fb), [fg] "v"(fg)
        : "scc");
}

// Keeps a rotation computed ahead of the branch on its operands' range: the
// test's result then arrives while the rotation is computed, not before it.
__device__ __forceinline__ void settle_core(double &c, double &s, double &r)
{
    asm volatile("" : "+v"(c), "+v"(s), "+v"(r));
}

// grid (handles), one workgroup per handle; see the notes above.
template <int CAP>
__global__ __launch_bounds__(kGenThreads) void gen_lds_kernel(HandleDev *const *hs, Gate gate)
{
    using G = GenLds<CAP>;
    extern __shared__ double smem[];
    if (gate.ranks && gate.pass >= gate.ranks[blockIdx.x]) return;
    const CONSTANT HandleDev *h = kptr(hs[blockIdx.x]);
    // a batch runs as many segments as its largest plan has; this
    // handle's pass may have ended already
    if (gate.part >= 3 && gate.part - 3 >= h->nseg) return;
    const int n = h->n, N = h->N;
    const LdsPtr lu = (LdsPtr)smem, lv = lu + G::UV, m1 = lu + 2 * G::UV, m2 = m1 + G::M;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int SN = 2 * N + 8;  // positions of M1 and M2 in use
    GLOBAL double *band = gptr(h->band);

    // ticks [t_begin, t_end) of this part; phase 1 ends (with the fold, at
    // tick split - 1) before phase 2 starts (at t2)
    const int ticks = (int)h->ticks, split = (int)h->split;
    const int t2 = (split + kGenStep - 1) / kGenStep * kGenStep;
    int t_begin = 0, t_end = ticks;
    if (gate.part == 1) t_end = split;
    if (gate.part == 2) t_begin = split;
    if (gate.part >= 3) {
        const int k = gate.part - 3;
        t_begin = k == 0 ? 0 : h->tcut[k - 1];
        t_end = h->tcut[k];
    }
    const bool run1 = t_begin < split - 1, run_fold = t_begin < split && t_end >= split;
    const bool run2 = t_end > t2;

    // the band as an earlier part left it in device memory (M1, M2, u, v in
    // order of position), into arrays stored by residue modulo R, and back
    auto load_image = [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        for (int s = tid; s < SN; s += nt) {
            const int x = gen_index<CAP, R>(s);
            m1[x] = band[s];
            m2[x] = band[SN + s];
        }
    };
    auto save_image = [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        for (int s = tid; s < SN; s += nt) {
            const int x = gen_index<CAP, R>(s);
            band[s] = m1[x];
            band[SN + s] = m2[x];
        }
    };
    using R1 = std::integral_constant<int, 4>;
    using R2 = std::integral_constant<int, 8>;
    if (t_begin == 0) {
        for (int x = tid; x < 2 * G::M; x += nt) m1[x] = 0.0;
        __syncthreads();
        for (int i = 1 + tid; i <= n; i += nt) {
            m1[gen_index<CAP, 4>(2 * i)] = h->d[i - 1];
            if (i < n) m2[gen_index<CAP, 4>(2 * i + 1)] = h->e[i - 1];
            lv[i] = h->v[i - 1];
        }
        for (int i = 1 + tid; i <= N; i += nt) lu[i] = h->u[i - 1];
    } else if (run1 || run_fold) {
        load_image(R1{});
        for (int i = tid; i <= N; i += nt) lu[i] = band[2 * SN + i];
        for (int i = tid; i <= n; i += nt) lv[i] = band[2 * SN + N + 1 + i];
    } else {
        load_image(R2{});
    }
    __syncthreads();

    const int nch1 = 2 * n - (N > n ? 2 : 3);  // phase-1 chains
    const uint32_t K16 = 16u * (uint32_t)h->K;
    const uint32_t bias = 8 * K16;  // keeps the offsets of a chain's step before its start non-negative
    GLOBAL char *csL = gptr((char *)h->csL) - bias, *csR = gptr((char *)h->csR) - bias;

    // carried window pairs of this lane's chain: phase 1 (w3, w4), phase 2
    // (w0, w1); bg is the bulge cell
    double a = 0.0, bg = 0.0, b = 0.0, g = 0.0;

    // The steps of one phase (1 or 2) from tick tb, a multiple of kGenStep,
    // to the last that starts below te.
    auto phase = [&](auto pc, int tb, int te) {
        constexpr bool P1 = decltype(pc)::value == 1;
        const int nch = P1 ? nch1 : 2 * n - (N > n ? 1 : 3);
        auto chain = [&](int c) {
            GenLane l;
            l.len = 0;
            l.tau = 1 << 30;
            l.sl = l.sr = 0;
            if (c < nch && (P1 || c != 2 * n - 3))  // no chain starts with R(n)
                l = gen_lane(h->chains, P1 ? c : nch1 + 1 + c - (c > 2 * n - 3 ? 1 : 0));
            return l;
        };
        GenCursor<GenLane> my;
        my.ci = tid;
        my.nt = nt;
        my.nch = nch;
        gen_first_chain(my, tb, chain);
        const int &ci = my.ci, &q0 = my.q0;
        const GenLane &cur = my.cur;
        if (cur.tau < tb && cur.tau + cur.len > tb) {  // in flight since an earlier part
            a = h->carry[4 * tid];
            bg = h->carry[4 * tid + 1];
            b = h->carry[4 * tid + 2];
            g = h->carry[4 * tid + 3];
        }
        // wait here for everything loaded: a load in flight in the loop
        // would make it wait for the coefficient stores, which the same
        // counter counts
        asm volatile("" ::"v"(a), "v"(bg), "v"(b), "v"(g), "v"(my.nxt.len), "v"(my.nxt.tau), "v"(my.nxt.sl),
                     "v"(my.nxt.sr));

        LdsPtr p1, p2;
        uint32_t oe, oo;  // stream offsets of the even ticks' side and the odd ticks'
        // cell M[s + k] of a lane, e = k plus the tick's constant part of s
        auto cell = [&](LdsPtr p, int e) -> LdsPtr { return p + gen_offset<CAP, P1>(e) / 8; };
        // What a chain's first rotation takes from memory, read a tick ahead
        // (it is final by then: the chains before it touched it at least two
        // ticks ago).  Phase 1: w3 and w4's second entry, and the pair of u
        // or v (at vec) that the rotation is generated from in place of w4;
        // the bulge cell is zero.  Phase 2: the generating pair is w1, in the
        // place of w0, and w0 = (x, 0) in the place of w1.
        double fa = 0.0, fbg = 0.0, fb = 0.0, fw = 0.0, fg = 0.0;
        LdsPtr vec = lu;
        auto fetch = [&](auto tc) {
            constexpr int T = decltype(tc)::value;
            constexpr bool RIGHT = P1 ? T % 2 == 0 : T % 2 == 1;
            constexpr int e = P1 ? 1 - 3 * T : 2 + 3 * T;
            const LdsPtr A = RIGHT ? p2 : p1, B = RIGHT ? p1 : p2;
            if constexpr (P1) {
                fbg = vec[0];
                fg = vec[1];
                fa = *cell(B, e + 2);
                fb = *cell(B, e + 3);
                fw = *cell(B, e + 4);
            } else {
                fa = *cell(A, e);
                fbg = *cell(A, e + 1);
                fb = *cell(A, e - 1);
            }
        };
        // One tick.  KIND 0: every lane in flight is past its first and
        // before its last rotation in the whole step; bit 0: some chains end
        // in this step (or ended, or have yet to start); bit 1: some start.
        // There the lanes not in flight compute along, on cells inside the
        // image, and only their writes are masked, so that ends and starts
        // cost a few instructions and no branch.
        auto tick = [&](auto tc, auto kind) {
            constexpr int T = decltype(tc)::value, KIND = decltype(kind)::value;
            constexpr bool RIGHT = P1 ? T % 2 == 0 : T % 2 == 1;
            constexpr int e = P1 ? 1 - 3 * T : 2 + 3 * T;
            const LdsPtr A = RIGHT ? p2 : p1, B = RIGHT ? p1 : p2;
            uint64_t live = 0, first = 0, last = 0;
            if constexpr (KIND > 0) {
                live = __builtin_amdgcn_ballot_w64((unsigned)(q0 + T) < (unsigned)cur.len);
                if constexpr (KIND & 1) last = __builtin_amdgcn_ballot_w64(q0 + T + 1 == cur.len);
            }
            if constexpr (KIND & 2) {
                first = __builtin_amdgcn_ballot_w64(q0 == -T);
                gen_enter(first, a, bg, b, g, fa, fbg, fb, P1 ? fg : 0.0);
            }
            double w2x = *cell(B, e + 1), w2y = *cell(A, e + 2);
            const double w4 = fw;
            double c, s, rr;
            double ka = a, kbg = bg, kb = b, kg = g;
            double z0, z1, z2, z3, z4;  // z0 .. z3 are carried to the next rotation
            bool in;
            auto out_of_range = [&]() {
                if constexpr (KIND > 0)
                    return (__builtin_amdgcn_ballot_w64(!in) & live) != 0;
                else
                    return !__all(in);
            };
            if constexpr (P1) {
                double w1x = *cell(A, e), w1y = *cell(A, e + 1), w0x = *cell(A, e - 1);
                if constexpr ((KIND & 2) && T + 1 < kGenStep) fetch(std::integral_constant<int, T + 1>{});
                in = givens_in_range(kbg, kg);
                givens_core<1>(kbg, kg, c, s, rr);
                settle_core(c, s, rr);
                z0 = c * w0x;  // w0's second entry is zero
                z1 = s * w0x;
                if (__builtin_expect(out_of_range(), 0)) {
                    givens_m<1>(kbg, kg, c, s, rr);
                    z0 = fma(c, w0x, -(s * 0.0));
                    z1 = fma(s, w0x, c * 0.0);
                }
                rot(c, s, ka, kb);
                rot(c, s, w2x, w2y);
                rot(c, s, w1x, w1y);
                z2 = w1x;
                z3 = w1y;
                z4 = rr;
                if constexpr (KIND & 2) {
                    const double w4n = fma(s, 0.0, c * w4);
                    z4 = __builtin_amdgcn_inverse_ballot_w64(first) ? w4n : rr;
                }
            } else {
                double w3x = *cell(B, e + 2), w3y = *cell(B, e + 3), w4y = *cell(B, e + 4);
                if constexpr ((KIND & 2) && T + 1 < kGenStep) fetch(std::integral_constant<int, T + 1>{});
                in = givens_in_range(ka, kbg);
                givens_core<2>(ka, kbg, c, s, rr);
                settle_core(c, s, rr);
                z1 = -(s * w4y);  // w4's first entry is zero
                z3 = c * w4y;
                if (__builtin_expect(out_of_range(), 0)) {
                    givens_m<2>(ka, kbg, c, s, rr);
                    z1 = fma(c, 0.0, -(s * w4y));
                    z3 = fma(s, 0.0, c * w4y);
                }
                rot(c, s, kb, kg);
                rot(c, s, w2x, w2y);
                rot(c, s, w3x, w3y);
                z0 = w3x;
                z2 = w3y;
                z4 = rr;
                if constexpr (KIND & 2) {
                    const bool f = __builtin_amdgcn_inverse_ballot_w64(first);
                    const double w0n = kb;
                    z4 = f ? w0n : rr;
                    kb = f ? rr : w0n;
                    kg = f ? 0.0 : kg;
                }
            }
            double2v value;
            value[0] = c;
            value[1] = s;
            GLOBAL char *stream = (RIGHT ? csR : csL) + (uint64_t)(T / 2) * K16;
            const uint32_t so = T % 2 == 0 ? oe : oo;
            if constexpr (KIND == 0) {
                if constexpr (P1) {
                    *cell(B, e + 2) = ka;
                    *cell(B, e + 3) = kb;
                    *cell(B, e + 4) = z4;
                } else {
                    *cell(A, e - 1) = z4;
                    *cell(A, e) = kb;
                    *cell(A, e + 1) = kg;
                }
                *cell(B, e + 1) = w2x;
                *cell(A, e + 2) = w2y;
                *(GLOBAL double2v *)(stream + (uint64_t)so) = value;
            } else {
                if constexpr (P1) {
                    gen_write<gen_offset<CAP, P1>(e + 2), gen_offset<CAP, P1>(e + 3), gen_offset<CAP, P1>(e + 4), gen_offset<CAP, P1>(e + 1), gen_offset<CAP, P1>(e + 2)>(
                        live, B, ka, kb, z4, B, w2x, A, w2y, stream, so, value);
                    if constexpr (KIND & 2) gen_write1<8>(first, vec, rr);
                    if constexpr (KIND & 1)
                        gen_write3<gen_offset<CAP, P1>(e - 1), gen_offset<CAP, P1>(e), gen_offset<CAP, P1>(e + 1)>(last, A, z0, z2, z3);
                } else {
                    gen_write<gen_offset<CAP, P1>(e - 1), gen_offset<CAP, P1>(e), gen_offset<CAP, P1>(e + 1), gen_offset<CAP, P1>(e + 1), gen_offset<CAP, P1>(e + 2)>(
                        live, A, z4, kb, kg, B, w2x, A, w2y, stream, so, value);
                    if constexpr (KIND & 1)
                        gen_write3<gen_offset<CAP, P1>(e + 2), gen_offset<CAP, P1>(e + 3), gen_offset<CAP, P1>(e + 4)>(last, B, z0, z2, z3);
                }
            }
            a = z0;
            bg = z1;
            b = z2;
            g = z3;
        };
        // the kGenStep ticks of a step: a tick's LDS accesses stay behind the
        // previous tick's (other lanes of the wavefront wrote what it reads)
        auto step = [&](auto kind) {
            auto one = [&](auto tc) {
                tick(tc, kind);
                asm volatile("" ::: "memory");
            };
            if constexpr (decltype(kind)::value & 2) {
                if constexpr (P1) vec = (ci & 1) ? lu + (ci + 1) / 2 : lv + (ci + 2) / 2;
                fetch(std::integral_constant<int, 0>{});
            }
            one(std::integral_constant<int, 0>{});
            one(std::integral_constant<int, 1>{});
            one(std::integral_constant<int, 2>{});
            one(std::integral_constant<int, 3>{});
            one(std::integral_constant<int, 4>{});
            one(std::integral_constant<int, 5>{});
            one(std::integral_constant<int, 6>{});
            one(std::integral_constant<int, 7>{});
        };
        // rotation, cells and slots of the lane's chain at the step from tick t
        auto place = [&](int t) {
            my.q0 = t - cur.tau;
            // base of the step's cells: its position without the constant part, over R
            const int beta = P1 ? (ci - 3 * q0) >> 2 : (ci + 3 * q0) >> 3;
            p1 = m1 + beta - (P1 ? 8 : 0);
            p2 = m2 + beta - (P1 ? 8 : 0);
            oe = bias + (P1 ? cur.sr : cur.sl) + K16 * (uint32_t)((t >> 1) - ((cur.tau + 1) >> 1));
            oo = bias + (P1 ? cur.sl : cur.sr) + K16 * (uint32_t)((t >> 1) - (cur.tau >> 1));
        };
        auto fetch_next = [&]() {
            my.more = ci + nt < nch;
            my.nxt = chain(ci + nt);
            asm volatile("" ::"v"(my.nxt.len), "v"(my.nxt.tau), "v"(my.nxt.sl), "v"(my.nxt.sr));
        };
        place(tb);
        for (int t = tb; t < te; t += kGenStep) {
            auto place_now = [&]() { place(t); };
            GenWave<decltype(place_now), decltype(fetch_next)> wave{my, place_now, fetch_next};
            gen_next_chain(wave);
            const bool touched = q0 > -kGenStep && q0 < cur.len;
            const bool starts = touched && q0 <= 0, ends = touched && q0 + kGenStep >= cur.len;
            const uint64_t any = __builtin_amdgcn_ballot_w64(touched);
            const int kind = (__any(starts) ? 2 : 0) + (__any(ends) ? 1 : 0);
            if (any != 0) {
                if (__builtin_amdgcn_inverse_ballot_w64(any)) {
                    if (kind == 0) step(std::integral_constant<int, 0>{});
                    else if (kind == 2) step(std::integral_constant<int, 2>{});
                    else if (kind == 1) step(std::integral_constant<int, 1>{});
                    else step(std::integral_constant<int, 3>{});
                }
            }
            my.q0 += kGenStep;
            p1 += P1 ? -3 * kGenStep / 4 : 3 * kGenStep / 8;
            p2 += P1 ? -3 * kGenStep / 4 : 3 * kGenStep / 8;
            oe += kGenStep / 2 * K16;
            oo += kGenStep / 2 * K16;
            // this step's LDS accesses are complete before the next step's
            // of any wavefront (the stores to the streams need no wait)
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
        if (te < ticks && cur.tau < te && cur.tau + cur.len > te) {
            h->carry[4 * tid] = a;
            h->carry[4 * tid + 1] = bg;
            h->carry[4 * tid + 2] = b;
            h->carry[4 * tid + 3] = g;
        }
    };

    if (run1) phase(std::integral_constant<int, 1>{}, t_begin, t_end < split - 1 ? t_end : split - 1);
    __syncthreads();
    if (run_fold) {
        // u v^T now touches only (N-1, n) and (N, n); u_N is the spike's
        // survivor when m > n, taken from device memory here because the
        // spike may run beside the earlier parts
        if (tid == 0) {
            const double vn = lv[n], uN = N > n ? h->u[N - 1] : lu[N];
            const LdsPtr f1 = N > n ? m1 + gen_index<CAP, 4>(2 * n) : m2 + gen_index<CAP, 4>(2 * n - 1);
            const LdsPtr f2 = N > n ? m1 + gen_index<CAP, 4>(2 * n + 1) : m1 + gen_index<CAP, 4>(2 * n);
            *f1 = fma(lu[N - 1], vn, *f1);
            *f2 = fma(uN, vn, *f2);
        }
        __syncthreads();
    }
    bool by8 = t_begin >= split;  // the arrays are stored for phase 2
    if (run2) {
        if (!by8) {
            save_image(R1{});
            __syncthreads();
            load_image(R2{});
            __syncthreads();
            by8 = true;
        }
        phase(std::integral_constant<int, 2>{}, t_begin > t2 ? t_begin : t2, t_end);
        __syncthreads();
    }
    if (t_end < ticks) {
        // a later part continues (no chain is in flight at the end of phase 1)
        if (by8) {
            save_image(R2{});
        } else {
            save_image(R1{});
            for (int i = tid; i <= N; i += nt) band[2 * SN + i] = lu[i];
            for (int i = tid; i <= n; i += nt) band[2 * SN + N + 1 + i] = lv[i];
        }
        return;
    }
    for (int i = 1 + tid; i <= n; i += nt) {
        h->d[i - 1] = m1[gen_index<CAP, 8>(2 * i)];
        if (i < n) h->e[i - 1] = m2[gen_index<CAP, 8>(2 * i + 1)];
    }
}

// ---- generation in device memory --------------------------------------------------

// Band storage: band_row (device.h).  Entries outside the band read as zero
// and are never written: the schedule keeps them zero.

// Chain descriptor held in registers.
struct ChainReg {
    int type, param, len, tau0;
    int64_t slot0, slot1;
};

__device__ __forceinline__ ChainReg load_chain(const GenChain *chains, int idx)
{
    const GLOBAL int *p = (const GLOBAL int *)gptr(chains) + 8 * idx;
    const GLOBAL int64_t *q = (const GLOBAL int64_t *)(p + 4);
    ChainReg c;
    c.type = p[0];
    c.param = p[1];
    c.len = p[2];
    c.tau0 = p[3];
    c.slot0 = q[0];
    c.slot1 = q[1];
    return c;
}

// A use that makes the compiler wait for a chain's loads at this point.  The
// vector memory counter also counts the coefficient stores, so a wait for a
// load left in flight across the tick loop would wait for the previous
// tick's store in every tick.
__device__ __forceinline__ void settle(const ChainReg &c)
{
    asm volatile("" ::"v"(c.type), "v"(c.param), "v"(c.len), "v"(c.tau0), "v"(c.slot0), "v"(c.slot1));
}

// Ticks between refills of a thread's prefetched chain descriptor.
constexpr int kRefill = 32;

__device__ __forceinline__ int band_cell(int r, int c)
{
    return band_row(r) + (c - r) + 2;
}

// Rotation s of chain g as band pointers (the offsets of rot_offsets):
// the pair a rotation is generated from is slot 1 in phase 1 and slot 0 in
// phase 2, except at a chain's first rotation: the u or v pair in phase 1,
// slot 1 in phase 2.  The next rotation's slots 0, 1 hold (x_3, y_3),
// (x_4, y_4) of this one's, in both phases and both directions.
//
// Rotations s and s + 2 of a chain have the same pattern three rows and
// columns further on: every band pointer moves by kBandStep3 doubles, the u
// or v pointer by 3 and the coefficient slot by K.
template <typename BP>
struct RotAddr {
    BP x[5], y[5];      // window pairs, in slot order
    BP vb;              // u or v pair (vb[0], vb[1])
    GLOBAL double *cs;  // coefficient slot (c, s)
};

template <typename BP>
__device__ __forceinline__ RotAddr<BP> decode(BP S, const ChainReg &g, int s, int K, int UO, int VO,
                                              GLOBAL double *csL, GLOBAL double *csR)
{
    const RotOff o = rot_offsets(g.type, g.param, s, UO, VO);
    RotAddr<BP> d;
    d.vb = S + o.vb;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        d.x[k] = S + o.x[k];
        d.y[k] = S + o.y[k];
    }
    d.cs = (o.side == 0 ? csL + 2 * g.slot0 : csR + 2 * g.slot1) + (int64_t)(s >> 1) * 2 * K;
    return d;
}

template <typename BP>
__device__ __forceinline__ void advance(RotAddr<BP> &a, int db, int du, int64_t dcs)
{
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        a.x[q] += db;
        a.y[q] += db;
    }
    a.vb += du;
    a.cs += dcs;
}

// Generation of one pass for one handle per workgroup.  Thread l runs chains
// l, l + blockDim, ... (non-empty chains in schedule order); chain c performs
// its rotation s at tick tau0(c) + s, and a barrier separates ticks.  The host
// chose the start ticks so that two rotations touching a common band row, u or
// v entry are ordered as in the sequential schedule; in particular no other
// rotation touches a band entry between two consecutive rotations of a chain
// that share it, so the thread keeps the two shared pairs in registers
// (k0, k1) instead of writing and reading them back.  A tick reads three
// window pairs and the u or v pair, generates the rotation from registers and
// writes three pairs and the u or v pair; a chain's first tick also reads
// slots 0 and 1, its last also writes slots 3 and 4.
//
// Each thread keeps the pointers of its chain's next rotation at an even tick
// (ae) and at an odd tick (ao) and moves the set it has just used on to the
// chain's rotation two ticks later.
__global__ __launch_bounds__(kGenThreads) void gen_mem_kernel(HandleDev *const *hs, Gate gate)
{
    if (gate.ranks && gate.pass >= gate.ranks[blockIdx.x]) return;
    const CONSTANT HandleDev *h = kptr(hs[blockIdx.x]);
    // a batch runs as many segments as its largest plan has; this
    // handle's pass may have ended already
    if (gate.part >= 3 && gate.part - 3 >= h->nseg) return;
    const int n = h->n, N = h->N;
    double *S = h->band;
    using BP = GLOBAL double *;
    const BP SB = (BP)S;
    const int UO = (int)band_doubles(N);  // u_i at S[UO + i + 3]
    const int VO = UO + (N + 8);          // v_j at S[VO + j + 3]
    const int tid = threadIdx.x;
    const int nt = blockDim.x;
    const int total = VO + (n + 8);
    // A part after the first continues from the band the previous one left;
    // otherwise start from d, e, u and v.  Parts: 0 all ticks, 1 phase 1,
    // 2 phase 2, 3 + k segment k.
    const int part = gate.part;
    const int ticks = (int)h->ticks, split = (int)h->split;
    int t_begin = 0, t_end = ticks;
    if (part == 1) t_end = split;
    if (part == 2) t_begin = split;
    if (part >= 3) {
        const int k = part - 3;
        t_begin = k == 0 ? 0 : h->tcut[k - 1];
        t_end = h->tcut[k];
    }
    if (t_begin > 0) {
        // u_N, the spike's survivor, is read only by the fold: a pass may
        // start generating before the spike has finished (the first segment
        // then read u_N early) and let only the fold's segment wait for it,
        // so every later segment takes u_N afresh
        if (N > n && tid == 0) S[UO + N + 3] = h->u[N - 1];
        __syncthreads();
    } else {
        for (int k = tid; k < total; k += nt) S[k] = 0.0;
        __syncthreads();
        for (int i = 1 + tid; i <= n; i += nt) {
            S[band_cell(i, i)] = h->d[i - 1];
            if (i < n) S[band_cell(i, i + 1)] = h->e[i - 1];
            S[VO + i + 3] = h->v[i - 1];
        }
        for (int i = 1 + tid; i <= N; i += nt) S[UO + i + 3] = h->u[i - 1];
        __syncthreads();
    }

    const int K = h->K;
    const int nch = h->nchains;
    GLOBAL double *csL = gptr((double *)h->csL), *csR = gptr((double *)h->csR);
    const int64_t dcs = 2 * (int64_t)K;
    // Thread tid runs chains tid, tid + nt, ...; gn holds the next one when
    // `next` is set.  Descriptors are loaded and waited for before the loop,
    // every kRefill ticks, or (when a chain ends before a refill) at the
    // switch, so the tick body itself never waits on vector memory.
    int ci = tid;
    ChainReg g = {}, gn = {};
    bool next = false;
    if (ci < nch) g = load_chain(h->chains, ci);
    settle(g);
    // part 2: skip the chains that finished before it (none is in flight at
    // the split)
    while (ci < nch && g.tau0 + g.len <= t_begin) {
        ci += nt;
        if (ci < nch) {
            g = load_chain(h->chains, ci);
            settle(g);
        }
    }
    if (ci + nt < nch) {
        gn = load_chain(h->chains, ci + nt);
        next = true;
    }
    settle(gn);

    RotAddr<BP> ae, ao;
    bool m1 = false, fold = false;
    int db = 0, du = 0;
    int tend = -1;
    auto start = [&]() {
        const RotAddr<BP> a0 = decode(SB, g, 0, K, UO, VO, csL, csR), a1 = decode(SB, g, 1, K, UO, VO, csL, csR);
        const bool odd0 = g.tau0 & 1;
        ae = odd0 ? a1 : a0;
        ao = odd0 ? a0 : a1;
        m1 = g.type <= CH_P1B;
        fold = g.type == CH_FOLD;
        db = m1 ? -kBandStep3 : kBandStep3;
        du = m1 ? -3 : 3;
        tend = g.tau0 + g.len - 1;
    };
    double kx0 = 0.0, kx1 = 0.0, ky0 = 0.0, ky1 = 0.0;  // slots 0, 1 carried from the previous rotation
    if (ci < nch) {
        start();
        if (g.tau0 < t_begin) {
            // in flight since an earlier segment: resume at rotation q with
            // the carried pairs that segment saved
            const int q = t_begin - g.tau0;
            const RotAddr<BP> aq = decode(SB, g, q, K, UO, VO, csL, csR),
                              aq1 = decode(SB, g, q + 1, K, UO, VO, csL, csR);
            const bool oddq = t_begin & 1;
            ae = oddq ? aq1 : aq;
            ao = oddq ? aq : aq1;
            kx0 = h->carry[4 * tid];
            kx1 = h->carry[4 * tid + 1];
            ky0 = h->carry[4 * tid + 2];
            ky1 = h->carry[4 * tid + 3];
        }
    }
    // wait for the carries here: a load still in flight at the tick loop
    // would make the loop wait on the vector memory counter in every tick,
    // and that counter also counts the coefficient stores
    asm volatile("" ::"v"(kx0), "v"(kx1), "v"(ky0), "v"(ky1));
    // One rotation with its window, for one phase (the phase is uniform
    // across a wavefront except where phase 2 starts, so a wavefront
    // normally runs one of the two bodies).
    auto rotate = [&](RotAddr<BP> &a, bool first, bool last, auto phase) {
        constexpr bool P1 = decltype(phase)::value;
        double xv[5], yv[5];
#pragma unroll
        for (int q = 2; q < 5; ++q) {
            xv[q] = *a.x[q];
            yv[q] = *a.y[q];
        }
        double ux = a.vb[0], uy = a.vb[1];
        // local copies: a select between captured variables would become a
        // load through a selected address
        xv[0] = kx0;
        xv[1] = kx1;
        yv[0] = ky0;
        yv[1] = ky1;
        double va = P1 ? xv[1] : xv[0], vb = P1 ? yv[1] : yv[0];
        if (first) {
            xv[0] = *a.x[0];
            xv[1] = *a.x[1];
            yv[0] = *a.y[0];
            yv[1] = *a.y[1];
            va = P1 ? ux : xv[1];
            vb = P1 ? uy : yv[1];
        }
        double c, sn, rr;
        givens_fast<P1 ? 1 : 2>(va, vb, c, sn, rr);
#pragma unroll
        for (int q = 0; q < 5; ++q) rot(c, sn, xv[q], yv[q]);
        rot(c, sn, ux, uy);
        // the generating pair becomes (0, r) (mode 1) or (r, 0) (mode 2)
        if (P1) {
            ux = first ? 0.0 : ux;
            uy = first ? rr : uy;
            xv[1] = first ? xv[1] : 0.0;
            yv[1] = first ? yv[1] : rr;
        } else {
            xv[1] = first ? rr : xv[1];
            yv[1] = first ? 0.0 : yv[1];
            xv[0] = first ? xv[0] : rr;
            yv[0] = first ? yv[0] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            *a.x[q] = xv[q];
            *a.y[q] = yv[q];
        }
        a.vb[0] = ux;
        a.vb[1] = uy;
        if (last) {
            *a.x[3] = xv[3];
            *a.y[3] = yv[3];
            *a.x[4] = xv[4];
            *a.y[4] = yv[4];
        }
        kx0 = xv[3];
        kx1 = yv[3];
        ky0 = xv[4];
        ky1 = yv[4];
        // one 16-byte store of the rotation's (c, s)
        HIP_vector_base<double, 2>::Native_vec_ value;
        value[0] = c;
        value[1] = sn;
        *(GLOBAL HIP_vector_base<double, 2>::Native_vec_ *)a.cs = value;
    };

    auto tick = [&](RotAddr<BP> &a, int t) {
        const bool live = ci < nch && t >= g.tau0;
        if (live) {
            if (fold) {
                // u v^T now touches only (N-1, n) and (N, n)
                const int fa = band_cell(N - 1, n), fb = band_cell(N, n);
                S[fa] = fma(S[UO + N - 1 + 3], S[VO + n + 3], S[fa]);
                S[fb] = fma(S[UO + N + 3], S[VO + n + 3], S[fb]);
            } else if (m1) {
                rotate(a, t == g.tau0, t == tend, std::true_type{});
            } else {
                rotate(a, t == g.tau0, t == tend, std::false_type{});
            }
            if (t == tend) {
                ci += nt;
                if (next) {
                    g = gn;
                    next = false;
                } else if (ci < nch) {
                    g = load_chain(h->chains, ci);
                    settle(g);
                }
                if (ci < nch) start();
            } else {
                advance(a, db, du, dcs);
            }
        }
        if (((t + 1) & (kRefill - 1)) == 0 && !next && ci + nt < nch) {
            gn = load_chain(h->chains, ci + nt);
            settle(gn);
            next = true;
        }
        __syncthreads();
    };

    int t = t_begin;
    if (t < t_end && (t & 1)) {
        tick(ao, t);
        ++t;
    }
    for (; t + 1 < t_end; t += 2) {
        tick(ae, t);
        tick(ao, t + 1);
    }
    if (t < t_end) tick(ae, t);

    if (t_end < ticks) {
        // a later part continues: keep the carries of a chain still in
        // flight (none at the end of phase 1)
        if (ci < nch && g.tau0 < t_end) {
            h->carry[4 * tid] = kx0;
            h->carry[4 * tid + 1] = kx1;
            h->carry[4 * tid + 2] = ky0;
            h->carry[4 * tid + 3] = ky1;
        }
        return;
    }
    for (int i = 1 + tid; i <= n; i += nt) {
        h->d[i - 1] = S[band_cell(i, i)];
        if (i < n) h->e[i - 1] = S[band_cell(i, i + 1)];
    }
}

// Row capacities of the LDS kernel's instances: a launch takes the smallest
// that holds its largest handle, so that small factorizations leave LDS for
// other workgroups of the CU.
#define BDU_GEN_CAPS(F) F(128) F(256) F(512) F(1024) F(2064) F(3392)
static_assert(kMaxGenLdsRows == 3392, "the largest capacity");

hipError_t prepare_kernels()
{
    static UntilDone once;
    return once([] {
        hipError_t e = hipSuccess;
#define BDU_GEN_ATTR(C)                                                                                       \
    if (e == hipSuccess)                                                                                      \
        e = hipFuncSetAttribute((const void *)gen_lds_kernel<C>, hipFuncAttributeMaxDynamicSharedMemorySize, \
                                GenLds<C>::BYTES);
        BDU_GEN_CAPS(BDU_GEN_ATTR)
#undef BDU_GEN_ATTR
        return e;
    });
}

hipError_t launch_gen(HandleDev *const *hs, int count, int64_t rows, bool in_lds, int threads, Gate gate,
                      hipStream_t st)
{
    if (threads < 64 || threads > kGenThreads || threads % 64) return hipErrorInvalidValue;
    if (in_lds) {
        hipError_t e = prepare_kernels();
        if (e != hipSuccess) return e;
#define BDU_GEN_CASE(C)                                                                                        \
    if (rows <= C) {                                                                                           \
        hipLaunchKernelGGL(gen_lds_kernel<C>, dim3(count), dim3(threads), GenLds<C>::BYTES, st, hs, gate);      \
        return hipGetLastError();                                                                              \
    }
        BDU_GEN_CAPS(BDU_GEN_CASE)
#undef BDU_GEN_CASE
        return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(gen_mem_kernel, dim3(count), dim3(threads), 0, st, hs, gate);
    return hipGetLastError();
}

}  // namespace bdu
