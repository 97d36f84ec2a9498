// apply_kernel.h -- gfx950 kernel accumulating the rotation streams into Q and P
// (Brust & Saunders, Section 3.4, eq. bidiagplus): the staged applier.  FP64
// throughout.
//
// A workgroup owns ROWS rows of Q or P (a panel) and sweeps the blocks of a
// launch over it, one front after the other (schedule.h).  A block's K =
// K0 * NW chains are dealt to NW pipeline stages of K0 chains; stage w holds
// local columns [3 (f - K0 + 1), 3 f + 6] of its rows in registers (f its own
// front, S = K0 + 3 fronts behind stage w - 1), applies its K0 rotations per
// front and hands finished columns to stage w + 1 through an LDS ring.  P
// pipelines of NW stages take the blocks in turn, each with a wavefront that
// moves columns between device memory and the pipeline's ends.
//
// What bounds it: a front is a dependent chain (pairs and columns from LDS,
// K0 rotations, columns to LDS, a barrier), so a wavefront alone on its SIMD
// needs about twice the time of its 4 K0 FP64 instructions, and the chip is
// only full with four wavefronts per SIMD on all 256 CUs.  One stream of
// n = 2048 has 64 panels of 64 rows.  Hence two splits for launches that do
// not fill the chip:
//   G stages share a wavefront, each on 64 / G lanes, and a lane owns R rows:
//   ROWS = 64 R / G.  All stages are S fronts apart and S is the length of
//   the unrolled loop, so they use the same registers at the same time.
//   P = 2 runs two blocks beside each other, twice the wavefronts per CU.
// Measured, all of one pass's application (both phases), with the generation
// beside it, against 64-row panels and one pipeline that also moved its
// pairs by the memory wavefront's loads of every line for three blocks:
//   n = 2048, K = 180        9.5 -> 6.3 ms (G 3, P 2: 196 workgroups)
//   4000 x 2000, K = 84     13.9 -> 8.4 ms (G 1, P 2)
//   10000 x 2000, K = 84    16.9 -> 9.9 ms (G 1, P 2; 1.0 ms of it the spike's
//                           rotations, in a kernel of their own, apply.hip)
//   n = 200, K = 84          420 -> 325 us (G 4)
//   64 streams of n = 2048, K = 180: 153 -> 143 ms (G 1, P 1)
//
// Coefficients.  A (c, s) pair serves all lanes of a stage.  With a wavefront
// to itself (G = 1) a stage holds its pairs in scalar registers
// (compute_run_sc).  Otherwise they go through the LDS: a front's pairs are
// loaded, coalesced, CD + 2 fronts ahead into a buffer of three fronts, and a
// stage reads each pair back as a 16-byte LDS read that all its lanes share
// (4 cycles on the LDS, against at least 20 for the rotation's FP64
// instructions; at four wavefronts per SIMD this would bound the kernel).
// LDS accesses of a wavefront complete in order, so every wait is for exactly
// the pair in use, and no compute wavefront waits on device memory.
//
// The memory and coefficient wavefronts run at the highest wave priority:
// all others wait for them at the barrier, and they share their SIMDs with
// up to four compute wavefronts (1 to 5 % of a launch).
#pragma once
#include <hip/hip_runtime.h>

#include <climits>
#include <type_traits>
#include <utility>

#include "device.h"
#include "kernels.h"
#include "primitives.h"
#include "schedule.h"

namespace bdu {

namespace {

typedef LOCAL double *LdsPtr;
typedef double double2v __attribute__((ext_vector_type(2)));
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));

__host__ __device__ constexpr int pmod(int a, int b) { return ((a % b) + b) % b; }

// Columns in the LDS ring between two stages: at most 14 columns are live
// (written but not yet read), and 3 r with r | (K0 + 3) keeps slots static.
__host__ __device__ constexpr int ring_cols(int K0)
{
    int U = K0 + 3, r = 5;
    while (U % r) ++r;
    return 3 * r;
}

template <int K0_, int NW_, int R_, int G_, int P_, int D_, int WAVES_>
struct Apply {
    static constexpr int K0 = K0_, NW = NW_, R = R_, G = G_, P = P_;
    static constexpr int WAVES = WAVES_;               // wavefronts a SIMD must hold
    static constexpr int U = K0 + 3, WSZ = 3 * U, K = K0 * NW;
    static constexpr int D = D_;                       // pairs in registers: D - 1 read ahead
    static constexpr int RC = ring_cols(K0);
    static constexpr int GL = 64 / G;                  // lanes of a stage
    static constexpr int ROWS = GL * R;                // rows of a panel
    static constexpr int NP = (NW + G - 1) / G;        // wavefronts of a pipeline
    static constexpr bool SC = G == 1;                 // pairs in scalar registers
    static constexpr bool OWN = !SC && P * (NP + 1) < 16 && P * K <= 192;  // a coefficient wavefront of its own?
    static constexpr int NT = 64 * (P * (NP + 1) + OWN);  // threads
    static constexpr int RING = RC * ROWS;             // doubles per ring
    static constexpr int NRING = NP * G + 1;           // rings 0 .. NW of a pipeline (and those of idle stages)
    static constexpr int DL = U / 3;                   // fronts of columns loaded ahead
    static constexpr int CD = U / 3;                   // fronts of pairs in flight
    static constexpr int CS = 3;                       // fronts in the pair buffer
    static constexpr int KB = P * K + (NP * G - NW) * K0;  // pairs of a front in it (idle stages read past their pipeline's)
    static constexpr int MAXB = 128;                   // blocks of a run
    static constexpr int COEF = P * NRING * RING;          // LDS offsets, in doubles
    static constexpr int TABLE = COEF + (SC ? 0 : 2 * CS * KB);
    static constexpr int LDS = TABLE + MAXB * 3 + 1;   // and the run's chunks and blocks
    static_assert(K0 % D == 0, "static pair registers");
    static_assert(U % 3 == 0 && U % DL == 0 && WSZ % RC == 0 && U % CS == 0 && U % CD == 0, "static ring slots");
};

// A block of a run, in the workgroup's table in LDS.
struct RunBlock {
    int rel, live, chunks;  // first chunk; live chunks of a stage; chunks swept
    int base, lmax;         // BlockDesc
    uint32_t off;           // first slot of the block's pairs, from the run's first
};
static_assert(sizeof(RunBlock) == 24, "three doubles");

// Writes of three finished columns by the lanes in `mask`, by narrowing the
// execution mask around them.
template <int O0, int O1, int O2>
__device__ __forceinline__ void masked_write3(uint64_t mask, LdsPtr p, double x0, double x1, double x2)
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

// The rotation at position P of a front in front_order, at front PHI of a chunk.
template <typename A, int MODE, int PHI, int P>
__device__ __forceinline__ void rotate_at(const double2v &cf, double (&buf)[A::R][A::WSZ])
{
    constexpr FrontOrder ord = front_order(MODE, A::K, A::K0);
    constexpr bool DESC = MODE < 2;
    constexpr int t = ord.t[P];
    constexpr int l0 = 3 * (PHI - t) + rho_of(MODE, A::K, t);
    constexpr int sx = pmod(l0 + (DESC ? 1 : 0), A::WSZ);
    constexpr int sy = pmod(l0 + (DESC ? 0 : 1), A::WSZ);
#pragma unroll
    for (int r = 0; r < A::R; ++r) rot(cf[0], cf[1], buf[r][sx], buf[r][sy]);
}

// f(integral_constant<0>), ..., f(integral_constant<N - 1>)
template <typename F, int... I>
__device__ __forceinline__ void unroll(F f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unroll(F f)
{
    unroll(f, std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ void front_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// A stage's place in a run: it is live in chunks [beg, end) of block b, for
// `live` chunks from the block's first plus its index.
struct Place {
    int b = -1, beg = 0, end = 0;
    uint32_t off = 0;
    // moves on to the block stage w is in at chunk ch, or to the last one,
    // among every step-th block
    __device__ __forceinline__ void enter(const RunBlock *table, int nb, int step, int w, int ch)
    {
        while (ch >= end && b + step < nb) {
            b += step;
            const RunBlock &t = table[b];
            const int a = t.live, c = t.chunks - w;
            beg = t.rel + w;
            end = beg + (a < c ? a : c);
            off = t.off;
        }
    }
};

// One compute wavefront over a run of T chunks of U fronts (nb blocks in the
// table), a barrier after every front.  Its G stages advance through the
// blocks on their own, at chunk boundaries, and outside of their live chunks
// compute along on whatever their registers hold with their ring writes
// masked.
template <typename A, int MODE>
__device__ __forceinline__ void compute_run(double *lds, int wave, int lane, int nb, int T)
{
    constexpr int U = A::U, WSZ = A::WSZ, K0 = A::K0, RC = A::RC, CS = A::CS, D = A::D;
    const RunBlock *table = (const RunBlock *)(lds + A::TABLE);
    const int pl = wave / A::NP;  // pipeline
    const int x = lane < A::GL * A::G ? lane : A::GL * A::G - 1;  // a lane to spare repeats the last one
    const int w = wave % A::NP * A::G + x / A::GL;  // this lane's stage
    const LdsPtr rin = (LdsPtr)lds + (pl * A::NRING + w) * A::RING + x % A::GL;
    const LdsPtr rout = rin + A::RING;
    typedef LOCAL double2v *PairPtr;
    const PairPtr mine = (PairPtr)((LdsPtr)lds + A::COEF) + pl * A::K + w * K0;
    double2v cf[D];  // pair p of a front in cf[p mod D], read D - 1 rotations ahead
    auto ahead = [&]() {  // a chunk's first pairs
#pragma unroll
        for (int p = 0; p < D - 1; ++p) cf[p] = mine[p];
    };
    double buf[A::R][WSZ];
    auto clear = [&]() {
#pragma unroll
        for (int r = 0; r < A::R; ++r)
#pragma unroll
            for (int i = 0; i < WSZ; ++i) buf[r][i] = 0.0;
    };
    clear();
    ahead();
    Place own;
    own.b = pl - A::P;
    for (int ch = 0; ch < T; ++ch) {
        if (__any(ch >= own.end)) own.enter(table, nb, A::P, w, ch);
        const int c = w < A::NW && ch < own.end ? ch - own.beg : -1;
        const uint64_t live = __builtin_amdgcn_ballot_w64(c >= 0);
        if (live == 0) {
            for (int phi = 0; phi < U; ++phi) front_barrier();
            ahead();
            clear();  // nothing in the window is needed any more
            continue;
        }
        if (__any(c == 0)) {
            if (c == 0) {
                // the block's first columns (the window starts finite: slots
                // not yet loaded meet identity rotations)
#pragma unroll
                for (int r = 0; r < A::R; ++r)
#pragma unroll
                    for (int i = 0; i < WSZ; ++i) buf[r][i] = i <= 3 ? rin[i * A::ROWS + r * A::GL] : 0.0;
            }
        }
        unroll<U>([&](auto pc) {
            constexpr int phi = decltype(pc)::value;
            // the next front's new columns 3 f + 4 .. 3 f + 6, read a front
            // early: their producer finished them two fronts ago
#pragma unroll
            for (int k = 4; k <= 6; ++k)
#pragma unroll
                for (int r = 0; r < A::R; ++r)
                    buf[r][pmod(3 * phi + k, WSZ)] = rin[pmod(3 * phi + k, RC) * A::ROWS + r * A::GL];
            unroll<K0>([&](auto qc) {
                constexpr int p = decltype(qc)::value, n = p + D - 1;
                cf[n % D] = mine[n < K0 ? phi % CS * A::KB + n : (phi + 1) % CS * A::KB + n - K0];
                rotate_at<A, MODE, phi, p>(cf[p % D], buf);
                if constexpr (p == K0 / 2 - 1) {
                    // the first rotations (chain K0 - 1) have finished the
                    // columns that leave the window
                    constexpr int l = 3 * (phi - K0 + 1), ROWB = 8 * A::ROWS;
#pragma unroll
                    for (int r = 0; r < A::R; ++r)
                        masked_write3<pmod(l, RC) * ROWB, pmod(l + 1, RC) * ROWB, pmod(l + 2, RC) * ROWB>(
                            live, rout + r * A::GL, buf[r][pmod(l, WSZ)], buf[r][pmod(l + 1, WSZ)],
                            buf[r][pmod(l + 2, WSZ)]);
                }
            });
            front_barrier();
            // keep fronts in order: the columns in use are materialised here,
            // so that two fronts are not interleaved
#pragma unroll
            for (int r = 0; r < A::R; ++r)
#pragma unroll
                for (int j = -3 * (K0 - 1); j <= 3; ++j) asm volatile("" : "+v"(buf[r][pmod(3 * phi + j, WSZ)]));
        });
    }
}

// A compute wavefront of one stage (G = 1), its pairs in scalar registers:
// the first half of a front's pairs is loaded in the middle of the previous
// front (once the first half of its rotations has freed those registers), the
// second half at the start of the front itself, so every scalar load has
// about half a front of work before its value is needed.  Scalar loads share
// their completion counter with LDS accesses and complete out of order, so
// every wait for one is a wait for all: the front's LDS accesses are all
// issued before the mid-front wait, and the barrier that ends the front waits
// for nothing more.
template <typename A, int MODE>
__device__ __forceinline__ void compute_run_sc(const CONSTANT double *__restrict__ cs, double *lds, int wave, int lane,
                                               int nb, int T)
{
    constexpr int U = A::U, WSZ = A::WSZ, K0 = A::K0, K = A::K, RC = A::RC, H = K0 / 2;
    const RunBlock *table = (const RunBlock *)(lds + A::TABLE);
    const int pl = wave / A::NW, w = wave % A::NW;
    const LdsPtr rin = (LdsPtr)lds + (pl * A::NRING + w) * A::RING + lane;
    const LdsPtr rout = rin + A::RING;
    double buf[A::R][WSZ];
    double c[K0], sn[K0];
    // pairs [p0, p1) of front phi of the chunk at q
    auto load = [&](const CONSTANT double *q, int phi, int p0, int p1) {
#pragma unroll
        for (int p = 0; p < K0; ++p)
            if (p >= p0 && p < p1) {
                c[p] = q[2 * (phi * K + p)];
                sn[p] = q[2 * (phi * K + p) + 1];
            }
    };
    int cur = 0;  // chunks of barriers run so far
    for (int b = pl; b < nb; b += A::P) {
        const int beg = __builtin_amdgcn_readfirstlane(table[b].rel) + w;
        const int live = __builtin_amdgcn_readfirstlane(table[b].live);
        const int most = __builtin_amdgcn_readfirstlane(table[b].chunks) - w;
        const int end = beg + (live < most ? live : most);
        const uint32_t off = __builtin_amdgcn_readfirstlane(table[b].off);
        for (int i = (beg - cur) * U; i > 0; --i) front_barrier();
        cur = end > beg ? end : beg;
        const CONSTANT double *q = cs + 2 * ((int64_t)off + (int64_t)w * (U * K) + w * K0);
#pragma unroll
        for (int r = 0; r < A::R; ++r)
#pragma unroll
            for (int i = 0; i < WSZ; ++i) buf[r][i] = i <= 3 ? rin[i * A::ROWS + r * 64] : 0.0;
        load(q, 0, 0, H);
        for (int ch = beg; ch < end; ++ch) {
            const CONSTANT double *const qn = ch + 1 < end ? q + 2 * U * K : q;  // past the end: this chunk's again
            unroll<U>([&](auto pc) {
                constexpr int phi = decltype(pc)::value;
                // the first half's pairs (loaded during the previous front)
                // have landed before the second half's loads are issued
                asm volatile("" ::"s"(c[0]));
                __builtin_amdgcn_sched_barrier(0);
                load(q, phi, H, K0);
                __builtin_amdgcn_sched_barrier(0);
                // the next front's new columns 3 f + 4 .. 3 f + 6
#pragma unroll
                for (int k = 4; k <= 6; ++k)
#pragma unroll
                    for (int r = 0; r < A::R; ++r)
                        buf[r][pmod(3 * phi + k, WSZ)] = rin[pmod(3 * phi + k, RC) * A::ROWS + r * 64];
                unroll<H>([&](auto qc) {
                    constexpr int p = decltype(qc)::value;
                    rotate_at<A, MODE, phi, p>(double2v{c[p], sn[p]}, buf);
                });
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int r = 0; r < A::R; ++r)
                        rout[pmod(3 * (phi - K0 + 1) + k, RC) * A::ROWS + r * 64] =
                            buf[r][pmod(3 * (phi - K0 + 1) + k, WSZ)];
                // wait here (not after the next loads) for this front's second
                // half; every LDS access of the front is complete after it
                asm volatile("" ::"s"(c[H]));
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (phi + 1 < U) load(q, phi + 1, 0, H);
                else load(qn, 0, 0, H);
                __builtin_amdgcn_sched_barrier(0);
                unroll<K0 - H>([&](auto qc) {
                    constexpr int p = H + decltype(qc)::value;
                    rotate_at<A, MODE, phi, p>(double2v{c[p], sn[p]}, buf);
                });
                asm volatile("s_barrier" ::: "memory");
#pragma unroll
                for (int r = 0; r < A::R; ++r)
#pragma unroll
                    for (int j = -3 * (K0 - 1); j <= 3; ++j) asm volatile("" : "+v"(buf[r][pmod(3 * phi + j, WSZ)]));
            });
            q = qn;
        }
    }
    for (int i = (T - cur) * U; i > 0; --i) front_barrier();
}

// Brings pairs [first, first + N) of every front of a run: at front F it
// writes front F + 2's to the buffer (the stages read a front's first ones at
// the end of the front before it) and loads those of front F + 2 + CD.  Lane l
// moves pairs l, l + 64, ... of them.  For stages that load their pairs by
// scalar loads (SC) it only brings them into the L2 cache, one word of every
// 128-byte line (eight pairs) per lane: without it those loads go to memory.
template <typename A, int N>
struct Pairs {
    static constexpr bool SC = A::SC;
    static constexpr int U = A::U, K = A::K, CD = A::CD, NL = SC ? 1 : (N + 63) / 64;
    static_assert(!SC || (N == K && K <= 8 * 63), "a lane for every line");
    typedef std::conditional_t<SC, int, double2v> Word;
    typedef LOCAL double2v *PairPtr;
    const RunBlock *table;
    const GLOBAL char *cs;
    PairPtr to;
    int lane, nb;
    Place src[NL];
    uint32_t at[NL], next[NL];  // byte offsets in the run's pairs, this chunk's and the next's
    int i[NL];
    Word fifo[CD][NL];

    __device__ __forceinline__ uint32_t source(int it, int ch)
    {
        const int x = i[it] % K, v = x / A::K0;
        Place &p = src[it];
        if (__any(ch >= p.end)) p.enter(table, nb, A::P, v, ch);
        int c = ch < p.end ? ch - p.beg : p.end - 1 - p.beg;  // past the end: the last chunk's again
        c = c < 0 ? 0 : c;
        return 16u * (p.off + (uint32_t)((c + v) * (U * K) + x));
    }
    // the pair at offset o of the chunk's front f
    __device__ __forceinline__ Word load(uint32_t o, int f) const
    {
        return *(const GLOBAL Word *)(cs + (int64_t)f * (16 * K) + (uint64_t)o);
    }
    __device__ __forceinline__ void put(int slot, int it, Word v)
    {
        if constexpr (SC) asm volatile("" ::"v"(v));  // here by now
        else if (it * 64 + 64 <= N || it * 64 + lane < N) to[slot * A::KB + it * 64] = v;
    }
    __device__ __forceinline__ void begin(const GLOBAL double2v *run, double *lds, int first, int lane_, int nb_)
    {
        table = (const RunBlock *)(lds + A::TABLE);
        cs = (const GLOBAL char *)run;
        lane = lane_;
        nb = nb_;
        to = (PairPtr)((LdsPtr)lds + A::COEF) + first + lane;
#pragma unroll
        for (int it = 0; it < NL; ++it) {
            const int x = SC ? 8 * lane : it * 64 + lane;
            i[it] = first + (x < N ? x : N - 1);
            src[it] = Place();
            src[it].b = i[it] / K - A::P;
            at[it] = source(it, 0);
            const Word v0 = load(at[it], 0), v1 = load(at[it], 1);
#pragma unroll
            for (int j = 0; j < CD; ++j) fifo[j][it] = load(at[it], j + 2);
            next[it] = source(it, 1);
            put(0, it, v0);
            put(1, it, v1);
        }
    }
    template <int PHI>
    __device__ __forceinline__ void front()
    {
        constexpr int f = PHI + 2 + CD;
#pragma unroll
        for (int it = 0; it < NL; ++it) {
            put((PHI + 2) % A::CS, it, fifo[PHI % CD][it]);
            fifo[PHI % CD][it] = f < U ? load(at[it], f) : load(next[it], f - U);
        }
    }
    __device__ __forceinline__ void chunk(int ch)
    {
#pragma unroll
        for (int it = 0; it < NL; ++it) {
            at[it] = next[it];
            next[it] = source(it, ch + 2);
        }
    }
};

// A coefficient wavefront of its own, for all pipelines.
template <typename A>
__device__ __forceinline__ void pairs_run(const GLOBAL double2v *__restrict__ cs, double *lds, int lane, int nb, int T)
{
    Pairs<A, A::P * A::K> pairs;
    pairs.begin(cs, lds, 0, lane, nb);
    front_barrier();
    for (int ch = 0; ch < T; ++ch) {
        unroll<A::U>([&](auto pc) {
            pairs.template front<decltype(pc)::value>();
            front_barrier();
        });
        pairs.chunk(ch);
    }
}

// First chunk of a block when P pipelines share the blocks.
template <int P, typename B>
__device__ __forceinline__ int start_of(const B &d)
{
    static_assert(P == 1 || P == 2, "planned starts");
    return P == 1 ? d.start : d.start2;
}

// The memory wavefront of pipeline pl over the nb blocks of a run's table, of
// which every P-th is its own; they run back to back (start chunks from the
// plan): T chunks of U fronts, one barrier per front.  Its load side follows
// the block of its latest prologue (the block stage 0 is in or waits for): at
// front F of that block it writes to ring 0 the columns stage 0 reads at front
// F + 1 (3F + 7 .. 3F + 9, loaded DL fronts earlier into a register FIFO); a
// block's columns 0..6 and first DL FIFO entries are loaded in its prologue,
// the front before it starts, which also overwrites whatever the load side
// wrote for the previous block past its end.  Its store side follows the
// oldest block not yet written back: at front F it stores the columns the
// last stage finished at front F - 1.
//
// Every load and store is issued at every front, from one place in the code,
// whether or not its data is needed, so that the compiler can count them and
// wait only for the FIFO entry in use.  (With the loads in two branches, or
// the stores under one, it waits for all in flight or for the entry of two
// fronts ago: 177 against 143 ms for 64 streams of n = 2048.)  Columns past
// the matrix's ends are loaded from its last column there; stores of columns
// outside of the block are dropped by the buffer's bounds.  A column is
// loaded for one block only after an earlier block's store of it has
// completed; the plan's start chunks guarantee that (stage_starts in
// plan.cpp).
//
// A front's three columns are 3 ROWS doubles: access q of NQ moves doubles
// 64 q .. 64 q + 63 of them (row x mod ROWS of column x / ROWS).
template <typename A>
__device__ __forceinline__ void memory_run(GLOBAL double *__restrict__ X, int ld, int ncols, int row0, bool desc,
                                           const GLOBAL double2v *__restrict__ cs, int pl, int nb, int T, double *lds,
                                           int lane)
{
    constexpr int U = A::U, RC = A::RC, DL = A::DL, ROWS = A::ROWS, NW = A::NW, K0 = A::K0, P = A::P;
    constexpr int NQ = (3 * ROWS + 63) / 64;
    const RunBlock *table = (const RunBlock *)(lds + A::TABLE);
    auto kof = [&](int q) { return ROWS % 64 == 0 ? q * 64 / ROWS : (q * 64 + lane) / ROWS; };  // column of the three
    auto rof = [&](int q) { return ROWS % 64 == 0 ? q * 64 % ROWS + lane : (q * 64 + lane) % ROWS; };  // row
    auto used = [&](int q) { return 3 * ROWS % 64 == 0 || q * 64 + lane < 3 * ROWS; };
    // rows of a last panel past the leading dimension: read from its last row, never written
    auto real = [&](int q) { return 128 % ROWS == 0 || row0 + rof(q) < ld; };
    auto at = [&](int q) { return 128 % ROWS == 0 || row0 + rof(q) < ld ? rof(q) : ld - 1 - row0; };
    const int dir = desc ? -1 : 1;
    // local column lam of a block: matrix column col0 + dir lam
    auto base_of = [&](int b) { return __builtin_amdgcn_readfirstlane(table[b].base); };
    // A front's three columns by their lowest one: its address, and each
    // lane's offsets from there, the same for every front.
    uint32_t off[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int k = kof(q) < 3 ? kof(q) : 2;
        off[q] = 8u * ((uint32_t)(desc ? 2 - k : k) * ld + at(q));
    }
    GLOBAL char *const X0 = (GLOBAL char *)(X + row0);
    const int64_t step = (int64_t)dir * 24 * ld;
    auto lowest = [&](int base, int lam) { return base - 1 + dir * lam - (desc ? 2 : 0); };
    auto address = [&](int c) { return X0 + (int64_t)c * (8 * ld); };

    // load side: the next three columns to load
    double fifo[DL][NQ];
    const LdsPtr first = (LdsPtr)lds + pl * A::NRING * A::RING, last = first + NW * A::RING;
    int lc = 0, lcstep = 0;
    GLOBAL char *lp = X0;
    int64_t lstep = 0;
    auto load_entry = [&](int slot) {
        uint32_t o[NQ];
        GLOBAL char *base = lp;
#pragma unroll
        for (int q = 0; q < NQ; ++q) o[q] = off[q];
        const bool inside = lc >= 0 && lc + 2 < ncols;
        if (!inside) {
            const int cb = lc < 0 ? 0 : (lc >= ncols ? ncols - 1 : lc);
            base = address(cb);
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int k = kof(q) < 3 ? kof(q) : 2;
                int c = lc + (desc ? 2 - k : k);
                c = c < 0 ? 0 : (c >= ncols ? ncols - 1 : c);
                o[q] = 8u * ((uint32_t)(c - cb) * ld + at(q));
            }
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) fifo[slot][q] = *(const GLOBAL double *)(base + (uint64_t)o[q]);
        if (desc ? lc + 2 < 0 : lc >= ncols) {  // past the block: wait at column 0
            lc = lcstep = 0;
            lp = X0;
            lstep = 0;
        }
        lc += lcstep;
        lp += lstep;
    };
    auto prologue = [&](int b) {
        constexpr int N = (7 * ROWS + 63) / 64;
        const int base = base_of(b);
#pragma unroll
        for (int q = 0; q < N; ++q) {
            if (q * 64 + lane < 7 * ROWS) {
                int c = base - 1 + dir * kof(q);
                c = c < 0 ? 0 : (c >= ncols ? ncols - 1 : c);
                first[kof(q) * ROWS + rof(q)] = X[(int64_t)c * ld + row0 + at(q)];
            }
        }
        lc = lowest(base, 7);
        lcstep = 3 * dir;
        lp = address(lc);
        lstep = step;
#pragma unroll
        for (int j = 0; j < DL; ++j) load_entry(j);
    };
    // the front before the next block starts
    int bl = pl, bs = pl, next_pro;
    auto plan_prologue = [&]() {
        bl += P;
        next_pro = bl < nb ? __builtin_amdgcn_readfirstlane(table[bl].rel) * U - 1 : -2;
    };
    // store side: at front F of the run the block's local columns slam .. slam + 2
    int slam, slo, shi, send;
    GLOBAL char *sp;
    auto store_block = [&](int F) {
        if (bs < nb) {
            const int base = base_of(bs);
            slam = 3 * (F - __builtin_amdgcn_readfirstlane(table[bs].rel) * U - (NW - 1) * U - K0);
            shi = __builtin_amdgcn_readfirstlane(table[bs].lmax) + 1;
            slo = desc && base > ncols ? base - ncols : 0;
            send = shi / 3 * 3;
            sp = address(lowest(base, slam));
        } else {  // nothing left to store
            slam = INT_MIN / 2;
            slo = shi = 0;
            send = INT_MAX;
            sp = X0;
        }
    };
    store_block(0);
    // a pipeline without blocks loads the first one's columns for nobody
    prologue(pl < nb ? pl : 0);  // the first block's; a later one's again, the front before it starts
    if (pl < nb && table[pl].rel > 0) next_pro = __builtin_amdgcn_readfirstlane(table[pl].rel) * U - 1;
    else plan_prologue();
    Pairs<A, A::K> pairs;
    if constexpr (!A::OWN) pairs.begin(cs, lds, pl * A::K, lane, nb);
    front_barrier();
    for (int G0 = 0; G0 < T * U; G0 += U) {
        unroll<U>([&](auto pc) {
            constexpr int phi = decltype(pc)::value, slot = phi % DL;
            const int F = G0 + phi;
            double out[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                int sl = pmod(3 * phi - 3 * K0, RC) + (kof(q) < 3 ? kof(q) : 2);
                sl = sl >= RC ? sl - RC : sl;
                out[q] = last[sl * ROWS + rof(q)];
            }
            // load side (past the block's end it feeds nobody; the next
            // prologue overwrites those slots)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                // ring slot of column 3 phi + 7 + k: consecutive modulo RC
                int sl = pmod(3 * phi + 7, RC) + kof(q);
                sl = sl >= RC ? sl - RC : sl;
                if (used(q)) first[sl * ROWS + rof(q)] = fifo[slot][q];
            }
            load_entry(slot);
            if constexpr (!A::OWN) pairs.template front<phi>();
            // store side
            {
                const __amdgpu_buffer_rsrc_t to =
                    __builtin_amdgcn_make_buffer_rsrc((void *)(uintptr_t)sp, 0, 0x7fffffff, 0x00027000);
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const int lam = slam + kof(q);
                    const bool mine = used(q) && real(q) && lam >= slo && lam <= shi;
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uint2v, out[q]), to,
                                                          mine ? off[q] : 0xffffffffu, 0, 0);
                }
            }
            // the block's last column is stored at this front
            if (slam >= send) {
                bs += P;
                store_block(F + 1);
            } else {
                slam += 3;
                sp += step;
            }
            // the next block's prologue, the front before it starts (always
            // the last front of a chunk: blocks start on chunk boundaries)
            if (phi == U - 1 && F == next_pro) {
                prologue(bl);
                plan_prologue();
            }
            front_barrier();
        });
        if constexpr (!A::OWN) pairs.chunk(G0 / U);
    }
    // a later run loads these columns again
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// grid (panels, handles): panels [0, ceil(m / ROWS)) update Q, the rest P.
// The pass's blocks go in runs of one phase and at most MAXB blocks.
template <typename A>
__global__ __launch_bounds__(A::NT) __attribute__((amdgpu_waves_per_eu(A::WAVES))) void apply_staged_kernel(HandleDev *const *hs, Gate gate)
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
    const int qp = (m + A::ROWS - 1) / A::ROWS, pp = (n + A::ROWS - 1) / A::ROWS;
    if (pid >= qp + pp) return;
    __shared__ double lds[A::LDS];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    // the rings start finite (stale slots may meet identity rotations)
    for (int i = threadIdx.x; i < A::COEF; i += A::NT) lds[i] = 0.0;
    const int nb1 = h->nb1;
    const bool onQ = pid < qp;
    const int row0 = (onQ ? pid : pid - qp) * A::ROWS;
    GLOBAL double *X = gptr(onQ ? h->Q : h->P);
    const int ld = onQ ? h->ldq : h->ldp;
    const int ncols = onQ ? m : n;
    const BlockDesc *blk = onQ ? h->blkL : h->blkR;
    const GLOBAL double2v *cs = (const GLOBAL double2v *)gptr((double *)(onQ ? h->csL : h->csR));
    int bbeg, bend;
    (void)part_blocks(h, gate.part, &bbeg, &bend);
    RunBlock *table = (RunBlock *)(lds + A::TABLE);
    int *chunks = (int *)(lds + A::TABLE + 3 * A::MAXB);
    for (int b0 = bbeg; b0 < bend;) {
        const bool phase1 = b0 < nb1;
        int b1 = phase1 && bend > nb1 ? nb1 : bend;
        // as many blocks as the table holds and 32-bit offsets reach
        const int64_t bytes = (int64_t)16 * A::K * (ncols / 3 + (A::NW + 2) * A::U);
        const int most = bytes * A::MAXB < (int64_t)1 << 31 ? A::MAXB : (int)(((int64_t)1 << 31) / bytes);
        b1 = b1 < b0 + most ? b1 : b0 + most;
        const int start0 = start_of<A::P>(kptr(blk)[b0]);
        const int64_t off0 = kptr(blk)[b0].off;
        const GLOBAL double2v *run = cs + off0;
        __syncthreads();  // the previous run has left the table
        if (threadIdx.x == 0) chunks[0] = chunks[1] = 0;
        __syncthreads();
        for (int x = threadIdx.x; x < b1 - b0; x += A::NT) {
            const GLOBAL BlockDesc *d = gptr((BlockDesc *)blk) + b0 + x;
            RunBlock r;
            r.rel = start_of<A::P>(*d) - start0;
            r.chunks = d->nfront / A::U;
            r.base = d->base;
            r.lmax = d->lmax;
            r.live = ((d->lmax + 1) / 3 + A::K0 - 1 + A::U) / A::U;
            r.off = (uint32_t)(d->off - off0);
            table[x] = r;
            // the run ends when its latest block's last column is stored;
            // blocks without work come last
            if (d->lmax >= 0) {
                atomicMax(&chunks[0], r.rel + r.chunks);
                atomicMax(&chunks[1], x + 1);
            }
        }
        __syncthreads();
        const int T = __builtin_amdgcn_readfirstlane(chunks[0]);
        const int nb = __builtin_amdgcn_readfirstlane(chunks[1]);
        if (T > 0) {
            if (w >= A::P * A::NP) __builtin_amdgcn_s_setprio(3);
            if (w >= A::P * A::NP && w < A::P * (A::NP + 1)) {
                memory_run<A>(X, ld, ncols, row0, phase1, run, w - A::P * A::NP, nb, T, lds, lane);
            } else if (A::OWN && w == A::P * (A::NP + 1)) {
                if constexpr (A::OWN) pairs_run<A>(run, lds, lane, nb, T);
            } else {
                front_barrier();  // the first columns and pairs are in LDS
                auto compute = [&](auto mode) {
                    constexpr int MODE = decltype(mode)::value;
                    if constexpr (A::SC) compute_run_sc<A, MODE>(kptr((const double *)run), lds, w, lane, nb, T);
                    else compute_run<A, MODE>(lds, w, lane, nb, T);
                };
                if (phase1) {
                    if (onQ) compute(std::integral_constant<int, 0>{});
                    else compute(std::integral_constant<int, 1>{});
                } else {
                    if (onQ) compute(std::integral_constant<int, 2>{});
                    else compute(std::integral_constant<int, 3>{});
                }
            }
        }
        b0 = b1;
    }
}

template <int K0, int NW, int R, int G, int P, int D, int WAVES>
hipError_t launch_t(HandleDev *const *hs, int count, int panels, Gate gate, hipStream_t st)
{
    using A = Apply<K0, NW, R, G, P, D, WAVES>;
    // Q's and P's rows are in whole panels each: one more where 64-row panels
    // do not divide into this kernel's
    const int wgs = (panels * 64 + A::ROWS - 1) / A::ROWS + (64 % A::ROWS && A::ROWS % 64 ? 1 : 0);
    hipLaunchKernelGGL(apply_staged_kernel<A>, dim3(wgs, count), dim3(A::NT), 0, st, hs, gate);
    return hipGetLastError();
}

}  // namespace
}  // namespace bdu
