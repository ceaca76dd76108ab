// stepper.h -- fused implicit time steps with the state kept on chip: every
// step builds the right-hand side of a system from its current state (an
// explicit stencil, possibly nonlinear) and solves the shared banded LHS,
// `steps` times per launch, reading the batch once and writing it once.
// The right-hand-side rule is a policy (Rhs); ch.hip (Cahn-Hilliard, Section
// 5.1) and cn_stencil.h (Crank-Nicolson diffusion and hyperdiffusion, Sections 3
// and 4 benchmark problems) instantiate it.
//
// An Rhs policy provides
//   static constexpr int R;   // rows of halo it reads on each side (1, 2 or 3)
//   struct State;             // per-lane data of the system it works on
//   State lane_state(int64_t k, int row0) const;   // system k, chunk from row0
//   template <int C, bool FULL>
//   void operator()(double (&c)[C], const Halo &h, int j, bool last_chunk, int nrow,
//                   const State &s) const;
// which overwrites the chunk c (rows j*C .. j*C + C - 1 of the system) with
// the right-hand side.  nrow = n - j*C (rows of the chunk that are real when
// the decomposition is ragged); last_chunk: j == P - 1.
#pragma once

#include <type_traits>

#include "sweep_core.h"

namespace bb {
namespace {

// Values around a chunk: the R rows above it (l1 = row j*C - 1, l2, l3;
// 0 for the first chunk) and below it (r1 = row j*C + C, r2, r3; 0 past the
// last chunk), and rows 0, 1, 2, n-3, n-2, n-1 of the system (for periodic
// wrap-around).  Entries a smaller R does not read stay 0.
struct Halo {
    double l1, l2, l3, r1, r2, r3;
    double e0, e1, e2, en3, en2, en1;
};

// Optional per-run statistic of the fused steps (Cahn-Hilliard coarsening,
// Section 5, batched 1D scaling), compiled in only where asked for (STATS):
// after every `every` steps, each system's typical domain size
// 1 / (1 - <c^2>), <c^2> = (1/n) sum_i c_i^2, summed over the systems of its
// group in a fixed order and stored at [group][sample] of `partial` (each
// entry written once; no read-modify-write inside the step loop).
struct StepStats {
    double *partial = nullptr;
    int64_t every = 1, samples = 0;
    double inv_n = 0.0;
    int64_t traj_stride = 0;   // TRAJ: elements between the states of consecutive steps in `out`
};

// sum of squares of this lane's rows (padding rows hold 0): four interleaved
// partial sums (rows t mod 4) keep the dependency chain short, combined in a
// fixed order
template <int C>
__device__ __forceinline__ double chunk_sum_sq(const double (&c)[C])
{
    double ss[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < C; ++t) ss[t & 3] = fma(c[t], c[t], ss[t & 3]);
    return (ss[0] + ss[1]) + (ss[2] + ss[3]);
}

// Sum of v over the S lanes of each block of S consecutive lanes (S a power
// of two), a fixed butterfly: every lane of the block gets the same sum.
__device__ __forceinline__ double block_sum(double v, int S)
{
    for (int off = 1; off < S; off <<= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// Whether a ragged group of one wave has all of a chunk's rows in flight before
// it selects the first, rather than selecting each as it comes.  With 64-row
// chunks the latter: launches of few steps start sooner (trajectory of 4 states,
// tri n = 777, m = 8192: 117 against 102 us, n = 1000, m = 8192 191 and 175; one
// step, penta n = 777, m = 2^16 424 and 409; 10 steps, periodic tri n = 1025,
// m = 8192 888 and 848).  The former for pentadiagonal systems that are periodic
// (n = 600, m = 2^16, states stored 400 against 411 us a step) or in shorter
// chunks (n = 600, m = 1000, 10 steps 96 and 102), and for trajectories of periodic
// tridiagonal systems of more than 16 chunks (4 states, n = 1025, m = 8192 447 and
// 470; n = 1000, of 16, 207 and 185).
constexpr bool step_rows_first(int K, bool cyclic, int C) { return K == 2 && (cyclic || C < 64); }

// One lane per chunk; the lanes of a system sit in one wave (shuffles) and
// the coefficient table is staged in LDS.
// TRAJ: the state after every step s (0-based) is stored at
// out + s * st.traj_stride instead of only the last one at out.
template <class Rhs, int K, bool CYC, int C, bool FULL, bool STATS, bool TRAJ,
          bool ALL = step_rows_first(K, CYC, C)>
__global__ __launch_bounds__(kMaxBlockThreads) void step_kernel(const double *__restrict__ table,
                                                             int64_t table_elems, CyclicQ cq,
                                                             SweepGeom g, Rhs rhs, int64_t steps,
                                                             StepStats st, const double *in,
                                                             double *out)
{
    extern __shared__ double smem_d[];
    stage_table(smem_d, table, table_elems);
    __syncthreads();

    const LaneGeom lg = lane_geom(g.log2P);
    const int lane = threadIdx.x % kWave;
    const int row0 = lg.j * C;
    const bool has_left = lg.j > 0, has_right = lg.j < lg.P - 1;
    const int left = has_left ? lane - lg.S : lane;
    const int right = has_right ? lane + lg.S : lane;
    const int exact = FULL || g.exact;
    const GroupRange gr = group_range(g.groups, 0, STATS ? 0 : g.linear);

    for (int64_t blk = gr.first; blk < gr.end; blk += gr.stride) {
        const int64_t grp = begin_block(gr, blk, g.lockstep);
        if (grp >= g.groups) continue;
        const int64_t k = grp * lg.S + lg.sl;
        const bool kval = k < g.m;
        double c[C];
        load_chunk<double, C, FULL, ALL>(c, in, row0, kval ? k : g.m - 1, g.ld, g.n);
        const typename Rhs::State ls = rhs.lane_state(kval ? k : g.m - 1, row0);

        for (int64_t step = 0; step < steps; ++step) {
            Halo h = {};
            h.l1 = shfl(c[C - 1], left);
            h.r1 = shfl(c[0], right);
            if (!has_left) h.l1 = 0.0;
            if (!has_right) h.r1 = 0.0;
            if constexpr (Rhs::R >= 2) {
                h.l2 = shfl(c[C - 2], left);
                h.r2 = shfl(c[1], right);
                if (!has_left) h.l2 = 0.0;
                if (!has_right) h.r2 = 0.0;
            }
            if constexpr (Rhs::R >= 3) {
                h.l3 = shfl(c[C - 3], left);
                h.r3 = shfl(c[2], right);
                if (!has_left) h.l3 = 0.0;
                if (!has_right) h.r3 = 0.0;
            }
            gather_ends<double, 2, C>(c, lg, g.n, exact, h.e0, h.e1, h.en2, h.en1);
            if constexpr (Rhs::R >= 3) {
                h.e2 = shfl(c[2], lg.sl);
                h.en3 = exact ? shfl(c[C - 3], (g.n / C - 1) * lg.S + lg.sl)
                              : shfl(pick(c, (g.n - 3) % C), ((g.n - 3) / C) * lg.S + lg.sl);
            }
            rhs.template operator()<C, FULL>(c, h, lg.j, lg.j == lg.P - 1, opaque_v(g.n - row0), ls);
            __builtin_amdgcn_sched_barrier(0);
            chunk_solve<double, K, C, CYC, FULL>(c, smem_d, lg, g.n, cq);
            if (STATS && (step + 1) % st.every == 0) {
                // chunks of a system: lanes j*S + sl of this wave, summed in chunk order
                const double ss = chunk_sum_sq<C>(c);
                double tot = 0.0;
                for (int i = 0; i < lg.P; ++i) tot += shfl(ss, i * lg.S + lg.sl);
                // l - 1 = <C^2> / (1 - <C^2>): summed without the 1 of every run,
                // so the ensemble sum keeps the digits that l - 1 carries
                const double msq = tot * st.inv_n;
                const double ell = kval ? msq / (1.0 - msq) : 0.0;
                const double sum = block_sum(ell, lg.S);   // the group: lanes 0 .. S-1
                if (lane == 0) st.partial[grp * st.samples + (step + 1) / st.every - 1] = sum;
            }
            if constexpr (TRAJ) {
                if (kval) store_chunk<double, C, FULL>(c, out + step * st.traj_stride, row0, k, g.ld, g.n);
            }
        }
        if constexpr (!TRAJ) {
            if (kval) store_chunk<double, C, FULL>(c, out, row0, k, g.ld, g.n);
        }
    }
}

// Any number of waves per group: chunks that tile n, or a last chunk with padding.
constexpr int kRagFull = 1, kRagTail = 2;

// x = v[t], or v[t] = x (PUT), for a wave-uniform t: a tree of scalar branches.
// The fence that ends each leaf keeps the compiler from merging them into one
// indexed access, for which it would put the whole chunk into scratch memory.
template <bool PUT, int LO, int HI, int C>
__device__ __forceinline__ void row_at(double (&v)[C], int t, double &x)
{
    if constexpr (HI - LO == 1) {
        if constexpr (PUT)
            v[LO] = x;
        else
            x = v[LO];
        asm volatile("" : "+v"(x));
    } else {
        constexpr int MID = (LO + HI) / 2;
        if (t < MID)
            row_at<PUT, LO, MID>(v, t, x);
        else
            row_at<PUT, MID, HI>(v, t, x);
    }
}

// Waves per SIMD a split kernel is held to.  Three, with 64-row chunks in 168
// VGPRs, in workgroups of four waves or fewer with at most two halo rows: a step
// waits at its barriers and for its recurrences, and the other workgroups of the
// CU fill in.  Most get there with a few VGPRs spilled (4-wave Cahn-Hilliard 4,
// with the statistic 2, periodic penta 6, tri of 16 chunks 10; three full chunks,
// periodic penta 22, penta 4, Cahn-Hilliard 16) and are faster all the same (us
// for 20 steps, two waves and three; n = 256, m = 2^18: Cahn-Hilliard 958 and 822,
// with the statistic 1149 and 967, periodic penta 961 and 769, penta, no spills,
// 793 and 803; n = 192, m = 2^18: periodic penta 950 and 800, penta 883 and 655,
// Cahn-Hilliard 949 and 772; tri n = 1024, m = 2^16: 606 and 600, periodic 605
// and 569).  The spills cost launches that store every state: periodic penta
// n = 192 one step 171 and 199 us, 4 states at m = 2^17 217 and 252.
constexpr int step_waves(int K, int C, int QL, bool scalar, int rows, int R, int rag)
{
    const bool three = C == 64 && QL <= 2 && R <= 2 && rag != kRagTail &&
                       (scalar || (rows == 4 && K == 1));
    return three ? 3 : QL == 3 ? 2 : 1;
}

// Whether a kernel with one chunk per wave takes its coefficients by row
// broadcast from an LDS table rather than through the scalar cache: the
// passes then need neither scalar loads nor the fenced blocks of rows that
// wait for them (us a step, scalar vs broadcast: tri n = 512, m = 2^17 39.2 vs
// 28.8, penta 57.9 vs 46.4; penta n = 500, m = 5000 9.4 vs 8.0; penta
// n = 200, m = 2^16 16.0 vs 14.3; 32-row chunks tri n = 128, m = 2^14 2.0 vs
// 1.6).  Not where the scalar kernel keeps three waves per SIMD and the other,
// which holds the pass's coefficients in VGPRs, two (Cahn-Hilliard n = 256,
// m = 2^18 36.8 vs 38.9), nor in groups of two or three such waves (penta
// n = 100, m = 2^17 15.5 vs 20.1).
constexpr bool chunk_by_rows(int K, int C, int waves, int R, bool full)
{
    if (C == 32) return waves >= 3;
    return C == 64 && (waves >= 5 || (waves == 4 && (!full || K == 1 || R > 2)));
}

// The same steps with a system group split over the Q = 2^QL waves of a
// workgroup (chunks tile n exactly): wave q holds chunks q*P/Q ..
// (q+1)*P/Q - 1 of S = 64Q/P systems, and every chunk-boundary value goes
// through the LDS exchange area: the first and last R rows of every chunk
// for the stencil and the wrap-around, then the phases of chunk_solve.
// SCALAR (one chunk per wave, P == Q): every lane of a wave needs the same
// coefficient row at the same time, so the coefficients come from the global
// table through the scalar cache (no LDS staging, no LDS reads).  Otherwise
// the table is staged in LDS ahead of the exchange area.
// ROWS: chunks per wave (1, 2 or 4) of a group whose LDS coefficients go by
// row broadcast, 0: plain LDS reads.
// RAG (one chunk per wave): any number of waves up to 2^QL, each with one chunk of C rows;
// kRagFull: they tile n, kRagTail: the last holds the rows that remain.  Only
// that wave loads and stores with row predicates, and periodic ghost rows in
// its padding let it run the right-hand side of a full chunk (a second,
// predicated copy of the right-hand side put 0.5-1.5 KB of every lane into
// scratch).  Times beside the rule (step_plan).
template <class Rhs, int K, bool CYC, int C, int QL, bool SCALAR, bool STATS, bool TRAJ,
          int ROWS = 0, int RAG = 0>
__global__ __launch_bounds__((kWave << QL) > kMaxBlockThreads ? (kWave << QL) : kMaxBlockThreads,
                             step_waves(K, C, QL, SCALAR, ROWS, Rhs::R, RAG))
void step_kernel_split(const double *__restrict__ table, int64_t table_elems, CyclicQ cq,
                       SweepGeom g, Rhs rhs, int64_t steps, StepStats st, const double *in,
                       double *out)
{
    constexpr bool ONE = SCALAR || ROWS == 1;   // one chunk per wave
    static_assert(RAG == 0 || ONE, "any number of waves: one chunk each");
    using Src = typename std::conditional<SCALAR, FromScalar<double>, FromLds<double>>::type;
    constexpr int R = Rhs::R;
    constexpr bool FULL = RAG != kRagTail;
    extern __shared__ double smem_d[];
    const int64_t tl = SCALAR ? 0 : table_elems;
    double *xch = smem_d + tl;                              // chunk_solve phases
    double *xd = xch + split_exchange_len(K, QL);              // [2R][P*S]: rows 0, C-1, 1, C-2, 2, C-3
    double *xs = xd + ((2LL * R * kWave) << QL);            // [P*S]: sums of squares
    typename Src::ptr tab;
    if constexpr (SCALAR) {
        tab = (typename Src::ptr)table;
    } else {
        stage_table(smem_d, table, table_elems);
        __syncthreads();
        tab = smem_d;
    }

    // ONE: P == Q (the host checks log2P == QL), so the geometry is known
    // at compile time: S = 64, one chunk per wave
    LaneGeom lg = lane_geom(ONE ? QL : ROWS > 0 ? QL + ROWS / 2 : g.log2P, QL);
    if constexpr (RAG != 0) {
        lg.P = g.waves;
        lg.S = kWave;
        lg.W = 1;
        lg.sl = threadIdx.x % kWave;
        lg.j0 = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    }
    if constexpr (ONE) lg.j = lg.j0;   // the wave's chunk
    const int row0 = lg.j * C;
    // kRagTail: rows of the system from this chunk on; whether the wave's rows
    // are all real, and its stencil's too
    const int nrow = g.n - row0;
    const bool all_real = FULL || nrow >= C;
    double *xe = xs + (STATS ? (kWave << QL) : 0);          // kRagTail: rows n-1 .. n-R
    const bool has_left = lg.j > 0, has_right = lg.j < lg.P - 1;
    const int PS = lg.P * lg.S;
    const int me = lg.j * lg.S + lg.sl;
    const int lft = (has_left ? lg.j - 1 : lg.j) * lg.S + lg.sl;
    const int rgt = (has_right ? lg.j + 1 : lg.j) * lg.S + lg.sl;
    const int first = lg.sl, last = (lg.P - 1) * lg.S + lg.sl;
    // STATS launches are persistent unless forced (the mapping code costs the
    // statistic kernel its third wave per SIMD); the persistent mapping also
    // serves a forced one-per-group grid
    GroupRange gr;
    if constexpr (RAG != 0)   // one group per workgroup, whatever its waves; no more than that
        gr = GroupRange{blockIdx.x, blockIdx.x < g.groups ? blockIdx.x + int64_t(1) : 0, 1, 1, 0};
    else
        gr = group_range(g.groups, QL, STATS ? 0 : g.linear);

    for (int64_t blk = gr.first; blk < gr.end; blk += gr.stride) {
        const int64_t grp = begin_block(gr, blk, g.lockstep);
        if (grp >= g.groups) continue;
        const int64_t k = grp * lg.S + lg.sl;
        const bool kval = k < g.m;
        double c[C];
        if (all_real)
            load_chunk<double, C, true>(c, in, row0, kval ? k : g.m - 1, g.ld, g.n);
        else
            load_chunk<double, C, false>(c, in, row0, kval ? k : g.m - 1, g.ld, g.n);
        const typename Rhs::State ls = rhs.lane_state(kval ? k : g.m - 1, row0);

        for (int64_t step = 0; step < steps; ++step) {
            xd[me] = c[0];
            xd[PS + me] = c[C - 1];
            if constexpr (R >= 2) {
                xd[2 * PS + me] = c[1];
                xd[3 * PS + me] = c[C - 2];
            }
            if constexpr (R >= 3) {
                xd[4 * PS + me] = c[2];
                xd[5 * PS + me] = c[C - 3];
            }
            if constexpr (!FULL) {
#pragma unroll
                for (int d = 1; d <= R; ++d)
                    if (nrow >= d && nrow - d < C) {
                        double x = 0.0;
                        row_at<false, 0, C>(c, opaque_u(nrow - d), x);
                        xe[(d - 1) * kWave + lg.sl] = x;
                    }
            }
            __syncthreads();
            Halo h = {};
            h.l1 = has_left ? xd[PS + lft] : 0.0;
            h.r1 = has_right ? xd[rgt] : 0.0;
            h.e0 = xd[first];
            h.en1 = xd[PS + last];
            if constexpr (R >= 2) {
                h.l2 = has_left ? xd[3 * PS + lft] : 0.0;
                h.r2 = has_right ? xd[2 * PS + rgt] : 0.0;
                h.e1 = xd[2 * PS + first];
                h.en2 = xd[3 * PS + last];
            }
            if constexpr (R >= 3) {
                h.l3 = has_left ? xd[5 * PS + lft] : 0.0;
                h.r3 = has_right ? xd[4 * PS + rgt] : 0.0;
                h.e2 = xd[4 * PS + first];
                h.en3 = xd[5 * PS + last];
            }
            if constexpr (!FULL) {
                h.en1 = xe[lg.sl];
                if constexpr (R >= 2) h.en2 = xe[kWave + lg.sl];
                if constexpr (R >= 3) h.en3 = xe[2 * kWave + lg.sl];
            }
            if constexpr (!FULL && CYC) {
                // rows 0 .. R-1 after row n-1, in the chunk's padding or its
                // halo: the stencil needs no wrap terms there, and what it
                // leaves in the padding meets zero coefficients
                double e[3] = {h.e0, h.e1, h.e2};
#pragma unroll
                for (int d = 0; d < R; ++d) {
                    const int t = opaque_u(nrow + d);
                    if (t < C) row_at<true, 0, C>(c, t, e[d]);
                    h.r1 = t == C ? e[d] : h.r1;
                    h.r2 = t == C + 1 ? e[d] : h.r2;
                    h.r3 = t == C + 2 ? e[d] : h.r3;
                }
            }
            rhs.template operator()<C, true>(c, h, lg.j, FULL && !has_right, C, ls);
            __builtin_amdgcn_sched_barrier(0);
            chunk_solve<double, K, C, CYC, FULL, true, Src, (ROWS > 0), (SCALAR && QL < 2 && RAG == 0 ? 1 << QL : ROWS > 0 && K == 1 ? 8 : 4)>(
                c, tab, lg, g.n, cq, xch);
            if (STATS && (step + 1) % st.every == 0) {
                // chunks of a system through LDS, summed in chunk order, by
                // wave 0 (it holds chunk 0: lanes 0 .. S-1 are the group)
                xs[me] = chunk_sum_sq<C>(c);
                __syncthreads();
                if (threadIdx.x < kWave) {
                    double tot = 0.0;
                    for (int i = 0; i < lg.P; ++i) tot += xs[i * lg.S + lg.sl];
                    const double msq = tot * st.inv_n;   // l - 1, as above
                    const double ell = kval ? msq / (1.0 - msq) : 0.0;
                    const double sum = block_sum(ell, lg.S);
                    if (threadIdx.x == 0)
                        st.partial[grp * st.samples + (step + 1) / st.every - 1] = sum;
                }
            }
            if constexpr (TRAJ) {
                if (kval && all_real)
                    store_chunk<double, C, true>(c, out + step * st.traj_stride, row0, k, g.ld, g.n);
                else if (kval)
                    store_chunk<double, C, false>(c, out + step * st.traj_stride, row0, k, g.ld, g.n);
            }
        }
        if constexpr (!TRAJ) {
            if (kval && all_real)
                store_chunk<double, C, true>(c, out, row0, k, g.ld, g.n);
            else if (kval)
                store_chunk<double, C, false>(c, out, row0, k, g.ld, g.n);
        }
    }
}

// LDS bytes of the split kernel beyond the staged table: the chunk_solve
// exchange, 2R rows per (chunk, slot), for the statistic one sum of squares
// per (chunk, slot) and, with any number of waves, R rows per slot.
constexpr size_t split_step_lds(int K, int QL, int R, bool stats, bool rag = false)
{
    return (size_t)(split_exchange_len(K, QL) + ((2LL * R * kWave) << QL) + (stats ? kWave << QL : 0) +
                    (rag ? R * kWave : 0)) *
           sizeof(double);
}

// Launch `steps` fused steps.  `scalar` selects the kernels with one chunk
// per wave (on g.waves waves, or on 2^log2Q == 2^log2P), otherwise
// g.log2Q > 0 the split kernel (full decomposition, log2Q <= 3) with the table
// in LDS, else the LDS kernel with one wave per group.  The split kernel takes
// its coefficients by row broadcast in groups of 16 64-row chunks and of 32
// chunks, by plain LDS reads in the others: 16 32-row chunks (n = 512 in small
// batches) fit the broadcast too, which has not been measured there.  The grid of the
// kernels with one chunk per wave follows g.linear (one that stages a table
// reads it from L2 and still gains: penta n = 512, m = 2^17, two steps per
// launch 171 vs 149 us a step); the other LDS kernels stage the table once per
// workgroup and stay persistent unless tuning grid_linear asks otherwise.
// TRAJ: every step's state, see step_kernel.
template <class Rhs, int K, bool CYC, bool STATS = false, bool TRAJ = false>
hipError_t launch_stepper(const double *table, int64_t table_elems, const CyclicQ &q,
                          const SweepGeom &g, bool scalar, const Rhs &rhs, int64_t steps,
                          const double *in, double *out, hipStream_t s,
                          StepStats st = StepStats{})
{
    if (scalar) {
        // one chunk per wave: 16-, 32- or 64-row chunks tiling n into 1, 2, 4
        // or 8, or (g.waves) 32- or 64-row chunks into any number up to 8
        const int waves = g.waves > 0 ? g.waves : 1 << g.log2Q;
        const int64_t rows = (int64_t)waves * g.C;
        const bool tail = rows != g.n;
        if (waves > 8 || rows < g.n || rows - g.C >= g.n || (g.waves == 0 && (tail || g.log2P != g.log2Q)))
            return hipErrorInvalidValue;
        const bool by_rows = chunk_by_rows(K, g.C, waves, Rhs::R, !tail);
        const bool linear = g.waves > 0 || g.linear;
        // QL: log2 of the waves, for any number 3 by rows and 2 (up to 3
        // waves) with scalar coefficients.  A scalar chunk with padding takes
        // 130 to 230 VGPRs at 64 rows: two waves per SIMD (three, with
        // spills: tri n = 100, m = 2^17 11.1 us a step against 9.9)
#define BB_ONE(CC, QQ, SC, RR)                                                                          \
        return launch_grid_mode(step_kernel_split<Rhs, K, CYC, CC, QQ, SC, STATS, TRAJ, SC ? 0 : 1, RR>,\
                                split_step_lds(K, QQ, Rhs::R, STATS, RR != 0) +                         \
                                    (SC ? 0 : (size_t)table_elems * sizeof(double)),                    \
                                g.groups, waves, linear, s, table, table_elems, q, g, rhs, steps, st, in, out)
        if (by_rows) {
            if (g.waves > 0) {
                if (g.C == 64 && tail) BB_ONE(64, 3, false, kRagTail);
                if (g.C == 64) BB_ONE(64, 3, false, kRagFull);
                if (tail) BB_ONE(32, 3, false, kRagTail);
                BB_ONE(32, 3, false, kRagFull);
            }
            if (g.C == 64 && g.log2Q == 3) BB_ONE(64, 3, false, 0);
            if constexpr (chunk_by_rows(K, 64, 4, Rhs::R, true))
                if (g.C == 64) BB_ONE(64, 2, false, 0);
            if (g.log2Q == 3) BB_ONE(32, 3, false, 0);
            BB_ONE(32, 2, false, 0);
        }
        if (g.waves > 0) {
            if (waves > 3) return hipErrorInvalidValue;
            if (g.C == 64 && tail) BB_ONE(64, 2, true, kRagTail);
            if (g.C == 64) BB_ONE(64, 2, true, kRagFull);
            if (g.C == 32 && tail) BB_ONE(32, 2, true, kRagTail);
            return hipErrorInvalidValue;
        }
        switch (g.C) {
        case 16:
            if (g.log2Q == 3) BB_ONE(16, 3, true, 0);
            if (g.log2Q == 2) BB_ONE(16, 2, true, 0);
            if (g.log2Q == 1) BB_ONE(16, 1, true, 0);
            BB_ONE(16, 0, true, 0);
        case 32:
            if (g.log2Q == 1) BB_ONE(32, 1, true, 0);
            BB_ONE(32, 0, true, 0);
        case 64:
            if constexpr (!chunk_by_rows(K, 64, 4, Rhs::R, true))
                if (g.log2Q == 2) BB_ONE(64, 2, true, 0);
            if (g.log2Q == 1) BB_ONE(64, 1, true, 0);
            BB_ONE(64, 0, true, 0);
        default: return hipErrorInvalidValue;
        }
#undef BB_ONE
    }
    if (g.log2Q > 0) {
        // LDS table, group split over 2^log2Q waves: 32- and 64-row chunks
        if (g.log2Q > 3 || g.log2Q > g.log2P || !is_full(g)) return hipErrorInvalidValue;
        const size_t xl = (size_t)table_elems * sizeof(double) + split_step_lds(K, g.log2Q, Rhs::R, STATS);
#define BB_SPLIT(CC)                                                                                     \
        case CC:                                                                                         \
            if (CC == 64 && g.log2Q == 2 && g.log2P == 4)                                                \
                return launch_grid_split(step_kernel_split<Rhs, K, CYC, CC, 2, false, STATS, TRAJ, 4>, xl, g.groups, 4, s, table, table_elems, q, g, rhs, steps, st, in, out); \
            if (CC == 64 && g.log2Q == 3 && g.log2P == 4)                                                \
                return launch_grid_split(step_kernel_split<Rhs, K, CYC, CC, 3, false, STATS, TRAJ, 2>, xl, g.groups, 8, s, table, table_elems, q, g, rhs, steps, st, in, out); \
            if (g.log2Q == 3 && g.log2P == 5)                                                            \
                return launch_grid_split(step_kernel_split<Rhs, K, CYC, CC, 3, false, STATS, TRAJ, 4>, xl, g.groups, 8, s, table, table_elems, q, g, rhs, steps, st, in, out); \
            switch (g.log2Q) {                                                                           \
            case 1: return launch_grid_split(step_kernel_split<Rhs, K, CYC, CC, 1, false, STATS, TRAJ>, xl, g.groups, 2, s, table, table_elems, q, g, rhs, steps, st, in, out); \
            case 2: return launch_grid_split(step_kernel_split<Rhs, K, CYC, CC, 2, false, STATS, TRAJ>, xl, g.groups, 4, s, table, table_elems, q, g, rhs, steps, st, in, out); \
            default: return launch_grid_split(step_kernel_split<Rhs, K, CYC, CC, 3, false, STATS, TRAJ>, xl, g.groups, 8, s, table, table_elems, q, g, rhs, steps, st, in, out); \
            }
        switch (g.C) {
            BB_SPLIT(32)
            BB_SPLIT(64)
        default: return hipErrorInvalidValue;
        }
#undef BB_SPLIT
    }
    const size_t lds = (size_t)table_elems * sizeof(double);
    if constexpr (K == 1 && CYC && TRAJ)
        if (g.C == 64 && g.log2P >= 5 && !is_full(g))   // step_rows_first
            return launch_grid(step_kernel<Rhs, K, CYC, 64, false, STATS, TRAJ, true>, lds, g.groups, s,
                               table, table_elems, q, g, rhs, steps, st, in, out);
#define BB_STEP(CC)                                                                            \
    case CC:                                                                                   \
        return is_full(g) ? launch_grid(step_kernel<Rhs, K, CYC, CC, true, STATS, TRAJ>, lds, g.groups, s,   \
                                        table, table_elems, q, g, rhs, steps, st, in, out)      \
                          : launch_grid(step_kernel<Rhs, K, CYC, CC, false, STATS, TRAJ>, lds, g.groups, s,  \
                                        table, table_elems, q, g, rhs, steps, st, in, out);
    switch (g.C) {
        BB_STEP(4)
        BB_STEP(8)
        BB_STEP(16)
        BB_STEP(32)
        BB_STEP(64)
    default: return hipErrorInvalidValue;
    }
#undef BB_STEP
}

}  // namespace
}  // namespace bb
