// sweep_core.h -- device building blocks shared by the gfx950 kernels of
// libbandbatch (sweep.hip, refine.hip, ch.hip): the per-lane chunk solve of a
// banded LU with one shared LHS, the lane/workgroup geometry, coefficient
// table sources, chunk loads and stores, and the persistent-grid launcher.
//
// Forward elimination + back substitution of the Thomas algorithm (Section
// 3.1; Appendix A batched sweep) and of the pentadiagonal LR solve (Section
// 4.1; Appendix B), on right-hand sides interleaved with the batch index
// fastest (Section 2).  The decomposition of a system over P lanes, the
// coefficient table and its LDS layout are described in internal.h.
//
// Per lane: load the C rows of its chunk (one coalesced wave-wide load per
// row), run the two recurrences in registers with the chunk-boundary scans,
// apply the periodic correction if any, store once.  HBM traffic is one read
// of the right-hand side and one write of the solution; coefficients come
// from LDS (staged once per workgroup) or through the scalar cache.
#pragma once

#include <type_traits>

#include "internal.h"
#include "row_bcast.h"

namespace bb {
namespace {

template <typename T>
__device__ __forceinline__ T shfl(T v, int src)
{
    return __shfl(v, src, kWave);
}

// Opaque copies of loop-invariant values.  The persistent loops below would
// otherwise let the compiler hoist every per-row LDS coefficient read and
// every per-row address offset out of the loop and keep them all live in
// registers; re-reading them each iteration is what the design wants.
__device__ __forceinline__ int opaque_v(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}

__device__ __forceinline__ int64_t opaque_s(int64_t x)
{
    asm volatile("" : "+s"(x));
    return x;
}

__device__ __forceinline__ int opaque_u(int x)   // wave-uniform (SGPR) copy
{
    asm volatile("" : "+s"(x));
    return x;
}

// Where a kernel reads its coefficient table: from LDS, staged once per
// workgroup (the lanes of a wave work on different chunks), or -- when every
// lane of a wave works on the same chunk -- straight from the global table
// through the scalar cache, the coefficient of each row arriving in SGPRs as
// an operand of the lanes' FMAs.  base() re-derives the pointer from a value
// the compiler cannot see through, so coefficient reads are not hoisted out
// of the persistent loop.
template <typename T>
struct FromLds {
    using ptr = const T *;
    __device__ static ptr base(ptr p) { return p + opaque_v(0); }
};

template <typename T>
struct FromScalar {
    typedef const T __attribute__((address_space(4))) elem;   // constant address space
    using ptr = elem *;
    __device__ static ptr base(ptr p) { return p + opaque_u(0); }
};

// A branch the compiler cannot fold (always taken, on a uniform value it
// cannot see).  Each pass runs in blocks of kFenceRows rows, each block inside
// such a branch: a separate basic block, so the coefficient reads of one block
// are not hoisted above the work of the previous one and only a few rows of
// coefficients are live at a time.
constexpr int kFenceRows = 8;
__device__ __forceinline__ bool opaque_true()
{
    int x = 1;
    asm volatile("" : "+s"(x));
    return x != 0;
}

// body(t) for t = 0 .. C-1 (rows_up) or C-1 .. 0 (rows_down), fully
// unrolled, in fenced blocks of kFenceRows rows.
template <int C, typename F>
__device__ __forceinline__ void rows_up(F &&body)
{
    constexpr int B = C < kFenceRows ? C : kFenceRows;
#pragma unroll
    for (int t0 = 0; t0 < C; t0 += B) {
        if (opaque_true()) {
#pragma unroll
            for (int tt = 0; tt < B; ++tt) body(t0 + tt);
        }
    }
}

template <int C, typename F>
__device__ __forceinline__ void rows_down(F &&body)
{
    constexpr int B = C < kFenceRows ? C : kFenceRows;
#pragma unroll
    for (int t0 = C - B; t0 >= 0; t0 -= B) {
        if (opaque_true()) {
#pragma unroll
            for (int tt = B - 1; tt >= 0; --tt) body(t0 + tt);
        }
    }
}

// runtime-indexed read of a register array without spilling it: C selects
template <typename T, int C>
__device__ __forceinline__ T pick(const T (&v)[C], int t)
{
    T r = T(0);
#pragma unroll
    for (int q = 0; q < C; ++q) r = (q == t) ? v[q] : r;
    return r;
}

// Where this lane sits: chunk j (of P) of system slot sl (of S) in its group;
// its wave holds chunks j0 .. j0 + W - 1 (uniform).
struct LaneGeom {
    int j, sl, S, P, j0, W;
};

// This lane's view of a coefficient table (layout in internal.h); Ptr is the
// pointer type of the table's source (LDS or scalar).
template <typename Ptr>
struct LaneTable {
    Ptr wE1, wE2, wS1, wS2;   // boundary-state weights (pass 1)
    Ptr s, l1, l2;            // forward recurrence (pass 2), l stored negated
    Ptr u1, u2;               // backward recurrence (pass 3), stored negated
    Ptr z0, z1;               // periodic correction, stored negated
    Ptr Mf, Mb, G;            // per-chunk KxK matrices
};

template <typename T, int K, int C, bool CYC, typename Ptr>
__device__ __forceinline__ LaneTable<Ptr> lane_table(Ptr tab, int P, int j)
{
    const int L = P * (C + 1);
    const int off = j * (C + 1);
    LaneTable<Ptr> tb;
    int q = 0;
    tb.wE1 = tab + (q++) * L + off;
    tb.wE2 = (K == 2) ? tab + (q++) * L + off : nullptr;
    tb.wS1 = tab + (q++) * L + off;
    tb.wS2 = (K == 2) ? tab + (q++) * L + off : nullptr;
    tb.s = tab + (q++) * L + off;
    tb.l1 = tab + (q++) * L + off;
    tb.l2 = (K == 2) ? tab + (q++) * L + off : nullptr;
    tb.u1 = tab + (q++) * L + off;
    tb.u2 = (K == 2) ? tab + (q++) * L + off : nullptr;
    tb.z0 = CYC ? tab + (q++) * L + off : nullptr;
    tb.z1 = (CYC && K == 2) ? tab + (q++) * L + off : nullptr;
    tb.Mf = tab + q * L;
    tb.Mb = tb.Mf + P * K * K;
    tb.G = tb.Mb + P * K * K;
    return tb;
}

// Gather rows 0, 1, n-2, n-1 of the system this lane works on (every lane of
// the system gets the same four values).  Row n-1 / n-2 sit at a compile-time
// position when the chunks tile n exactly, else they are picked at run time.
template <typename T, int K, int C>
__device__ __forceinline__ void gather_ends(const T (&v)[C], const LaneGeom &lg, int n, int exact,
                                            T &r0, T &r1, T &rn2, T &rn1)
{
    r0 = shfl(v[0], lg.sl);
    r1 = (K == 2) ? shfl(v[1], lg.sl) : T(0);
    if (exact) {
        const int src = (n / C - 1) * lg.S + lg.sl;
        rn1 = shfl(v[C - 1], src);
        rn2 = (K == 2) ? shfl(v[C - 2], src) : T(0);
    } else {
        rn1 = shfl(pick(v, (n - 1) % C), ((n - 1) / C) * lg.S + lg.sl);
        rn2 = (K == 2) ? shfl(pick(v, (n - 2) % C), ((n - 2) / C) * lg.S + lg.sl) : T(0);
    }
}

// y <- M y + e for a KxK matrix M (row-major) and K-vectors
template <typename T, int K, typename Ptr>
__device__ __forceinline__ void affine(Ptr M, T &y1, T &y2, T e1, T e2)
{
    if constexpr (K == 1) {
        y1 = fma(M[0], y1, e1);
    } else {
        const T n1 = fma(M[1], y2, fma(M[0], y1, e1));
        const T n2 = fma(M[3], y2, fma(M[2], y1, e2));
        y1 = n1;
        y2 = n2;
    }
}

// s = Q (r0, r1, rn2, rn1): the periodic correction scalars, with every
// product-sum written as an explicit fma chain so the rounding does not
// depend on how the compiler contracts a particular kernel.
template <typename T, int K>
__device__ __forceinline__ void correction_scalars(const CyclicQ &cq, T r0, T r1, T rn2, T rn1,
                                                   T &c0, T &c1)
{
    if constexpr (K == 1) {
        c0 = fma(T(cq.q[0][1]), rn1, T(cq.q[0][0]) * r0);
    } else {
        c0 = fma(T(cq.q[0][3]), rn1, fma(T(cq.q[0][2]), rn2, fma(T(cq.q[0][1]), r1, T(cq.q[0][0]) * r0)));
        c1 = fma(T(cq.q[1][3]), rn1, fma(T(cq.q[1][2]), rn2, fma(T(cq.q[1][1]), r1, T(cq.q[1][0]) * r0)));
    }
}

// Matrices of the 16 chunks from distance d0 along a scan, lane l of a row:
// chunk c0 + l.  With fewer than 16 chunks the other lanes read past or
// before them, inside the workgroup's LDS, and their values are not used.
template <typename T, int K, bool UP>
__device__ __forceinline__ void row_mats(const T *lds_mats, const LaneGeom &lg, int d0, T (&m)[K * K])
{
    const int c0 = UP ? d0 : lg.P < 16 ? lg.P - 8 : lg.P - 16 - d0;
    const int lane = threadIdx.x % kRowLanes;
#pragma unroll
    for (int q = 0; q < K * K; ++q) m[q] = lds_mats[(c0 + lane) * K * K + q];
}

// The scans of a split group.  Every lane walks the other chunks' boundary
// states in the exchange area xa (component c of chunk i at
// xa[c*P*S + i*S + slot]): state i = e_i + M_i state_{i-1} over the chunks
// before (UP) or after its own, taking the state that enters its chunk.  The
// chain's latency is what they cost, so everything four steps need is loaded
// before them: the boundary states, and the chunk matrices, which are the
// same for every lane -- held by the lanes of a row and taken by row
// broadcast (ROWS), else read from LDS or through the scalar cache like the
// coefficients.  With a load inside each
// step the two scans took 6000 of the 13400 clocks of a step of one group at
// 16 chunks.  The steps past the last chunk a wave needs run on clamped
// loads and are not taken.
// ENDS (periodic): every wave walks the first `steps` chunks of the chain and
// also takes the state that leaves the last of them, (y1, y2).
// BL: steps per block.
template <typename T, int K, bool ROWS, bool UP, bool ENDS, int BL, typename MP>
__device__ __forceinline__ void group_scan(const T *xa, MP mats, const LaneGeom &lg, int steps,
                                           T &h1, T &h2, T &y1, T &y2)
{
    constexpr int KK = K * K;
    static_assert(!ROWS || BL == 4 || (K == 1 && BL == 8), "steps of the row-broadcast chain");
    const int PS = lg.P * lg.S;
    // chunk at distance d along the chain: d, or P-1-d
    const int mine = UP ? lg.j : lg.P - 1 - lg.j;
    const int near = UP ? lg.j0 : lg.P - lg.j0 - lg.W;   // the wave's nearest chunk
    const int far = near + lg.W - 1;                     // ... and its farthest
    const int lim = ENDS && steps - 1 > far ? steps - 1 : far;   // last block runs to here
    T a1 = T(0), a2 = T(0);
    h1 = h2 = T(0);
    auto chunk_at = [&](int d) { return UP ? d : lg.P - 1 - d; };
    auto block = [&](auto lane0, int d0, const T (&m)[ROWS ? KK : BL * KK]) __attribute__((always_inline)) {
        T e[BL], g[BL];
#pragma unroll
        for (int b = 0; b < BL; ++b) {
            const int i = chunk_at(d0 + b < lg.P ? d0 + b : lg.P - 1);
            e[b] = xa[i * lg.S + lg.sl];
            g[b] = K == 2 ? xa[PS + i * lg.S + lg.sl] : T(0);
        }
        const T b1 = a1, b2 = a2;
        if constexpr (ROWS) {
            // four steps at a time; lanes hold the matrices by chunk number, so
            // a block going down the chunks runs over its lanes from the top
#pragma unroll
            for (int b0 = 0; b0 < BL; b0 += 4) {
                T e4[4], g4[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    e4[UP ? b : 3 - b] = e[b0 + b];
                    g4[UP ? b : 3 - b] = g[b0 + b];
                }
                constexpr int L0 = decltype(lane0)::value;
                if (b0 == 0)
                    chain4<K, UP, L0>(e4, g4, m, a1, a2);
                else
                    chain4<K, UP, UP ? (L0 + 4) % 16 : (L0 + 12) % 16>(e4, g4, m, a1, a2);
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    e[b0 + b] = e4[UP ? b : 3 - b];
                    g[b0 + b] = g4[UP ? b : 3 - b];
                }
                a1 = e[b0 + 3];
                a2 = g[b0 + 3];
            }
        } else {
#pragma unroll
            for (int b = 0; b < BL; ++b) {
                affine<T, K>(m + b * KK, a1, a2, e[b], g[b]);
                e[b] = a1;
                g[b] = a2;
            }
        }
        a1 = e[BL - 1];
        a2 = g[BL - 1];
        // the state entering the lane's chunk: before step `mine`
        if (near < d0 + BL && far >= d0) {
#pragma unroll
            for (int b = 0; b < BL; ++b) {
                const bool me = mine == d0 + b;
                h1 = me ? (b == 0 ? b1 : e[b == 0 ? 0 : b - 1]) : h1;
                if constexpr (K == 2) h2 = me ? (b == 0 ? b2 : g[b == 0 ? 0 : b - 1]) : h2;
            }
        }
        if (ENDS && steps - 1 >= d0 && steps - 1 < d0 + BL) {
#pragma unroll
            for (int b = 0; b < BL; ++b) {
                y1 = steps - 1 == d0 + b ? e[b] : y1;
                if constexpr (K == 2) y2 = steps - 1 == d0 + b ? g[b] : y2;
            }
        }
    };
    if constexpr (ROWS) {
        for (int d0 = 0; d0 <= lim; d0 += 16) {
            T m[KK];
            row_mats<T, K, UP>(mats, lg, d0, m);
            // lanes of the block's chunks: from the row's low end going up,
            // from its high end going down (from lane 7 with fewer than 16
            // chunks)
            auto at = [&](auto i) {
                constexpr int o = decltype(i)::value;
                if (d0 + o > lim) return;
                if (!UP && lg.P < 16)
                    block(std::integral_constant<int, (o < 8 ? 4 - o : 0)>{}, d0 + o, m);
                else
                    block(std::integral_constant<int, UP ? o : 12 - o>{}, d0 + o, m);
            };
            at(std::integral_constant<int, 0>{});
            if constexpr (BL == 4) at(std::integral_constant<int, 4>{});
            at(std::integral_constant<int, 8>{});
            if constexpr (BL == 4) at(std::integral_constant<int, 12>{});
        }
    } else {
        for (int d0 = 0; d0 <= lim; d0 += BL) {
            T m[BL * KK];
#pragma unroll
            for (int b = 0; b < BL; ++b)
#pragma unroll
                for (int q = 0; q < KK; ++q)
                    m[b * KK + q] = mats[chunk_at(d0 + b < lg.P ? d0 + b : lg.P - 1) * KK + q];
            block(std::integral_constant<int, 0>{}, d0, m);
        }
    }
}

// Coefficient array q of this lane's chunk for the row-broadcast passes.
template <int C>
__device__ __forceinline__ const double *row_base(const double *tab, const LaneGeom &lg, int q)
{
    return tab + q * lg.P * (C + 1) + lg.j * (C + 1) + (int)(threadIdx.x % kRowLanes);
}

// x += z0 c0 (+ z1 c1) on this lane's chunk, row-broadcast coefficients
template <int K, int C>
__device__ __forceinline__ void rows_correct(double (&v)[C], const double *tab, const LaneGeom &lg,
                                             double c0, double c1)
{
    constexpr int qz = 4 * K + 1;
    const RowCoef<C> z0 = row_coef<C>(row_base<C>(tab, lg, qz));
    if constexpr (K == 1) {
        blocks8_up<C>([&](auto t) {
            constexpr int t_ = decltype(t)::value;
            rows8_correct<t_, C>(v, c0, z0.r[t_ / 16]);
        });
    } else {
        const RowCoef<C> z1 = row_coef<C>(row_base<C>(tab, lg, qz + 1));
        blocks8_up<C>([&](auto t) {
            constexpr int t_ = decltype(t)::value;
            rows8_correct<t_, C>(v, c0, c1, z0.r[t_ / 16], z1.r[t_ / 16]);
        });
    }
}

// Solve this lane's chunk in place: v holds the right-hand side rows on entry
// and the solution rows on exit.  All 64 lanes of the wave must call it
// together (the scans shuffle across the wave).
//
//   pass 1: the chunk's zero-history forward end state e and the zero-future
//           backward start state o of that forward solution, both linear in
//           the right-hand side: dot products with precomputed weights (no
//           dependency chain, nothing written);
//   scans:  history H_j (prefix over chunks, H_{i+1} = e_i + Mf_i H_i), then
//           S_j = o_j + G_j H_j and the future F_j (suffix, F_{i-1} = S_i + Mb_i F_i);
//   pass 2: forward recurrence from H_j, writing y;
//   pass 3: backward recurrence from F_j, writing x.
// Periodic: the correction scalars follow from the scans; a full
// decomposition (FULL) puts them into H_j and F_j, a ragged one adds the
// correction's rows in pass 3 (internal.h, build_sweep_table).
// Each pass re-derives its table pointers (LDS or scalar) from an opaque base
// so the compiler re-reads coefficients instead of keeping C of them live
// across passes.
//
// SPLIT: the group spans several waves of the workgroup; boundary states go
// through the exchange area xch (split_exchange_len elements) with workgroup
// barriers, so every wave of the workgroup must call it the same number of
// times.
// ROWS: the passes take their coefficients by row broadcast (row_bcast.h):
// double, table in LDS, S a multiple of 16 so that a 16-lane row works on one
// chunk.
// BL: steps per block of the group's scans; 0 (K = 1, full or not periodic): no
// blocks, each lane walks to its own chunk, one load and step at a time, and the periodic end
// states go round in a third phase of the exchange area, of 2 P S elements more
// (for kernels without the registers of a block's loads).
template <typename T, int K, int C, bool CYC, bool FULL, bool SPLIT = false,
          typename Src = FromLds<T>, bool ROWS = false, int BL = 4>
__device__ __forceinline__ void chunk_solve(T (&v)[C], typename Src::ptr tab, const LaneGeom &lg,
                                            int n, const CyclicQ &cq, T *xch = nullptr)
{
    static_assert(!ROWS || (std::is_same<T, double>::value && std::is_same<Src, FromLds<T>>::value &&
                            C % kRowLanes == 0),
                  "row-broadcast coefficients: double, LDS table, 16-row blocks");
    static_assert(!SPLIT || BL > 0 || (K == 1 && (FULL || !CYC) && !ROWS), "step-by-step scans");
    // array indices of the table (internal.h)
    constexpr int qE = 0, qW = K, qs = 2 * K, ql = 2 * K + 1, qu = 3 * K + 1;
    constexpr bool ZROWS = CYC && !FULL;   // the table has z arrays
    const int real = FULL ? lg.P : (n - 1) / C + 1;   // real chunks
    // the chunk matrices, for the scans of a split group
    const auto mats = tab + sweep_arrays(K, CYC, FULL) * lg.P * (C + 1);
    T e1 = T(0), e2 = T(0), o1 = T(0), o2 = T(0);
    if constexpr (ROWS) {
        const double *t0 = Src::base(tab);
        const RowCoef<C> we1 = row_coef<C>(row_base<C>(t0, lg, qE));
        const RowCoef<C> ws1 = row_coef<C>(row_base<C>(t0, lg, qW));
        if constexpr (K == 1) {
            blocks8_up<C>([&](auto t) {
                constexpr int t_ = decltype(t)::value;
                rows8_ends<t_, C>(v, e1, o1, we1.r[t_ / 16], ws1.r[t_ / 16]);
            });
        } else {
            const RowCoef<C> we2 = row_coef<C>(row_base<C>(t0, lg, qE + 1));
            const RowCoef<C> ws2 = row_coef<C>(row_base<C>(t0, lg, qW + 1));
            blocks8_up<C>([&](auto t) {
                constexpr int t_ = decltype(t)::value;
                rows8_ends<t_, C>(v, e1, o1, e2, o2, we1.r[t_ / 16], ws1.r[t_ / 16], we2.r[t_ / 16],
                                  ws2.r[t_ / 16]);
            });
        }
    } else {
        const auto tb = lane_table<T, K, C, ZROWS>(Src::base(tab), lg.P, lg.j);
        rows_up<C>([&](int t) {
            e1 = fma(tb.wE1[t], v[t], e1);
            o1 = fma(tb.wS1[t], v[t], o1);
            if constexpr (K == 2) {
                e2 = fma(tb.wE2[t], v[t], e2);
                o2 = fma(tb.wS2[t], v[t], o2);
            }
        });
    }
    __builtin_amdgcn_sched_barrier(0);
    // history of this chunk: H_j = true (y_{start-1}, y_{start-2})
    const auto tb = lane_table<T, K, C, ZROWS>(Src::base(tab), lg.P, lg.j);
    T h1 = T(0), h2 = T(0);
    // periodic: y_{n-1} and y_{n-2} of the last real chunk's forward pass, x_0 and x_1
    T y1e = T(0), y2e = T(0), x0e = T(0), x1e = T(0);
    // exchange area: structure of arrays of P*S entries, (chunk, slot) at
    // chunk*S + slot, so a wave's accesses are consecutive words
    const int me = lg.j * lg.S + lg.sl;
    const int PS = lg.P * lg.S;
    if constexpr (SPLIT) {
        T *xa = xch;   // [K][P*S]
        xa[me] = e1;
        if constexpr (K == 2) xa[PS + me] = e2;
        __syncthreads();
        if constexpr (BL == 0) {
            for (int i = 0; i < lg.j; ++i) h1 = fma(tb.Mf[i], h1, xa[i * lg.S + lg.sl]);
        } else {
            group_scan<T, K, ROWS, true, CYC, BL>(xa, mats, lg, real, h1, h2, y1e, y2e);
        }
    } else {
        for (int i = 0; i < lg.P; ++i) {
            const int src = i * lg.S + lg.sl;
            const T a1 = shfl(e1, src);
            const T a2 = (K == 2) ? shfl(e2, src) : T(0);
            if (i < lg.j) affine<T, K>(tb.Mf + i * K * K, h1, h2, a1, a2);
        }
    }
    // zero-future start state of the true forward solution of this chunk
    T s1 = o1, s2 = o2;
    {
        const auto Gm = tb.G + lg.j * K * K;
        if constexpr (K == 1) {
            s1 = fma(Gm[0], h1, o1);
        } else {
            s1 = fma(Gm[1], h2, fma(Gm[0], h1, o1));
            s2 = fma(Gm[3], h2, fma(Gm[2], h1, o2));
        }
    }
    // future of this chunk: F_j = true (x_{end+1}, x_{end+2})
    T f1 = T(0), f2 = T(0);
    if constexpr (SPLIT) {
        T *xb = xch + K * PS;   // [K][P*S]
        xb[me] = s1;
        if constexpr (K == 2) xb[PS + me] = s2;
        __syncthreads();
        if constexpr (BL == 0) {
            for (int i = lg.P - 1; i > lg.j; --i) f1 = fma(tb.Mb[i], f1, xb[i * lg.S + lg.sl]);
        } else {
            group_scan<T, K, ROWS, false, CYC, BL>(xb, mats + lg.P * K * K, lg, lg.P, f1, f2, x0e, x1e);
        }
    } else {
        for (int i = lg.P - 1; i >= 0; --i) {
            const int src = i * lg.S + lg.sl;
            const T a1 = shfl(s1, src);
            const T a2 = (K == 2) ? shfl(s2, src) : T(0);
            if (i > lg.j) affine<T, K>(tb.Mb + i * K * K, f1, f2, a1, a2);
        }
    }
    // periodic correction scalars c = Q (x_0, x_1, x_{n-2}, x_{n-1}) of the
    // solution without it (the last chunk's future is zero, so x_{n-1} =
    // y_{n-1} and x_{n-2} = y_{n-2} - u1 y_{n-1})
    T c0 = T(0), c1 = T(0);
    if constexpr (CYC) {
        if constexpr (SPLIT && BL == 0) {
            T *xc = xch + 2 * PS;   // [2][P*S]: every chunk's start and forward end state
            xc[me] = fma(tb.Mb[lg.j], f1, s1);
            xc[PS + me] = fma(tb.Mf[lg.j], h1, e1);
            __syncthreads();
            x0e = xc[lg.sl];
            y1e = xc[PS + (lg.P - 1) * lg.S + lg.sl];
        } else if constexpr (!SPLIT) {
            T g1 = f1, g2 = f2, y1 = h1, y2 = h2;
            affine<T, K>(tb.Mb + lg.j * K * K, g1, g2, s1, s2);
            affine<T, K>(tb.Mf + lg.j * K * K, y1, y2, e1, e2);
            const int last = (real - 1) * lg.S + lg.sl;
            x0e = shfl(g1, lg.sl);
            x1e = (K == 2) ? shfl(g2, lg.sl) : T(0);
            y1e = shfl(y1, last);
            y2e = (K == 2) ? shfl(y2, last) : T(0);
        }
        const T xn2 = (K == 2) ? fma(T(cq.u1_nm2), y1e, y2e) : T(0);
        correction_scalars<T, K>(cq, x0e, x1e, xn2, y1e, c0, c1);
        if constexpr (FULL) {
            const auto HZ = tb.Mf + (3 * lg.P + lg.j) * K * K, FZ = tb.Mf + (4 * lg.P + lg.j) * K * K;
            if constexpr (K == 1) {
                h1 = fma(HZ[0], c0, h1);
                f1 = fma(FZ[0], c0, f1);
            } else {
                h1 = fma(HZ[1], c1, fma(HZ[0], c0, h1));
                h2 = fma(HZ[3], c1, fma(HZ[2], c0, h2));
                f1 = fma(FZ[1], c1, fma(FZ[0], c0, f1));
                f2 = fma(FZ[3], c1, fma(FZ[2], c0, f2));
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // pass 2: forward recurrence from the true history
    if constexpr (ROWS) {
        const double *t0 = Src::base(tab);
        const RowCoef<C> cs = row_coef<C>(row_base<C>(t0, lg, qs));
        const RowCoef<C> l1 = row_coef<C>(row_base<C>(t0, lg, ql));
        if constexpr (K == 1) {
            blocks8_up<C>([&](auto t) {
                constexpr int t_ = decltype(t)::value;
                const double y1 = t_ == 0 ? h1 : v[t_ == 0 ? 0 : t_ - 1];
                rows8_forward<t_, C>(v, y1, cs.r[t_ / 16], l1.r[t_ / 16]);
            });
        } else {
            const RowCoef<C> l2 = row_coef<C>(row_base<C>(t0, lg, ql + 1));
            blocks8_up<C>([&](auto t) {
                constexpr int t_ = decltype(t)::value;
                const double y1 = t_ == 0 ? h1 : v[t_ == 0 ? 0 : t_ - 1];
                const double y2 = t_ == 0 ? h2 : v[t_ == 0 ? 0 : t_ - 2];
                rows8_forward<t_, C>(v, y1, y2, cs.r[t_ / 16], l1.r[t_ / 16], l2.r[t_ / 16]);
            });
        }
    } else {
        const auto tp = lane_table<T, K, C, ZROWS>(Src::base(tab), lg.P, lg.j);
        T y1 = h1, y2 = h2;
        rows_up<C>([&](int t) {
            T y = tp.s[t] * v[t];
            if constexpr (K == 2) y = fma(tp.l2[t], y2, y);
            y = fma(tp.l1[t], y1, y);
            v[t] = y;
            y2 = y1;
            y1 = y;
        });
    }
    __builtin_amdgcn_sched_barrier(0);
    // pass 3: backward recurrence from the true future (+ correction rows, ragged periodic)
    if constexpr (ROWS) {
        const double *t0 = Src::base(tab);
        const RowCoef<C> u1 = row_coef<C>(row_base<C>(t0, lg, qu));
        if constexpr (K == 1) {
            blocks8_down<C>([&](auto t) {
                constexpr int t_ = decltype(t)::value;
                const double x1 = t_ + 8 == C ? f1 : v[t_ + 8 == C ? 0 : t_ + 8];
                rows8_backward<t_, C>(v, x1, u1.r[t_ / 16]);
            });
        } else {
            const RowCoef<C> u2 = row_coef<C>(row_base<C>(t0, lg, qu + 1));
            blocks8_down<C>([&](auto t) {
                constexpr int t_ = decltype(t)::value;
                const double x1 = t_ + 8 == C ? f1 : v[t_ + 8 == C ? 0 : t_ + 8];
                const double x2 = t_ + 8 == C ? f2 : v[t_ + 8 == C ? 0 : t_ + 9];
                rows8_backward<t_, C>(v, x1, x2, u1.r[t_ / 16], u2.r[t_ / 16]);
            });
        }
        if constexpr (ZROWS) rows_correct<K, C>(v, t0, lg, c0, c1);
    } else {
        const auto tp = lane_table<T, K, C, ZROWS>(Src::base(tab), lg.P, lg.j);
        T x1 = f1, x2 = f2;
        rows_down<C>([&](int t) {
            T x = v[t];
            if constexpr (K == 2) x = fma(tp.u2[t], x2, x);
            x = fma(tp.u1[t], x1, x);
            x2 = x1;
            x1 = x;
            if constexpr (ZROWS) {
                x = fma(tp.z0[t], c0, x);
                if constexpr (K == 2) x = fma(tp.z1[t], c1, x);
            }
            v[t] = x;
        });
    }
}

// Workgroup -> group-of-systems mapping.  A workgroup of W waves works on
// W consecutive groups at a time (one per wave); workgroups are dealt
// round-robin to the 8 XCDs, and each XCD gets a contiguous range of these
// blocks of groups, so segments that share 128 B lines are read inside one L2.
// The trip count of the loop over blocks is uniform across the workgroup, so a
// workgroup barrier inside it is reached by every wave the same number of times.
struct GroupRange {
    int64_t first, end, stride;   // blocks of W groups
    int W, wave;
};

__device__ __forceinline__ GroupRange group_range(int64_t groups, int log2Q = 0, int linear = 0)
{
    constexpr int kXcd = 8;
    GroupRange r;
    r.W = (blockDim.x / kWave) >> log2Q;     // groups per workgroup
    r.wave = (threadIdx.x / kWave) >> log2Q; // this wave's group in the workgroup
    const int64_t blocks = (groups + r.W - 1) / r.W;
    if (linear) {   // the host launched one workgroup per block of groups
        r.first = blockIdx.x;
        r.end = r.first < blocks ? r.first + 1 : r.first;
        r.stride = 1;
        return r;
    }
    const int xcd = blockIdx.x % kXcd;
    const int64_t per_xcd = (blocks + kXcd - 1) / kXcd;
    const int64_t base = (int64_t)xcd * per_xcd;
    r.first = base + blockIdx.x / kXcd;
    r.end = base + per_xcd < blocks ? base + per_xcd : blocks;
    r.stride = gridDim.x / kXcd;   // host launches a multiple of 8
    return r;
}

// Start of one iteration of the persistent loop.  With `lockstep`, the waves
// of a workgroup start their loads together, so the two halves of a 128 B
// line that two waves read (64 B segments) are requested close in time and
// the second request hits in L2 instead of refetching the line.
__device__ __forceinline__ int64_t begin_block(const GroupRange &r, int64_t b, int lockstep)
{
    if (lockstep) __syncthreads();
    return b * r.W + r.wave;
}

// Copy the shared table into LDS: four loads in flight per thread per round.
template <typename T>
__device__ __forceinline__ void stage_table(T *lds, const T *__restrict__ table, int64_t elems)
{
    const int64_t stride = blockDim.x;
    int64_t e = threadIdx.x;
    for (; e + 3 * stride < elems; e += 4 * stride) {
        const T a = table[e], b = table[e + stride], c = table[e + 2 * stride], d = table[e + 3 * stride];
        lds[e] = a;
        lds[e + stride] = b;
        lds[e + 2 * stride] = c;
        lds[e + 3 * stride] = d;
    }
    for (; e < elems; e += stride) lds[e] = table[e];
}

// Load the C rows of this lane's chunk; column k must be in bounds.
// FULL: every row of every chunk is a real row, no predicates at all.
// Ragged: the row pointer stops at row n-1 (in bounds) and rows past n read 0.
// The stride is laundered once per call so the C row offsets are recomputed
// here rather than hoisted out of the persistent loop and kept live.
// ALL (ragged): every load in flight before the first is looked at; otherwise
// each row is selected as it comes.
template <typename T, int C, bool FULL, bool ALL = true>
__device__ __forceinline__ void load_chunk(T (&v)[C], const T *base, int row0, int64_t k,
                                           int64_t ld, int n)
{
    ld = opaque_s(ld);
    if constexpr (FULL) {
        const T *p = base + (int64_t)row0 * ld + k;
#pragma unroll
        for (int t = 0; t < C; ++t) v[t] = p[(int64_t)t * ld];
    } else {
        const int nv = opaque_v(n - row0);   // rows of this chunk that are real
        const T *p = base + (int64_t)(row0 < n ? row0 : n - 1) * ld + k;
#pragma unroll
        for (int t = 0; t < C; ++t) {
            const T x = *p;
            v[t] = ALL || t < nv ? x : T(0);
            p += (t + 1 < nv) ? ld : 0;
        }
        if constexpr (ALL) {
            // left to itself the compiler may wait for each in turn
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < C; ++t) v[t] = t < nv ? v[t] : T(0);
        }
    }
}

// Store the chunk; the caller masks out lanes whose column is past m.  Ragged:
// the pointer stops at row n-1 and the rows past n rewrite row n-1 with its
// own value, so no store is predicated per row.
template <typename T, int C, bool FULL>
__device__ __forceinline__ void store_chunk(const T (&v)[C], T *base, int row0, int64_t k,
                                            int64_t ld, int n)
{
    ld = opaque_s(ld);
    if constexpr (FULL) {
        T *p = base + (int64_t)row0 * ld + k;
#pragma unroll
        for (int t = 0; t < C; ++t) p[(int64_t)t * ld] = v[t];
    } else if (row0 < n) {
        const int nv = opaque_v(n - row0);
        T *p = base + (int64_t)row0 * ld + k;
        T keep = v[0];
#pragma unroll
        for (int t = 0; t < C; ++t) {
            keep = t < nv ? v[t] : keep;
            *p = keep;
            p += (t + 1 < nv) ? ld : 0;
        }
    }
}

// store_chunk of value(t), computed row by row inside the fenced row blocks,
// so the values need not all be live at once.
template <int C, bool FULL, typename F>
__device__ __forceinline__ void store_chunk_fn(F &&value, double *base, int row0, int64_t k,
                                               int64_t ld, int n)
{
    ld = opaque_s(ld);
    if constexpr (FULL) {
        double *p = base + (int64_t)row0 * ld + k;
        rows_up<C>([&](int t) { p[(int64_t)t * ld] = value(t); });
    } else if (row0 < n) {
        const int nv = opaque_v(n - row0);
        double *p = base + (int64_t)row0 * ld + k;
        double keep = value(0);
        rows_up<C>([&](int t) {
            keep = t < nv ? value(t) : keep;
            *p = keep;
            p += (t + 1 < nv) ? ld : 0;
        });
    }
}

// Lane coordinates: a wave holds P/Q chunks of S = 64Q/P systems,
// lane = (chunk within the wave) * S + slot; wave q of a split group holds
// chunks q*P/Q .. (q+1)*P/Q - 1.
__device__ __forceinline__ LaneGeom lane_geom(int log2P, int log2Q = 0)
{
    LaneGeom lg;
    const int lw = log2P - log2Q;   // log2 of chunks per wave
    lg.P = 1 << log2P;
    lg.S = kWave >> lw;
    const int lane = threadIdx.x % kWave;
    const int q = (threadIdx.x / kWave) & ((1 << log2Q) - 1);
    lg.j = (q << lw) + (lane >> (6 - lw));
    lg.sl = lane & (lg.S - 1);
    lg.j0 = __builtin_amdgcn_readfirstlane(q << lw);
    lg.W = 1 << lw;
    return lg;
}

// ---------------------------------------------------------------- launch helpers
int cu_count()
{
    static int cached = 0;
    if (!cached) {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
            cus > 0)
            cached = cus;
        else
            return 256;
    }
    return cached;
}

// Workgroups of a kernel that fit a CU at once, asked of the runtime once per
// thread, device, kernel and launch shape (the questions took about 1 us of a
// 4 us call); a kernel that needs more than 64 KB of LDS is allowed it then.
struct ResidentKey {
    const void *kern = nullptr;
    size_t lds = 0;
    int threads = 0, dev = 0, blocks = 0;
};

inline hipError_t resident_blocks(const void *kern, int threads, size_t lds, int *blocks)
{
    constexpr int N = 64;   // direct-mapped, so bounded
    static thread_local ResidentKey cache[N];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    ResidentKey &c = cache[(((uintptr_t)kern >> 4) ^ (lds >> 3) ^ (uintptr_t)dev) % N];
    if (c.kern == kern && c.lds == lds && c.threads == threads && c.dev == dev) {
        *blocks = c.blocks;
        return hipSuccess;
    }
    if (lds > 65536) {
        // the CU's whole LDS: launches of one kernel differ in what they need
        e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
    }
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, kern, threads, lds);
    if (e != hipSuccess) return e;
    c.kern = kern;
    c.lds = lds;
    c.threads = threads;
    c.dev = dev;
    c.blocks = *blocks;
    return hipSuccess;
}

// Persistent-style launch: as many workgroups as can be resident at once
// (rounded to a multiple of the 8 XCDs), each looping over groups of systems.
// split_waves > 0: a split group of that many waves is the whole workgroup.
// Tuning grid_linear = 1: non-persistent grids for the kernels launched
// through launch_grid_split; the host sets SweepGeom::linear to match.
inline bool grid_linear() { return tuning(kTuneGridLinear) == 1; }

// linear: one workgroup per block of groups (the kernel's SweepGeom::linear
// must be set); otherwise a persistent grid of at most one wave of resident
// workgroups, each walking the blocks of its XCD's share (group_range).
template <typename... KArgs, typename... Args>
hipError_t launch_grid_mode(void (*kern)(KArgs...), size_t lds, int64_t groups, int split_waves,
                            bool linear, hipStream_t s, Args... args)
{
    // waves per workgroup: the workgroup is the unit that moves in step (see
    // begin_block); tuning waves_per_block (1, 2 or 4) overrides
    int waves_per_block = kBlockThreads / kWave;
    if (tuning(kTuneWavesPerBlock) > 0) waves_per_block = (int)tuning(kTuneWavesPerBlock);
    int groups_per_block = waves_per_block;
    if (split_waves > 0) {
        waves_per_block = split_waves;
        groups_per_block = 1;
    }
    const int threads = waves_per_block * kWave;
    int per_cu = 0;
    hipError_t e = resident_blocks((const void *)kern, threads, lds, &per_cu);
    if (e != hipSuccess) return e;
    if (per_cu < 1) return hipErrorInvalidConfiguration;
    int64_t need = (groups + groups_per_block - 1) / groups_per_block;
    int64_t cap = (int64_t)cu_count() * per_cu;
    int64_t blocks = need < cap ? need : cap;
    if (linear) blocks = need;
    blocks = ((blocks + 7) / 8) * 8;   // multiple of the XCD count, see group_range
    if (blocks < 8) blocks = 8;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(threads), lds, s, args...);
    return hipGetLastError();
}

template <typename... KArgs, typename... Args>
hipError_t launch_grid_split(void (*kern)(KArgs...), size_t lds, int64_t groups, int split_waves,
                             hipStream_t s, Args... args)
{
    return launch_grid_mode(kern, lds, groups, split_waves, grid_linear(), s, args...);
}

template <typename... KArgs, typename... Args>
hipError_t launch_grid(void (*kern)(KArgs...), size_t lds, int64_t groups, hipStream_t s,
                       Args... args)
{
    return launch_grid_split(kern, lds, groups, 0, s, args...);
}

bool is_full(const SweepGeom &g) { return ((int64_t)g.C << g.log2P) == g.n; }

}  // namespace
}  // namespace bb
