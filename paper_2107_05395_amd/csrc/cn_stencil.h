// cn_stencil.h -- the right-hand side of a Crank-Nicolson step as a policy of
// the fused stepper (stepper.h): periodic diffusion (Section 3 benchmark
// problem, K = 1) and periodic hyperdiffusion (Section 4 benchmark problem,
// K = 2), and their non-periodic forms.  cn_tri.hip and cn_penta.hip
// instantiate it.
#pragma once

#include "long_core.h"
#include "stepper.h"

namespace bb {
namespace {

// Eight rows of a full chunk's stencil, in place, rows in order.  A row's
// result takes its own register, so the rows after it have taken what they
// need of it before (two, four rows at a time); left to the compiler the rows
// of a chunk either sit in fenced blocks, each with a branch (64 tridiagonal
// rows: 1536 clocks, 911 without), or hold a second copy of the chunk.  The
// sums are the fma chains of StencilRhs.
// K = 1: s enters as w0 c_{-1} + w1 c_0 of the first row and leaves as that of
// the row after the eighth, r (old value).
#define BB_W1_4(SA, SB, c0, c1, c2, c3, c4)                                                        \
    "v_mul_f64 %[t1], %[w0], %[" c0 "]\n\tv_mul_f64 %[t2], %[w0], %[" c1 "]\n\t"                   \
    "v_mul_f64 %[t3], %[w0], %[" c2 "]\n\tv_mul_f64 %[" SB "], %[w0], %[" c3 "]\n\t"               \
    "v_fma_f64 %[t1], %[w1], %[" c1 "], %[t1]\n\tv_fma_f64 %[t2], %[w1], %[" c2 "], %[t2]\n\t"     \
    "v_fma_f64 %[t3], %[w1], %[" c3 "], %[t3]\n\tv_fma_f64 %[" SB "], %[w1], %[" c4 "], %[" SB "]\n\t" \
    "v_fma_f64 %[" c0 "], %[w2], %[" c1 "], %[" SA "]\n\t"                                         \
    "v_fma_f64 %[" c1 "], %[w2], %[" c2 "], %[t1]\n\t"                                             \
    "v_fma_f64 %[" c2 "], %[w2], %[" c3 "], %[t2]\n\t"                                             \
    "v_fma_f64 %[" c3 "], %[w2], %[" c4 "], %[t3]\n\t"

__device__ __forceinline__ void stencil_rows8(double *c, double r, double &s, const double (&w)[3])
{
    double sb, t1, t2, t3;
    asm(BB_W1_4("sa", "sb", "c0", "c1", "c2", "c3", "c4") BB_W1_4("sb", "sa", "c4", "c5", "c6", "c7", "r")
        : [c0] "+&v"(c[0]), [c1] "+&v"(c[1]), [c2] "+&v"(c[2]), [c3] "+&v"(c[3]), [c4] "+&v"(c[4]),
          [c5] "+&v"(c[5]), [c6] "+&v"(c[6]), [c7] "+&v"(c[7]), [sa] "+&v"(s), [sb] "=&v"(sb),
          [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3)
        : [r] "v"(r), [w0] "s"(w[0]), [w1] "s"(w[1]), [w2] "s"(w[2]));
}

// K = 2: (u, v) enter as w0 c_{-2} + w1 c_{-1} and w0 c_{-1}, the first terms
// of the first two rows, and leave as those of the two rows after the eighth;
// r0, r1: those rows (old values).
#define BB_W2_4(A, B, U, V, c0, c1, c2, c3, c4, c5)                                                \
    "v_mul_f64 %[t2], %[w0], %[" c0 "]\n\tv_mul_f64 %[t3], %[w0], %[" c1 "]\n\t"                   \
    "v_mul_f64 %[" U "], %[w0], %[" c2 "]\n\tv_fma_f64 %[" B "], %[w1], %[" c0 "], %[" B "]\n\t"   \
    "v_mul_f64 %[" V "], %[w0], %[" c3 "]\n\tv_fma_f64 %[" A "], %[w2], %[" c0 "], %[" A "]\n\t"   \
    "v_fma_f64 %[t2], %[w1], %[" c1 "], %[t2]\n\tv_fma_f64 %[t3], %[w1], %[" c2 "], %[t3]\n\t"     \
    "v_fma_f64 %[" U "], %[w1], %[" c3 "], %[" U "]\n\tv_fma_f64 %[" B "], %[w2], %[" c1 "], %[" B "]\n\t" \
    "v_fma_f64 %[" A "], %[w3], %[" c1 "], %[" A "]\n\t"                                           \
    "v_fma_f64 %[t2], %[w2], %[" c2 "], %[t2]\n\tv_fma_f64 %[t3], %[w2], %[" c3 "], %[t3]\n\t"     \
    "v_fma_f64 %[" B "], %[w3], %[" c2 "], %[" B "]\n\t"                                           \
    "v_fma_f64 %[" c0 "], %[w4], %[" c2 "], %[" A "]\n\t"                                          \
    "v_fma_f64 %[t2], %[w3], %[" c3 "], %[t2]\n\tv_fma_f64 %[t3], %[w3], %[" c4 "], %[t3]\n\t"     \
    "v_fma_f64 %[" c1 "], %[w4], %[" c3 "], %[" B "]\n\t"                                          \
    "v_fma_f64 %[" c2 "], %[w4], %[" c4 "], %[t2]\n\t"                                             \
    "v_fma_f64 %[" c3 "], %[w4], %[" c5 "], %[t3]\n\t"

__device__ __forceinline__ void stencil_rows8(double *c, double r0, double r1, double &u, double &v,
                                              const double (&w)[5])
{
    double qa, qb, t2, t3;
    asm(BB_W2_4("u", "v", "qa", "qb", "c0", "c1", "c2", "c3", "c4", "c5")
        BB_W2_4("qa", "qb", "u", "v", "c4", "c5", "c6", "c7", "r0", "r1")
        : [c0] "+&v"(c[0]), [c1] "+&v"(c[1]), [c2] "+&v"(c[2]), [c3] "+&v"(c[3]), [c4] "+&v"(c[4]),
          [c5] "+&v"(c[5]), [c6] "+&v"(c[6]), [c7] "+&v"(c[7]), [u] "+&v"(u), [v] "+&v"(v),
          [qa] "=&v"(qa), [qb] "=&v"(qb), [t2] "=&v"(t2), [t3] "=&v"(t3)
        : [r0] "v"(r0), [r1] "v"(r1), [w0] "s"(w[0]), [w1] "s"(w[1]), [w2] "s"(w[2]), [w3] "s"(w[3]),
          [w4] "s"(w[4]));
}
#undef BB_W1_4
#undef BB_W2_4

// f_i = sum_{d=-K..K} w[d+K] c_{i+d}: the explicit half B of the scheme, a
// constant stencil of 2K+1 weights.  Periodic (CYC): indices wrap mod n like
// the matrix.  Otherwise the terms whose row falls outside the system are left
// out.  The sum is one fma chain from the leftmost term, so every kernel that
// uses the policy rounds it the same way.
template <int K, bool CYC>
struct StencilRhs {
    static constexpr int R = K;
    double w[2 * K + 1];
    struct State {};
    __device__ State lane_state(int64_t, int) const { return State{}; }

    template <int C, bool FULL>
    __device__ __forceinline__ void operator()(double (&c)[C], const Halo &h, int j,
                                               bool last_chunk, int nrow, const State &) const
    {
        // rows j*C - 1, j*C - 2: the previous chunk, or rows n-1, n-2 (periodic)
        double m1 = h.l1, m2 = h.l2;
        if (j == 0) {
            m1 = CYC ? h.en1 : 0.0;
            m2 = CYC ? h.en2 : 0.0;
        }
        // rows j*C + C, j*C + C + 1: the next chunk, or rows 0, 1 (periodic)
        // after the last chunk of a full decomposition
        double q1 = h.r1, q2 = h.r2;
        if constexpr (FULL) {
            if (last_chunk) {
                q1 = CYC ? h.e0 : 0.0;
                q2 = CYC ? h.e1 : 0.0;
            }
        }
        if constexpr (FULL && C % 8 == 0) {
            if constexpr (K == 1) {
                double s = fma(w[1], c[0], w[0] * m1);
#pragma unroll
                for (int t = 0; t < C; t += 8)
                    stencil_rows8(c + t, t + 8 < C ? c[t + 8 < C ? t + 8 : 0] : q1, s, w);
            } else {
                double u = fma(w[1], m1, w[0] * m2), v = w[0] * m1;
#pragma unroll
                for (int t = 0; t < C; t += 8)
                    stencil_rows8(c + t, t + 8 < C ? c[t + 8 < C ? t + 8 : 0] : q1,
                                  t + 8 < C ? c[t + 8 < C ? t + 9 : 0] : q2, u, v, w);
            }
            return;
        }
        // ragged: rows past n-1 of the system are rows 0, 1 (periodic) or absent
        const double past0 = CYC ? h.e0 : 0.0, past1 = CYC ? h.e1 : 0.0;
        rows_up<C>([&](int t) {
            const double cur = c[t];
            double p1 = t + 1 < C ? c[t + 1] : q1;
            if constexpr (!FULL) p1 = t + 1 < nrow ? p1 : (t + 1 == nrow ? past0 : past1);
            double f;
            if constexpr (K == 1) {
                f = fma(w[2], p1, fma(w[1], cur, w[0] * m1));
            } else {
                double p2 = t + 2 < C ? c[t + 2] : (t + 2 == C ? q1 : q2);
                if constexpr (!FULL) p2 = t + 2 < nrow ? p2 : (t + 2 == nrow ? past0 : past1);
                f = fma(w[4], p2, fma(w[3], p1, fma(w[2], cur, fma(w[1], m1, w[0] * m2))));
            }
            if constexpr (!FULL) f = t < nrow ? f : 0.0;
            c[t] = f;
            m2 = m1;
            m1 = cur;
        });
    }
};

// traj_stride > 0: store the state after every step s at out + s * traj_stride
// (a trajectory) instead of only the last one.
template <int K, bool CYC>
hipError_t launch_cn_kc(const double *table, int64_t table_elems, const CyclicQ &q,
                        const SweepGeom &g, bool scalar, const double *w, int64_t steps,
                        int64_t traj_stride, const double *in, double *out, hipStream_t s)
{
    StencilRhs<K, CYC> r;
    for (int d = 0; d <= 2 * K; ++d) r.w[d] = w[d];
    if (traj_stride > 0) {
        StepStats st;
        st.traj_stride = traj_stride;
        return launch_stepper<StencilRhs<K, CYC>, K, CYC, false, true>(table, table_elems, q, g, scalar,
                                                                      r, steps, in, out, s, st);
    }
    return launch_stepper<StencilRhs<K, CYC>, K, CYC>(table, table_elems, q, g, scalar, r, steps, in,
                                                      out, s);
}

// The stencil as the source of the long-system launches (one step per call):
// a chunk's rows and the K rows on each side of it, read from the state
// before the step -- wrapped mod n (periodic) or zero outside the system.
// The halo takes the place of the wrap rows, so the policy sees every chunk
// as an inner one.
template <int K, bool CYC>
struct StencilLongSrc {
    StencilRhs<K, CYC> rhs;
    const double *c;
    __device__ __forceinline__ double row(int i, int64_t k, int64_t ld, int n) const
    {
        if constexpr (CYC) {
            i = i < 0 ? i + n : (i >= n ? i - n : i);
        } else {
            if (i < 0 || i >= n) return 0.0;
        }
        return c[(int64_t)i * ld + k];
    }
    template <int C>
    __device__ __forceinline__ void full(double (&v)[C], int row0, int64_t k, int64_t ld,
                                         int n) const
    {
        load_chunk<double, C, true>(v, c, row0, k, ld, n);
        Halo h{};
        h.l1 = row(row0 - 1, k, ld, n);
        h.l2 = row(row0 - 2, k, ld, n);
        h.r1 = row(row0 + C, k, ld, n);
        h.r2 = row(row0 + C + 1, k, ld, n);
        rhs.template operator()<C, true>(v, h, 1, false, C, typename StencilRhs<K, CYC>::State{});
    }
    // the last chunk: rows row0 .. n-1 (row0 >= C); past row n-1 come rows
    // 0, 1 (periodic) or nothing
    template <int C>
    __device__ __forceinline__ void tail(double (&v)[C], int row0, int64_t k, int64_t ld,
                                         int n) const
    {
        load_chunk<double, C, false>(v, c, row0, k, ld, n);
        Halo h{};
        h.l1 = row(row0 - 1, k, ld, n);
        h.l2 = row(row0 - 2, k, ld, n);
        if constexpr (CYC) {
            h.e0 = c[k];
            h.e1 = c[ld + k];
        }
        rhs.template operator()<C, false>(v, h, 1, false, n - row0,
                                          typename StencilRhs<K, CYC>::State{});
    }
};

// Three waves, as the other sources' kernels have: in 162 VGPRs without spills;
// left alone the compiler takes 184 and two (periodic n = 2049, m = 5000, one
// step: 91 us at two, 83 at three; n = 1500, m = 6000 86 and 80; the other way at
// n = 4000, m = 50001, 1197 and 1226).
template <>
constexpr int kSolveWaves<StencilLongSrc<2, true>> = 3;

template <int K>
hipError_t launch_cn_long_k(bool cyclic, const double *table, const CyclicQ &q, const LongGeom &g,
                            const double *w, const double *in, double *out, hipStream_t s)
{
    if (cyclic) {
        StencilLongSrc<K, true> src{{}, in};
        for (int d = 0; d <= 2 * K; ++d) src.rhs.w[d] = w[d];
        return launch_long_k<K, true>(table, q, g, src, out, s);
    }
    StencilLongSrc<K, false> src{{}, in};
    for (int d = 0; d <= 2 * K; ++d) src.rhs.w[d] = w[d];
    return launch_long_k<K, false>(table, q, g, src, out, s);
}

template <int K>
hipError_t launch_cn_k(bool cyclic, const double *table, int64_t table_elems, const CyclicQ &q,
                       const SweepGeom &g, bool scalar, const double *w, int64_t steps,
                       int64_t traj_stride, const double *in, double *out, hipStream_t s)
{
    return cyclic ? launch_cn_kc<K, true>(table, table_elems, q, g, scalar, w, steps, traj_stride, in, out, s)
                  : launch_cn_kc<K, false>(table, table_elems, q, g, scalar, w, steps, traj_stride, in, out, s);
}

}  // namespace
}  // namespace bb
