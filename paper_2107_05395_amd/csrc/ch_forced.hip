// ch_forced.hip -- fused steps of the forced Cahn-Hilliard equation in the
// frame of the travelling wave (the forced flow-pattern section, numerical
// scheme): the Section 5.1 right-hand side plus an advection term,
// differenced with the fifth-order Hamilton-Jacobi WENO scheme the paper
// cites, and a sinusoidal forcing; each run has its own advection speed and
// forcing.  A right-hand-side policy of the fused stepper (stepper.h).
#include <cmath>

#include "long_core.h"
#include "stepper.h"

namespace bb {
namespace {

__device__ __forceinline__ double nl3(double c) { return fma(c * c, c, -c); }

// N / S for S at least about 1 and far from overflow (or NaN): the reciprocal
// to about 24 bits, two Newton steps, the quotient and its remainder's
// correction (the IEEE division's scaling and fix-up of its exceptional
// operands left out: 8 instructions instead of 11 to 13).
__device__ __forceinline__ double divide_scaled(double N, double S)
{
    double r = __builtin_amdgcn_rcp(S);
    r = fma(r, fma(-S, r, 1.0), r);
    r = fma(r, fma(-S, r, 1.0), r);
    const double q = N * r;
    return fma(fma(-S, q, N), r, q);
}

// The five one-sided differences v1..v5 of the WENO5 scheme (Jiang and Peng;
// three third-order candidates blended with weights 0.1, 0.6, 0.3 over
// (smoothness + eps)^2, eps = 1e-6 max v_q^2 + 1e-99), ordered from the far
// upwind end, enter through the second differences
//   a = v2 - v1, b = v3 - v2, c = v4 - v3, d = v5 - v4:
// the candidates are v3 + (5b - 2a)/6, v3 + (b + 2c)/6 and v3 + (4c - d)/6, and
// four times the smoothness measures 13/3 (b - a)^2 + (3b - a)^2,
// 13/3 (c - b)^2 + (b + c)^2 and 13/3 (d - c)^2 + (d - 3c)^2.  From row to row
// these differences carry over, and for the other upwind side they are the
// same numbers mirrored and negated, so a row selects four of them instead of
// five differences of each side.  Returns dx times the derivative less v3.
// The weights gamma_k / t_k^2 times (t1 t2 t3)^2 need no division; the common
// scale 2^-e, e the exponent of eps, keeps the products in range (t_k is
// between eps and about 4e7 eps), states of any magnitude included.
__device__ __forceinline__ double weno5_rest(double a, double b, double c, double d, double vmax2)
{
    const double eps4 = fma(4e-6, vmax2, 4e-99);
    const double e1 = b - a, e2 = c - b, e3 = d - c;
    const double g1 = fma(3.0, b, -a), g2 = b + c, g3 = fma(-3.0, c, d);
    constexpr double k = 13.0 / 3.0;
    double t1 = fma(k * e1, e1, fma(g1, g1, eps4));
    double t2 = fma(k * e2, e2, fma(g2, g2, eps4));
    double t3 = fma(k * e3, e3, fma(g3, g3, eps4));
    const int e = -__builtin_amdgcn_frexp_exp(eps4);
    t1 = __builtin_ldexp(t1, e);
    t2 = __builtin_ldexp(t2, e);
    t3 = __builtin_ldexp(t3, e);
    const double r1 = t2 * t3, r2 = t1 * t3, r3 = t1 * t2;
    const double w1 = r1 * r1, w2 = r2 * r2, w3 = r3 * r3;
    // weights 1 : 6 : 3; six times their sum
    const double S = fma(6.0, w1, fma(36.0, w2, 18.0 * w3));
    const double N = fma(w1, fma(5.0, b, -2.0 * a), fma(w2, fma(12.0, c, 6.0 * b), w3 * fma(12.0, c, -3.0 * d)));
    return divide_scaled(N, S);
}

// f_i = C_i + alpha (N_{i-1} - 2 N_i + N_{i+1}) + beta W_i(C) + amp cos(kdx i),
// N = C^3 - C, periodic, W upwinded for dC/dt = v dC/deta (beta > 0:
// right-biased differences).  The scheme's per-run coefficients follow from
// the physical parameters of run k when its group is loaded: the advection
// term dt v dC/deta with the WENO derivative W/dx gives beta = dt v / dx, the
// forcing dt f0 k cos(k eta) at eta_i = i dx gives amp = dt f0 k and
// kdx = k dx.
// Bound by FP64 issue: 78 vector instructions a row (about 170 with five
// differences of each side formed and selected per row and two divisions),
// 92 with the solve; n = 512, m = 2^16: 131 -> 99 us a step, of 86 at one
// instruction per 4 clocks.
struct ForcedChRhs {
    static constexpr int R = 3;
    double alpha, dt, dx;
    const double *v, *f0, *k;   // device, one per run
    struct State {
        double beta, amp, c0, s0, cd, sd;   // cos, sin of kdx * row0 and of kdx
    };
    __device__ State lane_state(int64_t run, int row0) const
    {
        State st;
        const double kr = k[run];
        st.beta = dt * v[run] / dx;
        st.amp = dt * f0[run] * kr;
        const double kd = kr * dx;
        sincos(kd * (double)row0, &st.s0, &st.c0);
        sincos(kd, &st.sd, &st.cd);
        return st;
    }

    template <int C, bool FULL>
    __device__ __forceinline__ void operator()(double (&c)[C], const Halo &h, int j,
                                               bool last_chunk, int nrow, const State &st) const
    {
        // rows j*C - 1 .. j*C - 3: the previous chunk, or rows n-1 .. n-3
        double m1 = h.l1, m2 = h.l2, m3 = h.l3;
        if (j == 0) {
            m1 = h.en1;
            m2 = h.en2;
            m3 = h.en3;
        }
        // rows j*C + C .. j*C + C + 2: the next chunk, or rows 0 .. 2 after
        // the last chunk of a full decomposition
        double q1 = h.r1, q2 = h.r2, q3 = h.r3;
        if constexpr (FULL) {
            if (last_chunk) {
                q1 = h.e0;
                q2 = h.e1;
                q3 = h.e2;
            }
        }
        // row t + 3 of the chunk before this step
        auto ahead3 = [&](int t) -> double {
            const int u = t + 3;
            double x = u < C ? c[u < C ? u : C - 1] : (u == C ? q1 : (u == C + 1 ? q2 : q3));
            if constexpr (!FULL) {
                const int w = u - nrow;   // ragged: past row n-1 come rows 0, 1, 2
                x = w < 0 ? x : (w == 0 ? h.e0 : (w == 1 ? h.e1 : h.e2));
            }
            return x;
        };
        const bool plus = st.beta > 0.0;
        const double bsign = plus ? -st.beta : st.beta;
        // rows t + 1, t + 2; first differences D_i = C_{i+1} - C_i around row t
        // (dk: D_{t+k}), their squares, pairs' maxima and second differences
        // G_i = D_i - D_{i-1}
        double p1, p2;
        {
            auto first = [&](int u) -> double {
                double x = u < C ? c[u < C ? u : C - 1] : (u == C ? q1 : q2);
                if constexpr (!FULL) {
                    const int w = u - nrow;
                    x = w < 0 ? x : (w == 0 ? h.e0 : h.e1);
                }
                return x;
            };
            p1 = first(1);
            p2 = first(2);
        }
        double dm1 = c[0] - m1, d0 = p1 - c[0], d1 = p2 - p1;
        const double dm2 = m1 - m2, dm3 = m2 - m3;
        double gm2 = dm2 - dm3, gm1 = dm1 - dm2, g0 = d0 - dm1, g1 = d1 - d0;
        double sm3 = dm3 * dm3, sm2 = dm2 * dm2, sm1 = dm1 * dm1, s0 = d0 * d0, s1 = d1 * d1;
        double xm2 = fmax(sm2, sm1), xm1 = fmax(sm1, s0), x0 = fmax(s0, s1);
        double nprev = nl3(m1), ncur = nl3(c[0]);
        double cs = st.c0, sn = st.s0;
        rows_up<C>([&](int t) {
            const double cur = c[t];
            const double p3 = ahead3(t);
            const double nnext = nl3(p1);
            double f = fma(alpha, fma(-2.0, ncur, nprev) + nnext, cur);
            const double d2 = p3 - p2, g2 = d2 - d1, s2 = d2 * d2;
            // upwind: rows below (beta > 0) or above; the second differences of
            // the rows below enter negated, which the sign of bsign carries
            const double a = plus ? g2 : gm2, b = plus ? g1 : gm1, d = plus ? gm1 : g1;
            const double v3 = plus ? d0 : dm1;
            const double vmax2 = fmax(fmax(xm2, x0), plus ? s2 : sm3);
            const double rest = weno5_rest(a, b, g0, d, vmax2);
            f = fma(st.beta, v3, f);
            f = fma(bsign, rest, f);
            f = fma(st.amp, cs, f);
            if constexpr (!FULL) f = t < nrow ? f : 0.0;
            c[t] = f;
            p1 = p2;
            p2 = p3;
            dm1 = d0;
            d0 = d1;
            d1 = d2;
            gm2 = gm1;
            gm1 = g0;
            g0 = g1;
            g1 = g2;
            sm3 = sm2;
            sm2 = sm1;
            sm1 = s0;
            s0 = s1;
            s1 = s2;
            xm2 = xm1;
            xm1 = x0;
            x0 = fmax(s0, s1);
            nprev = ncur;
            ncur = nnext;
            const double cn = fma(cs, st.cd, -sn * st.sd);   // rotate to row t + 1
            sn = fma(sn, st.cd, cs * st.sd);
            cs = cn;
        });
    }
};

// The forced right-hand side as the source of the long-system launches
// (one step per call): a chunk's rows and the three rows on each side of it,
// indices mod n, read from the state before the step.  The halo takes the
// place of the wrap rows, so the policy sees every chunk as an inner one.
struct ForcedLongSrc {
    ForcedChRhs rhs;
    const double *c;
    __device__ __forceinline__ double row(int i, int64_t k, int64_t ld, int n) const
    {
        i = i < 0 ? i + n : (i >= n ? i - n : i);
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
        h.l3 = row(row0 - 3, k, ld, n);
        h.r1 = row(row0 + C, k, ld, n);
        h.r2 = row(row0 + C + 1, k, ld, n);
        h.r3 = row(row0 + C + 2, k, ld, n);
        rhs.template operator()<C, true>(v, h, 1, false, C, rhs.lane_state(k, row0));
    }
    // the last chunk: rows row0 .. n-1 (row0 >= C >= 16); past row n-1 come
    // rows 0, 1, 2
    template <int C>
    __device__ __forceinline__ void tail(double (&v)[C], int row0, int64_t k, int64_t ld,
                                         int n) const
    {
        load_chunk<double, C, false>(v, c, row0, k, ld, n);
        Halo h{};
        h.l1 = row(row0 - 1, k, ld, n);
        h.l2 = row(row0 - 2, k, ld, n);
        h.l3 = row(row0 - 3, k, ld, n);
        h.e0 = c[k];
        h.e1 = c[ld + k];
        h.e2 = c[2 * ld + k];
        rhs.template operator()<C, false>(v, h, 1, false, n - row0, rhs.lane_state(k, row0));
    }
};

}  // namespace

hipError_t launch_ch_forced_long(const double *table, const CyclicQ &q, const LongGeom &g,
                                 double alpha, double dt, double dx, const double *v,
                                 const double *f0, const double *k, const double *in, double *out,
                                 hipStream_t s)
{
    ForcedChRhs r;
    r.alpha = alpha;
    r.dt = dt;
    r.dx = dx;
    r.v = v;
    r.f0 = f0;
    r.k = k;
    return launch_long_k<2, true>(table, q, g, ForcedLongSrc{r, in}, out, s);
}

hipError_t launch_ch_forced(const double *table, int64_t table_elems, const CyclicQ &q,
                            const SweepGeom &g, bool scalar, double alpha, double dt, double dx,
                            const double *v, const double *f0, const double *k, int64_t steps,
                            const double *in, double *out, hipStream_t s)
{
    ForcedChRhs r;
    r.alpha = alpha;
    r.dt = dt;
    r.dx = dx;
    r.v = v;
    r.f0 = f0;
    r.k = k;
    return launch_stepper<ForcedChRhs, 2, true>(table, table_elems, q, g, scalar, r, steps, in,
                                                out, s);
}

}  // namespace bb
