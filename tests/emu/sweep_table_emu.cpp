// sweep_table_emu.cpp -- CPU model of a one-launch solve on its own table
// (build_sweep_table), for tests only: boundary-state dot products, both
// scans with the periodic end states taken from them, the correction put
// into the chunks' histories and futures (full decompositions) or added row
// by row (ragged ones), forward and backward passes.
#include <string>
#include <vector>

#include "../../paper_2107_05395_amd/csrc/factor.h"

extern "C" int emu_sweep(int kind, const double *a, const double *b, const double *c,
                         const double *d, const double *e, int64_t n, int adjoint, int C,
                         const double *f, double *x)
{
    bb::Factor F;
    std::string err;
    const double *bands[5] = {a, b, c, d, e};
    int st = bb::make_factor(kind, bands, n, F, err);
    if (st) return st;
    const int K = F.K, KK = K * K;
    const int P = bb::lanes_for(n, C);
    if ((int64_t)P * C < n) return -100;
    const bool full = (int64_t)P * C == n;
    const bb::Direction &dir = adjoint ? F.adjoint : F.primal;
    const std::vector<double> tab = bb::build_sweep_table(dir, K, F.cyclic, n, C, P);
    if ((int64_t)tab.size() != bb::sweep_table_len(K, F.cyclic, full, C, P)) return -101;
    const int64_t L = (int64_t)P * (C + 1);
    auto arr = [&](int q, int j, int t) { return tab[(size_t)(q * L + (int64_t)j * (C + 1) + t)]; };
    const double *Mf = tab.data() + bb::sweep_arrays(K, F.cyclic, full) * L, *Mb = Mf + P * KK,
                 *G = Mb + P * KK, *HZ = G + P * KK, *FZ = HZ + P * KK;
    const int qs = 2 * K, ql = 2 * K + 1, qu = 3 * K + 1, qz = 4 * K + 1;
    const int real = (int)((n - 1) / C) + 1;
    auto affine = [&](const double *M, double *y, const double *add) {
        double r[2] = {0, 0};
        for (int i = 0; i < K; ++i) {
            r[i] = add[i];
            for (int k = 0; k < K; ++k) r[i] += M[i * K + k] * y[k];
        }
        y[0] = r[0];
        y[1] = r[1];
    };
    std::vector<double> v((size_t)P * C, 0.0), E(2 * P, 0.0), O(2 * P, 0.0), H(2 * P, 0.0), Fu(2 * P, 0.0);
    for (int64_t i = 0; i < n; ++i) v[i] = f[i];
    for (int j = 0; j < P; ++j)
        for (int t = 0; t < C; ++t)
            for (int k = 0; k < K; ++k) {
                E[2 * j + k] += arr(k, j, t) * v[(size_t)j * C + t];
                O[2 * j + k] += arr(K + k, j, t) * v[(size_t)j * C + t];
            }
    double y[2] = {0, 0}, ye[2] = {0, 0}, g[2] = {0, 0};
    for (int j = 0; j < P; ++j) {
        H[2 * j] = y[0];
        H[2 * j + 1] = y[1];
        affine(Mf + j * KK, y, &E[2 * j]);
        if (j == real - 1) ye[0] = y[0], ye[1] = y[1];
    }
    for (int j = P - 1; j >= 0; --j) {
        Fu[2 * j] = g[0];
        Fu[2 * j + 1] = g[1];
        double s[2] = {H[2 * j], H[2 * j + 1]};
        affine(G + j * KK, s, &O[2 * j]);
        affine(Mb + j * KK, g, s);
    }
    double cs[2] = {0, 0};
    if (F.cyclic) {
        const bb::CyclicQ &q = dir.cor.q;
        if (K == 1) {
            cs[0] = q.q[0][0] * g[0] + q.q[0][1] * ye[0];
        } else {
            const double xn2 = ye[1] + q.u1_nm2 * ye[0];
            for (int r = 0; r < 2; ++r)
                cs[r] = q.q[r][0] * g[0] + q.q[r][1] * g[1] + q.q[r][2] * xn2 + q.q[r][3] * ye[0];
        }
        if (full)
            for (int j = 0; j < P; ++j)
                for (int i = 0; i < K; ++i)
                    for (int k = 0; k < K; ++k) {
                        H[2 * j + i] += HZ[j * KK + i * K + k] * cs[k];
                        Fu[2 * j + i] += FZ[j * KK + i * K + k] * cs[k];
                    }
    }
    for (int j = 0; j < P; ++j) {
        double y1 = H[2 * j], y2 = H[2 * j + 1];
        for (int t = 0; t < C; ++t) {
            double w = arr(qs, j, t) * v[(size_t)j * C + t] + arr(ql, j, t) * y1;
            if (K == 2) w += arr(ql + 1, j, t) * y2;
            v[(size_t)j * C + t] = w;
            y2 = y1;
            y1 = w;
        }
        double x1 = Fu[2 * j], x2 = Fu[2 * j + 1];
        for (int t = C - 1; t >= 0; --t) {
            double w = v[(size_t)j * C + t] + arr(qu, j, t) * x1;
            if (K == 2) w += arr(qu + 1, j, t) * x2;
            x2 = x1;
            x1 = w;
            if (F.cyclic && !full) {
                w += arr(qz, j, t) * cs[0];
                if (K == 2) w += arr(qz + 1, j, t) * cs[1];
            }
            v[(size_t)j * C + t] = w;
        }
    }
    for (int64_t i = 0; i < n; ++i) x[i] = v[i];
    return 0;
}
