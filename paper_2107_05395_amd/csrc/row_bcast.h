// row_bcast.h -- the three passes of a chunk solve with the coefficients
// broadcast from registers: v_fmac_f64 with the DPP control row_newbcast:i
// takes lane i's value of its first operand for all 16 lanes of a row, at the
// rate of the plain instruction (measured 2.16 against 2.12 ns per wave and
// SIMD; an 8-byte LDS read that feeds it costs 6.8).  When every 16-lane row
// of a wave works on one chunk, lane i of the row holds the coefficients of
// rows 16b + i, and one LDS read serves 16 rows: a pass reads each
// coefficient array C/16 times instead of C times.
//
// The passes are written in asm blocks of 8 rows because the compiler does
// not fold the broadcast into v_fmac_f64 (it emits v_mov_b64_dpp and the
// product).  Each block opens with s_nop 1: a DPP operand may not be read
// within two wait states of a VALU write, and the compiler, which does not
// see into the block, may have moved a coefficient just before it.  Operands
// written before the last one is read are early clobbers (+&v): without that an
// input of the same value would share their registers.  Nothing in a block is a
// memory access.  Operation order and rounding are those of
// chunk_solve's plain passes.
#pragma once

#include "internal.h"

namespace bb {
namespace {

constexpr int kRowLanes = 16;   // lanes of a DPP row

// Coefficients of one array for a chunk: lane i of each row holds rows 16b + i.
template <int C>
struct RowCoef {
    double r[C / kRowLanes];
};

// base: the array's chunk, plus this lane's position in its row
template <int C>
__device__ __forceinline__ RowCoef<C> row_coef(const double *base)
{
    RowCoef<C> k;
#pragma unroll
    for (int b = 0; b < C / kRowLanes; ++b) k.r[b] = base[b * kRowLanes];
    return k;
}

#define BB_DPP(lane) " row_newbcast:" #lane " row_mask:0xf bank_mask:0xf\n\t"
#define BB_FMAC(acc, coef, x, lane) "v_fmac_f64_dpp %[" acc "], %[" coef "], %[" x "]" BB_DPP(lane)
// v <- coefficient * v
#define BB_SCALE(v, coef, tmp, lane)                                                               \
    "v_mov_b64_dpp %[" tmp "], %[" coef "]" BB_DPP(lane)                                           \
    "v_mul_f64 %[" v "], %[" tmp "], %[" v "]\n\t"

#define BB_ROWS_UP(OP, a, b, c, d, e, f, g, h)                                                     \
    OP("v0", a) OP("v1", b) OP("v2", c) OP("v3", d) OP("v4", e) OP("v5", f) OP("v6", g) OP("v7", h)
#define BB_V_IN(v, t)                                                                              \
    [v0] "v"(v[t]), [v1] "v"(v[t + 1]), [v2] "v"(v[t + 2]), [v3] "v"(v[t + 3]), [v4] "v"(v[t + 4]), \
        [v5] "v"(v[t + 5]), [v6] "v"(v[t + 6]), [v7] "v"(v[t + 7])
#define BB_V_IO(v, t)                                                                              \
    [v0] "+&v"(v[t]), [v1] "+&v"(v[t + 1]), [v2] "+&v"(v[t + 2]), [v3] "+&v"(v[t + 3]),                \
        [v4] "+&v"(v[t + 4]), [v5] "+&v"(v[t + 5]), [v6] "+&v"(v[t + 6]), [v7] "+&v"(v[t + 7])

// pass 1, rows t .. t+7: e += wE v, o += wS v (K = 2: two of each)
#define BB_P1K1(v, lane) BB_FMAC("e1", "we1", v, lane) BB_FMAC("o1", "ws1", v, lane)
#define BB_P1K2(v, lane)                                                                           \
    BB_P1K1(v, lane) BB_FMAC("e2", "we2", v, lane) BB_FMAC("o2", "ws2", v, lane)

template <int T, int C>
__device__ __forceinline__ void rows8_ends(const double (&v)[C], double &e1, double &o1, double we1,
                                           double ws1)
{
    if constexpr (T / 8 % 2 == 0)
        asm("s_nop 1\n\t" BB_ROWS_UP(BB_P1K1, 0, 1, 2, 3, 4, 5, 6, 7)
            : [e1] "+&v"(e1), [o1] "+&v"(o1)
            : [we1] "v"(we1), [ws1] "v"(ws1), BB_V_IN(v, T));
    else
        asm("s_nop 1\n\t" BB_ROWS_UP(BB_P1K1, 8, 9, 10, 11, 12, 13, 14, 15)
            : [e1] "+&v"(e1), [o1] "+&v"(o1)
            : [we1] "v"(we1), [ws1] "v"(ws1), BB_V_IN(v, T));
}

template <int T, int C>
__device__ __forceinline__ void rows8_ends(const double (&v)[C], double &e1, double &o1, double &e2,
                                           double &o2, double we1, double ws1, double we2, double ws2)
{
    if constexpr (T / 8 % 2 == 0)
        asm("s_nop 1\n\t" BB_ROWS_UP(BB_P1K2, 0, 1, 2, 3, 4, 5, 6, 7)
            : [e1] "+&v"(e1), [o1] "+&v"(o1), [e2] "+&v"(e2), [o2] "+&v"(o2)
            : [we1] "v"(we1), [ws1] "v"(ws1), [we2] "v"(we2), [ws2] "v"(ws2), BB_V_IN(v, T));
    else
        asm("s_nop 1\n\t" BB_ROWS_UP(BB_P1K2, 8, 9, 10, 11, 12, 13, 14, 15)
            : [e1] "+&v"(e1), [o1] "+&v"(o1), [e2] "+&v"(e2), [o2] "+&v"(o2)
            : [we1] "v"(we1), [ws1] "v"(ws1), [we2] "v"(we2), [ws2] "v"(ws2), BB_V_IN(v, T));
}

// pass 2, rows t .. t+7: y = s v + l2 y2 + l1 y1, the scaling two rows ahead
// of the recurrence
#define BB_P2K1(a, b, c, d, e, f, g, h)                                                            \
    BB_SCALE("v0", "s", "ta", a) BB_SCALE("v1", "s", "tb", b) BB_FMAC("v0", "l1", "y1", a)         \
    BB_SCALE("v2", "s", "ta", c) BB_FMAC("v1", "l1", "v0", b)                                      \
    BB_SCALE("v3", "s", "tb", d) BB_FMAC("v2", "l1", "v1", c)                                      \
    BB_SCALE("v4", "s", "ta", e) BB_FMAC("v3", "l1", "v2", d)                                      \
    BB_SCALE("v5", "s", "tb", f) BB_FMAC("v4", "l1", "v3", e)                                      \
    BB_SCALE("v6", "s", "ta", g) BB_FMAC("v5", "l1", "v4", f)                                      \
    BB_SCALE("v7", "s", "tb", h) BB_FMAC("v6", "l1", "v5", g) BB_FMAC("v7", "l1", "v6", h)

#define BB_P2K2(a, b, c, d, e, f, g, h)                                                            \
    BB_SCALE("v0", "s", "ta", a) BB_SCALE("v1", "s", "tb", b)                                      \
    BB_FMAC("v0", "l2", "y2", a) BB_FMAC("v1", "l2", "y1", b) BB_FMAC("v0", "l1", "y1", a)         \
    BB_SCALE("v2", "s", "ta", c) BB_FMAC("v1", "l1", "v0", b) BB_FMAC("v2", "l2", "v0", c)         \
    BB_SCALE("v3", "s", "tb", d) BB_FMAC("v2", "l1", "v1", c) BB_FMAC("v3", "l2", "v1", d)         \
    BB_SCALE("v4", "s", "ta", e) BB_FMAC("v3", "l1", "v2", d) BB_FMAC("v4", "l2", "v2", e)         \
    BB_SCALE("v5", "s", "tb", f) BB_FMAC("v4", "l1", "v3", e) BB_FMAC("v5", "l2", "v3", f)         \
    BB_SCALE("v6", "s", "ta", g) BB_FMAC("v5", "l1", "v4", f) BB_FMAC("v6", "l2", "v4", g)         \
    BB_SCALE("v7", "s", "tb", h) BB_FMAC("v6", "l1", "v5", g) BB_FMAC("v7", "l2", "v5", h)         \
    BB_FMAC("v7", "l1", "v6", h)

template <int T, int C>
__device__ __forceinline__ void rows8_forward(double (&v)[C], double y1, double s, double l1)
{
    double ta, tb;
    if constexpr (T / 8 % 2 == 0)
        asm("s_nop 1\n\t" BB_P2K1(0, 1, 2, 3, 4, 5, 6, 7)
            : BB_V_IO(v, T), [ta] "=&v"(ta), [tb] "=&v"(tb)
            : [y1] "v"(y1), [s] "v"(s), [l1] "v"(l1));
    else
        asm("s_nop 1\n\t" BB_P2K1(8, 9, 10, 11, 12, 13, 14, 15)
            : BB_V_IO(v, T), [ta] "=&v"(ta), [tb] "=&v"(tb)
            : [y1] "v"(y1), [s] "v"(s), [l1] "v"(l1));
}

template <int T, int C>
__device__ __forceinline__ void rows8_forward(double (&v)[C], double y1, double y2, double s,
                                              double l1, double l2)
{
    double ta, tb;
    if constexpr (T / 8 % 2 == 0)
        asm("s_nop 1\n\t" BB_P2K2(0, 1, 2, 3, 4, 5, 6, 7)
            : BB_V_IO(v, T), [ta] "=&v"(ta), [tb] "=&v"(tb)
            : [y1] "v"(y1), [y2] "v"(y2), [s] "v"(s), [l1] "v"(l1), [l2] "v"(l2));
    else
        asm("s_nop 1\n\t" BB_P2K2(8, 9, 10, 11, 12, 13, 14, 15)
            : BB_V_IO(v, T), [ta] "=&v"(ta), [tb] "=&v"(tb)
            : [y1] "v"(y1), [y2] "v"(y2), [s] "v"(s), [l1] "v"(l1), [l2] "v"(l2));
}

// pass 3, rows t+7 .. t: x = y + u2 x2 + u1 x1
#define BB_P3K1(a, b, c, d, e, f, g, h)                                                            \
    BB_FMAC("v7", "u1", "x1", h) BB_FMAC("v6", "u1", "v7", g) BB_FMAC("v5", "u1", "v6", f)         \
    BB_FMAC("v4", "u1", "v5", e) BB_FMAC("v3", "u1", "v4", d) BB_FMAC("v2", "u1", "v3", c)         \
    BB_FMAC("v1", "u1", "v2", b) BB_FMAC("v0", "u1", "v1", a)

#define BB_P3K2(a, b, c, d, e, f, g, h)                                                            \
    BB_FMAC("v7", "u2", "x2", h) BB_FMAC("v6", "u2", "x1", g)                                      \
    BB_FMAC("v7", "u1", "x1", h) BB_FMAC("v6", "u1", "v7", g) BB_FMAC("v5", "u2", "v7", f)         \
    BB_FMAC("v5", "u1", "v6", f) BB_FMAC("v4", "u2", "v6", e)                                      \
    BB_FMAC("v4", "u1", "v5", e) BB_FMAC("v3", "u2", "v5", d)                                      \
    BB_FMAC("v3", "u1", "v4", d) BB_FMAC("v2", "u2", "v4", c)                                      \
    BB_FMAC("v2", "u1", "v3", c) BB_FMAC("v1", "u2", "v3", b)                                      \
    BB_FMAC("v1", "u1", "v2", b) BB_FMAC("v0", "u2", "v2", a) BB_FMAC("v0", "u1", "v1", a)

template <int T, int C>
__device__ __forceinline__ void rows8_backward(double (&v)[C], double x1, double u1)
{
    if constexpr (T / 8 % 2 == 0)
        asm("s_nop 1\n\t" BB_P3K1(0, 1, 2, 3, 4, 5, 6, 7)
            : BB_V_IO(v, T) : [x1] "v"(x1), [u1] "v"(u1));
    else
        asm("s_nop 1\n\t" BB_P3K1(8, 9, 10, 11, 12, 13, 14, 15)
            : BB_V_IO(v, T) : [x1] "v"(x1), [u1] "v"(u1));
}

template <int T, int C>
__device__ __forceinline__ void rows8_backward(double (&v)[C], double x1, double x2, double u1,
                                               double u2)
{
    if constexpr (T / 8 % 2 == 0)
        asm("s_nop 1\n\t" BB_P3K2(0, 1, 2, 3, 4, 5, 6, 7)
            : BB_V_IO(v, T) : [x1] "v"(x1), [x2] "v"(x2), [u1] "v"(u1), [u2] "v"(u2));
    else
        asm("s_nop 1\n\t" BB_P3K2(8, 9, 10, 11, 12, 13, 14, 15)
            : BB_V_IO(v, T) : [x1] "v"(x1), [x2] "v"(x2), [u1] "v"(u1), [u2] "v"(u2));
}

// periodic correction, rows t .. t+7: x += z0 c0 (+ z1 c1)
#define BB_ZK1(v, lane) BB_FMAC(v, "z0", "c0", lane)
#define BB_ZK2(v, lane) BB_FMAC(v, "z1", "c1", lane)

template <int T, int C>
__device__ __forceinline__ void rows8_correct(double (&v)[C], double c0, double z0)
{
    if constexpr (T / 8 % 2 == 0)
        asm("s_nop 1\n\t" BB_ROWS_UP(BB_ZK1, 0, 1, 2, 3, 4, 5, 6, 7)
            : BB_V_IO(v, T) : [c0] "v"(c0), [z0] "v"(z0));
    else
        asm("s_nop 1\n\t" BB_ROWS_UP(BB_ZK1, 8, 9, 10, 11, 12, 13, 14, 15)
            : BB_V_IO(v, T) : [c0] "v"(c0), [z0] "v"(z0));
}

template <int T, int C>
__device__ __forceinline__ void rows8_correct(double (&v)[C], double c0, double c1, double z0,
                                              double z1)
{
    if constexpr (T / 8 % 2 == 0)
        asm("s_nop 1\n\t" BB_ROWS_UP(BB_ZK1, 0, 1, 2, 3, 4, 5, 6, 7) BB_ROWS_UP(BB_ZK2, 0, 1, 2, 3, 4, 5, 6, 7)
            : BB_V_IO(v, T) : [c0] "v"(c0), [c1] "v"(c1), [z0] "v"(z0), [z1] "v"(z1));
    else
        asm("s_nop 1\n\t" BB_ROWS_UP(BB_ZK1, 8, 9, 10, 11, 12, 13, 14, 15) BB_ROWS_UP(BB_ZK2, 8, 9, 10, 11, 12, 13, 14, 15)
            : BB_V_IO(v, T) : [c0] "v"(c0), [c1] "v"(c1), [z0] "v"(z0), [z1] "v"(z1));
}

// Chain over the boundary states of four chunks, in place (the scans of a
// split group): state i = e_i + M_i state_{i-1}, lane LANE0 + i of
// each row holding M_i.  UP: e[0] follows (h1, h2); else the last does, down
// to e[0].
#define BB_UPK1(a, b, c, d)                                                                        \
    BB_FMAC("e0", "m0", "h1", a) BB_FMAC("e1", "m0", "e0", b) BB_FMAC("e2", "m0", "e1", c)         \
    BB_FMAC("e3", "m0", "e2", d)
#define BB_DOWNK1(a, b, c, d)                                                                      \
    BB_FMAC("e3", "m0", "h1", d) BB_FMAC("e2", "m0", "e3", c) BB_FMAC("e1", "m0", "e2", b)         \
    BB_FMAC("e0", "m0", "e1", a)
// (p, q) += M (x, y)
#define BB_AFF(p, q, x, y, lane)                                                                   \
    BB_FMAC(p, "m0", x, lane) BB_FMAC(q, "m2", x, lane) BB_FMAC(p, "m1", y, lane) BB_FMAC(q, "m3", y, lane)
#define BB_UPK2(a, b, c, d)                                                                        \
    BB_AFF("e0", "g0", "h1", "h2", a) BB_AFF("e1", "g1", "e0", "g0", b)                            \
    BB_AFF("e2", "g2", "e1", "g1", c) BB_AFF("e3", "g3", "e2", "g2", d)
#define BB_DOWNK2(a, b, c, d)                                                                      \
    BB_AFF("e3", "g3", "h1", "h2", d) BB_AFF("e2", "g2", "e3", "g3", c)                            \
    BB_AFF("e1", "g1", "e2", "g2", b) BB_AFF("e0", "g0", "e1", "g1", a)
#define BB_E_IO [e0] "+&v"(e[0]), [e1] "+&v"(e[1]), [e2] "+&v"(e[2]), [e3] "+&v"(e[3])
#define BB_CHAIN1(SEQ)                                                                             \
    asm("s_nop 1\n\t" SEQ : BB_E_IO : [m0] "v"(m[0]), [h1] "v"(h1))
#define BB_CHAIN2(SEQ)                                                                             \
    asm("s_nop 1\n\t" SEQ                                                                          \
        : BB_E_IO, [g0] "+&v"(g[0]), [g1] "+&v"(g[1]), [g2] "+&v"(g[2]), [g3] "+&v"(g[3])              \
        : [m0] "v"(m[0]), [m1] "v"(m[1]), [m2] "v"(m[2]), [m3] "v"(m[3]), [h1] "v"(h1), [h2] "v"(h2))

template <int K, bool UP, int LANE0>
__device__ __forceinline__ void chain4(double (&e)[4], double (&g)[4], const double (&m)[K * K],
                                       double h1, double h2)
{
#define BB_CHAIN_AT(a, b, c, d)                                                                    \
    do {                                                                                           \
        if constexpr (K == 1 && UP) BB_CHAIN1(BB_UPK1(a, b, c, d));                                \
        else if constexpr (K == 1) BB_CHAIN1(BB_DOWNK1(a, b, c, d));                               \
        else if constexpr (UP) BB_CHAIN2(BB_UPK2(a, b, c, d));                                     \
        else BB_CHAIN2(BB_DOWNK2(a, b, c, d));                                                     \
    } while (0)
    static_assert(LANE0 == 0 || LANE0 == 4 || LANE0 == 8 || LANE0 == 12, "first lane of the four");
    if constexpr (LANE0 == 0) BB_CHAIN_AT(0, 1, 2, 3);
    else if constexpr (LANE0 == 4) BB_CHAIN_AT(4, 5, 6, 7);
    else if constexpr (LANE0 == 8) BB_CHAIN_AT(8, 9, 10, 11);
    else BB_CHAIN_AT(12, 13, 14, 15);
#undef BB_CHAIN_AT
}

// body(integral_constant<int, t>) for t = 0, 8, .. C-8 (or down)
template <int C, int T = 0, typename F>
__device__ __forceinline__ void blocks8_up(F &&body)
{
    if constexpr (T < C) {
        body(std::integral_constant<int, T>{});
        blocks8_up<C, T + 8>(body);
    }
}

template <int C, int T = C - 8, typename F>
__device__ __forceinline__ void blocks8_down(F &&body)
{
    if constexpr (T >= 0) {
        body(std::integral_constant<int, T>{});
        blocks8_down<C, T - 8>(body);
    }
}

#undef BB_DPP
#undef BB_FMAC
#undef BB_SCALE
#undef BB_ROWS_UP
#undef BB_V_IN
#undef BB_V_IO
#undef BB_P1K1
#undef BB_P1K2
#undef BB_P2K1
#undef BB_P2K2
#undef BB_P3K1
#undef BB_P3K2
#undef BB_ZK1
#undef BB_ZK2
#undef BB_UPK1
#undef BB_DOWNK1
#undef BB_AFF
#undef BB_UPK2
#undef BB_DOWNK2
#undef BB_E_IO
#undef BB_CHAIN1
#undef BB_CHAIN2

}  // namespace
}  // namespace bb
