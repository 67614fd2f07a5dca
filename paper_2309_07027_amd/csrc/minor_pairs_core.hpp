// minor_pairs_core.hpp -- per-lane core of the leave-one-column-out walk over
// pairs of columns (the Laplace minors of the Clifford & Clifford step, Sec. 4,
// with Eq. bbfgrepeated; arXiv:2309.07027).
//
// Four wavefronts share the addends; each owns NP pairs of columns.  With
// Z_p = w prod_{p' != p} c_1 c_2 (pair p'), the minors without the columns of
// pair p are sum Z_p c_2 and sum Z_p c_1.  Per addend a wavefront forms its
// pairs' products, hands their product to the other three through LDS, and gets
// the Z_p of its pairs from the other three products and its own.
//
// One binary digit x is taken two addends at a time.  A pair's product is
// c_1 c_2 = y + x D with D linear in the sign counts of the other rows, so the
// second addend's costs one complex addition, and with c_2 = b_2 + x d_2
//   sum_x Z c_2 = b_2 sum_x Z + d_2 Z(1):
// the multiply-accumulates with the column sums are shared by the two addends,
// and the d terms are added once at a unit's end.
//
// A second binary digit, at four pairs a wavefront, makes a step of four addends
// that shares the sums and the multiply-accumulates once more (MinorLane).
//
// Bound by FP64 issue: 23.6 FP64 instructions per pair and addend with one digit
// (189 a step of two addends and four pairs, 11 other vector ones), 21.9 with
// two (351 a step of four addends), and about 40 registers per pair, so up to 40
// columns fit two wavefronts per SIMD without spills or accumulation registers
// (up to 24 columns three).  One wavefront for all columns, walk_minors_unit,
// issues 38 a pair and addend at 30 columns and 54 at 36, where half are register
// moves.  Measured (kernel): 24 columns, 2^22 addends, 0.193 -> 0.087 ms; 30
// columns, 2^28, 4.96 -> 3.1 ms; 35 columns, 34 photons at random, 12.5 -> 6.2 ms.
//
// Where an inner row dominates a column the products at x = 1 and x' = 1 are formed
// from the column sums there, not from differences, and each addend's Z is
// accumulated with its own column sums (DIRECT; the reason is pair_core.hpp's).
// The inner rows are then added to the sums of the others at each step, so that
// they leave no rounding of their size in a sum where they cancel.
//
// Compiled by hipcc for the kernel and by a host compiler for the CPU emulation.
#pragma once

#include "pair_core.hpp"

namespace bbfg {

// acc + a b
BBFG_FN void cmac(cpx& acc, cpx a, cpx b) { acc = cfma(a, b, acc); }
BBFG_FN cpx cmul_uniform(cpx a, double s) { return {a.r * s, a.i * s}; }

// DIGITS: inner binary digits, 1 or 2.  With a second digit x', taken as a second
// half of the step, b_1 and b_2 serve four addends: y and D move to x' = 1 by
// their differences (E, and the constant K of the two digits), and the sums over
// both halves are accumulated at once.  DIRECT: no differences, and the column sums
// held are those without the inner rows.
template <int NP, int DIGITS, bool DIRECT>
struct MinorLane {
    cpx b1[NP], b2[NP];                // column sums at x = x' = 0
    cpx D[DIRECT ? 1 : NP];            // difference of the product in x
    cpx E[DIGITS > 1 && !DIRECT ? NP : 1];  // its difference in x'
    cpx y[NP], v[NP];                  // product at x = 0 and x = 1 of the current half
    cpx acc1[NP], acc2[NP];            // sums of Z c_2, Z c_1
    cpx G[DIRECT ? 1 : NP];            // sum of the signed Z at x = 1
    cpx F[DIGITS > 1 && !DIRECT ? NP : 1];  // the same at x' = 1
    cpx S[DIGITS > 1 && !DIRECT ? NP : 1];  // the first half's sums

    // doubles per pair of a step: the changes of b_1, b_2, D (and E)
    static constexpr int kStep = 2 * (2 + DIGITS);

    // products over neighbouring pairs at one x
    static constexpr int H = (NP + 1) / 2;
    struct Half {
        cpx m[H];                      // of pairs 2i, 2i + 1
        cpx all;
    } half[2];

    BBFG_FN void clear()
    {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            acc1[p] = acc2[p] = {0.0, 0.0};
            if constexpr (!DIRECT) G[p] = {0.0, 0.0};
            if constexpr (DIGITS > 1 && !DIRECT) F[p] = {0.0, 0.0};
        }
    }

    static BBFG_FN void digit_step(kptr<double> row, int p, cpx& d1, cpx& d2)
    {
        d1 = {-2.0 * row[4 * p], -2.0 * row[4 * p + 1]};
        d2 = {-2.0 * row[4 * p + 2], -2.0 * row[4 * p + 3]};
    }

    // Column sums at one position: coef(k) is kept row k's coefficient, a points
    // at this wavefront's columns of row 0 (rows `ld` doubles apart, columns past
    // the matrix zero; `cols` of the wavefront's 2 NP columns are real).  The last
    // kept row is x's, the one before it x' 's, at coefficient +1.
    template <typename Coef>
    BBFG_FN void seed(kptr<double> a, size_t ld, int r, int cols, Coef coef)
    {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            b1[p] = {2 * p < cols ? 0.0 : 1.0, 0.0};
            b2[p] = {2 * p + 1 < cols ? 0.0 : 1.0, 0.0};
        }
        kptr<double> row = a;
        for (int k = 0; k < (DIRECT ? r - DIGITS : r); ++k) {
            const double c = coef(k);
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                b1[p] = {fmar(c, row[4 * p], b1[p].r), fmar(c, row[4 * p + 1], b1[p].i)};
                b2[p] = {fmar(c, row[4 * p + 2], b2[p].r), fmar(c, row[4 * p + 3], b2[p].i)};
            }
            if (k + 1 < r) row = row + (int64_t)ld;
        }
        if constexpr (DIRECT) return;
#pragma unroll
        for (int p = 0; p < (DIRECT ? 0 : NP); ++p) {
            cpx d1, d2;
            digit_step(row, p, d1, d2);
            D[p] = cfma(d1, b2[p], cfma(d2, b1[p], cmul(d1, d2)));
            if constexpr (DIGITS > 1) {
                digit_step(row + -(int64_t)ld, p, d1, d2);
                E[p] = cfma(d1, b2[p], cfma(d2, b1[p], cmul(d1, d2)));
            }
        }
    }

    // One step of the Gray walk: s holds per pair the changes.
    BBFG_FN void advance(const double* s)
    {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            b1[p] = cadd(b1[p], s + kStep * p);
            b2[p] = cadd(b2[p], s + kStep * p + 2);
            if constexpr (DIRECT) continue;
            D[p] = cadd(D[p], s + kStep * p + 4);
            if constexpr (DIGITS > 1) E[p] = cadd(E[p], s + kStep * p + 6);
        }
    }

    // b and f times a row's entry at e
    static BBFG_FN cpx joined(cpx b, double f, kptr<double> row, int e)
    {
        return {fmar(f, row[e], b.r), fmar(f, row[e + 1], b.i)};
    }
    // DIRECT: pair p's column sums at x' = 0 or 1 but for x's row
    template <bool SECOND>
    BBFG_FN void without_x(int p, kptr<double> inner, size_t ld, cpx& c1, cpx& c2) const
    {
        c1 = b1[p];
        c2 = b2[p];
        if constexpr (DIGITS > 1) {
            kptr<double> row = inner + -(int64_t)ld;
            c1 = joined(c1, SECOND ? -1.0 : 1.0, row, 4 * p);
            c2 = joined(c2, SECOND ? -1.0 : 1.0, row, 4 * p + 2);
        }
    }
    template <bool SECOND>
    BBFG_FN void direct_products(int p, kptr<double> inner, size_t ld)
    {
        cpx c1, c2;
        without_x<SECOND>(p, inner, ld, c1, c2);
        y[p] = cmul(joined(c1, 1.0, inner, 4 * p), joined(c2, 1.0, inner, 4 * p + 2));
        v[p] = cmul(joined(c1, -1.0, inner, 4 * p), joined(c2, -1.0, inner, 4 * p + 2));
    }

    // This wavefront's product at both x of the first half, or (after backward of
    // the first) of the second; K: K of the two digits; inner points at x's row.
    BBFG_FN void forward(kptr<double> inner, size_t ld)
    {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            if constexpr (DIRECT) {
                direct_products<false>(p, inner, ld);
            } else {
                y[p] = cmul(b1[p], b2[p]);
                v[p] = cadd(y[p], D[p]);
            }
        }
        products();
    }
    BBFG_FN void forward_second(const double* K, kptr<double> inner, size_t ld)
    {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            if constexpr (DIRECT) {
                direct_products<true>(p, inner, ld);
            } else {
                y[p] = cadd(y[p], E[p]);
                v[p] = cadd(cadd(y[p], D[p]), K + 2 * p);
            }
        }
        products();
    }

    BBFG_FN cpx value(int p, int x) const { return x ? v[p] : y[p]; }

    BBFG_FN void products()
    {
#pragma unroll
        for (int x = 0; x < 2; ++x) {
#pragma unroll
            for (int i = 0; i < H; ++i)
                half[x].m[i] = 2 * i + 1 < NP ? cmul(value(2 * i, x), value(2 * i + 1 < NP ? 2 * i + 1 : 0, x))
                                              : value(2 * i, x);
            half[x].all = half[x].m[0];
#pragma unroll
            for (int i = 1; i < H; ++i) half[x].all = cmul(half[x].all, half[x].m[i]);
        }
    }

    // z[p] = e prod of the other pairs' products at x
    BBFG_FN void others(int x, cpx e, cpx* z) const
    {
        const Half& h = half[x];
        cpx eh[H];  // e times the products of the other neighbour pairs
        if constexpr (H == 1) {
            eh[0] = e;
        } else if constexpr (H == 2) {
            eh[0] = cmul(e, h.m[1]);
            eh[1] = cmul(e, h.m[0]);
        } else {
            const cpx t = cmul(e, h.m[2]);
            eh[0] = cmul(t, h.m[1]);
            eh[1] = cmul(t, h.m[0]);
            eh[2] = cmul(e, cmul(h.m[0], h.m[1]));
        }
#pragma unroll
        for (int i = 0; i < H; ++i) {
            if (2 * i + 1 < NP) {
                z[2 * i] = cmul(eh[i], value(2 * i + 1 < NP ? 2 * i + 1 : 0, x));
                z[2 * i + 1 < NP ? 2 * i + 1 : 0] = cmul(eh[i], value(2 * i, x));
            } else {
                z[2 * i] = eh[i];
            }
        }
    }

    // Accumulates a half's two addends; e0, e1: the weight (its sign turned in the
    // second half) times the other wavefronts' products; x enters with (-1)^x.
    template <bool LAST>
    BBFG_FN void backward(cpx e0, cpx e1, kptr<double> inner, size_t ld)
    {
        cpx z0[NP], z1[NP];
        others(0, e0, z0);
        others(1, e1, z1);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            if constexpr (DIRECT) {
                cpx c1, c2;
                without_x<(DIGITS > 1 && LAST)>(p, inner, ld, c1, c2);
                cmac(acc1[p], joined(c2, 1.0, inner, 4 * p + 2), z0[p]);
                cmac(acc2[p], joined(c1, 1.0, inner, 4 * p), z0[p]);
                const cpx less = {-z1[p].r, -z1[p].i};
                cmac(acc1[p], joined(c2, -1.0, inner, 4 * p + 2), less);
                cmac(acc2[p], joined(c1, -1.0, inner, 4 * p), less);
                continue;
            }
            cpx s = csub(z0[p], z1[p]);
            G[p] = csub(G[p], z1[p]);
            if constexpr (DIGITS > 1) {
                if constexpr (!LAST) {
                    S[p] = s;
                } else {
                    F[p] = cadd(F[p], s);
                    s = cadd(s, S[p]);
                }
            }
            if constexpr (LAST) {
                cmac(acc1[p], s, b2[p]);
                cmac(acc2[p], s, b1[p]);
            }
        }
    }

    // The sums over the walked addends of the minors without columns 2p, 2p + 1;
    // inner points at x's row (x' 's lies ld doubles before).
    BBFG_FN void result(int p, kptr<double> inner, size_t ld, cpx& first, cpx& second) const
    {
        first = acc1[p];
        second = acc2[p];
        if constexpr (DIRECT) return;
        cpx d1, d2;
        digit_step(inner, p, d1, d2);
        first = cfma(d2, G[p], acc1[p]);
        second = cfma(d1, G[p], acc2[p]);
        if constexpr (DIGITS > 1) {
            digit_step(inner + -(int64_t)ld, p, d1, d2);
            first = cfma(d2, F[p], first);
            second = cfma(d1, F[p], second);
        }
    }
};

}  // namespace bbfg
