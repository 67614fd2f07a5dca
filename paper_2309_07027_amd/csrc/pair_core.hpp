// pair_core.hpp -- per-lane core of the pair walk of the generalized BB/FG
// permanent (arXiv:2309.07027, Eq. bbfgrepeated).
//
// The product of two column sums is a quadratic polynomial of the sign counts.
// Over four binary digits (16 addends) it is fixed by its value y at the first
// of them, the four differences D_k = y(k flipped) - y, and the six constants
//   K_kl = d_k1 d_l2 + d_l1 d_k2      (d_kj = -2 a_kj),
// which depend on the two columns only.  Every further value is one complex
// addition, and keeping the differences up to date 11 more: 26 complex additions
// give a pair's 16 products, where updating two sums and multiplying them at
// each addend takes 32 complex additions and 16 complex products.  Per addend
// and pair the pair walk issues 4 FP64 instructions for the running product
// over the pairs, 3.25 for the values and 1 for y and the D_k, against 12.
//
// The sums b_1, b_2 and the D_k are linear in the sign counts of the other
// rows, so each is the sum of a part that depends on the lane (lane and high
// digits; in LDS, shared by the wavefronts of a work group) and a part that is
// the same for every lane (the "mid" digits; a table read by scalar loads).
// Nothing is carried from one block of 16 addends to the next but the sums of
// the results, so no column sum drifts.
//
// Bound by FP64 issue: 133 VALU instructions a pair and block, 132 of them FP64,
// 89 % of the issue slots used at 30 columns.  16 wavefronts of at most 128
// registers share one unit's lane parts (6 KB a pair); 12 of 160 registers, with
// the lane parts fetched a pair ahead, measured 3 % slower.  Measured against
// the walk of walk_core.hpp: 30 columns, 2^29 addends, 2.98 -> 2.09 ms (kernel);
// 14 columns of multiplicity 2, 2^27 addends, 0.50 -> 0.32 ms; 4096 items of
// 23-24 photons 37.6 -> 29.1 ms.
//
// A value formed from differences carries an error of about 2^-53 of the largest
// of its pair's 16 products, where a product of two column sums has one relative
// to the sums.  The two are alike while the inner rows' entries are of the size
// of the others.  Where they dominate a column their signs can cancel there, and
// other columns can make up for the small product: with two rows of 1e4 that
// cancel in two columns and add up in two others the differences lose four
// digits, and the estimate, which is made of the addends, does not show it.  Such
// a permanent (differences_serve) has its products formed from the column sums
// (pair_block_direct), at the plain walk's 12 instructions an addend and pair:
// 30 columns, 2^29 addends, 3.13 ms a call instead of 2.24 (the plain walk 3.04-
// 3.12); 512 items of 23 photons 10.9 instead of 7.7 ms (10.0).  Fetching a pair's
// scalars a pair ahead made no difference there.
//
// Compiled by hipcc for the kernels and by a host compiler for the CPU
// emulation used in tests, as walk_core.hpp.
#pragma once

#include <type_traits>

#include "walk_core.hpp"

#if defined(__HIP_DEVICE_COMPILE__)
#define BBFG_SCHED_BARRIER() __builtin_amdgcn_sched_barrier(0)
#else
#define BBFG_SCHED_BARRIER()
#endif

namespace bbfg {

struct alignas(16) cpx {
    double r, i;
};

// a b - c, written over a on the device: the compiler's own choice, a multiply-
// accumulate into c's register, costs a register move per product at every turn
// of the loop over the pairs
BBFG_FN double fmar_sub(double a, double b, double c)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm("v_fma_f64 %0, %0, %1, -%2" : "+v"(a) : "v"(b), "v"(c));
    return a;
#else
    return fmar(a, b, -c);
#endif
}

BBFG_FN cpx cadd(cpx a, cpx b) { return {a.r + b.r, a.i + b.i}; }
BBFG_FN cpx csub(cpx a, cpx b) { return {a.r - b.r, a.i - b.i}; }
BBFG_FN cpx cadd(cpx a, const double* k) { return {a.r + k[0], a.i + k[1]}; }
BBFG_FN cpx cmul(cpx a, cpx b)
{
    cpx c;
    cmul<double>(a.r, a.i, b.r, b.i, c.r, c.i);
    return c;
}
// acc + a b, a uniform
BBFG_FN cpx cfma(cpx a, cpx b, cpx acc)
{
    return {fmar(-a.i, b.i, fmar(a.r, b.r, acc.r)), fmar(a.i, b.r, fmar(a.r, b.i, acc.i))};
}

// p *= v, with the real part written last so that it can stay in its register
BBFG_FN void cmul_into(cpx& p, cpx v)
{
    const double t = p.i * v.i;
    p.i = p.i * v.r;
    p.i = fmar(p.r, v.i, p.i);
    p.r = fmar_sub(p.r, v.r, t);
}

// Whether the inner rows (inner_rows: a bit each) leave a column of r kept rows
// to differences; mag(k) is the modulus |re| + |im| of row k's entry.  At least
// half of the other entries have to reach 1/16 of the largest inner one: with
// rows 16 times the others that cancel as above the differences are off by as
// much as the plain walk, with 64 times by ten times as much.  Entries of like
// distribution (Gaussian, Haar) fail it in fewer than one column of a million
// beside ten other rows, in 2e-5 of the columns beside five, 3e-4 beside three.
constexpr double kInnerRange = 16.0;
template <typename Mag>
BBFG_FN bool differences_serve(int r, uint64_t inner_rows, Mag mag)
{
    double top = 0.0;
    int inner = 0, near = 0;
    for (uint64_t rows = inner_rows; rows; rows &= rows - 1, ++inner) {
        const double m = mag(__builtin_ctzll(rows));
        top = m > top ? m : top;
    }
#pragma unroll 8
    for (int k = 0; k < r; ++k) {  // loads first: nothing here depends on the row before
        const double m = kInnerRange * mag(k);
        near += (int)((inner_rows >> k & 1u) == 0) & (int)(m >= top);
    }
    const int others = r - inner;
    return 2 * near >= others;
}

// The pair's column sums and differences: slot 0, 1: b_1, b_2; slot 2 + k: D_k.
struct PairSums {
    cpx s[kPairSlots];
};

// d_kj = -2 a_kj of inner digit k and column j of pair p; a pair whose second
// column lies beyond the matrix (odd n) is filled up with a column that is 1.
template <typename Ptr>
BBFG_FN void pair_steps(const PairDesc& d, Ptr a, uint32_t p, int k, cpx& d1, cpx& d2)
{
    Ptr row = a + 2 * ((size_t)d.inner[k] * d.n + 2 * p);
    d1 = {-2.0 * row[0], -2.0 * row[1]};
    d2 = {0.0, 0.0};
    if (2 * p + 1 < (uint32_t)d.n) d2 = {-2.0 * row[2], -2.0 * row[3]};
}

// Lane part of pair p: coef(k) is the coefficient of kept row k for this lane
// (its largest value for the mid and inner rows).
template <typename Coef>
BBFG_FN void pair_seed(const PairDesc& d, kptr<double> a, uint32_t p, Coef coef, PairSums& out)
{
    const bool full = 2 * p + 1 < (uint32_t)d.n;
    const int second = full ? 2 : 0;  // the column beyond an odd n is not read
    cpx b1 = {0.0, 0.0}, b2 = {0.0, 0.0};
    kptr<double> row = a + 4 * (size_t)p;
#pragma unroll 4
    for (int k = 0; k < d.r; ++k) {
        const double c = coef(k);
        b1 = {fmar(c, row[0], b1.r), fmar(c, row[1], b1.i)};
        b2 = {fmar(c, row[second], b2.r), fmar(c, row[second + 1], b2.i)};
        row = row + 2 * (size_t)d.n;
    }
    if (!full) b2 = {1.0, 0.0};
    out.s[0] = b1;
    out.s[1] = b2;
#pragma unroll
    for (int k = 0; k < kPairBits; ++k) {
        cpx d1, d2;
        pair_steps(d, a, p, k, d1, d2);
        out.s[2 + k] = cfma(d1, b2, cfma(d2, b1, cmul(d1, d2)));
    }
}

// Uniform part of pair p at mid position h: the mid rows' share of the sums.
BBFG_FN void pair_mid(const PairDesc& d, kptr<RowInfo> ri, const double* a, uint32_t p, uint32_t h, double* out)
{
    const bool full = 2 * p + 1 < (uint32_t)d.n;
    cpx b1 = {0.0, 0.0}, b2 = {0.0, 0.0};
    for (int i = 0; i < d.mids; ++i) {
        const int k = d.mid_row[i];
        const double c = -2.0 * (double)((h / ri[k].stride) % ri[k].radix);
        const double* row = a + 2 * ((size_t)k * d.n + 2 * p);
        b1 = {fmar(c, row[0], b1.r), fmar(c, row[1], b1.i)};
        if (full) b2 = {fmar(c, row[2], b2.r), fmar(c, row[3], b2.i)};
    }
    out[0] = b1.r;
    out[1] = b1.i;
    out[2] = b2.r;
    out[3] = b2.i;
#pragma unroll
    for (int k = 0; k < kPairBits; ++k) {
        cpx d1, d2;
        pair_steps(d, a, p, k, d1, d2);
        const cpx u = cfma(d1, b2, cmul(d2, b1));
        out[4 + 2 * k] = u.r;
        out[5 + 2 * k] = u.i;
    }
}

// The six constants K_01, K_02, K_03, K_12, K_13, K_23 of pair p.
BBFG_FN void pair_constants(const PairDesc& d, const double* a, uint32_t p, double* out)
{
    cpx d1[kPairBits], d2[kPairBits];
    for (int k = 0; k < kPairBits; ++k) pair_steps(d, a, p, k, d1[k], d2[k]);
    int q = 0;
    for (int k = 0; k < kPairBits; ++k)
        for (int l = k + 1; l < kPairBits; ++l, ++q) {
            const cpx v = cfma(d1[k], d2[l], cmul(d1[l], d2[k]));
            out[2 * q] = v.r;
            out[2 * q + 1] = v.i;
        }
}

// Signed weight prod (-1)^Delta C(M', Delta) over the mid rows at position h.
BBFG_FN double pair_mid_weight(const PairDesc& d, kptr<RowInfo> ri, const double* binom, uint32_t h)
{
    double w = 1.0;
    for (int i = 0; i < d.mids; ++i) {
        const int k = d.mid_row[i];
        const uint32_t delta = (h / ri[k].stride) % ri[k].radix;
        const double b = ri[k].mp <= 1 ? 1.0 : binom[ri[k].mp * kBinomDim + (int)delta];
        w *= (delta & 1u) ? -b : b;
    }
    return w;
}

// Sign count of a lane or high row, and its coefficient base - 2 Delta; mid and
// inner rows are at Delta = 0.
BBFG_FN int pair_coef(const RowInfo& x, uint32_t lane_idx, uint32_t high)
{
    uint32_t delta = 0;
    if (x.kind == ROW_LANE) delta = (lane_idx / x.stride) % x.radix;
    else if (x.kind == ROW_HIGH) delta = (high / x.stride) % x.radix;
    return x.base - 2 * (int)delta;
}

// Weight (-1)^Delta C(M', Delta) of a lane or high row at coefficient c.
BBFG_FN double pair_row_weight(const RowInfo& x, const double* binom, int c)
{
    if (x.kind != ROW_LANE && x.kind != ROW_HIGH) return 1.0;
    const int delta = (x.base - c) / 2;
    const double b = x.mp <= 1 ? 1.0 : binom[x.mp * kBinomDim + delta];
    return (delta & 1) ? -b : b;
}

// One pair's 16 values, multiplied into the running products P (or, FIRST,
// becoming them).  K: the pair's constants.
template <bool FIRST>
BBFG_FN void pair_block(const PairSums& q, const double* K, cpx* P)
{
    auto put = [&](int x, cpx v) {
        if constexpr (FIRST) P[x] = v;
        else cmul_into(P[x], v);
    };
    const double *K01 = K, *K02 = K + 2, *K03 = K + 4, *K12 = K + 6, *K13 = K + 8, *K23 = K + 10;
    cpx v[4];
    v[0] = cmul(q.s[0], q.s[1]);
    v[1] = cadd(v[0], q.s[2]);
    v[2] = cadd(v[0], q.s[3]);
    v[3] = cadd(v[1], cadd(q.s[3], K01));
    const cpx e1 = cadd(q.s[4], K02), f1 = cadd(q.s[5], K03);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        // D_2 and D_3 with digits 0 and 1 at c
        const cpx e = c == 0 ? q.s[4] : c == 1 ? e1 : c == 2 ? cadd(q.s[4], K12) : cadd(e1, K12);
        const cpx f = c == 0 ? q.s[5] : c == 1 ? f1 : c == 2 ? cadd(q.s[5], K13) : cadd(f1, K13);
        const cpx u = cadd(v[c], e);
        put(c, v[c]);
        put(4 + c, u);
        put(8 + c, cadd(v[c], f));
        put(12 + c, cadd(u, cadd(f, K23)));
    }
}

// The same values as products of the column sums c1, c2, walked over the inner
// digits in Gray order; a1, a2: the inner rows' entries.
template <bool FIRST>
BBFG_FN void pair_block_direct(cpx c1, cpx c2, const cpx* a1, const cpx* a2, cpx* P)
{
    int x = 0;
#pragma unroll
    for (int g = 0; g < kPairBlock; ++g) {
        if (g > 0) {
            const int k = __builtin_ctz((unsigned)g);
            x ^= 1 << k;
            const double f = x >> k & 1 ? -2.0 : 2.0;
            c1 = {fmar(f, a1[k].r, c1.r), fmar(f, a1[k].i, c1.i)};
            c2 = {fmar(f, a2[k].r, c2.r), fmar(f, a2[k].i, c2.i)};
        }
        const cpx v = cmul(c1, c2);
        if constexpr (FIRST) P[x] = v;
        else cmul_into(P[x], v);
    }
}

// Sum of the 16 products with the inner digits' signs, and of their moduli |re| + |im|.
BBFG_FN void pair_block_sum(const cpx* P, double& sr, double& si, double& sa)
{
    double r[kPairBlock], i[kPairBlock], a[kPairBlock];
#pragma unroll
    for (int x = 0; x < kPairBlock; ++x) {
        const bool odd = ((x ^ (x >> 1) ^ (x >> 2) ^ (x >> 3)) & 1) != 0;
        r[x] = odd ? -P[x].r : P[x].r;
        i[x] = odd ? -P[x].i : P[x].i;
        a[x] = __builtin_fabs(P[x].r) + __builtin_fabs(P[x].i);
    }
#pragma unroll
    for (int s = 1; s < kPairBlock; s *= 2) {
#pragma unroll
        for (int x = 0; x < kPairBlock; x += 2 * s) {
            r[x] += r[x + s];
            i[x] += i[x + s];
            a[x] += a[x + s];
        }
    }
    sr = r[0];
    si = i[0];
    sa = a[0];
}

// A lane's sums over the unit's wavefronts, in double-double as those over lanes
// and units are (a wavefront's own cover at most 512 addends): (r, i, m, w) starts
// as the first wavefront's, get(v, r, i, m, w) reads another's; each wavefront has
// a share w of the lane's weight.
template <typename Get>
BBFG_FN void pair_join(Get get, double r, double i, double m, double w, ddv& sr, ddv& si, double& sa)
{
    sr = {r, 0.0};
    si = {i, 0.0};
#pragma unroll
    for (int v = 1; v < kPairWaves; ++v) {
        double vr, vi, vm, vw;
        get(v, vr, vi, vm, vw);
        sr = dd_add(sr, vr);
        si = dd_add(si, vi);
        m += vm;
        w *= vw;
    }
    sr = dd_mul(sr, w);
    si = dd_mul(si, w);
    sa = __builtin_fabs(w) * m;
}

// What one pair of a block reads by scalar loads: its uniform part and constants.
struct PairInputs {
    double u[2 * kPairSlots];
    double k[2 * kPairConsts];
};

BBFG_FN void pair_fetch(kptr<double> U, kptr<double> K, PairInputs& in)
{
#pragma unroll
    for (int i = 0; i < 2 * kPairSlots; ++i) in.u[i] = U[i];
#pragma unroll
    for (int i = 0; i < 2 * kPairConsts; ++i) in.k[i] = K[i];
}

// A block's products, raised and added: the sums grow by the weighted ones.
template <bool POW>
BBFG_FN void pair_close(const PairDesc& d, cpx* P, double w, double& accr, double& acci, double& acca)
{
    if constexpr (POW) {
#pragma unroll
        for (int x = 0; x < kPairBlock; ++x) cpow_uint<double>(P[x].r, P[x].i, d.col_pow);
    }
    double sr, si, sa;
    pair_block_sum(P, sr, si, sa);
    accr = fmar(w, sr, accr);
    acci = fmar(w, si, acci);
    acca = fmar(__builtin_fabs(w), sa, acca);
}

// One lane's walk over mid positions [h0, h1): sum of the weighted addends and
// of their magnitudes.  lane(p, out) reads the lane part of pair p.  POW: every
// column has multiplicity d.col_pow, the product is (prod_j c_j)^col_pow.
// The next pair's scalar loads are issued before a pair's arithmetic (the last
// ones read past the walked positions, into the tables that follow).
template <bool POW, typename Lane>
BBFG_FN void pair_walk(const PairDesc& d, kptr<double> mid, kptr<double> weight, kptr<double> consts, uint32_t h0,
                       uint32_t h1, Lane lane, double& out_r, double& out_i, double& out_a)
{
    const uint32_t np = (uint32_t)d.np;
    double accr = 0.0, acci = 0.0, acca = 0.0;
    kptr<double> U = mid + (size_t)h0 * np * (2 * kPairSlots);
    PairInputs in;
    if (h0 < h1) pair_fetch(U, consts, in);
    for (uint32_t h = h0; h < h1; ++h) {
        cpx P[kPairBlock];
        const double w = weight[h];
        auto step = [&](auto first, uint32_t p, uint32_t next) {
            PairSums q;
            double k[2 * kPairConsts];
            lane(p, q);
#pragma unroll
            for (int s = 0; s < kPairSlots; ++s) q.s[s] = {q.s[s].r + in.u[2 * s], q.s[s].i + in.u[2 * s + 1]};
#pragma unroll
            for (int i = 0; i < 2 * kPairConsts; ++i) k[i] = in.k[i];
            U = U + 2 * kPairSlots;
            pair_fetch(U, consts + next * (2 * kPairConsts), in);
            BBFG_SCHED_BARRIER();
            pair_block<decltype(first)::value>(q, k, P);
            BBFG_SCHED_BARRIER();
        };
        step(std::true_type{}, 0u, np > 1 ? 1u : 0u);
        for (uint32_t p = 1; p < np; ++p) step(std::false_type{}, p, p + 1 < np ? p + 1 : 0u);
        pair_close<POW>(d, P, w, accr, acci, acca);
    }
    out_r = accr;
    out_i = acci;
    out_a = acca;
}

// The same walk with the products formed from the column sums; a: the kept rows.
template <bool POW, typename Lane>
BBFG_FN void pair_walk_direct(const PairDesc& d, kptr<double> a, kptr<double> mid, kptr<double> weight, uint32_t h0,
                              uint32_t h1, Lane lane, double& out_r, double& out_i, double& out_a)
{
    const uint32_t np = (uint32_t)d.np;
    double accr = 0.0, acci = 0.0, acca = 0.0;
    kptr<double> U = mid + (size_t)h0 * np * (2 * kPairSlots);
    for (uint32_t h = h0; h < h1; ++h) {
        cpx P[kPairBlock];
        const double w = weight[h];
        auto step = [&](auto first, uint32_t p) {
            cpx a1[kPairBits], a2[kPairBits], c[2];
#pragma unroll
            for (int k = 0; k < kPairBits; ++k) {
                kptr<double> row = a + 2 * ((size_t)d.inner[k] * d.n + 2 * p);
                a1[k] = {row[0], row[1]};
                a2[k] = {0.0, 0.0};
                if (2 * p + 1 < (uint32_t)d.n) a2[k] = {row[2], row[3]};
            }
            lane(p, c);
            c[0] = {c[0].r + U[0], c[0].i + U[1]};
            c[1] = {c[1].r + U[2], c[1].i + U[3]};
            U = U + 2 * kPairSlots;
            pair_block_direct<decltype(first)::value>(c[0], c[1], a1, a2, P);
        };
        step(std::true_type{}, 0u);
        for (uint32_t p = 1; p < np; ++p) step(std::false_type{}, p);
        pair_close<POW>(d, P, w, accr, acci, acca);
    }
    out_r = accr;
    out_i = acci;
    out_a = acca;
}

}  // namespace bbfg
