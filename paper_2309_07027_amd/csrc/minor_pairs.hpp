// minor_pairs.hpp -- gfx950 kernel of the leave-one-column-out walk over pairs
// of columns (minor_pairs_core.hpp), one translation unit per bucket.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.hpp"
#include "minor_pairs_core.hpp"
#include "walk_device.hpp"

namespace bbfg {

constexpr int kMinorThreads = kWave * kMinorWaves;

struct MinorShared {
    cpx prod[2][kMinorWaves][2][kWave];    // the wavefronts' products, two steps deep
    double mag[kMinorWaves][kWave];        // the wavefronts' moduli at a sampled position
    double weight[kMinorWaves][kWave];     // the wavefronts' shares of the lane weights
    int8_t coef[kMaxN][kWave];
    uint32_t next_unit;
};

// Coefficients of the kept rows at (block h, position t) into S.coef, each
// wavefront a share of the rows; returns the lane's weight over its lane and
// high digits (zero for idle lanes).
__device__ __forceinline__ double minor_coefs(const WalkArgs& A, const PermDesc& d, MinorShared& S, uint32_t lane,
                                              uint32_t wave, uint32_t lane_idx, bool valid, uint64_t h, uint32_t t)
{
    kptr<RowInfo> ri = kconst(A.rowinfo + d.rowinfo_off);
    double w = valid ? 1.0 : 0.0;
    for (int k = (int)wave; k < d.r; k += kMinorWaves) {
        RowInfo x;
        x.base = ri[k].base;
        x.kind = ri[k].kind;
        x.radix = ri[k].radix;
        x.stride = ri[k].stride;
        x.mp = ri[k].mp;
        uint32_t delta = 0;
        if (x.kind == ROW_LANE) {
            delta = (lane_idx / x.stride) % x.radix;
        } else if (x.kind == ROW_HIGH) {
            delta = digit_of(h, x.stride, x.radix);
        } else if (x.kind == ROW_LOW) {
            const uint32_t dg = (t / x.stride) % x.radix;
            const uint32_t q = t / (x.stride * x.radix);
            delta = (q & 1u) ? (x.radix - 1u - dg) : dg;
        }
        const int c = x.base - 2 * (int)delta;
        S.coef[k][lane] = (int8_t)c;
        w *= pair_row_weight(x, A.binom, c);
    }
    S.weight[wave][lane] = w;
    __syncthreads();
    w = S.weight[0][lane];
#pragma unroll
    for (int v = 1; v < kMinorWaves; ++v) w *= S.weight[v][lane];
    return w;
}

// One unit: the sums of the targets of this wavefront's NP pairs, from pair
// `first` on, over the unit's addends, then, for sampled units, the estimate of
// their magnitude sums (the modulus of the addend at the unit's last position,
// the inner digits at the lane's lowest bits, times the addends it stands for).
// The item's rows hold ROWNP pairs for each wavefront.
template <int NP, int DIGITS, int ROWNP, bool DIRECT>
__device__ __forceinline__ void minor_pairs_unit(const WalkArgs& A, const PermDesc& d, uint32_t u_local, MinorShared& S,
                                                 uint32_t wave, uint32_t first)
{
    uint32_t lane = threadIdx.x & (kWave - 1);
    // What is made of it is not held from unit to unit: for that the bucket of up to
    // 24 columns spilled, and a kernel that uses scratch memory costs a sampling step
    // 10 us (16 samples of 24 photons 1.51 -> 1.61 ms).
    asm volatile("" : "+v"(lane));
    const uint32_t upg = (uint32_t)d.units_per_group;
    const uint32_t g = u_local / upg;
    const uint32_t part = u_local - g * upg;
    const uint64_t base = d.span / upg;
    const uint32_t rem = (uint32_t)(d.span - base * upg);
    const uint64_t lin0 = (uint64_t)part * base + (part < rem ? part : rem);
    const uint64_t lin1 = lin0 + base + (part < rem ? 1u : 0u);
    uint32_t lane_idx = g * kWave + lane;
    const bool valid = lane_idx < d.lane_product;
    if (!valid) lane_idx = 0;

    constexpr int kCols = 2 * NP;
    const size_t ld = 4 * (size_t)ROWNP * kMinorWaves;              // doubles per kept row
    constexpr int kStep = MinorLane<NP, DIGITS, DIRECT>::kStep;
    const size_t step_ld = kStep * (size_t)ROWNP * kMinorWaves;     // doubles per step row
    kptr<double> a = kconst(A.a + 2 * d.a_off + first * 4);
    kptr<double> inner = a + (int64_t)((size_t)(d.r - 1) * ld);     // x's row
    kptr<double> steps = kconst(A.a2 + 2 * d.a2_off + first * kStep);
    kptr<TabEntry> tab = kconst(d.tab);
    const int cols = (int)d.n - 2 * (int)first;                     // real columns from there on (may be < 0)
    const uint32_t Q = d.Q;
    auto coef = [&](int k) { return (double)S.coef[k][lane]; };

    MinorLane<NP, DIGITS, DIRECT> L;
    L.clear();
    uint32_t buf = 0;
    // e of both x: the weight times the other wavefronts' products.  From its
    // column sums to here a wavefront is what the other three wait for, and has
    // little to issue; it goes before the accumulations of the other work groups'
    // wavefronts on its SIMD (25 columns, 2^24 addends, 0.156 -> 0.145 ms; 29 and
    // 30, 2^28, 2.28 -> 1.97 and 3.39 -> 3.25; 33 to 40 columns 2 to 5 % less).
    auto exchange = [&](double ws, cpx& e0, cpx& e1) {
        S.prod[buf][wave][0][lane] = L.half[0].all;
        S.prod[buf][wave][1][lane] = L.half[1].all;
        __syncthreads();
        const cpx(*const o0)[2][kWave] = &S.prod[buf][(wave + 1) % kMinorWaves];
        const cpx(*const o1)[2][kWave] = &S.prod[buf][(wave + 2) % kMinorWaves];
        const cpx(*const o2)[2][kWave] = &S.prod[buf][(wave + 3) % kMinorWaves];
        e0 = cmul_uniform(cmul(cmul((*o0)[0][lane], (*o1)[0][lane]), (*o2)[0][lane]), ws);
        e1 = cmul_uniform(cmul(cmul((*o0)[1][lane], (*o1)[1][lane]), (*o2)[1][lane]), ws);
        buf ^= 1u;
        __builtin_amdgcn_s_setprio(0);
        BBFG_SCHED_BARRIER();
    };
    // K of the two inner digits: the change of D when x' grows
    double K[DIGITS > 1 ? 2 * NP : 1];
    if constexpr (DIGITS > 1 && !DIRECT) {
        kptr<double> row = steps + (2 * (size_t)(d.r - 2) + 1) * step_ld;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            K[2 * p] = row[kStep * p + 4];
            K[2 * p + 1] = row[kStep * p + 5];
        }
    }
    for (uint64_t lin = lin0; lin < lin1;) {
        const uint64_t h = lin / Q;
        const uint32_t t0 = (uint32_t)(lin - h * Q);
        const uint64_t bend = (h + 1) * (uint64_t)Q;
        const uint32_t t1 = (uint32_t)(((lin1 < bend) ? lin1 : bend) - h * Q);
        const double w = minor_coefs(A, d, S, lane, wave, lane_idx, valid, h, t0);
        L.seed(a, ld, d.r, cols, coef);
        double ws = w * tab[t0].s;
        uint32_t next_row = t0 + 1 < t1 ? uniform_u32(tab[t0 + 1].row) : 0u;
        for (uint32_t t = t0; t < t1; ++t) {
            cpx e0, e1;
            kptr<double> here = inner;
            if constexpr (DIRECT) {
                // read the inner rows anew each step: held over the loop they take
                // registers that then spill
                int32_t zero = 0;
                asm volatile("" : "+s"(zero));
                here = inner + zero;
            }
            __builtin_amdgcn_s_setprio(1);
            BBFG_SCHED_BARRIER();
            L.forward(here, ld);
            exchange(ws, e0, e1);
            if constexpr (DIGITS > 1) {
                L.template backward<false>(e0, e1, here, ld);
                __builtin_amdgcn_s_setprio(1);
                BBFG_SCHED_BARRIER();
                L.forward_second(K, here, ld);
                exchange(-ws, e0, e1);
            }
            // the next step's changes are fetched under the rest of this step (not
            // earlier: a wait for LDS data waits for scalar loads as well); after
            // the last step they are row 0's, and go into sums that are seeded anew
            // (without differences registers are short, and the fetch follows that rest)
            BBFG_SCHED_BARRIER();
            if constexpr (DIRECT) {
                L.template backward<true>(e0, e1, here, ld);
                BBFG_SCHED_BARRIER();
            }
            double s[kStep * NP];
            kptr<double> row = steps + (size_t)next_row * step_ld;
#pragma unroll
            for (int i = 0; i < kStep * NP; ++i) s[i] = row[i];
            ws = w * tab[t + 1 < t1 ? t + 1 : t].s;
            next_row = uniform_u32(tab[t + 2 < t1 ? t + 2 : t].row);
            BBFG_SCHED_BARRIER();
            if constexpr (!DIRECT) L.template backward<true>(e0, e1, here, ld);
            L.advance(s);
        }
        lin += (uint64_t)(t1 - t0);
        __syncthreads();  // the coefficients and weights may be overwritten
    }
    const uint64_t slot = d.part_base + (uint64_t)u_local * d.targets + 2 * first;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        cpx m1, m2;
        L.result(p, inner, ld, m1, m2);
        if (2 * p < cols) store_partial_sums_all_lanes(A.partials, slot + 2 * p, m1.r, m1.i);
        if (2 * p + 1 < cols) store_partial_sums_all_lanes(A.partials, slot + 2 * p + 1, m2.r, m2.i);
    }
    const uint32_t every = d.mag_every;
    if (part % every != 0) {
#pragma unroll
        for (int j = 0; j < kCols; ++j)
            if (j < cols) A.partials[(slot + j) * kPartialDoubles + 4] = 0.0;
        return;
    }
    const uint32_t reps = (upg - part < every) ? upg - part : every;
    const uint64_t hl = (lin1 - 1) / Q;
    const uint32_t tl = (uint32_t)(lin1 - 1 - hl * Q);
    const double w = minor_coefs(A, d, S, lane, wave, lane_idx, valid, hl, tl);
    L.seed(a, ld, d.r, cols, coef);
    // moduli of the column sums, and their product
    double mod[kCols], own = 1.0;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        cpx c1 = L.b1[p], c2 = L.b2[p];
#pragma unroll
        for (int i = 0; i < DIGITS; ++i) {
            const double x = (lane >> i & 1u) ? (DIRECT ? -1.0 : -2.0) : (DIRECT ? 1.0 : 0.0);
            kptr<double> row = inner + -(int64_t)((size_t)i * ld);
            c1 = {fmar(x, row[4 * p], c1.r), fmar(x, row[4 * p + 1], c1.i)};
            c2 = {fmar(x, row[4 * p + 2], c2.r), fmar(x, row[4 * p + 3], c2.i)};
        }
        mod[2 * p] = __builtin_sqrt(fmar(c1.r, c1.r, c1.i * c1.i));
        mod[2 * p + 1] = __builtin_sqrt(fmar(c2.r, c2.r, c2.i * c2.i));
        own *= mod[2 * p] * mod[2 * p + 1];
    }
    S.mag[wave][lane] = own;
    __syncthreads();
    double lead = (double)(1 << DIGITS) * (double)(lin1 - lin0) * (double)reps * __builtin_fabs(w * tab[tl].s);
#pragma unroll
    for (int v = 1; v < kMinorWaves; ++v) lead *= S.mag[(wave + v) % kMinorWaves][lane];
    // leave-one-out products: no division, so zero moduli are harmless
    double pre[kCols];
    pre[0] = lead;
#pragma unroll
    for (int j = 1; j < kCols; ++j) pre[j] = pre[j - 1] * mod[j - 1];
    double suffix = 1.0;
#pragma unroll
    for (int j = kCols - 1; j >= 0; --j) {
        if (j < cols) store_partial_mag_all_lanes(A.partials, slot + j, pre[j] * suffix);
        suffix *= mod[j];
    }
}

// The wavefronts of a work group meet at the same barriers whether they own NP
// pairs or NP - 1: all that is walked is the unit's.
template <int NP, int DIGITS, bool DIRECT>
__device__ __forceinline__ void minor_pairs_share(const WalkArgs& A, const PermDesc& d, uint32_t u, MinorShared& S,
                                                  uint32_t wave)
{
    const uint32_t full = (uint32_t)minor_full_waves(d.n);
    if constexpr (NP > kMinorMinPairs) {
        if (wave >= full) {
            minor_pairs_unit<NP - 1, DIGITS, NP, DIRECT>(A, d, u, S, wave, wave * (NP - 1) + full);
            return;
        }
    }
    minor_pairs_unit<NP, DIGITS, NP, DIRECT>(A, d, u, S, wave, wave * NP);
}

template <int NPMIN, int NPMAX, bool DIRECT>
__device__ __forceinline__ void dispatch_minor_pairs(const WalkArgs& A, const PermDesc& d, uint32_t u, MinorShared& S,
                                                     uint32_t wave)
{
    if constexpr (NPMIN <= NPMAX) {
        if (minor_pairs_per_wave(d.n) == NPMIN) {
            if constexpr (NPMIN == kMinorTwoDigits) {
                if (d.col_pow == 2) {
                    minor_pairs_share<NPMIN, 2, DIRECT>(A, d, u, S, wave);
                    return;
                }
            }
            minor_pairs_share<NPMIN, 1, DIRECT>(A, d, u, S, wave);
        } else dispatch_minor_pairs<NPMIN + 1, NPMAX, DIRECT>(A, d, u, S, wave);
    }
}

// Persistent work groups of four wavefronts pull units from a counter.
template <int NPMAX>
__global__ __launch_bounds__(kMinorThreads) __attribute__((amdgpu_waves_per_eu(NPMAX <= 3 ? 3 : 2))) void minor_pairs_kernel(WalkArgs A)
{
    __shared__ MinorShared S;
    // the remainder tells the range, which saves registers (32 columns 9.6 -> 9.4 ms)
    const uint32_t wave = uniform_u32(threadIdx.x / kWave % kMinorWaves);
    for (;;) {
        if (threadIdx.x == 0) S.next_unit = atomicAdd(A.counter, 1u);
        __syncthreads();
        const uint32_t u = uniform_u32(S.next_unit);
        __syncthreads();
        if (u >= A.total_units) break;
        const uint32_t item = item_of_unit(A, u);
        // the gather's flag, at an address that does not wait for the descriptor (a unit
        // of a sampling step is a few us long)
        const double direct = kconst(A.a + 2 * (size_t)item)[0];
        const PermDesc d = A.descs[item];
        if (direct != 0.0)
            dispatch_minor_pairs<kMinorMinPairs, NPMAX, true>(A, d, u - (uint32_t)d.unit_base, S, wave);
        else dispatch_minor_pairs<kMinorMinPairs, NPMAX, false>(A, d, u - (uint32_t)d.unit_base, S, wave);
    }
}

}  // namespace bbfg
