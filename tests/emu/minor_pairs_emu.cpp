// minor_pairs_emu.cpp -- CPU emulation of the leave-one-column-out walk over
// pairs of columns, for tests.
//
// Runs the per-lane code of the gfx950 kernel (minor_pairs_core.hpp, compiled
// for the host with bounds-checked pointers) on the planner's split: the four
// wavefronts of a work group in step, lane by lane.  Built with
// AddressSanitizer/UBSan by the tests.
//
// stdin : n_rows K slots l_batch / n_rows multiplicities (sum K - 1) /
//         n_rows*K complex entries (re im, hex floats), row-major
// stdout: K lines "re im" (permanent without column l), or "general" when the
//         planner leaves the case to the other walk
#include <cmath>
#include <cstdio>
#include <vector>

#include "minor_pairs_core.hpp"
#include "plan.hpp"

using namespace bbfg;

namespace {

template <int NP, int DIGITS, bool DIRECT>
void run_way(const HostPlan& P, int K, const std::vector<double>& A, std::vector<double>& out)
{
    const int r = P.r, pairs = NP * kMinorWaves;
    constexpr int kStep = MinorLane<NP, DIGITS, DIRECT>::kStep;
    // the prep kernel's layout
    std::vector<double> rows(4 * (size_t)r * pairs, 0.0), steps(kStep * (size_t)(2 * (r - 1)) * pairs);
    for (int k = 0; k < r; ++k)
        for (int j = 0; j < K; ++j)
            for (int c = 0; c < 2; ++c)
                rows[4 * (size_t)k * pairs + 2 * j + c] = A[2 * ((size_t)P.src_row[(size_t)k] * K + j) + c];
    for (int k = 0; k + 1 < r; ++k)
        for (int p = 0; p < pairs; ++p) {
            const double* x = &rows[4 * ((size_t)k * pairs + p)];
            double v[kStep] = {2 * x[0], 2 * x[1], 2 * x[2], 2 * x[3]};
            for (int i = 0; i < DIGITS; ++i) {
                const double* c = &rows[4 * ((size_t)(r - 1 - i) * pairs + p)];
                v[4 + 2 * i] = -4.0 * (c[0] * x[2] - c[1] * x[3] + x[0] * c[2] - x[1] * c[3]);
                v[5 + 2 * i] = -4.0 * (c[0] * x[3] + c[1] * x[2] + x[0] * c[3] + x[1] * c[2]);
            }
            for (int q = 0; q < kStep; ++q) {
                steps[kStep * ((size_t)(2 * k) * pairs + p) + q] = v[q];
                steps[kStep * ((size_t)(2 * k + 1) * pairs + p) + q] = -v[q];
            }
        }
    emu_clear();
    emu_register(rows.data(), sizeof(double) * rows.size());
    emu_register(steps.data(), sizeof(double) * steps.size());
    std::vector<double> binom((size_t)kBinomDim * kBinomDim, 0.0);
    for (int m = 0; m < kBinomDim; ++m)
        for (int k = 0; k <= m; ++k) binom[(size_t)m * kBinomDim + k] = (double)binom_u64(m, k);
    const size_t ld = 4 * (size_t)pairs, step_ld = kStep * (size_t)pairs;
    const uint32_t upg = (uint32_t)P.units_per_group;
    for (uint64_t u = 0; u < P.units; ++u) {
        const uint32_t g = (uint32_t)(u / upg), part = (uint32_t)(u % upg);
        const uint64_t base = P.span / upg, rem = P.span - base * upg;
        const uint64_t lin0 = part * base + (part < rem ? part : rem), lin1 = lin0 + base + (part < rem ? 1 : 0);
        for (uint32_t lane = 0; lane < (uint32_t)kWave; ++lane) {
            const uint32_t lane_idx = g * kWave + lane;
            if (lane_idx >= P.lane_product) continue;
            // wavefronts of NP pairs, and those of one less
            constexpr int NL = NP > kMinorMinPairs ? NP - 1 : NP;
            MinorLane<NP, DIGITS, DIRECT> L[kMinorWaves];
            MinorLane<NL, DIGITS, DIRECT> less[kMinorWaves];
            const int full = minor_full_waves(K);
            auto wave = [&](int v, auto f) {
                if (v < full) f(L[v], NP, (size_t)(v * NP));
                else f(less[v], NL, (size_t)(v * NL + full));
            };
            auto waves = [&](auto f) {
                for (int v = 0; v < kMinorWaves; ++v)
                    wave(v, [&](auto& l, int pairs_of, size_t first) { f(v, l, pairs_of, first); });
            };
            waves([&](int, auto& l, int, size_t) { l.clear(); });
            for (uint64_t lin = lin0; lin < lin1;) {
                const uint64_t h = lin / P.Q;
                const uint32_t t0 = (uint32_t)(lin - h * P.Q);
                const uint64_t bend = (h + 1) * (uint64_t)P.Q;
                const uint32_t t1 = (uint32_t)((lin1 < bend ? lin1 : bend) - h * P.Q);
                std::vector<int> coef((size_t)r);
                double w = 1.0;
                for (int k = 0; k < r; ++k) {
                    const RowInfo& x = P.rows[(size_t)k];
                    uint32_t delta = 0;
                    if (x.kind == ROW_LANE) delta = (lane_idx / x.stride) % x.radix;
                    else if (x.kind == ROW_HIGH) delta = digit_of(h, x.stride, x.radix);
                    else if (x.kind == ROW_LOW) {
                        const uint32_t dg = (t0 / x.stride) % x.radix, q = t0 / (x.stride * x.radix);
                        delta = (q & 1u) ? (x.radix - 1u - dg) : dg;
                    }
                    coef[(size_t)k] = x.base - 2 * (int)delta;
                    w *= pair_row_weight(x, binom.data(), coef[(size_t)k]);
                }
                waves([&](int, auto& l, int, size_t first) {
                    l.seed(kconst(rows.data()) + (int64_t)(4 * first), ld, r, K - 2 * (int)first,
                           [&](int k) { return (double)coef[(size_t)k]; });
                });
                for (uint32_t t = t0; t < t1; ++t) {
                    const TabEntry e = (*P.table)[t];
                    if (t > t0)
                        waves([&](int, auto& l, int, size_t first) {
                            l.advance(&steps[(size_t)e.row * step_ld + kStep * first]);
                        });
                    cpx all[kMinorWaves][2], o[kMinorWaves][2];
                    auto exchange = [&](double ws) {
                        waves([&](int v, auto& l, int, size_t) {
                            for (int x = 0; x < 2; ++x) all[v][x] = l.half[x].all;
                        });
                        for (int v = 0; v < kMinorWaves; ++v)
                            for (int x = 0; x < 2; ++x)
                                o[v][x] = cmul_uniform(cmul(cmul(all[(v + 1) % kMinorWaves][x],
                                                                 all[(v + 2) % kMinorWaves][x]),
                                                            all[(v + 3) % kMinorWaves][x]),
                                                       ws);
                    };
                    auto inner = [&](size_t first) {
                        return kconst(rows.data()) + (int64_t)((size_t)(r - 1) * ld + 4 * first);
                    };
                    waves([&](int, auto& l, int, size_t first) { l.forward(inner(first), ld); });
                    exchange(w * e.s);
                    if constexpr (DIGITS > 1) {
                        waves([&](int v, auto& l, int, size_t first) {
                            l.template backward<false>(o[v][0], o[v][1], inner(first), ld);
                        });
                        waves([&](int, auto& l, int pairs_of, size_t first) {
                            double K[2 * NP];
                            const double* row = &steps[(size_t)(2 * (r - 2) + 1) * step_ld + kStep * first];
                            for (int p = 0; p < pairs_of; ++p) {
                                K[2 * p] = row[kStep * p + 4];
                                K[2 * p + 1] = row[kStep * p + 5];
                            }
                            l.forward_second(K, inner(first), ld);
                        });
                        exchange(-w * e.s);
                    }
                    waves([&](int v, auto& l, int, size_t first) {
                        l.template backward<true>(o[v][0], o[v][1], inner(first), ld);
                    });
                }
                lin += t1 - t0;
            }
            waves([&](int, auto& l, int pairs_of, size_t first) {
                for (int p = 0; p < pairs_of; ++p) {
                    cpx c[2];
                    l.result(p, kconst(rows.data()) + (int64_t)((size_t)(r - 1) * ld + 4 * first), ld, c[0], c[1]);
                    for (int q = 0; q < 2; ++q) {
                        const int j = 2 * (int)first + 2 * p + q;
                        if (j >= K) continue;
                        out[2 * (size_t)j] += c[q].r;
                        out[2 * (size_t)j + 1] += c[q].i;
                    }
                }
            });
        }
    }
}

// With differences or without, as the gather chooses.
template <int NP, int DIGITS>
void run(const HostPlan& P, int K, const std::vector<double>& A, std::vector<double>& out)
{
    const uint64_t inner_rows = ((uint64_t(1) << DIGITS) - 1) << (P.r - DIGITS);
    bool direct = false;
    for (int j = 0; j < K; ++j)
        direct = direct || !differences_serve(P.r, inner_rows, [&](int k) {
                     const double* x = &A[2 * ((size_t)P.src_row[(size_t)k] * K + j)];
                     return std::fabs(x[0]) + std::fabs(x[1]);
                 });
    if (direct) run_way<NP, DIGITS, true>(P, K, A, out);
    else run_way<NP, DIGITS, false>(P, K, A, out);
}

}  // namespace

int main()
{
    int n_rows = 0, K = 0;
    long long slots = 0, l_batch = 0;
    if (std::scanf("%d %d %lld %lld", &n_rows, &K, &slots, &l_batch) != 4) return 2;
    std::vector<int32_t> M((size_t)n_rows);
    for (int32_t& m : M)
        if (std::scanf("%d", &m) != 1) return 2;
    std::vector<double> A(2 * (size_t)n_rows * (size_t)K);
    for (double& x : A)
        if (std::scanf("%la", &x) != 1) return 2;
    HostPlan P;
    PlanParams pp;
    pp.l_batch = (uint64_t)l_batch;
    std::string err;
    if (!build_minor_pair_plan(M.data(), n_rows, K - 1, (uint64_t)slots, pp, P, err)) {
        if (!err.empty()) return 3;
        std::printf("general\n");
        return 0;
    }
    std::vector<double> out(2 * (size_t)K, 0.0);
    const bool two = P.minor_digits == 2;
    switch (minor_pairs_per_wave(K)) {
    case 2: run<2, 1>(P, K, A, out); break;
    case 3: run<3, 1>(P, K, A, out); break;
    case 4: two ? run<4, 2>(P, K, A, out) : run<4, 1>(P, K, A, out); break;
    case 5: run<5, 1>(P, K, A, out); break;
    case 6: run<6, 1>(P, K, A, out); break;
    default: return 4;
    }
    const double s = std::ldexp(1.0, P.scale_log2);
    for (int l = 0; l < K; ++l) std::printf("%a %a\n", out[2 * (size_t)l] * s, out[2 * (size_t)l + 1] * s);
    return 0;
}
