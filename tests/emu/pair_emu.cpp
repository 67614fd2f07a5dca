// pair_emu.cpp -- CPU emulation of the pair walk, for tests.
//
// Runs the per-lane code of the gfx950 kernel (pair_core.hpp, compiled for the
// host with bounds-checked pointers) on the planner's split, unit by unit,
// wavefront by wavefront and lane by lane, and adds the units' sums.  Built
// with AddressSanitizer/UBSan by the tests.
//
// stdin : n_rows n single ryser pow / n_rows multiplicities / n_rows*n complex
//         entries (re im, hex floats), row-major.  pow >= 2: every one of the n
//         columns has that multiplicity.
// stdout: re im kappa units mid (hex floats, then integers), or "general" when
//         the planner leaves the case to the general walk
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "pair_core.hpp"
#include "plan.hpp"

using namespace bbfg;

int main()
{
    int n_rows = 0, n = 0, single = 0, ryser = 0, pow = 0;
    if (std::scanf("%d %d %d %d %d", &n_rows, &n, &single, &ryser, &pow) != 5) return 2;
    std::vector<int32_t> M((size_t)n_rows);
    for (int32_t& m : M)
        if (std::scanf("%d", &m) != 1) return 2;
    std::vector<double> A(2 * (size_t)n_rows * (size_t)n);
    for (double& x : A)
        if (std::scanf("%la", &x) != 1) return 2;
    HostPlan P;
    PlanParams pp;
    pp.ryser = ryser != 0;
    std::string err;
    if (build_plan(M.data(), n_rows, pow >= 2 ? n * pow : n, 4096, pp, P, err)) {
        std::fprintf(stderr, "plan error: %s\n", err.c_str());
        return 2;
    }
    auto pair = build_pair_plan(P, n, single ? 256u : 0u);
    if (!pair) {
        std::printf("general\n");
        return 0;
    }
    const int r = P.r;
    std::vector<double> a(2 * (size_t)r * (size_t)n);
    for (int k = 0; k < r; ++k)
        std::memcpy(&a[2 * (size_t)k * n], &A[2 * (size_t)P.src_row[(size_t)k] * n], sizeof(double) * 2 * (size_t)n);
    std::vector<double> binom((size_t)kBinomDim * kBinomDim, 0.0);
    for (int m = 0; m < kBinomDim; ++m)
        for (int k = 0; k <= m; ++k) binom[(size_t)m * kBinomDim + k] = (double)binom_u64(m, k);
    PairDesc d;
    std::memset(&d, 0, sizeof d);
    d.units = (uint32_t)pair->units;
    d.lane_product = pair->lane_product;
    d.mid = pair->mid;
    d.high = pair->high;
    d.col_pow = pow >= 2 ? (uint32_t)pow : 1u;
    d.n = n;
    d.np = (n + 1) / 2;
    d.r = r;
    for (int k = 0; k < kPairBits; ++k) d.inner[k] = pair->inner[k];
    d.mids = (int32_t)pair->mid_rows.size();
    if (d.mids > kPairMids || d.mid > (uint32_t)kPairMidMax) return 3;
    for (int i = 0; i < d.mids; ++i) d.mid_row[i] = pair->mid_rows[(size_t)i];
    const uint32_t np = (uint32_t)d.np;
    // the tables in one buffer, in the library's order
    const size_t mid_doubles = (size_t)d.mid * np * 2 * kPairSlots;
    std::vector<double> tab(mid_doubles + d.mid + (size_t)np * 2 * kPairConsts);
    double *weight = tab.data() + mid_doubles, *consts = weight + d.mid;
    emu_clear();
    emu_register(a.data(), sizeof(double) * a.size());
    emu_register(tab.data(), sizeof(double) * tab.size());
    emu_register(pair->rows.data(), sizeof(RowInfo) * pair->rows.size());
    kptr<RowInfo> ri = kconst(pair->rows.data());
    for (uint32_t h = 0; h < d.mid; ++h) {
        for (uint32_t p = 0; p < np; ++p) pair_mid(d, ri, a.data(), p, h, &tab[((size_t)h * np + p) * 2 * kPairSlots]);
        weight[h] = pair_mid_weight(d, ri, binom.data(), h);
    }
    for (uint32_t p = 0; p < np; ++p) pair_constants(d, a.data(), p, consts + (size_t)p * 2 * kPairConsts);
    // the gather's choice between differences and products of column sums
    uint64_t inner_rows = 0;
    for (int k : pair->inner) inner_rows |= uint64_t(1) << k;
    bool direct = false;
    for (int j = 0; j < n; ++j)
        direct = direct || !differences_serve(r, inner_rows, [&](int k) {
                     const double* x = &a[2 * ((size_t)k * n + j)];
                     return std::fabs(x[0]) + std::fabs(x[1]);
                 });
    double sr = 0.0, si = 0.0, sa = 0.0;
    for (uint32_t u = 0; u < d.units; ++u) {
        const uint32_t g = u / d.high, high = u % d.high;
        for (uint32_t lane = 0; lane < (uint32_t)kWave; ++lane) {
            const uint32_t lane_idx = g * kWave + lane;
            if (lane_idx >= d.lane_product) continue;
            std::vector<int> coef((size_t)r);
            double w = 1.0;
            for (int k = 0; k < r; ++k) {
                coef[(size_t)k] = pair_coef(pair->rows[(size_t)k], lane_idx, high);
                if (coef[(size_t)k] < -128 || coef[(size_t)k] > 127) return 3;  // kept as a byte
                w *= pair_row_weight(pair->rows[(size_t)k], binom.data(), coef[(size_t)k]);
            }
            std::vector<PairSums> parts(np);
            for (uint32_t p = 0; p < np; ++p)
                pair_seed(d, kconst(a.data()), p, [&](int k) { return (double)coef[(size_t)k]; }, parts[p]);
            for (uint32_t wave = 0; wave < (uint32_t)kPairWaves; ++wave) {
                const uint32_t h0 = d.mid * wave / kPairWaves, h1 = d.mid * (wave + 1) / kPairWaves;
                double x, y, z;
                auto get = [&](uint32_t p, PairSums& q) { q = parts[p]; };
                auto sums = [&](uint32_t p, cpx* c) {
                    c[0] = parts[p].s[0];
                    c[1] = parts[p].s[1];
                };
                if (direct && pow >= 2)
                    pair_walk_direct<true>(d, kconst(a.data()), kconst(tab.data()), kconst(weight), h0, h1, sums, x, y, z);
                else if (direct)
                    pair_walk_direct<false>(d, kconst(a.data()), kconst(tab.data()), kconst(weight), h0, h1, sums, x, y, z);
                else if (pow >= 2)
                    pair_walk<true>(d, kconst(tab.data()), kconst(weight), kconst(consts), h0, h1, get, x, y, z);
                else
                    pair_walk<false>(d, kconst(tab.data()), kconst(weight), kconst(consts), h0, h1, get, x, y, z);
                sr += w * x;
                si += w * y;
                sa += std::fabs(w) * z;
            }
        }
    }
    const double s = std::ldexp(1.0, P.scale_log2);
    std::printf("%a %a %a %llu %u\n", sr * s, si * s, sa * s / std::hypot(sr * s, si * s), (unsigned long long)d.units, d.mid);
    return 0;
}
