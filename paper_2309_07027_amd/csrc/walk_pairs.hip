// walk_pairs.hip -- gfx950 kernels of the pair walk (pair_core.hpp).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.hpp"
#include "pair_core.hpp"
#include "walk_device.hpp"

namespace bbfg {

constexpr int kPairThreads = kWave * kPairWaves;

// LDS of a work group: the lane parts of every pair (after the walk: the
// wavefronts' sums and weights), the coefficients of the kept rows per lane,
// the next unit.
constexpr size_t kPairCoefBytes = size_t(kMaxN) * kWave;
constexpr size_t kPairRedBytes = sizeof(double) * 4 * kPairThreads;
constexpr size_t pair_lane_bytes(uint32_t np)
{
    const size_t bytes = sizeof(cpx) * kPairSlots * kWave * np;
    return bytes > kPairRedBytes ? bytes : kPairRedBytes;
}
static_assert(pair_lane_bytes(kPairMax) + kPairCoefBytes + 16 <= 160 * 1024, "LDS of a compute unit");
size_t pair_lds_bytes(uint32_t np) { return pair_lane_bytes(np) + kPairCoefBytes + 16; }

// ---------------------------------------------------------------------------
// tables of each item: uniform parts, weights and constants
// ---------------------------------------------------------------------------
// Bound by the stores of the uniform parts (96 bytes a pair and position): they
// go through LDS so that a wavefront writes whole lines.
constexpr uint32_t kTabThreads = 256;

__global__ __launch_bounds__(kTabThreads) void pair_tables_kernel(PairArgs A)
{
    __shared__ double stage[kTabThreads * (2 * kPairSlots + 1)];
    const PairDesc d = A.descs[blockIdx.x];
    kptr<RowInfo> ri = kconst(A.rowinfo + d.rowinfo_off);
    const double* a = A.a + 2 * d.a_off;
    const uint32_t np = (uint32_t)d.np;
    const uint32_t entries = d.mid * np;
    const uint32_t step = gridDim.y * kTabThreads;
    for (uint32_t e0 = blockIdx.y * kTabThreads; e0 < entries; e0 += step) {
        const uint32_t e = e0 + threadIdx.x;
        if (e < entries) {
            const uint32_t h = e / np, p = e - h * np;
            pair_mid(d, ri, a, p, h, stage + threadIdx.x * (2 * kPairSlots + 1));
        }
        __syncthreads();
        const uint32_t left = entries - e0 < kTabThreads ? entries - e0 : kTabThreads;
        double* const out = A.tables + d.mid_off + (size_t)e0 * (2 * kPairSlots);
        for (uint32_t i = threadIdx.x; i < left * (2 * kPairSlots); i += kTabThreads) {
            const uint32_t t = i / (2 * kPairSlots);
            out[i] = stage[t * (2 * kPairSlots + 1) + (i - t * (2 * kPairSlots))];
        }
        __syncthreads();
    }
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *A.counter = 0u;  // of the walk that follows
    if (A.unit_item)
        for (uint32_t u = blockIdx.y * blockDim.x + threadIdx.x; u < d.units; u += step) A.unit_item[d.unit_base + u] = blockIdx.x;
    if (blockIdx.y == 0) {
        for (uint32_t h = threadIdx.x; h < d.mid; h += blockDim.x)
            A.tables[d.weight_off + h] = pair_mid_weight(d, ri, A.binom, h);
        for (uint32_t p = threadIdx.x; p < np; p += blockDim.x)
            pair_constants(d, a, p, A.tables + d.const_off + (size_t)p * (2 * kPairConsts));
    }
}

// ---------------------------------------------------------------------------
// the walk: persistent work groups pull units from a counter
// ---------------------------------------------------------------------------
template <bool POW>
__global__ __launch_bounds__(kPairThreads) void pair_walk_kernel(PairArgs A)
{
    extern __shared__ __align__(16) char lds[];
    cpx* const parts = reinterpret_cast<cpx*>(lds);
    double* const red = reinterpret_cast<double*>(lds);
    int8_t* const coef = reinterpret_cast<int8_t*>(lds + pair_lane_bytes(A.np_max));
    uint32_t* const next_unit = reinterpret_cast<uint32_t*>(coef + kPairCoefBytes);
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = uniform_u32(threadIdx.x / kWave);
    // the first unit is the work group's own; each later one is taken from the
    // counter while its predecessor is walked
    uint32_t fetched = blockIdx.x;
    for (;;) {
        if (threadIdx.x == 0) *next_unit = fetched;
        __syncthreads();
        const uint32_t u = uniform_u32(*next_unit);
        if (u >= A.total_units) break;
        if (threadIdx.x == 0) fetched = gridDim.x + atomicAdd(A.counter, 1u);
        const uint32_t item = A.unit_item ? uniform_u32(A.unit_item[u]) : 0u;
        const PairDesc d = A.descs[item];
        const uint32_t u_local = u - d.unit_base;
        const uint32_t g = u_local / d.high;
        const uint32_t high = u_local - g * d.high;
        kptr<RowInfo> ri = kconst(A.rowinfo + d.rowinfo_off);
        kptr<double> a = kconst(A.a + 2 * d.a_off);
        const double direct = kconst(A.a + 2 * (size_t)d.direct_off)[0];  // set by the gather (walk.hip)
        uint32_t lane_idx = g * kWave + lane;
        const bool valid = lane_idx < d.lane_product;
        if (!valid) lane_idx = 0;
        // this wavefront's rows: their coefficients per lane, and the product of
        // their weights
        double w = valid ? 1.0 : 0.0;
        for (int k = (int)wave; k < d.r; k += kPairWaves) {
            RowInfo x;
            x.base = ri[k].base;
            x.kind = ri[k].kind;
            x.radix = ri[k].radix;
            x.stride = ri[k].stride;
            x.mp = ri[k].mp;
            const int c = pair_coef(x, lane_idx, high);
            coef[k * kWave + (int)lane] = (int8_t)c;
            w *= pair_row_weight(x, A.binom, c);
        }
        __syncthreads();
        auto lane_coef = [&](int k) { return (double)coef[k * kWave + (int)lane]; };
        for (uint32_t p = wave; p < (uint32_t)d.np; p += kPairWaves) {
            PairSums q;
            pair_seed(d, a, p, lane_coef, q);
#pragma unroll
            for (int s = 0; s < kPairSlots; ++s) parts[(p * kPairSlots + s) * kWave + lane] = q.s[s];
        }
        __syncthreads();
        const uint32_t h0 = d.mid * wave / kPairWaves, h1 = d.mid * (wave + 1) / kPairWaves;
        double r, i, m;
        if (direct != 0.0) {
            pair_walk_direct<POW>(d, a, kconst(A.tables + d.mid_off), kconst(A.tables + d.weight_off), h0, h1,
                                  [&](uint32_t p, cpx* c) {
                                      c[0] = parts[p * kPairSlots * kWave + lane];
                                      c[1] = parts[(p * kPairSlots + 1) * kWave + lane];
                                  },
                                  r, i, m);
        } else {
            pair_walk<POW>(d, kconst(A.tables + d.mid_off), kconst(A.tables + d.weight_off),
                           kconst(A.tables + d.const_off), h0, h1,
                           [&](uint32_t p, PairSums& q) {
#pragma unroll
                               for (int s = 0; s < kPairSlots; ++s) q.s[s] = parts[(p * kPairSlots + s) * kWave + lane];
                           },
                           r, i, m);
        }
        __syncthreads();  // the lane parts are no longer read
        red[threadIdx.x] = r;
        red[kPairThreads + threadIdx.x] = i;
        red[2 * kPairThreads + threadIdx.x] = m;
        red[3 * kPairThreads + threadIdx.x] = w;
        __syncthreads();
        if (wave == 0) {
            ddv sr, si;
            double sa;
            pair_join(
                [&](int v, double& vr, double& vi, double& vm, double& vw) {
                    const int at = v * kWave + (int)lane;
                    vr = red[at];
                    vi = red[kPairThreads + at];
                    vm = red[2 * kPairThreads + at];
                    vw = red[3 * kPairThreads + at];
                },
                r, i, m, w, sr, si, sa);
            store_partial(A.partials, d.part_base + u_local, sr, si, sa);
        }
    }
}

const void* pair_walk_fn(bool pow)
{
    return pow ? reinterpret_cast<const void*>(&pair_walk_kernel<true>)
               : reinterpret_cast<const void*>(&pair_walk_kernel<false>);
}

hipError_t launch_pair_tables(uint32_t items, uint32_t blocks, hipStream_t s, const PairArgs& A)
{
    if (items == 0) return hipSuccess;
    hipLaunchKernelGGL(pair_tables_kernel, dim3(items, blocks), dim3(256), 0, s, A);
    return hipGetLastError();
}

hipError_t launch_pair_walk(bool pow, uint32_t grid, hipStream_t s, const PairArgs& A)
{
    void* args[] = {const_cast<PairArgs*>(&A)};
    return hipLaunchKernel(pair_walk_fn(pow), dim3(grid), dim3(kPairThreads), args, pair_lds_bytes(A.np_max), s);
}

}  // namespace bbfg
