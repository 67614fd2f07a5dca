// walk_short.hip -- a short single permanent in one launch.
//
// A sum of up to a few thousand wavefront steps leaves a compute unit with at
// most a few wavefronts, and nothing hides the latency of the walk's scalar
// loads, each of which depends on the one before (row record -> row, Gray entry
// -> row) and misses the first time; around it stood a gather launch before and
// a finalize launch after.  Here everything that describes the permanent comes
// with the kernel's arguments, each work group gathers the rows itself, all at
// once, into LDS, each wavefront its Gray entries to one lane each, and the work
// group that stores the last partial adds them all up.  The arithmetic and its order are
// those of walk_single_kernel and finalize_kernel.
//
// Bound by latency.  perm_bbfg, a call: 8 columns (one unit) 37.5 -> 21.2 us, 16
// columns, 2^15 addends, 57 -> 30 us, 20 columns, 2^19 addends (1024 units of 8
// steps), 69 -> 38 us (kernel: 6, 15, 23 us).  Above 32 columns, 2048 units or 40 KB of rows the
// general sequence runs: there the rows no longer fit several times into a
// compute unit's LDS and the walks are long enough to hide their loads.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "kernels.hpp"
#include "walk_core.hpp"
#include "walk_device.hpp"

namespace bbfg {

namespace {

constexpr uint32_t kShortWaves = 4;
constexpr int kWaitVector = 0x0F70;  // s_waitcnt vmcnt(0)

__device__ __forceinline__ double readlane_f64(double x, int k)
{
    const uint64_t bits = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bits, k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(bits >> 32), k);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

struct UnitSum {
    ddv r, i;
    double a;
};

// Adds unit u's partial record, stored by another work group of this launch.
__device__ __forceinline__ void add_partial(const double* partials, uint64_t u, UnitSum& s)
{
    const double* p = partials + u * kPartialDoubles;
    double x[kPartialDoubles];
#pragma unroll
    for (int q = 0; q < kPartialDoubles; ++q)
        x[q] = __hip_atomic_load(p + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s.r = dd_add(s.r, {x[0], x[1]});
    s.i = dd_add(s.i, {x[2], x[3]});
    s.a += x[4];
}

// What finalize_kernel's 256 threads compute, by a work group of one wavefront
// (at most 256 units; lane l stands for threads l, l + 64, l + 128, l + 192) or
// four.  A single unit's record comes in registers.
__device__ __forceinline__ void finalize_group(const PermDesc& d, const double* partials, uint32_t waves,
                                               UnitSum* shared, ddv unit_r, ddv unit_i, double unit_a, unsigned long long start,
                                               double* out)
{
    const uint32_t lane = threadIdx.x & (kWave - 1);
    UnitSum v4[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) v4[v] = {{0.0, 0.0}, {0.0, 0.0}, 0.0};
    if (d.units == 1) {
        if (lane == 0) v4[0] = {dd_add(v4[0].r, unit_r), dd_add(v4[0].i, unit_i), unit_a};
    } else if (waves == 1) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (lane + 64 * v < d.units) add_partial(partials, lane + 64 * v, v4[v]);
    } else {
#pragma unroll 2
        for (uint64_t u = threadIdx.x; u < d.units; u += 256) add_partial(partials, u, v4[0]);
        shared[threadIdx.x] = v4[0];
        __syncthreads();
        if (threadIdx.x >= kWave) return;
#pragma unroll
        for (int v = 1; v < 4; ++v) v4[v] = shared[lane + 64 * v];
    }
    ddv sr[4], si[4];
    double sa[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        sr[v] = v4[v].r;
        si[v] = v4[v].i;
        sa[v] = v4[v].a;
    }
#pragma unroll
    for (int half = 2; half > 0; half >>= 1)
#pragma unroll
        for (int v = 0; v < half; ++v) {
            sr[v] = dd_add(sr[v], sr[v + half]);
            si[v] = dd_add(si[v], si[v + half]);
            sa[v] = sa[v] + sa[v + half];
        }
    ddv r = sr[0], i = si[0];
    double a = sa[0];
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        const ddv orr = {__shfl_down(r.hi, s), __shfl_down(r.lo, s)};
        const ddv oi = {__shfl_down(i.hi, s), __shfl_down(i.lo, s)};
        const double oa = __shfl_down(a, s);
        r = dd_add(r, orr);
        i = dd_add(i, oi);
        a = a + oa;
    }
    if (lane == 0) {
        const double re = (r.hi + r.lo) * d.scale;
        const double im = (i.hi + i.lo) * d.scale;
        const double mag = __builtin_sqrt(re * re + im * im);
        const double kappa = mag > 0.0 ? a * d.scale / mag : __builtin_inf();
        out[0] = re;
        out[1] = im;
        out[2] = kappa * d.err_coeff;
        out[3] = kappa;
        out[4] = (double)(wall_clock64() - start);
    }
}

template <int N>
__global__ __launch_bounds__(kWave * kShortWaves) void walk_short_kernel(ShortArgs by_value)
{
    extern __shared__ __align__(16) double rows[];
    __shared__ uint32_t last;
    const unsigned long long began = wall_clock64();
    // the arguments where the launch put them: lanes index the row records
    const ShortArgs& S = *(const ShortArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    const PermDesc d = by_value.d;
    const uint32_t lane = threadIdx.x & (kWave - 1), waves = blockDim.x / kWave;
    const uint32_t u = blockIdx.x * waves + uniform_u32(threadIdx.x / kWave);
    // the kept rows, and behind them +2a and -2a of each
    double2* const a = reinterpret_cast<double2*>(rows);
    double2* const a2 = a + d.r * N;
    const double* const src = by_value.src;  // a caller's matrix: aligned to its doubles only
#pragma unroll 4
    for (uint32_t e = threadIdx.x; e < (uint32_t)d.r * N; e += blockDim.x) {
        const uint32_t k = e / N, j = e - k * N;
        const double* const at = src + 2 * ((uint64_t)S.src_row[k] * by_value.ld + j);
        const double2 x = {at[0], at[1]};
        a[e] = x;
        a2[2 * k * N + j] = {2.0 * x.x, 2.0 * x.y};
        a2[(2 * k + 1) * N + j] = {-2.0 * x.x, -2.0 * x.y};
    }
    uint32_t held = 0xFFFFFFFFu;  // the Gray entries in the lanes: positions 64 held + lane
    TabEntry mine = {0u, 0u, 0.0};
    auto tab = [&](uint32_t t) {
        if (t / kWave != held) {
            held = t / kWave;
            const uint32_t at = held * kWave + lane;
            mine = d.tab[at < d.Q ? at : d.Q - 1];
        }
        const int k = (int)(t % kWave);
        return TabEntry{(uint32_t)__builtin_amdgcn_readlane((int)mine.row, k), 0u, readlane_f64(mine.s, k)};
    };
    WalkArgs W;
    W.rowinfo = S.rows;
    W.binom = by_value.binom;
    __syncthreads();
    ddv sr = {0.0, 0.0}, si = {0.0, 0.0};
    double r = 0.0, i = 0.0, m = 0.0;
    if (u < d.units) {
        walk_unit_from<N, double, false, true>(static_cast<const double*>(rows), static_cast<const double*>(rows + 2 * d.r * N),
                                         tab, W, d, u, lane, r, i, m);
        wave_sum(r, i, m, sr, si);
        if (d.units > 1 && lane == 0) {
            double* p = by_value.partials + (uint64_t)u * kPartialDoubles;
            const double x[kPartialDoubles] = {sr.hi, sr.lo, si.hi, si.lo, m};
#pragma unroll
            for (int q = 0; q < kPartialDoubles; ++q)
                __hip_atomic_store(p + q, x[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // Each wavefront waits for its own stores: the work group's barrier does
            // not, and the release before its count waits for wavefront 0's alone (what
            // it writes back covers the compute unit's stores that have arrived).  A
            // release fence here would write back the cache once a wavefront: 20 columns
            // 45 us a call instead of 39.
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(kWaitVector);
            asm volatile("" ::: "memory");
        }
    }
    if (d.units == 1) {
        finalize_group(d, nullptr, 1, nullptr, sr, si, m, began, by_value.out);
        return;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        // Work groups count themselves in kShortCounters counters, the last of each
        // of those in another: a thousand increments of one word take 20 us.
        if (blockIdx.x == 0) __hip_atomic_store(by_value.start, began, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t mine = blockIdx.x % kShortCounters;
        const uint32_t members = (gridDim.x - mine + kShortCounters - 1) / kShortCounters;
        uint32_t* own = by_value.done + (1 + mine) * kCounterStride;
        last = 0;
        if (__hip_atomic_fetch_add(own, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) + 1u == members) {
            __hip_atomic_store(own, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next launch
            const uint32_t groups = gridDim.x < kShortCounters ? gridDim.x : kShortCounters;
            if (__hip_atomic_fetch_add(by_value.done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) + 1u == groups) {
                __hip_atomic_store(by_value.done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                last = 1;
            }
        }
    }
    __syncthreads();
    if (last) {
        // every unit's partial had left its wavefront before its work group's count
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        const unsigned long long start = __hip_atomic_load(by_value.start, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        finalize_group(d, by_value.partials, waves, reinterpret_cast<UnitSum*>(rows), sr, si, m, start, by_value.out);
    }
}

template <int... Is>
const void* short_ptr(int n, std::integer_sequence<int, Is...>)
{
    const void* t[] = {reinterpret_cast<const void*>(&walk_short_kernel<Is + 1>)...};
    return t[n - 1];
}

}  // namespace

uint32_t walk_short_lds(int n, int r) { return 3u * (uint32_t)r * (uint32_t)n * 16u; }

hipError_t launch_walk_short(hipStream_t s, const ShortArgs& A)
{
    if (A.d.n < 1 || A.d.n > kShortMaxN || A.d.r > kShortMaxN || A.d.units > kShortMaxUnits) return hipErrorInvalidValue;
    void* args[] = {const_cast<ShortArgs*>(&A)};
    // one wavefront a work group while the compute units are not all used
    const uint32_t waves = A.d.units <= 256 ? 1 : kShortWaves;
    uint32_t lds = walk_short_lds(A.d.n, A.d.r);
    if (waves > 1) lds = std::max<uint32_t>(lds, sizeof(UnitSum) * kWave * waves);  // the last work group's sums
    return hipLaunchKernel(short_ptr(A.d.n, std::make_integer_sequence<int, kShortMaxN>{}),
                           dim3(((uint32_t)A.d.units + waves - 1) / waves), dim3(kWave * waves), args, lds, s);
}

}  // namespace bbfg
