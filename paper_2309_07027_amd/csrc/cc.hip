// cc.hip -- gfx950 kernels of the Clifford & Clifford sampler step (Sec. 4).
//
// Step k of a sample draws the k-th output mode r_k with probability
// proportional to |perm A[(r_1..r_{k-1}, r), (pi_1..pi_k)]|^2.  Expanding that
// k x k permanent along its last row gives
//     w_r = | sum_{l=1..k} A[r, pi_l] * minor_l |^2,
//     minor_l = perm A[(r_1..r_{k-1}), (pi_1..pi_k) without pi_l],
// so one batch of k permanents of size k-1 (rows with multiplicities) serves
// every candidate row.  The minors come from the permanent engine; this kernel
// forms the weights of all candidates and draws r_k by inverse CDF.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "cc_kernels.hpp"
#include "internal.hpp"
#include "walk_core.hpp"

namespace bbfg {

// A (rows x n) = the input columns of U (ideal), or of the 2m x 2m dilation
// [[se U, sl I], [sl U, -se I]] (lossy; inputs lie in the first m modes, so
// only the U blocks are ever selected).
__global__ void build_job_matrix_kernel(const double* __restrict__ U, int m, const int32_t* __restrict__ cols, int n,
                                        double se, double sl, int lossy, double* __restrict__ A)
{
    const int rows = lossy ? 2 * m : m;
    const int total = rows * n;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gridDim.x * blockDim.x) {
        const int r = e / n, b = e - r * n;
        const int ur = r < m ? r : r - m;
        const double f = lossy ? (r < m ? se : sl) : 1.0;
        const double* u = U + 2 * ((size_t)ur * m + cols[b]);
        A[2 * (size_t)e] = f * u[0];
        A[2 * (size_t)e + 1] = f * u[1];
    }
}

constexpr int kCCThreads = 256;
constexpr int kCCRows = 256;    // most candidate rows (2 x 128 modes, or 256)

// What the draw of one step works on: the first k permuted columns, their
// minors (values, moduli, error estimates), the candidates' weights.
struct CCShared {
    double w[kCCRows], dw[kCCRows];
    double mr[kMaxN], mi[kMaxN], ma[kMaxN], me[kMaxN];
    double sums[2];
    int32_t p[kMaxN];
    int choice;
};

// Draws row r_k by inverse CDF from the minors in S (all threads of the block;
// S.choice is the drawn row and the return value its error estimate afterwards,
// for thread 0).  The loads of a candidate's sum are independent of each other,
// and one thread adds the weights in row order, keeping the running sums for a
// search by all threads.
__device__ __forceinline__ double cc_draw(CCShared& S, const double* A, int rows, int n, int k, double u)
{
    if (threadIdx.x == 0) S.choice = rows;
    for (int r = threadIdx.x; r < rows; r += kCCThreads) {
        const double* arow = A + 2 * (size_t)r * n;
        double sr = 0.0, si = 0.0, e = 0.0;
        if (k == 1) {
            sr = arow[2 * S.p[0]];
            si = arow[2 * S.p[0] + 1];
        } else {
#pragma unroll 8
            for (int l = 0; l < k; ++l) {
                const double ar = arow[2 * S.p[l]], ai = arow[2 * S.p[l] + 1];
                sr = __builtin_fma(ar, S.mr[l], sr);
                sr = __builtin_fma(-ai, S.mi[l], sr);
                si = __builtin_fma(ar, S.mi[l], si);
                si = __builtin_fma(ai, S.mr[l], si);
                e += __builtin_sqrt(ar * ar + ai * ai) * S.ma[l] * S.me[l];
            }
        }
        S.w[r] = __builtin_fma(sr, sr, si * si);
        S.dw[r] = e * (2.0 * __builtin_sqrt(S.w[r]) + e);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double total = 0.0, dtotal = 0.0;
#pragma unroll 8
        for (int r = 0; r < rows; ++r) {
            total += S.w[r];
            dtotal += S.dw[r];
            S.dw[r] = total;  // the running sum of the weights
        }
        S.sums[0] = total;
        S.sums[1] = dtotal;
    }
    __syncthreads();
    const double total = S.sums[0], target = u * total;
    for (int r = threadIdx.x; r < rows; r += kCCThreads)
        if (S.dw[r] > target) atomicMin(&S.choice, r);
    __syncthreads();
    if (threadIdx.x == 0 && S.choice >= rows) {
        // rounding left the draw past the total: the last row with a weight
        int c = rows - 1;
        for (int r = rows - 1; r >= 0; --r)
            if (S.w[r] > 0.0) {
                c = r;
                break;
            }
        S.choice = c;
    }
    __syncthreads();
    return total > 0.0 ? S.sums[1] / total : 0.0;
}

// One block per sample's step.  Bound by latency: the step's record, columns and
// minors are gathered once into LDS.  (With the loads chained through the slot
// map inside the sums, and a serial search, a step of 20 photons on 60 modes
// took 10.5 us.)
__global__ __launch_bounds__(kCCThreads) void cc_weights_kernel(const CCStep* __restrict__ steps,
                                                                const int32_t* __restrict__ pi,
                                                                const uint32_t* __restrict__ slot,
                                                                const double* __restrict__ minors,
                                                                const double* __restrict__ minor_err,
                                                                int32_t* __restrict__ drawn, double* __restrict__ tv_est)
{
    const CCStep st = steps[blockIdx.x];
    __shared__ CCShared S;
    if ((int)threadIdx.x < st.k) {
        const int l = threadIdx.x;
        S.p[l] = pi[st.pi_off + l];
        if (st.k > 1) {
            const size_t q = slot[st.minor_off + l];
            const double x = minors[2 * q], y = minors[2 * q + 1];
            S.mr[l] = x;
            S.mi[l] = y;
            S.ma[l] = __builtin_sqrt(x * x + y * y);
            S.me[l] = minor_err[2 * q];
        }
    }
    __syncthreads();
    const double tv = cc_draw(S, st.A, st.rows, st.n, st.k, st.u);
    if (threadIdx.x == 0) {
        drawn[blockIdx.x] = S.choice;
        tv_est[blockIdx.x] = tv;
    }
}

// ---------------------------------------------------------------------------
// the first steps of a sample, all in one launch
// ---------------------------------------------------------------------------
// Step k's minors are sums of 2^{k-2} addends over the signs of the k - 1
// prefix rows (the first at +1; a row drawn twice is two rows): too short to be
// worth a round trip to the host each.  One block takes a sample through its
// first kEarlySteps steps.  A thread holds one pattern of the first eight signs
// and walks the others in Gray order; the threads' sums meet in LDS.  Bound by
// the latency of a step's chain of gathers, sums and draw: about 7 us a step
// against 60 us for a step of its own launches and round trip.  16 samples on 60
// modes: 12 photons 736 -> 144 us, 20 photons 1.41 -> 0.73 ms.  At 14 columns a
// thread walks 16 patterns; each further step would double that, and a step's
// own launches fill the device better from there on.
constexpr int kEarlySigns = 8;
static_assert(kCCThreads == 1 << kEarlySigns, "a thread per sign pattern");

struct EarlyShared {
    CCShared draw;
    double row[kEarlySteps][kEarlySteps][2];           // drawn rows at the sample's columns
    double acc[3 * kEarlySteps][kCCThreads + 1];       // per target: re, im, |re| + |im| of every thread
    double sum[3 * kEarlySteps];
};

template <int K>
__device__ __forceinline__ void early_minors(EarlyShared& S)
{
    constexpr int kSigns = K - 2;
    constexpr int kHeld = kSigns < kEarlySigns ? kSigns : kEarlySigns;
    const uint32_t t = threadIdx.x;
    double accr[K], acci[K], acca[K];
#pragma unroll
    for (int j = 0; j < K; ++j) accr[j] = acci[j] = acca[j] = 0.0;
    if (t < (1u << kHeld)) {
        double re[K], im[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            re[j] = S.row[0][j][0];
            im[j] = S.row[0][j][1];
        }
        double sign = 1.0;
        for (int i = 0; i < kSigns; ++i) {
            const double d = i < kHeld && (t >> i & 1u) ? -1.0 : 1.0;
            sign *= d;
#pragma unroll
            for (int j = 0; j < K; ++j) {
                re[j] = __builtin_fma(d, S.row[1 + i][j][0], re[j]);
                im[j] = __builtin_fma(d, S.row[1 + i][j][1], im[j]);
            }
        }
        for (uint32_t g = 0;;) {
            double pr[K], pm[K];
            pr[0] = sign;
            pm[0] = 0.0;
#pragma unroll
            for (int j = 1; j < K; ++j) {
                pr[j] = __builtin_fma(pr[j - 1], re[j - 1], -(pm[j - 1] * im[j - 1]));
                pm[j] = __builtin_fma(pr[j - 1], im[j - 1], pm[j - 1] * re[j - 1]);
            }
            double sr = 1.0, si = 0.0;
#pragma unroll
            for (int j = K - 1; j >= 0; --j) {
                const double zr = __builtin_fma(pr[j], sr, -(pm[j] * si));
                const double zi = __builtin_fma(pr[j], si, pm[j] * sr);
                accr[j] += zr;
                acci[j] += zi;
                acca[j] += __builtin_fabs(zr) + __builtin_fabs(zi);
                const double nr = __builtin_fma(sr, re[j], -(si * im[j]));
                si = __builtin_fma(sr, im[j], si * re[j]);
                sr = nr;
            }
            if (++g >= (1u << (kSigns - kHeld))) break;
            const int b = __builtin_ctz(g);
            const double d = ((g ^ (g >> 1)) >> b & 1u) ? -2.0 : 2.0;
            sign = -sign;
#pragma unroll
            for (int j = 0; j < K; ++j) {
                re[j] = __builtin_fma(d, S.row[1 + kHeld + b][j][0], re[j]);
                im[j] = __builtin_fma(d, S.row[1 + kHeld + b][j][1], im[j]);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
        S.acc[3 * j][t] = accr[j];
        S.acc[3 * j + 1][t] = acci[j];
        S.acc[3 * j + 2][t] = acca[j];
    }
    __syncthreads();
    // the threads' sums are added in double-double, as a wavefront's lanes are in the
    // walks: kParts threads a sum, neighbours starting in different banks
    constexpr uint32_t kParts = 3 * K * 8 <= kCCThreads ? 8 : 4;
    constexpr uint32_t kShare = kCCThreads / kParts;
    if (t < 3 * K * kParts) {
        const double* a = S.acc[t / kParts] + t % kParts * kShare;
        const uint32_t turn = t % kParts * (32 / kParts);
        ddv s = {0.0, 0.0};
#pragma unroll 8
        for (uint32_t i = 0; i < kShare; ++i) dd_gather(s, a[(i + turn) & (kShare - 1)]);
        s = dd_fast(s.hi, s.lo);
#pragma unroll
        for (uint32_t off = 1; off < kParts; off <<= 1)
            s = dd_add(s, {__shfl_xor(s.hi, (int)off), __shfl_xor(s.lo, (int)off)});
        if (t % kParts == 0) S.sum[t / kParts] = s.hi + s.lo;
    }
    __syncthreads();
    if (t < K) {
        const double scale = 1.0 / (double)(1u << (K - 2));
        double v[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c] = S.sum[3 * t + c] * scale;
        S.draw.mr[t] = v[0];
        S.draw.mi[t] = v[1];
        S.draw.ma[t] = __builtin_sqrt(v[0] * v[0] + v[1] * v[1]);
        // kappa u (n + sqrt(Q)): K - 1 columns, Q Gray positions without a new seed
        const double coeff = (double)(K - 1) + __builtin_sqrt((double)(1u << (kSigns - kHeld)));
        S.draw.me[t] = S.draw.ma[t] > 0.0 ? v[2] / S.draw.ma[t] * coeff * 0x1.0p-53 : __builtin_inf();
    }
    __syncthreads();
}

template <int K>
__device__ __forceinline__ void early_minors_of(int k, EarlyShared& S)
{
    if constexpr (K <= kEarlySteps) {
        if (k == K) early_minors<K>(S);
        else early_minors_of<K + 1>(k, S);
    }
}

__global__ __launch_bounds__(kCCThreads) void cc_early_kernel(const CCEarly* __restrict__ early,
                                                              const int32_t* __restrict__ pi,
                                                              const double* __restrict__ us,
                                                              int32_t* __restrict__ drawn, double* __restrict__ tv_est)
{
    __shared__ EarlyShared S;
    const CCEarly e = early[blockIdx.x];
    if ((int)threadIdx.x < e.steps) S.draw.p[threadIdx.x] = pi[e.pi_off + threadIdx.x];
    __syncthreads();
    double tv = 0.0;
    for (int k = 1; k <= e.steps; ++k) {
        if (k > 1) early_minors_of<2>(k, S);
        tv += cc_draw(S.draw, e.A, e.rows, e.n, k, us[e.out_off + k - 1]);
        const int c = S.draw.choice;
        if ((int)threadIdx.x < e.steps) {
            const double* x = e.A + 2 * ((size_t)c * e.n + S.draw.p[threadIdx.x]);
            S.row[k - 1][threadIdx.x][0] = x[0];
            S.row[k - 1][threadIdx.x][1] = x[1];
        }
        if (threadIdx.x == 0) drawn[e.out_off + k - 1] = c;
        __syncthreads();
    }
    if (threadIdx.x == 0) tv_est[blockIdx.x] = tv;
}

hipError_t launch_build_job_matrix(const double* U, int m, const int32_t* cols, int n, double se, double sl, int lossy,
                                   double* A, hipStream_t s)
{
    const int rows = lossy ? 2 * m : m;
    const int total = rows * n;
    if (total == 0) return hipSuccess;
    const int blocks = (total + 255) / 256;
    hipLaunchKernelGGL(build_job_matrix_kernel, dim3(blocks), dim3(256), 0, s, U, m, cols, n, se, sl, lossy, A);
    return hipGetLastError();
}

hipError_t launch_cc_early(uint32_t samples, const CCEarly* early, const int32_t* pi, const double* us, int32_t* drawn,
                           double* tv_est, hipStream_t s)
{
    if (samples == 0) return hipSuccess;
    hipLaunchKernelGGL(cc_early_kernel, dim3(samples), dim3(kCCThreads), 0, s, early, pi, us, drawn, tv_est);
    return hipGetLastError();
}

hipError_t launch_cc_weights(uint32_t nsteps, const CCStep* steps, const int32_t* pi, const uint32_t* slot,
                             const double* minors, const double* minor_err, int32_t* drawn, double* tv_est,
                             hipStream_t s)
{
    if (nsteps == 0) return hipSuccess;
    hipLaunchKernelGGL(cc_weights_kernel, dim3(nsteps), dim3(kCCThreads), 0, s, steps, pi, slot, minors, minor_err,
                       drawn, tv_est);
    return hipGetLastError();
}

}  // namespace bbfg
