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

// One block per sample's step.  Bound by latency: the step's record, columns and
// minors are gathered once into LDS, so that the loads of a candidate's sum are
// independent of each other, and one thread adds the weights in row order,
// keeping the running sums for a search by all threads.  (With the loads
// chained through the slot map inside the sums, and a serial search, a step of
// 20 photons on 60 modes took 10.5 us.)
constexpr int kCCThreads = 256;
constexpr int kCCRows = 256;    // most candidate rows (2 x 128 modes, or 256)

__global__ __launch_bounds__(kCCThreads) void cc_weights_kernel(const CCStep* __restrict__ steps,
                                                                const int32_t* __restrict__ pi,
                                                                const uint32_t* __restrict__ slot,
                                                                const double* __restrict__ minors,
                                                                const double* __restrict__ minor_err,
                                                                int32_t* __restrict__ drawn, double* __restrict__ tv_est)
{
    const CCStep st = steps[blockIdx.x];
    __shared__ double w[kCCRows];
    __shared__ double dw[kCCRows];
    __shared__ double mr[kMaxN], mi[kMaxN], ma[kMaxN], me[kMaxN];
    __shared__ int32_t p[kMaxN];
    __shared__ int choice;
    __shared__ double sums[2];
    if ((int)threadIdx.x < st.k) {
        const int l = threadIdx.x;
        p[l] = pi[st.pi_off + l];
        if (st.k > 1) {
            const size_t q = slot[st.minor_off + l];
            const double x = minors[2 * q], y = minors[2 * q + 1];
            mr[l] = x;
            mi[l] = y;
            ma[l] = __builtin_sqrt(x * x + y * y);
            me[l] = minor_err[2 * q];
        }
    }
    if (threadIdx.x == 0) choice = st.rows;
    __syncthreads();
    for (int r = threadIdx.x; r < st.rows; r += kCCThreads) {
        const double* arow = st.A + 2 * (size_t)r * st.n;
        double sr = 0.0, si = 0.0, e = 0.0;
        if (st.k == 1) {
            sr = arow[2 * p[0]];
            si = arow[2 * p[0] + 1];
        } else {
#pragma unroll 8
            for (int l = 0; l < st.k; ++l) {
                const double ar = arow[2 * p[l]], ai = arow[2 * p[l] + 1];
                sr = __builtin_fma(ar, mr[l], sr);
                sr = __builtin_fma(-ai, mi[l], sr);
                si = __builtin_fma(ar, mi[l], si);
                si = __builtin_fma(ai, mr[l], si);
                e += __builtin_sqrt(ar * ar + ai * ai) * ma[l] * me[l];
            }
        }
        w[r] = __builtin_fma(sr, sr, si * si);
        dw[r] = e * (2.0 * __builtin_sqrt(w[r]) + e);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double total = 0.0, dtotal = 0.0;
#pragma unroll 8
        for (int r = 0; r < st.rows; ++r) {
            total += w[r];
            dtotal += dw[r];
            dw[r] = total;  // the running sum of the weights
        }
        sums[0] = total;
        sums[1] = dtotal;
    }
    __syncthreads();
    const double total = sums[0], target = st.u * total;
    for (int r = threadIdx.x; r < st.rows; r += kCCThreads)
        if (dw[r] > target) atomicMin(&choice, r);
    __syncthreads();
    if (threadIdx.x == 0) {
        int c = choice;
        if (c >= st.rows) {  // rounding left the draw past the total: the last row with a weight
            c = st.rows - 1;
            for (int r = st.rows - 1; r >= 0; --r)
                if (w[r] > 0.0) {
                    c = r;
                    break;
                }
        }
        drawn[blockIdx.x] = c;
        tv_est[blockIdx.x] = total > 0.0 ? sums[1] / total : 0.0;
    }
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
