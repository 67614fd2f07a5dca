// kernels.hpp -- launch interface between the host runtime and walk.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.hpp"

namespace bbfg {

const void* walk_single_fn(int n, int f32);
const void* walk_batch_fn(int bucket, int f32);
int batch_bucket_max(int nmax, int f32);
// smallest leave-one-column-out kernel for nmax columns (adds a 30-column one)
int minors_bucket_max(int nmax);

hipError_t launch_walk_single(int n, int f32, uint32_t grid, hipStream_t s, const WalkArgs& A, uint32_t item);
hipError_t launch_walk_batch(int bucket, int f32, uint32_t grid, hipStream_t s, const WalkArgs& A);
// uniform column multiplicities (items with col_pow >= 2), FP64, buckets 16 and
// 24 (at most 24 distinct columns)
const void* walk_cols_fn(int bucket);
const void* walk_cols_fn_b16();
const void* walk_cols_fn_b24();
hipError_t launch_walk_cols(int bucket, uint32_t grid, hipStream_t s, const WalkArgs& A);
// leave-one-column-out walks (items with targets > 0), FP64, same buckets
const void* walk_minors_fn(int bucket);
const void* walk_minors_fn_b16();
const void* walk_minors_fn_b24();
const void* walk_minors_fn_b30();
const void* walk_minors_fn_b32();
const void* walk_minors_fn_b48();
hipError_t launch_walk_minors(int bucket, uint32_t grid, hipStream_t s, const WalkArgs& A);
// a short single permanent in one launch (walk_short.hip)
uint32_t walk_short_lds(int n, int r);
hipError_t launch_walk_short(hipStream_t s, const ShortArgs& A);
// leave-one-column-out walk over pairs, np pairs of columns a wavefront at most
const void* minor_pairs_fn(int np);
const void* minor_pairs_fn_b3();
const void* minor_pairs_fn_b4();
const void* minor_pairs_fn_b6();
hipError_t launch_minor_pairs(int np, uint32_t grid, hipStream_t s, const WalkArgs& A);
// pair walk (walk_pairs.hip): tables of the items, then the walk; pow: items with
// col_pow >= 2
const void* pair_walk_fn(bool pow);
size_t pair_lds_bytes(uint32_t np);
hipError_t launch_pair_tables(uint32_t items, uint32_t blocks, hipStream_t s, const PairArgs& A);
hipError_t launch_pair_walk(bool pow, uint32_t grid, hipStream_t s, const PairArgs& A);
// counters: the unit counters, cleared.  image_bytes > 0: it, srcrow and srccol
// point into the pinned host image, which is copied to image_copy.
hipError_t launch_prep(uint32_t items, hipStream_t s, const PrepItem* it, const uint32_t* srcrow, const uint32_t* srccol,
                       double* a, double* a2, float* af, float* a2f, uint32_t* counters, const void* image = nullptr,
                       void* image_copy = nullptr, size_t image_bytes = 0);
hipError_t launch_finalize(uint32_t results, hipStream_t s, const PermDesc* descs, const uint32_t* res_item,
                           const double* partials, double* out, double* diag);
hipError_t launch_init_binom(double* tab, hipStream_t s);
// FP64 FMA throughput probe over `blocks` blocks of 256 lanes; *flops = the work
hipError_t launch_fma_peak(uint32_t blocks, uint32_t iters, double* out, hipStream_t s, double* flops);

}  // namespace bbfg
