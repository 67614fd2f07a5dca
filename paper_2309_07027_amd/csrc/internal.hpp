// internal.hpp -- data structures shared by the host planner and the gfx950
// kernels of the generalized BB/FG permanent (arXiv:2309.07027, Sec. 2).
#pragma once

#include <cstdint>

namespace bbfg {

constexpr int kWave = 64;       // CDNA wavefront width
constexpr int kMaxN = 48;       // largest column count of the FP64 path
constexpr int kMaxNF32 = 24;    // largest column count of the FP32 path
constexpr int kBinomDim = kMaxN + 1;

// How the sign count Delta_k of a row is obtained inside a work unit.
//   FIXED: the row has no free sign (the pivot with M = 1); coefficient = base.
//   LANE : a lane-prefix digit; Delta = (lane_index / stride) % radix.
//   HIGH : a per-segment digit;  Delta = (h / stride) % radix, h = block index.
//   LOW  : a Gray-walked digit;  Delta = reflected decode of the position t
//          inside the block (Sec. 2.2 reflected n-ary Gray code).
//   MID, INNER: digits of the pair walk (pair_core.hpp): a position of its
//          uniform table, and one of the four binary digits of its blocks.
enum RowKind : int32_t { ROW_FIXED = 0, ROW_LANE = 1, ROW_HIGH = 2, ROW_LOW = 3, ROW_MID = 4, ROW_INNER = 5 };

// One kept row.  Column-sum coefficient = base - 2 * Delta  (Eq. Deltak), where
// base = M'_k + (1 if the row is the pivot).  Weight factor (-1)^Delta C(mp, Delta).
struct RowInfo {
    int32_t base;
    int32_t kind;
    uint32_t radix;   // mp + 1
    uint32_t stride;  // product of the radices of the earlier digits of the same kind
    int32_t mp;       // M'_k
    int32_t pad;
};

// Gray-walk table entry for position t of a block: the +-2a row that is added
// when stepping from t-1 to t, and the signed low-digit weight at t:
//   s(t) = prod_{low k} (-1)^{Delta_k(t)} C(M'_k, Delta_k(t)).
// The planner numbers the kept rows so that low digit i is kept row i; a table
// then depends on the radices of the low digits only and is shared by every
// permanent with the same low radices.
struct TabEntry {
    uint32_t row;  // index into the 2r x n array of +-2a rows (2i: +2a_i, 2i+1: -2a_i)
    uint32_t pad;
    double s;
};

// Device descriptor of one permanent.
struct PermDesc {
    uint64_t a_off;          // element offset of the r x n kept rows (complex)
    uint64_t a2_off;         // element offset of the 2r x n +-2a rows (complex)
    const TabEntry* tab;     // Gray table (Q entries, device memory)
    uint64_t unit_base;      // slot of this permanent's unit 0 in the partial arrays
    uint64_t units;          // number of units  (= groups * units_per_group)
    uint64_t units_per_group;
    uint64_t span;           // block positions per lane group (H * Q)
    uint32_t rowinfo_off;    // entry offset of the r RowInfo records
    int32_t n;               // columns
    int32_t r;               // kept rows
    uint32_t Q;              // Gray block length
    uint32_t lane_product;   // number of valid lane indices
    uint32_t groups;         // lane groups
    double scale;            // 2^{1-n} of the permanents computed (n - 1 columns of them for minors)
    double err_coeff;        // u * (n + sqrt(Q)), u the unit roundoff: error estimate = kappa * err_coeff
    uint64_t part_base;      // first partial slot; unit u, target t -> part_base + u * max(1, targets) + t
    uint32_t targets;        // 0: one permanent of the n columns.  G > 0: the G permanents that each
                             //   leave out one of the last G columns (Laplace minors)
    uint32_t res_base;       // index of the first result
    uint32_t col_pow;        // every one of the n (distinct) columns has multiplicity col_pow
                             //   (Eq. bbfgrepeated): the product is (prod_j c_j)^col_pow; in a
                             //   leave-one-column-out walk over pairs, its inner digits (1 or 2)
    uint32_t mag_every;      // leave-one-column-out walks: units whose index in their lane group is
                             //   a multiple of mag_every sample the magnitude estimate (>= 1)
};

// Leave-one-column-out walks over K columns cover the targets in groups of
// minor_group(K): one group keeps K column sums, G prefix products and G
// accumulators per lane (4K + 8G FP64 registers).  Up to 30 columns the groups
// stay small enough for two wavefronts per SIMD (<= 256 VGPRs): up to 24
// columns groups of at most 27 - K/2 targets, at 25-30 columns two groups (the
// kernel for up to 30 columns is built for two wavefronts per SIMD).  Above,
// where the sums are long and work dominates, one wavefront per SIMD with the
// fewest groups that fit 512 registers without spilling to scratch does fewer
// products per addend (one group up to 36 columns: K + 2G - 4 complex products
// instead of about 1.6 times that), which measured 1.2-1.25 times faster at
// 31-36 columns than three groups at two wavefronts; at 25-30 columns two
// groups at two wavefronts measured 4-9 % faster than one group at one.
constexpr int minor_group(int K)
{
    int gmax = K <= 24 ? 27 - K / 2 : (K <= 30 ? (K + 1) / 2 : 54 - K / 2);
    if (gmax < 1) gmax = 1;
    if (gmax > K) gmax = K;
    const int groups = (K + gmax - 1) / gmax;
    return (K + groups - 1) / groups;
}

// Leave-one-column-out walks estimate each target's sum of |addend| from about
// this many sampled units per lane group (64 lanes each), all units if fewer.
constexpr uint64_t kMagUnitsPerGroup = 32;
inline uint32_t mag_every_for(uint64_t units_per_group)
{
    const uint64_t e = units_per_group / kMagUnitsPerGroup;
    return e > 1 ? (uint32_t)e : 1u;
}

// Unit counters of a launch sequence: the walk's and the pair walk's, on cache
// lines of their own.
constexpr uint32_t kCounters = 2;
constexpr uint32_t kCounterStride = 32;

constexpr uint32_t kUnitChunkLog2 = 6;
constexpr uint32_t kUnitChunk = 1u << kUnitChunkLog2;

// Sizes of the partial record of one unit: a complex double-double (4 doubles)
// plus the sum of |addend| (1 double).
constexpr int kPartialDoubles = 5;

// Gather job for one matrix: element (k, j) of the kept rows is
//   src[src_off + srcrow[srcrow_off + k] * ld + col(j)]   (complex elements)
// with col(j) = j when srccol_off == kIdentityCols, else srccol[srccol_off + j].
constexpr uint32_t kIdentityCols = 0xFFFFFFFFu;
struct PrepItem {
    const double* src;
    uint64_t src_off;
    uint64_t a_off;
    uint64_t a2_off;
    uint32_t srcrow_off;
    uint32_t srccol_off;
    uint32_t ld;
    int32_t n;
    int32_t r;
    int32_t f32;
    int32_t rows_only;  // no +-2a rows
    int32_t digits;     // inner digits of that walk
    int32_t np;         // > 0: the layout of the leave-one-column-out walk over pairs, np pairs a wavefront
    uint64_t inner_rows;  // walks over pairs: the kept rows of the inner digits, a bit each (0: other walks)
    uint64_t direct_off;  // their flag in a (complex elements): not zero where products are formed from the sums
};

// ---------------------------------------------------------------------------
// short single permanents (walk_short.hip)
// ---------------------------------------------------------------------------
constexpr int kShortMaxN = 32;                // most columns, hence kept rows
constexpr uint32_t kShortMaxUnits = 2048;
constexpr uint32_t kShortCounters = 16;
constexpr uint32_t kShortLdsBytes = 40 << 10;  // rows and +-2a rows of a wavefront

// Everything one short permanent needs, passed by value with its launch.
struct ShortArgs {
    PermDesc d;               // its table resident, its offsets zero
    RowInfo rows[kShortMaxN];
    uint32_t src_row[kShortMaxN];  // kept row -> row of src
    const double* src;        // rows of ld complex elements
    const double* binom;
    double* partials;
    uint32_t* done;           // counters of finished work groups; zero between launches
    unsigned long long* start;  // clock at the first work group's start
    double* out;              // value, diagnostics, clock ticks of the launch (pinned host memory)
    uint32_t ld;
};

// ---------------------------------------------------------------------------
// pair walk (pair_core.hpp)
// ---------------------------------------------------------------------------
constexpr int kPairBits = 4;                  // inner binary digits
constexpr int kPairBlock = 1 << kPairBits;    // addends of a block
constexpr int kPairSlots = 2 + kPairBits;     // complex values of a pair: two column sums, the differences
constexpr int kPairConsts = kPairBits * (kPairBits - 1) / 2;  // constants of a pair
constexpr int kPairWaves = 16;               // wavefronts of a work group
constexpr int kPairMidMax = 512;              // most mid positions
constexpr int kPairMids = 9;                  // most mid digits
constexpr int kPairMax = (kMaxN + 1) / 2;     // most pairs of columns

// The pair walk takes sums of more than this many addends (with column
// multiplicities, more than the second number).  A unit's start costs about
// 7 us, which shorter sums do not earn back in full; up to these sizes the walk
// stays the one whose bits the CPU emulation of walk_core.hpp pins.
constexpr uint64_t kPairMinAddends = uint64_t(1) << 19;
constexpr uint64_t kPairMinAddendsCols = uint64_t(1) << 22;
constexpr int kPairMinCols = 4;

// Device descriptor of one permanent evaluated by the pair walk.  Its units are
// (lane group, high position) in that order; a unit covers every mid position.
struct PairDesc {
    uint64_t a_off;        // element offset of the r x n kept rows (complex)
    uint64_t mid_off;      // double offsets into the tables: mid x np x kPairSlots complex uniform parts,
    uint64_t weight_off;   //   the mid positions' signed weights,
    uint64_t const_off;    //   np x 6 complex constants
    uint64_t part_base;    // first partial slot (one per unit)
    uint32_t unit_base;    // first unit of the item in the launch
    uint32_t direct_off;   // PrepItem's
    uint32_t units;        // groups * high
    uint32_t rowinfo_off;  // entry offset of the r RowInfo records
    uint32_t lane_product;
    uint32_t mid;          // mid positions
    uint32_t high;         // high positions
    uint32_t col_pow;
    int32_t n;             // columns
    int32_t np;            // pairs of columns, (n + 1) / 2
    int32_t r;             // kept rows
    int32_t inner[kPairBits];  // kept rows of the inner digits
    int32_t mids;              // mid digits and their kept rows
    int32_t mid_row[kPairMids];
};

// ---------------------------------------------------------------------------
// leave-one-column-out walk over pairs (minor_pairs_core.hpp)
// ---------------------------------------------------------------------------
constexpr int kMinorWaves = 4;                // wavefronts that share a walk's columns
constexpr int kMinorMinPairs = 2;             // pairs of a wavefront, at least
constexpr int kMinorMinCols = 9;              // fewest columns it is used for
// It takes sums of more addends than this in a sampler step (16 samples of 20
// photons: 0.79, 0.80, 1.05 ms with 2^6, 2^10, 2^12; 1024 samples of 16: 3.07,
// 3.18, 3.22 ms) and in a lone call (where the walk of shorter sums stays the one
// whose bits the CPU emulation of walk_core.hpp pins; 24 columns, 2^22 addends:
// 0.193 -> 0.089 ms).
constexpr uint64_t kMinorMinAddendsBatch = uint64_t(1) << 6;
constexpr uint64_t kMinorMinAddends = uint64_t(1) << 17;
// An item of a sampler step is split into about so many units, down to units of
// so many steps of two addends.  The split depends on the item alone, so that a
// sample's bits do not depend on its neighbours; few samples want many units, a
// full launch few (128, 64, 32 units: 16 samples of 24 photons 1.56, 1.52, 1.66
// ms; 256 of them 10.6, 9.6, 9.1; 24 jobs on the server 47.1, 45.3, 44.4).
constexpr uint64_t kMinorItemUnits = 64;
constexpr uint64_t kMinorMinUnit = 16;
// Two inner digits instead of one: at four pairs a wavefront (25-32 columns),
// where they fill the 256 registers of two wavefronts per SIMD, and for longer
// sums.  30 photons: 10.1 -> 9.4 ms, 24 jobs on the server 47.9 -> 45.1 ms; at
// three pairs one digit and three wavefronts per SIMD are faster, and short sums
// want the more and shorter steps (24 photons with two throughout: 1.44 -> 1.54
// ms).
constexpr int kMinorTwoDigits = 4;
constexpr uint64_t kMinorTwoAddends = uint64_t(1) << 18;
constexpr int minor_pairs_per_wave(int K)
{
    const int np = ((K + 1) / 2 + kMinorWaves - 1) / kMinorWaves;
    return np > kMinorMinPairs ? np : kMinorMinPairs;
}
// Complex elements of a walk's steps: per kept row but the last two rows with the
// changes of b_1, b_2 and the digits' differences for each pair.
constexpr uint64_t minor_step_elems(int r, int digits, int np)
{
    return 2 * (uint64_t)(r - 1) * (uint64_t)(2 + digits) * (uint64_t)np * kMinorWaves;
}
// Wavefronts that own so many pairs; the others own one less (two at least: with
// one the chain of a step is all that is left).  Which SIMD has the smaller
// shares changes from work group to work group by itself; turning them by hand in
// every second one made no difference.  Equal shares padded with columns that are
// 1 -> these: 25 columns, 2^24 addends, 0.160 -> 0.156 ms; 33 columns 16.8 ->
// 15.4, 35 25.2 -> 24.1, 42 64.5 -> 60.2 ms (2^29 addends and more).
constexpr int minor_full_waves(int K)
{
    const int np = minor_pairs_per_wave(K);
    return np > kMinorMinPairs ? (K + 1) / 2 - kMinorWaves * (np - 1) : kMinorWaves;
}

// Kernel arguments of the pair walk (passed by value).
struct PairArgs {
    const PairDesc* descs;
    const RowInfo* rowinfo;
    const double* a;
    double* tables;
    const double* binom;
    double* partials;
    uint32_t* unit_item;     // item of each unit (null: one item)
    uint32_t* counter;
    uint32_t total_units;
    uint32_t np_max;
};

// Kernel arguments of the walk kernels (passed by value).
struct WalkArgs {
    const PermDesc* descs;
    const RowInfo* rowinfo;
    const double* a;     // FP64 kept rows (interleaved complex)
    const double* a2;    // FP64 +-2a rows
    const float* af;     // FP32 copies
    const float* a2f;
    const double* binom; // kBinomDim x kBinomDim
    double* partials;    // kPartialDoubles per unit slot
    // batch: units are numbered item by item in "unit order"; position p of that
    // order is item uorder[p], whose units start at ubase[p] (ubase has one more
    // entry: the total).  uchunk[c] is the position of the item holding unit
    // c * kUnitChunk (one more entry: the last position), which bounds the
    // search for the item of a unit to the items of its chunk.
    const uint32_t* ubase;
    const uint32_t* uorder;
    const uint32_t* uchunk;
    uint32_t* counter;          // batch: next unit
    uint32_t total_units;       // batch: number of units
    uint32_t nitem;             // batch: number of items
};

}  // namespace bbfg
