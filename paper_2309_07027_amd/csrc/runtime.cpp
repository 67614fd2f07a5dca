// runtime.cpp -- device context, buffers, plan cache and the permanent engine.
#include "runtime.hpp"

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <numeric>
#include <unordered_set>

namespace bbfg {

// ---------------------------------------------------------------------------
// errors
// ---------------------------------------------------------------------------
namespace {
thread_local std::string t_err = "no error";
thread_local hipStream_t t_stream = nullptr;
std::mutex g_ctx_mu;
// Contexts live until the process ends (never destroyed: freeing device memory
// during static destruction could race the HIP runtime's own teardown).
std::map<int, Context*> g_ctx;
}  // namespace

int set_error(int code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    t_err = buf;
    return code;
}

const char* last_error() { return t_err.c_str(); }

int validate_shape(const int32_t* mult, int32_t n_rows, int32_t n_cols, int max_n)
{
    if (n_rows < 0) return set_error(BBFG_EINVAL, "n_rows = %d < 0", n_rows);
    if (n_cols < 0) return set_error(BBFG_EINVAL, "n_cols = %d < 0", n_cols);
    if (n_cols > max_n) return set_error(BBFG_ERANGE, "n_cols = %d exceeds the maximum %d", n_cols, max_n);
    if (n_rows > 0 && !mult) return set_error(BBFG_EINVAL, "row_mult is NULL");
    int64_t sum = 0;
    for (int32_t i = 0; i < n_rows; ++i) {
        if (mult[i] < 0) return set_error(BBFG_EINVAL, "row_mult[%d] = %d < 0", i, mult[i]);
        sum += mult[i];
    }
    if (sum != n_cols)
        return set_error(BBFG_EINVAL, "sum(row_mult) = %lld differs from n_cols = %d", (long long)sum, n_cols);
    return BBFG_OK;
}

hipStream_t current_stream() { return t_stream; }
void set_current_stream(hipStream_t s) { t_stream = s; }

// ---------------------------------------------------------------------------
// buffers: grow-only, reused across calls (calls are serialised per device)
// ---------------------------------------------------------------------------
int DevBuf::ensure(size_t bytes)
{
    if (bytes <= cap) return BBFG_OK;
    size_t want = std::max<size_t>(bytes, cap + cap / 2);
    want = (want + 4095) / 4096 * 4096;
    if (p) {
        (void)hipFree(p);
        p = nullptr;
        cap = 0;
    }
    if (hipMalloc(&p, want) != hipSuccess) {
        p = nullptr;
        (void)hipGetLastError();
        return set_error(BBFG_ENOMEM, "hipMalloc(%zu) failed", want);
    }
    cap = want;
    return BBFG_OK;
}

void DevBuf::release()
{
    if (p) (void)hipFree(p);
    p = nullptr;
    cap = 0;
}

int PinnedBuf::ensure(size_t bytes)
{
    if (bytes <= cap) return BBFG_OK;
    size_t want = std::max<size_t>(bytes, cap + cap / 2);
    want = (want + 4095) / 4096 * 4096;
    if (p) {
        (void)hipHostFree(p);
        p = nullptr;
        cap = 0;
    }
    if (hipHostMalloc(&p, want, hipHostMallocDefault) != hipSuccess) {
        p = nullptr;
        (void)hipGetLastError();
        return set_error(BBFG_ENOMEM, "hipHostMalloc(%zu) failed", want);
    }
    cap = want;
    return BBFG_OK;
}

void PinnedBuf::release()
{
    if (p) (void)hipHostFree(p);
    p = nullptr;
    cap = 0;
}

Workspace::~Workspace()
{
    if (ev0) (void)hipEventDestroy(ev0);
    if (ev1) (void)hipEventDestroy(ev1);
    if (done) (void)hipEventDestroy(done);
    if (early0) (void)hipEventDestroy(early0);
    if (early1) (void)hipEventDestroy(early1);
}

int Workspace::init()
{
    if (!ev0) BBFG_HIP(hipEventCreate(&ev0));
    if (!ev1) BBFG_HIP(hipEventCreate(&ev1));
    if (!early0) BBFG_HIP(hipEventCreate(&early0));
    if (!early1) BBFG_HIP(hipEventCreate(&early1));
    if (!done) BBFG_HIP(hipEventCreateWithFlags(&done, hipEventDisableTiming));
    BBFG_TRY(counter.ensure(256));
    if (!short_done.p) {
        const size_t bytes = sizeof(uint32_t) * (2 + kShortCounters) * kCounterStride;
        BBFG_TRY(short_done.ensure(bytes));
        // zero here, and again after each launch that counts in it
        BBFG_HIP(hipMemset(short_done.p, 0, bytes));
        BBFG_HIP(hipDeviceSynchronize());
    }
    return BBFG_OK;
}

bool is_device_ptr(const void* p)
{
    if (!p) return false;
    hipPointerAttribute_t attr;
    std::memset(&attr, 0, sizeof attr);
    if (hipPointerGetAttributes(&attr, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return attr.type == hipMemoryTypeDevice || attr.type == hipMemoryTypeManaged;
}

// ---------------------------------------------------------------------------
// context
// ---------------------------------------------------------------------------
int get_context(Context** out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return set_error(BBFG_EDEVICE, "no HIP device available");
    }
    std::lock_guard<std::mutex> lk(g_ctx_mu);
    auto it = g_ctx.find(dev);
    if (it != g_ctx.end()) {
        *out = it->second;
        return BBFG_OK;
    }
    auto c = std::make_unique<Context>();
    c->device = dev;
    hipDeviceProp_t prop;
    BBFG_HIP(hipGetDeviceProperties(&prop, dev));
    c->n_cu = prop.multiProcessorCount;
    BBFG_HIP(hipDeviceGetAttribute(&c->clock_khz, hipDeviceAttributeWallClockRate, dev));
    BBFG_HIP(hipMalloc(&c->binom, sizeof(double) * kBinomDim * kBinomDim));
    BBFG_HIP(launch_init_binom(c->binom, nullptr));
    BBFG_HIP(hipDeviceSynchronize());
    BBFG_TRY(c->ws.init());
    if (const char* path = std::getenv("BBFG_AUTOTUNE_CACHE")) {
        FILE* f = std::fopen(path, "r");
        if (f) {
            std::fclose(f);
            (void)load_autotune_file(*c, path);
        }
    }
    *out = c.get();
    g_ctx[dev] = c.release();
    return BBFG_OK;
}

int walk_slots(Context& c, int n, int f32, uint64_t* slots)
{
    const auto key = std::make_pair(n, f32);
    auto it = c.occ_single.find(key);
    int waves = 0;
    if (it == c.occ_single.end()) {
        const void* fn = walk_single_fn(n, f32);
        if (!fn) return set_error(BBFG_ERANGE, "no walk kernel for n=%d", n);
        int blocks = 0;
        BBFG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, fn, kWave, 0));
        waves = std::max(1, blocks);
        c.occ_single[key] = waves;
    } else {
        waves = it->second;
    }
    *slots = (uint64_t)waves * (uint64_t)c.n_cu;
    return BBFG_OK;
}

int batch_waves(Context& c, int bucket, int kind, int* waves)
{
    const auto key = std::make_pair(bucket, kind);
    auto it = c.occ_batch.find(key);
    if (it != c.occ_batch.end()) {
        *waves = it->second;
        return BBFG_OK;
    }
    const void* fn = kind == kKindMinors ? walk_minors_fn(bucket)
                     : kind == kKindCols  ? walk_cols_fn(bucket)
                                          : walk_batch_fn(bucket, kind);
    if (!fn) return set_error(BBFG_ERANGE, "no batch kernel for bucket %d", bucket);
    int blocks = 0;
    BBFG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, fn, kWave, 0));
    *waves = std::max(1, blocks);
    c.occ_batch[key] = *waves;
    return BBFG_OK;
}

int pair_occupancy(int np, bool pow, int* groups)
{
    const void* fn = pair_walk_fn(pow);
    const size_t lds = pair_lds_bytes((uint32_t)np);
    // the largest any launch needs: the attribute belongs to the function
    BBFG_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)pair_lds_bytes(kPairMax)));
    int blocks = 0;
    BBFG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, fn, kWave * kPairWaves, lds));
    *groups = std::max(1, blocks);
    return BBFG_OK;
}

uint32_t pair_table_blocks(uint64_t items, uint64_t positions, uint64_t np)
{
    return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(1024 / items, positions * np / 256));
}

int pair_groups(Context& c, int np, bool pow, int* groups)
{
    const auto key = std::make_pair(np, pow ? 1 : 0);
    auto it = c.occ_pair.find(key);
    if (it == c.occ_pair.end()) {
        int n = 1;
        BBFG_TRY(pair_occupancy(np, pow, &n));
        it = c.occ_pair.emplace(key, n).first;
    }
    *groups = it->second;
    return BBFG_OK;
}

int minor_groups(Context& c, int np, int* groups)
{
    const auto key = std::make_pair(-np, 0);
    auto it = c.occ_pair.find(key);
    if (it == c.occ_pair.end()) {
        int blocks = 0;
        BBFG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, minor_pairs_fn(np), kWave * kMinorWaves, 0));
        it = c.occ_pair.emplace(key, std::max(1, blocks)).first;
    }
    *groups = it->second;
    return BBFG_OK;
}

uint64_t batch_unit_length(Context& c, int n, int f32)
{
    auto it = c.batch_L.find(std::make_pair(n, f32));
    return it == c.batch_L.end() ? kDefaultBatchUnit : it->second;
}

int load_autotune_file(Context& c, const char* path)
{
    FILE* f = std::fopen(path, "r");
    if (!f) return set_error(BBFG_EINVAL, "cannot open autotune cache %s", path);
    int prec = 0, n = 0;
    unsigned long long L = 0;
    int count = 0;
    while (std::fscanf(f, "%d %d %llu", &prec, &n, &L) == 3) {
        if (n >= 1 && n <= kMaxN && L >= 1 && (prec == BBFG_FP64 || prec == BBFG_FP32 || prec == BBFG_MINORS)) {
            c.batch_L[std::make_pair(n, prec)] = (uint64_t)L;
            ++count;
            ++c.plan_epoch;
        }
    }
    std::fclose(f);
    return count > 0 ? BBFG_OK : set_error(BBFG_EINVAL, "no entries in autotune cache %s", path);
}

uint64_t PlanIndex::hash(const char* p, size_t n)
{
    uint64_t h = 0x9E3779B97F4A7C15ull ^ n;
    for (; n >= 8; p += 8, n -= 8) {
        uint64_t x;
        std::memcpy(&x, p, 8);
        h = (h ^ x) * 0xBF58476D1CE4E5B9ull;
        h ^= h >> 29;
    }
    uint64_t x = 0;
    std::memcpy(&x, p, n);
    h = (h ^ x) * 0x94D049BB133111EBull;
    return h ^ (h >> 32);
}

const std::shared_ptr<const HostPlan>* PlanIndex::find(uint64_t h, const char* p, size_t n) const
{
    if (slots.empty()) return nullptr;
    for (size_t i = h & (slots.size() - 1); slots[i].key; i = (i + 1) & (slots.size() - 1))
        if (slots[i].hash == h && slots[i].key->size() == n && std::memcmp(slots[i].key->data(), p, n) == 0)
            return slots[i].plan;
    return nullptr;
}

void PlanIndex::add(uint64_t h, const std::string* key, const std::shared_ptr<const HostPlan>* plan)
{
    if (2 * (used + 1) > slots.size()) {
        std::vector<Slot> old(std::max<size_t>(1024, 2 * slots.size()));
        old.swap(slots);
        used = 0;
        for (const Slot& o : old)
            if (o.key) add(o.hash, o.key, o.plan);
    }
    size_t i = h & (slots.size() - 1);
    while (slots[i].key) i = (i + 1) & (slots.size() - 1);
    slots[i].hash = h;
    slots[i].key = key;
    slots[i].plan = plan;
    ++used;
}

void PlanIndex::clear()
{
    std::vector<Slot>().swap(slots);
    used = 0;
}

int get_plan(Context& c, const int32_t* mult, int n_rows, int n_cols, int f32, int mode,
             std::shared_ptr<const HostPlan>* out, int kernel_cols, bool ryser, uint64_t pair_min)
{
    PlanParams pp = c.params;
    pp.ryser = ryser;
    if (mode == PLAN_BATCH) pp.l_batch = batch_unit_length(c, n_cols, f32);
    // everything the plan depends on, as bytes
    thread_local std::vector<char> key;
    const struct {
        int32_t n_cols, f32, ryser, kernel_cols;
        uint64_t l_batch, pair_min;
    } head = {n_cols, f32, ryser ? 1 : 0, kernel_cols, pp.l_batch, pair_min};
    const size_t mult_bytes = sizeof(int32_t) * (size_t)n_rows;
    key.resize(sizeof head + mult_bytes);
    std::memcpy(key.data(), &head, sizeof head);
    if (mult_bytes) std::memcpy(key.data() + sizeof head, mult, mult_bytes);
    const uint64_t hash = PlanIndex::hash(key.data(), key.size());
    if (const auto* found = c.plan_index.find(hash, key.data(), key.size())) {
        *out = *found;
        return BBFG_OK;
    }
    auto remember = [&](const std::shared_ptr<const HostPlan>& plan) {
        const auto it = c.plans.emplace(std::string(key.data(), key.size()), plan).first;
        c.plan_index.add(hash, &it->first, &it->second);
        *out = plan;
    };
    uint64_t slots = 1;
    if (f32 == kKindMinors && mode == PLAN_SINGLE) {
        // a lone leave-one-column-out walk fills the minors kernel's own
        // resident wavefronts (K = n_cols + 1 columns)
        const int bucket = minors_bucket_max(n_cols + 1);
        if (bucket < 0) return set_error(BBFG_ERANGE, "no minors kernel for %d columns", n_cols + 1);
        int waves = 1;
        BBFG_TRY(batch_waves(c, bucket, kKindMinors, &waves));
        slots = (uint64_t)waves * (uint64_t)c.n_cu;
    } else if (f32 == kKindCols && mode == PLAN_SINGLE) {
        // (prod_j c_j)^e over kernel_cols distinct columns: the column-power
        // kernel's resident wavefronts
        const int bucket = batch_bucket_max(kernel_cols, 0);
        if (bucket < 0) return set_error(BBFG_ERANGE, "no column-power kernel for %d columns", kernel_cols);
        int waves = 1;
        BBFG_TRY(batch_waves(c, bucket, kKindCols, &waves));
        slots = (uint64_t)waves * (uint64_t)c.n_cu;
    } else if (n_cols >= 1) {
        BBFG_TRY(walk_slots(c, n_cols, f32 == 1 ? 1 : 0, &slots));
    }
    if (c.tables.entries > c.table_entry_cap || c.plans.size() >= c.plan_cap) BBFG_TRY(flush_plans(c));
    auto p = std::make_shared<HostPlan>();
    std::string err;
    if (f32 == kKindMinors) {
        uint64_t groups = 1;
        if (mode == PLAN_SINGLE) {
            int per_cu = 1;
            BBFG_TRY(minor_groups(c, minor_pairs_per_wave(n_cols + 1), &per_cu));
            groups = (uint64_t)per_cu * (uint64_t)c.n_cu;
        }
        if (build_minor_pair_plan(mult, n_rows, n_cols, groups, pp, *p, err, &c.tables)) {
            remember(p);
            return BBFG_OK;
        }
        if (!err.empty()) return set_error(BBFG_ERANGE, "%s", err.c_str());
    }
    const int rc = build_plan(mult, n_rows, n_cols, slots, pp, *p, err, &c.tables);
    if (rc != BBFG_OK) return set_error(rc, "%s", err.c_str());
    if (f32 == 0 || f32 == kKindCols)
        p->pair = build_pair_plan(*p, kernel_cols > 0 ? kernel_cols : n_cols, mode == PLAN_SINGLE ? (uint32_t)c.n_cu : 0u,
                                  pair_min);
    remember(p);
    return BBFG_OK;
}

int table_reserve(Context& c, size_t bytes, TabEntry** out)
{
    const size_t need = (bytes + 255) / 256 * 256;
    if (c.tab_chunk < c.tab_chunks.size() && c.tab_used + need > c.tab_chunks[c.tab_chunk]->cap) {
        ++c.tab_chunk;
        c.tab_used = 0;
    }
    if (c.tab_chunk == c.tab_chunks.size()) {
        auto b = std::make_unique<DevBuf>();
        BBFG_TRY(b->ensure(std::max<size_t>(need, kTableChunkBytes)));
        c.tab_chunks.push_back(std::move(b));
        c.tab_used = 0;
    }
    *out = reinterpret_cast<TabEntry*>(c.tab_chunks[c.tab_chunk]->as<char>() + c.tab_used);
    c.tab_used += need;
    return BBFG_OK;
}

int flush_plans(Context& c)
{
    // device tables are about to be reused: nothing may still read them
    BBFG_HIP(hipDeviceSynchronize());
    for (auto& kv : c.graphs) (void)hipGraphExecDestroy(kv.second);
    c.graphs.clear();
    c.graph_seen.clear();
    c.dev_tables.clear();
    c.tab_chunk = 0;
    c.tab_used = 0;
    c.tables.tables.clear();
    c.tables.entries = 0;
    c.plan_index.clear();
    c.plans.clear();
    return BBFG_OK;
}

// ---------------------------------------------------------------------------
// the permanent engine
// ---------------------------------------------------------------------------
namespace {

// A positive cost as 16 ordered bits (its exponent and five bits of fraction):
// what the order of units needs.
uint16_t coarse_cost(double x)
{
    uint64_t bits;
    std::memcpy(&bits, &x, sizeof bits);
    return (uint16_t)(bits >> 47);
}

// Sorts item indices by falling cost, equal ones in their order (two counting
// passes; comparing through the plans took 0.15 ms for 4096 items).
void longest_first(const std::vector<uint16_t>& cost, std::vector<size_t>& order)
{
    std::vector<size_t> other(order.size());
    for (int shift = 0; shift < 16; shift += 8) {
        size_t first[257] = {};
        for (size_t i : order) ++first[256 - (cost[i] >> shift & 255)];
        for (int b = 1; b <= 256; ++b) first[b] += first[b - 1];
        for (size_t i : order) other[first[255 - (cost[i] >> shift & 255)]++] = i;
        order.swap(other);
    }
}

// The fields of a descriptor that depend on its plan alone.
void fill_walk_desc(PermDesc& d, const HostPlan& p, int n_cols, bool f32)
{
    d.units_per_group = p.units_per_group;
    d.span = p.span;
    d.n = n_cols;
    d.r = p.r;
    d.Q = p.Q;
    d.lane_product = p.lane_product;
    d.groups = p.groups;
    d.scale = std::ldexp(1.0, p.scale_log2);
    d.err_coeff = p.err_coeff * (f32 ? 0x1.0p-24 : 0x1.0p-53);
    d.col_pow = 1;
    d.mag_every = 1;
}

}  // namespace

uint64_t pair_inner_rows(const PairPlan& p)
{
    uint64_t rows = 0;
    for (int k : p.inner) rows |= uint64_t(1) << k;
    return rows;
}

uint64_t fill_pair_desc(PairDesc& q, const PermDesc& d, const HostPlan& p, uint64_t unit_base, uint64_t direct_off,
                        uint64_t* table_doubles)
{
    const PairPlan& pp = *p.pair;
    std::memset(&q, 0, sizeof q);
    q.a_off = d.a_off;
    q.part_base = d.part_base;
    q.direct_off = (uint32_t)direct_off;
    q.unit_base = (uint32_t)unit_base;
    q.units = (uint32_t)pp.units;
    q.rowinfo_off = d.rowinfo_off;
    q.lane_product = pp.lane_product;
    q.mid = pp.mid;
    q.high = pp.high;
    q.col_pow = d.col_pow;
    q.n = d.n;
    q.np = (d.n + 1) / 2;
    q.r = d.r;
    for (int k = 0; k < kPairBits; ++k) q.inner[k] = pp.inner[k];
    q.mids = (int32_t)pp.mid_rows.size();
    for (int i = 0; i < q.mids; ++i) q.mid_row[i] = pp.mid_rows[(size_t)i];
    // 64-byte aligned tables
    auto take = [table_doubles](uint64_t doubles) {
        const uint64_t off = *table_doubles;
        *table_doubles += (doubles + 7) / 8 * 8;
        return off;
    };
    q.mid_off = take((uint64_t)q.mid * (uint64_t)q.np * 2 * kPairSlots);
    q.weight_off = take(q.mid);
    q.const_off = take((uint64_t)q.np * 2 * kPairConsts);
    return q.mid;
}

int run_short(Context& c, Workspace& w, const PermItem& item, double* out, RunResult* rr, bool* done)
{
    *done = false;
    const HostPlan& p = *item.plan;
    if (p.pair || p.n > kShortMaxN || p.units > kShortMaxUnits || walk_short_lds(p.n, p.r) > kShortLdsBytes ||
        item.row_map || item.col_map || item.targets || item.col_pow)
        return BBFG_OK;
    hipStream_t s = current_stream();
    auto te = c.dev_tables.find(p.table.get());
    if (te == c.dev_tables.end()) return BBFG_OK;
    if (te->second.ready && te->second.stream != s) {
        if (hipEventQuery(te->second.ready.get()) != hipSuccess) return BBFG_OK;
        te->second.ready.reset();
    }
    BBFG_TRY(w.partials.ensure(sizeof(double) * kPartialDoubles * (size_t)p.units));
    BBFG_TRY(w.hres.ensure(sizeof(double) * 5));
    ShortArgs A;
    std::memset(&A, 0, sizeof A);
    A.d.tab = te->second.dev;
    fill_walk_desc(A.d, p, p.n, false);
    A.d.units = p.units;
    for (int k = 0; k < p.r; ++k) {
        A.rows[k] = p.rows[(size_t)k];
        A.src_row[k] = (uint32_t)p.src_row[(size_t)k];
    }
    A.src = item.src + 2 * item.src_off;
    A.ld = item.ld;
    A.binom = c.binom;
    A.partials = w.partials.as<double>();
    A.done = w.short_done.as<uint32_t>();
    A.start = reinterpret_cast<unsigned long long*>(A.done + (1 + kShortCounters) * kCounterStride);
    A.out = w.hres.as<double>();
    BBFG_HIP(launch_walk_short(s, A));
    BBFG_HIP(hipStreamSynchronize(s));
    std::memcpy(out, w.hres.p, sizeof(double) * 4);
    // the launch times itself: two recorded events take 5 us of a call
    rr->kernel_ms = c.clock_khz > 0 ? w.hres.as<double>()[4] / c.clock_khz : 0.0;
    rr->units = p.units;
    *done = true;
    return BBFG_OK;
}

int run_perms(Context& c, Workspace& w, std::vector<PermItem>& items, int f32, bool single, double* out_host,
              double* diag_host, RunResult* rr, bool sync, bool use_graph)
{
    const size_t nitem = items.size();
    if (nitem == 0) return BBFG_OK;
    if (single && nitem != 1) return set_error(BBFG_EINVAL, "internal: single launch with %zu items", nitem);
    hipStream_t s = current_stream();
    // leave-one-column-out items (targets > 0) run in their own launches
    const bool minors = items[0].targets > 0;
    const bool powcols = items[0].col_pow >= 2;
    for (auto& it : items) {
        if ((it.targets > 0) != minors || (minors && (single || f32 || it.targets > it.plan->n + 1)))
            return set_error(BBFG_EINVAL, "internal: bad mix of minor items");
        if ((it.col_pow >= 2) != powcols ||
            (powcols && (single || f32 || minors || it.arena_cols < 1 || it.arena_cols * it.col_pow != it.plan->n)))
            return set_error(BBFG_EINVAL, "internal: bad mix of column-multiplicity items");
    }
    // columns held per item: the plan's n, plus the left-out column for minors,
    // or the distinct columns of an item with column multiplicities
    auto cols_of = [&](const PermItem& it) {
        return it.arena_cols > 0 ? it.arena_cols : it.plan->n + (it.targets > 0 ? 1 : 0);
    };
    auto stride_of = [](const PermItem& it) { return (uint64_t)(it.targets > 0 ? it.targets : 1); };

    // distinct plans (row records are shared between equal shapes; Gray tables
    // are resident on the device and shared between equal low radices); each
    // plan records its slot for this evaluation in its slot_* fields
    static std::atomic<uint64_t> evaluations{0};
    const uint64_t call = ++evaluations;
    std::vector<const HostPlan*> distinct;
    size_t n_rowinfo = 0, n_srcrow = 0, n_srccol = 0;
    struct Upload {
        const HostPlan* plan;
        TabEntry* dst;
        size_t bytes, off;
    };
    std::vector<Upload> uploads;        // tables this evaluation brings to the device
    std::unordered_map<const void*, TabEntry*> uploading;  // their host tables -> pool space
    std::vector<EventPtr> table_waits;  // uploads queued on other streams, maybe still running
    size_t upload_bytes = 0;
    uint64_t a_elems = 0;
    int nmax = 0;
    // items that go over pairs of columns have a launch of their own: the pair
    // walk (plans that hold its split) or the leave-one-column-out walk over pairs
    auto by_pairs = [&](const PermItem& it) { return minors ? it.plan->minor_digits > 0 : !f32 && it.plan->pair != nullptr; };
    auto arena_of = [&](const PermItem& it, int nc) -> uint64_t {
        const uint64_t rows = (uint64_t)it.plan->r;
        if (!by_pairs(it)) return rows * (uint64_t)nc * 3u;  // a (r x n) + a2 (2r x n)
        if (!minors) return rows * (uint64_t)nc;
        const int np = minor_pairs_per_wave(nc);  // rows, steps
        return rows * 2 * (uint64_t)np * kMinorWaves + minor_step_elems(it.plan->r, it.plan->minor_digits, np);
    };
    size_t npair = 0;
    int np_max = 0;
    for (auto& it : items) {
        const HostPlan* p = it.plan.get();
        if (by_pairs(it)) {
            const int nc = cols_of(it);
            ++npair;
            np_max = std::max(np_max, minors ? minor_pairs_per_wave(nc) : (nc + 1) / 2);
        }
        if (by_pairs(it) && !minors) {
            const int nc = cols_of(it);
            if (p->slot_call != call) {
                p->slot_call = call;
                p->slot_rowinfo = n_rowinfo;
                p->slot_table = nullptr;
                distinct.push_back(p);
                n_rowinfo += (size_t)p->r;
            }
            n_srcrow += (size_t)p->r;
            if (it.col_map) n_srccol += (size_t)nc;
            a_elems += arena_of(it, nc);
            continue;
        }
        if (p->slot_call != call) {
            auto te = c.dev_tables.find(p->table.get());
            auto up = uploading.find(p->table.get());
            const TabEntry* dt = nullptr;
            if (te != c.dev_tables.end()) {
                DevTable& e = te->second;
                if (e.ready && e.stream != s) {
                    if (hipEventQuery(e.ready.get()) == hipSuccess) e.ready.reset();
                    else table_waits.push_back(e.ready);
                }
                dt = e.dev;
            } else if (up != uploading.end()) {
                dt = up->second;
            } else {
                // listed as resident only once its upload is queued (below)
                const size_t bytes = sizeof(TabEntry) * p->table->size();
                TabEntry* dst = nullptr;
                BBFG_TRY(table_reserve(c, bytes, &dst));
                uploads.push_back({p, dst, bytes, upload_bytes});
                uploading[p->table.get()] = dst;
                upload_bytes += (bytes + 255) / 256 * 256;
                dt = dst;
            }
            p->slot_call = call;
            p->slot_rowinfo = n_rowinfo;
            p->slot_table = dt;
            distinct.push_back(p);
            n_rowinfo += (size_t)p->r;
        }
        const int nc = cols_of(it);
        n_srcrow += (size_t)p->r;
        if (it.col_map) n_srccol += (size_t)nc;
        a_elems += arena_of(it, nc);
        if (!by_pairs(it)) nmax = std::max(nmax, nc);
    }

    // the arena starts with a flag per item, for the walks over pairs
    const uint64_t n_flags = npair ? nitem : 0;
    a_elems += n_flags;

    // unit numbering of each launch: longest units first (items ordered by
    // per-unit cost)
    const size_t nwalk = nitem - npair;
    std::vector<size_t> order, order_pair;
    order.reserve(nwalk);
    order_pair.reserve(npair);
    for (size_t i = 0; i < nitem; ++i) (by_pairs(items[i]) ? order_pair : order).push_back(i);
    if (!single) {
        std::vector<uint16_t> cost(nitem);
        for (size_t i = 0; i < nitem; ++i) {
            const HostPlan& p = *items[i].plan;
            const double nc = cols_of(items[i]);
            if (by_pairs(items[i]) && !minors) cost[i] = coarse_cost((double)p.pair->mid * nc);
            else
                cost[i] = coarse_cost((double)p.span / (double)p.units_per_group *
                                      (6.0 * nc - 2.0 + 12.0 * items[i].targets));
        }
        longest_first(cost, order);
        longest_first(cost, order_pair);
    }
    auto units_of = [&](const PermItem& it) {
        return by_pairs(it) && !minors ? it.plan->pair->units : it.plan->units;
    };
    std::vector<uint64_t> unit_base(nitem), part_base(nitem);
    uint64_t total_units = 0, pair_units = 0, total_parts = 0;
    for (size_t i : order) {
        unit_base[i] = total_units;
        part_base[i] = total_parts;
        total_units += items[i].plan->units;
        total_parts += items[i].plan->units * stride_of(items[i]);
    }
    for (size_t i : order_pair) {
        unit_base[i] = pair_units;
        part_base[i] = total_parts;
        pair_units += units_of(items[i]);
        total_parts += units_of(items[i]) * stride_of(items[i]);
    }
    if (total_units > 0xFFFFFFF0ull || pair_units > 0xFFFFFFF0ull)
        return set_error(BBFG_ERANGE, "too many work units (%llu)", (unsigned long long)(total_units + pair_units));
    // results: one per plain item, `targets` per minor item (item order)
    std::vector<uint32_t> res_base(nitem);
    uint64_t nres = 0;
    for (size_t i = 0; i < nitem; ++i) {
        res_base[i] = (uint32_t)nres;
        nres += stride_of(items[i]);
    }
    if (nres > 0x7FFFFFFFull) return set_error(BBFG_ERANGE, "too many results (%llu)", (unsigned long long)nres);

    // host metadata image
    Layout L;
    const size_t off_desc = L.add(sizeof(PermDesc) * nitem);
    const size_t off_row = L.add(sizeof(RowInfo) * std::max<size_t>(1, n_rowinfo));
    const size_t off_prep = L.add(sizeof(PrepItem) * nitem);
    const size_t off_src = L.add(sizeof(uint32_t) * std::max<size_t>(1, n_srcrow));
    const size_t off_col = L.add(sizeof(uint32_t) * std::max<size_t>(1, n_srccol));
    // unit -> item index of a launch (a single walk needs none, the pair walk
    // makes its own on the device)
    struct UnitIndex {
        bool on = false;
        size_t nchunk = 0, base = 0, order = 0, chunk = 0;
    } ix_walk, ix_pair;
    auto place_index = [&L](UnitIndex& ix, size_t count, uint64_t units) {
        ix.on = true;
        ix.nchunk = (size_t)((units + kUnitChunk - 1) / kUnitChunk);
        ix.base = L.add(sizeof(uint32_t) * (count + 1));
        ix.order = L.add(sizeof(uint32_t) * count);
        ix.chunk = L.add(sizeof(uint32_t) * (ix.nchunk + 1));
    };
    if (!single && nwalk) place_index(ix_walk, nwalk, total_units);
    if (minors && npair) place_index(ix_pair, npair, pair_units);
    const size_t off_pair = npair && !minors ? L.add(sizeof(PairDesc) * npair) : 0;
    const size_t off_ritem = L.add(sizeof(uint32_t) * (size_t)nres);
    const size_t off_tabs = L.add(std::max<size_t>(1, upload_bytes));
    BBFG_TRY(w.hmeta.ensure(L.size));
    BBFG_TRY(w.meta.ensure(L.size));
    char* H = w.hmeta.as<char>();
    PermDesc* hd = reinterpret_cast<PermDesc*>(H + off_desc);
    RowInfo* hr = reinterpret_cast<RowInfo*>(H + off_row);
    PrepItem* hp = reinterpret_cast<PrepItem*>(H + off_prep);
    uint32_t* hs = reinterpret_cast<uint32_t*>(H + off_src);
    uint32_t* hc = reinterpret_cast<uint32_t*>(H + off_col);
    uint32_t* hri = reinterpret_cast<uint32_t*>(H + off_ritem);
    for (const HostPlan* p : distinct)
        std::memcpy(hr + p->slot_rowinfo, (p->pair && !f32 ? p->pair->rows : p->rows).data(),
                    sizeof(RowInfo) * (size_t)p->r);
    for (const Upload& u : uploads) std::memcpy(H + off_tabs + u.off, u.plan->table->data(), u.bytes);
    uint64_t a_cursor = n_flags;
    size_t s_cursor = 0, c_cursor = 0;
    for (size_t i = 0; i < nitem; ++i) {
        const HostPlan& p = *items[i].plan;
        const int nc = cols_of(items[i]);
        PermDesc& d = hd[i];
        std::memset(&d, 0, sizeof d);
        d.a_off = a_cursor;
        const bool pair = by_pairs(items[i]);
        const int np = pair && minors ? minor_pairs_per_wave(nc) : 0;
        d.a2_off = a_cursor + (uint64_t)p.r * (np ? 2u * (uint64_t)np * kMinorWaves : (uint64_t)nc);
        a_cursor += arena_of(items[i], nc);
        d.tab = p.slot_table;
        d.unit_base = unit_base[i];
        d.units = units_of(items[i]);
        fill_walk_desc(d, p, nc, f32 != 0);
        d.rowinfo_off = (uint32_t)p.slot_rowinfo;
        d.part_base = part_base[i];
        d.targets = (uint32_t)items[i].targets;
        d.res_base = res_base[i];
        d.col_pow = np ? (uint32_t)p.minor_digits : items[i].col_pow >= 2 ? (uint32_t)items[i].col_pow : 1u;
        d.mag_every = mag_every_for(p.units_per_group);
        for (uint64_t t = 0; t < stride_of(items[i]); ++t) hri[res_base[i] + t] = (uint32_t)i;
        PrepItem& q = hp[i];
        std::memset(&q, 0, sizeof q);
        q.src = items[i].src;
        q.src_off = items[i].src_off;
        q.ld = items[i].ld;
        q.a_off = d.a_off;
        q.a2_off = d.a2_off;
        q.srcrow_off = (uint32_t)s_cursor;
        q.n = nc;
        q.r = p.r;
        q.f32 = f32;
        q.rows_only = pair ? 1 : 0;
        q.np = np;
        q.digits = p.minor_digits;
        q.direct_off = i;
        if (np) q.inner_rows = ((uint64_t(1) << p.minor_digits) - 1) << (p.r - p.minor_digits);
        else if (pair) q.inner_rows = pair_inner_rows(*p.pair);
        for (int k = 0; k < p.r; ++k) {
            const int ur = p.src_row[(size_t)k];
            hs[s_cursor++] = (uint32_t)(items[i].row_map ? items[i].row_map[ur] : ur);
        }
        if (items[i].col_map) {
            q.srccol_off = (uint32_t)c_cursor;
            for (int j = 0; j < nc; ++j) hc[c_cursor++] = (uint32_t)items[i].col_map[j];
        } else {
            q.srccol_off = kIdentityCols;
        }
    }
    auto fill_index = [&](const UnitIndex& ix, const std::vector<size_t>& ord, uint64_t units) {
        if (!ix.on) return;
        uint32_t* hb = reinterpret_cast<uint32_t*>(H + ix.base);
        uint32_t* ho = reinterpret_cast<uint32_t*>(H + ix.order);
        uint32_t* hk = reinterpret_cast<uint32_t*>(H + ix.chunk);
        for (size_t oi = 0; oi < ord.size(); ++oi) {
            const size_t i = ord[oi];
            const uint64_t b = unit_base[i], e = b + units_of(items[i]);
            hb[oi] = (uint32_t)b;
            ho[oi] = (uint32_t)i;
            for (uint64_t c = (b + kUnitChunk - 1) / kUnitChunk; c * kUnitChunk < e; ++c) hk[c] = (uint32_t)oi;
        }
        hb[ord.size()] = (uint32_t)units;
        hk[ix.nchunk] = (uint32_t)(ord.size() - 1);
    };
    fill_index(ix_walk, order, total_units);
    fill_index(ix_pair, order_pair, pair_units);
    // the pair walk's items in launches whose tables stay within their bound
    struct PairLaunch {
        size_t first = 0, items = 0;  // in order_pair
        uint64_t units = 0, doubles = 0, unit_map = 0, mid_max = 0, grid = 0;
        uint32_t table_blocks = 0;
        PairArgs args;
    };
    std::vector<PairLaunch> pair_launches;
    if (npair && !minors) {
        PairDesc* hpd = reinterpret_cast<PairDesc*>(H + off_pair);
        uint64_t most = 0, unit_first = 0;
        for (size_t oi = 0; oi < npair;) {
            PairLaunch l;
            l.first = oi;
            for (; oi < npair; ++oi, ++l.items) {
                const size_t i = order_pair[oi];
                uint64_t doubles = l.doubles;
                const uint64_t mid = fill_pair_desc(hpd[oi], hd[i], *items[i].plan, unit_base[i] - unit_first, i, &doubles);
                if (l.items && sizeof(double) * doubles > kPairTableBytes) break;
                l.doubles = doubles;
                l.mid_max = std::max(l.mid_max, mid);
                l.units += units_of(items[i]);
            }
            unit_first += l.units;
            l.unit_map = l.doubles;  // the units' items follow the tables
            if (l.items > 1) l.doubles += (l.units + 1) / 2;
            most = std::max(most, l.doubles);
            pair_launches.push_back(l);
        }
        BBFG_TRY(w.pair_tables.ensure(sizeof(double) * most));
    }

    // device buffers
    if (f32) BBFG_TRY(w.arena_f.ensure(sizeof(float) * 2 * std::max<uint64_t>(1, a_elems)));
    else BBFG_TRY(w.arena_d.ensure(sizeof(double) * 2 * std::max<uint64_t>(1, a_elems)));
    BBFG_TRY(w.partials.ensure(sizeof(double) * kPartialDoubles * (size_t)total_parts));
    BBFG_TRY(w.results.ensure(sizeof(double) * 4 * (size_t)nres));
    BBFG_TRY(w.hres.ensure(sizeof(double) * 4 * (size_t)nres));
    char* D = w.meta.as<char>();

    WalkArgs W;
    std::memset(&W, 0, sizeof W);
    W.descs = reinterpret_cast<const PermDesc*>(D + off_desc);
    W.rowinfo = reinterpret_cast<const RowInfo*>(D + off_row);
    W.a = w.arena_d.as<double>();
    W.a2 = w.arena_d.as<double>();
    W.af = w.arena_f.as<float>();
    W.a2f = w.arena_f.as<float>();
    W.binom = c.binom;
    W.partials = w.partials.as<double>();
    auto set_index = [&](WalkArgs& w_, const UnitIndex& ix) {
        w_.ubase = ix.on ? reinterpret_cast<const uint32_t*>(D + ix.base) : nullptr;
        w_.uorder = ix.on ? reinterpret_cast<const uint32_t*>(D + ix.order) : nullptr;
        w_.uchunk = ix.on ? reinterpret_cast<const uint32_t*>(D + ix.chunk) : nullptr;
    };
    set_index(W, ix_walk);
    W.nitem = (uint32_t)nitem;
    W.counter = w.counter.as<uint32_t>();
    W.total_units = (uint32_t)total_units;

    WalkArgs WP = W;  // the leave-one-column-out walk over pairs
    uint64_t pair_grid = 0;
    if (npair && minors) {
        set_index(WP, ix_pair);
        WP.counter = W.counter + kCounterStride;
        WP.total_units = (uint32_t)pair_units;
        int groups = 1;
        BBFG_TRY(minor_groups(c, np_max, &groups));
        pair_grid = std::min<uint64_t>((uint64_t)groups * (uint64_t)c.n_cu, pair_units);
    }
    for (PairLaunch& l : pair_launches) {
        PairArgs& PA = l.args;
        std::memset(&PA, 0, sizeof PA);
        PA.descs = reinterpret_cast<const PairDesc*>(D + off_pair) + l.first;
        PA.rowinfo = W.rowinfo;
        PA.a = W.a;
        PA.tables = w.pair_tables.as<double>();
        PA.binom = c.binom;
        PA.partials = W.partials;
        PA.unit_item = l.items > 1 ? reinterpret_cast<uint32_t*>(PA.tables + l.unit_map) : nullptr;
        PA.counter = W.counter + kCounterStride;
        PA.total_units = (uint32_t)l.units;
        PA.np_max = (uint32_t)np_max;
        int groups = 1;
        BBFG_TRY(pair_groups(c, np_max, powcols, &groups));
        l.grid = std::min<uint64_t>((uint64_t)groups * (uint64_t)c.n_cu, l.units);
        l.table_blocks = pair_table_blocks(l.items, l.mid_max, (uint64_t)np_max);
    }
    int bucket = 0;
    uint64_t grid = total_units;
    if (!single && nwalk) {
        bucket = minors ? minors_bucket_max(nmax) : batch_bucket_max(nmax, f32);
        if (bucket < 0) return set_error(BBFG_ERANGE, "no batch kernel for n=%d", nmax);
        int waves = 1;
        BBFG_TRY(batch_waves(c, bucket, minors ? kKindMinors : (powcols ? kKindCols : f32), &waves));
        grid = std::min<uint64_t>((uint64_t)waves * (uint64_t)c.n_cu, total_units);
    }
    double* R = w.results.as<double>();
    double* HR = w.hres.as<double>();

    // Everything one evaluation puts on a stream (also what a graph captures):
    // metadata upload, gather, walks and finalize.  No memset: the unit counters
    // are cleared by the gather kernel.  A short metadata image is read and copied
    // by the gather kernel itself, and a few results that the host waits for go
    // straight to pinned host memory (many small writes over the bus take longer
    // than a copy: 4096 results 0.05 ms).
    const bool short_image = off_tabs <= kShortImageBytes;
    const char* M = short_image ? H : D;
    const bool direct = sync && nres <= kDirectResults;
    double* out = direct ? HR : R;
    auto enqueue = [&](hipStream_t q, bool timed) -> int {
        if (!short_image) BBFG_HIP(hipMemcpyAsync(D, H, off_tabs, hipMemcpyHostToDevice, q));
        BBFG_HIP(launch_prep((uint32_t)nitem, q, reinterpret_cast<const PrepItem*>(M + off_prep),
                             reinterpret_cast<const uint32_t*>(M + off_src),
                             reinterpret_cast<const uint32_t*>(M + off_col), w.arena_d.as<double>(),
                             w.arena_d.as<double>(), w.arena_f.as<float>(), w.arena_f.as<float>(), W.counter,
                             H, D, short_image ? off_tabs : 0));
        if (timed && pair_launches.empty()) BBFG_HIP(hipEventRecord(w.ev0, q));
        if (npair && minors) BBFG_HIP(launch_minor_pairs(np_max, (uint32_t)pair_grid, q, WP));
        for (const PairLaunch& l : pair_launches) {
            BBFG_HIP(launch_pair_tables((uint32_t)l.items, l.table_blocks, q, l.args));
            if (timed && l.first == 0) BBFG_HIP(hipEventRecord(w.ev0, q));
            BBFG_HIP(launch_pair_walk(powcols, (uint32_t)l.grid, q, l.args));
        }
        if (!nwalk) {
        } else if (single) BBFG_HIP(launch_walk_single(items[0].plan->n, f32, (uint32_t)total_units, q, W, 0u));
        else if (minors) BBFG_HIP(launch_walk_minors(bucket, (uint32_t)grid, q, W));
        else if (powcols) BBFG_HIP(launch_walk_cols(bucket, (uint32_t)grid, q, W));
        else BBFG_HIP(launch_walk_batch(bucket, f32, (uint32_t)grid, q, W));
        if (timed) BBFG_HIP(hipEventRecord(w.ev1, q));
        BBFG_HIP(launch_finalize((uint32_t)nres, q, W.descs, reinterpret_cast<const uint32_t*>(D + off_ritem),
                                 W.partials, out, out + 2 * nres));
        if (sync && !direct) BBFG_HIP(hipMemcpyAsync(HR, R, sizeof(double) * 4 * nres, hipMemcpyDeviceToHost, q));
        return BBFG_OK;
    };

    // Gray tables new to the device: copied from the pinned image in stream
    // order (outside any captured graph), then an event that other streams wait
    // for; tables uploaded on other streams and maybe not yet complete are waited
    // for on the device
    for (const EventPtr& e : table_waits) BBFG_HIP(hipStreamWaitEvent(s, e.get(), 0));
    if (!uploads.empty()) {
        hipEvent_t ev = nullptr;
        BBFG_HIP(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
        EventPtr ready(ev, [](hipEvent_t e) { (void)hipEventDestroy(e); });
        for (const Upload& u : uploads)
            BBFG_HIP(hipMemcpyAsync(u.dst, H + off_tabs + u.off, u.bytes, hipMemcpyHostToDevice, s));
        BBFG_HIP(hipEventRecord(ev, s));
        for (const Upload& u : uploads) {
            DevTable e;
            e.host = u.plan->table;
            e.dev = u.dst;
            e.ready = ready;
            e.stream = s;
            c.dev_tables[u.plan->table.get()] = std::move(e);
        }
    }

    bool launched = false;
    if (use_graph && sync) {
        // A launch sequence seen before is captured once and replayed.  The
        // captured nodes hold sizes and addresses only (every kernel reads its
        // shapes from the uploaded metadata), so the key is the layout of the
        // metadata image, the launch shapes and every buffer address; the image
        // itself is copied again by each replay.
        uint64_t key = 1469598103934665603ull;
        auto mix = [&key](const void* p, size_t n) {
            const unsigned char* b = static_cast<const unsigned char*>(p);
            for (size_t i = 0; i < n; ++i) key = (key ^ b[i]) * 1099511628211ull;
        };
        mix(&W, sizeof W);
        mix(&WP, sizeof WP);
        for (const PairLaunch& l : pair_launches) {
            mix(&l.args, sizeof l.args);
            const uint64_t shape[] = {l.items, l.grid, l.table_blocks};
            mix(shape, sizeof shape);
        }
        const uint64_t extra[] = {nitem, nres, (uint64_t)single, (uint64_t)minors, (uint64_t)powcols, (uint64_t)f32,
                                  (uint64_t)bucket,
                                  grid, L.size, off_desc, off_row, off_prep, off_src, off_col, ix_walk.base, ix_walk.order, ix_walk.chunk,
                                  ix_pair.base, ix_pair.order, ix_pair.chunk, off_pair, off_ritem, off_tabs,
                                  npair, pair_grid,
                                  (uint64_t)(uintptr_t)H, (uint64_t)(uintptr_t)D, (uint64_t)(uintptr_t)R,
                                  (uint64_t)(uintptr_t)HR, (uint64_t)(uintptr_t)w.arena_d.p,
                                  (uint64_t)(uintptr_t)w.arena_f.p};
        mix(extra, sizeof extra);
        auto git = c.graphs.find(key);
        if (git == c.graphs.end() && c.graph_seen.count(key)) {
            if (!c.cstream) BBFG_HIP(hipStreamCreateWithFlags(&c.cstream, hipStreamNonBlocking));
            hipGraph_t g = nullptr;
            BBFG_HIP(hipStreamBeginCapture(c.cstream, hipStreamCaptureModeThreadLocal));
            const int rc = enqueue(c.cstream, false);
            hipGraph_t gcap = nullptr;
            const hipError_t ec = hipStreamEndCapture(c.cstream, &gcap);
            if (rc != BBFG_OK) return rc;
            if (ec != hipSuccess) return set_error(BBFG_EDEVICE, "hipStreamEndCapture: %s", hipGetErrorString(ec));
            g = gcap;
            hipGraphExec_t exec = nullptr;
            BBFG_HIP(hipGraphInstantiate(&exec, g, nullptr, nullptr, 0));
            (void)hipGraphDestroy(g);
            if (c.graphs.size() >= 64) {
                for (auto& kv : c.graphs) (void)hipGraphExecDestroy(kv.second);
                c.graphs.clear();
            }
            git = c.graphs.emplace(key, exec).first;
        }
        if (git != c.graphs.end()) {
            BBFG_HIP(hipEventRecord(w.ev0, s));
            BBFG_HIP(hipGraphLaunch(git->second, s));
            BBFG_HIP(hipEventRecord(w.ev1, s));
            launched = true;
            if (rr) rr->graph = true;
        } else {
            if (c.graph_seen.size() > 4096) c.graph_seen.clear();
            c.graph_seen.insert(key);
        }
    }
    if (!launched) BBFG_TRY(enqueue(s, true));
    if (rr) rr->units = total_units + pair_units;
    if (!sync) return BBFG_OK;
    BBFG_HIP(hipStreamSynchronize(s));
    if (out_host) std::memcpy(out_host, HR, sizeof(double) * 2 * nres);
    if (diag_host) std::memcpy(diag_host, HR + 2 * nres, sizeof(double) * 2 * nres);
    if (rr) {
        float ms = 0.f;
        BBFG_HIP(hipEventElapsedTime(&ms, w.ev0, w.ev1));
        rr->kernel_ms = ms;
        rr->units = total_units + pair_units;
    }
    return BBFG_OK;
}

}  // namespace bbfg
