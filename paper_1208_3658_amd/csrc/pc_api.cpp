// pc_api.cpp -- the C ABI of libpc.so: validation, device memory, edge-set
// tables, catalogue conversion and residency, and the batched launch.
#include <hip/hip_runtime.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <unordered_map>
#include <vector>

#include "../../include/pc.h"
#include "pc_internal.hpp"
#include "pc_math.h"
#include "pc_runtime.hpp"
#include "../../include/pc_debug.h"

namespace pc {

// preparation steps that do not depend on the tile size (pc_prep.hip)
hipError_t launch_zero(void *p, size_t bytes, hipStream_t st);
hipError_t launch_zero_put(void *p, size_t bytes, void *dst, const void *src, size_t n, hipStream_t st);
int64_t convert_blocks(int64_t n);
int64_t order_blocks(int64_t n);
uint32_t order_buckets(int64_t n, int per_point);
size_t scan_sums_words(int64_t m);
hipError_t launch_convert(const SrcDesc *srcs, int n_srcs, int64_t blocks, hipStream_t st);
hipError_t launch_order(const ViewDesc *views, int n_views, int64_t blocks, uint32_t *hist, int64_t buckets,
                        uint32_t *sums, hipStream_t st);
hipError_t launch_add_copies(unsigned long long *dst, const unsigned long long *src, int64_t n, int32_t n_copies,
                             hipStream_t st);

// the per-tile-size steps (pc_kernels.hip, pc_prep.hip; one instance per size)
#define PC_TILE_STEPS                                                                                              \
    hipError_t launch_count(bool fp64, bool mc, bool compact, const SegDesc *segs, int32_t n_segs,                 \
                            const TableDesc *tabs,                                                                 \
                            const uint64_t *items, const unsigned long long *n_items, const uint64_t *sub,         \
                            uint64_t total_items, uint32_t lut_lds_off, uint32_t stage_lds_off,                    \
                            unsigned long long *queue, unsigned long long *rechecked, int chunk,                   \
                            uint32_t lds_bytes, int grid, uint64_t flush_cap, hipStream_t st);                     \
    hipError_t launch_bounds(const ViewDesc *views, int n_views, int64_t tiles, hipStream_t st);                   \
    hipError_t launch_prune(const SegDesc *segs, int32_t n_segs, const TableDesc *tabs, int64_t total_rows,        \
                            uint64_t *survivors, uint64_t *sub, unsigned long long *meta, int32_t mfma_ok,         \
                            int32_t split_ok, bool blocks, hipStream_t st);                                        \
    hipError_t count_occupancy(bool fp64, bool mc, bool compact, uint32_t lds_bytes, int *blocks_per_cu);          \
    hipError_t set_max_lds(uint32_t bytes);
namespace t256 { PC_TILE_STEPS }
// the block kernel (pc_blocks.hip)
namespace blk {
hipError_t launch_bounds(const ViewDesc *views, int n_views, int64_t tiles, hipStream_t st);
hipError_t launch_products(int32_t n, const uint16_t *a, const uint16_t *b, const float *c, float *out);
void lds_layout(bool fp64, bool few_pairs, double edges_met, int32_t max_edges, int32_t max_cells, int32_t cols, int32_t *cols_out, int32_t *cells_out,
                uint32_t *lds_bytes);
hipError_t occupancy(bool fp64, bool global_table, uint32_t lds_bytes, int *per_cu);
hipError_t launch_count(bool fp64, bool global_table, const SegDesc *segs, const TableDesc *tabs, const uint64_t *items, const uint64_t *tiles,
                        const unsigned long long *n_items, unsigned long long *queue, unsigned long long *rechecked,
                        unsigned long long *stats, unsigned long long *counts, const unsigned long long *copies,
                        int64_t count_words, int32_t max_edges, int32_t max_cells, int32_t cols, uint32_t lds_bytes, int chunk, uint64_t flush_cap, int grid, hipStream_t st);
}
namespace t128 { PC_TILE_STEPS }
#undef PC_TILE_STEPS

// One tile size's steps.  tile = points per tile (both axes); 64-point
// sub-blocks, tile / 64 of them per tile; the matrix-core path needs 256.
struct TileOps {
    int tile;
    int subs;
    bool matrix_cores;
    decltype(&t256::launch_count) launch_count;
    decltype(&t256::launch_bounds) launch_bounds;
    decltype(&t256::launch_prune) launch_prune;
    decltype(&t256::count_occupancy) count_occupancy;
    decltype(&t256::set_max_lds) set_max_lds;
};
static const TileOps kTile256 = {256, 4, true, t256::launch_count, t256::launch_bounds, t256::launch_prune,
                                 t256::count_occupancy, t256::set_max_lds};
static const TileOps kTile128 = {128, 2, false, t128::launch_count, t128::launch_bounds, t128::launch_prune,
                                 t128::count_occupancy, t128::set_max_lds};
// the block kernel's preparation (its launch has its own arguments)
static const TileOps kTileBlocks = {kBlockTile, 0, false, nullptr, blk::launch_bounds, t256::launch_prune,
                                    nullptr, nullptr};
// resident catalogues are ordered, and bounded for 256-point tiles and the
// block kernel's
static const TileOps &kResidentTile = kTile256;

#ifndef PC_SPLIT
#define PC_SPLIT 1  // split surviving tile pairs into j sub-blocks in the prune pass
#endif

// ------------------------------------------------------------------ errors

static thread_local std::string t_err;

int fail(int code, const std::string &msg) {
    t_err = msg;
    return code;
}

int hip_fail(hipError_t e, const char *what) {
    if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation)
        return fail(PC_ERR_NOMEM, std::string(what) + ": " + hipGetErrorString(e));
    return fail(PC_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

#define PC_HIP(call, what)                                  \
    do {                                                    \
        hipError_t e_ = (call);                             \
        if (e_ != hipSuccess) return hip_fail(e_, (what));  \
    } while (0)

void clear_error() { t_err.clear(); }

// per-thread count of device allocations still to fail (testing)
static thread_local int32_t t_fail_allocs = 0;

bool injected_alloc_failure() {
    if (t_fail_allocs <= 0) return false;
    --t_fail_allocs;
    return true;
}

// ------------------------------------------------------------------ device

static std::mutex g_dev_mu;
static std::map<int, DeviceInfo> g_dev;

int device_info(DeviceInfo **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    std::lock_guard<std::mutex> lk(g_dev_mu);
    auto it = g_dev.find(dev);
    if (it == g_dev.end()) {
        hipDeviceProp_t prop;
        e = hipGetDeviceProperties(&prop, dev);
        if (e != hipSuccess) return hip_fail(e, "hipGetDeviceProperties");
        DeviceInfo d;
        d.device = dev;
        d.cus = prop.multiProcessorCount;
        d.lds_per_block = static_cast<uint32_t>(prop.sharedMemPerBlock);
        d.lds_per_cu = static_cast<uint32_t>(prop.maxSharedMemoryPerMultiProcessor);
        d.arch = prop.gcnArchName;
        d.ok = d.arch.rfind("gfx950", 0) == 0;
        if (d.ok) {
            const uint32_t want = std::max<uint32_t>(d.lds_per_block, 64u * 1024u);
            if (kTile256.set_max_lds(want) == hipSuccess && kTile128.set_max_lds(want) == hipSuccess)
                d.lds_per_block = want;
        }
        it = g_dev.emplace(dev, d).first;
    }
    if (!it->second.ok)
        return fail(PC_ERR_DEVICE, "libpc needs an AMD gfx950 (MI355X) device; current device is " +
                                       it->second.arch);
    *out = &it->second;
    return PC_OK;
}

// ------------------------------------------------------------------ tables

struct TableKey {
    int device;
    int cols;
    std::vector<uint64_t> bits;
    bool operator<(const TableKey &o) const {
        if (device != o.device) return device < o.device;
        if (cols != o.cols) return cols < o.cols;
        return bits < o.bits;
    }
};

static std::mutex g_tab_mu;
// Device tables by (device, cols, edges), least recently used dropped past
// kMaxCachedTables (a launch holds its own references, so dropping an entry
// never frees a table in use).  A server with a new edge set per request
// would otherwise keep every table.
constexpr size_t kMaxCachedTables = 256;
struct CachedTable {
    std::shared_ptr<DevTable> t;
    uint64_t last_use = 0;
};
static std::map<TableKey, CachedTable> g_tabs;
static uint64_t g_tab_tick = 0;

DevTable::~DevTable() {
    if (d_mem) (void)hipFree(d_mem);
}

void table_blob(const HostTable &h, TableBlob *out, TableParts parts) {
    // one device block: e64 | band | band_g | fband | fband_g | lut32 | lutc | lut64 | lutb
    const bool vec = parts == kAllTables || parts == kMixedTables, vec64 = parts == kAllTables || parts == kFp64Table,
               blk = parts == kAllTables || parts == kBlockTable;
    const size_t b_e = sizeof(double) * h.e64.size();
    const size_t b_b = vec ? 2 * sizeof(float) * h.e64.size() : 0;
    out->o_band = (b_e + 255) & ~size_t(255);
    out->o_band_g = (out->o_band + b_b + 255) & ~size_t(255);
    out->o_fband = (out->o_band_g + b_b + 255) & ~size_t(255);
    out->o_fband_g = (out->o_fband + b_b + 255) & ~size_t(255);
    out->o_lut32 = (out->o_fband_g + b_b + 255) & ~size_t(255);
    const size_t b_l32 = vec ? sizeof(LutEntry32) * h.lut32.entries.size() : 0;
    out->o_lutc = (out->o_lut32 + b_l32 + 255) & ~size_t(255);
    const size_t b_lc = vec ? sizeof(LutEntryC) * h.lut32.compact.size() : 0;
    out->o_lut64 = (out->o_lutc + b_lc + 255) & ~size_t(255);
    const size_t b_l64 = vec64 ? sizeof(LutEntry64) * h.lut64.size() : 0;
    out->o_lutb = (out->o_lut64 + b_l64 + 255) & ~size_t(255);
    const size_t b_lb = blk ? sizeof(LutEntryB) * h.lutb.size() : 0;
    std::vector<unsigned char> &blob = out->bytes;
    blob.assign(out->o_lutb + b_lb + 256, 0);
    memcpy(blob.data(), h.e64.data(), b_e);
    for (size_t k = 0; vec && k < h.e64.size(); ++k) {
        const float bb[4] = {h.lo[k], h.hi[k], h.lo_g[k], h.hi_g[k]};
        memcpy(blob.data() + out->o_band + 8 * k, bb, 8);
        memcpy(blob.data() + out->o_band_g + 8 * k, bb + 2, 8);
        const float fb[4] = {h.fh[k], h.fw[k], h.fh_g[k], h.fw_g[k]};
        memcpy(blob.data() + out->o_fband + 8 * k, fb, 8);
        memcpy(blob.data() + out->o_fband_g + 8 * k, fb + 2, 8);
    }
    if (b_l32) memcpy(blob.data() + out->o_lut32, h.lut32.entries.data(), b_l32);
    if (b_lc) memcpy(blob.data() + out->o_lutc, h.lut32.compact.data(), b_lc);
    if (b_l64) memcpy(blob.data() + out->o_lut64, h.lut64.data(), b_l64);
    if (b_lb) memcpy(blob.data() + out->o_lutb, h.lutb.data(), b_lb);
}

void table_place(DevTable *t, const TableBlob &b, unsigned char *base) {
    t->d_e64 = reinterpret_cast<const double *>(base);
    t->d_band = reinterpret_cast<const float *>(base + b.o_band);
    t->d_band_g = reinterpret_cast<const float *>(base + b.o_band_g);
    t->d_fband = reinterpret_cast<const float *>(base + b.o_fband);
    t->d_fband_g = reinterpret_cast<const float *>(base + b.o_fband_g);
    t->d_lut32 = base + b.o_lut32;
    t->d_lutc = t->host.lut32.compact.empty() ? nullptr : base + b.o_lutc;
    t->d_lut64 = base + b.o_lut64;
    t->d_lutb = base + b.o_lutb;
}

int get_table(const double *theta, int32_t n_edges, std::shared_ptr<DevTable> *out, int cols) {
    if (!theta) return fail(PC_ERR_INVALID, "theta_edges_deg is NULL");
    if (n_edges < 2) return fail(PC_ERR_INVALID, "n_edges must be >= 2");
    DeviceInfo *di = nullptr;
    int rc = device_info(&di);
    if (rc) return rc;
    TableKey key;
    key.device = di->device;
    key.cols = cols;
    key.bits.resize(static_cast<size_t>(n_edges));
    memcpy(key.bits.data(), theta, sizeof(double) * static_cast<size_t>(n_edges));
    {
        std::lock_guard<std::mutex> lk(g_tab_mu);
        auto it = g_tabs.find(key);
        if (it != g_tabs.end()) {
            it->second.last_use = ++g_tab_tick;
            *out = it->second.t;
            return PC_OK;
        }
    }
    auto t = std::make_shared<DevTable>();
    std::string err;
    if (!build_table(theta, n_edges, t->host, err, cols)) return fail(PC_ERR_INVALID, err);
    TableBlob blob;
    table_blob(t->host, &blob);
    void *d = nullptr;
    PC_HIP(injected_alloc_failure() ? hipErrorOutOfMemory : hipMalloc(&d, blob.bytes.size()), "hipMalloc(tables)");
    t->d_mem = d;
    PC_HIP(hipMemcpy(d, blob.bytes.data(), blob.bytes.size(), hipMemcpyHostToDevice), "hipMemcpy(tables)");
    table_place(t.get(), blob, static_cast<unsigned char *>(d));
    std::lock_guard<std::mutex> lk(g_tab_mu);
    auto it = g_tabs.find(key);
    if (it != g_tabs.end()) {
        it->second.last_use = ++g_tab_tick;
        *out = it->second.t;  // another thread won; ours is freed
        return PC_OK;
    }
    if (g_tabs.size() >= kMaxCachedTables) {
        auto lru = g_tabs.begin();
        for (auto c = g_tabs.begin(); c != g_tabs.end(); ++c)
            if (c->second.last_use < lru->second.last_use) lru = c;
        g_tabs.erase(lru);
    }
    g_tabs.emplace(key, CachedTable{t, ++g_tab_tick});
    *out = t;
    return PC_OK;
}

TableDesc table_desc(const DevTable &t, bool fp64) {
    TableDesc d;
    memset(&d, 0, sizeof(d));
    const HostTable &h = t.host;
    d.e64 = t.d_e64;
    d.n_edges = static_cast<int32_t>(h.e64.size());
    d.lutb = t.d_lutb;
    d.b_shift = h.b_shift;
    d.b_key0 = h.b_key0;
    d.b_cells = static_cast<int32_t>(h.lutb.size());
    if (fp64) {
        d.cols = h.cols64;
        d.lut = t.d_lut64;
        d.clamp_lo = h.clamp_lo64;
        d.clamp_hi = h.clamp_hi64;
        d.shift = h.shift64;
        d.key0 = h.clamp_lo64 >> h.shift64;
        d.n_cells = static_cast<int32_t>(h.lut64.size());
        d.search = h.search64 ? 1 : 0;
    } else {
        d.cols = h.cols32;
        d.lut = t.d_lut32;
        d.lutc = t.d_lutc;
        d.clamp_lo = h.lut32.clamp_lo;
        d.clamp_hi = h.lut32.clamp_hi;
        d.shift = h.lut32.shift;
        d.key0 = h.lut32.clamp_lo >> h.lut32.shift;
        d.n_cells = static_cast<int32_t>(h.lut32.entries.size());
        d.search = 0;
        d.band = t.d_band;
        d.band_g = t.d_band_g;
        d.fband = t.d_fband;
        d.fband_g = t.d_fband_g;
    }
    return d;
}

// LDS bytes a table needs: histogram rows, then the cell table (or edges;
// compact: the 8-byte cells)
static void table_lds(const DevTable &t, bool fp64, bool compact, uint32_t *hist, uint32_t *lut) {
    const HostTable &h = t.host;
    *hist = static_cast<uint32_t>(h.e64.size() + 3) * (fp64 ? h.row_bytes64 : h.row_bytes32);
    if (fp64) {
        *lut = h.search64 ? static_cast<uint32_t>(8 * h.e64.size())
                          : static_cast<uint32_t>(16 * h.lut64.size());
    } else {
        *lut = static_cast<uint32_t>((compact ? 8 : 16) * h.lut32.entries.size());
    }
}

// ------------------------------------------------------------- catalogues

static std::mutex g_cat_mu;
static std::unordered_map<uint64_t, std::shared_ptr<Resident>> g_cats;
static std::atomic<uint64_t> g_next_handle{1};

Resident::~Resident() {
    if (d_mem) (void)hipFree(d_mem);
}

int validate_catalog(const pc_catalog *c, const char *name) {
    if (!c) return fail(PC_ERR_INVALID, std::string(name) + " is NULL");
    if (c->n < 0) return fail(PC_ERR_INVALID, std::string(name) + ".n < 0");
    if (c->n > 0 && (!c->ra_deg || !c->dec_deg))
        return fail(PC_ERR_INVALID, std::string(name) + " has NULL coordinate pointers");
    if (c->n > (int64_t(1) << 40)) return fail(PC_ERR_INVALID, std::string(name) + ".n too large");
    if (!c->on_device) {
        for (int64_t i = 0; i < c->n; ++i) {
            const double r = c->ra_deg[i], d = c->dec_deg[i];
            if (!std::isfinite(r) || !std::isfinite(d) || d < -90.0 || d > 90.0)
                return fail(PC_ERR_INVALID, std::string(name) + ": RA must be finite and Dec in [-90, 90] (index " +
                                                std::to_string(i) + ")");
        }
    }
    return PC_OK;
}

static int get_resident(uint64_t h, std::shared_ptr<Resident> *out) {
    std::lock_guard<std::mutex> lk(g_cat_mu);
    auto it = g_cats.find(h);
    if (it == g_cats.end()) return fail(PC_ERR_INVALID, "unknown catalogue handle");
    *out = it->second;
    return PC_OK;
}

// Stream-ordered device allocation released when the batch ends.
struct Workspace {
    void *mem = nullptr;
    hipStream_t st = nullptr;
    ~Workspace() {
        if (mem) (void)hipFreeAsync(mem, st);
    }
};

struct Arena {
    size_t size = 0;
    size_t take(size_t bytes) {
        // a cache line; small pieces, of which a batch of small views has many, half
        const size_t align = bytes >= 1024 ? 128 : 64;
        const size_t o = (size + align - 1) & ~(align - 1);
        size = o + bytes;
        return o;
    }
};

static int64_t n_tiles(int64_t n, int tile) { return (n + tile - 1) / tile; }

// ------------------------------------------------------------------- batch

// optional per-thread timing of the counting kernel (HIP events on its stream)
static thread_local bool t_timing = false;

bool thread_timing() { return t_timing; }
void set_thread_timing(bool on) { t_timing = on; }
static thread_local hipEvent_t t_ev0 = nullptr, t_ev1 = nullptr;
// per-thread cap on the counting kernel's histogram flush interval (testing)
static thread_local uint64_t t_flush_cap = 0;
// compact cell tables: 0 when they raise the waves per CU, 1 whenever built, -1 never
static thread_local int t_compact_mode = 0;
// per-thread tile size for launches without explicit parameters (testing; 0: as chosen)
static thread_local int t_force_tile = 0;
// spatial ordering of the block kernel's launches: 0 as chosen, 1 always, -1
// only where a chord table does not fit into LDS (testing)
static thread_local int t_order = 0;
static thread_local BatchStats t_last;

int run_batch(const std::vector<BatchJob> &jobs, int mode_flags, hipStream_t st, BatchStats *stats,
              const LaunchTune *tune) {
    BatchOpts o;
    o.tune = tune;
    return run_batch_opts(jobs, mode_flags, st, stats, o);
}

int run_batch_opts(const std::vector<BatchJob> &jobs, int mode_flags, hipStream_t st, BatchStats *stats,
                   const BatchOpts &opts) {
    const LaunchTune *tune = opts.tune;
    const bool plan_only = opts.plan_bytes != nullptr;
    const bool ext = !plan_only && opts.ws != nullptr;  // caller's workspace: allocate nothing
    const bool fixed = opts.ws_bytes > 0;               // run, or planned, for a workspace of that size
    if (jobs.empty()) return fail(PC_ERR_INVALID, "no jobs");
    const int mode = mode_flags & ~(PC_NO_PRUNE | PC_MATRIX_CORES | PC_TUNED);
    const bool prune = (mode_flags & PC_NO_PRUNE) == 0;
    if (mode != PC_MIXED && mode != PC_FP64_PLAIN) return fail(PC_ERR_INVALID, "unknown mode");
    const bool fp64 = mode == PC_FP64_PLAIN;
    // launch parameters: explicit, tuned for this shape (PC_TUNED), or defaults
    LaunchTune lt;
    bool vector_tuned = false;
    if (tune) {
        lt = *tune;
    } else if (mode_flags & PC_TUNED) {
        TuneEntry te;
        if (tune_lookup(tune_key_of(jobs), &te) == PC_OK) {
            lt = te.tune;
            vector_tuned = !te.blocks;
        } else {
            lt.matrix_cores = (mode_flags & PC_MATRIX_CORES) != 0;
        }
    } else {
        lt.matrix_cores = (mode_flags & PC_MATRIX_CORES) != 0;
    }
    if (!tune && t_force_tile) {
        lt.tile = t_force_tile;
        lt.vector = true;
    }
    if (lt.chunk < 1 || lt.chunk > 64) return fail(PC_ERR_INVALID, "work chunk must be in [1, 64]");
    // the matrix-core path needs the prune pass's marks; binary32 only
    if (lt.tile != 0 && lt.tile != 128 && lt.tile != 256) return fail(PC_ERR_INVALID, "tile must be 128 or 256 points");
    const bool mc = lt.matrix_cores && prune && !fp64 && lt.tile != 128;
    // the block kernel runs the pruned launches, mixed and binary64.  The vector
    // kernels stay for 128-point tiles, for visiting every pair and for
    // PC_MATRIX_CORES.
    const bool blocks = prune && !mc && lt.tile != 128 && !lt.vector;
    // columns and chunk that were chosen for the vector kernel say nothing about
    // this one (four columns, a choice for large edge sets there, take 3.15 ms for
    // 300,000 x 400,000 points in 24 bins, its own sixteen 1.59)
    if (blocks && vector_tuned) {
        lt.cols = LaunchTune().cols;
        lt.chunk = LaunchTune().chunk;
    }
    const TileOps &T = blocks ? kTileBlocks : lt.tile == 128 ? kTile128 : kTile256;
    const int tile = T.tile;
    // host-side validation first, so bad arguments are reported as such
    for (const BatchJob &j : jobs) {
        if (j.auto_flag != 0 && j.auto_flag != 1) return fail(PC_ERR_INVALID, "auto_flag must be 0 or 1");
        std::string err;
        if (!validate_edges(j.theta, j.n_edges, err)) return fail(PC_ERR_INVALID, err);
        if (!j.counts && !plan_only) return fail(PC_ERR_INVALID, "counts is NULL");
        // inputs the caller already checked point by point (the server's
        // copies) skip the per-point scan here
        const pc_catalog *A = j.hA ? nullptr : j.A, *B = (j.auto_flag || j.hB) ? nullptr : j.B;
        if (opts.trusted_inputs) {
            if ((!j.hA && !A) || (!j.auto_flag && !j.hB && !B)) return fail(PC_ERR_INVALID, "catalogue is NULL");
        } else {
            int r = A ? validate_catalog(A, "A") : PC_OK;
            if (r) return r;
            r = B ? validate_catalog(B, "B") : PC_OK;
            if (r) return r;
        }
        if (!j.hA) {
            const int64_t nA = j.A->n;
            const int64_t r0 = j.row_begin, r1 = j.row_end < 0 ? nA : j.row_end;
            if (r0 < 0 || r1 > nA || r0 > r1)
                return fail(PC_ERR_INVALID, "row range [" + std::to_string(r0) + ", " + std::to_string(r1) +
                                                ") outside [0, " + std::to_string(nA) + "]");
        }
    }
    DeviceInfo *di = nullptr;
    int rc = PC_OK;
    if (!plan_only) {
        rc = device_info(&di);
        if (rc) return rc;
    }

    Arena ar;
    // ---- sources: catalogues as binary64 unit vectors in the caller's order
    struct Source {
        const pc_catalog *c = nullptr;
        std::shared_ptr<Resident> res;
        int64_t n = 0;
        size_t o_a64 = 0;
        size_t at_ra = 0, at_dec = 0;  // host arrays: place in the call's host data, in doubles
    };
    std::vector<Source> srcs;
    size_t host_doubles = 0;
    std::map<std::tuple<const double *, const double *, int64_t>, int> src_of_ptr;
    std::map<uint64_t, int> src_of_handle;
    auto add_source = [&](const pc_catalog *c, uint64_t h, int *out) -> int {
        if (h) {
            auto it = src_of_handle.find(h);
            if (it != src_of_handle.end()) { *out = it->second; return PC_OK; }
            Source sc;
            auto v = plan_only && opts.plan_sizes ? opts.plan_sizes->find(h) : std::map<uint64_t, int64_t>::const_iterator();
            if (plan_only && opts.plan_sizes && v != opts.plan_sizes->end()) {
                // planning against a catalogue described only by its size
                sc.res = std::make_shared<Resident>();
                sc.res->n = v->second;
            } else {
                int r = get_resident(h, &sc.res);
                if (r) return r;
            }
            sc.n = sc.res->n;
            *out = static_cast<int>(srcs.size());
            src_of_handle.emplace(h, *out);
            srcs.push_back(sc);
            return PC_OK;
        }
        auto key = std::make_tuple(c->ra_deg, c->dec_deg, c->n);
        auto it = src_of_ptr.find(key);
        if (it != src_of_ptr.end()) { *out = it->second; return PC_OK; }
        Source sc;
        sc.c = c;
        sc.n = c->n;
        sc.o_a64 = ar.take(sizeof(double4) * static_cast<size_t>(std::max<int64_t>(c->n, 1)));
        if (!c->on_device && c->n > 0) {
            sc.at_ra = host_doubles;
            sc.at_dec = sc.at_ra + static_cast<size_t>(c->n);
            host_doubles = sc.at_dec + static_cast<size_t>(c->n);
        }
        *out = static_cast<int>(srcs.size());
        src_of_ptr.emplace(key, *out);
        srcs.push_back(sc);
        return PC_OK;
    };

    // ---- views: spatially ordered copies of source index ranges
    struct View {
        int src = -1;
        int64_t b = 0, e = 0;
        bool resident_full = false;
        size_t o_a64s = 0, o_a32s = 0, o_g32s = 0, o_bounds = 0, o_groups = 0;
        // the ordering's scratch (see plan_order): keys, of their own or from the
        // region's counters on, first counter
        size_t o_keys = 0;
        int64_t hist0 = 0;
        uint32_t buckets = 0;
    };
    std::vector<View> views;
    std::map<std::tuple<int, int64_t, int64_t>, int> view_of;
    // which ordered forms the launch's kernels read: plain binary32 (vector
    // paths), tile-centred Gram form (pruned mixed launches)
    const bool need_a32 = !fp64 && !blocks, need_g32 = prune && !fp64;
    // the ordering's keys: in the Gram form's place where a workspace is tight
    // (beside the points' places, both done with when the form is written), of
    // their own otherwise, or in the ordering's region where there is no Gram form
    const bool own_keys = need_g32 && blocks && !fixed;
    auto add_view = [&](int src, int64_t b, int64_t e) -> int {
        auto key = std::make_tuple(src, b, e);
        auto it = view_of.find(key);
        if (it != view_of.end()) return it->second;
        View v;
        v.src = src;
        v.b = b;
        v.e = e;
        const int64_t n = e - b;
        // a resident catalogue's own ordered copy and bounds serve a view of
        // all of it when the launch uses the tile size they were built for
        if (srcs[src].res && b == 0 && e == srcs[src].n && (&T == &kResidentTile || blocks)) {
            v.resident_full = true;
        } else if (n > 0) {
            v.o_a64s = ar.take(sizeof(double4) * static_cast<size_t>(n));
            // binary32 copies padded: the vector kernels read a step of j-points ahead
            if (need_a32) v.o_a32s = ar.take(sizeof(float4) * static_cast<size_t>(n + kJPad));
            if (need_g32) v.o_g32s = ar.take(sizeof(float4) * static_cast<size_t>(blocks ? n : n + kJPad));
            if (own_keys) v.o_keys = ar.take(sizeof(uint32_t) * static_cast<size_t>(n));
            v.o_bounds = ar.take(sizeof(double4) * static_cast<size_t>(n_tiles(n, tile) * (1 + T.subs)));
            if (blocks) v.o_groups = ar.take(sizeof(float4) * static_cast<size_t>(n_tiles(n, tile) * kGroups));
        }
        const int id = static_cast<int>(views.size());
        view_of.emplace(key, id);
        views.push_back(v);
        return id;
    };

    std::vector<std::shared_ptr<DevTable>> tabs;
    std::map<const DevTable *, int> tab_idx;
    // planning, or the caller's workspace: the batch's own tables by edge set
    // (in the workspace, not the allocating per-device cache)
    std::map<std::pair<int, std::vector<uint64_t>>, int> local_tab;
    std::vector<TableBlob> blobs;
    struct JobPlan {
        int tab = 0;
        size_t o_counts = 0;
        int vi_tri = -1, vi_rect = -1, vj_rect = -1;
    };
    std::vector<JobPlan> plan(jobs.size());
    for (size_t q = 0; q < jobs.size(); ++q) {
        const BatchJob &j = jobs[q];
        int sa = -1, sb = -1;
        rc = add_source(j.A, j.hA, &sa);
        if (rc) return rc;
        if (!j.auto_flag) {
            rc = add_source(j.B, j.hB, &sb);
            if (rc) return rc;
        }
        const int64_t nA = srcs[sa].n;
        const int64_t r0 = j.row_begin, r1 = j.row_end < 0 ? nA : j.row_end;
        if (r0 < 0 || r1 > nA || r0 > r1)
            return fail(PC_ERR_INVALID, "row range [" + std::to_string(r0) + ", " + std::to_string(r1) +
                                            ") outside [0, " + std::to_string(nA) + "]");
        if (plan_only || ext) {
            std::vector<uint64_t> bits(static_cast<size_t>(j.n_edges));
            memcpy(bits.data(), j.theta, sizeof(double) * bits.size());
            auto key = std::make_pair(fp64 ? 0 : lt.cols, std::move(bits));
            auto it = local_tab.find(key);
            if (it == local_tab.end()) {
                auto t = std::make_shared<DevTable>();
                if (fixed) {
                    std::string err;
                    if (!build_table(j.theta, j.n_edges, t->host, err, fp64 ? 0 : lt.cols))
                        return fail(PC_ERR_INVALID, err);
                    blobs.emplace_back();
                    table_blob(t->host, &blobs.back(), blocks ? kBlockTable : fp64 ? kFp64Table : kMixedTables);
                }
                it = local_tab.emplace(std::move(key), static_cast<int>(tabs.size())).first;
                tabs.push_back(t);
            }
            plan[q].tab = it->second;
        } else {
            std::shared_ptr<DevTable> t;
            rc = get_table(j.theta, j.n_edges, &t, fp64 ? 0 : lt.cols);
            if (rc) return rc;
            auto it = tab_idx.find(t.get());
            if (it == tab_idx.end()) {
                it = tab_idx.emplace(t.get(), static_cast<int>(tabs.size())).first;
                tabs.push_back(t);
            }
            plan[q].tab = it->second;
        }
        if (j.auto_flag) {
            // pairs i<j with i in [r0, r1): triangle on [r0, r1) + rectangle [r0, r1) x [r1, n)
            plan[q].vi_tri = add_view(sa, r0, r1);
            if (r1 < nA && r1 > r0) {
                plan[q].vi_rect = plan[q].vi_tri;
                plan[q].vj_rect = add_view(sa, r1, nA);
            }
        } else {
            plan[q].vi_rect = add_view(sa, r0, r1);
            plan[q].vj_rect = add_view(sb, 0, srcs[sb].n);
        }
    }
    // results block, read back with one copy: meta[kMetaWords] | each job's counts | conversion flags
    // (meta[0]: survivors, meta[7]: re-check tally, from meta[kPruneStatBase]:
    // the prune pass's statistics in kPruneStripes copies, from
    // meta[kQueueBase]: the counting kernel's work queue, 8 counters
    // kQueueStride words apart)
    constexpr size_t kMetaWords = kQueueBase + 8 * kQueueStride;
    size_t res_words = kMetaWords;
    for (size_t q = 0; q < jobs.size(); ++q) res_words += static_cast<size_t>(jobs[q].n_edges + 1);
    const size_t err_words = (std::max<size_t>(srcs.size(), 1) + 1) / 2;
    const size_t o_host = ar.take(sizeof(double) * host_doubles);
    const size_t o_res = ar.take(sizeof(unsigned long long) * (res_words + err_words));
    {
        size_t w = kMetaWords;
        for (size_t q = 0; q < jobs.size(); ++q) {
            plan[q].o_counts = o_res + sizeof(unsigned long long) * w;
            w += static_cast<size_t>(jobs[q].n_edges + 1);
        }
    }
    const size_t o_err = o_res + sizeof(unsigned long long) * res_words;
    const size_t o_meta = o_res;
    // the prune pass's copies of every job's counters, the sources' extents
    // and the ordering counters follow the results: zeroed by one launch
    const size_t count_words = res_words - kMetaWords;
    const size_t o_pcopies = ar.take(sizeof(unsigned long long) * kPruneStripes * count_words);
    const size_t o_ext = ar.take(sizeof(uint32_t) * kExtWords * srcs.size());

    // ---- segments
    std::vector<SegDesc> segs;
    uint64_t items = 0;
    uint64_t limit_items = 0;
    bool items_overflow = false;  // more tile pairs than an item number holds
    int64_t prune_rows = 0;
    auto view_n = [&](int v) { return views[v].e - views[v].b; };
    for (size_t q = 0; q < jobs.size(); ++q) {
        auto add = [&](bool tri, int vi, int vj) {
            const int64_t ni = view_n(vi), nj = view_n(vj);
            if (ni <= 0 || nj <= 0 || (tri && ni < 2)) return;
            SegDesc sd;
            memset(&sd, 0, sizeof(sd));
            sd.tri = tri ? 1 : 0;
            sd.i0 = 0;
            sd.ni = ni;
            sd.j0 = 0;
            sd.nj = nj;
            sd.tiles_i = n_tiles(ni, tile);
            sd.tiles_j = n_tiles(nj, tile);
            // in 128 bits: up to 2^32 tiles per side, whose products pass 2^64
            const unsigned __int128 n_items =
                tri ? static_cast<unsigned __int128>(sd.tiles_i) * static_cast<unsigned __int128>(sd.tiles_i + 1) / 2
                    : static_cast<unsigned __int128>(sd.tiles_i) * static_cast<unsigned __int128>(sd.tiles_j);
            // the limit counts pairs of 256-point tiles, whatever the tile size
            const int64_t li = blocks ? n_tiles(ni, 256) : sd.tiles_i, lj = blocks ? n_tiles(nj, 256) : sd.tiles_j;
            const unsigned __int128 l_items =
                tri ? static_cast<unsigned __int128>(li) * static_cast<unsigned __int128>(li + 1) / 2
                    : static_cast<unsigned __int128>(li) * static_cast<unsigned __int128>(lj);
            if (l_items > kItemMask || limit_items + static_cast<uint64_t>(l_items) > kItemMask) items_overflow = true;
            limit_items = std::min<uint64_t>(limit_items + static_cast<uint64_t>(std::min<unsigned __int128>(l_items, kItemMask)), kItemMask + 1);
            sd.n_items = static_cast<uint64_t>(std::min<unsigned __int128>(n_items, kItemMask));
            sd.item0 = items;
            items = std::min<uint64_t>(items + sd.n_items, kItemMask + 1);
            // rows of the prune pass (see k_prune)
            sd.prow0 = prune_rows;
            prune_rows += tri ? (sd.tiles_i + 1) / 2 : sd.tiles_i;
            sd.tab = plan[q].tab;
            sd.job = static_cast<int32_t>(q);
            // view indices parked in the pointer slots until the workspace exists
            sd.i0 = vi;
            sd.j0 = vj;
            segs.push_back(sd);
        };
        if (plan[q].vi_tri >= 0) add(true, plan[q].vi_tri, plan[q].vi_tri);
        if (plan[q].vi_rect >= 0 && plan[q].vj_rect >= 0) add(false, plan[q].vi_rect, plan[q].vj_rect);
    }
    if (items_overflow || items > kItemMask)
        return fail(PC_ERR_INVALID, "too many tile pairs in one call (more than " + std::to_string(kItemMask) +
                                        "); split the catalogues into row ranges");
    // split survivors: the prune pass looks at the j-tile's sub-blocks too
    // (mixed mode); their descriptions sit beside the survivors
    // (block kernel: the survivors' tiles do)
    const bool split = prune && (blocks || (PC_SPLIT && !fp64));
    // The survivors.  A mixed plan, and a fixed workspace, count 16 bytes per pair of
    // 256-point tiles, what the vector kernels need, so that admission and the
    // fixed area's limit are the same whichever kernel runs; the block kernel
    // writes 16 per pair of 512-point tiles, and an ordinary call allocates only
    // those (4M x 8M points: 2.0 GB instead of 7.8).
    const bool as_vector = !blocks || (!fp64 && (plan_only || fixed));
    const uint64_t slots = std::max<uint64_t>(!prune ? 1 : as_vector ? std::max(items, limit_items) : items, 1);
    const size_t surv_bytes = sizeof(uint64_t) * slots, surv_region = surv_bytes * (split ? 2 : 1);
    // The ordering's counters, and the keys where no ordered copy has room for
    // them until it is written, are done with when the prune pass writes the
    // survivors: one region holds the one, then the other.  Views are ordered
    // together in rounds of as many as fit `cap` bytes (a view by itself may
    // take more, but where `limited`, a workspace that would not hold it,
    // it gets fewer counters and a coarser order).
    struct OrderRound {
        size_t first = 0, count = 0;  // of the views to order
        int64_t words = 0, blocks = 0;
    };
    std::vector<OrderRound> rounds;
    constexpr size_t kOrderBytes = size_t(64) << 20;
    auto plan_order = [&](size_t cap, bool limited) -> size_t {
        rounds.clear();
        size_t most = 0, used = 0, place = 0;
        for (View &v : views) {
            if (v.resident_full || v.e <= v.b) continue;
            const size_t keys = need_g32 ? 0 : sizeof(uint32_t) * static_cast<size_t>((v.e - v.b + 3) & ~int64_t(3));
            v.buckets = order_buckets(v.e - v.b, prune ? 4 : 2);
            if (limited && keys + sizeof(uint32_t) * v.buckets > cap)
                v.buckets = std::max<uint32_t>(kMinBuckets, cap > keys ? static_cast<uint32_t>((cap - keys) / sizeof(uint32_t)) & ~3u : 0u);
            const size_t need = keys + sizeof(uint32_t) * v.buckets;
            if (rounds.empty() || used + need > cap) {
                rounds.push_back(OrderRound());
                rounds.back().first = place;
                used = 0;
            }
            OrderRound &r = rounds.back();
            v.hist0 = r.words;
            if (!need_g32) v.o_keys = used - sizeof(uint32_t) * static_cast<size_t>(r.words);  // behind the round's counters
            r.words += v.buckets;
            ++r.count;
            ++place;
            used += need;
            most = std::max(most, used);
        }
        return most;
    };
    // descriptors, sent with one copy: sources | views | segments | tables
    // (written in whole 16-byte words, see launch_zero_put)
    size_t to_convert = 0, to_order = 0;
    for (const Source &sc : srcs) to_convert += !sc.res && sc.n > 0 ? 1 : 0;
    for (const View &v : views) to_order += !v.resident_full && v.e > v.b ? 1 : 0;
    const size_t b_srcs = sizeof(SrcDesc) * to_convert, b_views = sizeof(ViewDesc) * to_order,
                 b_segs = sizeof(SegDesc) * segs.size(), b_tabs = sizeof(TableDesc) * tabs.size();
    const size_t before_region = ar.size;
    size_t o_region = 0, o_sums = 0, o_desc = 0, order_bytes = 0;
    int64_t hist_words = 0;  // the largest round's
    std::vector<size_t> o_blob(blobs.size());
    auto place_rest = [&](size_t cap, bool limited) {
        ar.size = before_region;
        order_bytes = plan_order(cap, limited);
        hist_words = 0;
        for (const OrderRound &r : rounds) hist_words = std::max(hist_words, r.words);
        o_region = ar.take(std::max(order_bytes, surv_region));
        o_sums = ar.take(sizeof(uint32_t) * std::max<size_t>(scan_sums_words(hist_words), 4));
        o_desc = ar.take((b_srcs + b_views + b_segs + b_tabs + 15) & ~size_t(15));
        for (size_t k = 0; k < blobs.size(); ++k) o_blob[k] = ar.take(blobs[k].bytes.size());
    };
    place_rest(std::max(kOrderBytes, surv_region), false);
    if (fixed && ar.size > opts.ws_bytes) {
        // a workspace that does not hold this: more rounds, and if they do not
        // help no chord tables (they are the larger ones of dense edge sets)
        auto fit = [&] {
            const size_t others = ar.size - std::max(order_bytes, surv_region);
            place_rest(std::max(surv_region, opts.ws_bytes > others ? (opts.ws_bytes - others) & ~size_t(127) : 0), true);
            return ar.size <= opts.ws_bytes;
        };
        if (!fit() && blocks) {
            for (size_t k = 0; k < blobs.size(); ++k) {
                tabs[k]->host.lutb.clear();
                table_blob(tabs[k]->host, &blobs[k], kBlockTable);
            }
            place_rest(std::max(kOrderBytes, surv_region), false);
            if (ar.size > opts.ws_bytes) fit();
        }
    }
    const size_t o_surv = o_region, o_sub = o_region + surv_bytes;
    if (plan_only) {
        *opts.plan_bytes = ar.size;
        return PC_OK;
    }

    // ---- the workspace: allocated here, or the caller's
    Workspace ws;
    ws.st = st;
    unsigned char *W = nullptr;
    if (ext) {
        if (ar.size > opts.ws_bytes)
            return fail(PC_ERR_INVALID, "the call needs " + std::to_string(ar.size) +
                                            " bytes of device workspace; the fixed workspace holds " +
                                            std::to_string(opts.ws_bytes));
        W = static_cast<unsigned char *>(opts.ws);
        for (size_t k = 0; k < blobs.size(); ++k) {
            PC_HIP(hipMemcpyAsync(W + o_blob[k], blobs[k].bytes.data(), blobs[k].bytes.size(), hipMemcpyHostToDevice,
                                  st),
                   "H2D tables");
            table_place(tabs[k].get(), blobs[k], W + o_blob[k]);
        }
    } else {
        PC_HIP(injected_alloc_failure() ? hipErrorOutOfMemory : hipMallocAsync(&ws.mem, ar.size, st),
               "hipMallocAsync(workspace)");
        W = static_cast<unsigned char *>(ws.mem);
    }

    // ---- the sources to convert (validity flags read back at the end) and
    // the views to order
    std::vector<const double4 *> src_a64(srcs.size(), nullptr);
    std::vector<const uint32_t *> src_ext(srcs.size(), nullptr);
    // Host catalogues of a small call go up in one copy: a copy from the caller's
    // memory costs 13 us at 80 KB, one of 320 KB 19, gathering that 5.  Whole calls
    // of two catalogues, separate / gathered: 128 / 115 us at 32 KB, 245 / 223 at 320,
    // 267 / 254 at 640, but 383 / 400 at 1280, where the extra pass shows.
    constexpr size_t kGatherDoubles = 96 * 1024;
    double *const d_host = reinterpret_cast<double *>(W + o_host);
    const std::unique_ptr<double[]> gathered(
        host_doubles > 0 && host_doubles <= kGatherDoubles ? new (std::nothrow) double[host_doubles] : nullptr);
    std::vector<SrcDesc> sds;
    int64_t conv_blocks = 0;
    for (size_t k = 0; k < srcs.size(); ++k) {
        if (srcs[k].res) {
            src_a64[k] = srcs[k].res->a64;
            src_ext[k] = srcs[k].res->ext;
            continue;
        }
        const pc_catalog *c = srcs[k].c;
        src_a64[k] = reinterpret_cast<const double4 *>(W + srcs[k].o_a64);
        src_ext[k] = reinterpret_cast<const uint32_t *>(W + o_ext) + k * kExtWords;
        if (c->n <= 0) continue;
        SrcDesc d;
        d.ra = c->ra_deg;
        d.dec = c->dec_deg;
        if (!c->on_device) {
            double *const dra = d_host + srcs[k].at_ra, *const ddec = d_host + srcs[k].at_dec;
            if (gathered) {
                memcpy(gathered.get() + srcs[k].at_ra, c->ra_deg, sizeof(double) * static_cast<size_t>(c->n));
                memcpy(gathered.get() + srcs[k].at_dec, c->dec_deg, sizeof(double) * static_cast<size_t>(c->n));
            } else {
                PC_HIP(hipMemcpyAsync(dra, c->ra_deg, sizeof(double) * c->n, hipMemcpyHostToDevice, st), "H2D ra");
                PC_HIP(hipMemcpyAsync(ddec, c->dec_deg, sizeof(double) * c->n, hipMemcpyHostToDevice, st), "H2D dec");
            }
            d.ra = dra;
            d.dec = ddec;
        }
        d.a64 = reinterpret_cast<double4 *>(W + srcs[k].o_a64);
        d.err = reinterpret_cast<int *>(W + o_err) + k;
        d.ext = reinterpret_cast<uint32_t *>(W + o_ext) + k * kExtWords;
        d.n = c->n;
        d.blk0 = conv_blocks;
        conv_blocks += convert_blocks(c->n);
        sds.push_back(d);
    }
    if (gathered)
        PC_HIP(hipMemcpyAsync(d_host, gathered.get(), sizeof(double) * host_doubles, hipMemcpyHostToDevice, st),
               "H2D catalogues");
    struct ViewPtrs {
        const double4 *a64s = nullptr;
        const float4 *a32s = nullptr;
        const float4 *g32s = nullptr;
        const double4 *bounds = nullptr;
        const double4 *sub_bounds = nullptr;  // T.subs per tile, after the tiles' own
        const float4 *groups = nullptr;       // kGroups per tile (block kernel)
    };
    std::vector<ViewPtrs> vp(views.size());
    // LDS of the block kernel, and whether every edge set's chord table is in it
    int32_t max_edges = 0, max_cells = 0, bcols = 0;
    uint32_t blocks_lds = 0;
    bool global_table = false;
    bool ordered = !blocks;
    if (blocks) {
        bool all = true;
        for (auto &t : tabs) {
            max_edges = std::max(max_edges, static_cast<int32_t>(t->host.e64.size()));
            max_cells = std::max(max_cells, static_cast<int32_t>(t->host.lutb.size()));
            all = all && !t->host.lutb.empty();
        }
        const bool any = max_cells > 0;
        // The pairs, and over them the mean of the edges that a block meets: its
        // size, of 32 points, over the last bin's width, if the catalogues fill a
        // field about as wide as the last edge (their extent is not on the host).
        double pairs = 0.0, edges_met = 0.0;
        for (const SegDesc &sd : segs) {
            const double ni = static_cast<double>(sd.ni), nj = static_cast<double>(sd.nj), p = ni * nj * (sd.tri ? 0.5 : 1.0);
            const std::vector<double> &e = tabs[static_cast<size_t>(sd.tab)]->host.e64;
            const double last = std::sqrt(e[e.size() - 1]);
            pairs += p;
            edges_met += p * std::sqrt(kGroup / std::sqrt(ni * nj)) * last / (last - std::sqrt(e[e.size() - 2]));
        }
        edges_met /= std::max(pairs, 1.0);
        const bool few_pairs = t_order ? t_order < 0 : pairs <= kUnorderedPairs;
        blk::lds_layout(fp64, few_pairs, edges_met, max_edges, max_cells, lt.cols ? std::min(lt.cols, 16) : 16, &bcols, &max_cells, &blocks_lds);
        // Few pairs are counted in the caller's order: unordered groups prune
        // nothing and put every block through the chord table (hence only with
        // one), but the four ordering launches cost more than that.  Whole
        // calls, ordered / caller's order: 100 / 79 us for the pairs of 1003
        // points, 111 / 95 of 4096, 123 / 110 of 6000; 122 / 108 for 4096 x 4096,
        // 156 / 144 for 8192 x 8192 in bins of all scales, but 131 / 136 where the
        // bins end at 2 degrees and the order lets most pairs go.  In binary64 110 / 79
        // for 1003 points, 115 / 90 for 4096, 127 / 101 for 4096 x 4096, 158 / 140 for 8192
        // x 8192, 129 / 137 with bins to 2 degrees: the same line.
        global_table = any && max_cells == 0;
        ordered = !all || max_cells == 0 || !few_pairs;
    }
    std::vector<ViewDesc> vds;
    int64_t all_tiles = 0;
    uint32_t points = 0;  // of the round's views so far
    size_t round = 0;
    for (size_t v = 0; v < views.size(); ++v) {
        const View &vw = views[v];
        if (vw.resident_full) {
            const Resident &r = *srcs[vw.src].res;
            vp[v].a64s = r.a64s;
            vp[v].a32s = r.a32s;
            vp[v].g32s = blocks ? r.g512 : r.g32s;
            vp[v].bounds = blocks ? r.b512 : r.bounds;
            vp[v].sub_bounds = r.bounds + n_tiles(r.n, kResidentTile.tile);
            vp[v].groups = r.groups;
            continue;
        }
        const int64_t n = vw.e - vw.b;
        if (n <= 0) continue;
        ViewDesc d;
        d.src = src_a64[vw.src] + vw.b;
        d.ext = src_ext[vw.src];
        if (vds.size() == rounds[round].first + rounds[round].count) {
            ++round;
            points = 0;
        }
        d.hist = reinterpret_cast<uint32_t *>(W + o_region) + vw.hist0;
        // (read only where the order is the caller's)
        d.a64s = ordered ? reinterpret_cast<double4 *>(W + vw.o_a64s) : const_cast<double4 *>(d.src);
        d.a32s = need_a32 ? reinterpret_cast<float4 *>(W + vw.o_a32s) : nullptr;
        d.g32s = need_g32 ? reinterpret_cast<float4 *>(W + vw.o_g32s) : nullptr;
        // (done with when the bounds step writes the Gram form)
        d.slots = reinterpret_cast<uint32_t *>(d.g32s);
        d.keys = own_keys   ? reinterpret_cast<uint32_t *>(W + vw.o_keys)
                 : need_g32 ? d.slots + n
                            : reinterpret_cast<uint32_t *>(W + o_region + sizeof(uint32_t) * static_cast<size_t>(rounds[round].words) + vw.o_keys);
        d.bounds = reinterpret_cast<double4 *>(W + vw.o_bounds);
        d.groups = blocks ? reinterpret_cast<float4 *>(W + vw.o_groups) : nullptr;
        d.n = n;
        d.hist0 = vw.hist0;
        d.blk0 = rounds[round].blocks;
        d.tile0 = all_tiles;
        d.tiles = n_tiles(n, tile);
        d.buckets = vw.buckets;
        d.points0 = points;
        rounds[round].blocks += order_blocks(n);
        all_tiles += d.tiles;
        points += static_cast<uint32_t>(n);
        vds.push_back(d);
        vp[v].a64s = d.a64s;
        vp[v].a32s = d.a32s;
        vp[v].g32s = d.g32s;
        vp[v].bounds = d.bounds;
        vp[v].sub_bounds = d.bounds + d.tiles;
        vp[v].groups = d.groups;
    }

    // ---- descriptors
    for (SegDesc &sd : segs) {
        const int vi = static_cast<int>(sd.i0), vj = static_cast<int>(sd.j0);
        sd.i0 = 0;
        sd.j0 = 0;
        sd.i32 = vp[vi].a32s;
        sd.i64 = vp[vi].a64s;
        sd.ib = vp[vi].bounds;
        sd.j32 = vp[vj].a32s;
        sd.j64 = vp[vj].a64s;
        sd.jb = vp[vj].bounds;
        sd.ig = vp[vi].g32s;
        sd.jg = vp[vj].g32s;
        sd.ib32 = vp[vi].groups;
        sd.jb32 = vp[vj].groups;
        sd.jb_sub = vp[vj].sub_bounds;
        sd.counts = reinterpret_cast<unsigned long long *>(W + plan[static_cast<size_t>(sd.job)].o_counts);
        sd.pcounts = reinterpret_cast<unsigned long long *>(W + o_pcopies + plan[static_cast<size_t>(sd.job)].o_counts -
                                                            o_res - sizeof(unsigned long long) * kMetaWords);
        sd.pstride = static_cast<int64_t>(count_words);
    }
    std::vector<TableDesc> tds;
    bool compact_ok = !fp64 && !mc && !blocks;
    for (auto &t : tabs) {
        tds.push_back(table_desc(*t, fp64));
        compact_ok = compact_ok && t->d_lutc != nullptr;
    }
    // LDS: histogram | cell table (or edges) | matrix-core A operands
    auto layout = [&](bool compact, uint32_t *lut_off, uint32_t *stage_off, uint32_t *lds) {
        uint32_t hist_max = 0, lut_max = 0;
        for (auto &t : tabs) {
            uint32_t h, l;
            table_lds(*t, fp64, compact, &h, &l);
            hist_max = std::max(hist_max, h);
            lut_max = std::max(lut_max, l);
        }
        *lut_off = (hist_max + 15u) & ~15u;
        *stage_off = *lut_off + ((std::max<uint32_t>(lut_max, 16u) + 15u) & ~15u);
        *lds = *stage_off + (mc ? 16u * kWave * 4u : 0u);
    };
    uint32_t lut_off = 0, stage_off = 0, lds_bytes = 0;
    layout(false, &lut_off, &stage_off, &lds_bytes);
    // the compact cell table costs one instruction per cell-table chord; it
    // is taken when its smaller LDS footprint lets more waves share a CU
    bool compact = false;
    if (compact_ok && t_compact_mode >= 0 && items > 0) {
        uint32_t lo_c = 0, so_c = 0, lds_c = 0;
        layout(true, &lo_c, &so_c, &lds_c);
        bool take = t_compact_mode > 0;
        if (!take && lds_bytes <= di->lds_per_block) {
            int full = 0, small = 0;
            PC_HIP(T.count_occupancy(false, false, false, lds_bytes, &full), "occupancy");
            PC_HIP(T.count_occupancy(false, false, true, lds_c, &small), "occupancy");
            take = small > full;
        } else if (!take) {
            take = true;  // only the compact table fits
        }
        if (take) {
            compact = true;
            lut_off = lo_c;
            stage_off = so_c;
            lds_bytes = lds_c;
        }
    }
    if (!blocks && lds_bytes > di->lds_per_block)
        return fail(PC_ERR_INVALID, "edge set needs " + std::to_string(lds_bytes) +
                                        " bytes of LDS per wave; the device allows " +
                                        std::to_string(di->lds_per_block));
    // ---- send the descriptors; zero, convert, order, bound
    std::vector<unsigned char> desc(b_srcs + b_views + b_segs + b_tabs);
    auto put = [&](size_t at, const void *p, size_t bytes) {
        if (bytes) memcpy(desc.data() + at, p, bytes);
    };
    put(0, sds.data(), sizeof(SrcDesc) * sds.size());
    put(b_srcs, vds.data(), sizeof(ViewDesc) * vds.size());
    put(b_srcs + b_views, segs.data(), b_segs);
    put(b_srcs + b_views + b_segs, tds.data(), b_tabs);
    // (the counters of the ordering's first round too, where there is one)
    const int64_t first_words = ordered && !rounds.empty() ? rounds[0].words : 0;
    const size_t zero_bytes = (o_region - o_res + sizeof(uint32_t) * static_cast<size_t>(first_words) + 15) & ~size_t(15);
    if (desc.size() <= kPutBytes) {
        PC_HIP(launch_zero_put(W + o_res, zero_bytes, W + o_desc, desc.data(), desc.size(), st), "zero results");
    } else {
        PC_HIP(hipMemcpyAsync(W + o_desc, desc.data(), desc.size(), hipMemcpyHostToDevice, st), "H2D descriptors");
        PC_HIP(launch_zero(W + o_res, zero_bytes, st), "zero results");
    }
    const SrcDesc *d_srcs = reinterpret_cast<const SrcDesc *>(W + o_desc);
    const ViewDesc *d_views = reinterpret_cast<const ViewDesc *>(W + o_desc + b_srcs);
    PC_HIP(launch_convert(d_srcs, static_cast<int>(sds.size()), conv_blocks, st), "convert");
    for (const OrderRound &r : rounds) {
        if (!ordered) break;
        uint32_t *const hist = reinterpret_cast<uint32_t *>(W + o_region);
        if (r.first > 0) PC_HIP(launch_zero(hist, sizeof(uint32_t) * static_cast<size_t>(r.words), st), "zero counters");
        PC_HIP(launch_order(d_views + r.first, static_cast<int>(r.count), r.blocks, hist, r.words,
                            reinterpret_cast<uint32_t *>(W + o_sums), st),
               "order");
    }
    PC_HIP(T.launch_bounds(d_views, static_cast<int>(vds.size()), all_tiles, st), "bounds");
    unsigned long long *meta = reinterpret_cast<unsigned long long *>(W + o_meta);

    // ---- whole-tile-pair binning, then the counting kernel over the rest
    const SegDesc *d_segs = reinterpret_cast<const SegDesc *>(W + o_desc + b_srcs + b_views);
    const TableDesc *d_tabs = reinterpret_cast<const TableDesc *>(W + o_desc + b_srcs + b_views + b_segs);
    uint64_t *surv = reinterpret_cast<uint64_t *>(W + o_surv);
    uint64_t *sub_words = reinterpret_cast<uint64_t *>(W + o_sub);
    int grid = 0;
    if (items > 0) {
        if (prune) {
            PC_HIP(T.launch_prune(d_segs, static_cast<int32_t>(segs.size()), d_tabs, prune_rows, surv,
                                split ? sub_words : nullptr, meta, mc ? 1 : 0, split ? 1 : 0, blocks, st),
                   "prune");
            if (!blocks)  // (the block kernel adds them itself)
                PC_HIP(launch_add_copies(reinterpret_cast<unsigned long long *>(W + o_res) + kMetaWords,
                                         reinterpret_cast<const unsigned long long *>(W + o_pcopies),
                                         static_cast<int64_t>(count_words), kPruneStripes, st),
                       "add prune counts");
        }
        int per_cu = 0;
        if (blocks) {
            lds_bytes = blocks_lds;
            PC_HIP(blk::occupancy(fp64, global_table, lds_bytes, &per_cu), "occupancy");
        } else {
            PC_HIP(T.count_occupancy(fp64, mc, compact, lds_bytes, &per_cu), "occupancy");
        }
        per_cu = std::max(per_cu, 1);
        int64_t g = static_cast<int64_t>(di->cus) * per_cu;
        // (the block kernel cuts few survivors into up to sixteen units)
        g = std::min<int64_t>(g, static_cast<int64_t>(std::min<uint64_t>(items, 1u << 20)) * (blocks ? 16 : 1));
        if (g >= 8) g -= g % 8;
        grid = static_cast<int>(std::max<int64_t>(g, 1));
        const bool timed = t_timing && !ext;  // events are not created in the caller's-workspace mode
        if (timed) {
            if (!t_ev0) {
                PC_HIP(hipEventCreate(&t_ev0), "hipEventCreate");
                PC_HIP(hipEventCreate(&t_ev1), "hipEventCreate");
            }
            PC_HIP(hipEventRecord(t_ev0, st), "hipEventRecord");
        }
        if (blocks)
            PC_HIP(blk::launch_count(fp64, global_table, d_segs, d_tabs, surv, sub_words, meta, meta + kQueueBase, meta + 7,
                                     meta + kPruneStatBase, reinterpret_cast<unsigned long long *>(W + o_res) + kMetaWords,
                                     reinterpret_cast<const unsigned long long *>(W + o_pcopies),
                                     static_cast<int64_t>(count_words), max_edges, max_cells, bcols, lds_bytes, lt.chunk, t_flush_cap,
                                     grid, st),
                   "block kernel");
        else
            PC_HIP(T.launch_count(fp64, mc, compact, d_segs, static_cast<int32_t>(segs.size()), d_tabs, prune ? surv : nullptr,
                            prune ? meta : nullptr, split ? sub_words : nullptr, items, lut_off, stage_off, meta + kQueueBase,
                            meta + 7, lt.chunk, lds_bytes, grid, t_flush_cap, st),
               "count kernel");
        if (timed) PC_HIP(hipEventRecord(t_ev1, st), "hipEventRecord");
    }

    // ---- results: counts, validity flags and pruning figures under one sync
    std::vector<unsigned long long> hres(res_words + err_words, 0ull);
    PC_HIP(hipMemcpyAsync(hres.data(), W + o_res, sizeof(unsigned long long) * hres.size(), hipMemcpyDeviceToHost, st),
           "D2H results");
    PC_HIP(hipStreamSynchronize(st), "hipStreamSynchronize");
    const int *flags = reinterpret_cast<const int *>(hres.data() + res_words);
    for (size_t k = 0; k < srcs.size(); ++k)
        if (flags[k]) return fail(PC_ERR_INVALID, "catalogue has non-finite RA/Dec or |Dec| > 90");
    for (size_t q = 0; q < jobs.size(); ++q)
        memcpy(jobs[q].counts, hres.data() + (plan[q].o_counts - o_res) / sizeof(unsigned long long),
               sizeof(uint64_t) * static_cast<size_t>(jobs[q].n_edges + 1));
    const unsigned long long *hmeta = hres.data();
    uint64_t ps[kPruneStats] = {};  // the prune pass's statistics, stripes added up
    for (int c = 0; c < kPruneStripes; ++c)
        for (int k = 1; k < kPruneStats; ++k) ps[k] += hmeta[kPruneStatBase + c * kPruneStripeWords + k];

    uint64_t total_pairs = 0;
    for (const SegDesc &sd : segs) {
        const uint64_t ni = static_cast<uint64_t>(sd.ni), nj = static_cast<uint64_t>(sd.nj);
        total_pairs += sd.tri ? ni * (ni - 1) / 2 : ni * nj;
    }
    t_last = BatchStats();
    t_last.items = items;
    t_last.grid = grid;
    t_last.lds_bytes = lds_bytes;
    t_last.segments = static_cast<int>(segs.size());
    t_last.kernel_ms = -1.0;
    t_last.survivors = prune ? hmeta[0] : items;
    t_last.pairs_total = total_pairs;
    t_last.pairs_computed = prune ? ps[1] : total_pairs;
    t_last.mfma_items = prune ? ps[2] : 0;
    t_last.few_items = prune ? ps[3] : 0;
    t_last.gram_items = prune ? ps[4] : 0;
    t_last.split_items = prune ? ps[5] : 0;
    t_last.rechecked = hmeta[7];
    for (int m = 0; m < 4; ++m) t_last.pairs_by_m[m] = prune ? ps[6 + m] : 0;
    t_last.pairs_gram = prune ? ps[10] : 0;
    if (!prune || fp64) {
        // every computed pair through the cell table (the binary64 kernel
        // ignores the few-edge tags)
        t_last.pairs_by_m[0] = t_last.pairs_computed;
        for (int m = 1; m < 4; ++m) t_last.pairs_by_m[m] = 0;
        t_last.pairs_gram = 0;
    }
    t_last.pairs_mfma = prune ? ps[11] : 0;
    t_last.workspace_bytes = ar.size;
    t_last.ordered = ordered && !vds.empty();
    if (t_timing && !ext && items > 0) {
        float ms = 0.0f;
        PC_HIP(hipEventElapsedTime(&ms, t_ev0, t_ev1), "hipEventElapsedTime");
        t_last.kernel_ms = ms;
    }
    if (stats) *stats = t_last;
    return PC_OK;
}

int upload_catalog(const pc_catalog *c, hipStream_t st, uint64_t *handle) {
    int rc = validate_catalog(c, "catalogue");
    if (rc) return rc;
    if (!handle) return fail(PC_ERR_INVALID, "handle is NULL");
    DeviceInfo *di = nullptr;
    rc = device_info(&di);
    if (rc) return rc;
    auto r = std::make_shared<Resident>();
    r->n = c->n;
    r->device = di->device;
    const size_t n = static_cast<size_t>(std::max<int64_t>(c->n, 1));
    Arena ar;
    const size_t o64 = ar.take(sizeof(double4) * n);
    const size_t o64s = ar.take(sizeof(double4) * n);
    const size_t o32s = ar.take(sizeof(float4) * (n + kJPad));  // padded as in run_batch
    const size_t og32s = ar.take(sizeof(float4) * (n + kJPad));
    const int64_t t512 = n_tiles(static_cast<int64_t>(n), kBlockTile);
    const size_t og512 = ar.take(std::max(sizeof(float4) * n, sizeof(uint32_t) * order_buckets(static_cast<int64_t>(n), 4)));
    const size_t ob512 = ar.take(sizeof(double4) * static_cast<size_t>(t512));
    const size_t og = ar.take(sizeof(float4) * static_cast<size_t>(t512 * kGroups));
    const size_t ob = ar.take(sizeof(double4) * static_cast<size_t>(n_tiles(static_cast<int64_t>(n), kResidentTile.tile) *
                                                                     (1 + kResidentTile.subs)));
    struct alignas(16) Desc {
        SrcDesc s;
        ViewDesc v, v512;          // v512: the bounds of the block kernel's tiles
        uint32_t ext[kExtWords];   // zeroed with the rest: the extent,
        int err[4];                // the validity flag
    };
    static_assert(sizeof(Desc) % 16 == 0 && sizeof(Desc) <= kPutBytes, "goes to the device as arguments");
    const size_t odesc = ar.take(sizeof(Desc));
    const size_t oext = odesc + offsetof(Desc, ext), oerr = odesc + offsetof(Desc, err);
    // scratch of the conversion and the ordering lies in copies that are
    // written after it is done with: counters and keys in the two Gram forms,
    // the caller's host arrays in the ordered binary32 copy
    const uint32_t buckets = order_buckets(static_cast<int64_t>(n), 4);
    const size_t ohist = og512, okeys = og32s, ora = o32s, odec = o32s + sizeof(double) * n;
    const size_t osums = ar.take(sizeof(uint32_t) * std::max<size_t>(scan_sums_words(buckets), 4));
    PC_HIP(injected_alloc_failure() ? hipErrorOutOfMemory : hipMalloc(&r->d_mem, ar.size), "hipMalloc(catalogue)");
    unsigned char *W = static_cast<unsigned char *>(r->d_mem);
    r->a64 = reinterpret_cast<double4 *>(W + o64);
    r->a64s = reinterpret_cast<double4 *>(W + o64s);
    r->a32s = reinterpret_cast<float4 *>(W + o32s);
    r->g32s = reinterpret_cast<float4 *>(W + og32s);
    r->bounds = reinterpret_cast<double4 *>(W + ob);
    r->g512 = reinterpret_cast<float4 *>(W + og512);
    r->b512 = reinterpret_cast<double4 *>(W + ob512);
    r->groups = reinterpret_cast<float4 *>(W + og);
    r->ext = reinterpret_cast<uint32_t *>(W + oext);
    Desc d = {};
    if (c->n <= 0) {
        PC_HIP(launch_zero(W + odesc, sizeof(d), st), "zero");
    } else {
        d.s.ra = c->ra_deg;
        d.s.dec = c->dec_deg;
        if (!c->on_device) {
            PC_HIP(hipMemcpyAsync(W + ora, c->ra_deg, sizeof(double) * c->n, hipMemcpyHostToDevice, st), "H2D ra");
            PC_HIP(hipMemcpyAsync(W + odec, c->dec_deg, sizeof(double) * c->n, hipMemcpyHostToDevice, st), "H2D dec");
            d.s.ra = reinterpret_cast<const double *>(W + ora);
            d.s.dec = reinterpret_cast<const double *>(W + odec);
        }
        d.s.a64 = r->a64;
        d.s.err = reinterpret_cast<int *>(W + oerr);
        d.s.ext = r->ext;
        d.s.n = c->n;
        d.v.src = r->a64;
        d.v.ext = r->ext;
        d.v.keys = reinterpret_cast<uint32_t *>(W + okeys);
        d.v.hist = reinterpret_cast<uint32_t *>(W + ohist);
        d.v.slots = d.v.keys + c->n;
        d.v.a64s = r->a64s;
        d.v.a32s = r->a32s;
        d.v.g32s = r->g32s;
        d.v.bounds = r->bounds;
        d.v.n = c->n;
        d.v.tiles = n_tiles(c->n, kResidentTile.tile);
        d.v.buckets = buckets;
        d.v512 = d.v;
        d.v512.g32s = r->g512;
        d.v512.bounds = r->b512;
        d.v512.groups = r->groups;
        d.v512.tiles = t512;
        const SrcDesc *ds = reinterpret_cast<const SrcDesc *>(W + odesc);
        const ViewDesc *dv = reinterpret_cast<const ViewDesc *>(W + odesc + offsetof(Desc, v));
        PC_HIP(launch_zero_put(W + ohist, sizeof(uint32_t) * buckets, W + odesc, &d, sizeof(d), st), "zero");
        PC_HIP(launch_convert(ds, 1, convert_blocks(c->n), st), "convert");
        PC_HIP(launch_order(dv, 1, order_blocks(c->n), reinterpret_cast<uint32_t *>(W + ohist), buckets,
                            reinterpret_cast<uint32_t *>(W + osums), st),
               "order");
        PC_HIP(kResidentTile.launch_bounds(dv, 1, d.v.tiles, st), "bounds");
        PC_HIP(kTileBlocks.launch_bounds(dv + 1, 1, t512, st), "bounds");
    }
    int flag = 0;
    PC_HIP(hipMemcpyAsync(&flag, W + oerr, sizeof(int), hipMemcpyDeviceToHost, st), "D2H flag");
    PC_HIP(hipStreamSynchronize(st), "hipStreamSynchronize");
    if (flag) return fail(PC_ERR_INVALID, "catalogue has non-finite RA/Dec or |Dec| > 90");
    const uint64_t h = g_next_handle.fetch_add(1);
    {
        std::lock_guard<std::mutex> lk(g_cat_mu);
        g_cats.emplace(h, r);
    }
    *handle = h;
    return PC_OK;
}

int release_catalog(uint64_t h) {
    std::shared_ptr<Resident> r;
    {
        std::lock_guard<std::mutex> lk(g_cat_mu);
        auto it = g_cats.find(h);
        if (it == g_cats.end()) return fail(PC_ERR_INVALID, "unknown catalogue handle");
        r = it->second;
        g_cats.erase(it);
    }
    // the allocation goes when the last user (a running batch) drops it
    return PC_OK;
}

int resident_catalog(uint64_t h, std::shared_ptr<Resident> *out) { return get_resident(h, out); }

int jobs_from_abi(const pc_job *jobs, int32_t n_jobs, std::vector<BatchJob> *out) {
    if (!jobs || n_jobs < 1) return fail(PC_ERR_INVALID, "jobs is NULL or n_jobs < 1");
    std::vector<BatchJob> &v = *out;
    v.assign(static_cast<size_t>(n_jobs), BatchJob());
    for (int32_t q = 0; q < n_jobs; ++q) {
        v[q].A = jobs[q].A;
        v[q].B = jobs[q].B;
        v[q].theta = jobs[q].theta_edges_deg;
        v[q].n_edges = jobs[q].n_edges;
        v[q].auto_flag = jobs[q].auto_flag;
        v[q].row_begin = jobs[q].row_begin;
        v[q].row_end = jobs[q].row_end;
        v[q].counts = jobs[q].counts;
    }
    return PC_OK;
}

}  // namespace pc

// ===================================================================== C ABI

using namespace pc;

extern "C" {

const char *pc_last_error(void) { return t_err.c_str(); }

const char *pc_version(void) { return "pc 0.1 gfx950"; }

int pc_count_ex(const pc_catalog *A, const pc_catalog *B, const double *theta_edges_deg, int32_t n_edges,
                int32_t auto_flag, int32_t mode, int64_t row_begin, int64_t row_end, uint64_t *counts,
                void *stream) {
    clear_error();
    BatchJob j;
    j.A = A;
    j.B = B;
    j.theta = theta_edges_deg;
    j.n_edges = n_edges;
    j.auto_flag = auto_flag;
    j.row_begin = row_begin;
    j.row_end = row_end;
    j.counts = counts;
    std::vector<BatchJob> v(1, j);
    return run_batch(v, mode, static_cast<hipStream_t>(stream), nullptr);
}

int pc_count(const pc_catalog *A, const pc_catalog *B, const double *theta_edges_deg, int32_t n_edges,
             int32_t auto_flag, uint64_t *counts, void *stream) {
    return pc_count_ex(A, B, theta_edges_deg, n_edges, auto_flag, PC_MIXED, 0, -1, counts, stream);
}

int pc_count_batch(const pc_job *jobs, int32_t n_jobs, int32_t mode, void *stream) {
    clear_error();
    std::vector<BatchJob> v;
    const int rc = jobs_from_abi(jobs, n_jobs, &v);
    if (rc) return rc;
    return run_batch(v, mode, static_cast<hipStream_t>(stream), nullptr);
}

int pc_wtheta(const uint64_t *DD, const uint64_t *DR, const uint64_t *RR, int32_t n_bins, int64_t nD, int64_t nR,
              double *w) {
    clear_error();
    if (!DD || !DR || !RR || !w) return fail(PC_ERR_INVALID, "NULL argument");
    if (n_bins < 1) return fail(PC_ERR_INVALID, "n_bins must be >= 1");
    if (nD < 2 || nR < 2) return fail(PC_ERR_INVALID, "nD and nR must be >= 2");
    landy_szalay(DD, DR, RR, n_bins, nD, nR, w);
    return PC_OK;
}

int pc_estimator(int32_t kind, const uint64_t *DD, const uint64_t *DR, const uint64_t *RR, int32_t n_bins,
                 int64_t nD, int64_t nR, double *w) {
    clear_error();
    if (kind < PC_EST_LANDY_SZALAY || kind > PC_EST_HAMILTON) return fail(PC_ERR_INVALID, "unknown estimator");
    const bool need_dr = kind != PC_EST_NATURAL, need_rr = kind != PC_EST_DAVIS_PEEBLES;
    if (!DD || !w || (need_dr && !DR) || (need_rr && !RR)) return fail(PC_ERR_INVALID, "NULL argument");
    if (n_bins < 1) return fail(PC_ERR_INVALID, "n_bins must be >= 1");
    if (nD < 2 || nR < 2) return fail(PC_ERR_INVALID, "nD and nR must be >= 2");
    estimator(kind, DD, DR, RR, n_bins, nD, nR, w);
    return PC_OK;
}

int pc_catalog_upload(const pc_catalog *c, void *stream, uint64_t *handle) {
    clear_error();
    return upload_catalog(c, static_cast<hipStream_t>(stream), handle);
}

int pc_catalog_release(uint64_t handle) {
    clear_error();
    return release_catalog(handle);
}

int pc_count_h(uint64_t hA, uint64_t hB, const double *theta_edges_deg, int32_t n_edges, int32_t auto_flag,
               int32_t mode, int64_t row_begin, int64_t row_end, uint64_t *counts, void *stream) {
    clear_error();
    if (!hA || (!auto_flag && !hB)) return fail(PC_ERR_INVALID, "catalogue handle is 0");
    BatchJob j;
    j.hA = hA;
    j.hB = auto_flag ? 0 : hB;
    j.theta = theta_edges_deg;
    j.n_edges = n_edges;
    j.auto_flag = auto_flag;
    j.row_begin = row_begin;
    j.row_end = row_end;
    j.counts = counts;
    std::vector<BatchJob> v(1, j);
    return run_batch(v, mode, static_cast<hipStream_t>(stream), nullptr);
}

int pc_unit_vectors(const pc_catalog *c, double *xyz64, float *xyz32, void *stream) {
    clear_error();
    uint64_t h = 0;
    hipStream_t st = static_cast<hipStream_t>(stream);
    int rc = upload_catalog(c, st, &h);
    if (rc) return rc;
    std::shared_ptr<Resident> r;
    get_resident(h, &r);
    release_catalog(h);
    const size_t n = static_cast<size_t>(c->n);
    if (n > 0) {
        std::vector<double4> v64(n);
        PC_HIP(hipMemcpyAsync(v64.data(), r->a64, sizeof(double4) * n, hipMemcpyDeviceToHost, st), "D2H a64");
        PC_HIP(hipStreamSynchronize(st), "hipStreamSynchronize");
        for (size_t i = 0; i < n; ++i) {
            if (xyz64) {
                xyz64[3 * i + 0] = v64[i].x;
                xyz64[3 * i + 1] = v64[i].y;
                xyz64[3 * i + 2] = v64[i].z;
            }
            if (xyz32) {
                xyz32[3 * i + 0] = static_cast<float>(v64[i].x);
                xyz32[3 * i + 1] = static_cast<float>(v64[i].y);
                xyz32[3 * i + 2] = static_cast<float>(v64[i].z);
            }
        }
    }
    return PC_OK;
}

int pc_chord2_edges(const double *theta_edges_deg, int32_t n_edges, double *e) {
    clear_error();
    if (!theta_edges_deg || !e) return fail(PC_ERR_INVALID, "NULL argument");
    HostTable t;
    std::string err;
    if (!build_table(theta_edges_deg, n_edges, t, err)) return fail(PC_ERR_INVALID, err);
    memcpy(e, t.e64.data(), sizeof(double) * static_cast<size_t>(n_edges));
    return PC_OK;
}

int pc_guard_band(const double *theta_edges_deg, int32_t n_edges, float *lo, float *hi) {
    clear_error();
    if (!theta_edges_deg || !lo || !hi) return fail(PC_ERR_INVALID, "NULL argument");
    HostTable t;
    std::string err;
    if (!build_table(theta_edges_deg, n_edges, t, err)) return fail(PC_ERR_INVALID, err);
    memcpy(lo, t.lo.data(), sizeof(float) * static_cast<size_t>(n_edges));
    memcpy(hi, t.hi.data(), sizeof(float) * static_cast<size_t>(n_edges));
    return PC_OK;
}

}  // extern "C"

extern "C" int pc_debug_lut32(const double *theta_edges_deg, int32_t n_edges, int64_t *info, uint32_t *entries,
                              int64_t max_cells) {
    clear_error();
    if (!theta_edges_deg || !info) return fail(PC_ERR_INVALID, "NULL argument");
    HostTable t;
    std::string err;
    if (!build_table(theta_edges_deg, n_edges, t, err)) return fail(PC_ERR_INVALID, err);
    const Lut32 &L = t.lut32;
    info[0] = static_cast<int64_t>(L.entries.size());
    info[1] = L.shift;
    info[2] = L.clamp_lo;
    info[3] = L.clamp_hi;
    info[4] = t.row_bytes32;
    info[5] = t.cols32;
    info[6] = L.multi;
    info[7] = 0;
    if (entries && static_cast<int64_t>(L.entries.size()) <= max_cells)
        memcpy(entries, L.entries.data(), sizeof(LutEntry32) * L.entries.size());
    return PC_OK;
}

extern "C" int pc_debug_last_workspace(uint64_t *bytes) {
    clear_error();
    if (!bytes) return fail(PC_ERR_INVALID, "bytes is NULL");
    *bytes = t_last.workspace_bytes;
    return PC_OK;
}

extern "C" int pc_debug_static_plan(const pc_job *jobs, int32_t n_jobs, int32_t mode, uint64_t bytes,
                                    uint64_t *need) {
    clear_error();
    if (!need || bytes == 0) return fail(PC_ERR_INVALID, "need is NULL or bytes is 0");
    std::vector<BatchJob> v;
    const int rc = jobs_from_abi(jobs, n_jobs, &v);
    if (rc) return rc;
    BatchOpts o;
    o.plan_bytes = need;
    o.ws_bytes = bytes;
    return run_batch_opts(v, mode, nullptr, nullptr, o);
}

extern "C" int pc_debug_products(int32_t n, const uint16_t *a, const uint16_t *b, const float *c, float *out) {
    clear_error();
    if (n < 0 || n > (1 << 20)) return fail(PC_ERR_INVALID, "n must be in [0, 2^20]");
    if (n == 0) return PC_OK;
    if (!a || !b || !c || !out) return fail(PC_ERR_INVALID, "NULL argument");
    DeviceInfo *di = nullptr;
    const int rc = device_info(&di);
    if (rc) return rc;
    const size_t k = static_cast<size_t>(n);
    struct Free {
        void *p = nullptr;
        ~Free() {
            if (p) (void)hipFree(p);
        }
    } m;
    PC_HIP(hipMalloc(&m.p, 136 * k), "hipMalloc(products)");
    float *const dc = static_cast<float *>(m.p), *const dout = dc + k;
    uint16_t *const da = reinterpret_cast<uint16_t *>(dout + k), *const db = da + 32 * k;
    PC_HIP(hipMemcpy(da, a, 64 * k, hipMemcpyHostToDevice), "H2D a");
    PC_HIP(hipMemcpy(db, b, 64 * k, hipMemcpyHostToDevice), "H2D b");
    PC_HIP(hipMemcpy(dc, c, 4 * k, hipMemcpyHostToDevice), "H2D c");
    PC_HIP(blk::launch_products(n, da, db, dc, dout), "products");
    PC_HIP(hipMemcpy(out, dout, 4 * k, hipMemcpyDeviceToHost), "D2H products");
    return PC_OK;
}

extern "C" int pc_debug_chord_table(const double *theta_edges_deg, int32_t n_edges, int64_t *info, uint32_t *cells,
                                    int64_t max_cells) {
    clear_error();
    if (!theta_edges_deg || !info) return fail(PC_ERR_INVALID, "NULL argument");
    HostTable t;
    std::string err;
    if (!build_table(theta_edges_deg, n_edges, t, err)) return fail(PC_ERR_INVALID, err);
    info[0] = static_cast<int64_t>(t.lutb.size());
    info[1] = t.b_shift;
    info[2] = t.b_key0;
    if (cells && static_cast<int64_t>(t.lutb.size()) <= max_cells && !t.lutb.empty())
        memcpy(cells, t.lutb.data(), sizeof(LutEntryB) * t.lutb.size());
    return PC_OK;
}

extern "C" int pc_debug_fused_band(const double *theta_edges_deg, int32_t n_edges, int32_t gram, float *h,
                                   float *w) {
    clear_error();
    if (!theta_edges_deg || !h || !w) return fail(PC_ERR_INVALID, "NULL argument");
    HostTable t;
    std::string err;
    if (!build_table(theta_edges_deg, n_edges, t, err)) return fail(PC_ERR_INVALID, err);
    memcpy(h, (gram ? t.fh_g : t.fh).data(), sizeof(float) * static_cast<size_t>(n_edges));
    memcpy(w, (gram ? t.fw_g : t.fw).data(), sizeof(float) * static_cast<size_t>(n_edges));
    return PC_OK;
}

extern "C" int pc_debug_guard_band_gram(const double *theta_edges_deg, int32_t n_edges, float *lo, float *hi) {
    clear_error();
    if (!theta_edges_deg || !lo || !hi) return fail(PC_ERR_INVALID, "NULL argument");
    HostTable t;
    std::string err;
    if (!build_table(theta_edges_deg, n_edges, t, err)) return fail(PC_ERR_INVALID, err);
    memcpy(lo, t.lo_g.data(), sizeof(float) * static_cast<size_t>(n_edges));
    memcpy(hi, t.hi_g.data(), sizeof(float) * static_cast<size_t>(n_edges));
    return PC_OK;
}

extern "C" int pc_debug_fail_allocations(int32_t n) {
    clear_error();
    if (n < 0) return fail(PC_ERR_INVALID, "n must be >= 0");
    t_fail_allocs = n;
    return PC_OK;
}

extern "C" int pc_debug_set_tile(int32_t tile) {
    clear_error();
    if (tile != 0 && tile != 128 && tile != 256) return fail(PC_ERR_INVALID, "tile must be 0, 128 or 256");
    t_force_tile = tile;
    return PC_OK;
}

extern "C" int pc_debug_set_order(int32_t mode) {
    clear_error();
    if (mode < -1 || mode > 1) return fail(PC_ERR_INVALID, "mode must be -1, 0 or 1");
    t_order = mode;
    return PC_OK;
}

extern "C" int pc_debug_last_ordered(int32_t *ordered) {
    clear_error();
    if (!ordered) return fail(PC_ERR_INVALID, "ordered is NULL");
    *ordered = t_last.ordered ? 1 : 0;
    return PC_OK;
}

extern "C" int pc_debug_set_flush_every(uint64_t items) {
    clear_error();
    t_flush_cap = items;
    return PC_OK;
}

extern "C" int pc_debug_set_compact_table(int32_t mode) {
    clear_error();
    if (mode < -1 || mode > 1) return fail(PC_ERR_INVALID, "mode must be -1, 0 or 1");
    t_compact_mode = mode;
    return PC_OK;
}

extern "C" int pc_debug_set_timing(int32_t on) {
    clear_error();
    t_timing = on != 0;
    return PC_OK;
}

extern "C" int pc_debug_last_pruning(uint64_t *survivors, uint64_t *pairs_computed, uint64_t *pairs_total,
                                     uint64_t *mfma_items, uint64_t *few_items, uint64_t *gram_items,
                                     uint64_t *split_items) {
    clear_error();
    if (split_items) *split_items = t_last.split_items;
    if (gram_items) *gram_items = t_last.gram_items;
    if (few_items) *few_items = t_last.few_items;
    if (mfma_items) *mfma_items = t_last.mfma_items;
    if (survivors) *survivors = t_last.survivors;
    if (pairs_computed) *pairs_computed = t_last.pairs_computed;
    if (pairs_total) *pairs_total = t_last.pairs_total;
    return PC_OK;
}

extern "C" int pc_debug_last_paths(uint64_t *pairs_by_edges, uint64_t *gram_pairs, uint64_t *mfma_pairs) {
    clear_error();
    if (pairs_by_edges)
        for (int m = 0; m < 4; ++m) pairs_by_edges[m] = t_last.pairs_by_m[m];
    if (gram_pairs) *gram_pairs = t_last.pairs_gram;
    if (mfma_pairs) *mfma_pairs = t_last.pairs_mfma;
    return PC_OK;
}

extern "C" int pc_debug_last_rechecks(uint64_t *pairs_rechecked) {
    clear_error();
    if (!pairs_rechecked) return fail(PC_ERR_INVALID, "pairs_rechecked is NULL");
    *pairs_rechecked = t_last.rechecked;
    return PC_OK;
}

extern "C" int pc_debug_last_launch(double *kernel_ms, uint64_t *items, int32_t *grid, uint32_t *lds_bytes) {
    clear_error();
    if (kernel_ms) *kernel_ms = t_last.kernel_ms;
    if (items) *items = t_last.items;
    if (grid) *grid = t_last.grid;
    if (lds_bytes) *lds_bytes = t_last.lds_bytes;
    return PC_OK;
}
