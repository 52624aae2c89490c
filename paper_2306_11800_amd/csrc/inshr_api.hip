// Host side of the C ABI (include/inshr.h): argument checks, work partition, scratch memory and
// kernel sequencing.  No arithmetic of the method runs here.
#include "../../include/inshr.h"
#include "inshr_launch.h"
#include "inshr_sketch.h"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <string>
#include <unordered_map>
#include <vector>

using namespace inshr;

namespace {

struct DevBuf { // grow-only device allocation
    void *p = nullptr;
    size_t cap = 0;
};

struct HostBuf { // grow-only pinned host allocation
    void *p = nullptr;
    size_t cap = 0;
    bool lent = false; // a part of the context's own pinned block
};

} // namespace

struct inshr_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    uint64_t scratch_limit = 0;
    int n_cu = 256;
    int wg_per_cu = 0; // workgroups that a sweep deals a CU, 0: by sweep_workgroups (INSHR_WG_PER_CU)
    bool lds_ordered = false; // same-address LDS atomics return in lane order (checked at creation)
    // tensors of at least this many elements get a sampled first sweep (INSHR_SAMPLE_MIN_N; 0 = never)
    uint64_t sample_min_n = 16ull << 20;
    bool sample_force_miss = false; // INSHR_SAMPLE_FORCE_MISS=1 (tests): always take the exact sweeps again
    // keys a wave may gather per tile of its 1024 elements, on average over its tiles (of 1024): the
    // gather pools are sized by it; a search that finds them too small doubles it and runs again
    // (INSHR_POOL_WCAP sets the start)
    uint32_t pool_wcap = 136;
    std::string last_err;

    char *pinned = nullptr;     // host memory allocated with the context (an allocation takes 80 us and more):
                                // the flags and what the host buffers begin with
    u32 *flags = nullptr;       // flag words of the delta kernels (DF_*), then those of calls that wait for theirs
    bool delta_pending = false; // an asynchronous delta call has not had its flags read yet
    bool static_pending = false; // the same for inshr_delta_static (its flag words are in its own scratch)
    DevBuf search_mem; // everything a search leaves behind for inshr_quantize
    DevBuf aux_mem;    // quantize descriptors, delta scratch
    DevBuf totals_mem; // symbol populations of a delta or reconstruct call, when aux_mem has a limit
    DevBuf sketch_mem; // sketch tables, histograms, bucket lists and the centres they give
    DevBuf sens_mem;   // scores, compacted values and block counts of inshr_quantize_sens
    double sketch_alpha = 0.0;                 // the bucket tables last built, and for which alpha
    int sketch_i_lo = 0;
    std::vector<u32> sketch_cell, sketch_tops;
    std::vector<double> sketch_rep;
    HostBuf h_up;      // staging for descriptor uploads
    HostBuf h_down;    // results of a call, stored there by the kernels or downloaded
    HostBuf h_res;     // what a search and the calls that work from its state say of every tensor (SearchResult)

    // state of the last search
    bool have_search = false;
    Batch batch{};
    GridDesc grid{};
    std::vector<inshr_config> grid_cfgs;
    std::vector<inshr_tensor> tensors;
    std::vector<u32> pos;       // device position of tensors[t]
    size_t scores_off = 0;
    // (what the state holds of boundaries and centres, and what it takes to work out more of them)
    std::vector<u32> resolved;  // per device position: VIEW_NONE, VIEW_ALL or the one configuration
    std::vector<TDesc> td;
    std::vector<u32> groups;    // of the search, empty: none
    double eps = 0.0;
    int mode = 0;
    bool any_pooled = false;
    uint32_t wcap = 0;          // pool_wcap of the pools' layout
    uint64_t pool_len = 0;      // u32 entries of the second pool
    size_t view_off = 0, gw_off = 0, tgo_off = 0, gun_off = 0, view_end = 0;
};

// ------------------------------------------------------------------------------------------
// optional per-kernel timing (HIP events on the launch stream)
// ------------------------------------------------------------------------------------------
namespace {
struct ProfState {
    bool on = false;
    std::vector<hipEvent_t> pool;       // event pairs, reused
    std::vector<const char *> pending;  // name of each recorded pair
    std::vector<std::string> names;
    std::vector<double> total_ms;
    std::vector<uint64_t> launches;
} g_prof;
} // namespace

namespace inshr {
void prof_begin(const char *name, hipStream_t s)
{
    if (!g_prof.on) return;
    const size_t k = g_prof.pending.size();
    while (g_prof.pool.size() < 2 * (k + 1)) {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) return;
        g_prof.pool.push_back(e);
    }
    g_prof.pending.push_back(name);
    (void)hipEventRecord(g_prof.pool[2 * k], s);
}
void prof_end(hipStream_t s)
{
    if (!g_prof.on || g_prof.pending.empty()) return;
    const size_t k = g_prof.pending.size() - 1;
    (void)hipEventRecord(g_prof.pool[2 * k + 1], s);
}
} // namespace inshr

namespace {

void prof_collect()
{
    for (size_t k = 0; k < g_prof.pending.size(); k++) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, g_prof.pool[2 * k], g_prof.pool[2 * k + 1]) != hipSuccess) continue;
        size_t i = 0;
        for (; i < g_prof.names.size(); i++)
            if (g_prof.names[i] == g_prof.pending[k]) break;
        if (i == g_prof.names.size()) {
            g_prof.names.push_back(g_prof.pending[k]);
            g_prof.total_ms.push_back(0.0);
            g_prof.launches.push_back(0);
        }
        g_prof.total_ms[i] += ms;
        g_prof.launches[i]++;
    }
    g_prof.pending.clear();
}

#define HIPCHK(ctx, call)                                                                         \
    do {                                                                                          \
        hipError_t e__ = (call);                                                                  \
        if (e__ != hipSuccess) {                                                                  \
            (ctx)->last_err = std::string(#call) + ": " + hipGetErrorString(e__);                 \
            return INSHR_E_DEVICE;                                                                \
        }                                                                                         \
    } while (0)

int ensure_dev(inshr_ctx *c, DevBuf &b, size_t bytes)
{
    if (bytes <= b.cap) return INSHR_OK;
    if (c->scratch_limit && bytes > c->scratch_limit) return INSHR_E_CAPACITY;
    if (b.p) HIPCHK(c, hipFree(b.p));
    b.p = nullptr;
    b.cap = 0;
    hipError_t e = hipMalloc(&b.p, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        c->last_err = std::string("hipMalloc of scratch: ") + hipGetErrorString(e);
        b.p = nullptr;
        return INSHR_E_CAPACITY;
    }
    b.cap = bytes;
    return INSHR_OK;
}

// After the stream has been synchronised: the flags that the kernels of the last inshr_delta raised.
int take_delta_flags(inshr_ctx *c)
{
    if (!c->delta_pending && !c->static_pending) return INSHR_OK;
    u32 f = 0, g[FLAG_WORDS] = {};
    if (c->delta_pending) f = raised_flags(c->flags);
    if (c->static_pending) HIPCHK(c, hipMemcpy(g, delta_static_flags(c->device), sizeof(g), hipMemcpyDeviceToHost));
    c->delta_pending = c->static_pending = false;
    f |= raised_flags(g);
    if (f & DF_ORDER) {
        c->last_err = "delta: ranks from returning LDS atomics disagree with ballot ranks (set INSHR_NO_LDS_ORDER=1)";
        return INSHR_E_INTERNAL;
    }
    if (f & DF_PERM) return INSHR_E_ARG;
    return INSHR_OK;
}

int ensure_host(inshr_ctx *c, HostBuf &b, size_t bytes)
{
    if (bytes <= b.cap) return INSHR_OK;
    if (b.p && !b.lent) HIPCHK(c, hipHostFree(b.p));
    b.p = nullptr;
    b.cap = 0;
    b.lent = false;
    bytes = (bytes + 255) & ~(size_t)255; // (copies are made in whole pieces)
    HIPCHK(c, hipHostMalloc(&b.p, bytes, hipHostMallocDefault));
    b.cap = bytes;
    return INSHR_OK;
}

// The flag words of a call that waits for them, clear.  Nothing in flight raises any.
u32 *call_flags(inshr_ctx *c)
{
    u32 *f = c->flags + FLAG_WORDS;
    memset(f, 0, FLAG_WORDS * sizeof(u32));
    return f;
}

struct Carver { // lays sub-buffers out in one allocation, 256-byte aligned
    size_t off = 0;
    size_t take(size_t bytes)
    {
        size_t o = off;
        off = (off + bytes + 255) & ~(size_t)255;
        return o;
    }
};

struct QuantScratch { // of inshr_quantize; the first up_bytes are uploaded
    size_t qd, wg, un, up_bytes, bytes;
    QuantScratch(uint32_t nT, uint32_t nB, int n_wg)
    {
        Carver cv;
        qd = cv.take(sizeof(QDesc) * nT);
        wg = cv.take(sizeof(u32) * (n_wg + 1));
        un = cv.take(sizeof(Unit) * ((size_t)n_wg + nB));
        up_bytes = cv.off;
        bytes = cv.off;
    }
};

uint32_t bins_of(const inshr_config &c) { return c.bins ? c.bins : (1u << c.bits); }
bool same_config(const inshr_config &a, const inshr_config &b)
{
    return bins_of(a) == bins_of(b) && a.prune_ppm == b.prune_ppm && a.outlier_ppm == b.outlier_ppm;
}

int check_config(const inshr_config &c)
{
    if (c.bins) {
        if (!bins_supported(c.bins)) return INSHR_E_CONFIG;
    } else if (c.bits < 1 || c.bits > 8) {
        return INSHR_E_CONFIG;
    }
    if ((uint64_t)c.prune_ppm + (uint64_t)c.outlier_ppm >= 1000000ull) return INSHR_E_CONFIG;
    return INSHR_OK;
}

int build_grid(const inshr_config *grid, uint32_t n_cfg, double eps, GridDesc &g)
{
    if (n_cfg == 0 || n_cfg > (uint32_t)MAX_CFG) return INSHR_E_CONFIG;
    memset(&g, 0, sizeof(g));
    g.n_cfg = n_cfg;
    g.eps = eps;
    g.n_all = NB8;
    g.K_top = 1u;
    bool used[NBT] = {};
    for (uint32_t i = 0; i < n_cfg; i++) {
        int rc = check_config(grid[i]);
        if (rc) return rc;
        uint32_t ip = 0, io = 0;
        for (ip = 0; ip < g.n_p; ip++)
            if (g.p_ppm[ip] == grid[i].prune_ppm) break;
        if (ip == g.n_p) {
            if (g.n_p == (uint32_t)MAX_FRAC) return INSHR_E_CONFIG;
            g.p_ppm[g.n_p++] = grid[i].prune_ppm;
        }
        for (io = 0; io < g.n_o; io++)
            if (g.o_ppm[io] == grid[i].outlier_ppm) break;
        if (io == g.n_o) {
            if (g.n_o == (uint32_t)MAX_FRAC) return INSHR_E_CONFIG;
            g.o_ppm[g.n_o++] = grid[i].outlier_ppm;
        }
        uint32_t q = 0;
        for (q = 0; q < g.n_pairs; q++)
            if (g.pair_p[q] == ip && g.pair_o[q] == io) break;
        if (q == g.n_pairs) {
            if (g.n_pairs == (uint32_t)MAX_PAIRS) return INSHR_E_CONFIG;
            g.pair_p[q] = ip;
            g.pair_o[q] = io;
            g.n_pairs++;
        }
        g.cfg_pair[i] = q;
        const uint32_t K = bins_of(grid[i]);
        g.cfg_K[i] = K;
        g.cfg_bits[i] = symbol_bits(K) - 1u;
        g.cfg_l16[i] = (uint32_t)std::floor(std::log2((double)K) * 65536.0 + 0.5);
        if (K & (K - 1u))
            g.n_all = NBT; // 3, 6 or 12 bins: the twelfths are boundaries too
        else
            g.K_top = std::max(g.K_top, K);
        for (uint32_t j = 1; j < K; j++) used[bnd_index(K, j)] = true;
    }
    for (uint32_t i = 0; i < (uint32_t)NBT; i++)
        if (used[i]) g.bnd[g.n_bnd++] = (u16)i;
    return INSHR_OK;
}

// The tiles of the tensors ts (device positions, ascending) dealt out evenly to at most n_wg workgroups, in
// order, and the waves' shares of a gather pool: every wave of a unit owns room for wcap keys per tile of the
// unit plus one full tile (the sweeps stop gathering when the share cannot take a whole tile any more), and
// never more than the wave's elements.
struct Partition {
    std::vector<Unit> units;
    std::vector<u32> wg0;   // [workgroups + 1]
    std::vector<u32> t_off; // [tensors of the search by sweeps + 1] units of every tensor
    u64 pool = 0;
};
void deal_tiles(const std::vector<TDesc> &td, uint32_t nB, const std::vector<u32> &ts, int n_wg, uint32_t wcap,
                Partition &p)
{
    auto tiles_of = [&](u32 t) { return (td[t].n + TILE - 1) / TILE; };
    if (ts.empty()) {
        p.wg0.assign(1, 0u);
        p.t_off.assign(nB + 1, 0u);
        return;
    }
    u64 total = 0;
    for (u32 t : ts) total += tiles_of(t);
    n_wg = (int)std::min<u64>(total, (u64)n_wg);
    p.units.clear();
    p.wg0.assign(1, 0u);
    p.t_off.assign(nB + 1, 0u);
    p.pool = 0;
    const u64 per_wave = TILE / (BLOCK / 64);
    size_t k = 0;
    u64 done = 0; // tiles of the tensors before ts[k]
    for (int w = 0; w < n_wg; w++) {
        const u64 lo = total * (u64)w / (u64)n_wg, hi = total * (u64)(w + 1) / (u64)n_wg;
        for (u64 at = lo; at < hi;) {
            while (at >= done + tiles_of(ts[k])) done += tiles_of(ts[k++]);
            const u64 end = std::min(hi, done + tiles_of(ts[k]));
            Unit u;
            u.tile0 = (u32)(td[ts[k]].tile0 + (at - done));
            u.tile1 = (u32)(td[ts[k]].tile0 + (end - done));
            u.off16 = (u32)(p.pool / (BLOCK / 64));
            u.capw = (u32)std::min((end - at) * per_wave, (end - at) * (u64)wcap + per_wave);
            u.tensor = ts[k];
            p.t_off[u.tensor + 1]++;
            p.units.push_back(u);
            p.pool += (u64)u.capw * (BLOCK / 64);
            at = end;
        }
        p.wg0.push_back((u32)p.units.size());
    }
    for (uint32_t t = 0; t < nB; t++) p.t_off[t + 1] += p.t_off[t];
}

// Workgroups of a sweep over so many tiles.  One is resident on a CU (its tables fill the LDS).  A second one in turn
// evens out what tiles cost and makes more, shorter units for the kernels that take a workgroup per unit, but starts and
// empties its tables once more, which tensors of a few hundred tiles take as long for as for their tiles.  One / two, ms of
// kernels: 12 M values scored 0.47 / 0.55, 54 M step 0.80 / 0.94, 330 M step 2.44 / 2.56, 355 M scored 2.66 / 2.82,
// 615 M step 3.26 / 3.25, 6.7 G step 33.7 / 33.2: two from 96 tiles per CU (400 M values) on.
int sweep_workgroups(const inshr_ctx *c, u64 tiles)
{
    const u64 per = c->wg_per_cu ? (u64)c->wg_per_cu : tiles >= 96ull * (u64)c->n_cu ? 2ull : 1ull;
    return (int)std::min<u64>(tiles, (u64)c->n_cu * per);
}

// Gather units for the tensors ts (device positions, ascending), in p and, with st, on the device.  The copy is staged
// at offset at of h_up: nothing in flight reads that part of it, and where it is too small to
// hold it, nothing in flight reads any of it.
int upload_units(inshr_ctx *c, const std::vector<u32> &view, const std::vector<u32> &ts, Partition &p, size_t at, Stage &st)
{
    Batch &bt = c->batch;
    const uint32_t nB = (uint32_t)bt.nB;
    for (int n_wg = bt.n_wg;; n_wg = (n_wg + 1) / 2) { // (fewer workgroups need less of the pool)
        deal_tiles(c->td, nB, ts, n_wg, c->wcap, p);
        if (p.pool <= c->pool_len || n_wg == 1) break;
    }
    if (p.pool > c->pool_len || p.units.size() > (size_t)bt.n_wg + nB) {
        c->last_err = "gather units do not fit the search's scratch";
        return INSHR_E_INTERNAL;
    }
    int rc = ensure_host(c, c->h_up, at + (c->view_end - c->view_off));
    if (rc) return rc;
    char *hb = (char *)c->h_up.p + at, *db = (char *)c->search_mem.p;
    memcpy(hb, view.data(), sizeof(u32) * nB);
    memcpy(hb + (c->gw_off - c->view_off), p.wg0.data(), sizeof(u32) * p.wg0.size());
    memcpy(hb + (c->tgo_off - c->view_off), p.t_off.data(), sizeof(u32) * (nB + 1));
    memcpy(hb + (c->gun_off - c->view_off), p.units.data(), sizeof(Unit) * p.units.size());
    st.add(db + c->view_off, hb, c->gun_off - c->view_off + sizeof(Unit) * p.units.size());
    bt.n_gwg = (int)p.wg0.size() - 1;
    bt.n_gunits = (int)p.units.size();
    return INSHR_OK;
}

// Enqueues the work that gives boundaries, centres and errors of the configurations in view (per device
// position; VIEW_NONE: nothing; at: see upload_units).  The state is complete once the work is done and
// its results (TState::pool_overflow among them) have been looked at.
int resolve(inshr_ctx *c, const std::vector<u32> &view, size_t at)
{
    std::vector<u32> ts;
    for (uint32_t t = 0; t < (uint32_t)c->batch.nB; t++)
        if (view[t] != VIEW_NONE) ts.push_back(t);
    if (ts.empty()) return INSHR_OK;
    Partition p;
    Stage st;
    const int rc = upload_units(c, view, ts, p, at, st);
    if (rc) return rc;
    HIPCHK(c, launch_stage(st, c->n_cu, c->stream));
    HIPCHK(c, launch_resolve(c->batch, c->stream));
    return INSHR_OK;
}

// Tensors that launch_fused takes: its lists of protected values (one entry per protected value, in 1 / 16 of
// a unit's share of a pool for each wave) are made for small fractions.
constexpr uint32_t FUSE_MAX_PPM = 10000, FUSE_MIN_WCAP = 32;

// a tensor's span of the gather pools, which its units' lists share
void enter_span(QDesc &q, const Partition &p, u32 t)
{
    const u32 u0 = p.t_off[t], u1 = p.t_off[t + 1];
    q.fused = 1u;
    q.span = p.units[u0].off();
    q.span_len = p.units[u1 - 1].off() + (u64)p.units[u1 - 1].capw * (BLOCK / 64) - q.span;
}

bool fusable(const inshr_ctx *c, u32 g)
{
    return c->wcap >= FUSE_MIN_WCAP && c->grid_cfgs[g].outlier_ppm <= FUSE_MAX_PPM;
}

// Room in h_up that score_one takes: what upload_units stages, and the descriptors.
size_t score_one_bytes(const inshr_ctx *c) { return (c->view_end - c->view_off) + sizeof(QDesc) * (size_t)c->batch.nB + 256; }

// Enqueues the work that gives boundaries, centres and the exact error of one configuration per tensor (cfg: per device
// position, VIEW_NONE: none; all of them fusable) by the quantizer's sweep without its outputs.  A tensor that
// its means do not hold says so in its results (fuse_bad) and is left as it was.  Staged at offset at of h_up.
int score_one(inshr_ctx *c, const std::vector<u32> &cfg, size_t at)
{
    const uint32_t nB = (uint32_t)c->batch.nB;
    std::vector<u32> ts;
    for (uint32_t t = 0; t < nB; t++)
        if (cfg[t] != VIEW_NONE) ts.push_back(t);
    if (ts.empty()) return INSHR_OK;
    int rc = ensure_dev(c, c->aux_mem, sizeof(QDesc) * nB); // (less than the search took)
    if (rc) return rc;
    rc = ensure_host(c, c->h_up, at + score_one_bytes(c));
    if (rc) return rc;
    Partition p;
    Stage st;
    if ((rc = upload_units(c, std::vector<u32>(nB, VIEW_NONE), ts, p, at, st))) return rc;
    const size_t o_qd = (at + (c->view_end - c->view_off) + 255) & ~(size_t)255;
    QDesc *qd = (QDesc *)((char *)c->h_up.p + o_qd);
    memset(qd, 0, sizeof(QDesc) * nB);
    for (u32 t : ts) {
        qd[t].cfg = cfg[t];
        enter_span(qd[t], p, t);
    }
    st.add(c->aux_mem.p, qd, sizeof(QDesc) * nB);
    HIPCHK(c, launch_stage(st, c->n_cu, c->stream));
    HIPCHK(c, launch_fused(c->batch, (const QDesc *)c->aux_mem.p, nullptr, c->stream));
    return INSHR_OK;
}

// What a search is for.  CHOOSE: best and feasible alone; where bounds of the errors settle the choice of a
// tensor, nothing else is worked out for it (resolve() does so for the configurations that
// inshr_quantize asks for).  SCORES: every configuration's score.  GIVEN: thresholds and class counts for
// a quantizer whose configuration is given.  LIGHT: the same for the sketch quantizer, which
// brings its own bins and takes the protected counts per tile in its own sweep; the state is then
// not offered to INSHR_REUSE_SEARCH.
enum { CHOOSE, SCORES, GIVEN, LIGHT };

// The results of a search or of resolve(), which are in h_res: 1 when a wave's share of a gather pool was
// too small and the search has to be repeated (with the larger pools that pool_wcap stands for now).
int check_results(inshr_ctx *c, uint32_t nT, bool any_pooled)
{
    const std::vector<u32> &pos = c->pos;
    const SearchResult *res = (const SearchResult *)c->h_res.p;
    for (uint32_t t = 0; t < nT; t++) {
        if (res[t].nonfinite) return INSHR_E_NONFINITE;
    }
    for (uint32_t t = 0; t < nT; t++) {
        if (any_pooled && (res[pos[t]].internal_err & 32u)) { // (a tensor alone always keeps the value of rank P)
            c->last_err = "the shared thresholds leave tensor " + std::to_string(t) + " without quantized values";
            return INSHR_E_CONFIG;
        }
    }
    for (uint32_t t = 0; t < nT; t++) {
        const SearchResult &r = res[pos[t]];
        if (!r.pool_overflow) continue;
        // some wave gathered more keys than its share of a pool holds: larger pools, once more
        const uint32_t full = TILE / (BLOCK / 64);
        if (c->wcap >= full) {
            c->last_err = "gather pool overflow with full-size pools on tensor " + std::to_string(t);
            return INSHR_E_INTERNAL;
        }
        c->pool_wcap = std::min<uint32_t>(full, c->wcap * 2);
        if (getenv("INSHR_SAMPLE_DEBUG"))
            fprintf(stderr, "inshr_search: gather pools too small (tensor %u, code %u): again with %u keys per wave and tile\n",
                    t, r.pool_overflow, c->pool_wcap);
        return 1;
    }
    for (uint32_t t = 0; t < nT; t++) {
        if (res[pos[t]].internal_err) {
            c->last_err = "kernel self-check failed on tensor " + std::to_string(t) + ", code " +
                          std::to_string(res[pos[t]].internal_err);
            return INSHR_E_INTERNAL;
        }
    }
    return INSHR_OK;
}

// group: NULL, or one number per tensor; tensors with equal numbers share their thresholds, which
// are then order statistics of the group's pooled magnitudes (Sec. 4.2, per-layer-type pruning).
int run_search(inshr_ctx *c, const inshr_tensor *tensors, uint32_t nT, const inshr_config *grid,
               uint32_t n_cfg, double eps, int mode, const uint32_t *group = nullptr)
{
    const bool light = mode == LIGHT, want_scores = mode == SCORES;
    c->have_search = false;
    if (!tensors || !grid || nT == 0) return INSHR_E_ARG;
    // leader of every tensor's group and the group's size
    std::vector<u32> leader(nT);
    std::vector<u64> n_pool(nT, 0);
    std::vector<u32> members(nT, 0);
    bool any_pooled = false;
    {
        std::unordered_map<uint32_t, u32> first;
        for (uint32_t t = 0; t < nT; t++) {
            leader[t] = group ? first.emplace(group[t], t).first->second : t;
            n_pool[leader[t]] += tensors[t].n;
            members[leader[t]]++;
        }
        for (uint32_t t = 0; t < nT; t++) {
            if (members[leader[t]] > 1) any_pooled = true;
            if (n_pool[leader[t]] >= (1ull << 32)) {
                c->last_err = "a group of tensors that share thresholds holds 2^32 values or more";
                return INSHR_E_ARG;
            }
        }
    }
    GridDesc g;
    int rc = build_grid(grid, n_cfg, eps, g);
    if (rc) return rc;
    for (uint32_t t = 0; t < nT; t++) {
        if (!tensors[t].data || tensors[t].n == 0 || tensors[t].n >= (1ull << 32)) return INSHR_E_ARG;
        if ((uintptr_t)tensors[t].data & 3u) return INSHR_E_ARG;
    }
    // Order on the device: the tensors the sweeps search, then the small ones, each of which one
    // workgroup searches by itself (k_small).  A tensor that shares its thresholds is not searched by
    // itself, and a light search leaves the sketch what only the sweeps count.
    std::vector<u32> user_of(nT); // position in the caller's arrays of the tensor at a device position
    std::vector<u32> &pos = c->pos;
    pos.resize(nT);
    uint32_t nB = 0, nS1 = 0, nS0 = 0;
    {
        auto cls = [&](uint32_t t) { // 0: sweeps, 1 / 2: small
            if (light || members[leader[t]] > 1 || tensors[t].n > (u64)SMALL_MAX) return 0;
            return tensors[t].n > (u64)SMALL_TINY ? 1 : 2;
        };
        uint32_t cnt[3] = {0, 0, 0};
        for (uint32_t t = 0; t < nT; t++) cnt[cls(t)]++;
        nB = cnt[0];
        nS1 = cnt[1];
        nS0 = cnt[2];
        uint32_t at[3] = {0, nB, nB + nS1};
        for (uint32_t t = 0; t < nT; t++) {
            pos[t] = at[cls(t)]++;
            user_of[pos[t]] = t;
        }
    }
    uint64_t total_tiles = 0, all_tiles = 0; // of the tensors the sweeps search, of all
    for (uint32_t t = 0; t < nT; t++) {
        const u64 k = (tensors[t].n + TILE - 1) / TILE;
        all_tiles += k;
        if (pos[t] < nB) total_tiles += k;
    }
    HIPCHK(c, hipSetDevice(c->device));
    HIPCHK(c, hipStreamSynchronize(c->stream)); // staging buffers may be in flight (inshr_delta)

    // work partition: tiles are dealt out evenly to workgroups in order
    const int n_wg = sweep_workgroups(c, total_tiles), n_wg_all = sweep_workgroups(c, all_tiles);
    std::vector<TDesc> &td = c->td;
    td.assign(nT, TDesc());
    std::vector<u64> wg_tile0(n_wg + 1);
    size_t view_at = 0; // in h_up, behind what this call and a quantizer upload
    c->wcap = c->pool_wcap;
    {
        u64 tile = 0;
        bool any_sampled = false;
        for (uint32_t t = 0; t < nT; t++) {
            const uint32_t u = user_of[t];
            td[t].data = tensors[u].data;
            td[t].n = tensors[u].n;
            td[t].tile0 = tile;
            td[t].pool_grp = td[t].pool_len = 0;
            td[t].leader = pos[leader[u]];
            td[t].pooled = members[leader[u]] > 1 ? 1u : 0u;
            td[t].n_pool = n_pool[leader[u]];
            // (a sampled first sweep predicts where a tensor's own order statistics lie; a group's
            // come from the exact histograms of all its tensors)
            td[t].sampled = (!td[t].pooled && c->sample_min_n && td[t].n >= c->sample_min_n && t < nB &&
                             td[t].n < (1ull << 31)) ? 1u : 0u;
            any_sampled = any_sampled || td[t].sampled;
            tile += (td[t].n + TILE - 1) / TILE;
        }
        for (int w = 0; w <= n_wg; w++) wg_tile0[w] = n_wg ? total_tiles * (u64)w / (u64)n_wg : 0;
        Partition part;
        {
            std::vector<u32> all(nB);
            for (uint32_t t = 0; t < nB; t++) all[t] = t;
            deal_tiles(td, nB, all, n_wg, c->wcap, part);
        }
        const u32 units = (u32)part.units.size();
        const u64 pool = part.pool;
        for (u32 u = units; u-- > 0;) { // a tensor's span of the pool: its units'
            TDesc &d = td[part.units[u].tensor];
            d.pool_grp = part.units[u].off();
            d.pool_len += (u64)part.units[u].capw * (BLOCK / 64);
        }
        c->pool_len = pool;
        // device layout; what only boundaries and scores need is left out of a light search (k_plan2 ends it)
        Carver cv;
        auto full = [&](size_t bytes) { return light ? (size_t)0 : bytes; };
        const size_t o_td = cv.take(sizeof(TDesc) * nT);
        const size_t o_gd = cv.take(sizeof(GridDesc));
        const size_t o_wt = cv.take(sizeof(u64) * (n_wg + 1));
        const size_t o_wa = cv.take(sizeof(u64) * (n_wg_all + 1));
        const size_t o_wf = cv.take(sizeof(u32) * (n_wg + 1));
        const size_t o_tfo = cv.take(sizeof(u32) * (nB + 1));
        const size_t o_un = cv.take(sizeof(Unit) * units);
        const size_t up_bytes = cv.off;
        const size_t o_ts = cv.take(sizeof(TState) * nT);
        const size_t o_h1 = cv.off; // once the thresholds stand, the first histogram makes room for ...
        cv.take(((size_t)n_wg + nB) * 16 * 4); // ... counts and sums of the gather units (unit_prot, sq_prot), ...
        const size_t o_uc = cv.take(((size_t)n_wg + nB) * 16 * 4); // ... the keys they gathered (unit_cand) and ...
        c->view_off = cv.take(sizeof(u32) * nB); // ... what upload_units writes
        c->gw_off = cv.take(nB ? sizeof(u32) * (n_wg + 1) : 0);
        c->tgo_off = cv.take(nB ? sizeof(u32) * (nB + 1) : 0);
        c->gun_off = cv.take(sizeof(Unit) * ((size_t)n_wg + nB));
        c->view_end = cv.off;
        cv.off = std::max(cv.off, o_h1 + (size_t)nB * L1_BINS * 4);
        const size_t o_h2 = cv.take((size_t)nB * L2_BINS * 4);
        const size_t o_ph1 = cv.take(any_pooled ? (size_t)nB * L1_BINS * 4 : 0);
        const size_t zero_full = cv.off; // [o_ts, here) is cleared before the sweeps, and for a light search
        const size_t o_to = cv.take((size_t)total_tiles * MAX_FRAC * 4);
        const size_t zero_end = light ? cv.off : zero_full; // ... up to here (launch_resolve clears what it adds to)
        const size_t o_ngt = cv.take(256);
        const size_t o_gcn = cv.take(full((size_t)nB * 2 * MAX_EDGES * 4));
        const size_t o_gsx = cv.take(full((size_t)nB * 2 * MAX_EDGES * 8));
        const size_t o_ms = cv.take(full((size_t)nB * MAX_SUB * 8));
        const size_t o_psel = cv.take(any_pooled ? (size_t)nB * 2 * SEL_WORDS * 4 : 0);
        const size_t o_tab = cv.take((size_t)nT * COARSE * 4);
        const size_t o_ut = cv.take((size_t)units * 16 * 4);
        const size_t o_bi = cv.take(full((size_t)nB * L2_BINS * 4));
        const size_t o_tb = cv.take(full((size_t)nB * TGT_STRIDE * 4));
        const size_t o_tr = cv.take(full((size_t)nB * TGT_STRIDE * 4));
        const size_t o_tk = cv.take(full((size_t)nT * TGT_STRIDE * 4));
        const size_t o_sq = cv.take((size_t)units * SQ_STRIDE * 8);
        const size_t o_ed = cv.take(full((size_t)nB * MAX_EDGES * 4));
        const size_t o_sl = cv.take(full((size_t)nB * (L2_BINS + 64) * 2));
        const size_t o_pe = cv.take(full((size_t)nB * MAX_PAIRS * EIDX_STRIDE * 2));
        const size_t o_eb = cv.take(full((size_t)nB * MAX_EDGES * 4));
        const size_t o_ei = cv.take(full((size_t)nB * MAX_EDGES * 2));
        const size_t o_gel = cv.take(full((size_t)nB * MAX_GROUPS * 4));
        const size_t o_geh = cv.take(full((size_t)nB * MAX_GROUPS * 4));
        const size_t o_sgc = cv.take(full((size_t)nB * MAX_EDGES * 4));
        const size_t o_sbc = cv.take(full((size_t)nB * MAX_SUB * 4));
        const size_t o_sbn = cv.take(full((size_t)nB * MAX_SUB * 4));
        const size_t o_cb = cv.take(full((size_t)nT * n_cfg * CB_STRIDE * 4));
        const size_t o_sc = cv.take(full((size_t)nT * n_cfg * sizeof(Score)));
        const size_t o_bg = cv.take(full((size_t)nB * L2_BINS * 2));
        const size_t o_go = cv.take(full((size_t)nB * MAX_GROUPS * 4));
        const size_t o_ge = cv.take(full((size_t)nB * MAX_GROUPS * 4));
        const size_t o_gc = cv.take(full((size_t)nB * MAX_GROUPS * 4));
        const size_t o_tgg = cv.take(full((size_t)nB * TGT_STRIDE * 4));
        const size_t o_tkl = cv.take(full((size_t)nB * TGT_STRIDE * 4));
        const size_t o_tkh = cv.take(full((size_t)nB * TGT_STRIDE * 4));
        const size_t o_gl = cv.take(full((size_t)nB * MAX_GROUPS * 4));
        const size_t o_pool = cv.take((size_t)pool * 4);
        const size_t o_pool2 = cv.take(full((size_t)pool * 4));
        rc = ensure_dev(c, c->search_mem, cv.off);
        if (rc) return rc;
        // (as large as quantizing from this state will want it)
        view_at = std::max(up_bytes, QuantScratch(nT, nB, n_wg).up_bytes);
        rc = ensure_host(c, c->h_up, view_at + (c->view_end - c->view_off));
        if (rc) return rc;
        rc = ensure_host(c, c->h_res, sizeof(SearchResult) * nT);
        if (rc) return rc;
        char *hb = (char *)c->h_up.p;
        char *db = (char *)c->search_mem.p;
        memcpy(hb + o_td, td.data(), sizeof(TDesc) * nT);
        memcpy(hb + o_gd, &g, sizeof(GridDesc));
        memcpy(hb + o_wt, wg_tile0.data(), sizeof(u64) * (n_wg + 1));
        memcpy(hb + o_wf, part.wg0.data(), sizeof(u32) * part.wg0.size());
        memcpy(hb + o_tfo, part.t_off.data(), sizeof(u32) * (nB + 1));
        memcpy(hb + o_un, part.units.data(), sizeof(Unit) * units);
        {
            u64 *wa = (u64 *)(hb + o_wa);
            for (int w = 0; w <= n_wg_all; w++) wa[w] = all_tiles * (u64)w / (u64)n_wg_all;
        }
        Stage up;
        up.add(db, hb, up_bytes);
        up.zero(db + o_ts, zero_end - o_ts);
        HIPCHK(c, launch_stage(up, c->n_cu, c->stream));

        Batch &bt = c->batch;
        bt.td = (const TDesc *)(db + o_td);
        bt.gd = (const GridDesc *)(db + o_gd);
        bt.wg_tile0 = (const u64 *)(db + o_wt);
        bt.wg_fu0 = (const u32 *)(db + o_wf);
        bt.t_fu_off = (const u32 *)(db + o_tfo);
        bt.wg_gu0 = (const u32 *)(db + c->gw_off);
        bt.t_gu_off = (const u32 *)(db + c->tgo_off);
        bt.grp_list = (u32 *)(db + o_gl);
        bt.n_grp_total = (u32 *)(db + o_ngt);
        bt.n_units = (int)units;
        bt.n_bucket_blocks = c->n_cu * 4;
        bt.n_cu = c->n_cu;
        bt.lds_ordered = c->lds_ordered;
        bt.any_sampled = any_sampled;
        bt.any_pooled = any_pooled;
        bt.force_miss = c->sample_force_miss;
        bt.wg_tile0_all = (const u64 *)(db + o_wa);
        bt.nT = (int)nT;
        bt.nB = (int)nB;
        bt.nS1 = (int)nS1;
        bt.nS0 = (int)nS0;
        bt.n_wg = n_wg;
        bt.n_wg_all = n_wg_all;
        bt.n_pairs = g.n_pairs;
        bt.n_cfg = n_cfg;
        bt.n_tiles = all_tiles;
        Bufs &B = bt.bufs;
        B.ts = (TState *)(db + o_ts);
        B.res = (SearchResult *)c->h_res.p;
        B.hist1 = (u32 *)(db + o_h1);
        B.pool_h1 = (u32 *)(db + o_ph1);
        B.pool_sel = (u32 *)(db + o_psel);
        B.hist2 = (u32 *)(db + o_h2);
        B.table2 = (u32 *)(db + o_tab);
        B.units = (const Unit *)(db + o_un);
        B.gunits = (const Unit *)(db + c->gun_off);
        B.view = (const u32 *)(db + c->view_off);
        B.unit_thr = (u32 *)(db + o_ut);
        B.binfo = (u32 *)(db + o_bi);
        B.tgt_bin = (u32 *)(db + o_tb);
        B.tgt_res = (u32 *)(db + o_tr);
        B.tgt_key = (u32 *)(db + o_tk);
        B.pool = (u32 *)(db + o_pool);
        B.pool2 = (u32 *)(db + o_pool2);
        B.unit_cand = (u32 *)(db + o_uc);
        B.unit_prot = (u32 *)(db + o_h1);
        B.bin_group = (u16 *)(db + o_bg);
        B.grp_off = (u32 *)(db + o_go);
        B.grp_end = (u32 *)(db + o_ge);
        B.grp_cur = (u32 *)(db + o_gc);
        B.tgt_rank = (u32 *)(db + o_tgg);
        B.tgt_klo = (u32 *)(db + o_tkl);
        B.tgt_khi = (u32 *)(db + o_tkh);
        B.tile_out = (u32 *)(db + o_to);
        B.sq_part = (double *)(db + o_sq);
        B.sq_prot = (double *)(db + o_h1);
        static_assert(MAX_FRAC * sizeof(double) == 16 * sizeof(u32), "sq_prot and unit_prot take the same room");
        B.edges = (u32 *)(db + o_ed);
        B.sl = (u16 *)(db + o_sl);
        B.pair_eidx = (u16 *)(db + o_pe);
        B.edge_bin = (u32 *)(db + o_eb);
        B.edge_item = (u16 *)(db + o_ei);
        B.grp_elo = (u32 *)(db + o_gel);
        B.grp_ehi = (u32 *)(db + o_geh);
        B.seg_cnt = (u32 *)(db + o_sgc);
        B.grp_cnt = (u32 *)(db + o_gcn);
        B.grp_sx = (double *)(db + o_gsx);
        B.mom_sx = (u64 *)(db + o_ms);
        B.sub_code = (u32 *)(db + o_sbc);
        B.sub_cnt = (u32 *)(db + o_sbn);
        B.codebook = (float *)(db + o_cb);
        B.scores = (Score *)(db + o_sc);
        c->scores_off = o_sc;
    }
    c->grid_cfgs.assign(grid, grid + n_cfg);
    c->batch.light = light;
    c->batch.spread = mode == CHOOSE || mode == LIGHT;
    if (mode != CHOOSE) HIPCHK(c, launch_small(c->batch, c->stream));
    HIPCHK(c, launch_select(c->batch, c->stream));
    c->resolved.assign(nT, VIEW_ALL); // (the small tensors are searched completely)
    std::fill(c->resolved.begin(), c->resolved.begin() + nB, VIEW_NONE);
    if (mode == CHOOSE) {
        HIPCHK(c, launch_decide(c->batch, c->stream));
    } else if (mode == SCORES) {
        std::fill(c->resolved.begin(), c->resolved.begin() + nB, VIEW_ALL);
        if ((rc = resolve(c, c->resolved, view_at))) return rc;
    } else {
        HIPCHK(c, launch_counts(c->batch, c->stream));
    }

    // results, in device order
    const size_t sc_bytes = want_scores ? sizeof(Score) * (size_t)nT * n_cfg : 0;
    rc = ensure_host(c, c->h_down, std::max(sc_bytes, sizeof(QInfo) * nT));
    if (rc) return rc;
    char *db = (char *)c->search_mem.p;
    const SearchResult *res = (const SearchResult *)c->h_res.p;
    std::vector<char> tried(nB, 0);
    for (;;) {
        if (sc_bytes)
            HIPCHK(c, hipMemcpyAsync(c->h_down.p, db + c->scores_off, sc_bytes, hipMemcpyDeviceToHost, c->stream));
        HIPCHK(c, hipStreamSynchronize(c->stream));
        rc = check_results(c, nT, any_pooled);
        if (rc == 1) return run_search(c, tensors, nT, grid, n_cfg, eps, mode, group);
        if (rc) return rc;
        // Tensors whose choice the bounds leave open are scored: the configuration it hangs on, by the quantizer's
        // sweep where its means hold all of them (they go along where a tensor's whole grid is scored: the other
        // chain of kernels takes longer than they do on top of it, BERT-base with Adam state 3.11 instead of 3.03 ms),
        // or the whole grid.
        std::vector<u32> open(nB, VIEW_NONE);
        bool any_open = false, fuse = true;
        for (uint32_t t = 0; t < nB; t++)
            if (res[t].best >= CHOICE_IF) {
                open[t] = c->resolved[t] = res[t].best == VIEW_NONE ? VIEW_ALL : res[t].best & ~CHOICE_IF;
                fuse = fuse && open[t] != VIEW_ALL && !tried[t] && fusable(c, open[t]);
                tried[t] = any_open = true;
            }
        if (!any_open) break;
        if (fuse) {
            rc = ensure_host(c, c->h_up, view_at + score_one_bytes(c)); // (nothing is in flight)
            if (rc) return rc;
        }
        if ((rc = fuse ? score_one(c, open, view_at) : resolve(c, open, view_at))) return rc;
    }
    if (getenv("INSHR_SAMPLE_DEBUG")) { // how many sampled first sweeps had to be repeated exactly
        uint32_t n_sampled = 0, n_redo = 0;
        for (uint32_t t = 0; t < nT; t++) {
            n_sampled += td[pos[t]].sampled ? 1u : 0u;
            const uint32_t redo = res[pos[t]].redo;
            n_redo += redo ? 1u : 0u;
            if (redo)
                fprintf(stderr, "inshr_search: tensor %u (n = %llu) repeated, thresholds missed: 0x%x\n", t,
                        (unsigned long long)tensors[t].n, redo >> 1);
        }
        fprintf(stderr, "inshr_search: %u tensors, %u with a sampled first sweep, %u of them repeated\n",
                nT, n_sampled, n_redo);
    }
    c->grid = g;
    c->tensors.assign(tensors, tensors + nT);
    c->groups.clear();
    if (group) c->groups.assign(group, group + nT);
    c->eps = eps;
    c->mode = mode;
    c->any_pooled = any_pooled;
    c->have_search = !light;
    return INSHR_OK;
}

// The last search once more, for larger pools (check_results).
int repeat_search(inshr_ctx *c)
{
    const std::vector<inshr_tensor> tensors = c->tensors;
    const std::vector<inshr_config> grid = c->grid_cfgs;
    const std::vector<u32> groups = c->groups;
    return run_search(c, tensors.data(), (uint32_t)tensors.size(), grid.data(), (uint32_t)grid.size(), c->eps, c->mode,
                      groups.empty() ? nullptr : groups.data());
}

// Boundaries, centres and scores of one configuration per tensor (cfg: by the caller's order) after a search for given
// configurations; the scores go to h_down, for every configuration of the grid and device position.  1: the search has to
// be repeated for larger pools.
int score_given(inshr_ctx *c, const std::vector<uint32_t> &cfg)
{
    const uint32_t nT = (uint32_t)c->batch.nT, nB = (uint32_t)c->batch.nB;
    const size_t sc_bytes = sizeof(Score) * (size_t)nT * c->batch.n_cfg;
    int rc = ensure_host(c, c->h_down, sc_bytes);
    if (rc) return rc;
    std::vector<u32> want(nB, VIEW_NONE), one(nB, VIEW_NONE), apart(nB, VIEW_NONE);
    for (uint32_t t = 0; t < nT; t++)
        if (c->pos[t] < nB) want[c->pos[t]] = cfg[t];
    for (uint32_t t = 0; t < nB; t++) (fusable(c, want[t]) ? one : apart)[t] = want[t];
    const SearchResult *res = (const SearchResult *)c->h_res.p;
    for (;;) {
        // (each of the two stages its units in a place of its own)
        const size_t one_at = (c->view_end - c->view_off + 255) & ~(size_t)255;
        rc = ensure_host(c, c->h_up, one_at + score_one_bytes(c)); // (nothing is in flight)
        if (rc) return rc;
        if ((rc = score_one(c, one, one_at))) return rc;
        if ((rc = resolve(c, apart, 0))) return rc;
        HIPCHK(c, hipMemcpyAsync(c->h_down.p, (char *)c->search_mem.p + c->scores_off, sc_bytes, hipMemcpyDeviceToHost, c->stream));
        HIPCHK(c, hipStreamSynchronize(c->stream));
        rc = check_results(c, nT, c->any_pooled);
        if (rc) return rc;
        bool again = false;
        for (uint32_t t = 0; t < nB; t++) {
            apart[t] = one[t] != VIEW_NONE && res[t].fuse_bad ? one[t] : VIEW_NONE;
            again = again || apart[t] != VIEW_NONE;
            one[t] = VIEW_NONE;
        }
        if (!again) return INSHR_OK;
    }
}

// Everything a search with scores leaves behind, for all tensors.
int resolve_all(inshr_ctx *c)
{
    const uint32_t nT = (uint32_t)c->batch.nT;
    for (;;) {
        std::vector<u32> view(nT, VIEW_NONE);
        bool any = false;
        for (uint32_t t = 0; t < (uint32_t)c->batch.nB; t++)
            if (c->resolved[t] != VIEW_ALL) {
                view[t] = VIEW_ALL;
                any = true;
            }
        if (!any) return INSHR_OK;
        HIPCHK(c, hipStreamSynchronize(c->stream));
        int rc = resolve(c, view, 0);
        if (rc) return rc;
        HIPCHK(c, hipStreamSynchronize(c->stream));
        rc = check_results(c, nT, c->any_pooled);
        if (rc == 1) {
            if ((rc = repeat_search(c))) return rc;
            continue;
        }
        if (rc) return rc;
        std::fill(c->resolved.begin(), c->resolved.end(), VIEW_ALL);
    }
}

} // namespace

extern "C" {

int inshr_create(inshr_ctx **out, int device, void *hip_stream, uint64_t scratch_bytes)
{
    if (!out) return INSHR_E_ARG;
    *out = nullptr;
    int n_dev = 0;
    if (hipGetDeviceCount(&n_dev) != hipSuccess || device < 0 || device >= n_dev) return INSHR_E_DEVICE;
    inshr_ctx *c = new inshr_ctx();
    c->device = device;
    c->stream = (hipStream_t)hip_stream;
    c->scratch_limit = scratch_bytes;
    hipDeviceProp_t pr;
    if (hipSetDevice(device) != hipSuccess || hipGetDeviceProperties(&pr, device) != hipSuccess) {
        delete c;
        return INSHR_E_DEVICE;
    }
    c->n_cu = pr.multiProcessorCount > 0 ? pr.multiProcessorCount : 256;
    if (const char *e = getenv("INSHR_WG_PER_CU")) {
        int v = atoi(e);
        if (v >= 1 && v <= 16) c->wg_per_cu = v;
    }
    // the delta scatter and the group sort have a fast path that needs same-address LDS atomics to
    // be served in lane order; it is used only if this device passes the check
    // (INSHR_NO_LDS_ORDER=1, or its older name INSHR_DELTA_SLOTS=1, forces it off)
    {
        u32 *viol = nullptr;
        u32 h = 1;
        if (hipMalloc(&viol, 4) == hipSuccess) {
            if (hipMemsetAsync(viol, 0, 4, c->stream) == hipSuccess &&
                launch_lds_order_check(viol, c->stream) == hipSuccess &&
                hipMemcpyAsync(&h, viol, 4, hipMemcpyDeviceToHost, c->stream) == hipSuccess &&
                hipStreamSynchronize(c->stream) == hipSuccess)
                c->lds_ordered = (h == 0);
            (void)hipFree(viol);
        }
        for (const char *name : {"INSHR_NO_LDS_ORDER", "INSHR_DELTA_SLOTS"})
            if (const char *e = getenv(name))
                if (atoi(e) != 0) c->lds_ordered = false;
    }
    {
        const size_t n_flags = 256;
        const struct { HostBuf *b; size_t bytes; } first[3] = {{&c->h_res, 16 << 10}, {&c->h_down, 16 << 10}, {&c->h_up, 64 << 10}};
        size_t bytes = n_flags;
        for (auto &f : first) bytes += f.bytes;
        if (hipHostMalloc((void **)&c->pinned, bytes, hipHostMallocDefault) != hipSuccess || delta_static_init(device) != hipSuccess) {
            if (c->pinned) (void)hipHostFree(c->pinned);
            delete c;
            return INSHR_E_DEVICE;
        }
        c->flags = (u32 *)c->pinned;
        size_t at = n_flags;
        for (auto &f : first) {
            f.b->p = c->pinned + at;
            f.b->cap = f.bytes;
            f.b->lent = true;
            at += f.bytes;
        }
    }
    if (const char *e = getenv("INSHR_SAMPLE_MIN_N")) c->sample_min_n = strtoull(e, nullptr, 10);
    if (const char *e = getenv("INSHR_SAMPLE_FORCE_MISS")) c->sample_force_miss = atoi(e) != 0;
    if (const char *e = getenv("INSHR_POOL_WCAP")) {
        const long v = atol(e);
        if (v >= 1 && v <= TILE / (BLOCK / 64)) c->pool_wcap = (uint32_t)v;
    }
    *out = c;
    return INSHR_OK;
}

void inshr_destroy(inshr_ctx *c)
{
    if (!c) return;
    (void)hipSetDevice(c->device);
    (void)hipStreamSynchronize(c->stream);
    if (c->search_mem.p) (void)hipFree(c->search_mem.p);
    if (c->aux_mem.p) (void)hipFree(c->aux_mem.p);
    if (c->totals_mem.p) (void)hipFree(c->totals_mem.p);
    if (c->sketch_mem.p) (void)hipFree(c->sketch_mem.p);
    if (c->sens_mem.p) (void)hipFree(c->sens_mem.p);
    for (const HostBuf *h : {&c->h_up, &c->h_down, &c->h_res})
        if (h->p && !h->lent) (void)hipHostFree(h->p);
    if (c->pinned) (void)hipHostFree(c->pinned);
    delete c;
}

const char *inshr_strerror(int code)
{
    switch (code) {
    case INSHR_OK: return "ok";
    case INSHR_E_ARG: return "bad argument";
    case INSHR_E_CONFIG: return "bad configuration or grid too large";
    case INSHR_E_NONFINITE: return "NaN or Inf in a tensor";
    case INSHR_E_CAPACITY: return "buffer or scratch too small";
    case INSHR_E_SHAPE: return "shape mismatch";
    case INSHR_E_DEVICE: return "HIP error";
    case INSHR_E_INTERNAL: return "internal self-check failed";
    default: return "unknown error";
    }
}

const char *inshr_last_device_error(const inshr_ctx *c) { return c ? c->last_err.c_str() : ""; }

int inshr_sync(inshr_ctx *c)
{
    if (!c) return INSHR_E_ARG;
    HIPCHK(c, hipSetDevice(c->device));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    return take_delta_flags(c);
}

int inshr_lds_ordered(const inshr_ctx *c) { return (c && c->lds_ordered) ? 1 : 0; }

int inshr_profile(inshr_ctx *c, int enable)
{
    if (!c) return INSHR_E_ARG;
    HIPCHK(c, hipSetDevice(c->device));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    prof_collect();
    g_prof.on = enable != 0;
    if (enable) {
        g_prof.names.clear();
        g_prof.total_ms.clear();
        g_prof.launches.clear();
    }
    return INSHR_OK;
}

int inshr_profile_read(inshr_ctx *c, inshr_kernel_time *out, uint32_t cap, uint32_t *n)
{
    if (!c || !n) return INSHR_E_ARG;
    HIPCHK(c, hipSetDevice(c->device));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    prof_collect();
    *n = (uint32_t)g_prof.names.size();
    for (uint32_t i = 0; i < *n && i < cap && out; i++) {
        memset(&out[i], 0, sizeof(out[i]));
        strncpy(out[i].name, g_prof.names[i].c_str(), sizeof(out[i].name) - 1);
        out[i].total_ms = g_prof.total_ms[i];
        out[i].launches = g_prof.launches[i];
    }
    return INSHR_OK;
}

// what the last search downloaded, in the caller's order
static void take_results(const inshr_ctx *c, uint32_t nT, uint32_t n_cfg, uint32_t *best, uint8_t *feasible,
                         inshr_score *scores)
{
    static_assert(sizeof(Score) == sizeof(inshr_score), "score layout");
    const SearchResult *res = (const SearchResult *)c->h_res.p;
    const Score *hsc = (const Score *)c->h_down.p;
    for (uint32_t t = 0; t < nT; t++) {
        const u32 p = c->pos[t];
        best[t] = res[p].best;
        feasible[t] = (uint8_t)res[p].feasible;
        if (scores) memcpy(scores + (size_t)t * n_cfg, hsc + (size_t)p * n_cfg, sizeof(Score) * n_cfg);
    }
}

int inshr_search(inshr_ctx *c, const inshr_tensor *tensors, uint32_t n_tensors,
                 const inshr_config *grid, uint32_t n_cfg, double eps, uint32_t *best,
                 uint8_t *feasible, inshr_score *scores)
{
    if (!c || !best || !feasible) return INSHR_E_ARG;
    int rc = run_search(c, tensors, n_tensors, grid, n_cfg, eps, scores ? SCORES : CHOOSE);
    if (rc) return rc;
    take_results(c, n_tensors, n_cfg, best, feasible, scores);
    return INSHR_OK;
}

int inshr_search_pooled(inshr_ctx *c, const inshr_tensor *tensors, const uint32_t *group,
                        uint32_t n_tensors, const inshr_config *grid, uint32_t n_cfg, double eps,
                        uint32_t *best, uint8_t *feasible, inshr_score *scores)
{
    if (!c || !best || !feasible || !group) return INSHR_E_ARG;
    int rc = run_search(c, tensors, n_tensors, grid, n_cfg, eps, scores ? SCORES : CHOOSE, group);
    if (rc) return rc;
    take_results(c, n_tensors, n_cfg, best, feasible, scores);
    return INSHR_OK;
}

int inshr_quantize_bound(uint64_t n, const inshr_config *cfg, uint64_t *packed_words,
                         uint64_t *outlier_cap)
{
    if (!cfg || n == 0 || n >= (1ull << 32)) return INSHR_E_ARG;
    int rc = check_config(*cfg);
    if (rc) return rc;
    if (packed_words) *packed_words = (n * (uint64_t)symbol_bits(bins_of(*cfg)) + 63) / 64;
    if (outlier_cap) *outlier_cap = n * (uint64_t)cfg->outlier_ppm / 1000000ull;
    return INSHR_OK;
}

static int quantize_with_state(inshr_ctx *c, const inshr_config *cfg, inshr_quantized *out,
                               const uint32_t *which, uint32_t n_sel, const u32 *alt_key = nullptr,
                               const float *alt_cb = nullptr, bool val_bf16 = false)
{
    // alt_key / alt_cb: device arrays with 256 entries per tensor of the batch that replace the
    // search's boundaries and centres
    // which[k] = position in the search batch of the k-th tensor to quantize (cfg / out indexed by k)
    const uint32_t nT = (uint32_t)c->batch.nT;
    std::vector<QDesc> qd(nT);
    for (auto &q : qd) memset(&q, 0, sizeof(q));
    uint32_t gi = 0;
    for (uint32_t k = 0; k < n_sel; k++) {
        const uint32_t u = which[k], t = c->pos[u]; // in the caller's order, on the device
        if (k == 0 || !same_config(c->grid_cfgs[gi], cfg[k])) { // (neighbours often have the same one)
            for (gi = 0; gi < c->grid.n_cfg; gi++)
                if (same_config(c->grid_cfgs[gi], cfg[k])) break;
            if (gi == c->grid.n_cfg) return INSHR_E_SHAPE;
        }
        uint64_t words = 0, cap = 0;
        inshr_quantize_bound(c->tensors[u].n, &cfg[k], &words, &cap);
        if (!out[k].packed || !out[k].codebook || out[k].packed_words < words) return INSHR_E_CAPACITY;
        if (out[k].outlier_cap && (!out[k].outlier_idx || !out[k].outlier_val)) return INSHR_E_ARG;
        qd[t].packed = (unsigned long long *)out[k].packed;
        qd[t].codebook = out[k].codebook;
        qd[t].boundaries = out[k].boundaries;
        qd[t].out_idx = out[k].outlier_idx;
        qd[t].out_val = out[k].outlier_val;
        qd[t].out_cap = out[k].outlier_cap;
        qd[t].cfg = gi;
        qd[t].val_bf16 = val_bf16 ? 1u : 0u;
        qd[t].alt_key = alt_key ? alt_key + (size_t)t * 256 : nullptr;
        qd[t].alt_cb = alt_cb ? alt_cb + (size_t)t * 256 : nullptr;
    }
    const uint32_t nB = (uint32_t)c->batch.nB;
    const QuantScratch lay(nT, nB, c->batch.n_wg);
    const size_t o_qd = lay.qd, o_wg = lay.wg, o_un = lay.un, up_bytes = lay.up_bytes;
    HIPCHK(c, hipStreamSynchronize(c->stream)); // staging buffers and scratch may be in use (inshr_delta)
    int rc = ensure_dev(c, c->aux_mem, lay.bytes);
    if (rc) return rc;
    rc = ensure_host(c, c->h_up, up_bytes);
    if (rc) return rc;
    rc = ensure_host(c, c->h_down, sizeof(QInfo) * nT);
    if (rc) return rc;
    char *db = (char *)c->aux_mem.p;
    QInfo *const qi = (QInfo *)c->h_down.p;
    // Tensors whose boundaries and centres the state does not hold are quantized in one sweep that works them
    // out (launch_fused).  Where that does not do (a protect fraction whose lists are long, or what the
    // kernels find too much for them), and for those the state holds, the ordinary way.
    std::vector<char> done(nT, 0), apart(nT, 0);
    const std::vector<QDesc> asked = nB ? qd : std::vector<QDesc>();
    for (;;) {
        std::vector<u32> fuse, ready, view(nT, VIEW_NONE);
        bool open = false;
        for (uint32_t t = 0; t < nB; t++) {
            if (!asked[t].packed || done[t]) continue;
            if (alt_key || c->resolved[t] == VIEW_ALL || c->resolved[t] == asked[t].cfg)
                ready.push_back(t);
            else if (!apart[t] && fusable(c, asked[t].cfg))
                fuse.push_back(t);
            else
                open = true;
        }
        Partition p;
        Stage up;
        if (!fuse.empty()) {
            if ((rc = upload_units(c, view, fuse, p, up_bytes, up))) return rc;
            for (u32 t : fuse) c->resolved[t] = VIEW_NONE;
        } else if (open) {
            ready.clear();
            for (uint32_t t = 0; t < nB; t++) {
                if (!asked[t].packed || done[t]) continue;
                if (c->resolved[t] != VIEW_ALL && c->resolved[t] != asked[t].cfg) view[t] = asked[t].cfg;
                ready.push_back(t);
            }
            if ((rc = resolve(c, view, up_bytes))) return rc;
        }
        for (uint32_t t = 0; nB && t < nT; t++) { // (the state holds nothing yet for those that wait for a later pass)
            qd[t] = asked[t];
            if (done[t] || t < nB) qd[t].packed = nullptr;
        }
        for (u32 t : ready) qd[t].packed = asked[t].packed;
        for (u32 t : fuse) {
            qd[t].packed = asked[t].packed;
            enter_span(qd[t], p, t);
        }
        Partition pq;
        deal_tiles(c->td, nB, ready, c->batch.n_wg, c->wcap, pq);
        char *hb = (char *)c->h_up.p;
        memcpy(hb + o_qd, qd.data(), sizeof(QDesc) * nT);
        memcpy(hb + o_wg, pq.wg0.data(), sizeof(u32) * pq.wg0.size());
        memcpy(hb + o_un, pq.units.data(), sizeof(Unit) * pq.units.size());
        up.add(db, hb, o_un + sizeof(Unit) * pq.units.size());
        HIPCHK(c, launch_stage(up, c->n_cu, c->stream));
        const QDesc *dq = (const QDesc *)(db + o_qd);
        if (!fuse.empty()) HIPCHK(c, launch_fused(c->batch, dq, qi, c->stream));
        HIPCHK(c, launch_quantize(c->batch, dq, (const Unit *)(db + o_un), (const u32 *)(db + o_wg),
                                  (int)pq.wg0.size() - 1, qi, c->stream));
        const bool any = !fuse.empty() || open;
        HIPCHK(c, hipStreamSynchronize(c->stream));
        if (!any) break;
        rc = check_results(c, nT, c->any_pooled);
        if (rc < 0) return rc;
        if (rc == 1) { // larger pools: from the start
            if ((rc = repeat_search(c))) return rc;
            std::fill(done.begin(), done.end(), 0);
            continue;
        }
        const SearchResult *res = (const SearchResult *)c->h_res.p;
        for (uint32_t t = 0; t < nT; t++) done[t] = asked[t].packed && (t >= nB || done[t]);
        for (u32 t : ready) done[t] = 1;
        for (u32 t : fuse) {
            (res[t].fuse_bad ? apart : done)[t] = 1;
            if (!res[t].fuse_bad) c->resolved[t] = asked[t].cfg; // (what the sweep worked out is in the state)
        }
        for (uint32_t t = 0; t < nB; t++)
            if (view[t] != VIEW_NONE) c->resolved[t] = view[t];
        bool all = true;
        for (uint32_t t = 0; t < nT; t++) all = all && (done[t] || !asked[t].packed);
        if (all) break;
    }
    int result = INSHR_OK;
    for (uint32_t k = 0; k < n_sel; k++) {
        const QInfo &r = qi[c->pos[which[k]]];
        out[k].n_pruned = r.n_pruned;
        out[k].n_outlier = r.n_outlier;
        out[k].n_kept = r.n_kept;
        out[k].n_bins = bins_of(cfg[k]);
        out[k].sym_bits = symbol_bits(out[k].n_bins);
        uint32_t tp = r.tau_p, to = r.tau_o;
        memcpy(&out[k].tau_prune, &tp, 4);
        memcpy(&out[k].tau_outlier, &to, 4);
        if (r.flags & 1u) {
            c->last_err = "protected-value count self-check failed";
            result = INSHR_E_INTERNAL;
        } else if ((r.flags & 2u) && result == INSHR_OK) {
            result = INSHR_E_CAPACITY;
        }
    }
    return result;
}

int inshr_quantize(inshr_ctx *c, const inshr_tensor *tensors, const inshr_config *cfg,
                   inshr_quantized *out, uint32_t n_tensors, uint32_t flags)
{
    if (!c || !tensors || !cfg || !out || n_tensors == 0) return INSHR_E_ARG;
    for (uint32_t t = 0; t < n_tensors; t++) {
        int rc = check_config(cfg[t]);
        if (rc) return rc;
    }
    HIPCHK(c, hipSetDevice(c->device));
    if (flags & INSHR_REUSE_SEARCH) {
        if (!c->have_search || c->tensors.size() != n_tensors) return INSHR_E_SHAPE;
        std::vector<uint32_t> which(n_tensors);
        for (uint32_t t = 0; t < n_tensors; t++) {
            if (c->tensors[t].data != tensors[t].data || c->tensors[t].n != tensors[t].n) return INSHR_E_SHAPE;
            which[t] = t;
        }
        return quantize_with_state(c, cfg, out, which.data(), n_tensors, nullptr, nullptr,
                                   (flags & INSHR_PROTECT_BF16) != 0);
    }
    // stand-alone: one internal single-configuration search per distinct configuration
    std::vector<char> done(n_tensors, 0);
    for (uint32_t t0 = 0; t0 < n_tensors; t0++) {
        if (done[t0]) continue;
        std::vector<inshr_tensor> sub;
        std::vector<inshr_config> subcfg;
        std::vector<uint32_t> idx;
        for (uint32_t t = t0; t < n_tensors; t++) {
            if (!done[t] && same_config(cfg[t], cfg[t0])) {
                done[t] = 1;
                sub.push_back(tensors[t]);
                subcfg.push_back(cfg[t]);
                idx.push_back(t);
            }
        }
        int rc = run_search(c, sub.data(), (uint32_t)sub.size(), &cfg[t0], 1, 0.0, GIVEN);
        if (rc) return rc;
        std::vector<inshr_quantized> subout(sub.size());
        std::vector<uint32_t> which(sub.size());
        for (size_t k = 0; k < sub.size(); k++) {
            subout[k] = out[idx[k]];
            which[k] = (uint32_t)k;
        }
        rc = quantize_with_state(c, subcfg.data(), subout.data(), which.data(), (uint32_t)sub.size(), nullptr,
                                 nullptr, (flags & INSHR_PROTECT_BF16) != 0);
        for (size_t k = 0; k < sub.size(); k++) out[idx[k]] = subout[k];
        if (rc) return rc;
    }
    return INSHR_OK;
}

// ------------------------------------------------------------------------------------------
// sketch + weighted K-Means boundaries
// ------------------------------------------------------------------------------------------
namespace {

struct SketchTables {
    std::vector<u32> cell, tops;
    std::vector<double> rep;
    int i_lo = 0; // tops[b] belongs to bucket index i_lo + b
};

// Tables of the bucket law ceil(log_gamma |x|): tops[b] = magnitude image of the largest fp32
// number <= gamma^(i_lo + b) (extended precision; a value x lies in the first bucket whose top
// reaches it), rep[b] = the bucket's value, cell[c] = first bucket and its top for the magnitudes
// c << 17 .. (c << 17) + 2^17 - 1.
int build_sketch_tables(inshr_ctx *ctx, double alpha, SketchTables &T)
{
    if (!(alpha >= 0.01 && alpha <= 0.5)) return INSHR_E_CONFIG;
    if (ctx && ctx->sketch_alpha == alpha) { // the tables of the call before
        T.i_lo = ctx->sketch_i_lo;
        T.cell = ctx->sketch_cell;
        T.tops = ctx->sketch_tops;
        T.rep = ctx->sketch_rep;
        return INSHR_OK;
    }
    const double gamma = (1.0 + alpha) / (1.0 - alpha);
    const long double lg = logl((long double)gamma);
    const int i_lo = (int)floorl(-149.0L * logl(2.0L) / lg) - 2;
    const int i_hi = (int)ceill(128.0L * logl(2.0L) / lg) + 1;
    const int n_idx = i_hi - i_lo + 1;
    if (n_idx > SK_MAX_IDX) return INSHR_E_CONFIG;
    T.i_lo = i_lo;
    T.tops.resize(n_idx);
    T.rep.resize(n_idx);
    for (int b = 0; b < n_idx; b++) {
        const int i = i_lo + b;
        const long double v = powl((long double)gamma, (long double)i);
        float f;
        if (v >= (long double)3.402823466e+38F) {
            f = 3.402823466e+38F;
        } else {
            f = (float)v;
            if ((long double)f > v) f = nextafterf(f, -1.0f); // round down (v > 0)
        }
        u32 bits;
        memcpy(&bits, &f, 4);
        T.tops[b] = bits;
        T.rep[b] = 2.0 * pow(gamma, (double)i) / (gamma + 1.0);
    }
    T.cell.assign(SK_CELLS, (u32)(n_idx - 1) << 17);
    for (u32 c = 64; c < (0x7f800000u >> 17); c++) { // normal numbers
        const u32 first = c << 17, last = first | 0x1FFFFu;
        const u32 b0 = (u32)(std::lower_bound(T.tops.begin(), T.tops.end(), first) - T.tops.begin());
        if (b0 + 1u >= (u32)n_idx || T.tops[b0 + 1u] < last) return INSHR_E_CONFIG; // more than two buckets
        const u32 split = T.tops[b0] <= last ? (T.tops[b0] & 0x1FFFFu) : 0x1FFFFu;
        T.cell[c] = (b0 << 17) | (0x1FFFFu - split); // adding the low magnitude bits carries above the split
    }
    if (ctx) {
        ctx->sketch_cell = T.cell;
        ctx->sketch_tops = T.tops;
        ctx->sketch_rep = T.rep;
        ctx->sketch_i_lo = i_lo;
        ctx->sketch_alpha = alpha;
    }
    return INSHR_OK;
}

} // namespace

namespace {

// Sketch and clustering for tensors which[k] of the searched batch with configurations cfg[k] (all
// in the search's grid); src[k] = the tensor's position in the caller's arrays (uniforms, info).
// Leaves 256 boundary keys and centres per tensor of the batch in *alt_key / *alt_cb (device).
int sketch_with_state(inshr_ctx *c, const inshr_config *cfg, const uint32_t *which, const uint32_t *src,
                      uint32_t n_sel, const inshr_sketch_params *params, const SketchTables &T,
                      inshr_sketch_info *info, const u32 **alt_key, const float **alt_cb,
                      bool multi = false, double eps = 0.0, inshr_sketch_choice *choice = nullptr)
{
    // multi: centres for 2 .. 8 bits, their exact errors and the choice (cfg[k].bits must be 8 then:
    // it names the grid entry that carries the tensor's prune / protect fractions)
    if (!c->batch.light) { // (protected counts per tile and sums of squares, as a search with scores leaves them)
        int rr = resolve_all(c);
        if (rr) return rr;
    }
    const uint32_t nT = (uint32_t)c->batch.nT;
    std::vector<SketchDesc> sd(nT);
    for (auto &d : sd) d.active = d.cfg = 0u;
    for (uint32_t k = 0; k < n_sel; k++) {
        uint32_t gi = 0;
        for (gi = 0; gi < c->grid.n_cfg; gi++)
            if (c->grid_cfgs[gi].bits == cfg[k].bits && c->grid_cfgs[gi].prune_ppm == cfg[k].prune_ppm &&
                c->grid_cfgs[gi].outlier_ppm == cfg[k].outlier_ppm)
                break;
        if (gi == c->grid.n_cfg) return INSHR_E_SHAPE;
        sd[c->pos[which[k]]].active = 1u;
        sd[c->pos[which[k]]].cfg = gi;
    }
    const size_t n_idx = T.tops.size();
    Carver cv;
    const size_t o_cell = cv.take(sizeof(u32) * SK_CELLS);
    const size_t o_tops = cv.take(sizeof(u32) * n_idx);
    const size_t o_rep = cv.take(sizeof(double) * n_idx);
    const size_t o_uni = cv.take(sizeof(double) * 256 * nT);
    const size_t o_sd = cv.take(sizeof(SketchDesc) * nT);
    const size_t upload = cv.off; // everything up to here comes from the host
    const size_t o_hist = cv.take(sizeof(u32) * SK_HIST * nT);
    const size_t o_xq = cv.take(sizeof(double) * SK_HIST * nT);
    const size_t o_wd = cv.take(2 * sizeof(double) * SK_HIST * nT); // (read up to 240 bytes past a row: more follows)
    const size_t n_sets = multi ? SK_SETS : 1;
    const size_t o_key = cv.take(sizeof(u32) * 256 * n_sets * nT);
    const size_t o_cb = cv.take(sizeof(float) * 256 * n_sets * nT);
    const size_t o_sr = cv.take(sizeof(u32) * SK_SETS * nT);
    const size_t o_fk = cv.take(sizeof(u32) * 256 * nT);
    const size_t o_fc = cv.take(sizeof(float) * 256 * nT);
    const size_t o_se = cv.take(sizeof(u32) * SK_SLOTS * nT);
    const size_t o_slot = cv.off; // slot moments, cleared before the scoring sweep
    const size_t o_sc = cv.take(sizeof(u32) * SK_SLOTS * nT);
    const size_t o_sx = cv.take(sizeof(double) * SK_SLOTS * nT);
    const size_t slot_end = cv.off;
    HIPCHK(c, hipStreamSynchronize(c->stream)); // the staging buffer may still be in use (inshr_delta)
    int rc = ensure_dev(c, c->sketch_mem, cv.off);
    if (rc) return rc;
    rc = ensure_host(c, c->h_up, upload);
    if (rc) return rc;
    rc = ensure_host(c, c->h_down, (sizeof(SketchInfo) + sizeof(SketchChoice)) * nT);
    if (rc) return rc;
    char *hb = (char *)c->h_up.p, *db = (char *)c->sketch_mem.p;
    memcpy(hb + o_cell, T.cell.data(), sizeof(u32) * SK_CELLS);
    memcpy(hb + o_tops, T.tops.data(), sizeof(u32) * n_idx);
    memcpy(hb + o_rep, T.rep.data(), sizeof(double) * n_idx);
    memset(hb + o_uni, 0, sizeof(double) * 256 * nT);
    for (uint32_t k = 0; k < n_sel; k++)
        memcpy(hb + o_uni + sizeof(double) * 256 * c->pos[which[k]], params->uniforms + (size_t)src[k] * 256,
               sizeof(double) * 256);
    memcpy(hb + o_sd, sd.data(), sizeof(SketchDesc) * nT);
    Stage up;
    up.add(db, hb, upload);
    up.zero(db + o_hist, sizeof(u32) * SK_HIST * nT);
    if (multi) up.zero(db + o_slot, slot_end - o_slot);
    HIPCHK(c, launch_stage(up, c->n_cu, c->stream));
    // (results of a few bytes per tensor: the kernels store them to the host)
    SketchChoice *const hch = (SketchChoice *)c->h_down.p;
    SketchInfo *const hinfo = (SketchInfo *)(hch + nT);
    SketchParams P;
    P.sigma = params->sigma;
    P.max_iter = params->max_iter;
    P.n_idx = (u32)n_idx;
    P.cell = (const u32 *)(db + o_cell);
    P.tops = (const u32 *)(db + o_tops);
    P.rep = (const double *)(db + o_rep);
    P.uniforms = (const double *)(db + o_uni);
    P.hist = (u32 *)(db + o_hist);
    P.xq = (double *)(db + o_xq);
    P.wd = (double *)(db + o_wd);
    P.alt_key = (u32 *)(db + o_key);
    P.alt_cb = (float *)(db + o_cb);
    P.info = hinfo;
    P.multi = multi ? 1u : 0u;
    P.light = c->batch.light ? 1u : 0u;
    P.eps = eps;
    P.set_rounds = (u32 *)(db + o_sr);
    P.slot_cnt = (u32 *)(db + o_sc);
    P.slot_sx = (double *)(db + o_sx);
    P.slot_edge = (u32 *)(db + o_se);
    P.choice = hch;
    P.final_key = (u32 *)(db + o_fk);
    P.final_cb = (float *)(db + o_fc);
    HIPCHK(c, launch_sketch(c->batch, (const SketchDesc *)(db + o_sd), P, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    if (info) {
        for (uint32_t k = 0; k < n_sel; k++) {
            info[src[k]].n_buckets = hinfo[c->pos[which[k]]].n_buckets;
            info[src[k]].rounds = hinfo[c->pos[which[k]]].rounds;
        }
    }
    if (multi && choice) {
        for (uint32_t k = 0; k < n_sel; k++) {
            const SketchChoice &r = hch[c->pos[which[k]]];
            inshr_sketch_choice &o = choice[src[k]];
            for (int b = 0; b < SK_SETS; b++) {
                o.sse[b] = r.sse[b];
                o.rounds[b] = r.rounds[b];
            }
            o.sumsq = r.sumsq;
            o.best_bits = r.best_bits;
            o.feasible = r.feasible;
        }
    }
    *alt_key = multi ? P.final_key : P.alt_key;
    *alt_cb = multi ? P.final_cb : P.alt_cb;
    return INSHR_OK;
}

} // namespace

int inshr_quantize_sketch(inshr_ctx *c, const inshr_tensor *tensors, const inshr_config *cfg,
                          const inshr_sketch_params *params, inshr_quantized *out,
                          inshr_sketch_info *info, uint32_t n_tensors, uint32_t flags)
{
    if (!c || !tensors || !cfg || !params || !out || n_tensors == 0 || !params->uniforms) return INSHR_E_ARG;
    if (!(params->sigma >= 0.0 && params->sigma <= 1.0)) return INSHR_E_CONFIG;
    for (uint32_t t = 0; t < n_tensors; t++) {
        int rc = check_config(cfg[t]);
        if (rc) return rc;
        if (cfg[t].bins) return INSHR_E_CONFIG; // the clustered bins come in powers of two, by bits
        for (int r = 0; r < (1 << cfg[t].bits); r++) {
            const double u = params->uniforms[(size_t)t * 256 + r];
            if (!(u >= 0.0 && u < 1.0)) return INSHR_E_ARG;
        }
    }
    SketchTables T;
    int rc = build_sketch_tables(c, params->alpha, T);
    if (rc) return rc;
    HIPCHK(c, hipSetDevice(c->device));
    const u32 *alt_key = nullptr;
    const float *alt_cb = nullptr;
    if (flags & INSHR_REUSE_SEARCH) {
        if (!c->have_search || c->tensors.size() != n_tensors) return INSHR_E_SHAPE;
        std::vector<uint32_t> which(n_tensors);
        for (uint32_t t = 0; t < n_tensors; t++) {
            if (c->tensors[t].data != tensors[t].data || c->tensors[t].n != tensors[t].n) return INSHR_E_SHAPE;
            which[t] = t;
        }
        rc = sketch_with_state(c, cfg, which.data(), which.data(), n_tensors, params, T, info, &alt_key, &alt_cb);
        if (rc) return rc;
        return quantize_with_state(c, cfg, out, which.data(), n_tensors, alt_key, alt_cb);
    }
    // stand-alone: one single-configuration search per distinct configuration gives the thresholds
    std::vector<char> done(n_tensors, 0);
    for (uint32_t t0 = 0; t0 < n_tensors; t0++) {
        if (done[t0]) continue;
        std::vector<inshr_tensor> sub;
        std::vector<inshr_config> subcfg;
        std::vector<uint32_t> idx;
        for (uint32_t t = t0; t < n_tensors; t++) {
            if (!done[t] && cfg[t].bits == cfg[t0].bits && cfg[t].prune_ppm == cfg[t0].prune_ppm &&
                cfg[t].outlier_ppm == cfg[t0].outlier_ppm) {
                done[t] = 1;
                sub.push_back(tensors[t]);
                subcfg.push_back(cfg[t]);
                idx.push_back(t);
            }
        }
        const uint32_t nS = (uint32_t)sub.size();
        rc = run_search(c, sub.data(), nS, &cfg[t0], 1, 0.0, LIGHT);
        if (rc) return rc;
        std::vector<inshr_quantized> subout(nS);
        std::vector<uint32_t> which(nS);
        for (uint32_t k = 0; k < nS; k++) {
            subout[k] = out[idx[k]];
            which[k] = k;
        }
        rc = sketch_with_state(c, subcfg.data(), which.data(), idx.data(), nS, params, T, info, &alt_key, &alt_cb);
        if (rc) return rc;
        rc = quantize_with_state(c, subcfg.data(), subout.data(), which.data(), nS, alt_key, alt_cb);
        for (uint32_t k = 0; k < nS; k++) out[idx[k]] = subout[k];
        if (rc) return rc;
    }
    return INSHR_OK;
}

int inshr_search_sketch(inshr_ctx *c, const inshr_tensor *tensors, const inshr_config *cfg,
                        const inshr_sketch_params *params, double eps, inshr_quantized *out,
                        inshr_sketch_choice *choice, inshr_sketch_info *info, uint32_t n_tensors,
                        uint32_t flags)
{
    if (!c || !tensors || !cfg || !params || !out || !choice || n_tensors == 0 || !params->uniforms)
        return INSHR_E_ARG;
    if (!(params->sigma >= 0.0 && params->sigma <= 1.0) || !(eps >= 0.0)) return INSHR_E_CONFIG;
    std::vector<inshr_config> wide(n_tensors); // the tensor's fractions with 8 bits
    for (uint32_t t = 0; t < n_tensors; t++) {
        if (cfg[t].bins) return INSHR_E_CONFIG;
        wide[t] = cfg[t];
        wide[t].bits = 8;
        int rc = check_config(wide[t]);
        if (rc) return rc;
        for (int r = 0; r < 256; r++) {
            const double u = params->uniforms[(size_t)t * 256 + r];
            if (!(u >= 0.0 && u < 1.0)) return INSHR_E_ARG;
        }
    }
    SketchTables T;
    int rc = build_sketch_tables(c, params->alpha, T);
    if (rc) return rc;
    HIPCHK(c, hipSetDevice(c->device));
    const u32 *alt_key = nullptr;
    const float *alt_cb = nullptr;
    auto finish = [&](const inshr_config *sub_wide, inshr_quantized *sub_out, const uint32_t *which,
                      const uint32_t *src, uint32_t n) -> int {
        int r = sketch_with_state(c, sub_wide, which, src, n, params, T, info, &alt_key, &alt_cb, true, eps, choice);
        if (r) return r;
        std::vector<inshr_config> chosen(n);
        for (uint32_t k = 0; k < n; k++) {
            chosen[k] = sub_wide[k];
            chosen[k].bits = (uint8_t)choice[src[k]].best_bits;
        }
        return quantize_with_state(c, chosen.data(), sub_out, which, n, alt_key, alt_cb);
    };
    if (flags & INSHR_REUSE_SEARCH) {
        if (!c->have_search || c->tensors.size() != n_tensors) return INSHR_E_SHAPE;
        std::vector<uint32_t> which(n_tensors);
        for (uint32_t t = 0; t < n_tensors; t++) {
            if (c->tensors[t].data != tensors[t].data || c->tensors[t].n != tensors[t].n) return INSHR_E_SHAPE;
            which[t] = t;
        }
        return finish(wide.data(), out, which.data(), which.data(), n_tensors);
    }
    // stand-alone: one search over 2 .. 8 bits per distinct pair of fractions gives the thresholds
    std::vector<char> done(n_tensors, 0);
    for (uint32_t t0 = 0; t0 < n_tensors; t0++) {
        if (done[t0]) continue;
        std::vector<inshr_tensor> sub;
        std::vector<inshr_config> subcfg;
        std::vector<uint32_t> idx;
        for (uint32_t t = t0; t < n_tensors; t++) {
            if (!done[t] && cfg[t].prune_ppm == cfg[t0].prune_ppm && cfg[t].outlier_ppm == cfg[t0].outlier_ppm) {
                done[t] = 1;
                sub.push_back(tensors[t]);
                subcfg.push_back(wide[t]);
                idx.push_back(t);
            }
        }
        const uint32_t nS = (uint32_t)sub.size();
        inshr_config grid7[SK_SETS];
        for (int b = 0; b < SK_SETS; b++) {
            grid7[b] = wide[t0];
            grid7[b].bits = (uint8_t)(2 + b);
        }
        rc = run_search(c, sub.data(), nS, grid7, SK_SETS, eps, LIGHT);
        if (rc) return rc;
        std::vector<inshr_quantized> subout(nS);
        std::vector<uint32_t> which(nS);
        for (uint32_t k = 0; k < nS; k++) {
            subout[k] = out[idx[k]];
            which[k] = k;
        }
        rc = finish(subcfg.data(), subout.data(), which.data(), idx.data(), nS);
        for (uint32_t k = 0; k < nS; k++) out[idx[k]] = subout[k];
        if (rc) return rc;
    }
    return INSHR_OK;
}

int inshr_search_sketch_grid(inshr_ctx *c, const inshr_tensor *tensors, const inshr_config *pairs,
                             uint32_t n_pairs, const inshr_sketch_params *params, double eps,
                             inshr_quantized *out, uint32_t *best_pair, inshr_sketch_choice *choice,
                             inshr_sketch_choice *table, uint32_t n_tensors)
{
    if (!c || !tensors || !pairs || !params || !out || !best_pair || !choice || n_tensors == 0 || n_pairs == 0)
        return INSHR_E_ARG;
    const uint32_t nT = n_tensors;
    std::vector<inshr_config> cfg(nT);
    std::vector<inshr_sketch_choice> ch(nT);
    std::vector<inshr_quantized> tmp(nT);
    struct Best {
        bool any = false, feasible = false;
        uint64_t cost = 0;
        double sse8 = 0.0;
        uint32_t pair = 0;
    };
    std::vector<Best> best(nT);
    // every pair in turn: all widths of the pair scored for all tensors (the outputs are scratch here)
    for (uint32_t q = 0; q < n_pairs; q++) {
        for (uint32_t t = 0; t < nT; t++) {
            cfg[t] = pairs[q];
            cfg[t].bits = 8;
            cfg[t].bins = 0;
            tmp[t] = out[t];
        }
        int rc = inshr_search_sketch(c, tensors, cfg.data(), params, eps, tmp.data(), ch.data(), nullptr, nT, 0);
        if (rc) return rc;
        for (uint32_t t = 0; t < nT; t++) {
            if (table) table[(size_t)t * n_pairs + q] = ch[t];
            Best &b = best[t];
            if (ch[t].feasible) {
                const uint32_t bits = ch[t].best_bits; // the fewest feasible bits of a pair are its cheapest
                const uint64_t cost = tmp[t].n_kept * bits + 32ull * tmp[t].n_outlier + (32ull << bits);
                if (!b.feasible || cost < b.cost) {
                    b.feasible = true;
                    b.cost = cost;
                    b.pair = q;
                }
            } else if (!b.feasible && (!b.any || ch[t].sse[6] < b.sse8)) {
                b.sse8 = ch[t].sse[6];
                b.pair = q;
            }
            b.any = true;
        }
    }
    // the winners once more, pair by pair, into the caller's buffers (same uniforms: same result)
    std::vector<char> done(nT, 0);
    for (uint32_t t0 = 0; t0 < nT; t0++) {
        if (done[t0]) continue;
        std::vector<inshr_tensor> sub;
        std::vector<inshr_config> subcfg;
        std::vector<inshr_quantized> subout;
        std::vector<uint32_t> idx;
        std::vector<double> uni;
        for (uint32_t t = t0; t < nT; t++) {
            if (!done[t] && best[t].pair == best[t0].pair) {
                done[t] = 1;
                sub.push_back(tensors[t]);
                inshr_config k = pairs[best[t].pair];
                k.bits = 8;
                k.bins = 0;
                subcfg.push_back(k);
                subout.push_back(out[t]);
                idx.push_back(t);
                uni.insert(uni.end(), params->uniforms + (size_t)t * 256, params->uniforms + (size_t)t * 256 + 256);
            }
        }
        inshr_sketch_params p2 = *params;
        p2.uniforms = uni.data();
        std::vector<inshr_sketch_choice> ch2(sub.size());
        int rc = inshr_search_sketch(c, sub.data(), subcfg.data(), &p2, eps, subout.data(), ch2.data(), nullptr,
                                     (uint32_t)sub.size(), 0);
        if (rc) return rc;
        for (size_t k = 0; k < sub.size(); k++) {
            out[idx[k]] = subout[k];
            choice[idx[k]] = ch2[k];
            best_pair[idx[k]] = best[idx[k]].pair;
        }
    }
    return INSHR_OK;
}

int inshr_sketch_buckets(double alpha, int32_t *i_lo, uint32_t *n_buckets, float *tops, double *values,
                         uint32_t cap)
{
    if (!i_lo || !n_buckets) return INSHR_E_ARG;
    SketchTables T;
    int rc = build_sketch_tables(nullptr, alpha, T);
    if (rc) return rc;
    *i_lo = T.i_lo;
    *n_buckets = (uint32_t)T.tops.size();
    if (cap < T.tops.size() && (tops || values)) return INSHR_E_CAPACITY;
    for (size_t b = 0; b < T.tops.size(); b++) {
        if (tops) memcpy(&tops[b], &T.tops[b], 4);
        if (values) values[b] = T.rep[b];
    }
    return INSHR_OK;
}

int inshr_sketch_quantiles(inshr_ctx *c, const inshr_tensor *tensors, uint32_t n_tensors, const double *q,
                           uint32_t n_q, double alpha, double *estimates)
{
    if (!c || !tensors || !q || !estimates || n_tensors == 0 || n_q == 0 || n_q > 4096u) return INSHR_E_ARG;
    SketchTables T;
    int rc = build_sketch_tables(c, alpha, T);
    if (rc) return rc;
    const uint32_t nT = n_tensors;
    const size_t n_idx = T.tops.size();
    std::vector<MagDesc> md(nT);
    std::vector<u64> ranks((size_t)nT * n_q);
    u64 chunks = 0;
    for (uint32_t t = 0; t < nT; t++) {
        if (!tensors[t].data || tensors[t].n == 0 || tensors[t].n >= (1ull << 32)) return INSHR_E_ARG;
        if ((uintptr_t)tensors[t].data & 3u) return INSHR_E_ARG;
        md[t].x = tensors[t].data;
        md[t].n = tensors[t].n;
        md[t].chunk0 = chunks;
        chunks += (tensors[t].n + SK_MAG_CHUNK - 1) / SK_MAG_CHUNK;
        for (uint32_t k = 0; k < n_q; k++) {
            if (!(q[k] >= 0.0 && q[k] <= 1.0)) return INSHR_E_ARG;
            ranks[(size_t)t * n_q + k] = (u64)floor(q[k] * (double)(tensors[t].n - 1)); // rank floor(q (n - 1))
        }
    }
    HIPCHK(c, hipSetDevice(c->device));
    Carver cv;
    const size_t o_cell = cv.take(sizeof(u32) * SK_CELLS);
    const size_t o_tops = cv.take(sizeof(u32) * n_idx);
    const size_t o_rep = cv.take(sizeof(double) * n_idx);
    const size_t o_md = cv.take(sizeof(MagDesc) * nT);
    const size_t o_rk = cv.take(sizeof(u64) * ranks.size());
    const size_t upload = cv.off;
    const size_t o_hist = cv.take(sizeof(u32) * SK_MAG_HIST * nT);
    const size_t o_nf = cv.take(256);
    const size_t zero_end = cv.off;
    const size_t o_est = cv.take(sizeof(double) * ranks.size());
    HIPCHK(c, hipStreamSynchronize(c->stream)); // the staging buffer may still be in use (inshr_delta)
    rc = ensure_dev(c, c->sketch_mem, cv.off);
    if (rc) return rc;
    rc = ensure_host(c, c->h_up, upload);
    if (rc) return rc;
    rc = ensure_host(c, c->h_down, sizeof(double) * ranks.size() + 256);
    if (rc) return rc;
    char *hb = (char *)c->h_up.p, *db = (char *)c->sketch_mem.p;
    memcpy(hb + o_cell, T.cell.data(), sizeof(u32) * SK_CELLS);
    memcpy(hb + o_tops, T.tops.data(), sizeof(u32) * n_idx);
    memcpy(hb + o_rep, T.rep.data(), sizeof(double) * n_idx);
    memcpy(hb + o_md, md.data(), sizeof(MagDesc) * nT);
    memcpy(hb + o_rk, ranks.data(), sizeof(u64) * ranks.size());
    HIPCHK(c, hipMemcpyAsync(db, hb, upload, hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipMemsetAsync(db + o_hist, 0, zero_end - o_hist, c->stream));
    HIPCHK(c, launch_sketch_quantiles((const MagDesc *)(db + o_md), (int)nT, chunks, c->n_cu, (const u32 *)(db + o_cell),
                                      (const u32 *)(db + o_tops), (const double *)(db + o_rep), (u32)n_idx,
                                      (u32 *)(db + o_hist), (u32 *)(db + o_nf), (const u64 *)(db + o_rk), n_q,
                                      (double *)(db + o_est), c->stream));
    HIPCHK(c, hipMemcpyAsync(c->h_down.p, db + o_est, sizeof(double) * ranks.size(), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipMemcpyAsync((char *)c->h_down.p + sizeof(double) * ranks.size(), db + o_nf, 4,
                             hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    u32 nf = 0;
    memcpy(&nf, (const char *)c->h_down.p + sizeof(double) * ranks.size(), 4);
    if (nf) return INSHR_E_NONFINITE;
    memcpy(estimates, c->h_down.p, sizeof(double) * ranks.size());
    return INSHR_OK;
}

// number of bins of a symbol stream; nonzero return: not a valid description
static int codes_bins(const inshr_codes &c, uint32_t &K)
{
    if (c.bins) {
        if (c.bins < 2 || c.bins > 256) return 1;
        K = c.bins;
    } else {
        if (c.bits < 1 || c.bits > 8) return 1;
        K = 1u << c.bits;
    }
    return 0;
}

int inshr_quantize_sens(inshr_ctx *c, const inshr_tensor *tensors, const float *const *grads,
                        const inshr_config *cfg, const uint8_t *prune_by_sensitivity,
                        inshr_quantized *out, inshr_sens_info *info, uint32_t n_tensors)
{
    if (!c || !tensors || !grads || !cfg || !out || n_tensors == 0 || n_tensors > 65535u) return INSHR_E_ARG;
    const uint32_t nT = n_tensors;
    c->have_search = false;
    // the distinct configurations: their fractions for the two threshold searches, their numbers
    // of bins for the search over the quantized values
    std::vector<inshr_config> frac_grid, bin_grid;
    std::vector<uint32_t> frac_of(nT), bin_of_t(nT);
    u64 n_total = 0, n_runs = 0;
    for (uint32_t t = 0; t < nT; t++) {
        int rc = check_config(cfg[t]);
        if (rc) return rc;
        if (!tensors[t].data || !grads[t] || tensors[t].n == 0 || tensors[t].n >= (1ull << 32)) return INSHR_E_ARG;
        if (((uintptr_t)tensors[t].data | (uintptr_t)grads[t]) & 3u) return INSHR_E_ARG;
        if (!out[t].packed || !out[t].codebook) return INSHR_E_ARG;
        if (out[t].outlier_cap && (!out[t].outlier_idx || !out[t].outlier_val)) return INSHR_E_ARG;
        if (out[t].packed_words < (tensors[t].n * (u64)symbol_bits(bins_of(cfg[t])) + 63) / 64) return INSHR_E_CAPACITY;
        inshr_config f = cfg[t], b = cfg[t];
        f.bits = 1;
        f.bins = 0;
        b.prune_ppm = b.outlier_ppm = 0;
        size_t i;
        for (i = 0; i < frac_grid.size(); i++)
            if (same_config(frac_grid[i], f)) break;
        if (i == frac_grid.size()) frac_grid.push_back(f);
        frac_of[t] = (uint32_t)i;
        for (i = 0; i < bin_grid.size(); i++)
            if (same_config(bin_grid[i], b)) break;
        if (i == bin_grid.size()) bin_grid.push_back(b);
        bin_of_t[t] = (uint32_t)i;
        n_total += tensors[t].n;
        n_runs += (tensors[t].n + SENS_RUN - 1) / SENS_RUN;
    }
    if (n_runs >= (1ull << 31)) return INSHR_E_ARG; // (2^45 values)
    HIPCHK(c, hipSetDevice(c->device));
    Carver cv;
    const size_t o_sd = cv.take(sizeof(SDesc) * nT);
    const size_t o_st = cv.take(n_runs * 8 + 256); // [ticket, pad to 256 bytes; states of the runs]: cleared
    const size_t o_bp = cv.take(n_runs * 4);
    const size_t o_bq = cv.take(n_runs * 16);
    const size_t o_S = cv.take(n_total * 4 + 64ull * nT);
    const size_t o_W = cv.take(n_total * 4 + 64ull * nT);
    int rc = ensure_dev(c, c->sens_mem, cv.off);
    if (rc) return rc;
    char *db = (char *)c->sens_mem.p;
    std::vector<SDesc> sd(nT);
    {
        u64 run = 0, off = 0;
        for (uint32_t t = 0; t < nT; t++) {
            memset(&sd[t], 0, sizeof(SDesc));
            sd[t].w = tensors[t].data;
            sd[t].g = grads[t];
            sd[t].n = tensors[t].n;
            sd[t].run0 = (u32)run;
            sd[t].S = (float *)(db + o_S) + off;
            sd[t].Wm = (float *)(db + o_W) + off;
            sd[t].by_sens = (prune_by_sensitivity && prune_by_sensitivity[t]) ? 1u : 0u;
            run += (tensors[t].n + SENS_RUN - 1) / SENS_RUN;
            off += (tensors[t].n + 15) / 16 * 16; // every tensor's scratch starts 64-byte aligned
        }
    }
    auto upload = [&](size_t clear) -> int { // the descriptors; bytes at o_st to clear
        HIPCHK(c, hipStreamSynchronize(c->stream)); // the staging buffer may still be in flight
        const int ru = ensure_host(c, c->h_up, sizeof(SDesc) * nT);
        if (ru) return ru;
        memcpy(c->h_up.p, sd.data(), sizeof(SDesc) * nT);
        Stage up;
        up.add(db + o_sd, c->h_up.p, sizeof(SDesc) * nT);
        up.zero(db + o_st, clear);
        HIPCHK(c, launch_stage(up, c->n_cu, c->stream));
        return INSHR_OK;
    };
    if ((rc = upload(0))) return rc;
    HIPCHK(c, launch_sens_score((const SDesc *)(db + o_sd), (int)nT, (u32)n_runs, c->stream));

    // thresholds: order statistics of the scores and of the weights (threshold searches only), in one
    // search where the scratch memory allows it
    std::vector<inshr_tensor> sub(2 * (size_t)nT);
    for (uint32_t t = 0; t < nT; t++) {
        sub[t].data = sd[t].S;
        sub[nT + t].data = tensors[t].data;
        sub[t].n = sub[nT + t].n = tensors[t].n;
    }
    auto thresholds = [&](uint32_t from, uint32_t to) -> int {
        const int rs = run_search(c, sub.data() + from, to - from, frac_grid.data(), (uint32_t)frac_grid.size(), 0.0,
                                  LIGHT);
        if (rs) return rs;
        const SearchResult *res = (const SearchResult *)c->h_res.p;
        for (uint32_t k = from; k < to; k++) {
            const uint32_t t = k % nT;
            uint32_t qp = 0, qo = 0;
            while (qp < c->grid.n_p && c->grid.p_ppm[qp] != cfg[t].prune_ppm) qp++;
            while (qo < c->grid.n_o && c->grid.o_ppm[qo] != cfg[t].outlier_ppm) qo++;
            if (qp == c->grid.n_p || qo == c->grid.n_o) return INSHR_E_INTERNAL;
            const u32 *thr = res[c->pos[k - from]].thr_mag;
            (k < nT ? sd[t].tau_os : sd[t].tau_om) = thr[c->grid.n_p + qo];
            if ((k < nT) == (sd[t].by_sens != 0u)) sd[t].tau_p = thr[qp];
        }
        return INSHR_OK;
    };
    rc = nT < 32768u ? thresholds(0, 2 * nT) : INSHR_E_CAPACITY;
    if (rc == INSHR_E_CAPACITY) {
        rc = thresholds(0, nT);
        if (!rc) rc = thresholds(nT, 2 * nT);
    }
    if (rc) return rc;
    sub.resize(nT);
    c->have_search = false;
    if ((rc = upload(n_runs * 8 + 256))) return rc;
    rc = ensure_host(c, c->h_down, sizeof(SInfo) * nT);
    if (rc) return rc;
    HIPCHK(c, launch_sens_partition((const SDesc *)(db + o_sd), (int)nT, (u32)n_runs, (u32 *)(db + o_st),
                                    (u64 *)(db + o_st + 256), (u32 *)(db + o_bp), (double *)(db + o_bq),
                                    (SInfo *)c->h_down.p, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    const std::vector<SInfo> si((const SInfo *)c->h_down.p, (const SInfo *)c->h_down.p + nT);
    for (uint32_t t = 0; t < nT; t++) {
        if (si[t].n_kept == 0) {
            c->last_err = "the thresholds leave tensor " + std::to_string(t) + " without quantized values";
            return INSHR_E_CONFIG;
        }
        if (si[t].n_outlier > out[t].outlier_cap) return INSHR_E_CAPACITY;
        sub[t].data = sd[t].Wm;
        sub[t].n = si[t].n_kept;
    }
    // the bins: the quantized values as tensors of their own, nothing pruned, nothing protected
    // (every tensor's own number of bins is all that is scored)
    do {
        rc = run_search(c, sub.data(), nT, bin_grid.data(), (uint32_t)bin_grid.size(), 0.0, GIVEN);
        if (rc) return rc;
        c->have_search = false; // (the state describes the compacted values, not the caller's tensors)
        rc = score_given(c, bin_of_t);
        if (rc < 0) return rc;
    } while (rc == 1); // larger pools
    const Score *hsc = (const Score *)c->h_down.p;
    const uint32_t n_bg = (uint32_t)bin_grid.size();
    std::vector<double> sse_q(nT), sq_q(nT);
    for (uint32_t t = 0; t < nT; t++) {
        const uint32_t gi = bin_of_t[t];
        const u32 p = c->pos[t];
        sse_q[t] = hsc[(size_t)p * n_bg + gi].sse;
        sq_q[t] = hsc[(size_t)p * n_bg + gi].sumsq;
        sd[t].packed = (unsigned long long *)out[t].packed;
        sd[t].out_idx = out[t].outlier_idx;
        sd[t].out_val = out[t].outlier_val;
        sd[t].out_cap = out[t].outlier_cap;
        sd[t].codebook = out[t].codebook;
        sd[t].boundaries = out[t].boundaries;
        sd[t].bkeys = c->batch.bufs.tgt_key + (size_t)p * TGT_STRIDE; // (one pair: nothing pruned or protected)
        sd[t].cb = c->batch.bufs.codebook + ((size_t)p * n_bg + gi) * CB_STRIDE;
        sd[t].K = bins_of(cfg[t]);
        sd[t].sym_bits = symbol_bits(sd[t].K);
    }
    if ((rc = upload(0))) return rc;
    u32 *const flags = call_flags(c);
    HIPCHK(c, launch_sens_quant((const SDesc *)(db + o_sd), (int)nT, (u32)n_runs, (const u32 *)(db + o_bp), flags,
                                c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    if (raised_flags(flags) & 2u) return INSHR_E_CAPACITY;
    for (uint32_t t = 0; t < nT; t++) {
        out[t].n_pruned = si[t].n_pruned;
        out[t].n_outlier = si[t].n_outlier;
        out[t].n_kept = si[t].n_kept;
        out[t].n_bins = sd[t].K;
        out[t].sym_bits = sd[t].sym_bits;
        memcpy(&out[t].tau_prune, &sd[t].tau_p, 4);
        memcpy(&out[t].tau_outlier, &sd[t].tau_om, 4);
        if (info) {
            memcpy(&info[t].tau_outlier_sens, &sd[t].tau_os, 4);
            info[t].sse = sse_q[t] + si[t].sq_pruned;
            info[t].sumsq = sq_q[t] + si[t].sq_pruned + si[t].sq_prot;
        }
    }
    return INSHR_OK;
}

int inshr_delta_bound(const inshr_codes *prev, const inshr_codes *cur, uint64_t *packed_words)
{
    if (!prev || !cur || !packed_words) return INSHR_E_ARG;
    if (prev->n != cur->n) return INSHR_E_SHAPE;
    uint32_t Kp = 0, Kc = 0;
    if (codes_bins(*prev, Kp) || codes_bins(*cur, Kc)) return INSHR_E_CONFIG;
    const uint32_t wB = symbol_bits(std::max(Kp, Kc));
    *packed_words = (prev->n * (uint64_t)wB + 63) / 64;
    return INSHR_OK;
}

// Tiles per chunk of a call; longer chunks where the counts of so many would not fit the scratch limit.
static u32 call_chunk_tiles(const inshr_ctx *c, const inshr_codes *prev, uint32_t n_tensors)
{
    u64 tiles = 0; // (sizes are checked by the caller)
    for (uint32_t t = 0; t < n_tensors; t++) tiles += (prev[t].n + DELTA_TILE - 1) / DELTA_TILE;
    u32 ct = delta_chunk_tiles(tiles, c->n_cu);
    if (!c->scratch_limit) return ct;
    auto scratch = [&] { // of a reconstruct call, which takes the most
        u64 chunks = 0;
        for (uint32_t t = 0; t < n_tensors; t++) chunks += ((prev[t].n + DELTA_TILE - 1) / DELTA_TILE + ct - 1) / ct;
        return (sizeof(DDesc) + sizeof(XDesc) + sizeof(u64) * (DELTA_SS + 8)) * n_tensors +
               chunks * 4 * (1 + DELTA_SS) + 6 * 256;
    };
    while (ct < (u32)DELTA_CHUNK && scratch() > c->scratch_limit) ct = std::min(2 * ct, (u32)DELTA_CHUNK);
    return ct;
}

// The parts of a call's tensors: where their symbol populations are added up and, behind those, the tensor of every
// part.  None where no tensor has enough chunks for them to be added up; every tensor is one part then.
struct Parts {
    std::vector<u32> tensor;
    bool many = false;
    void enter(DDesc &d, u32 t)
    {
        d.part0 = (u32)tensor.size();
        tensor.insert(tensor.end(), delta_parts(d.n_chunks), t);
        many = many || d.n_chunks > DELTA_FEW;
    }
    size_t sums() const { return many ? sizeof(u32) * DELTA_SS * tensor.size() : 0; }
    size_t bytes() const { return many ? sums() + sizeof(u32) * tensor.size() : 0; }
};
// They lie at offset o of aux_mem, or in an allocation of its own where the caller limits the size of one (a call that
// fitted the limit without them still does: aux_mem holds as much for every chunk, and there are no more parts than
// chunks).  The tensors' numbers are staged at offset at of h_up.
static int place_parts(inshr_ctx *c, const Parts &parts, size_t o, size_t at, DeltaCall &call, Stage &st)
{
    call.totals = nullptr;
    call.part_tensor = nullptr;
    call.n_parts = parts.tensor.size();
    if (!parts.many) return INSHR_OK;
    if (c->scratch_limit) {
        const int rc = ensure_dev(c, c->totals_mem, (parts.bytes() + 255) & ~(size_t)255);
        if (rc) return rc;
    }
    char *p = c->scratch_limit ? (char *)c->totals_mem.p : (char *)c->aux_mem.p + o;
    call.totals = (u32 *)p;
    st.zero(p, parts.sums());
    memcpy((char *)c->h_up.p + at, parts.tensor.data(), sizeof(u32) * parts.tensor.size());
    call.part_tensor = (const u32 *)(p + parts.sums());
    st.add(p + parts.sums(), (char *)c->h_up.p + at, sizeof(u32) * parts.tensor.size());
    return INSHR_OK;
}

int inshr_delta(inshr_ctx *c, const inshr_codes *prev, const uint32_t *const *prev_perm,
                const inshr_codes *cur, inshr_delta_out *out, uint32_t n_tensors)
{
    if (!c || !prev || !cur || !out || n_tensors == 0) return INSHR_E_ARG;
    std::vector<DDesc> dd(n_tensors);
    std::vector<u32> chunk_tensor;
    Parts parts;
    u64 chunk = 0;
    const u32 ctiles = call_chunk_tiles(c, prev, n_tensors);
    bool any_scatter = false, any_gather = false, any_perm = false, any_long = false;
    for (uint32_t t = 0; t < n_tensors; t++) {
        uint64_t words = 0;
        int rc = inshr_delta_bound(&prev[t], &cur[t], &words);
        if (rc) return rc;
        const uint64_t n = prev[t].n;
        if (n == 0 || n >= (1ull << 32) || !prev[t].packed || !cur[t].packed) return INSHR_E_ARG;
        uint32_t Kp = 0, Kc = 0;
        (void)codes_bins(prev[t], Kp); // (checked by inshr_delta_bound)
        (void)codes_bins(cur[t], Kc);
        if (prev[t].sym_bits != symbol_bits(Kp) || cur[t].sym_bits != symbol_bits(Kc)) return INSHR_E_CONFIG;
        if (!out[t].packed || !out[t].group_off || out[t].packed_words < words) return INSHR_E_CAPACITY;
        if (out[t].group_off_entries && out[t].group_off_entries < Kp + 3u) return INSHR_E_CAPACITY;
        if (prev_perm && prev_perm[t] && out[t].perm) return INSHR_E_ARG; // a given permutation is not written again
        DDesc &d = dd[t];
        memset(&d, 0, sizeof(d));
        d.prev = (const unsigned long long *)prev[t].packed;
        d.cur = (const unsigned long long *)cur[t].packed;
        d.out = (unsigned long long *)out[t].packed;
        d.group_off = out[t].group_off;
        d.perm = out[t].perm;
        d.prev_perm = prev_perm ? prev_perm[t] : nullptr;
        d.n = n;
        d.out_words = words;
        d.wp = prev[t].sym_bits;
        d.wc = cur[t].sym_bits;
        d.Kp = Kp;
        d.B = std::max(Kp, Kc) + 2u;
        d.wB = symbol_bits(std::max(Kp, Kc));
        out[t].delta_bits = d.wB;
        d.chunk0 = chunk;
        const u64 nt = (n + DELTA_TILE - 1) / DELTA_TILE;
        d.n_chunks = (nt + ctiles - 1) / ctiles;
        d.ctiles = ctiles;
        for (u64 k = 0; k < d.n_chunks; k++) chunk_tensor.push_back(t);
        parts.enter(d, t);
        any_long = any_long || !delta_single(d);
        chunk += d.n_chunks;
        if (d.prev_perm)
            any_gather = true;
        else if (d.perm)
            any_perm = true;
        else
            any_scatter = true;
    }
    HIPCHK(c, hipSetDevice(c->device));
    Carver cv;
    const size_t o_dd = cv.take(sizeof(DDesc) * n_tensors);
    const size_t o_ct = cv.take(sizeof(u32) * chunk_tensor.size());
    const size_t up_bytes = cv.off;
    const size_t o_tt = cv.take(c->scratch_limit ? 0 : parts.bytes());
    const size_t o_ck = cv.take((size_t)chunk * DELTA_SS * 4);
    // the staging buffer and the scratch may still be in use by an earlier asynchronous delta call
    HIPCHK(c, hipStreamSynchronize(c->stream));
    int rc = ensure_dev(c, c->aux_mem, cv.off);
    if (rc) return rc;
    rc = ensure_host(c, c->h_up, up_bytes + sizeof(u32) * parts.tensor.size());
    if (rc) return rc;
    rc = take_delta_flags(c); // (of a call whose flags nobody has asked for yet)
    if (rc) return rc;
    char *hb = (char *)c->h_up.p, *db = (char *)c->aux_mem.p;
    memcpy(hb + o_dd, dd.data(), sizeof(DDesc) * n_tensors);
    memcpy(hb + o_ct, chunk_tensor.data(), sizeof(u32) * chunk_tensor.size());
    DeltaCall call;
    Stage up;
    if ((rc = place_parts(c, parts, o_tt, up_bytes, call, up))) return rc;
    up.add(db, hb, up_bytes);
    HIPCHK(c, launch_stage(up, c->n_cu, c->stream));
    memset(c->flags, 0, FLAG_WORDS * sizeof(u32));
    c->delta_pending = true;
    call.dd = (const DDesc *)(db + o_dd);
    call.chunk_tensor = (const u32 *)(db + o_ct);
    call.chunk_tot = (u32 *)(db + o_ck);
    call.flags = c->flags;
    call.n_chunks = chunk;
    call.any_long = any_long;
    call.lds_ordered = c->lds_ordered;
    HIPCHK(c, launch_delta(call, any_scatter, any_perm, any_gather, c->stream));
    return INSHR_OK;
}

int inshr_delta_static(inshr_ctx *c, const inshr_codes *prev, const inshr_codes *cur,
                       inshr_delta_out *out, uint32_t n_tensors)
{
    if (!c || !prev || !cur || !out || n_tensors == 0) return INSHR_E_ARG;
    if (n_tensors > (uint32_t)DELTA_STATIC_MAX_TENSORS) {
        c->last_err = "inshr_delta_static: more than " + std::to_string(DELTA_STATIC_MAX_TENSORS) + " tensors";
        return INSHR_E_CAPACITY;
    }
    DeltaStaticArgs a;
    memset(&a, 0, sizeof(a));
    a.n_tensors = n_tensors;
    u64 chunk = 0;
    u32 ctiles = call_chunk_tiles(c, prev, n_tensors);
    { // (the static scratch holds a fixed number of chunks: longer ones where they would not fit)
        auto chunks_with = [&](u32 ct) {
            u64 k = 0;
            for (uint32_t t = 0; t < n_tensors; t++) k += ((prev[t].n + DELTA_TILE - 1) / DELTA_TILE + ct - 1) / ct;
            return k;
        };
        while (ctiles < (u32)DELTA_CHUNK && chunks_with(ctiles) > (u64)DELTA_STATIC_MAX_CHUNKS) ctiles++;
    }
    bool any_scatter = false, any_perm = false, any_long = false;
    u64 parts = 0;
    for (uint32_t t = 0; t < n_tensors; t++) {
        uint64_t words = 0;
        int rc = inshr_delta_bound(&prev[t], &cur[t], &words);
        if (rc) return rc;
        const uint64_t n = prev[t].n;
        if (n == 0 || n >= (1ull << 32) || !prev[t].packed || !cur[t].packed) return INSHR_E_ARG;
        uint32_t Kp = 0, Kc = 0;
        (void)codes_bins(prev[t], Kp); // (checked by inshr_delta_bound)
        (void)codes_bins(cur[t], Kc);
        if (prev[t].sym_bits != symbol_bits(Kp) || cur[t].sym_bits != symbol_bits(Kc)) return INSHR_E_CONFIG;
        if (!out[t].packed || !out[t].group_off || out[t].packed_words < words) return INSHR_E_CAPACITY;
        if (out[t].group_off_entries && out[t].group_off_entries < Kp + 3u) return INSHR_E_CAPACITY;
        DDesc &d = a.dd[t];
        d.prev = (const unsigned long long *)prev[t].packed;
        d.cur = (const unsigned long long *)cur[t].packed;
        d.out = (unsigned long long *)out[t].packed;
        d.group_off = out[t].group_off;
        d.perm = out[t].perm;
        d.n = n;
        d.out_words = words;
        d.wp = prev[t].sym_bits;
        d.wc = cur[t].sym_bits;
        d.Kp = Kp;
        d.B = std::max(Kp, Kc) + 2u;
        d.wB = symbol_bits(std::max(Kp, Kc));
        out[t].delta_bits = d.wB;
        d.chunk0 = chunk;
        const u64 nt = (n + DELTA_TILE - 1) / DELTA_TILE;
        d.n_chunks = (nt + ctiles - 1) / ctiles;
        d.ctiles = ctiles;
        d.part0 = (u32)parts;
        parts += delta_parts(d.n_chunks);
        any_long = any_long || !delta_single(d);
        chunk += d.n_chunks;
        if (d.perm)
            any_perm = true;
        else
            any_scatter = true;
    }
    if (chunk > (u64)DELTA_STATIC_MAX_CHUNKS) {
        c->last_err = "inshr_delta_static: the tensors need " + std::to_string(chunk) + " chunks of " +
                      std::to_string((u64)DELTA_TILE * DELTA_CHUNK) + " elements, the static scratch holds " +
                      std::to_string(DELTA_STATIC_MAX_CHUNKS);
        return INSHR_E_CAPACITY;
    }
    HIPCHK(c, hipSetDevice(c->device));
    c->static_pending = true;
    HIPCHK(c, launch_delta_static(c->device, a, chunk, parts, any_long, any_scatter, any_perm, c->lds_ordered, c->stream));
    return INSHR_OK;
}

int inshr_dequantize(inshr_ctx *c, const inshr_dequant_in *in, float *const *out, uint32_t n_tensors)
{
    if (!c || !in || !out || n_tensors == 0 || n_tensors > 65535u) return INSHR_E_ARG;
    std::vector<RDesc> rd(n_tensors);
    u64 tile = 0, max_out = 0;
    for (uint32_t t = 0; t < n_tensors; t++) {
        const inshr_dequant_in &q = in[t];
        inshr_codes as_codes;
        as_codes.bits = q.bits;
        as_codes.bins = q.bins;
        uint32_t K = 0;
        if (codes_bins(as_codes, K)) return INSHR_E_CONFIG;
        if (q.n == 0 || q.n >= (1ull << 32) || !q.packed || !q.codebook || !out[t]) return INSHR_E_ARG;
        if (q.n_outlier && (!q.outlier_idx || !q.outlier_val)) return INSHR_E_ARG;
        if (q.n_outlier > q.n) return INSHR_E_SHAPE;
        RDesc &d = rd[t];
        memset(&d, 0, sizeof(d));
        d.packed = (const unsigned long long *)q.packed;
        d.codebook = q.codebook;
        d.out_idx = q.outlier_idx;
        d.out_val = q.outlier_val;
        d.dst = out[t];
        d.n = q.n;
        d.n_outlier = q.n_outlier;
        d.tile0 = tile;
        d.w = symbol_bits(K);
        d.K = K;
        d.val_bf16 = q.protected_bf16 ? 1u : 0u;
        tile += (q.n + DEQUANT_TILE - 1) / DEQUANT_TILE;
        max_out = std::max<u64>(max_out, q.n_outlier);
    }
    HIPCHK(c, hipSetDevice(c->device));
    Carver cv;
    const size_t o_rd = cv.take(sizeof(RDesc) * n_tensors);
    const size_t o_one = cv.take(sizeof(u32) * n_tensors); // symbol-1 counts
    HIPCHK(c, hipStreamSynchronize(c->stream)); // staging buffer and scratch may still be in use (inshr_delta)
    int rc = ensure_dev(c, c->aux_mem, cv.off);
    if (rc) return rc;
    rc = ensure_host(c, c->h_up, o_one);
    if (rc) return rc;
    char *hb = (char *)c->h_up.p, *db = (char *)c->aux_mem.p;
    memcpy(hb + o_rd, rd.data(), sizeof(RDesc) * n_tensors);
    Stage up;
    up.add(db, hb, o_one);
    up.zero(db + o_one, sizeof(u32) * n_tensors);
    HIPCHK(c, launch_stage(up, c->n_cu, c->stream));
    u32 *const flags = call_flags(c);
    HIPCHK(c, launch_dequantize((const RDesc *)(db + o_rd), (int)n_tensors, tile, max_out, flags,
                                (u32 *)(db + o_one), c->n_cu, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    const u32 f = raised_flags(flags);
    if (f & RF_SYMBOL) return INSHR_E_ARG;
    if (f & RF_LIST) return INSHR_E_SHAPE;
    return INSHR_OK;
}

int inshr_reconstruct(inshr_ctx *c, const inshr_codes *prev, const inshr_delta_out *delta,
                      inshr_codes_out *cur, uint32_t n_tensors)
{
    if (!c || !prev || !delta || !cur || n_tensors == 0) return INSHR_E_ARG;
    std::vector<DDesc> dd(n_tensors);
    std::vector<XDesc> xd(n_tensors);
    std::vector<u32> chunk_tensor;
    Parts parts;
    u64 chunk = 0;
    bool any_long = false;
    const u32 ctiles = call_chunk_tiles(c, prev, n_tensors);
    for (uint32_t t = 0; t < n_tensors; t++) {
        const uint64_t n = prev[t].n;
        inshr_codes cur_codes;
        cur_codes.bits = cur[t].bits;
        cur_codes.bins = cur[t].bins;
        uint32_t Kp = 0, Kc = 0;
        if (codes_bins(prev[t], Kp) || codes_bins(cur_codes, Kc)) return INSHR_E_CONFIG;
        if (prev[t].sym_bits != symbol_bits(Kp)) return INSHR_E_CONFIG;
        if (n == 0 || n >= (1ull << 32) || !prev[t].packed || !delta[t].packed || !cur[t].packed) return INSHR_E_ARG;
        const uint32_t wB = symbol_bits(std::max(Kp, Kc));
        if (delta[t].delta_bits != wB) return INSHR_E_CONFIG;
        if (delta[t].packed_words < (n * wB + 63) / 64) return INSHR_E_CAPACITY;
        const uint32_t wc = symbol_bits(Kc);
        if (cur[t].packed_words < (n * wc + 63) / 64) return INSHR_E_CAPACITY;
        DDesc &d = dd[t];
        memset(&d, 0, sizeof(d));
        d.prev = (const unsigned long long *)prev[t].packed;
        d.out = (unsigned long long *)delta[t].packed; // read only on this side
        d.n = n;
        d.out_words = (n * wB + 63) / 64;
        d.wp = prev[t].sym_bits;
        d.wc = wc;
        d.Kp = Kp;
        d.B = std::max(Kp, Kc) + 2u;
        d.wB = wB;
        d.chunk0 = chunk;
        const u64 nt = (n + DELTA_TILE - 1) / DELTA_TILE;
        d.n_chunks = (nt + ctiles - 1) / ctiles;
        d.ctiles = ctiles;
        for (u64 k = 0; k < d.n_chunks; k++) chunk_tensor.push_back(t);
        parts.enter(d, t);
        any_long = any_long || !delta_single(d);
        chunk += d.n_chunks;
        XDesc &x = xd[t];
        memset(&x, 0, sizeof(x));
        x.cur_out = (unsigned long long *)cur[t].packed;
        x.group_off_in = delta[t].group_off;
        x.Sc = Kc + 2u;
    }
    HIPCHK(c, hipSetDevice(c->device));
    Carver cv;
    const size_t o_dd = cv.take(sizeof(DDesc) * n_tensors);
    const size_t o_xd = cv.take(sizeof(XDesc) * n_tensors);
    const size_t o_ct = cv.take(sizeof(u32) * chunk_tensor.size());
    const size_t up_bytes = cv.off;
    const size_t o_go = cv.take(sizeof(u64) * (DELTA_SS + 8) * n_tensors); // group offsets from prev
    const size_t o_tt = cv.take(c->scratch_limit ? 0 : parts.bytes());
    const size_t o_ck = cv.take((size_t)chunk * DELTA_SS * 4);
    HIPCHK(c, hipStreamSynchronize(c->stream)); // staging buffer and scratch may still be in use (inshr_delta)
    int rc = ensure_dev(c, c->aux_mem, cv.off);
    if (rc) return rc;
    rc = ensure_host(c, c->h_up, up_bytes + sizeof(u32) * parts.tensor.size());
    if (rc) return rc;
    char *hb = (char *)c->h_up.p, *db = (char *)c->aux_mem.p;
    DeltaCall call;
    Stage up;
    if ((rc = place_parts(c, parts, o_tt, up_bytes, call, up))) return rc;
    for (uint32_t t = 0; t < n_tensors; t++) dd[t].group_off = (u64 *)(db + o_go) + (size_t)t * (DELTA_SS + 8);
    memcpy(hb + o_dd, dd.data(), sizeof(DDesc) * n_tensors);
    memcpy(hb + o_xd, xd.data(), sizeof(XDesc) * n_tensors);
    memcpy(hb + o_ct, chunk_tensor.data(), sizeof(u32) * chunk_tensor.size());
    up.add(db, hb, up_bytes);
    HIPCHK(c, launch_stage(up, c->n_cu, c->stream));
    u32 *const flags = call_flags(c);
    call.dd = (const DDesc *)(db + o_dd);
    call.chunk_tensor = (const u32 *)(db + o_ct);
    call.chunk_tot = (u32 *)(db + o_ck);
    call.flags = flags;
    call.n_chunks = chunk;
    call.any_long = any_long;
    call.lds_ordered = c->lds_ordered;
    HIPCHK(c, launch_reconstruct(call, (const XDesc *)(db + o_xd), c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    const u32 f = raised_flags(flags);
    if (f & RF_ORDER) {
        c->last_err = "reconstruct: ranks from returning LDS atomics disagree with ballot ranks (set INSHR_NO_LDS_ORDER=1)";
        return INSHR_E_INTERNAL;
    }
    if (f & RF_GROUPS) return INSHR_E_SHAPE;
    if (f & RF_DELTA) return INSHR_E_ARG;
    return INSHR_OK;
}

} // extern "C"
