// Batches of independent periodic systems advanced together: one launch per
// phase covers every system (work items name the system and its local block),
// and a call's whole step sequence runs as one captured HIP graph, launched on
// the caller's stream. Each system keeps its own buffers, parameters and particles, and
// its arithmetic is exactly that of a single-system run: a batch changes the
// launch shape, never the result.
#include <math.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "lbe_internal.h"

namespace lbe {

// Fused-kernel tile shapes the batch tuner tries: BX x (256 / BX) nodes of one
// xy-plane per 256-thread block (wide tiles coalesce better, square ones
// stage a smaller halo).
constexpr int kTileWidths[LB_TUNE_CANDIDATES] = {64, 32, 16};

struct BatchState {
    std::vector<lb_handle*> subs;
    int precision = LB_FP64;
    SysDev* d_sys = nullptr;
    WorkItem* d_items[BI_COUNT] = {};
    size_t cap_items[BI_COUNT] = {};
    std::vector<SysDev> h_sys;
    std::vector<WorkItem> h_items[BI_COUNT];
    BatchLaunch bl;
    bool dirty = true;
    int bx = 64;      // fused tile width in use
    int parity = 0;   // index of the current population and owner copies, shared by all systems
    bool dens_ready = false;  // every system's Psi / rho match its current populations
    bool walls = false;       // some system has wall nodes
    hipStream_t cap = nullptr;  // records graphs only; nothing is launched on it
    // the graph of the last step count, per starting parity
    hipGraph_t graph[2] = {nullptr, nullptr};
    hipGraphExec_t exec[2] = {nullptr, nullptr};
    int graph_steps[2] = {0, 0};
    int last_steps = 0;          // steps of the graph launched last
    int64_t last_nodes = 0;      // its kernel nodes
};

namespace {

void tiles_for(const lb_params& p, int bx, int& tx, int& ty) {
    const int by = 256 / bx;
    tx = (p.nx + bx - 1) / bx;
    ty = (p.ny + by - 1) / by;
}

// Most work items a system can ever need, per kind.
void item_capacity(const lb_params& p, size_t cap[BI_COUNT]) {
    const size_t N = (size_t)p.nx * p.ny * p.nz;
    int tx, ty;
    size_t tiles = 0;
    for (int bx : kTileWidths) {
        tiles_for(p, bx, tx, ty);
        tiles = std::max(tiles, (size_t)tx * ty * p.nz);
    }
    const size_t np = (size_t)std::max(p.max_particles, 0);
    const bool mom = in_moments(p);
    cap[BI_NODE] = (N + 255) / 256;
    cap[BI_NODE_POP] = mom ? 0 : cap[BI_NODE];
    cap[BI_TILE] = cap[BI_TILE_PLAIN] = mom ? 0 : tiles;
    cap[BI_MTILE] = cap[BI_MTILE_PLAIN] = mom ? tiles : 0;
    const size_t shares = np > 0 ? max_shares(np) : 0;
    cap[BI_PART] = np;
    cap[BI_SHARE] = shares;
    cap[BI_SHARE_POP] = mom ? 0 : shares;
    cap[BI_SHARE_MOM] = mom ? shares : 0;
}

struct BatchLayout {
    size_t sys = 0;
    size_t items[BI_COUNT] = {};
    size_t cap[BI_COUNT] = {};
    std::vector<size_t> sub;  // workspace bytes of each system
    size_t total = 0;
};

bool batch_layout(int nsys, const lb_params* prm, BatchLayout& L, std::string* why) {
    if (nsys <= 0) {
        *why = "a batch needs at least one system";
        return false;
    }
    if (!prm) {
        *why = "per-system parameters are NULL";
        return false;
    }
    L.sub.resize(nsys);
    for (int s = 0; s < nsys; s++) {
        std::string w;
        if (!params_ok(&prm[s], &w)) {
            *why = "system " + std::to_string(s) + ": " + w;
            return false;
        }
        if (prm[s].precision != prm[0].precision) {
            *why = "all systems of a batch share one precision";
            return false;
        }
        size_t c[BI_COUNT];
        item_capacity(prm[s], c);
        for (int k = 0; k < BI_COUNT; k++) L.cap[k] += c[k];
        L.sub[s] = layout_of(&prm[s]).total;
    }
    for (int k = 0; k < BI_COUNT; k++) {
        if (L.cap[k] > (size_t)INT32_MAX) {
            *why = "batch too large for one launch";
            return false;
        }
        L.items[k] = align_up(std::max<size_t>(L.cap[k], 1) * sizeof(WorkItem));
    }
    L.sys = align_up((size_t)nsys * sizeof(SysDev));
    L.total = L.sys;
    for (int k = 0; k < BI_COUNT; k++) L.total += L.items[k];
    for (int s = 0; s < nsys; s++) L.total += L.sub[s];
    return true;
}

void drop_graph(BatchState* B, int k) {
    if (B->exec[k]) (void)hipGraphExecDestroy(B->exec[k]);
    if (B->graph[k]) (void)hipGraphDestroy(B->graph[k]);
    B->exec[k] = nullptr;
    B->graph[k] = nullptr;
    B->graph_steps[k] = 0;
}
void drop_graphs(BatchState* B) {
    for (int k = 0; k < 2; k++) drop_graph(B, k);
}

}  // namespace

SysDev sys_dev(const lb_handle* q) {
    SysDev d{};
    d.box = q->box;
    d.f[0] = q->b.f[0];
    d.f[1] = q->b.f[1];
    d.psi = q->b.psi;
    d.rho = q->b.rho;
    d.owner[0] = q->b.owner[0];
    d.owner[1] = q->b.owner[1];
    d.part = q->b.part;
    d.bmask[0] = q->b.bmask[0];
    d.bmask[1] = q->b.bmask[1];
    d.rec = q->b.rec;
    d.pfast[0] = q->b.pfast[0];
    d.pfast[1] = q->b.pfast[1];
    d.mv[0] = q->b.mv[0];
    d.mv[1] = q->b.mv[1];
    d.mom = q->mom ? 1 : 0;
    d.kpart = q->b.kpart;
    d.fpart = q->b.fpart;
    d.health = q->b.health;
    d.counters = q->b.counters;
    d.cap = q->cap;
    d.np = q->np;
    return d;
}

namespace {

// Rebuild the device descriptors and work lists from the systems' state.
int refresh(lb_handle* h) {
    BatchState* B = h->batch;
    const int nsys = (int)B->subs.size();
    B->h_sys.resize(nsys);
    B->walls = false;
    for (int k = 0; k < BI_COUNT; k++) B->h_items[k].clear();
    // the systems without and with solids are a launch of the moment step each
    int64_t columns[2] = {0, 0};
    int deep[2] = {1, 1};
    for (lb_handle* q : B->subs) {
        if (!q->mom) continue;
        int tx, ty;
        tiles_for(q->prm, B->bx, tx, ty);
        const int k = q->has_solid ? 1 : 0;
        columns[k] += (int64_t)tx * ty;
        deep[k] = std::max(deep[k], (int)q->box.nz);
    }
    for (int k = 0; k < 2; k++) B->bl.zc[k] = mstep_planes(columns[k], deep[k], k == 1);
    B->bl.mom = columns[0] + columns[1] > 0;
    for (int s = 0; s < nsys; s++) {
        lb_handle* q = B->subs[s];
        SysDev& d = B->h_sys[s];
        d = sys_dev(q);
        B->walls = B->walls || q->box.walls != 0;
        tiles_for(q->prm, B->bx, d.tiles_x, d.tiles_y);
        d.kext = kill_ext(q);
        const int nnode = (int)((q->box.N + 255) / 256);
        const int ntile = d.tiles_x * d.tiles_y * q->box.nz;
        const int zc = B->bl.zc[q->has_solid ? 1 : 0];
        const int ncol = d.tiles_x * d.tiles_y * ((q->box.nz + zc - 1) / zc);
        for (int i = 0; i < nnode; i++) B->h_items[BI_NODE].push_back({s, i});
        for (int i = 0; i < q->np; i++) B->h_items[BI_PART].push_back({s, i});
        for (int i = 0; i < q->np * particle_split(q->np); i++) {
            B->h_items[BI_SHARE].push_back({s, i});
            B->h_items[d.mom ? BI_SHARE_MOM : BI_SHARE_POP].push_back({s, i});
        }
        if (d.mom) {
            for (int i = 0; i < ncol; i++) B->h_items[q->has_solid ? BI_MTILE : BI_MTILE_PLAIN].push_back({s, i});
        } else {
            for (int i = 0; i < nnode; i++) B->h_items[BI_NODE_POP].push_back({s, i});
            for (int i = 0; i < ntile; i++) B->h_items[q->has_solid ? BI_TILE : BI_TILE_PLAIN].push_back({s, i});
        }
    }
    for (int k = 0; k < BI_COUNT; k++)
        if (B->h_items[k].size() > B->cap_items[k]) return fail(h, LB_EINVAL, "batch work list exceeds its capacity");
    LBE_HIP_OR_FAIL(h, hipMemcpyAsync(B->d_sys, B->h_sys.data(), nsys * sizeof(SysDev), hipMemcpyHostToDevice, h->stream));
    for (int k = 0; k < BI_COUNT; k++) {
        if (!B->h_items[k].empty())
            LBE_HIP_OR_FAIL(h, hipMemcpyAsync(B->d_items[k], B->h_items[k].data(),
                                              B->h_items[k].size() * sizeof(WorkItem), hipMemcpyHostToDevice,
                                              h->stream));
        B->bl.items[k] = B->d_items[k];
        B->bl.n[k] = (int)B->h_items[k].size();
    }
    B->bl.sys = B->d_sys;
    B->bl.bx = B->bx;
    LBE_HIP_OR_FAIL(h, hipStreamSynchronize(h->stream));
    drop_graphs(B);
    B->dirty = false;
    return LB_OK;
}

// One step of every system, parity c (populations and owner maps at index c),
// starting from densities of the current populations and ending with those
// of the next step (formed before kill / fill, as in a single-system step).
hipError_t enqueue_batch_step(BatchState* B, hipStream_t st, int c) {
    const BatchLaunch& bl = B->bl;
    const int prec = B->precision;
    hipError_t e;
    if ((e = launch_batch_shell(bl, prec, st, c)) != hipSuccess) return e;
    if (B->walls && (e = launch_batch_wall_shell(bl, prec, st, c)) != hipSuccess) return e;
    if ((e = launch_batch_fused(bl, prec, st, c, c)) != hipSuccess) return e;
    if (bl.mom && (e = launch_batch_mstep(bl, st, c)) != hipSuccess) return e;
    if ((e = launch_batch_forces(bl, st)) != hipSuccess) return e;
    if ((e = launch_batch_bodies(bl, st, c)) != hipSuccess) return e;
    if ((e = launch_batch_clear_owner(bl, st, 1 - c)) != hipSuccess) return e;
    if ((e = launch_batch_raster(bl, st, 1 - c)) != hipSuccess) return e;
    if ((e = launch_batch_density(bl, prec, st, 1 - c, 1 - c, c)) != hipSuccess) return e;
    if (bl.mom && (e = launch_batch_check(bl, (int)B->subs.size(), st, c)) != hipSuccess) return e;
    return launch_batch_killfill(bl, prec, st, c, 1 - c);
}

// Graph of n steps starting at parity c (it ends at parity c when n is even),
// recorded on the capture stream.
int capture(lb_handle* h, int c, int n) {
    BatchState* B = h->batch;
    drop_graph(B, c);
    LBE_HIP_OR_FAIL(h, hipStreamBeginCapture(B->cap, hipStreamCaptureModeThreadLocal));
    hipError_t e = hipSuccess;
    for (int k = 0; k < n && e == hipSuccess; k++) e = enqueue_batch_step(B, B->cap, (c + k) & 1);
    hipGraph_t g = nullptr;
    const hipError_t e2 = hipStreamEndCapture(B->cap, &g);
    if (e != hipSuccess || e2 != hipSuccess) {
        if (g) (void)hipGraphDestroy(g);
        return fail(h, LB_EHIP, std::string("graph capture: ") + hipGetErrorString(e != hipSuccess ? e : e2));
    }
    hipGraphExec_t x = nullptr;
    e = hipGraphInstantiate(&x, g, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        (void)hipGraphDestroy(g);
        return fail(h, LB_EHIP, std::string("graph instantiate: ") + hipGetErrorString(e));
    }
    B->graph[c] = g;
    B->exec[c] = x;
    B->graph_steps[c] = n;
    return LB_OK;
}

int check_ready(lb_handle* h) {
    BatchState* B = h->batch;
    for (size_t s = 0; s < B->subs.size(); s++)
        if (!B->subs[s]->inited)
            return fail(h, LB_ESTATE, "system " + std::to_string(s) + " has no fields (lb_init_fields)");
    if (B->dirty) return refresh(h);
    return LB_OK;
}

}  // namespace

// n steps of every system as one graph launch on the caller's stream. The
// graph of the last step count is kept per starting parity and replayed
// while the count and the systems stay the same.
int batch_sys(lb_handle* h, const SysDev** d_sys, int* nsys, int* parity, bool refresh_ok) {
    BatchState* B = h->batch;
    if (!refresh_ok && B->dirty)
        return fail(h, LB_ESTATE, "the batch changed since its tables were last uploaded: step it (or call "
                                  "lb_batch_tune) first");
    const int rc = check_ready(h);
    if (rc != LB_OK) return rc;
    *d_sys = B->d_sys;
    *nsys = (int)B->subs.size();
    *parity = B->parity;
    return LB_OK;
}

int batch_step_async(lb_handle* h, int nsteps) {
    BatchState* B = h->batch;
    int rc = check_ready(h);
    if (rc != LB_OK) return rc;
    if (nsteps == 0) return LB_OK;
    if (!B->dens_ready) {
        LBE_HIP_OR_FAIL(h, launch_batch_density(B->bl, B->precision, h->stream, B->parity, B->parity, -1));
        B->dens_ready = true;
    }
    const int c = B->parity;
    if (!B->exec[c] || B->graph_steps[c] != nsteps) {
        rc = capture(h, c, nsteps);
        if (rc != LB_OK) return rc;
    }
    LBE_HIP_OR_FAIL(h, hipGraphLaunch(B->exec[c], h->stream));
    size_t nodes = 0;
    LBE_HIP_OR_FAIL(h, hipGraphGetNodes(B->graph[c], nullptr, &nodes));
    B->last_steps = nsteps;
    B->last_nodes = (int64_t)nodes;
    B->parity = (c + nsteps) & 1;
    for (lb_handle* q : B->subs) {
        q->ocur = B->parity;
        if (q->mom) {
            q->mc = B->parity;
            q->oprev = 1 - B->parity;
        } else {
            q->cur = B->parity;
            q->dens_ready = true;
        }
    }
    return LB_OK;
}

int batch_health(lb_handle* h) {
    BatchState* B = h->batch;
    const int nsys = (int)B->subs.size();
    std::vector<int> bad(nsys, 0);
    for (int s = 0; s < nsys; s++)
        LBE_HIP_OR_FAIL(h, hipMemcpyAsync(&bad[s], B->subs[s]->b.health, sizeof(int), hipMemcpyDeviceToHost, h->stream));
    LBE_HIP_OR_FAIL(h, hipStreamSynchronize(h->stream));
    for (int s = 0; s < nsys; s++) {
        if (bad[s] & 2)
            return fail(h, LB_EUNSTABLE,
                        "system " + std::to_string(s) + ": a particle moved more than two lattice spacings in one step");
        if (bad[s]) return fail(h, LB_EUNSTABLE, "system " + std::to_string(s) + ": NaN or negative density detected");
    }
    return LB_OK;
}

void batch_destroy(lb_handle* h) {
    BatchState* B = h->batch;
    if (!B) return;
    (void)hipStreamSynchronize(h->stream);
    drop_graphs(B);
    if (B->cap) (void)hipStreamDestroy(B->cap);
    for (lb_handle* q : B->subs) {
        for (hipEvent_t e : q->ev_pool) (void)hipEventDestroy(e);
        delete q;
    }
    delete B;
    h->batch = nullptr;
}

void batch_touch(lb_handle* sub) {
    if (sub && sub->parent && sub->parent->batch) {
        sub->parent->batch->dirty = true;
        sub->parent->batch->dens_ready = false;
    }
}

}  // namespace lbe

using namespace lbe;

extern "C" {

size_t lb_batch_workspace_bytes(int32_t nsys, const lb_params* per_sys) {
    BatchLayout L;
    std::string why;
    if (!batch_layout(nsys, per_sys, L, &why)) return 0;
    return L.total;
}

int lb_create_batch(int32_t nsys, const lb_params* per_sys, void* dev_ws, size_t ws_bytes, void* hip_stream,
                    lb_handle** out) {
    if (!out) return fail(nullptr, LB_EINVAL, "out is NULL");
    *out = nullptr;
    BatchLayout L;
    std::string why;
    if (!batch_layout(nsys, per_sys, L, &why)) return fail(nullptr, LB_EINVAL, why);
    if (!dev_ws) return fail(nullptr, LB_EINVAL, "workspace is NULL");
    if (ws_bytes < L.total)
        return fail(nullptr, LB_ENOMEM, "workspace too small: need " + std::to_string(L.total) + " bytes");
    if (((uintptr_t)dev_ws) % kAlign != 0) return fail(nullptr, LB_EINVAL, "workspace must be 256-byte aligned");
    lb_handle* h = new lb_handle();
    h->prm = per_sys[0];
    h->stream = (hipStream_t)hip_stream;
    h->ws = (char*)dev_ws;
    h->ws_bytes = ws_bytes;
    h->batch = new BatchState();
    BatchState* B = h->batch;
    B->precision = per_sys[0].precision;
    char* p = (char*)dev_ws;
    B->d_sys = (SysDev*)p;
    p += L.sys;
    for (int k = 0; k < BI_COUNT; k++) {
        B->d_items[k] = (WorkItem*)p;
        B->cap_items[k] = L.cap[k];
        p += L.items[k];
    }
    // default tile: 64 x 4 when every system is at least 64 wide
    B->bx = 64;
    for (int s = 0; s < nsys; s++)
        if (per_sys[s].nx < 64) B->bx = 32;
    int rc = LB_OK;
    for (int s = 0; s < nsys && rc == LB_OK; s++) {
        lb_handle* q = new lb_handle();
        q->parent = h;
        rc = setup_handle(q, &per_sys[s], p, L.sub[s], h->stream);
        p += L.sub[s];
        if (rc != LB_OK) {
            delete q;
            break;
        }
        B->subs.push_back(q);
    }
    // a stream to record graphs on (the caller's may be the null stream,
    // which cannot be captured); default priority
    if (rc == LB_OK && hipStreamCreateWithFlags(&B->cap, hipStreamNonBlocking) != hipSuccess)
        rc = fail(nullptr, LB_EHIP, "capture stream creation failed");
    if (rc != LB_OK) {
        batch_destroy(h);
        delete h;
        return rc;
    }
    h->inited = true;
    *out = h;
    return LB_OK;
}

int lb_batch_size(const lb_handle* h) {
    if (!h || !h->batch) return LB_EINVAL;
    return (int)h->batch->subs.size();
}

int lb_batch_system(lb_handle* h, int32_t sys, lb_handle** out) {
    if (!h || !out) return LB_EINVAL;
    *out = nullptr;
    if (!h->batch) return fail(h, LB_EINVAL, "not a batch handle");
    if (sys < 0 || sys >= (int)h->batch->subs.size()) return fail(h, LB_EINVAL, "system index out of range");
    *out = h->batch->subs[sys];
    return LB_OK;
}

static lb_handle* sys_of(lb_handle* h, int32_t sys) {
    if (!h || !h->batch || sys < 0 || sys >= (int32_t)h->batch->subs.size()) return nullptr;
    return h->batch->subs[sys];
}

#define LBE_SYS_OR_FAIL(h, sys, q)                                                                  \
    lb_handle* q = sys_of(h, sys);                                                                  \
    if (!q) {                                                                                       \
        if (h) (void)fail(h, LB_EINVAL, h->batch ? "system index out of range" : "not a batch handle"); \
        return LB_EINVAL;                                                                           \
    }

int lb_init_fields_sys(lb_handle* h, int32_t sys, const double* rho_a, const double* rho_b, const double* u) {
    LBE_SYS_OR_FAIL(h, sys, q);
    return lb_init_fields(q, rho_a, rho_b, u);
}

int lb_add_ellipsoids_sys(lb_handle* h, int32_t sys, int32_t n, const double* radii, const double* pos,
                          const double* quat, const double* delta_rho, const double* density) {
    LBE_SYS_OR_FAIL(h, sys, q);
    return lb_add_ellipsoids(q, n, radii, pos, quat, delta_rho, density);
}

int lb_read_fields_sys(lb_handle* h, int32_t sys, double* rho_a, double* rho_b, double* u, int32_t* owner) {
    LBE_SYS_OR_FAIL(h, sys, q);
    return lb_read_fields(q, rho_a, rho_b, u, owner);
}

int lb_read_particles_sys(lb_handle* h, int32_t sys, double* pos, double* quat, double* vel, double* omega,
                          double* force, double* torque) {
    LBE_SYS_OR_FAIL(h, sys, q);
    return lb_read_particles(q, pos, quat, vel, omega, force, torque);
}

int lb_stats_sys(lb_handle* h, int32_t sys, double out[8]) {
    LBE_SYS_OR_FAIL(h, sys, q);
    return lb_stats(q, out);
}

}  // extern "C"

namespace {

// Tuning results kept for the life of the process, keyed by the precision and
// the shape of every system (box, whether it holds solids, and whether it steps in
// moments, which is another kernel): a batch of the same systems is not timed
// again.
struct TuneEntry {
    int bx;
    double ms[LB_TUNE_CANDIDATES];
};
std::map<std::string, TuneEntry>& tune_cache() {
    static std::map<std::string, TuneEntry> c;
    return c;
}
std::mutex& tune_mutex() {
    static std::mutex m;
    return m;
}
std::string tune_key(const BatchState* B) {
    std::string k = std::to_string(B->precision);
    for (const lb_handle* q : B->subs)
        k += ";" + std::to_string(q->box.nx) + "x" + std::to_string(q->box.ny) + "x" + std::to_string(q->box.nz) +
             (q->has_solid ? "s" : "f") + (q->mom ? "m" : "");
    return k;
}

}  // namespace

extern "C" {

int lb_batch_last_graph(const lb_handle* h, int32_t* steps, int64_t* kernel_nodes) {
    if (!h || !h->batch) return LB_EINVAL;
    if (steps) *steps = h->batch->last_steps;
    if (kernel_nodes) *kernel_nodes = h->batch->last_nodes;
    return LB_OK;
}

int lb_batch_tune(lb_handle* h, lb_tune_result* out) {
    if (!h) return LB_EINVAL;
    if (!h->batch) return fail(h, LB_EINVAL, "not a batch handle");
    BatchState* B = h->batch;
    int rc = check_ready(h);
    if (rc != LB_OK) return rc;
    const std::string key = tune_key(B);
    TuneEntry te{};
    bool cached = false;
    {
        std::lock_guard<std::mutex> lk(tune_mutex());
        auto it = tune_cache().find(key);
        if (it != tune_cache().end()) {
            te = it->second;
            cached = true;
        }
    }
    if (!cached) {
        // the fused launch only writes the next population copy and its masks,
        // which the next step rewrites whole, and link records (cleared
        // below): timing it leaves the state untouched
        const int c = B->parity;
        hipEvent_t e0, e1;
        LBE_HIP_OR_FAIL(h, hipEventCreate(&e0));
        LBE_HIP_OR_FAIL(h, hipEventCreate(&e1));
        float best = 0.0f;
        te.bx = B->bx;
        // (in moments it writes the copy from which a checkpoint would form the
        // populations: they are formed first)
        for (lb_handle* q : B->subs)
            if (q->mom) LBE_HIP_OR_FAIL(h, launch_expand(q));
        for (int k = 0; k < LB_TUNE_CANDIDATES && rc == LB_OK; k++) {
            B->bx = kTileWidths[k];
            rc = refresh(h);
            if (rc != LB_OK) break;
            LBE_HIP_OR_FAIL(h, launch_batch_density(B->bl, B->precision, h->stream, c, c, -1));
            LBE_HIP_OR_FAIL(h, launch_batch_shell(B->bl, B->precision, h->stream, c));
            auto fluid = [&]() -> hipError_t {
                const hipError_t e = launch_batch_fused(B->bl, B->precision, h->stream, c, c);
                return e == hipSuccess && B->bl.mom ? launch_batch_mstep(B->bl, h->stream, c) : e;
            };
            LBE_HIP_OR_FAIL(h, fluid());
            LBE_HIP_OR_FAIL(h, hipEventRecord(e0, h->stream));
            constexpr int reps = 3;
            for (int r = 0; r < reps; r++) LBE_HIP_OR_FAIL(h, fluid());
            LBE_HIP_OR_FAIL(h, hipEventRecord(e1, h->stream));
            LBE_HIP_OR_FAIL(h, hipEventSynchronize(e1));
            float ms = 0.0f;
            LBE_HIP_OR_FAIL(h, hipEventElapsedTime(&ms, e0, e1));
            te.ms[k] = (double)ms / reps;
            if (best == 0.0f || ms < best) {
                best = ms;
                te.bx = kTileWidths[k];
            }
        }
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        if (rc != LB_OK) return rc;
        // the timed launches also wrote link records, which the force pass
        // would otherwise have read and cleared: clear them
        for (lb_handle* q : B->subs) {
            const size_t rb = layout_of(&q->prm).rec;
            if (rb) LBE_HIP_OR_FAIL(h, launch_fill_f64(h, q->b.rec, 0.0, (int64_t)(rb / sizeof(double))));
            if (!q->mom) continue;
            LBE_HIP_OR_FAIL(h, launch_fill_u32(h, (uint32_t*)q->b.health + ST_SUSPECT, 0u, 1));
            LBE_HIP_OR_FAIL(h, launch_set_from(q, FROM_POPS));
        }
        std::lock_guard<std::mutex> lk(tune_mutex());
        tune_cache()[key] = te;
    }
    B->bx = te.bx;
    rc = refresh(h);
    if (rc != LB_OK) return rc;
    if (out) {
        out->tile_width = te.bx;
        out->cached = cached ? 1 : 0;
        for (int k = 0; k < LB_TUNE_CANDIDATES; k++) {
            out->tile_widths[k] = kTileWidths[k];
            out->ms[k] = te.ms[k];
        }
    }
    return LB_OK;
}

}  // extern "C"
