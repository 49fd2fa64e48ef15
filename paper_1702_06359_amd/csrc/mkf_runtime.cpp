// Host runtime and C ABI of the track builder (everything except serving).
#include "mkf_runtime.hpp"

#include "mkf_pack.hpp"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <functional>

namespace mkf {

static thread_local char g_err[512] = "";

mkf_status fail(mkf_status st, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return st;
}

// ---------------------------------------------------------------- memory

static std::atomic<unsigned long long> g_broken{0};   // one bit per device

void note_device_error(hipError_t e)
{
    switch (e) {
    case hipErrorIllegalAddress:
    case hipErrorLaunchFailure:
    case hipErrorAssert: {
        int dev = 0;
        (void)hipGetDevice(&dev);
        g_broken.fetch_or(1ull << (dev & 63));
        break;
    }
    default:
        break;
    }
}

bool device_broken(int device) { return (g_broken.load() >> (device & 63)) & 1ull; }

void *CtxHeap::alloc(size_t bytes)
{
    if (bytes == 0) bytes = 256;
    if (ctx->has_alloc) return ctx->alloc.alloc(bytes, (void *)ctx->stream, ctx->alloc.user);
    void *p = nullptr;
    if (hipMalloc(&p, bytes) != hipSuccess) {
        (void)hipGetLastError();   // not left for the next launch to report
        return nullptr;
    }
    return p;
}

void CtxHeap::release(void *p)
{
    if (!p) return;
    if (ctx->has_alloc) ctx->alloc.free(p, (void *)ctx->stream, ctx->alloc.user);
    else (void)hipFree(p);
}

SlabHeap::SlabHeap(char *base, size_t bytes) : base_(base), cap_(bytes) { free_[0] = bytes; }

void *SlabHeap::alloc(size_t bytes)
{
    bytes = (bytes + 255) & ~size_t(255);
    std::lock_guard<std::mutex> lk(mu_);
    for (auto it = free_.begin(); it != free_.end(); ++it) {
        if (it->second < bytes) continue;
        const size_t off = it->first, sz = it->second;
        free_.erase(it);
        if (sz > bytes) free_[off + bytes] = sz - bytes;
        taken_[off] = bytes;
        used_ += bytes;
        return base_ + off;
    }
    return nullptr;
}

void SlabHeap::release(void *p)
{
    if (!p) return;
    std::lock_guard<std::mutex> lk(mu_);
    const size_t off = static_cast<char *>(p) - base_;
    auto t = taken_.find(off);
    if (t == taken_.end()) return;
    size_t sz = t->second;
    taken_.erase(t);
    used_ -= sz;
    size_t start = off;
    auto nx = free_.lower_bound(off);
    if (nx != free_.end() && nx->first == off + sz) {
        sz += nx->second;
        free_.erase(nx);
    }
    auto pv = free_.lower_bound(off);
    if (pv != free_.begin()) {
        --pv;
        if (pv->first + pv->second == off) {
            start = pv->first;
            sz += pv->second;
            free_.erase(pv);
        }
    }
    free_[start] = sz;
}

// ---------------------------------------------------------------- layout

namespace {

struct Carver {
    char *base;
    size_t off = 0;
    explicit Carver(void *b) : base(static_cast<char *>(b)) {}
    template <class T>
    T *take(size_t count)
    {
        off = (off + 255) & ~size_t(255);
        T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
        off += count * sizeof(T);
        return p;
    }
};

// The event's inputs come first (hits, seeds, tracks as the host packs them,
// cleared work counters and the descriptor: one copy moves them all), then
// the binned hits and the results.
size_t carve_data(const EventShape &s, void *base, DevEvent *v, DevEvent **dev_view, size_t *input_end = nullptr)
{
    Carver c(base);
    const size_t n = (size_t)s.n_hits(), ns = (size_t)s.n_seeds, nt = (size_t)s.n_tracks, nl = (size_t)s.n_layers;
    v->hits = c.take<float4>(n);
    v->seed_par = c.take<float>(6 * ns);
    v->seed_cov = c.take<float>(21 * ns);
    v->seed_hits = c.take<int>((size_t)s.n_seed_layers * ns);
    v->seed_order = c.take<int>(ns);
    v->track_par = c.take<float>(6 * nt);
    v->track_cov = c.take<float>(21 * nt);
    v->track_hits = c.take<int>(nl * nt);
    v->stats = c.take<unsigned long long>(5);
    DevEvent *dv = c.take<DevEvent>(1);
    if (dev_view) *dev_view = dv;
    if (input_end) *input_end = c.off;
    v->binned = c.take<float4>(n);
    v->bin_of = c.take<int>(n);
    v->out_rec = c.take<float>(kRecWords * ns);
    v->out_hits = c.take<int>(nl * ns);
    v->fit_rec = c.take<float>(kRecWords * nt);
    v->rf_rec = c.take<float>(kRecWords * ns);
    return c.off;
}

// Bytes of the working arrays of the bucketed index build (k_index_hist ff.).
size_t index_work_bytes(const EventShape &s, int *chunk, int *chunks)
{
    const int most = max_layer_hits(s);
    *chunk = idx_chunk_of(most);
    *chunks = (most + *chunk - 1) / *chunk;
    return (sizeof(float4) + sizeof(int)) * (size_t)s.n_hits() +
           sizeof(int) * (size_t)s.n_layers * ((size_t)*chunks * kBuckets + kBuckets + 1) + 4 * 256;
}

// What the budget of a served event allows it beyond its inputs, FP32 result rows, binned
// hits and bin offsets: its results counted in the caller's types (the FP64
// fields make 27 words more a row for the build's, 26 for a final fit's), an
// int per hit and one per bin.
size_t index_allowance(const EventShape &s, int nb)
{
    return sizeof(int) * ((27 + 26) * (size_t)s.n_seeds + (size_t)s.n_hits() + (size_t)s.n_layers * nb);
}

// Whether an event asks for those arrays: one loaded for itself always, a
// served one where its budget covers them or its layers' counters exceed a
// block's LDS (the one-block-per-layer build then takes several times as
// long).  Where the memory is not to be had it does without.
bool wants_index_work(const EventShape &s, int nb, bool served)
{
    int chunk, chunks;
    return !served || index_work_bytes(s, &chunk, &chunks) <= index_allowance(s, nb) ||
           !layer_block_fits(max_layer_hits(s), nb);
}

size_t carve_index(const EventShape &s, int nb, bool work, void *base, DevEvent *v)
{
    Carver c(base);
    const size_t nl = (size_t)s.n_layers, n = (size_t)s.n_hits();
    v->bin_off = c.take<int>(nl * bin_off_stride(nb));
    v->part = nullptr;
    if (work) {
        index_work_bytes(s, &v->idx_chunk, &v->idx_chunks);
        v->bucket_shift = bucket_shift_of(nb);
        v->part = c.take<float4>(n);
        v->part_bin = c.take<int>(n);
        v->hist = c.take<int>(nl * v->idx_chunks * kBuckets);
        v->bucket_off = c.take<int>(nl * (kBuckets + 1));
    }
    return c.off;
}

int plain_slots(int n_seeds, int spw)
{
    return ((n_seeds + spw - 1) / spw) * kWave;
}

size_t carve_plain(const EventShape &s, int slots, void *base, DevEvent *v)
{
    Carver c(base);
    const size_t S = (size_t)slots;
    v->st_par = c.take<float>(6 * S);
    v->st_cov = c.take<float>(21 * S);
    v->st_trig = c.take<float>(4 * S);
    v->st_chi2 = c.take<float>(S);
    v->st_meta = c.take<int>(S);
    v->st_hist = c.take<int>((size_t)s.n_layers * S);
    v->st_slots = slots;
    return c.off;
}

// Host threads that pack inputs, started on first use and kept for the life
// of the process.  A caller posts a job (n tasks, at most `threads` workers
// including itself), takes tasks itself and waits until every task is done;
// jobs of concurrent callers share the workers.
class HostPool {
  public:
    static HostPool &get()
    {
        static HostPool *pool = new HostPool();   // never destroyed: workers may outlive static destructors
        return *pool;
    }

    void run(int n_tasks, int threads, const std::function<void(int)> &f)
    {
        Job job;
        job.f = &f;
        job.n = n_tasks;
        job.helpers = std::min(threads, n_tasks) - 1;
        if (job.helpers > 0 && !workers_.empty()) {
            std::lock_guard<std::mutex> lk(mu_);
            jobs_.push_back(&job);
            cv_.notify_all();
        }
        work(job);
        std::unique_lock<std::mutex> lk(mu_);
        auto it = std::find(jobs_.begin(), jobs_.end(), &job);
        if (it != jobs_.end()) jobs_.erase(it);
        done_cv_.wait(lk, [&] { return job.done.load() == job.n && job.active == 0; });
    }

  private:
    struct Job {
        const std::function<void(int)> *f = nullptr;
        int n = 0;
        int helpers = 0;                 // workers still allowed to join (under mu_)
        int active = 0;                  // workers inside the job (under mu_)
        std::atomic<int> next{0};
        std::atomic<int> done{0};
    };

    HostPool()
    {
        const unsigned hw = std::max(1u, std::thread::hardware_concurrency());
        const int n = (int)std::min(15u, hw > 1 ? hw - 1 : 0u);
        for (int i = 0; i < n; ++i) workers_.emplace_back([this] { loop(); });
        for (auto &t : workers_) t.detach();
    }

    void work(Job &job)
    {
        for (int t = job.next.fetch_add(1); t < job.n; t = job.next.fetch_add(1)) {
            (*job.f)(t);
            if (job.done.fetch_add(1) + 1 == job.n) {
                std::lock_guard<std::mutex> lk(mu_);
                done_cv_.notify_all();
            }
        }
    }

    void loop()
    {
        std::unique_lock<std::mutex> lk(mu_);
        for (;;) {
            Job *job = nullptr;
            for (Job *j : jobs_)
                if (j->helpers > 0 && j->next.load() < j->n) {
                    job = j;
                    break;
                }
            if (!job) {
                cv_.wait(lk);
                continue;
            }
            --job->helpers;
            ++job->active;
            lk.unlock();
            work(*job);
            lk.lock();
            --job->active;
            done_cv_.notify_all();
        }
    }

    std::mutex mu_;
    std::condition_variable cv_, done_cv_;
    std::deque<Job *> jobs_;
    std::vector<std::thread> workers_;
};

// Runs f(task) for task = 0 .. n_tasks-1 on up to `threads` host threads.
template <class F>
void run_tasks(int n_tasks, int threads, F f)
{
    threads = std::max(1, std::min(threads, n_tasks));
    if (threads == 1) {
        for (int t = 0; t < n_tasks; ++t) f(t);
        return;
    }
    const std::function<void(int)> fn = f;
    HostPool::get().run(n_tasks, threads, fn);
}


void derive_params(mkf_ctx *ctx)
{
    Params &P = ctx->params;
    const mkf_config &c = ctx->cfg;
    const mkf_tuning &t = ctx->tuning;
    std::memset(&P, 0, sizeof(P));
    for (int L = 0; L < c.n_layers; ++L) {
        LayerParam &lp = P.layer[L];
        lp.r = (float)c.layer_r[L];
        lp.x0 = (float)c.layer_x0[L];
        lp.inv_dphi = (float)(t.bins_phi / (2.0 * M_PI));
        lp.inv_r = (float)(1.0 / c.layer_r[L]);
        lp.kind = c.layer_kind[L];
        lp.half_thick = (float)(0.5 * c.layer_thickness[L]);
        if (lp.kind == 0) {
            lp.half_z = (float)c.layer_half_z[L];
            lp.inv_dz = (float)(t.bins_z / (2.0 * c.layer_half_z[L]));
            lp.grid_lo = -lp.half_z;
        } else {
            lp.zplane = (float)c.layer_z[L];
            lp.inv_dz = (float)(t.bins_z / (c.layer_r[L] - c.layer_rmin[L]));
            lp.grid_lo = (float)c.layer_rmin[L];
        }
    }
    P.n_layers = c.n_layers;
    P.n_seed_layers = c.n_seed_layers;
    P.max_cands = c.max_cands;
    P.max_holes = c.max_holes;
    P.hole_always = (c.flags & MKF_HOLE_ALWAYS) ? 1 : 0;
    P.update3d = (c.flags & MKF_UPDATE_3D) ? 1 : 0;
    P.geo = (c.layer_kind[0] == 1 ? 1 : 0) | (c.layer_thickness[0] > 0.0 || P.update3d ? 2 : 0);
    P.bins_phi = t.bins_phi;
    P.bins_z = t.bins_z;
    P.w_per_qpt = (float)(-0.00299792458 * c.bz);
    P.var_u = (float)(c.sigma_rphi * c.sigma_rphi);
    P.var_z = (float)(c.sigma_z * c.sigma_z);
    P.var_r = (float)(c.sigma_r * c.sigma_r);
    P.chi2_cut = (float)c.chi2_cut;
    P.mass2 = (float)(c.mass * c.mass);
    P.win_scale = 1.05f;
}

mkf_status check_config(const mkf_config *c)
{
    if (!c) return fail(MKF_E_INVALID, "config is NULL");
    if (c->n_seed_layers < 1 || c->n_layers <= c->n_seed_layers || c->n_layers > kMaxLayers)
        return fail(MKF_E_INVALID, "need 1 <= n_seed_layers < n_layers <= %d", kMaxLayers);
    if (c->max_cands < 1 || c->max_cands > kMaxCands) return fail(MKF_E_INVALID, "max_cands must be 1..%d", kMaxCands);
    if (c->max_holes < 0 || c->max_holes > 7) return fail(MKF_E_INVALID, "max_holes must be 0..7");
    if (c->flags & ~(MKF_HOLE_ALWAYS | MKF_UPDATE_3D)) return fail(MKF_E_INVALID, "unknown config flags");
    bool any_disk = false;
    for (int L = 0; L < c->n_layers; ++L) {
        const int kind = c->layer_kind[L];
        if (kind != 0 && kind != 1) return fail(MKF_E_INVALID, "layer_kind must be 0 (cylinder) or 1 (disk)");
        if (!(c->layer_r[L] > 0) || !std::isfinite(c->layer_r[L])) return fail(MKF_E_INVALID, "layer_r must be positive");
        if (kind == 0) {
            if (L > 0 && c->layer_kind[L - 1] == 0 && !(c->layer_r[L] > c->layer_r[L - 1]))
                return fail(MKF_E_INVALID, "consecutive cylinder radii must increase");
            if (!(c->layer_half_z[L] > 0) || !std::isfinite(c->layer_half_z[L]))
                return fail(MKF_E_INVALID, "layer_half_z must be positive");
        } else {
            any_disk = true;
            if (!std::isfinite(c->layer_z[L]) || c->layer_z[L] == 0.0)
                return fail(MKF_E_INVALID, "a disk needs a finite nonzero layer_z");
            if (!(c->layer_rmin[L] >= 0) || !(c->layer_rmin[L] < c->layer_r[L]))
                return fail(MKF_E_INVALID, "a disk needs 0 <= layer_rmin < layer_r");
        }
        if (!(c->layer_x0[L] >= 0) || !std::isfinite(c->layer_x0[L])) return fail(MKF_E_INVALID, "layer_x0 must be >= 0");
    }
    if ((any_disk || (c->flags & MKF_UPDATE_3D)) && (!(c->sigma_r > 0) || !std::isfinite(c->sigma_r)))
        return fail(MKF_E_INVALID, "sigma_r must be positive with a disk or the 3x3 measurement");
    for (int L = 1; L < c->n_layers; ++L)
        if (c->layer_kind[L] != c->layer_kind[0])
            return fail(MKF_E_INVALID, "layers must be all cylinders or all disks (mixed lists are not supported)");
    for (int L = 0; L < c->n_layers; ++L) {
        const double t = c->layer_thickness[L];
        if (!(t >= 0.0) || !std::isfinite(t)) return fail(MKF_E_INVALID, "layer_thickness must be >= 0");
        if ((t > 0.0) != (c->layer_thickness[0] > 0.0))
            return fail(MKF_E_INVALID, "layers must be all thin or all thick (mixed lists are not supported)");
        const double ref = c->layer_kind[L] == 0 ? c->layer_r[L] : std::fabs(c->layer_z[L]);
        if (!(0.5 * t < ref)) return fail(MKF_E_INVALID, "layer_thickness must be below twice the layer's r or |z|");
    }
    if (!std::isfinite(c->bz)) return fail(MKF_E_INVALID, "bz must be finite");
    if (!(c->sigma_rphi > 0) || !(c->sigma_z > 0) || !std::isfinite(c->sigma_rphi) || !std::isfinite(c->sigma_z))
        return fail(MKF_E_INVALID, "hit resolutions must be positive");
    if (!(c->chi2_cut > 0) || !std::isfinite(c->chi2_cut)) return fail(MKF_E_INVALID, "chi2_cut must be positive");
    if (!(c->mass >= 0) || !std::isfinite(c->mass)) return fail(MKF_E_INVALID, "mass must be >= 0");
    return MKF_OK;
}

mkf_status check_tuning(const mkf_config &c, mkf_tuning *t)
{
    static const int kLanes[] = {1, 2, 4, 6, 8};
    if (t->lanes_per_seed == 0) {
        for (int g : kLanes)
            if (g >= c.max_cands) {
                t->lanes_per_seed = g;
                break;
            }
    }
    const int G = t->lanes_per_seed;
    if (G != 1 && G != 2 && G != 4 && G != 6 && G != 8)
        return fail(MKF_E_INVALID, "lanes_per_seed must be 1, 2, 4, 6 or 8");
    if (G < c.max_cands) return fail(MKF_E_INVALID, "lanes_per_seed must be >= max_cands");
    if (t->waves_per_block == 0) t->waves_per_block = 1;
    if (t->waves_per_block < 1 || t->waves_per_block > 4) return fail(MKF_E_INVALID, "waves_per_block must be 1..4");
    if (t->bins_phi == 0) t->bins_phi = 2048;
    if (t->bins_z == 0) t->bins_z = 32;
    if (t->bins_phi < 1 || t->bins_phi > 4096 || t->bins_z < 1 || t->bins_z > 1024 ||
        (long long)t->bins_phi * t->bins_z > (1 << 20))
        return fail(MKF_E_INVALID, "bins out of range (phi 1..4096, z 1..1024, product <= 2^20)");
    if (t->persistent != 0 && t->persistent != 1) return fail(MKF_E_INVALID, "persistent must be 0 or 1");
    if (t->blocks_per_cu == 0) t->blocks_per_cu = 4;
    if (t->blocks_per_cu < 1 || t->blocks_per_cu > 32) return fail(MKF_E_INVALID, "blocks_per_cu must be 1..32");
    return MKF_OK;
}

void timers_collect(mkf_ctx *ctx, bool wait);

// Opens an interval; returns where its start stamp goes (null: not timed, as
// under a capture by the caller: the launches do not run now, and replays of
// them would stamp the ring's words while other calls use them).
unsigned long long *timer_open(mkf_ctx *ctx, int which, hipStream_t s)
{
    Timer &t = ctx->timers[which];
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (s != ctx->stream || hipStreamIsCapturing(s, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone)
        return nullptr;
    if (t.count == Timer::kRing) timers_collect(ctx, true);
    const int slot = (t.head + t.count) % Timer::kRing;
    t.start[slot] = t.stop[slot] = 0;
    t.open = true;
    return t.start + slot;
}

unsigned long long *timer_close(mkf_ctx *ctx, int which, hipStream_t s, long long launches)
{
    Timer &t = ctx->timers[which];
    if (s != ctx->stream || !t.open) return nullptr;
    const int slot = (t.head + t.count) % Timer::kRing;
    t.ring_launches[slot] = launches;
    ++t.count;
    t.open = false;
    return t.stop + slot;
}

// The stamp due, for a launch that writes it; stamp_now() for where none will.
Stamp take_stamp(mkf_ctx *ctx)
{
    const Stamp st = ctx->stamp_due;
    ctx->stamp_due = Stamp{};
    return st;
}

void stamp_now(mkf_ctx *ctx) { (void)launch_stamp(take_stamp(ctx), ctx->stream); }

void timer_begin(mkf_ctx *ctx, int which, hipStream_t s)
{
    stamp_now(ctx);
    ctx->stamp_due.a = timer_open(ctx, which, s);
}

void timer_end(mkf_ctx *ctx, int which, hipStream_t s, long long launches)
{
    stamp_now(ctx);
    ctx->stamp_due.a = timer_close(ctx, which, s, launches);
}

// one phase ends, another begins
void timer_switch(mkf_ctx *ctx, int from, int to, hipStream_t s, long long launches)
{
    stamp_now(ctx);
    unsigned long long *b = timer_open(ctx, to, s);   // first: it may collect
    unsigned long long *a = timer_close(ctx, from, s, launches);
    if (a) ctx->stamp_due = Stamp{a, b};
    else ctx->stamp_due.a = b;
}

// Adds the recorded intervals to the totals: all of them (waiting for the
// device) or only those already complete.
void timers_collect(mkf_ctx *ctx, bool wait)
{
    bool waited = false;
    for (auto &t : ctx->timers) {
        while (t.count > 0) {
            const int slot = t.head;
            if (wait && !waited) {
                (void)hipStreamSynchronize(ctx->stream);
                waited = true;
            }
            const unsigned long long a = __atomic_load_n(t.start + slot, __ATOMIC_RELAXED);
            const unsigned long long b = __atomic_load_n(t.stop + slot, __ATOMIC_RELAXED);
            if (b == 0 && !wait) break;
            if (a != 0 && b > a) {
                t.total_ms += (double)(b - a) * ctx->ms_per_tick;
                t.launches += t.ring_launches[slot];
            }
            t.head = (t.head + 1) % Timer::kRing;
            --t.count;
        }
    }
}

EventRec *find_event(mkf_ctx *ctx, int32_t h)
{
    auto it = ctx->events.find(h);
    return it == ctx->events.end() ? nullptr : it->second.get();
}

void drop_graphs_with(mkf_ctx *ctx, int32_t handle)
{
    auto &g = ctx->graphs;
    for (size_t i = 0; i < g.size();) {
        const bool hit = handle < 0 || std::find(g[i]->handles.begin(), g[i]->handles.end(), handle) != g[i]->handles.end();
        if (hit) {
            (void)hipStreamSynchronize(ctx->stream);   // a queued replay may still use its scratch
            (void)hipGraphExecDestroy(g[i]->exec);
            ctx->heap.release(g[i]->scratch);
            g.erase(g.begin() + i);
        } else {
            ++i;
        }
    }
}

void drop_plain_graph(EventRec *rec)
{
    if (rec->plain_graph) (void)hipGraphExecDestroy(rec->plain_graph);
    rec->plain_graph = nullptr;
}

mkf_status upload_view(EventRec *rec, hipStream_t s)
{
    MKF_HIP(hipMemcpyAsync(rec->dev_view, &rec->view, sizeof(DevEvent), hipMemcpyHostToDevice, s));
    MKF_HIP(hipStreamSynchronize(s));
    return MKF_OK;
}

mkf_status ensure_batch_scratch(mkf_ctx *ctx, int n)
{
    const size_t need = batch_scratch_bytes(n);
    if (ctx->batch_dev_bytes < need || ctx->batch_host_bytes < need) {
        MKF_HIP(hipStreamSynchronize(ctx->stream));   // queued work may still read the buffers
        ctx->stage_pending = false;
        ctx->staged_image.clear();
    }
    if (ctx->batch_dev_bytes < need) {
        ctx->heap.release(ctx->batch_dev);
        ctx->batch_dev = ctx->heap.alloc(need);
        ctx->batch_dev_bytes = ctx->batch_dev ? need : 0;
        if (!ctx->batch_dev) return fail(MKF_E_NOMEM, "batch scratch of %zu bytes", need);
    }
    if (ctx->batch_host_bytes < need) {
        if (ctx->batch_host) (void)hipHostFree(ctx->batch_host);
        ctx->batch_host = nullptr;
        ctx->batch_host_bytes = 0;
        MKF_HIP(hipHostMalloc(&ctx->batch_host, need, hipHostMallocDefault));
        ctx->batch_host_bytes = need;
    }
    return MKF_OK;
}

mkf_status gather_events(mkf_ctx *ctx, const int32_t *handles, int32_t n, std::vector<EventRec *> *recs)
{
    if (n < 0 || (n > 0 && !handles)) return fail(MKF_E_INVALID, "bad handle list");
    if ((long long)n * ctx->cfg.n_layers > 65535)
        return fail(MKF_E_INVALID, "at most %d events per batch", 65535 / ctx->cfg.n_layers);
    std::vector<int32_t> seen(handles, handles + n);
    std::sort(seen.begin(), seen.end());
    if (std::adjacent_find(seen.begin(), seen.end()) != seen.end())
        return fail(MKF_E_INVALID, "an event appears twice in the batch");
    recs->clear();
    for (int i = 0; i < n; ++i) {
        EventRec *r = find_event(ctx, handles[i]);
        if (!r) return fail(MKF_E_NOTFOUND, "unknown event handle %d", handles[i]);
        recs->push_back(r);
    }
    return MKF_OK;
}

}  // namespace

size_t event_data_bytes(const EventShape &s)
{
    DevEvent v{};
    return carve_data(s, nullptr, &v, nullptr);
}

int pack_threads(size_t n_values, size_t per_thread)
{
    const unsigned hw = std::max(1u, std::thread::hardware_concurrency());
    return (int)std::min<size_t>({(size_t)16, (size_t)hw, 1 + n_values / per_thread});
}

void touch_pages(const void *p, size_t bytes)
{
    constexpr size_t kPage = 4096, kTask = 16 * kPage;   // 22 us; a thread takes 30 to 50 us to wake
    const volatile char *at = static_cast<const volatile char *>(p);
    const size_t tasks = (bytes + kTask - 1) / kTask;
    const unsigned hw = std::max(1u, std::thread::hardware_concurrency());
    run_tasks((int)tasks, (int)std::min<size_t>({(size_t)16, (size_t)hw, (tasks + 1) / 2}), [=](int t) {
        for (size_t i = t * kTask; i < std::min(bytes, (t + 1) * kTask); i += kPage) (void)at[i];
    });
}

// the hits, at the front of the inputs, up to where the seeds begin
size_t event_hit_bytes(const EventShape &s) { return round_up_256(sizeof(float4) * (size_t)s.n_hits()); }

size_t event_view_offset(const EventShape &s)
{
    DevEvent v{};
    DevEvent *dv = nullptr;
    char origin = 0;   // only offsets from it are taken
    carve_data(s, &origin, &v, &dv);
    return reinterpret_cast<char *>(dv) - &origin;
}

size_t event_input_bytes(const EventShape &s)
{
    DevEvent v{};
    size_t end = 0;
    carve_data(s, nullptr, &v, nullptr, &end);
    return end;
}

size_t event_budget_bytes(const EventShape &s, int nb)
{
    const size_t off = sizeof(int) * (size_t)s.n_layers * bin_off_stride(nb);
    return round_up_256(event_data_bytes(s)) + round_up_256(off) + round_up_256(index_allowance(s, nb));
}

size_t batch_scratch_bytes(int n)
{
    size_t b = ((size_t)n * sizeof(DevEvent) + 255) & ~size_t(255);
    b += 4 * (((size_t)(n + 1) * sizeof(int) + 255) & ~size_t(255));
    return b + 256;
}

int resolve_lanes(const mkf_ctx *ctx) { return ctx->tuning.lanes_per_seed; }
int seeds_per_item(int geo, int G, long long seeds)
{
    const int most = kWave / G, resident = geo & 2 ? 1024 : 4096;
    const long long want = std::max<long long>({(seeds + resident - 1) / resident, 5, (10 + G - 1) / G});
    for (int spi : {5, 8, 10, 16, 20, 32, 40, 64})
        if (spi >= want && spi < most) return spi;
    return most;
}

int seeds_per_item(int geo, int G, EventRec *const *recs, int n)
{
    long long seeds = 0;
    for (int i = 0; i < n; ++i) seeds += recs[i]->shape.n_seeds;
    return seeds_per_item(geo, G, seeds);
}

// ---------------------------------------------------------------- events

// Counts and pointers of an event: its shape.  The values are checked while
// they are packed (pack_event).
mkf_status validate_event(const mkf_ctx *ctx, const mkf_event *ev, EventShape *shape)
{
    const mkf_config &c = ctx->cfg;
    if (!ev) return fail(MKF_E_INVALID, "event is NULL");
    if (ev->n_layers != c.n_layers) return fail(MKF_E_INVALID, "event has %d layers, config %d", ev->n_layers, c.n_layers);
    if (ev->n_seeds < 0 || ev->n_tracks < 0) return fail(MKF_E_INVALID, "negative seed or track count");
    if (!ev->n_hits || !ev->hit_xyz) return fail(MKF_E_INVALID, "n_hits / hit_xyz is NULL");
    EventShape s;
    s.n_layers = c.n_layers;
    s.n_seed_layers = c.n_seed_layers;
    s.n_seeds = ev->n_seeds;
    s.n_tracks = ev->n_tracks;
    long long tot = 0;
    for (int L = 0; L < c.n_layers; ++L) {
        const int n = ev->n_hits[L];
        if (n < 0 || n > kMaxHitsPerLayer) return fail(MKF_E_INVALID, "layer %d: %d hits out of range", L, n);
        if (n > 0 && !ev->hit_xyz[L]) return fail(MKF_E_INVALID, "layer %d: hit_xyz is NULL", L);
        s.layer_off[L] = (int)tot;
        tot += n;
        if (tot > (1LL << 30)) return fail(MKF_E_INVALID, "too many hits in one event");
    }
    s.layer_off[c.n_layers] = (int)tot;
    if (ev->n_seeds > 0 && (!ev->seed_par || !ev->seed_cov || !ev->seed_hits))
        return fail(MKF_E_INVALID, "seed arrays are NULL");
    if (ev->n_tracks > 0 && (!ev->track_par || !ev->track_cov || !ev->track_hits))
        return fail(MKF_E_INVALID, "track arrays are NULL");
    *shape = s;
    return MKF_OK;
}

// Writes the FP32 states, covariances and hit indices of n seeds or tracks
// (n_hit_layers indices a row) and checks them: finite, theta in (0, pi), off
// the axis, indices in range.  -1, or the first row that fails, *bad_hit set
// when by a hit index.
static long long pack_states(const double *par, const double *cov, const int32_t *hits, size_t n, int n_hit_layers,
                             const int32_t *n_hits, float *fpar, float *fcov, int *ohits, int *bad_hit)
{
    bool ok = narrow_all(par, fpar, 6 * n) & narrow_all(cov, fcov, 21 * n) & states_in_range(par, n);
    int out = 0;
    for (size_t i = 0; i < n; ++i)
        for (int L = 0; L < n_hit_layers; ++L) {
            const int32_t h = hits[i * n_hit_layers + L];
            out |= (h < -1) | (h >= n_hits[L]);
            ohits[i * n_hit_layers + L] = h;
        }
    if (ok && !out) return -1;
    for (size_t i = 0; i < n; ++i) {   // the first that failed
        if (!narrow_all(par + 6 * i, fpar + 6 * i, 6) || !narrow_all(cov + 21 * i, fcov + 21 * i, 21) ||
            !states_in_range(par + 6 * i, 1))
            return (long long)i;
        for (int L = 0; L < n_hit_layers; ++L) {
            const int32_t h = hits[i * n_hit_layers + L];
            if (h < -1 || h >= n_hits[L]) {
                *bad_hit = 1;
                return (long long)i;
            }
        }
    }
    return 0;   // what was refused once stays refused, whatever a second look says
}

// Packs an event's inputs into `image` in the device layout of its data
// block (carve_data) and checks every value on the way: each hit becomes
// the FP32 form the kernels read (geo: bit 0 disks, bit 1 layers of finite
// thickness or the 3x3 measurement), computed in FP64; seeds and tracks
// FP32 states and covariances, finite, theta in (0, pi), hit indices in
// range.  The layers and the seeds are packed in parallel for large events.
// The seeds of each block of rows in order of the azimuth of their direction: a counting sort over
// 1024 sectors that keeps the caller's order within a sector.  The batched
// builder takes the seeds of one wavefront, and of the wavefronts that run
// together, from neighbouring sectors, so the hits and bins their windows read
// are shared in cache instead of each wavefront reading a different part of
// every layer.  The outputs stay in the caller's order.
constexpr int kSeedSectors = 1024;

static inline uint16_t seed_sector(double phi)
{
    const double x = (phi + M_PI) * (kSeedSectors / (2 * M_PI));
    return (uint16_t)(x >= 0.0 ? (x < kSeedSectors ? (int)x : kSeedSectors - 1) : 0);   // NaN: sector 0
}

static void order_seeds(const std::vector<uint16_t> &sector, int *order)
{
    for (int b0 = 0; b0 < (int)sector.size(); b0 += kSeedBlock) {
        const int b1 = std::min((int)sector.size(), b0 + kSeedBlock);
        int start[kSeedSectors + 1] = {0};
        for (int i = b0; i < b1; ++i) ++start[sector[i] + 1];
        start[0] = b0;
        for (int k = 0; k < kSeedSectors; ++k) start[k + 1] += start[k];
        for (int i = b0; i < b1; ++i) order[start[sector[i]]++] = i;
    }
}

mkf_status pack_event(const mkf_event *ev, const EventShape &sh, int geo, void *image, int threads, std::string *why,
                      PackPart part)
{
    DevEvent v{};
    carve_data(sh, image, &v, nullptr);
    const int nsl = sh.n_seed_layers;
    const int nl = part == PackPart::kRows ? 0 : sh.n_layers;   // layers packed by this call
    const bool rows = part != PackPart::kHits;
    const int chunk = 4096;
    const int seed_tasks = rows ? (sh.n_seeds + chunk - 1) / chunk : 0;
    const int track_tasks = rows ? (sh.n_tracks + chunk - 1) / chunk : 0;
    const int n_tasks = nl + seed_tasks + track_tasks;
    if (rows) std::memset(v.stats, 0, 5 * sizeof(*v.stats));
    const HitForm form = geo & 2 ? HitForm::kXyz : geo & 1 ? HitForm::kDisk : HitForm::kCylinder;
    // first failure of each task: (index, kind), index -1 for none
    std::vector<int> bad(n_tasks, -1), kind(n_tasks, 0);
    std::vector<uint16_t> sector(rows ? sh.n_seeds : 0);   // azimuth sector of each seed, taken while it is packed
    run_tasks(n_tasks, threads, [&](int t) {
        if (t < nl) {
            // a hit as the kernels read it: its direction and second grid
            // coordinate computed here in FP64 and rounded once
            const size_t n = (size_t)ev->n_hits[t];
            float *o = reinterpret_cast<float *>(const_cast<float4 *>(v.hits) + sh.layer_off[t]);
            if (pack_hits(ev->hit_xyz[t], n, form, o)) return;
            bad[t] = 0;   // what was refused once stays refused, whatever a second look says
            for (size_t i = 0; i < n; ++i)   // the first that failed
                if (!pack_hits(ev->hit_xyz[t] + 3 * i, 1, form, o + 4 * i)) {
                    bad[t] = (int)i;
                    break;
                }
            return;
        }
        const bool seeds = t < nl + seed_tasks;
        const size_t i0 = (size_t)(seeds ? t - nl : t - nl - seed_tasks) * chunk;
        const size_t n = std::min<size_t>(chunk, (seeds ? sh.n_seeds : sh.n_tracks) - i0);
        const int nh = seeds ? nsl : sh.n_layers;   // hit indices of a row
        const double *par = (seeds ? ev->seed_par : ev->track_par) + 6 * i0;
        const double *cov = (seeds ? ev->seed_cov : ev->track_cov) + 21 * i0;
        const int32_t *hits = (seeds ? ev->seed_hits : ev->track_hits) + nh * i0;
        float *fpar = const_cast<float *>(seeds ? v.seed_par : v.track_par) + 6 * i0;
        float *fcov = const_cast<float *>(seeds ? v.seed_cov : v.track_cov) + 21 * i0;
        int *ohits = const_cast<int *>(seeds ? v.seed_hits : v.track_hits) + nh * i0;
        int bad_hit = 0;
        const long long failed = pack_states(par, cov, hits, n, nh, ev->n_hits, fpar, fcov, ohits, &bad_hit);
        if (failed >= 0) {
            bad[t] = (int)(i0 + failed);
            kind[t] = bad_hit;
            return;
        }
        if (seeds)
            for (size_t i = 0; i < n; ++i) sector[i0 + i] = seed_sector(par[6 * i + 4]);
    });
    for (int t = 0; t < n_tasks; ++t) {
        if (bad[t] < 0) continue;
        char msg[200];
        if (t < nl) {
            std::snprintf(msg, sizeof(msg), "layer %d hit %d: not finite (in FP32) or on the axis", t, bad[t]);
        } else {
            const char *what = t < nl + seed_tasks ? "seed" : "track";
            if (kind[t]) std::snprintf(msg, sizeof(msg), "%s %d: hit index out of range", what, bad[t]);
            else std::snprintf(msg, sizeof(msg), "%s %d: state or covariance not finite (in FP32), theta outside "
                                                 "(0, pi) or position on the axis", what, bad[t]);
        }
        *why = msg;
        return MKF_E_INVALID;
    }
    if (rows) order_seeds(sector, const_cast<int *>(v.seed_order));
    return MKF_OK;
}

mkf_status create_event(mkf_ctx *ctx, const EventShape &shape, DeviceHeap *heap, std::unique_ptr<EventRec> *out)
{
    auto rec = std::make_unique<EventRec>();
    rec->shape = shape;
    rec->heap = heap;
    const size_t bytes = event_data_bytes(shape);
    rec->data = heap->alloc(bytes);
    if (!rec->data) return fail(MKF_E_NOMEM, "event data: %zu bytes", bytes);
    DevEvent &v = rec->view;
    std::memset(&v, 0, sizeof(v));
    carve_data(shape, rec->data, &v, &rec->dev_view);
    v.n_layers = shape.n_layers;
    v.n_seeds = shape.n_seeds;
    v.n_tracks = shape.n_tracks;
    v.n_hits = shape.n_hits();
    for (int L = 0; L <= shape.n_layers; ++L) v.layer_off[L] = shape.layer_off[L];
    (void)ctx;
    *out = std::move(rec);
    return MKF_OK;
}

// Copies an event's packed inputs (pack_event) and its descriptor, now that
// its addresses are known, into its device data block.
mkf_status upload_packed(EventRec *rec, void *image, hipStream_t s)
{
    std::memcpy(static_cast<char *>(image) + event_view_offset(rec->shape), &rec->view, sizeof(DevEvent));
    MKF_HIP(hipMemcpyAsync(rec->data, image, event_input_bytes(rec->shape), hipMemcpyHostToDevice, s));
    return MKF_OK;
}

void destroy_event(mkf_ctx *ctx, EventRec *rec)
{
    (void)ctx;
    drop_plain_graph(rec);
    rec->heap->release(rec->plain);
    rec->heap->release(rec->index);
    rec->heap->release(rec->data);
    rec->heap->release(rec->beam);
    rec->plain = rec->index = rec->data = rec->beam = nullptr;
}

// Storage for every rank of the final beam of an event (max_cands per seed).
mkf_status ensure_beam(mkf_ctx *ctx, EventRec *rec)
{
    if (rec->beam) return MKF_OK;
    const size_t n = (size_t)rec->shape.n_seeds * ctx->cfg.max_cands, nl = (size_t)rec->shape.n_layers;
    auto carve = [&](void *base) {
        Carver c(base);
        DevEvent &v = rec->beam_view;
        v.beam_rec = c.take<float>(kRecWords * n);
        v.beam_hits = c.take<int>(nl * n);
        return c.off;
    };
    const size_t bytes = carve(nullptr);
    rec->beam = rec->heap->alloc(bytes);
    if (!rec->beam) return fail(MKF_E_NOMEM, "final beam: %zu bytes", bytes);
    carve(rec->beam);
    return MKF_OK;
}

// Make sure the event's index tables match the current bin grid.  *rebuilt is
// set when the tables were (re)allocated and the index must be built.
mkf_status ensure_index(mkf_ctx *ctx, EventRec *rec, bool *rebuilt, hipStream_t s)
{
    return ensure_index_grid(ctx, rec, ctx->tuning.bins_phi, ctx->tuning.bins_z, rebuilt, s);
}

int max_layer_hits(const EventShape &s)
{
    int m = 0;
    for (int L = 0; L < s.n_layers; ++L) m = std::max(m, s.layer_off[L + 1] - s.layer_off[L]);
    return m;
}

int event_bins(const EventShape &s, int bins_phi, int bins_z)
{
    const int k = event_grid_shift(max_layer_hits(s), bins_phi, bins_z);
    return (bins_phi >> k) * (bins_z >> k);
}

mkf_status ensure_index_grid(mkf_ctx *ctx, EventRec *rec, int bp, int bz, bool *rebuilt, hipStream_t s)
{
    *rebuilt = false;
    if (rec->index && rec->index_bins_phi == bp && rec->index_bins_z == bz) return MKF_OK;
    if (rec->index) MKF_HIP(hipStreamSynchronize(ctx->stream));   // queued builds may still read it
    rec->heap->release(rec->index);
    // the event's own grid: the context's, coarsened for a small event
    const int k = event_grid_shift(max_layer_hits(rec->shape), bp, bz);
    const int nb = (bp >> k) * (bz >> k);
    const bool served = rec->heap != &ctx->heap;   // in the budget's slab
    bool work = wants_index_work(rec->shape, nb, served);
    DevEvent sized{};
    size_t bytes = carve_index(rec->shape, nb, work, nullptr, &sized);
    rec->index = rec->heap->alloc(bytes);
    if (!rec->index && work) {
        work = false;
        bytes = carve_index(rec->shape, nb, work, nullptr, &sized);
        rec->index = rec->heap->alloc(bytes);
    }
    if (!rec->index) {
        rec->index_bins_phi = rec->index_bins_z = 0;
        return fail(MKF_E_NOMEM, "hit index: %zu bytes", bytes);
    }
    carve_index(rec->shape, nb, work, rec->index, &rec->view);
    rec->view.grid_k = k;
    rec->index_bins_phi = bp;
    rec->index_bins_z = bz;
    drop_plain_graph(rec);
    *rebuilt = true;
    return MKF_OK;
}

// Lays out the batch descriptors of recs[0..n) - the event views, the work,
// hit, track and seed prefixes and the work-queue counter - into `image`
// (batch_scratch_bytes(n) bytes, all written) and points `args` at the same
// layout starting at device address `dev`.  Allocates nothing.
mkf_status compose_batch(EventRec *const *recs, int n, int spi, bool beam, char *image, char *dev, BatchArgs *args)
{
    size_t off = 0;
    auto place = [&](size_t bytes) {
        const size_t o = off;
        off = (off + bytes + 255) & ~size_t(255);
        return o;
    };
    const size_t o_ev = place((size_t)n * sizeof(DevEvent));
    const size_t o_item = place((size_t)(n + 1) * sizeof(int));
    const size_t o_hit = place((size_t)(n + 1) * sizeof(int));
    const size_t o_trk = place((size_t)(n + 1) * sizeof(int));
    const size_t o_seed = place((size_t)(n + 1) * sizeof(int));
    const size_t o_q = place(sizeof(unsigned));
    std::memset(image, 0, off);
    char *h = image;
    DevEvent *ev = reinterpret_cast<DevEvent *>(h + o_ev);
    int *ip = reinterpret_cast<int *>(h + o_item);
    int *hp = reinterpret_cast<int *>(h + o_hit);
    int *tp = reinterpret_cast<int *>(h + o_trk);
    int *sp = reinterpret_cast<int *>(h + o_seed);
    long long items = 0, hits = 0, trks = 0, seeds = 0;
    IndexExtent all{}, layer_only{};
    int max_chunks = 0, max_shift = 0;
    for (int i = 0; i < n; ++i) {
        const EventShape &sh = recs[i]->shape;
        const int k = recs[i]->view.grid_k;
        const int bins = (recs[i]->index_bins_phi >> k) * (recs[i]->index_bins_z >> k);
        all.add(max_layer_hits(sh), bins);
        if (recs[i]->view.part) {
            max_chunks = std::max(max_chunks, recs[i]->view.idx_chunks);
            max_shift = std::max(max_shift, recs[i]->view.bucket_shift);
        } else {
            layer_only.add(max_layer_hits(sh), bins);
        }
        ev[i] = recs[i]->view;
        if (beam) {   // this launch also writes every rank of the final beam
            const DevEvent &b = recs[i]->beam_view;
            ev[i].beam_rec = b.beam_rec;
            ev[i].beam_hits = b.beam_hits;
        }
        ip[i] = (int)items;
        hp[i] = (int)hits;
        tp[i] = (int)trks;
        sp[i] = (int)seeds;
        seeds += recs[i]->shape.n_seeds;
        items += (recs[i]->shape.n_seeds + spi - 1) / spi;
        hits += recs[i]->shape.n_hits();
        trks += recs[i]->shape.n_tracks;
    }
    if (items > INT32_MAX || hits > INT32_MAX || trks > INT32_MAX || seeds > INT32_MAX)
        return fail(MKF_E_INVALID, "batch too large");
    ip[n] = (int)items;
    hp[n] = (int)hits;
    tp[n] = (int)trks;
    sp[n] = (int)seeds;
    args->events = reinterpret_cast<const DevEvent *>(dev + o_ev);
    args->item_prefix = reinterpret_cast<const int *>(dev + o_item);
    args->hit_prefix = reinterpret_cast<const int *>(dev + o_hit);
    args->track_prefix = reinterpret_cast<const int *>(dev + o_trk);
    args->seed_prefix = reinterpret_cast<const int *>(dev + o_seed);
    args->queue = reinterpret_cast<unsigned *>(dev + o_q);
    args->n_events = n;
    args->total_items = (int)items;
    args->total_hits = (int)hits;
    args->total_tracks = (int)trks;
    args->total_seeds = (int)seeds;
    args->seeds_per_item = spi;
    args->first_item = 0;
    args->end_item = (int)items;
    args->all = all;
    args->layer_only = layer_only;
    args->max_chunks = max_chunks;
    args->max_bucket_shift = max_shift;
    return MKF_OK;
}

mkf_status stage_batch(mkf_ctx *ctx, const std::vector<EventRec *> &recs, void *dev, void *host, int spi,
                       BatchArgs *args, hipStream_t s, bool beam)
{
    const int n = (int)recs.size();
    std::vector<char> image(batch_scratch_bytes(n));
    mkf_status st = compose_batch(recs.data(), n, spi, beam, image.data(), static_cast<char *>(dev), args);
    if (st != MKF_OK) return st;
    // The context's own buffer keeps the last image: an identical batch (same
    // events, views and tuning) is not copied again.  Its pinned staging
    // buffer is rewritten only once the previous copy out of it has run.
    const bool own = dev == ctx->batch_dev;
    if (!own || image != ctx->staged_image) {
        if (host == ctx->batch_host && ctx->stage_pending) {
            MKF_HIP(hipEventSynchronize(ctx->stage_done));
            ctx->stage_pending = false;
        }
        std::memcpy(host, image.data(), image.size());
        MKF_HIP(hipMemcpyAsync(dev, host, image.size(), hipMemcpyHostToDevice, s));
        if (host == ctx->batch_host) {
            MKF_HIP(hipEventRecord(ctx->stage_done, s));
            ctx->stage_pending = true;
        }
        if (own) ctx->staged_image.swap(image);
    }
    return MKF_OK;
}

size_t field_bytes(int f, int n_layers)
{
    const size_t b[kOutFields] = {48, 168, 8, 4 * (size_t)n_layers, 4, 4, 4, 4};
    return b[f];
}

void *field_of(const mkf_tracks &t, int f)
{
    void *const p[kOutFields] = {t.par, t.cov, t.chi2, t.hits, t.n_hits, t.n_holes, t.ndof, t.status};
    return p[f];
}

void set_field(DeliverJob &j, int f, void *p)
{
    switch (f) {
    case 0: j.par = static_cast<double *>(p); break;
    case 1: j.cov = static_cast<double *>(p); break;
    case 2: j.chi2 = static_cast<double *>(p); break;
    case 3: j.hits_out = static_cast<int *>(p); break;
    case 4: j.n_hits = static_cast<int *>(p); break;
    case 5: j.n_holes = static_cast<int *>(p); break;
    case 6: j.ndof = static_cast<int *>(p); break;
    default: j.status = static_cast<int *>(p); break;
    }
}

void *device_writable(void *p, size_t bytes, size_t align, int device, char **host, size_t *range, char **dev)
{
    if (reinterpret_cast<uintptr_t>(p) % align) return nullptr;
    hipPointerAttribute_t a{};
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    if (!a.devicePointer || !(a.type == hipMemoryTypeHost || (a.type == hipMemoryTypeDevice && a.device == device)))
        return nullptr;
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipMemGetAddressRange(&base, &size, a.devicePointer) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    const size_t off = static_cast<char *>(a.devicePointer) - static_cast<char *>(base);
    if (off > size || bytes > size - off) return nullptr;
    if (host) {   // the whole allocation
        *host = static_cast<char *>(p) - off;
        *dev = static_cast<char *>(base);
        *range = size;
    }
    return a.devicePointer;
}

// Page-locked staging of at least `bytes` (contents undefined when it grows).
static mkf_status ensure_pin(mkf_ctx *ctx, size_t bytes)
{
    if (ctx->load_pin_bytes >= bytes) return MKF_OK;
    MKF_HIP(hipStreamSynchronize(ctx->stream));   // a queued copy may still read it
    if (ctx->load_pin) (void)hipHostFree(ctx->load_pin);
    ctx->load_pin = nullptr;
    ctx->load_pin_bytes = 0;
    MKF_HIP(hipHostMalloc(&ctx->load_pin, bytes, hipHostMallocDefault));
    ctx->load_pin_bytes = bytes;
    return MKF_OK;
}

// Staging for `bytes` of `sets` sets of rows with the padding of their fields,
// in however many slots.
static size_t out_need_bytes(size_t bytes, size_t sets) { return bytes + 256 * kOutFields * (sets + 2 * kOutSlots); }

// Staging that lets `rows` result rows of `sets` events leave without another
// allocation.
static size_t out_pin_bytes(size_t rows, size_t sets, int n_layers)
{
    size_t row = 0;
    for (int f = 0; f < kOutFields; ++f) row += field_bytes(f, n_layers);
    return std::min(kOutSlots * kOutSlotMax, out_need_bytes(row * rows, sets));
}

// Result rows to the caller's arrays by launches of k_deliver on the
// context's stream: add() everything, then finish(), which waits for the
// stream.  A batched build calls place() for the rows of each of its parts as
// it launches them and carries the pending ones in its next launch.  The
// staging is copied from by one thread: waking the packing
// threads for it took longer than they saved (event of 7,001 tracks 423 us
// with 8 threads, 389 with one; fitted tracks of 8 x 5,000: 1,023 and 809).
class Delivery {
  public:
    // fixed: no allocation, whatever staging the context has is used (a load of
    // small events leaves less than a tile's: then the kOutLeast made with the
    // context)
    explicit Delivery(mkf_ctx *ctx, bool fixed = false) : ctx_(ctx), fixed_(fixed)
    {
        args_.n_jobs = args_.n_tiles = 0;
        args_.n_layers = ctx->cfg.n_layers;
    }
    // an early return leaves no launch pending that writes the caller's arrays
    ~Delivery()
    {
        if (!finished_) (void)hipStreamSynchronize(ctx_->stream);
    }

    void add(const OutRows &o)
    {
        if (o.n <= 0) return;
        const long long before = total_;
        total_ += o.n;
        Rows r{o, {}, 0, 0};
        bool any = false;
        const int nl = args_.n_layers;
        for (int f = 0; f < kOutFields; ++f) {
            void *p = field_of(o.out, f);
            if (!p) continue;
            any = true;
            r.direct[f] = writable(static_cast<char *>(p), field_bytes(f, nl) * o.n, f < kOutDoubles ? 8 : 4);
            if (!r.direct[f]) r.staged += field_bytes(f, nl);
        }
        if (!any) return;
        r.before = before;
        staged_ += r.staged * o.n;
        for (int f = 0; f < kOutFields; ++f)
            if (r.direct[f]) link_bytes_ += (double)field_bytes(f, nl) * o.n;
        rows_.push_back(r);
    }

    // The rows of a batch's events, added by prepare(): once the launches that
    // do not need to know of them are queued.
    void later(EventRec *const *recs, int n, const mkf_tracks *outs)
    {
        recs_ = recs;
        n_recs_ = outs ? n : 0;
        outs_ = outs;
    }
    // whether adding and preparing the rows of n events may take longer than the
    // shortest phase, an index of 9 us behind a launch of 5: the arrays of an
    // event take 0.6 us to look up.  (Where it may, a stamp in front or the
    // look-ups before the launch cost a call of 20 small events 2 of 128 us.)
    bool slow_to_prepare(size_t rows, int n) const
    {
        return n > 16 || (!fixed_ && n && out_pin_bytes(rows, n, args_.n_layers) > ctx_->load_pin_bytes);
    }
    bool slow_to_prepare() const
    {
        size_t rows = 0;
        for (int i = 0; i < n_recs_; ++i) rows += (size_t)recs_[i]->shape.n_seeds;
        return slow_to_prepare(rows, n_recs_);
    }

    // What may take the host long - looking up the arrays of many events, growing
    // the staging - before the launch whose end the delivery's will stamp, so
    // that the phase's time holds none of it.  Nothing is added afterwards.
    mkf_status prepare()
    {
        for (int i = 0; i < n_recs_; ++i)
            add(OutRows{recs_[i]->view.out_rec, recs_[i]->view.out_hits, recs_[i]->shape.n_seeds, outs_[i]});
        n_recs_ = 0;
        return begun_ ? MKF_OK : begin();
    }

    // Rows [first, end) of the rows added, in their order (after prepare()).
    mkf_status place(long long first, long long end)
    {
        mkf_status st;
        for (const Rows &r : rows_) {
            const long long a = std::max(first - r.before, 0LL), b = std::min<long long>(end - r.before, r.o.n);
            if (a < b && (st = place_rows(r, (int)a, (int)b)) != MKF_OK) return st;
        }
        placed_ = end;
        return MKF_OK;
    }

    // The jobs placed and not launched, for a launch of the caller's that
    // delivers them; launched() once it is queued.
    const DeliverArgs &pending() const { return args_; }
    void launched() { args_.n_jobs = args_.n_tiles = 0; }

    long long total_rows() const { return total_; }
    // us per row on its way out: bytes over the host link, or copied out of
    // the staging
    double us_per_row() const { return total_ ? (link_bytes_ / kLinkBytesPerUs + staged_ / kCopyBytesPerUs) / (double)total_ : 0.0; }

    mkf_status finish()
    {
        mkf_status st = prepare();
        if (st != MKF_OK || (st = place(placed_, total_)) != MKF_OK) return st;
        if ((st = launch()) != MKF_OK) return st;
        stamp_now(ctx_);   // of a phase that nothing was launched after
        if (n_slots_ > 1) {
            if ((st = mark_slot()) != MKF_OK) return st;
            for (int k = 1; k <= n_slots_; ++k)   // oldest first
                if ((st = empty(slot_[(cur_ + k) % n_slots_])) != MKF_OK) return st;
            // the last mark was the last of the stream; but arrays written
            // directly may be of a kind that only its end makes visible
            if (link_bytes_ > 0.0) MKF_HIP(hipStreamSynchronize(ctx_->stream));
        } else {
            MKF_HIP(hipStreamSynchronize(ctx_->stream));
            copy_out(slot_[0]);
        }
        finished_ = true;
        return MKF_OK;
    }

  private:
    struct Rows {
        OutRows o;
        void *direct[kOutFields];
        size_t staged;                  // bytes per row that go through the staging
        long long before;               // rows added before these
    };
    struct Slot {
        std::vector<HostCopy> copies;   // not yet made
        const unsigned *flag = nullptr; // `mark` once the device has filled the slot
        unsigned mark = 0;
    };

    mkf_status begin()
    {
        begun_ = true;
        if (!staged_) return MKF_OK;
        mkf_status st;
        const size_t need = out_need_bytes(staged_, rows_.size());
        if (!fixed_ && (st = ensure_pin(ctx_, std::min(need, kOutSlots * kOutSlotMax))) != MKF_OK) return st;
        const bool small = ctx_->load_pin_bytes < std::min(need, kOutLeast);   // only when fixed
        stage_ = small ? ctx_->least_pin : static_cast<char *>(ctx_->load_pin);
        // equal slots for everything where the staging holds it, else a ring
        const size_t have = std::min(need, small ? kOutLeast : ctx_->load_pin_bytes);
        n_slots_ = have < need ? kOutSlots : (int)std::min<size_t>(kOutSlots, std::max<size_t>(1, need / kOutSlotMin));
        if (have / n_slots_ < kOutLeast) n_slots_ = 1;
        slot_bytes_ = have / n_slots_ & ~size_t(255);
        return MKF_OK;
    }

    // device_writable(), asked once for each allocation that this call's arrays
    // lie in
    void *writable(char *p, size_t bytes, size_t align)
    {
        if (reinterpret_cast<uintptr_t>(p) % align) return nullptr;
        for (const Range &r : ranges_)
            if (p >= r.host && p + bytes <= r.host + r.bytes) return r.dev + (p - r.host);
        Range r{};
        void *dev = device_writable(p, bytes, align, ctx_->device, &r.host, &r.bytes, &r.dev);
        if (dev && r.host) ranges_.push_back(r);
        return dev;
    }

    // jobs for the rows of r: all at once, or as many as a slot still holds
    mkf_status place_rows(const Rows &r, int r0, int r1)
    {
        const int nl = args_.n_layers;
        while (r0 < r1) {
            int m = r1 - r0;
            mkf_status st;
            if (r.staged) {
                const size_t pad = 256 * kOutFields;
                const size_t least = r.staged * std::min(m, kDeliverTile) + pad;
                if ((cur_ < 0 || used_ + least > slot_bytes_) && (st = next_slot()) != MKF_OK) return st;
                m = (int)std::min<size_t>(m, (slot_bytes_ - used_ - pad) / r.staged);
            }
            if (args_.n_jobs == kDeliverJobs && (st = launch()) != MKF_OK) return st;
            DeliverJob &j = args_.job[args_.n_jobs++];
            j = DeliverJob{};
            j.rec = r.o.rec + (size_t)kRecWords * r0;
            j.hits = r.o.hits + (size_t)nl * r0;
            j.n = m;
            j.first_tile = args_.n_tiles;
            args_.n_tiles += (m + kDeliverTile - 1) / kDeliverTile;
            for (int f = 0; f < kOutFields; ++f) {
                char *p = static_cast<char *>(field_of(r.o.out, f));
                if (!p) continue;
                const size_t fb = field_bytes(f, nl);
                if (r.direct[f]) {
                    set_field(j, f, static_cast<char *>(r.direct[f]) + fb * r0);
                } else {
                    char *stage = stage_ + cur_ * slot_bytes_ + used_;
                    used_ += (fb * m + 255) & ~size_t(255);
                    set_field(j, f, stage);
                    slot_[cur_].copies.push_back(HostCopy{p + fb * r0, stage, fb * m});
                }
            }
            r0 += m;
        }
        return MKF_OK;
    }

    mkf_status launch()
    {
        if (args_.n_jobs == 0) return MKF_OK;
        MKF_HIP(launch_deliver(args_, ctx_->stream, take_stamp(ctx_)));
        launched();
        return MKF_OK;
    }

    // everything placed in the current slot has been launched
    mkf_status mark_slot()
    {
        Slot &sl = slot_[cur_];
        if (sl.copies.empty()) return MKF_OK;
        if (++ctx_->out_mark == 0) ++ctx_->out_mark;   // 0: never written
        sl.mark = ctx_->out_mark;
        sl.flag = ctx_->out_marks + cur_;
        MKF_HIP(launch_mark(ctx_->out_marks + cur_, sl.mark, ctx_->stream));
        return MKF_OK;
    }

    mkf_status next_slot()
    {
        mkf_status st = launch();   // ends the current slot's part
        if (st != MKF_OK || (cur_ >= 0 && (st = mark_slot()) != MKF_OK)) return st;
        cur_ = (cur_ + 1) % n_slots_;
        used_ = 0;
        return empty(slot_[cur_]);
    }

    // Waits until the device has filled the slot and copies its contents out.
    // The stream is asked from time to time, so that a failed launch ends the
    // wait.
    mkf_status empty(Slot &sl)
    {
        if (sl.copies.empty()) return MKF_OK;
        for (unsigned spin = 1; __atomic_load_n(sl.flag, __ATOMIC_ACQUIRE) != sl.mark; ++spin) {
            __builtin_ia32_pause();
            if (spin % 8192) continue;   // some 100 us
            const hipError_t e = hipStreamQuery(ctx_->stream);
            if (e == hipErrorNotReady) continue;
            MKF_HIP(e);
            if (__atomic_load_n(sl.flag, __ATOMIC_ACQUIRE) != sl.mark)
                return fail(MKF_E_DEVICE, "results: a finished launch left its mark unwritten");
        }
        copy_out(sl);
        return MKF_OK;
    }

    void copy_out(Slot &sl)
    {
        for (const HostCopy &c : sl.copies) std::memcpy(c.dst, c.src, c.bytes);
        sl.copies.clear();
    }

    mkf_ctx *ctx_;
    const bool fixed_;
    DeliverArgs args_;
    struct Range {
        char *host, *dev;
        size_t bytes;
    };
    std::vector<Range> ranges_;
    std::vector<Rows> rows_;
    EventRec *const *recs_ = nullptr;
    const mkf_tracks *outs_ = nullptr;
    int n_recs_ = 0;
    char *stage_ = nullptr;
    size_t staged_ = 0, slot_bytes_ = 0, used_ = 0;
    double link_bytes_ = 0.0;
    long long total_ = 0, placed_ = 0;
    Slot slot_[kOutSlots];
    int cur_ = -1, n_slots_ = 0;
    bool begun_ = false, finished_ = false;
};

mkf_status run_pipeline(mkf_ctx *ctx, const Params &P, const mkf_tuning &t, const BatchArgs &args, uint32_t flags,
                        bool timed, hipStream_t s, Delivery *d, const std::vector<EventLoad> &loads)
{
    const bool stats = flags & MKF_BATCH_STATS, reindex = flags & MKF_BATCH_REINDEX;
    if (stats) MKF_HIP(launch_batch_zero(args, s));
    if (reindex) {
        if (timed) timer_begin(ctx, 1, s);
        MKF_HIP(launch_index(P, args, s, timed ? take_stamp(ctx) : Stamp{}));
    }
    if (t.persistent) MKF_HIP(launch_fill_i32(reinterpret_cast<int *>(args.queue), 0, 1, s));
    // one index build of the batch, its end stamped by the build's launch, or by
    // a launch of its own (1.5 us) where the host may be late with that
    if (timed && reindex && !(d && d->slow_to_prepare())) {
        timer_switch(ctx, 1, 0, s, 1);
    } else if (timed) {
        if (reindex) timer_end(ctx, 1, s, 1);
        timer_begin(ctx, 0, s);
    }
    if (d) {
        const mkf_status st = d->prepare();
        if (st != MKF_OK) return st;
    }
    std::vector<long long> ends{0};   // one part, however many rows
    if (d && !t.persistent) ends = plan_parts(loads, P, d->us_per_row());
    if (ends.size() == 1) {
        MKF_HIP(launch_build_batch(P, args, t.lanes_per_seed, t.waves_per_block, t.persistent,
                                   ctx->n_cu * t.blocks_per_cu, stats, nullptr, s, timed ? take_stamp(ctx) : Stamp{}));
    } else {
        BatchArgs part = args;
        long long at = 0;
        for (size_t k = 0; k < ends.size(); ++k) {
            part.first_item = k ? part.end_item : 0;
            part.end_item = items_before(loads, ends[k], args.seeds_per_item);
            DeliverArgs *jobs = nullptr;
            mkf_status st;
            if (k) {   // the rows of the part before
                if ((st = d->place(at, ends[k - 1])) != MKF_OK) return st;
                at = ends[k - 1];
                jobs = ctx->build_jobs + k;
                *jobs = d->pending();
            }
            MKF_HIP(launch_build_batch(P, part, t.lanes_per_seed, t.waves_per_block, 0, 0, stats, jobs, s,
                                       timed && k == 0 ? take_stamp(ctx) : Stamp{}));
            if (k) d->launched();
        }
    }
    if (flags & MKF_BATCH_FIT) {
        if (timed) timer_switch(ctx, 0, 2, s, 1);
        MKF_HIP(launch_refit(P, args, s, timed ? take_stamp(ctx) : Stamp{}));
        if (timed) timer_end(ctx, 2, s, 1);
    } else if (timed) {
        timer_end(ctx, 0, s, 1);
    }
    return MKF_OK;
}

namespace {

OutRows build_rows(const EventRec *rec, const mkf_tracks &out)
{
    return OutRows{rec->view.out_rec, rec->view.out_hits, rec->shape.n_seeds, out};
}

// Delivers one set of rows and waits for the stream.
mkf_status deliver_one(mkf_ctx *ctx, const OutRows &o)
{
    Delivery d(ctx);
    d.add(o);
    return d.finish();
}

std::vector<EventLoad> event_loads(EventRec *const *recs, int n)
{
    std::vector<EventLoad> c(n);
    for (int i = 0; i < n; ++i) c[i] = EventLoad{recs[i]->shape.n_seeds, max_layer_hits(recs[i]->shape)};
    return c;
}

}  // namespace

static mkf_status check_tracks(const mkf_tracks *out, int n, const char *what)
{
    if (!out) return MKF_OK;
    if (out->n != n) return fail(MKF_E_INVALID, "%s: output has %d rows, need %d", what, out->n, n);
    return MKF_OK;
}

}  // namespace mkf

using namespace mkf;

// ====================================================================== ABI

extern "C" {

const char *mkf_version(void) { return "mkf 0.1 (gfx950, FP32 Kalman filter)"; }

const char *mkf_last_error(const mkf_ctx *ctx)
{
    (void)ctx;   // the message is per thread
    return g_err;
}

int32_t mkf_ctx_broken(const mkf_ctx *ctx) { return ctx && device_broken(ctx->device) ? 1 : 0; }

mkf_status mkf_create(const mkf_config *cfg, const mkf_allocator *alloc, void *hip_stream, mkf_ctx **out)
{
    if (!out) return fail(MKF_E_INVALID, "out is NULL");
    mkf_status st = check_config(cfg);
    if (st != MKF_OK) return st;
    if (alloc && (!alloc->alloc || !alloc->free)) return fail(MKF_E_INVALID, "allocator needs alloc and free");
    int dev = 0;
    MKF_HIP(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    MKF_HIP(hipGetDeviceProperties(&prop, dev));
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
        return fail(MKF_E_DEVICE, "device %d is %s, this library is built for gfx950", dev, prop.gcnArchName);
    auto ctx = std::make_unique<mkf_ctx>();
    ctx->cfg = *cfg;
    ctx->device = dev;
    ctx->n_cu = prop.multiProcessorCount;
    ctx->heap.ctx = ctx.get();
    if (alloc) {
        ctx->alloc = *alloc;
        ctx->has_alloc = true;
    }
    if (hip_stream) {
        ctx->stream = static_cast<hipStream_t>(hip_stream);
    } else {
        MKF_HIP(hipStreamCreateWithFlags(&ctx->stream, hipStreamNonBlocking));
        ctx->own_stream = true;
    }
    std::memset(&ctx->tuning, 0, sizeof(ctx->tuning));
    if ((st = check_tuning(ctx->cfg, &ctx->tuning)) != MKF_OK) return st;
    derive_params(ctx.get());
    int khz = 0;
    MKF_HIP(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
    if (khz <= 0) return fail(MKF_E_DEVICE, "device %d has no wall clock", dev);
    ctx->ms_per_tick = 1.0 / khz;
    constexpr size_t kStampBytes = 3 * 2 * Timer::kRing * sizeof(unsigned long long);
    constexpr size_t kJobBytes = kBuildParts * sizeof(DeliverArgs), kMarkBytes = kOutSlots * sizeof(unsigned);
    constexpr size_t kWords = round_up_256(kStampBytes + kJobBytes + kMarkBytes);
    MKF_HIP(hipHostMalloc(reinterpret_cast<void **>(&ctx->stamps), kWords + kOutLeast, hipHostMallocDefault));
    ctx->build_jobs = reinterpret_cast<DeliverArgs *>(reinterpret_cast<char *>(ctx->stamps) + kStampBytes);
    ctx->out_marks = reinterpret_cast<unsigned *>(reinterpret_cast<char *>(ctx->build_jobs) + kJobBytes);
    std::memset(ctx->out_marks, 0, kMarkBytes);
    ctx->least_pin = reinterpret_cast<char *>(ctx->stamps) + kWords;
    for (int k = 0; k < 3; ++k) {
        ctx->timers[k].start = ctx->stamps + (2 * k) * Timer::kRing;
        ctx->timers[k].stop = ctx->stamps + (2 * k + 1) * Timer::kRing;
    }
    MKF_HIP(hipEventCreateWithFlags(&ctx->stage_done, hipEventDisableTiming));
    // device address of this GPU's fixed batch-descriptor array (the
    // no-allocation builder); looked up once per device
    MKF_HIP(noalloc_scratch_init(dev));
    *out = ctx.release();
    return MKF_OK;
}

void mkf_destroy(mkf_ctx *ctx)
{
    if (!ctx) return;
    shutdown_server(ctx);
    (void)hipStreamSynchronize(ctx->stream);
    drop_graphs_with(ctx, -1);
    for (auto &kv : ctx->events) destroy_event(ctx, kv.second.get());
    ctx->events.clear();
    ctx->heap.release(ctx->batch_dev);
    if (ctx->batch_host) (void)hipHostFree(ctx->batch_host);
    if (ctx->load_pin) (void)hipHostFree(ctx->load_pin);
    if (ctx->stamps) (void)hipHostFree(ctx->stamps);   // and the build jobs, marks and staging behind them
    if (ctx->stage_done) (void)hipEventDestroy(ctx->stage_done);
    if (ctx->own_stream) (void)hipStreamDestroy(ctx->stream);
    delete ctx;
}

mkf_status mkf_set_tuning(mkf_ctx *ctx, const mkf_tuning *t)
{
    if (!ctx || !t) return fail(MKF_E_INVALID, "NULL argument");
    mkf_tuning nt = *t;
    mkf_status st = check_tuning(ctx->cfg, &nt);
    if (st != MKF_OK) return st;
    if (build_lds_bytes(ctx->params.geo, ctx->cfg.n_layers, nt.waves_per_block) > 65536)
        return fail(MKF_E_INVALID, "waves_per_block too large for %d layers", ctx->cfg.n_layers);
    ctx->tuning = nt;
    derive_params(ctx);
    drop_graphs_with(ctx, -1);
    for (auto &kv : ctx->events) drop_plain_graph(kv.second.get());
    return MKF_OK;
}

mkf_status mkf_get_tuning(const mkf_ctx *ctx, mkf_tuning *t)
{
    if (!ctx || !t) return fail(MKF_E_INVALID, "NULL argument");
    *t = ctx->tuning;
    return MKF_OK;
}

mkf_status mkf_load_events(mkf_ctx *ctx, const mkf_event *evs, int32_t n, int32_t *handles)
{
    if (!ctx || !handles || n < 0 || (n > 0 && !evs)) return fail(MKF_E_INVALID, "NULL argument");
    if ((long long)n * ctx->cfg.n_layers > 65535)
        return fail(MKF_E_INVALID, "at most %d events per call", 65535 / ctx->cfg.n_layers);
    if (n == 0) return MKF_OK;
    std::vector<EventShape> shapes(n);
    std::vector<size_t> off(n + 1, 0);
    size_t values = 0;
    for (int i = 0; i < n; ++i) {
        const mkf_status st = validate_event(ctx, &evs[i], &shapes[i]);
        if (st != MKF_OK) return n == 1 ? st : fail(st, "event %d: %s", i, mkf_last_error(ctx));
        off[i + 1] = off[i] + ((event_input_bytes(shapes[i]) + 255) & ~size_t(255));
        values += (size_t)shapes[i].n_hits() * 3 + (size_t)(shapes[i].n_seeds + shapes[i].n_tracks) * 27;
    }
    // room for the results of these events too, so that the first build of a
    // batch allocates none
    size_t rows = 0;
    for (const EventShape &sh : shapes) rows += (size_t)std::max(sh.n_seeds, sh.n_tracks);
    mkf_status st = ensure_pin(ctx, std::max(off[n], out_pin_bytes(rows, (size_t)n, ctx->cfg.n_layers)));
    if (st != MKF_OK) return st;
    char *pin = static_cast<char *>(ctx->load_pin);
    std::vector<std::unique_ptr<EventRec>> recs(n);
    auto undo = [&](mkf_status st) {
        (void)hipStreamSynchronize(ctx->stream);
        for (auto &r : recs)
            if (r) destroy_event(ctx, r.get());
        return st;
    };
    hipStream_t s = ctx->stream;
    // device memory first (the allocator may call back into the caller, so
    // on this thread)
    for (int i = 0; i < n; ++i) {
        bool rebuilt = false;
        if ((st = create_event(ctx, shapes[i], &ctx->heap, &recs[i])) != MKF_OK) return undo(st);
        if ((st = ensure_index(ctx, recs[i].get(), &rebuilt, s)) != MKF_OK) return undo(st);
    }
    // the hits of every event, then the index, then the seeds and tracks: a
    // part's copy is queued as soon as it is packed, so that the copies and the
    // index overlap the packing of what follows
    std::vector<mkf_status> sts(n, MKF_OK);
    std::vector<std::string> why(n);
    std::vector<hipError_t> copied(n, hipSuccess);
    const int threads = pack_threads(values, kLoadValuesPerThread);
    auto pack_send = [&](PackPart part) -> mkf_status {
        run_tasks(n, n == 1 ? 1 : threads, [&](int i) {
            char *image = pin + off[i];
            sts[i] = pack_event(&evs[i], shapes[i], ctx->params.geo, image, n == 1 ? threads : 1, &why[i], part);
            if (sts[i] != MKF_OK) return;
            const size_t hits = event_hit_bytes(shapes[i]);
            const size_t from = part == PackPart::kRows ? hits : 0;
            const size_t bytes = (part == PackPart::kHits ? hits : event_input_bytes(shapes[i])) - from;
            if (part != PackPart::kHits)
                std::memcpy(image + event_view_offset(shapes[i]), &recs[i]->view, sizeof(DevEvent));
            if (bytes)
                copied[i] = hipMemcpyAsync(static_cast<char *>(recs[i]->data) + from, image + from, bytes,
                                           hipMemcpyHostToDevice, s);
        });
        for (int i = 0; i < n; ++i)
            if (sts[i] != MKF_OK)
                return n == 1 ? fail(sts[i], "%s", why[i].c_str()) : fail(sts[i], "event %d: %s", i, why[i].c_str());
        for (int i = 0; i < n; ++i)
            if (copied[i] != hipSuccess) {
                note_device_error(copied[i]);
                return fail(MKF_E_DEVICE, "load: %s", hipGetErrorString(copied[i]));
            }
        return MKF_OK;
    };
    // (small inputs in one part: a second copy takes longer than it hides)
    const bool two = off[n] >= (512u << 10);
    if ((st = pack_send(two ? PackPart::kHits : PackPart::kAll)) != MKF_OK) return undo(st);
    if ((st = ensure_batch_scratch(ctx, n)) != MKF_OK) return undo(st);
    std::vector<EventRec *> raw(n);
    for (int i = 0; i < n; ++i) raw[i] = recs[i].get();
    BatchArgs args{};
    if ((st = stage_batch(ctx, raw, ctx->batch_dev, ctx->batch_host,
                          seeds_per_item(ctx->params.geo, ctx->tuning.lanes_per_seed, raw.data(), n), &args, s)) !=
        MKF_OK)
        return undo(st);
    hipError_t e = launch_index(ctx->params, args, s);
    if (e == hipSuccess) {
        if (two && (st = pack_send(PackPart::kRows)) != MKF_OK) return undo(st);
        e = hipStreamSynchronize(s);
    }
    if (e != hipSuccess) {
        note_device_error(e);
        return undo(fail(MKF_E_DEVICE, "load: %s", hipGetErrorString(e)));
    }
    for (int i = 0; i < n; ++i) {
        const int32_t h = ctx->next_handle++;
        ctx->events[h] = std::move(recs[i]);
        handles[i] = h;
    }
    return MKF_OK;
}

mkf_status mkf_load_event(mkf_ctx *ctx, const mkf_event *ev, int32_t *handle)
{
    if (!ctx || !handle || !ev) return fail(MKF_E_INVALID, "NULL argument");
    return mkf_load_events(ctx, ev, 1, handle);
}

mkf_status mkf_unload_event(mkf_ctx *ctx, int32_t handle)
{
    if (!ctx) return fail(MKF_E_INVALID, "NULL context");
    auto it = ctx->events.find(handle);
    if (it == ctx->events.end()) return fail(MKF_E_NOTFOUND, "unknown event handle %d", handle);
    MKF_HIP(hipStreamSynchronize(ctx->stream));
    drop_graphs_with(ctx, handle);
    destroy_event(ctx, it->second.get());
    ctx->events.erase(it);
    return MKF_OK;
}

static mkf_status reindex_if_needed(mkf_ctx *ctx, const std::vector<EventRec *> &recs, bool *any)
{
    *any = false;
    for (EventRec *r : recs) {
        bool rebuilt = false;
        mkf_status st = ensure_index(ctx, r, &rebuilt, ctx->stream);
        if (st != MKF_OK) return st;
        if (rebuilt) {
            if ((st = upload_view(r, ctx->stream)) != MKF_OK) return st;
            drop_graphs_with(ctx, -1);
            *any = true;
        }
    }
    return MKF_OK;
}

mkf_status mkf_build(mkf_ctx *ctx, int32_t handle, mkf_tracks *out)
{
    if (!ctx) return fail(MKF_E_INVALID, "NULL context");
    EventRec *rec = find_event(ctx, handle);
    if (!rec) return fail(MKF_E_NOTFOUND, "unknown event handle %d", handle);
    mkf_status st = check_tracks(out, rec->shape.n_seeds, "build");
    if (st != MKF_OK) return st;
    std::vector<EventRec *> one{rec};
    bool need_index = false;
    if ((st = reindex_if_needed(ctx, one, &need_index)) != MKF_OK) return st;
    const int G = ctx->tuning.lanes_per_seed, wpb = ctx->tuning.waves_per_block;
    const int spi = seeds_per_item(ctx->params.geo, G, &rec, 1);
    if (need_index) {
        if ((st = ensure_batch_scratch(ctx, 1)) != MKF_OK) return st;
        BatchArgs args{};
        if ((st = stage_batch(ctx, one, ctx->batch_dev, ctx->batch_host, spi, &args, ctx->stream)) !=
            MKF_OK)
            return st;
        MKF_HIP(launch_index(ctx->params, args, ctx->stream));
    }
    if (rec->plain_G != G || !rec->plain) {
        if (rec->plain) MKF_HIP(hipStreamSynchronize(ctx->stream));
        drop_plain_graph(rec);
        rec->heap->release(rec->plain);
        rec->plain = nullptr;
        rec->plain_G = 0;
        // fewer seeds per wavefront take more slots: where the memory for those
        // is not to be had, full wavefronts
        size_t bytes = 0;
        for (int spw : {spi, kWave / G}) {
            const int slots = plain_slots(rec->shape.n_seeds, spw);
            bytes = carve_plain(rec->shape, slots, nullptr, &rec->view);
            rec->plain = rec->heap->alloc(bytes);
            if (!rec->plain) continue;
            carve_plain(rec->shape, slots, rec->plain, &rec->view);
            rec->plain_spw = spw;
            break;
        }
        if (!rec->plain) return fail(MKF_E_NOMEM, "builder state: %zu bytes", bytes);
        rec->plain_G = G;
        if ((st = upload_view(rec, ctx->stream)) != MKF_OK) return st;
    }
    const int n_launch = rec->shape.n_layers - rec->shape.n_seed_layers;
    if (rec->shape.n_seeds > 0) {
        if (!rec->plain_graph || rec->plain_graph_G != G || rec->plain_graph_wpb != wpb) {
            drop_plain_graph(rec);
            hipGraph_t graph = nullptr;
            MKF_HIP(hipStreamBeginCapture(ctx->stream, hipStreamCaptureModeThreadLocal));
            hipError_t cap = hipSuccess;
            for (int L = rec->shape.n_seed_layers; L < rec->shape.n_layers && cap == hipSuccess; ++L)
                cap = launch_build_layer(ctx->params, rec->dev_view, rec->view, L, G, rec->plain_spw, wpb, false, ctx->stream);
            hipError_t end = hipStreamEndCapture(ctx->stream, &graph);
            if (cap != hipSuccess || end != hipSuccess) {
                if (graph) (void)hipGraphDestroy(graph);
                return fail(MKF_E_DEVICE, "capturing the layer loop: %s",
                            hipGetErrorString(cap != hipSuccess ? cap : end));
            }
            hipError_t ins = hipGraphInstantiate(&rec->plain_graph, graph, nullptr, nullptr, 0);
            (void)hipGraphDestroy(graph);
            if (ins != hipSuccess) return fail(MKF_E_DEVICE, "instantiating the layer loop: %s", hipGetErrorString(ins));
            rec->plain_graph_G = G;
            rec->plain_graph_wpb = wpb;
        }
        Delivery d(ctx);
        const bool first = out && d.slow_to_prepare((size_t)rec->shape.n_seeds, 1);
        if (first) {
            d.add(build_rows(rec, *out));
            if ((st = d.prepare()) != MKF_OK) return st;
        }
        timer_begin(ctx, 0, ctx->stream);
        stamp_now(ctx);
        MKF_HIP(hipGraphLaunch(rec->plain_graph, ctx->stream));
        timer_end(ctx, 0, ctx->stream, n_launch);
        if (out && !first) d.add(build_rows(rec, *out));
        if ((st = d.finish()) != MKF_OK) return st;
    } else {
        MKF_HIP(hipStreamSynchronize(ctx->stream));
    }
    timers_collect(ctx, false);   // all has run
    return MKF_OK;
}

mkf_status mkf_build_batch(mkf_ctx *ctx, const int32_t *handles, int32_t n, uint32_t flags, mkf_tracks *outs)
{
    if (!ctx) return fail(MKF_E_INVALID, "NULL context");
    if (flags & ~(MKF_BATCH_REINDEX | MKF_BATCH_STATS | MKF_BATCH_GRAPH | MKF_BATCH_ASYNC | MKF_BATCH_FIT |
                  MKF_BATCH_BEAM))
        return fail(MKF_E_INVALID, "unknown flags");
    const bool beam = flags & MKF_BATCH_BEAM;
    const bool async = flags & MKF_BATCH_ASYNC;
    flags &= ~MKF_BATCH_ASYNC;
    if (async && outs) return fail(MKF_E_INVALID, "an asynchronous batch returns no host outputs (outs must be NULL)");
    std::vector<EventRec *> recs;
    mkf_status st = gather_events(ctx, handles, n, &recs);
    if (st != MKF_OK) return st;
    if (outs)
        for (int i = 0; i < n; ++i)
            if ((st = check_tracks(&outs[i], recs[i]->shape.n_seeds, "build_batch")) != MKF_OK) return st;
    if (n == 0) return MKF_OK;
    if (beam)
        for (EventRec *r : recs)
            if ((st = ensure_beam(ctx, r)) != MKF_OK) return st;
    bool need_index = false;
    if ((st = reindex_if_needed(ctx, recs, &need_index)) != MKF_OK) return st;
    if (need_index) flags |= MKF_BATCH_REINDEX;
    std::unique_ptr<Delivery> d;   // none for an asynchronous batch: its destructor waits
    if (!async) d = std::make_unique<Delivery>(ctx);
    if (d) d->later(recs.data(), n, outs);
    const int spi = seeds_per_item(ctx->params.geo, ctx->tuning.lanes_per_seed, recs.data(), n);
    if (flags & MKF_BATCH_GRAPH) {
        BatchGraph *bg = nullptr;
        std::vector<int32_t> key(handles, handles + n);
        for (auto &g : ctx->graphs)
            if (g->handles == key && g->flags == flags && std::memcmp(&g->tuning, &ctx->tuning, sizeof(mkf_tuning)) == 0)
                bg = g.get();
        if (!bg) {
            auto g = std::make_unique<BatchGraph>();
            g->handles = key;
            g->flags = flags;
            g->tuning = ctx->tuning;
            g->scratch = ctx->heap.alloc(batch_scratch_bytes(n));
            if (!g->scratch) return fail(MKF_E_NOMEM, "graph scratch");
            if ((st = ensure_batch_scratch(ctx, n)) != MKF_OK) {
                ctx->heap.release(g->scratch);
                return st;
            }
            BatchArgs args{};
            if ((st = stage_batch(ctx, recs, g->scratch, ctx->batch_host, spi, &args, ctx->stream, beam)) != MKF_OK) {
                ctx->heap.release(g->scratch);
                return st;
            }
            hipError_t e = hipStreamSynchronize(ctx->stream);
            if (e != hipSuccess) {
                ctx->heap.release(g->scratch);
                return fail(MKF_E_DEVICE, "staging: %s", hipGetErrorString(e));
            }
            hipGraph_t graph = nullptr;
            MKF_HIP(hipStreamBeginCapture(ctx->stream, hipStreamCaptureModeThreadLocal));
            mkf_status cst = run_pipeline(ctx, ctx->params, ctx->tuning, args, flags, false, ctx->stream);
            hipError_t end = hipStreamEndCapture(ctx->stream, &graph);
            if (cst != MKF_OK || end != hipSuccess) {
                if (graph) (void)hipGraphDestroy(graph);
                ctx->heap.release(g->scratch);
                return cst != MKF_OK ? cst : fail(MKF_E_DEVICE, "capture: %s", hipGetErrorString(end));
            }
            hipError_t ins = hipGraphInstantiate(&g->exec, graph, nullptr, nullptr, 0);
            (void)hipGraphDestroy(graph);
            if (ins != hipSuccess) {
                ctx->heap.release(g->scratch);
                return fail(MKF_E_DEVICE, "instantiate: %s", hipGetErrorString(ins));
            }
            bg = g.get();
            ctx->graphs.push_back(std::move(g));
        }
        if (d && (st = d->prepare()) != MKF_OK) return st;
        timer_begin(ctx, 0, ctx->stream);
        stamp_now(ctx);
        MKF_HIP(hipGraphLaunch(bg->exec, ctx->stream));
        timer_end(ctx, 0, ctx->stream, 1);
    } else {
        if ((st = ensure_batch_scratch(ctx, n)) != MKF_OK) return st;
        BatchArgs args{};
        if ((st = stage_batch(ctx, recs, ctx->batch_dev, ctx->batch_host, spi, &args, ctx->stream, beam)) != MKF_OK)
            return st;
        if ((st = run_pipeline(ctx, ctx->params, ctx->tuning, args, flags, true, ctx->stream, d.get(),
                               event_loads(recs.data(), n))) != MKF_OK)
            return st;
    }
    if (async) {
        stamp_now(ctx);
        timers_collect(ctx, false);
        return MKF_OK;
    }
    if ((st = d->finish()) != MKF_OK) return st;
    timers_collect(ctx, false);   // all has run
    return MKF_OK;
}

mkf_status mkf_build_batch_noalloc(mkf_ctx *ctx, const int32_t *handles, int32_t n, uint32_t flags,
                                   mkf_tracks *outs)
{
    if (!ctx) return fail(MKF_E_INVALID, "NULL context");
    if (flags & ~(MKF_BATCH_REINDEX | MKF_BATCH_STATS | MKF_BATCH_ASYNC | MKF_BATCH_FIT))
        return fail(MKF_E_INVALID, "only MKF_BATCH_REINDEX, _STATS, _ASYNC and _FIT build without allocating");
    const bool async = flags & MKF_BATCH_ASYNC;
    flags &= ~MKF_BATCH_ASYNC;
    if (async && outs) return fail(MKF_E_INVALID, "an asynchronous batch returns no host outputs (outs must be NULL)");
    if (n < 0 || (n > 0 && !handles)) return fail(MKF_E_INVALID, "bad handle list");
    if (n > kNoAllocMaxEvents)
        return fail(MKF_E_INVALID, "%d events: the no-allocation builder takes at most %d", n, kNoAllocMaxEvents);
    if ((long long)n * ctx->cfg.n_layers > 65535)
        return fail(MKF_E_INVALID, "at most %d events per batch", 65535 / ctx->cfg.n_layers);
    char *dev = static_cast<char *>(noalloc_scratch(ctx->device));
    if (!dev) return fail(MKF_E_DEVICE, "no descriptor array on device %d", ctx->device);
    EventRec *recs[kNoAllocMaxEvents];
    for (int i = 0; i < n; ++i) {
        for (int j = 0; j < i; ++j)
            if (handles[j] == handles[i]) return fail(MKF_E_INVALID, "an event appears twice in the batch");
        recs[i] = find_event(ctx, handles[i]);
        if (!recs[i]) return fail(MKF_E_NOTFOUND, "unknown event handle %d", handles[i]);
        if (!recs[i]->index || recs[i]->index_bins_phi != ctx->tuning.bins_phi ||
            recs[i]->index_bins_z != ctx->tuning.bins_z)
            return fail(MKF_E_STATE, "event %d has no index for the current bin grid (mkf_build_batch makes one)",
                        handles[i]);
        if (outs && outs[i].n != recs[i]->shape.n_seeds)
            return fail(MKF_E_INVALID, "build_batch_noalloc: output has %d rows, need %d", outs[i].n,
                        recs[i]->shape.n_seeds);
    }
    if (n == 0) return MKF_OK;
    // the descriptors go through one host image and the device array of this
    // GPU; earlier work of this context may still read the array
    static std::mutex image_mu;
    static char image[kNoAllocScratchBytes];
    MKF_HIP(hipStreamSynchronize(ctx->stream));
    BatchArgs args{};
    {
        std::lock_guard<std::mutex> lk(image_mu);
        mkf_status st = compose_batch(recs, n, seeds_per_item(ctx->params.geo, ctx->tuning.lanes_per_seed, recs, n),
                                      false, image, dev, &args);
        if (st != MKF_OK) return st;
        MKF_HIP(hipMemcpyAsync(dev, image, batch_scratch_bytes(n), hipMemcpyHostToDevice, ctx->stream));
        MKF_HIP(hipStreamSynchronize(ctx->stream));
    }
    std::unique_ptr<Delivery> d;
    if (!async) d = std::make_unique<Delivery>(ctx, true);
    if (d) d->later(recs, n, outs);
    mkf_status st = run_pipeline(ctx, ctx->params, ctx->tuning, args, flags, true, ctx->stream, d.get(),
                                 event_loads(recs, n));
    if (st != MKF_OK) return st;
    if (async) {
        stamp_now(ctx);
        timers_collect(ctx, false);
        return MKF_OK;
    }
    if ((st = d->finish()) != MKF_OK) return st;
    timers_collect(ctx, false);   // all has run
    return MKF_OK;
}

mkf_status mkf_fetch_tracks(mkf_ctx *ctx, int32_t handle, mkf_tracks *out)
{
    if (!ctx || !out) return fail(MKF_E_INVALID, "NULL argument");
    EventRec *rec = find_event(ctx, handle);
    if (!rec) return fail(MKF_E_NOTFOUND, "unknown event handle %d", handle);
    mkf_status st = check_tracks(out, rec->shape.n_seeds, "fetch");
    if (st != MKF_OK) return st;
    return deliver_one(ctx, build_rows(rec, *out));
}

mkf_status mkf_fetch_fit(mkf_ctx *ctx, int32_t handle, mkf_tracks *out)
{
    if (!ctx || !out) return fail(MKF_E_INVALID, "NULL argument");
    EventRec *rec = find_event(ctx, handle);
    if (!rec) return fail(MKF_E_NOTFOUND, "unknown event handle %d", handle);
    mkf_status st = check_tracks(out, rec->shape.n_seeds, "fetch_fit");
    if (st != MKF_OK) return st;
    return deliver_one(ctx, OutRows{rec->view.rf_rec, rec->view.out_hits, rec->shape.n_seeds, *out});
}

mkf_status mkf_fetch_beam(mkf_ctx *ctx, int32_t handle, mkf_tracks *out)
{
    if (!ctx || !out) return fail(MKF_E_INVALID, "NULL argument");
    EventRec *rec = find_event(ctx, handle);
    if (!rec) return fail(MKF_E_NOTFOUND, "unknown event handle %d", handle);
    if (!rec->beam) return fail(MKF_E_STATE, "no build of this event kept its beam (MKF_BATCH_BEAM)");
    const size_t n = (size_t)rec->shape.n_seeds * ctx->cfg.max_cands;
    mkf_status st = check_tracks(out, (int)n, "fetch_beam");
    if (st != MKF_OK) return st;
    return deliver_one(ctx, OutRows{rec->beam_view.beam_rec, rec->beam_view.beam_hits, (int)n, *out});
}

mkf_status mkf_index_grid(mkf_ctx *ctx, int32_t handle, int32_t *bins_phi, int32_t *bins_z)
{
    if (!ctx || !bins_phi || !bins_z) return fail(MKF_E_INVALID, "NULL argument");
    EventRec *rec = find_event(ctx, handle);
    if (!rec) return fail(MKF_E_NOTFOUND, "unknown event handle %d", handle);
    if (!rec->index || rec->index_bins_phi != ctx->tuning.bins_phi || rec->index_bins_z != ctx->tuning.bins_z)
        return fail(MKF_E_STATE, "the index was built for another bin grid");
    *bins_phi = rec->index_bins_phi >> rec->view.grid_k;
    *bins_z = rec->index_bins_z >> rec->view.grid_k;
    return MKF_OK;
}

mkf_status mkf_fetch_index(mkf_ctx *ctx, int32_t handle, int32_t layer, int32_t *bin_off, int32_t *bin_of,
                           int32_t *order)
{
    if (!ctx) return fail(MKF_E_INVALID, "NULL context");
    EventRec *rec = find_event(ctx, handle);
    if (!rec) return fail(MKF_E_NOTFOUND, "unknown event handle %d", handle);
    if (layer < 0 || layer >= rec->shape.n_layers) return fail(MKF_E_INVALID, "layer %d out of range", layer);
    if (!rec->index || rec->index_bins_phi != ctx->tuning.bins_phi || rec->index_bins_z != ctx->tuning.bins_z)
        return fail(MKF_E_STATE, "the index was built for another bin grid");
    const int k = rec->view.grid_k;
    const int nb = (ctx->tuning.bins_phi >> k) * (ctx->tuning.bins_z >> k);
    const int h0 = rec->shape.layer_off[layer], n = rec->shape.layer_off[layer + 1] - h0;
    const DevEvent &v = rec->view;
    std::vector<int32_t> off(bin_off ? nb + 1 : 0);
    std::vector<float4> binned(order ? n : 0);
    hipStream_t s = ctx->stream;
    if (bin_off)
        MKF_HIP(hipMemcpyAsync(off.data(), v.bin_off + (size_t)layer * bin_off_stride(nb), 4 * (size_t)(nb + 1),
                               hipMemcpyDeviceToHost, s));
    if (bin_of && n) MKF_HIP(hipMemcpyAsync(bin_of, v.bin_of + h0, 4 * (size_t)n, hipMemcpyDeviceToHost, s));
    if (order && n) MKF_HIP(hipMemcpyAsync(binned.data(), v.binned + h0, sizeof(float4) * (size_t)n,
                                           hipMemcpyDeviceToHost, s));
    MKF_HIP(hipStreamSynchronize(s));
    if (bin_off)
        for (int i = 0; i <= nb; ++i) bin_off[i] = off[i] - h0;
    if (order)
        for (int i = 0; i < n; ++i) {
            int32_t id;
            std::memcpy(&id, &binned[i].w, 4);
            order[i] = id;
        }
    return MKF_OK;
}

mkf_status mkf_get_stats(mkf_ctx *ctx, int32_t handle, mkf_build_stats *out)
{
    if (!ctx || !out) return fail(MKF_E_INVALID, "NULL argument");
    EventRec *rec = find_event(ctx, handle);
    if (!rec) return fail(MKF_E_NOTFOUND, "unknown event handle %d", handle);
    unsigned long long v[5];
    MKF_HIP(hipMemcpyAsync(v, rec->view.stats, sizeof(v), hipMemcpyDeviceToHost, ctx->stream));
    MKF_HIP(hipStreamSynchronize(ctx->stream));
    out->cand_layers = (int64_t)v[0];
    out->chi2_evals = (int64_t)v[1];
    out->accepted = (int64_t)v[2];
    out->updates = (int64_t)v[3];
    out->hits_scanned = (int64_t)v[4];
    return MKF_OK;
}

mkf_status mkf_fit_batch(mkf_ctx *ctx, const int32_t *handles, int32_t n, mkf_tracks *outs)
{
    if (!ctx) return fail(MKF_E_INVALID, "NULL context");
    std::vector<EventRec *> recs;
    mkf_status st = gather_events(ctx, handles, n, &recs);
    if (st != MKF_OK) return st;
    if (outs)
        for (int i = 0; i < n; ++i)
            if ((st = check_tracks(&outs[i], recs[i]->shape.n_tracks, "fit_batch")) != MKF_OK) return st;
    if (n == 0) return MKF_OK;
    if ((st = ensure_batch_scratch(ctx, n)) != MKF_OK) return st;
    BatchArgs args{};
    if ((st = stage_batch(ctx, recs, ctx->batch_dev, ctx->batch_host, 64, &args, ctx->stream)) != MKF_OK)
        return st;
    Delivery d(ctx);
    size_t rows = 0;
    for (const EventRec *r : recs) rows += (size_t)r->shape.n_tracks;
    auto add = [&] {
        for (int i = 0; outs && i < n; ++i)
            d.add(OutRows{recs[i]->view.fit_rec, recs[i]->view.track_hits, recs[i]->shape.n_tracks, outs[i]});
    };
    const bool first = outs && d.slow_to_prepare(rows, n);
    if (first) {
        add();
        if ((st = d.prepare()) != MKF_OK) return st;
    }
    timer_begin(ctx, 2, ctx->stream);
    MKF_HIP(launch_fit(ctx->params, args, ctx->stream, take_stamp(ctx)));
    timer_end(ctx, 2, ctx->stream, 1);
    if (!first) add();
    if ((st = d.finish()) != MKF_OK) return st;
    timers_collect(ctx, false);   // all has run
    return MKF_OK;
}

mkf_status mkf_fit(mkf_ctx *ctx, int32_t handle, int32_t n_tracks, const double *init_par, const double *init_cov,
                   const int32_t *track_hits, mkf_tracks *out)
{
    if (!ctx) return fail(MKF_E_INVALID, "NULL context");
    EventRec *rec = find_event(ctx, handle);
    if (!rec) return fail(MKF_E_NOTFOUND, "unknown event handle %d", handle);
    mkf_status st = check_tracks(out, n_tracks, "fit");
    if (st != MKF_OK) return st;
    if (n_tracks < 0) return fail(MKF_E_INVALID, "negative track count");
    if (n_tracks > 0 && (!init_par || !init_cov || !track_hits)) return fail(MKF_E_INVALID, "track arrays are NULL");
    if (n_tracks == 0) return MKF_OK;
    // a temporary event view: the loaded event's hits with these tracks, whose
    // inputs are checked and narrowed to FP32 in the load staging and copied
    // in one piece
    EventShape ts = rec->shape;
    ts.n_seeds = 0;
    ts.n_tracks = n_tracks;
    const size_t nt = (size_t)n_tracks, nl = (size_t)ts.n_layers;
    auto layout = [&](char *base, DevEvent *v) {
        size_t o = 0;
        auto take = [&](size_t b) {
            char *p = base + o;
            o = (o + b + 255) & ~size_t(255);
            return p;
        };
        v->track_par = reinterpret_cast<float *>(take(24 * nt));
        v->track_cov = reinterpret_cast<float *>(take(84 * nt));
        v->track_hits = reinterpret_cast<int *>(take(4 * nl * nt));
        const size_t inputs = o;
        v->fit_rec = reinterpret_cast<float *>(take(4 * (size_t)kRecWords * nt));
        return std::make_pair(inputs, o);
    };
    DevEvent hv{};
    const auto sizes = layout(nullptr, &hv);
    // the inputs now, the results later
    if ((st = ensure_pin(ctx, std::max(sizes.first, out_pin_bytes(nt, 1, (int)nl)))) != MKF_OK) return st;
    layout(static_cast<char *>(ctx->load_pin), &hv);
    std::vector<int32_t> nh(nl);
    for (size_t L = 0; L < nl; ++L) nh[L] = rec->shape.layer_off[L + 1] - rec->shape.layer_off[L];
    int bad_hit = 0;
    const long long failed = pack_states(init_par, init_cov, track_hits, nt, (int)nl, nh.data(),
                                         const_cast<float *>(hv.track_par), const_cast<float *>(hv.track_cov),
                                         const_cast<int *>(hv.track_hits), &bad_hit);
    if (failed >= 0)
        return fail(MKF_E_INVALID, bad_hit ? "track %d: hit index out of range"
                                           : "track %d: state or covariance not finite (in FP32), theta "
                                             "outside (0, pi) or position on the axis", (int)failed);
    char *buf = static_cast<char *>(ctx->heap.alloc(sizes.second + sizeof(DevEvent) + 256));
    if (!buf) return fail(MKF_E_NOMEM, "fit buffers: %zu bytes", sizes.second);
    DevEvent v = rec->view;
    v.n_seeds = 0;
    v.n_tracks = n_tracks;
    layout(buf, &v);
    auto cleanup = [&](mkf_status s) {
        (void)hipStreamSynchronize(ctx->stream);
        ctx->heap.release(buf);
        return s;
    };
    hipStream_t s = ctx->stream;
    if (hipMemcpyAsync(buf, ctx->load_pin, sizes.first, hipMemcpyHostToDevice, s) != hipSuccess)
        return cleanup(fail(MKF_E_DEVICE, "fit upload failed"));
    if ((st = ensure_batch_scratch(ctx, 1)) != MKF_OK) return cleanup(st);
    EventRec tmp;
    tmp.shape = ts;
    tmp.view = v;
    std::vector<EventRec *> one{&tmp};
    BatchArgs args{};
    if ((st = stage_batch(ctx, one, ctx->batch_dev, ctx->batch_host, 64, &args, s)) != MKF_OK) return cleanup(st);
    {
        Delivery d(ctx);
        timer_begin(ctx, 2, s);
        const hipError_t e = launch_fit(ctx->params, args, s, take_stamp(ctx));
        timer_end(ctx, 2, s, 1);
        if (e != hipSuccess) return cleanup(fail(MKF_E_DEVICE, "fit launch: %s", hipGetErrorString(e)));
        if (out) d.add(OutRows{v.fit_rec, v.track_hits, n_tracks, *out});   // (its staging is there)
        if ((st = d.finish()) != MKF_OK) return cleanup(st);
    }
    timers_collect(ctx, false);   // all has run
    ctx->heap.release(buf);
    return MKF_OK;
}

mkf_status mkf_timer_read(mkf_ctx *ctx, int32_t which, double *total_ms, int64_t *launches)
{
    if (!ctx || which < 0 || which > 2) return fail(MKF_E_INVALID, "bad timer");
    MKF_HIP(hipStreamSynchronize(ctx->stream));
    timers_collect(ctx, true);
    if (total_ms) *total_ms = ctx->timers[which].total_ms;
    if (launches) *launches = ctx->timers[which].launches;
    return MKF_OK;
}

mkf_status mkf_timer_reset(mkf_ctx *ctx)
{
    if (!ctx) return fail(MKF_E_INVALID, "NULL context");
    MKF_HIP(hipStreamSynchronize(ctx->stream));
    timers_collect(ctx, true);
    for (auto &t : ctx->timers) {
        t.total_ms = 0;
        t.launches = 0;
    }
    return MKF_OK;
}

mkf_status mkf_sync(mkf_ctx *ctx)
{
    if (!ctx) return fail(MKF_E_INVALID, "NULL context");
    MKF_HIP(hipStreamSynchronize(ctx->stream));
    timers_collect(ctx, true);
    return MKF_OK;
}

mkf_status mkf_autotune(mkf_ctx *ctx, const int32_t *handles, int32_t n, mkf_tuning *best)
{
    if (!ctx) return fail(MKF_E_INVALID, "NULL context");
    std::vector<EventRec *> recs;
    mkf_status st = gather_events(ctx, handles, n, &recs);
    if (st != MKF_OK) return st;
    if (n == 0) return fail(MKF_E_INVALID, "no events to tune on");
    const mkf_tuning start = ctx->tuning;
    auto measure = [&](const mkf_tuning &t, double *ms) -> mkf_status {
        mkf_status s2 = mkf_set_tuning(ctx, &t);
        if (s2 != MKF_OK) return s2;
        s2 = mkf_build_batch(ctx, handles, n, MKF_BATCH_REINDEX, nullptr);
        if (s2 != MKF_OK) return s2;
        double best_ms = 1e30;
        for (int rep = 0; rep < 3; ++rep) {
            MKF_HIP(hipStreamSynchronize(ctx->stream));
            const auto t0 = std::chrono::steady_clock::now();
            s2 = mkf_build_batch(ctx, handles, n, MKF_BATCH_REINDEX, nullptr);
            if (s2 != MKF_OK) return s2;
            const auto t1 = std::chrono::steady_clock::now();
            best_ms = std::min(best_ms, std::chrono::duration<double, std::milli>(t1 - t0).count());
        }
        *ms = best_ms;
        return MKF_OK;
    };
    mkf_tuning cur = start;
    double cur_ms = 0;
    if ((st = measure(cur, &cur_ms)) != MKF_OK) return st;
    std::vector<int> lanes;
    for (int G : {1, 2, 4, 6, 8})
        if (G >= ctx->cfg.max_cands) lanes.push_back(G);
    const std::vector<int> waves = {1, 2, 4};
    const std::vector<int> bphi = {128, 256, 512, 1024, 2048};
    const std::vector<int> bz = {4, 8, 16, 32, 64};
    const std::vector<int> pers = {0, 1};
    const std::vector<int> bpc = {2, 4, 8, 16};
    for (int pass = 0; pass < 2; ++pass) {
        for (int dim = 0; dim < 6; ++dim) {
            const std::vector<int> &vals = dim == 0 ? lanes : dim == 1 ? waves : dim == 2 ? bphi : dim == 3 ? bz
                                                                                        : dim == 4 ? pers : bpc;
            for (int v : vals) {
                mkf_tuning t = cur;
                int *field = dim == 0 ? &t.lanes_per_seed : dim == 1 ? &t.waves_per_block : dim == 2 ? &t.bins_phi
                             : dim == 3 ? &t.bins_z : dim == 4 ? &t.persistent : &t.blocks_per_cu;
                if (*field == v) continue;
                *field = v;
                double ms = 0;
                if (measure(t, &ms) != MKF_OK) continue;
                if (ms < cur_ms * 0.98) {
                    cur = t;
                    cur_ms = ms;
                }
            }
        }
    }
    if ((st = mkf_set_tuning(ctx, &cur)) != MKF_OK) return st;
    if (best) *best = ctx->tuning;
    return MKF_OK;
}

mkf_status mkf_calib_copy(mkf_ctx *ctx, const void *src_dev, void *dst_dev, size_t bytes)
{
    if (!ctx || !src_dev || !dst_dev || bytes % 16) return fail(MKF_E_INVALID, "bad copy arguments");
    MKF_HIP(launch_copy(src_dev, dst_dev, bytes, ctx->stream));
    MKF_HIP(hipStreamSynchronize(ctx->stream));
    return MKF_OK;
}

mkf_status mkf_calib_fma(mkf_ctx *ctx, float *dst_dev, int32_t n_blocks, int32_t iters, double *ms, double *flop)
{
    if (!ctx || !dst_dev || n_blocks < 1 || iters < 4 || iters % 4 || !ms || !flop)
        return fail(MKF_E_INVALID, "bad FMA calibration arguments");
    hipEvent_t ev[2] = {nullptr, nullptr};
    MKF_HIP(hipEventCreate(&ev[0]));
    hipError_t e = hipEventCreate(&ev[1]);
    if (e == hipSuccess) e = hipEventRecord(ev[0], ctx->stream);
    if (e == hipSuccess) e = launch_calib_fma(dst_dev, n_blocks, iters, ctx->stream);
    if (e == hipSuccess) e = hipEventRecord(ev[1], ctx->stream);
    if (e == hipSuccess) e = hipEventSynchronize(ev[1]);
    float t = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&t, ev[0], ev[1]);
    hipEventDestroy(ev[0]);
    if (ev[1]) hipEventDestroy(ev[1]);
    MKF_HIP(e);
    *ms = t;
    *flop = 2.0 * calib_fma_chains() * (double)iters * 256.0 * (double)n_blocks;
    return MKF_OK;
}

}  // extern "C"
