// Host runtime of the track builder: context, device memory, loaded events.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <condition_variable>
#include <cstdarg>
#include <deque>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <unordered_map>
#include <vector>

#include "mkf_internal.hpp"

namespace mkf {

// thread-local message of the last failure
mkf_status fail(mkf_status st, const char *fmt, ...);

// Records errors after which the device's HIP context is unusable (a faulting
// kernel); mkf_ctx_broken reports them.
void note_device_error(hipError_t e);
bool device_broken(int device);

#define MKF_HIP(expr)                                                                          \
    do {                                                                                       \
        hipError_t e_ = (expr);                                                                \
        if (e_ != hipSuccess) {                                                                \
            ::mkf::note_device_error(e_);                                                      \
            return ::mkf::fail(MKF_E_DEVICE, "%s: %s", #expr, hipGetErrorString(e_));          \
        }                                                                                      \
    } while (0)

// Source of device memory for events: the caller's hooks / hipMalloc, or
// the serving slab.
struct DeviceHeap {
    virtual ~DeviceHeap() = default;
    virtual void *alloc(size_t bytes) = 0;
    virtual void release(void *p) = 0;
};

// First-fit sub-allocator over one reserved device slab (serving budget).
class SlabHeap : public DeviceHeap {
  public:
    SlabHeap(char *base, size_t bytes);
    void *alloc(size_t bytes) override;
    void release(void *p) override;
    size_t used() const { return used_; }
    size_t capacity() const { return cap_; }

  private:
    char *base_;
    size_t cap_;
    size_t used_ = 0;
    std::map<size_t, size_t> free_;     // offset -> size
    std::map<size_t, size_t> taken_;    // offset -> size
    std::mutex mu_;
};

// Sizes of one event, from which its device layout follows.
struct EventShape {
    int n_layers = 0;
    int n_seed_layers = 0;
    int n_seeds = 0;
    int n_tracks = 0;
    int layer_off[kMaxLayers + 1] = {0};
    int n_hits() const { return layer_off[n_layers]; }
};

size_t event_data_bytes(const EventShape &s);
size_t event_input_bytes(const EventShape &s);   // the packed inputs at the start of the data block
size_t event_budget_bytes(const EventShape &s, int n_bins);   // what a served event holds of the budget
int max_layer_hits(const EventShape &s);
int event_bins(const EventShape &s, int bins_phi, int bins_z);   // bins per layer of the event's grid

// One loaded event.
struct EventRec {
    EventShape shape;
    DeviceHeap *heap = nullptr;
    void *data = nullptr;          // hits, seeds, tracks, outputs, stats, descriptor
    void *index = nullptr;         // bin counts and offsets
    void *plain = nullptr;         // per-layer builder state
    void *beam = nullptr;          // every rank of the final beam (allocated on first request)
    DevEvent beam_view{};          // its arrays (only the beam_* members are set)
    int index_bins_phi = 0, index_bins_z = 0;   // grid the index was built for (0 = none)
    int plain_G = 0, plain_spw = 0;   // its lanes per seed and seeds per wavefront
    DevEvent view{};               // host copy of the device descriptor
    DevEvent *dev_view = nullptr;  // device copy (inside `data`)
    hipGraphExec_t plain_graph = nullptr;
    int plain_graph_G = 0;
    int plain_graph_wpb = 0;
};

struct BatchGraph {
    std::vector<int32_t> handles;
    uint32_t flags = 0;
    mkf_tuning tuning{};
    void *scratch = nullptr;       // descriptors + prefixes + queue, owned
    hipGraphExec_t exec = nullptr;
};

// Device time of the timed phases: a ring of (start, stop) wall-clock stamps
// in page-locked memory, so that calls that return before the device finishes
// (asynchronous batches) each keep their own interval until it is collected.
// The stamps are written by the launch that begins a phase or follows its end,
// or by a one-thread kernel in the stream where none does: 1.5-4.5 us, where a
// pair of HIP events around a kernel adds 5.6-6.5 us to a call.
struct Timer {
    static constexpr int kRing = 32;
    unsigned long long *start = nullptr, *stop = nullptr;   // kRing each; 0: not written yet
    long long ring_launches[kRing] = {};
    int head = 0, count = 0;   // recorded intervals not yet collected
    bool open = false;         // between timer_begin and timer_end
    double total_ms = 0.0;
    long long launches = 0;
};

// Rows of results bound for a caller's arrays: n rows at `rec` / `hits` on
// the device, `out` the arrays (pointers at the first of these rows).
struct OutRows {
    const float *rec = nullptr;
    const int *hits = nullptr;
    int n = 0;
    mkf_tracks out{};
};

struct HostCopy {   // staged bytes to copy once the device has written them
    void *dst;
    const void *src;
    size_t bytes;
};

// The way out of results (k_deliver): arrays that the device can write
// (page-locked memory) are written directly, the others through page-locked
// staging (the context's) that the host copies from.  The staging is used as
// a ring of slots, so that the device fills one while the host empties
// another and large outputs need no staging of their size.  With several slots
// the device tells the host of a filled one by a word that it waits for in a
// loop (k_mark; an event recorded and waited for makes a call up to 20 us
// longer: 20,000 tracks of one event built by mkf_build 393 us, 365 with
// marks); up to twice kOutSlotMin leave in one slot, copied after the stream's
// end (2,000 fitted tracks, 576 KB: 168 us in two slots, 121 in one).
constexpr int kOutSlots = 4;
constexpr int kBuildParts = 8;   // parts a batch with host outputs is built in, at most
constexpr size_t kOutSlotMin = size_t(512) << 10, kOutSlotMax = size_t(4) << 20;
constexpr size_t kOutLeast = size_t(64) << 10;   // the smallest staging used: a tile of rows and more

struct Server;   // serving state (mkf_serve.cpp)
struct ServerDeleter {
    void operator()(Server *s) const;
};

struct CtxHeap : public DeviceHeap {
    mkf_ctx *ctx = nullptr;
    void *alloc(size_t bytes) override;
    void release(void *p) override;
};

}  // namespace mkf

struct mkf_ctx {
    mkf_config cfg{};
    mkf_tuning tuning{};
    mkf::Params params{};          // derived from cfg + tuning
    int device = 0;
    int n_cu = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    bool has_alloc = false;
    mkf_allocator alloc{};
    mkf::CtxHeap heap;
    std::unordered_map<int32_t, std::unique_ptr<mkf::EventRec>> events;
    int32_t next_handle = 1;
    // batch scratch (descriptor array + prefixes + queue), device and pinned host
    void *batch_dev = nullptr;
    size_t batch_dev_bytes = 0;
    void *batch_host = nullptr;
    size_t batch_host_bytes = 0;
    hipEvent_t stage_done = nullptr;    // last copy out of batch_host
    bool stage_pending = false;
    std::vector<char> staged_image;     // what batch_dev holds (empty: unknown)
    // pinned staging of the packed inputs of loads and fits on their way in and
    // of results on their way out; every call that uses it ends waiting for
    // all that it queued to have passed through it, so it is free at the start
    // of the next
    void *load_pin = nullptr;
    size_t load_pin_bytes = 0;
    char *least_pin = nullptr;                      // page-locked, kOutLeast: for a call that may not make load_pin larger
    mkf::DeliverArgs *build_jobs = nullptr;         // page-locked: rows that build launches of the current call deliver
    unsigned *out_marks = nullptr;                  // page-locked: one a slot of the result staging (k_mark)
    unsigned out_mark = 0;                          // the last value used
    std::vector<std::unique_ptr<mkf::BatchGraph>> graphs;
    mkf::Timer timers[3];
    unsigned long long *stamps = nullptr;       // their rings, page-locked
    mkf::Stamp stamp_due;                       // of the next launch on the context's stream
    double ms_per_tick = 0.0;
    std::unique_ptr<mkf::Server, mkf::ServerDeleter> server;
};

namespace mkf {

// context-level helpers used by the ABI and the scheduler
// the counts and pointers of an event (its shape); values are checked by pack_event
mkf_status validate_event(const mkf_ctx *ctx, const mkf_event *ev, EventShape *shape);
// the event's inputs, checked and narrowed to FP32, in its device layout
// (event_input_bytes of them)
enum class PackPart { kAll, kHits, kRows };   // all inputs, the hits alone, the seeds and tracks
mkf_status pack_event(const mkf_event *ev, const EventShape &shape, int geo, void *image, int threads,
                      std::string *why, PackPart part = PackPart::kAll);
// Host threads worth using for packing that many FP64 values, up to 16.  One
// packs 3 to 4.5 values a nanosecond, and waking others takes 30 to 50 us: a
// load of 7,001 seeds (460,000 values) takes 102 us to pack on one thread, 131
// on two, 117 on eight.  A submit to the server, whose staging is colder, packs
// 717,000 values in 151 us on one thread, 142 on two, 116 on four.
constexpr size_t kLoadValuesPerThread = 1500000, kServeValuesPerThread = 400000;
int pack_threads(size_t n_values, size_t per_thread);
// Touches the pages of new page-locked memory (contents undefined) on several
// host threads.  The host's first touch of a page takes 1.4 us: 32 MB 10.9 ms
// on one thread, 3.9 on four, 1.9 on sixteen, and a single thread that packs
// into the memory or copies out of it would bear it all.  Reads only: another
// thread may be using some of them already.  p: where a page starts.
void touch_pages(const void *p, size_t bytes);
mkf_status create_event(mkf_ctx *ctx, const EventShape &shape, DeviceHeap *heap, std::unique_ptr<EventRec> *out);
size_t event_view_offset(const EventShape &s);   // of the event's descriptor in its packed inputs
mkf_status upload_packed(EventRec *rec, void *image, hipStream_t s);
void destroy_event(mkf_ctx *ctx, EventRec *rec);
mkf_status ensure_index(mkf_ctx *ctx, EventRec *rec, bool *rebuilt, hipStream_t s);
mkf_status ensure_index_grid(mkf_ctx *ctx, EventRec *rec, int bins_phi, int bins_z, bool *rebuilt, hipStream_t s);
mkf_status compose_batch(EventRec *const *recs, int n, int spi, bool beam, char *image, char *dev, BatchArgs *args);
mkf_status stage_batch(mkf_ctx *ctx, const std::vector<EventRec *> &recs, void *dev, void *host, int spi,
                       BatchArgs *args, hipStream_t s, bool beam = false);
mkf_status ensure_beam(mkf_ctx *ctx, EventRec *rec);
size_t batch_scratch_bytes(int n_events);
int resolve_lanes(const mkf_ctx *ctx);
// Seeds of a wavefront's work item, up to 64 / G lanes' worth: as many as keep
// the batch's wavefronts resident at once (4,096; one a SIMD, 1,024, of the
// deep-layer kernels, which gain nothing from more), for fewer search rounds
// and smaller selections in each; at least five (fewer gain nothing) and ten
// lanes; a divisor of kSeedBlock.
// Measured (us; 6 candidates, ten / five seeds): 500 seeds 37.4 / 35.9, 5,000
// 46.2 / 44.5, 20,000 68.4 / 62.4, on disks 123 / 94, but 40,000 82 / 116; one
// candidate (64 / 16 / 10 / 5 seeds): 5,000 43 / 38 / 38 / 38, 20,000 59 / 43
// / 42 / 48; deep layers 5,000 78 / 71, 20,000 (ten / eight)
// 135 / 137.
int seeds_per_item(int geo, int G, long long seeds);
int seeds_per_item(int geo, int G, EventRec *const *recs, int n);
// The batched pipeline on stream s: optional counter reset and re-index, then
// the build and the final fit.  `d`: the way out of the results, which the
// build launches then overlap, `loads` the events' sizes for it.  Serving keeps its own parameters and shapes.
class Delivery;
struct EventLoad {
    int seeds;
    int layer_hits;   // of its fullest layer
};
// The rows each part of a batch ends at, and the work items before a row: see
// their definitions.  Rows leave at the host link's rate, or at that of one
// host thread copying them out of the staging.
constexpr double kLinkBytesPerUs = 55e3, kCopyBytesPerUs = 28e3;
std::vector<long long> plan_parts(const std::vector<EventLoad> &loads, const Params &P, double us_per_row);
int items_before(const std::vector<EventLoad> &loads, long long rows, int spi);
mkf_status run_pipeline(mkf_ctx *ctx, const Params &P, const mkf_tuning &t, const BatchArgs &args, uint32_t flags,
                        bool timed, hipStream_t s, Delivery *d = nullptr, const std::vector<EventLoad> &loads = {});
// The fields of a result row (par, cov, chi2 in FP64, then hits, n_hits,
// n_holes, ndof, status): bytes per row, array in mkf_tracks, array of a job.
constexpr int kOutFields = 8;
constexpr int kOutDoubles = 3;
size_t field_bytes(int f, int n_layers);
void *field_of(const mkf_tracks &t, int f);
void set_field(DeliverJob &j, int f, void *p);
// the device's address of `bytes` of host memory at p when all of it is
// page-locked for this device (or device memory of it) and p a multiple of
// `align`, else null; with `host`, the allocation it lies in too
void *device_writable(void *p, size_t bytes, size_t align, int device, char **host = nullptr, size_t *range = nullptr,
                      char **dev = nullptr);
void shutdown_server(mkf_ctx *ctx);

}  // namespace mkf
