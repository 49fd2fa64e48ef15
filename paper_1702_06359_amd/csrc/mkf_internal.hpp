// Internal structures shared by the HIP kernels and the host runtime.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/mkf.h"

namespace mkf {

constexpr int kMaxLayers = MKF_MAX_LAYERS;
constexpr int kMaxCands = MKF_MAX_CANDS;
constexpr int kWave = 64;
constexpr uint32_t kHoleId = 0xFFFFFFu;   // hit-id field of a hole or stopped entry
constexpr int kMaxHitsPerLayer = 0xFFFFFE;

// Per-layer geometry and the hit-index grid, in FP32 as the kernels use it.
// The grid's second coordinate is z on a cylinder and r on a disk.
struct LayerParam {
    float r;           // cylinder radius; disk outer radius
    float half_z;
    float x0;
    float inv_dphi;    // bins_phi / (2 pi)
    float inv_dz;      // bins_z / extent of the second coordinate
    float inv_r;
    float grid_lo;     // lower edge of the second coordinate: -half_z, or the disk's r_min
    float zplane;      // disk plane
    int kind;          // 0 cylinder, 1 disk
    float half_thick;  // half the layer's depth (radial or along z); 0: hits on the surface
    int pad[2];
};

// Building and fitting parameters for one launch.
struct Params {
    LayerParam layer[kMaxLayers];
    int n_layers;
    int n_seed_layers;
    int max_cands;
    int max_holes;
    int hole_always;
    int bins_phi;
    int bins_z;
    int geo;             // bit 0: every layer a disk (else a cylinder); bit 1: hits carry (x, y, z) and every
                         // pair is carried to the hit's surface (thick layers, or the 3x3 measurement)
    float w_per_qpt;     // -kappa * B: curvature w = w_per_qpt * q/pT
    float var_u;         // sigma_rphi^2
    float var_z;         // sigma_z^2
    float chi2_cut;
    float mass2;         // scattering mass hypothesis squared
    float win_scale;     // (1 + window margin)
    float var_r;         // sigma_r^2 (disks; the radial axis of the 3x3 measurement)
    int update3d;        // 3x3 global-Cartesian measurement (needs the (x, y, z) hit layout)
};

// Device view of one loaded event.  All pointers are device pointers.
struct DevEvent {
    int n_layers;
    int n_seeds;
    int n_tracks;
    int n_hits;                          // all layers
    int layer_off[kMaxLayers + 1];       // first hit of each layer in the flat hit arrays
    const float4 *hits;                  // [n_hits] caller order, packed by the host from the FP64 input:
                                         // (cos phi_h, sin phi_h, z, r) on a cylinder, (cos, sin, r, z) on a
                                         // disk; (x, y, z, 0) for thick layers and the 3x3 measurement
    float4 *binned;                      // [n_hits] grouped by layer then bin: (c, s, z or r, id bits)
    int *bin_of;                         // [n_hits] bin of each caller-order hit
    // the bucketed index build's working arrays (k_index_hist, _part, _place)
    float4 *part;                        // [n_hits] hits grouped by layer then bucket, as in `binned`; null: none
    int *part_bin;                       // [n_hits] and their bins
    int *hist;                           // [n_layers][idx_chunks][kBuckets] hits per chunk and bucket
    int *bucket_off;                     // [n_layers][kBuckets + 1] first hit of each bucket in its layer
    int *bin_off;                        // [n_layers][bin_off_stride(n_bins)]: n_bins + 1 absolute indices into
                                         // `binned` per layer
    const float *seed_par;               // [n_seeds][6]
    const float *seed_cov;               // [n_seeds][21]
    const int *seed_hits;                // [n_seeds][n_seed_layers]
    const int *seed_order;               // [n_seeds] the seeds by azimuth of their direction: the batched
                                         // builder takes them in this order
    const float *track_par;              // [n_tracks][6]
    const float *track_cov;              // [n_tracks][21]
    const int *track_hits;               // [n_tracks][n_layers]
    // results, FP32: one record of kRecWords words per row (see below), widened to FP64 on their way out
    float *out_rec;                      // [n_seeds] build
    int *out_hits;                       // [n_seeds][n_layers]
    float *fit_rec;                      // [n_tracks] fit
    float *rf_rec;                       // [n_seeds] final fit of the built tracks
    // the whole final beam (set only for a build that asks for it; null otherwise)
    float *beam_rec;                     // [n_seeds * max_cands]
    int *beam_hits;                      // [n_seeds * max_cands][n_layers]
    unsigned long long *stats;           // [5] mkf_build_stats counters
    // plain per-layer builder state (slots = n_seeds * lanes_per_seed)
    float *st_par;                       // [6][slots]
    float *st_cov;                       // [21][slots]
    float *st_trig;                      // [4][slots] sin, cos of phi and theta
    float *st_chi2;                      // [slots]
    int *st_meta;                        // [slots]
    int *st_hist;                        // [n_layers][slots] parent rank << 24 | hit (0xFFFFFF: hole)
    int st_slots;
    int grid_k;                          // the event's bin grid: (bins_phi >> grid_k) x (bins_z >> grid_k)
    int bucket_shift;                    // log2 of the bins of a bucket
    int idx_chunk, idx_chunks;           // hits of a chunk of a layer; chunks of the fullest layer
};

// The bucketed index build sorts a layer's hits by bucket (a run of
// 2^bucket_shift bins, at most kBuckets of them) and then each bucket by bin.
// A chunk is the hits one block counts: 2,048, more for layers over kBuckets
// chunks' worth, so that a block sums at most 64 x 64 counts.
constexpr int kBuckets = 64;
constexpr int kBlockThreads = 256;
inline int bucket_shift_of(int n_bins)
{
    int s = 3;   // a bucket's first bin offset is 16-byte aligned, its counts come in eights
    while ((kBuckets << s) < n_bins) ++s;
    return s;
}
inline int idx_chunk_of(int max_layer_hits)
{
    const int most = (max_layer_hits + 63) / 64;
    const int c = most > 2048 ? most : 2048;
    return (c + kBlockThreads - 1) / kBlockThreads * kBlockThreads;
}

// A result row on the device: the state (6 words), the packed covariance
// (21), then the words named here; the counts and the status are integer
// bits.  32 words are one 128-byte cache line, so that a row written by one
// lane in an arbitrary order of rows (the batched builder takes the seeds in
// azimuth order) leaves the L2 as a whole line, and rows are half the size of
// the FP64 arrays the caller gets.
constexpr int kRecWords = 32;
enum : int {
    kRecCov = 6,
    kRecChi2 = 27,
    kRecHits = 28,      // hits on the track / updates of a fit
    kRecHoles = 29,
    kRecStatus = 30,    // -1: no candidate at that rank of the beam
};

// Result rows on their way to the caller's arrays (k_deliver): n rows from
// `rec` and `hits`, the arrays in memory the device can write (page-locked
// host memory), any of them null when not wanted.
struct DeliverJob {
    const float *rec;
    const int *hits;         // [n][n_layers]
    double *par, *cov, *chi2;
    int *hits_out, *n_hits, *n_holes, *ndof, *status;
    int n;
    int first_tile;          // tiles of the launch before this job's
};
constexpr int kDeliverTile = kWave;   // rows a wavefront moves at a time
constexpr int kDeliverJobs = 32;      // jobs of one launch
template <int kJobs>
struct DeliverArgsT {
    int n_jobs;
    int n_tiles;
    int n_layers;
    DeliverJob job[kJobs];
};
typedef DeliverArgsT<kDeliverJobs> DeliverArgs;

// Largest layer and bin grid of some events.
struct IndexExtent {
    int layer_hits = 0;
    int bins = 0;
    int events = 0;
    void add(int hits, int nb)
    {
        layer_hits = hits > layer_hits ? hits : layer_hits;
        bins = nb > bins ? nb : bins;
        ++events;
    }
};

// LDS counters of a layer indexed by one block: two 16-bit ones a word for
// layers of at most 65,535 hits.
inline size_t layer_block_lds(int layer_hits, int bins)
{
    return sizeof(int) * (size_t)(layer_hits <= 0xFFFF ? (bins + 1) / 2 : bins);
}
constexpr size_t kLayerBlockLds = size_t(128) << 10;   // of a block's 160 KB
inline bool layer_block_fits(int layer_hits, int bins) { return layer_block_lds(layer_hits, bins) <= kLayerBlockLds; }

// A batch: events plus the flattened work decomposition over them.
struct BatchArgs {
    const DevEvent *events;
    const int *item_prefix;      // [n_events + 1] work items (seed groups) before each event
    const int *hit_prefix;       // [n_events + 1] hits before each event
    const int *track_prefix;     // [n_events + 1] tracks before each event
    const int *seed_prefix;      // [n_events + 1] seeds before each event
    unsigned int *queue;         // work-queue counter (persistent kernels)
    int n_events;
    int total_items;
    int total_hits;
    int total_tracks;
    int total_seeds;
    int seeds_per_item;
    int first_item, end_item;    // the work items of a build launch (not a persistent one)
    // index launch shapes
    IndexExtent all;             // of every event
    IndexExtent layer_only;      // of the events without arrays for the bucketed build
    int max_chunks;              // most chunks and bins per bucket of the other events
    int max_bucket_shift;
};

// Ints per layer in the bin-offset array: its n_bins + 1 offsets, padded to
// a multiple of four so that every layer's row starts 16-byte aligned.
__host__ __device__ constexpr int bin_off_stride(int n_bins) { return (n_bins + 4) & ~3; }

// The bin grid of one event: the context's grid (bins_phi x bins_z, set for
// the fullest events) coarsened by halving both axes while the event's
// fullest layer keeps at least three bins per hit (the headline's 20,000-
// track events have three), both counts stay divisible, and at least 64
// azimuth bins and 2 rows remain.  Small events so get an index and windows
// sized for their hit density instead of an index as large as the largest.
inline int event_grid_shift(int max_layer_hits, int bins_phi, int bins_z)
{
    int k = 0;
    for (;;) {
        const int k1 = k + 1;
        if ((bins_phi >> k1) << k1 != bins_phi || (bins_z >> k1) << k1 != bins_z) break;
        if ((bins_phi >> k1) < 64 || (bins_z >> k1) < 2) break;
        if ((long long)(bins_phi >> k1) * (bins_z >> k1) < 3LL * max_layer_hits) break;
        k = k1;
    }
    return k;
}

// The batched builder takes the seeds of an event in azimuth order within
// blocks of this many rows, so that a batch can be built, and its rows
// delivered, in parts that are whole runs of rows.  A multiple of every
// seeds_per_item.  (Blocks against the order over a whole 20,000-seed event:
// 328.7 and 328.2 us for ten of them.)
constexpr int kSeedBlock = 10240;

// Batch descriptors of the no-allocation builder: a fixed device array per
// GPU (mkf_kernels.hip), as laid out for up to kNoAllocMaxEvents events.
constexpr int kNoAllocMaxEvents = 256;
constexpr size_t round_up_256(size_t b) { return (b + 255) & ~size_t(255); }
constexpr size_t kNoAllocScratchBytes =
    round_up_256(kNoAllocMaxEvents * sizeof(DevEvent)) + 4 * round_up_256((kNoAllocMaxEvents + 1) * sizeof(int)) + 256;
hipError_t noalloc_scratch_init(int device);   // with `device` current; once per device
void *noalloc_scratch(int device);              // its device address (null before init)

// Where a launch puts the time at its start (page-locked words; null: nowhere).
struct Stamp {
    unsigned long long *a = nullptr, *b = nullptr;
};

// Launch helpers implemented in mkf_kernels.hip.
size_t build_lds_bytes(int geo, int n_layers, int waves_per_block);   // dynamic LDS of a batched build block
hipError_t launch_fill_i32(int *ptr, int value, int n, hipStream_t s);
hipError_t launch_stamp(const Stamp &st, hipStream_t s);
hipError_t launch_mark(unsigned *flag, unsigned value, hipStream_t s);   // flag: page-locked
hipError_t launch_batch_zero(const BatchArgs &b, hipStream_t s);   // work counters of a batch
hipError_t launch_index(const Params &p, const BatchArgs &b, hipStream_t s, const Stamp &st = {});
// deliver: page-locked, unchanged until the launch has run, or null: rows that
// the launch delivers beside its build (not a persistent one)
hipError_t launch_build_batch(const Params &p, const BatchArgs &b, int lanes_per_seed, int waves_per_block,
                              int persistent, int n_blocks, bool stats, const DeliverArgs *deliver, hipStream_t s,
                              const Stamp &st = {});
hipError_t launch_build_layer(const Params &p, const DevEvent *ev_dev, const DevEvent &ev_host, int layer,
                              int lanes_per_seed, int seeds_per_wave, int waves_per_block, bool stats,
                              hipStream_t s);
hipError_t launch_fit(const Params &p, const BatchArgs &b, hipStream_t s, const Stamp &st = {});
hipError_t launch_refit(const Params &p, const BatchArgs &b, hipStream_t s, const Stamp &st = {});
hipError_t launch_deliver(const DeliverArgs &a, hipStream_t s, const Stamp &st = {});
hipError_t launch_copy(const void *src, void *dst, size_t bytes, hipStream_t s);
hipError_t launch_calib_fma(float *dst, int n_blocks, int iters, hipStream_t s);   // iters: multiple of 4
int calib_fma_chains();

}  // namespace mkf
