// HIP kernels of the Kalman-filter track builder and fit (gfx950): the hit
// index, the batched and the per-layer builders, the fit and the final fit
// of built tracks, on barrel cylinders or endcap disks, thin or of finite
// thickness, plus two calibration kernels (a streaming copy, an FP32
// multiply-add loop).
//
// Layout: one lane = one track candidate.  A seed owns G consecutive lanes
// (G = lanes_per_seed >= max_cands), so a wavefront carries 64/G seeds and a
// seed's beam never leaves its wavefront: ranking and pruning use lane
// shuffles only.  Candidate state (27 floats) lives in registers; the
// per-layer choice of every kept candidate (parent rank, hit) is recorded in
// LDS (batched builder) or device memory (per-layer builder) and unwound at
// the end to produce the hit list.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>

#include "mkf_device.hpp"

namespace mkf {

// ---------------------------------------------------------------------------
// small helpers

__device__ __forceinline__ int upper_bound_i32(const int *a, int n, int v)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] <= v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ unsigned long long shfl_xor_u64(unsigned long long v, int m)
{
    const unsigned lo = __shfl_xor((unsigned)v, m);
    const unsigned hi = __shfl_xor((unsigned)(v >> 32), m);
    return ((unsigned long long)hi << 32) | lo;
}

// Exclusive prefix sum over the wavefront with DPP moves (no LDS round
// trips): within each row of 16 lanes by shifts of 1, 2, 3, 4 and 8 lanes,
// then across rows by broadcasting lane 15 into rows 1 and 3 and lane 31
// into rows 2 and 3.  Disabled lanes of a step add 0.
__device__ __forceinline__ int wave_exclusive_sum(int x, int lane)
{
    (void)lane;
    int v = x;
    v += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, x, 0x113, 0xf, 0xf, true);   // row_shr:3
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xe, true);   // row_shr:4, banks 1-3
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xc, true);   // row_shr:8, banks 2-3
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, true);   // row_bcast:15 into rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, true);   // row_bcast:31 into rows 2, 3
    return v - x;
}

__global__ void k_fill_i32(int *__restrict__ p, int v, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// The device's wall clock (constant rate, one for the whole chip) at this
// place of a stream, to one or two words of page-locked host memory.
__global__ void k_stamp(unsigned long long *a, unsigned long long *b)
{
    const unsigned long long t = (unsigned long long)wall_clock64();
    __hip_atomic_store(a, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (b) __hip_atomic_store(b, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The same at the start of another kernel, from its first block: a phase that
// begins with a launch, or ends where the next launch begins, needs none of
// its own.
__device__ __forceinline__ void stamp_start(const Stamp &st)
{
    if (st.a == nullptr || (blockIdx.x | blockIdx.y | threadIdx.x) != 0) return;
    const unsigned long long t = (unsigned long long)wall_clock64();
    __hip_atomic_store(st.a, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (st.b) __hip_atomic_store(st.b, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Tells the host that everything before it in the stream has been done and is
// visible to it: the kernels before have finished and released their writes
// to the device (stream order), the fence passes them on to the host.
__global__ void k_mark(unsigned *flag, unsigned value)
{
    __threadfence_system();
    __hip_atomic_store(flag, value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Plain streaming copy used to calibrate memory-traffic counters.
__global__ void k_copy16(const float4 *__restrict__ src, float4 *__restrict__ dst, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

// FP32 multiply-add throughput of the vector ALUs: every lane runs
// kFmaChains independent chains x <- x a + b for `iters` rounds, with no
// memory traffic, and stores the sum of its chains (so nothing folds away).
constexpr int kFmaChains = 8;

__global__ void __launch_bounds__(256) k_calib_fma(float *__restrict__ out, int iters, float a, float b)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    float x[kFmaChains];
#pragma unroll
    for (int i = 0; i < kFmaChains; ++i) x[i] = (float)(t & 1023) * 1e-3f + (float)i;
    for (int it = 0; it < iters; it += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int i = 0; i < kFmaChains; ++i) x[i] = fmaf(x[i], a, b);
        }
    }
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < kFmaChains; ++i) sum += x[i];
    store_global(out + t, sum);
}

// Clears the per-event work counters of a batch (a kernel rather than a
// memset so that it can sit in a captured graph).
__global__ void k_batch_zero(const BatchArgs B)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g < B.n_events * 5) B.events[g / 5].stats[g % 5] = 0ull;
}

// Geometries the kernels are specialised for: bit 0 disks (else cylinders);
// bit 1 hits that carry their position (x, y, z), to whose own surface every
// (candidate, hit) pair is carried before its chi2 - layers of finite
// thickness (the two-step propagation) and the 3x3 measurement.
constexpr bool geo_disk(int geo) { return (geo & 1) != 0; }
constexpr bool geo_xyz(int geo) { return (geo & 2) != 0; }

// ---------------------------------------------------------------------------
// Hit index: per layer, hits are grouped by an (eta, phi) grid.  On a cylinder
// eta is a function of z, on a disk a function of r, so the grid is (z, phi)
// or (r, phi): bin = iz * bins_phi + iphi.  A counting sort over all events
// of a batch at once.

// An event's bin grid (event_grid_shift): bins_phi x bins_z, and the factor
// 2^-k that turns the context grid's per-layer scales into the event's
// (exact, so the scaled products round as the unscaled ones would).
struct EvGrid {
    int bp, bz;
    float sc;
};

__device__ __forceinline__ EvGrid ev_grid(const Params &P, CEvent &E)
{
    const int k = E.grid_k;
    return EvGrid{P.bins_phi >> k, P.bins_z >> k, __builtin_ldexpf(1.f, -k)};
}

// The bin of a hit as the host packed it: (cos phi_h, sin phi_h, g2, -) with
// g2 = z on a cylinder and r on a disk, or, on layers of finite thickness and
// for the 3x3 measurement, (x, y, z, 0), whose own surface the second
// propagation step needs.  bin = row * bins_phi + (phi bin).
__device__ __forceinline__ int bin_hit(const Params &P, const LayerParam &lp, const EvGrid &g, const float4 v)
{
    // the azimuth to 3.8e-7 rad: far inside the 1e-5 rad the search window
    // adds to its own azimuth range, which uses the same function
    const float phi = fast_atan2(v.y, v.x);
    const float g2 = geo_xyz(P.geo) ? (lp.kind ? sqrtf(fmaf(v.x, v.x, v.y * v.y)) : v.z) : v.z;
    int ip = (int)floorf((phi + kPi) * (lp.inv_dphi * g.sc));
    int iz = (int)floorf((g2 - lp.grid_lo) * (lp.inv_dz * g.sc));
    ip = min(max(ip, 0), g.bp - 1);
    iz = min(max(iz, 0), g.bz - 1);
    return iz * g.bp + ip;
}

// Bin counters in LDS: one 32-bit counter per bin, or two 16-bit counters per
// word when kShort (layers of at most 65,535 hits, so that neither half
// carries into the other).
template <bool kShort>
__device__ __forceinline__ int lds_count(const unsigned *s_cnt, int i)
{
    return kShort ? (int)((s_cnt[i >> 1] >> ((i & 1) * 16)) & 0xFFFFu) : (int)s_cnt[i];
}

// Adds one to counter `bin` and returns its previous value.
template <bool kShort>
__device__ __forceinline__ int lds_bump(unsigned *s_cnt, int bin)
{
    if (kShort) {
        const int sh = (bin & 1) * 16;
        return (int)((atomicAdd(&s_cnt[bin >> 1], 1u << sh) >> sh) & 0xFFFFu);
    }
    return (int)atomicAdd(&s_cnt[bin], 1u);
}

// In-place exclusive scan of the nr counters in s_cnt, starting from
// `carry`; each offset plus `gbase` is also written to gout[0, nr) as it is
// formed when gout is not null (16-byte aligned).  Each thread owns kPer (a multiple of 8)
// consecutive bins per step: one step for up to 1024 kPer bins in a block of
// 1024.  Every thread of the block calls it; it ends on a barrier.
template <bool kShort, int kPer>
__device__ __forceinline__ void lds_scan_counts(unsigned *s_cnt, int nr, int carry, int *s_wave, int *gout,
                                                int gbase)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
    const int nw = kShort ? (nr + 1) / 2 : nr;
    constexpr int kWords = kShort ? kPer / 2 : kPer;
    for (int base = 0; base < nr; base += blockDim.x * kPer) {
        const int b0 = base + threadIdx.x * kPer;   // a multiple of 8: its words are 16-byte aligned
        const int w0 = kShort ? b0 / 2 : b0;
        unsigned w[kWords];
        if (w0 + kWords <= nw) {
#pragma unroll
            for (int j = 0; j < kWords; j += 4) {
                const uint4 q = *reinterpret_cast<const uint4 *>(s_cnt + w0 + j);
                w[j] = q.x; w[j + 1] = q.y; w[j + 2] = q.z; w[j + 3] = q.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < kWords; ++j) w[j] = w0 + j < nw ? s_cnt[w0 + j] : 0u;
        }
        int v[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            v[j] = b0 + j >= nr ? 0 : kShort ? (int)((w[j >> 1] >> ((j & 1) * 16)) & 0xFFFFu) : (int)w[j];
        int sum = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) sum += v[j];
        int x = sum;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int t = __shfl_up(x, o);
            if (lane >= o) x += t;
        }
        if (lane == kWave - 1) s_wave[wave] = x;
        __syncthreads();
        if (wave == 0) {
            int t2 = lane < n_waves ? s_wave[lane] : 0;
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) {
                const int t = __shfl_up(t2, o);
                if (lane >= o) t2 += t;
            }
            if (lane < n_waves) s_wave[lane] = t2;
        }
        __syncthreads();
        int run = carry + (wave > 0 ? s_wave[wave - 1] : 0) + x - sum;
        int o[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            o[j] = run;
            if (kShort) {
                if (j & 1) w[j >> 1] |= (unsigned)run << 16;
                else w[j >> 1] = (unsigned)run;
            } else {
                w[j] = (unsigned)run;
            }
            run += v[j];
        }
        if (gout == nullptr) {
        } else if (b0 + kPer <= nr) {
#pragma unroll
            for (int j = 0; j < kPer; j += 4)
                store_global(reinterpret_cast<int4 *>(gout + b0 + j),
                             make_int4(gbase + o[j], gbase + o[j + 1], gbase + o[j + 2], gbase + o[j + 3]));
        } else {
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if (b0 + j < nr) store_global(gout + b0 + j, gbase + o[j]);
        }
        if (w0 + kWords <= nw) {
#pragma unroll
            for (int j = 0; j < kWords; j += 4)
                *reinterpret_cast<uint4 *>(s_cnt + w0 + j) = make_uint4(w[j], w[j + 1], w[j + 2], w[j + 3]);
        } else {
#pragma unroll
            for (int j = 0; j < kWords; ++j)
                if (w0 + j < nw) s_cnt[w0 + j] = w[j];
        }
        carry += s_wave[n_waves - 1];
        __syncthreads();
    }
}

// Hit index of one layer in one 1024-thread block per (event, layer), for
// batches of many (event, layer) pairs or of small layers (`only`: events
// without arrays for the bucketed build): every hit
// binned (bin_of kept) and counted with LDS atomics, the counts scanned in LDS
// (the offsets written out as they are formed), then every hit placed at its
// bin's running offset (a second LDS atomic), so that no rank is stored.  The
// order inside a bin is that of the atomics, which does not matter: every hit
// of a window is tested and ties are broken by hit index.  `kU` hits per
// thread and step, their loads issued together; the ragged end of the layer
// takes steps of one hit so that the full steps carry no bounds tests.  A
// thread reads back only the bins it wrote itself.
template <bool kShort>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4))) k_index_layer(const Params P,
                                                                                                   const BatchArgs B,
                                                                                                   int only,
                                                                                                   const Stamp st)
{
    extern __shared__ unsigned s_cnt[];
    __shared__ int s_wave[16];
    stamp_start(st);
    const int e = blockIdx.x / P.n_layers;
    const int L = blockIdx.x - e * P.n_layers;
    CEvent &E = event_desc(B.events, e);
    if (only && E.part) return;               // the whole block: the bucketed build has this event
    const int h0 = E.layer_off[L], n = E.layer_off[L + 1] - h0;
    const LayerParam lp = P.layer[L];
    const EvGrid g = ev_grid(P, E);
    const int nb = g.bp * g.bz;
    int *off = E.bin_off + L * bin_off_stride(nb);
    const float4 *hits = E.hits + h0;
    int *bin_of = E.bin_of + h0;
    float4 *binned = E.binned + h0;
    const int nw = kShort ? (nb + 1) / 2 : nb;
    for (int i = threadIdx.x; i < nw; i += blockDim.x) s_cnt[i] = 0u;
    __syncthreads();
    constexpr int kU = 8;
    const int stride = blockDim.x, step = kU * stride;
    const int n_full = n - n % step;
    for (int i = threadIdx.x; i < n_full; i += step) {
        float4 v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) v[u] = load_global(hits + i + u * stride);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int b = bin_hit(P, lp, g, v[u]);
            store_global(bin_of + i + u * stride, b);
            lds_bump<kShort>(s_cnt, b);
        }
    }
    for (int i = n_full + threadIdx.x; i < n; i += stride) {
        const int b = bin_hit(P, lp, g, load_global(hits + i));
        store_global(bin_of + i, b);
        lds_bump<kShort>(s_cnt, b);
    }
    __syncthreads();
    lds_scan_counts<kShort, 32>(s_cnt, nb, 0, s_wave, nullptr, 0);   // ends on a barrier
    // the offsets written out four consecutive bins per lane, so that each
    // store instruction covers one contiguous kilobyte
    for (int i = 4 * (int)threadIdx.x; i < nb; i += 4 * (int)blockDim.x) {
        if (i + 4 <= nb) {
            store_global(reinterpret_cast<int4 *>(off + i),
                         make_int4(h0 + lds_count<kShort>(s_cnt, i), h0 + lds_count<kShort>(s_cnt, i + 1),
                                   h0 + lds_count<kShort>(s_cnt, i + 2), h0 + lds_count<kShort>(s_cnt, i + 3)));
        } else {
            for (int j = i; j < nb; ++j) store_global(off + j, h0 + lds_count<kShort>(s_cnt, j));
        }
    }
    if (threadIdx.x == 0) off[nb] = h0 + n;
    __syncthreads();   // every offset read before the placement moves them
    for (int i = threadIdx.x; i < n_full; i += step) {
        int b[kU];
        float4 v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            b[u] = load_global(bin_of + i + u * stride);
            v[u] = load_global(hits + i + u * stride);
        }
        int pos[kU];   // all atomics of the step in flight before the stores
#pragma unroll
        for (int u = 0; u < kU; ++u) pos[u] = lds_bump<kShort>(s_cnt, b[u]);
#pragma unroll
        for (int u = 0; u < kU; ++u)
            store_global(binned + pos[u], make_float4(v[u].x, v[u].y, v[u].z, __int_as_float(i + u * stride)));
    }
    for (int i = n_full + threadIdx.x; i < n; i += stride) {
        const float4 v = load_global(hits + i);
        const int pos = lds_bump<kShort>(s_cnt, load_global(bin_of + i));
        store_global(binned + pos, make_float4(v.x, v.y, v.z, __int_as_float(i)));
    }
}

// The same for layers whose counters exceed a block's LDS, of events without
// arrays for the bucketed build (their memory was not to be had): one range of
// kIndexRange bins after the other, the layer's bins read twice for each.  The
// counter of a range's last bin ends, after the placement, at the offset of
// the next range's first.  Bound, as the form above, by one block's walk
// through the layer's hits: ten layers of 68,000 hits 141 us on 65,536 bins (two
// ranges), 304 on 262,144 (eight); the bucketed build 31 and 33, so an event
// asks for its arrays first.
constexpr int kIndexRange = (int)(kLayerBlockLds / sizeof(unsigned));

__global__ void __launch_bounds__(1024) k_index_ranges(const Params P, const BatchArgs B, int only, const Stamp st)
{
    extern __shared__ unsigned s_cnt[];
    __shared__ int s_wave[16];
    stamp_start(st);
    const int e = blockIdx.x / P.n_layers;
    const int L = blockIdx.x - e * P.n_layers;
    CEvent &E = event_desc(B.events, e);
    if (only && E.part) return;               // the whole block: the bucketed build has this event
    const int h0 = E.layer_off[L], n = E.layer_off[L + 1] - h0;
    const LayerParam lp = P.layer[L];
    const EvGrid g = ev_grid(P, E);
    const int nb = g.bp * g.bz;
    int *off = E.bin_off + L * bin_off_stride(nb);
    const float4 *hits = E.hits + h0;
    int *bin_of = E.bin_of + h0;
    float4 *binned = E.binned + h0;
    constexpr int kU = 4;
    const int tid = threadIdx.x, stride = blockDim.x, step = kU * stride;
    for (int base = tid; base < n; base += step) {
        float4 v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) v[u] = load_global(hits + min(base + u * stride, n - 1));
#pragma unroll
        for (int u = 0; u < kU; ++u)
            if (base + u * stride < n) store_global(bin_of + base + u * stride, bin_hit(P, lp, g, v[u]));
    }
    int first = 0;   // offset of the range's first bin in the layer
    for (int lo = 0; lo < nb; lo += kIndexRange) {
        const int nr = min(kIndexRange, nb - lo);
        for (int i = tid; i < nr; i += stride) s_cnt[i] = 0u;
        __syncthreads();
        for (int base = tid; base < n; base += step) {   // a thread reads the bins it wrote itself
            int b[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) b[u] = load_global(bin_of + (base + u * stride < n ? base + u * stride : base)) - lo;
#pragma unroll
            for (int u = 0; u < kU; ++u)
                if (base + u * stride < n && (unsigned)b[u] < (unsigned)nr) atomicAdd(&s_cnt[b[u]], 1u);
        }
        __syncthreads();
        lds_scan_counts<false, 32>(s_cnt, nr, first, s_wave, off + lo, h0);   // ends on a barrier
        for (int base = tid; base < n; base += step) {
            int b[kU];
            float4 v[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int i = base + u * stride < n ? base + u * stride : base;
                b[u] = load_global(bin_of + i) - lo;
                v[u] = load_global(hits + i);
            }
#pragma unroll
            for (int u = 0; u < kU; ++u)
                if (base + u * stride < n && (unsigned)b[u] < (unsigned)nr)
                    store_global(binned + atomicAdd(&s_cnt[b[u]], 1u),
                                 make_float4(v[u].x, v[u].y, v[u].z, __int_as_float(base + u * stride)));
        }
        __syncthreads();
        first = (int)s_cnt[nr - 1];
        __syncthreads();
    }
    if (tid == 0) store_global(off + nb, h0 + n);
}

// Hit index of layers that each get many blocks, in three launches.  First
// (k_index_hist) every chunk of a layer's hits is binned and its hits per
// bucket of bins counted in LDS; then (k_index_part) each chunk takes its place
// in every bucket from the counts of the chunks before it and writes its hits
// there; then (k_index_place) a block per bucket counts its hits per bin, scans
// the counts into the bin offsets and places the hits.  Every hit is read by
// one block per launch (splitting the bins over blocks that each read the
// whole layer instead took 51 us for one 50,000-track event, its time the
// 2 x 64 hits each thread went through whatever the split), no counter leaves
// LDS, and the last pass writes into one run of lines per block, which so
// leave its L2 whole.
__global__ void __launch_bounds__(kBlockThreads) k_index_hist(const Params P, const BatchArgs B, const Stamp st)
{
    __shared__ int s_n[kBuckets];
    stamp_start(st);
    const int e = blockIdx.y / P.n_layers;
    const int L = blockIdx.y - e * P.n_layers;
    CEvent &E = event_desc(B.events, e);
    const int h0 = E.layer_off[L], n = E.layer_off[L + 1] - h0;
    const int i0 = blockIdx.x * E.idx_chunk, i1 = min(i0 + E.idx_chunk, n);
    if (!E.part || i0 >= n) return;           // the whole block
    const LayerParam lp = P.layer[L];
    const EvGrid g = ev_grid(P, E);
    if (threadIdx.x < kBuckets) s_n[threadIdx.x] = 0;
    __syncthreads();
    const float4 *hits = E.hits + h0;
    int *bin_of = E.bin_of + h0;
    constexpr int kU = 8;
    for (int base = i0; base < i1; base += kU * kBlockThreads) {
        float4 v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) v[u] = load_global(hits + min(base + u * kBlockThreads + (int)threadIdx.x, i1 - 1));
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int i = base + u * kBlockThreads + threadIdx.x;
            const int b = bin_hit(P, lp, g, v[u]);
            if (i < i1) {
                store_global(bin_of + i, b);
                atomicAdd(&s_n[b >> E.bucket_shift], 1);
            }
        }
    }
    __syncthreads();
    if (threadIdx.x < kBuckets)
        store_global(E.hist + (L * E.idx_chunks + (int)blockIdx.x) * kBuckets + threadIdx.x, s_n[threadIdx.x]);
}

__global__ void __launch_bounds__(kBlockThreads) k_index_part(const Params P, const BatchArgs B)
{
    constexpr int kParts = kBlockThreads / kBuckets;   // threads that share the sums of a bucket
    __shared__ int s_before[kParts][kBuckets], s_all[kParts][kBuckets], s_next[kBuckets];
    const int e = blockIdx.y / P.n_layers;
    const int L = blockIdx.y - e * P.n_layers;
    CEvent &E = event_desc(B.events, e);
    const int h0 = E.layer_off[L], n = E.layer_off[L + 1] - h0;
    const int i0 = blockIdx.x * E.idx_chunk, i1 = min(i0 + E.idx_chunk, n);
    if (!E.part || i0 >= n) return;           // the whole block
    const int chunks = (n + E.idx_chunk - 1) / E.idx_chunk;
    const int b = threadIdx.x % kBuckets, part = threadIdx.x / kBuckets;
    const int *hist = E.hist + L * E.idx_chunks * kBuckets;
    int before = 0, all = 0;
    for (int c = part; c < chunks; c += kParts) {
        const int v = load_global(hist + c * kBuckets + b);
        all += v;
        before += c < (int)blockIdx.x ? v : 0;
    }
    s_before[part][b] = before;
    s_all[part][b] = all;
    __syncthreads();
    if (threadIdx.x < kBuckets) {   // one wavefront: kBuckets lanes
#pragma unroll
        for (int p = 1; p < kParts; ++p) {
            before += s_before[p][b];
            all += s_all[p][b];
        }
        const int start = wave_exclusive_sum(all, b);
        s_next[b] = start + before;
        if (blockIdx.x == 0) {
            store_global(E.bucket_off + L * (kBuckets + 1) + b, start);
            if (b == 0) store_global(E.bucket_off + L * (kBuckets + 1) + kBuckets, n);
        }
    }
    __syncthreads();
    const int *bin_of = E.bin_of + h0;
    const float4 *hits = E.hits + h0;
    float4 *part_hits = E.part + h0;
    int *part_bins = E.part_bin + h0;
    constexpr int kU = 8;
    for (int base = i0; base < i1; base += kU * kBlockThreads) {
        int bin[kU], pos[kU];
        float4 v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int i = min(base + u * kBlockThreads + (int)threadIdx.x, i1 - 1);
            bin[u] = load_global(bin_of + i);
            v[u] = load_global(hits + i);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u)
            pos[u] = base + u * kBlockThreads + (int)threadIdx.x < i1 ? atomicAdd(&s_next[bin[u] >> E.bucket_shift], 1)
                                                                    : -1;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (pos[u] < 0) continue;
            const int i = base + u * kBlockThreads + (int)threadIdx.x;
            store_global(part_hits + pos[u], make_float4(v[u].x, v[u].y, v[u].z, __int_as_float(i)));
            store_global(part_bins + pos[u], bin[u]);
        }
    }
}

__global__ void __launch_bounds__(kBlockThreads) k_index_place(const Params P, const BatchArgs B)
{
    extern __shared__ unsigned s_cnt[];
    __shared__ int s_wave[16];
    const int e = blockIdx.y / P.n_layers;
    const int L = blockIdx.y - e * P.n_layers;
    CEvent &E = event_desc(B.events, e);
    const EvGrid g = ev_grid(P, E);
    const int nb = g.bp * g.bz;
    const int lo = (int)blockIdx.x << E.bucket_shift;
    if (!E.part || lo >= nb) return;          // the whole block
    const int nr = min(1 << E.bucket_shift, nb - lo);
    const int h0 = E.layer_off[L], n = E.layer_off[L + 1] - h0;
    const int *edge = E.bucket_off + L * (kBuckets + 1) + blockIdx.x;
    const int s0 = n > 0 ? load_global(edge) : 0, s1 = n > 0 ? load_global(edge + 1) : 0;
    int *off = E.bin_off + L * bin_off_stride(nb);
    const float4 *part_hits = E.part + h0;
    const int *part_bins = E.part_bin + h0;
    float4 *binned = E.binned + h0;
    if (lo + nr == nb && threadIdx.x == 0) store_global(off + nb, h0 + n);
    // the bucket's first kP hits per thread stay in registers, their loads in
    // flight through the count and the scan; a fuller bucket reads the rest
    // twice
    constexpr int kP = 4;
    int bin[kP];
    float4 v[kP];
    const int first = s0 + (int)threadIdx.x;
#pragma unroll
    for (int u = 0; u < kP; ++u) {
        const int i = first + u * kBlockThreads;
        bin[u] = i < s1 ? load_global(part_bins + i) - lo : -1;
        v[u] = i < s1 ? load_global(part_hits + i) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int i = threadIdx.x; i < nr; i += kBlockThreads) s_cnt[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kP; ++u)
        if (bin[u] >= 0) atomicAdd(&s_cnt[bin[u]], 1u);
    for (int i = first + kP * kBlockThreads; i < s1; i += kBlockThreads) atomicAdd(&s_cnt[load_global(part_bins + i) - lo], 1u);
    __syncthreads();
    lds_scan_counts<false, 8>(s_cnt, nr, s0, s_wave, off + lo, h0);   // ends on a barrier
#pragma unroll
    for (int u = 0; u < kP; ++u)
        if (bin[u] >= 0) store_global(binned + atomicAdd(&s_cnt[bin[u]], 1u), v[u]);
    for (int i = first + kP * kBlockThreads; i < s1; i += kBlockThreads) {
        const float4 h = load_global(part_hits + i);
        store_global(binned + atomicAdd(&s_cnt[load_global(part_bins + i) - lo], 1u), h);
    }
}

// The blocks of a launch are dealt to the chip's eight XCDs in turn (block b
// runs on XCD b mod 8), and each XCD has its own L2.  Renumbering them so
// that every XCD takes one contiguous range of the work keeps what that
// range reads (the hits of the few events it covers) in that XCD's L2
// instead of every L2 holding a little of every event.  A bijection of
// [0, n) for any n; blocks of one XCD keep their dispatch order.
constexpr int kXcds = 8;

__device__ __forceinline__ int xcd_contiguous(int b, int n)
{
    const int q = n / kXcds, r = n % kXcds;
    const int x = b % kXcds;
    return x * q + min(x, r) + b / kXcds;
}

// ---------------------------------------------------------------------------
// Track building

struct Lane {
    float p[6];
    float c[21];
    Trig tg;           // sines and cosines of p[4] (phi) and p[5] (theta)
    float chi2;
    int n_hits;
    int n_holes;
    int status;
    int live;
    int stopped;
};

// Per-layer record of every kept candidate: parent rank << 24 | hit index
// (kHoleId for a hole).
struct Hist {
    int *rec;
    int stride;        // elements between layers
    __device__ void put(int L, int lane, int h, int parent) const
    {
        rec[L * stride + lane] = (parent << 24) | (h & (int)kHoleId);
    }
    __device__ int hit(int L, int lane) const
    {
        const int v = rec[L * stride + lane] & (int)kHoleId;
        return v == (int)kHoleId ? -1 : v;
    }
    __device__ int parent(int L, int lane) const { return (int)((unsigned)rec[L * stride + lane] >> 24); }
};

struct Count {
    unsigned long long prop = 0, chi2 = 0, acc = 0, upd = 0, scan = 0;
};

// ---------------------------------------------------------------------------
// Wavefront-cooperative hit search and beam selection.
//
// Each lane owns one candidate whose window is a few (z row, phi segment)
// runs of the binned hit array.  The non-empty runs of all lanes are listed
// in LDS with running offsets; the (candidate, hit) pairs they define are then
// evaluated 64 at a time, one pair per lane whatever candidate it belongs to,
// and the accepted ones are appended to an LDS list.  A wavefront's work so
// follows the total number of hits in its windows instead of its largest
// window, and no lane idles through another lane's chi2.  The next beam of
// every seed is then chosen straight from that list (plus each candidate's
// hole or stop entry) by rounds of LDS atomic minima over the child keys,
// one rank per round; when the list fills up first, it is cut down to the
// entries that can still make a beam.

constexpr int kRuns = 128;         // run records held before their pairs are evaluated
constexpr int kAcc = 2 * kWave;    // accepted entries held (two per lane) before the list is cut down

// kOwn rows of owner data per lane: 3 on thin layers ({x, y, z or r, chi2},
// {Cxx, Cxy, Cyy, Cxz}, {Cyz, Czz, du, dz}); 8 on thick ones, where every
// pair carries its candidate to the hit's own surface and so needs the whole
// predicted state ({x, y, z, chi2}, {q/pT, sin phi, cos phi, sin theta},
// {cos theta, phi, theta, C0}, then C1..C20), from which the kept children
// also take their parent's state.
template <int kOwn>
struct SearchLdsT {
    float4 own[kOwn][kWave];
    int4 run[kRuns];              // {first binned index, first pair index, owner lane, -}
    int2 acc[kAcc];               // {accumulated chi2 bits, hit id << 6 | owner lane}
    unsigned long long best[kWave + 1];   // per seed group: the best child key of the current round; + a sink
    int tally[kWave];             // per owner: child hit count << 16 | accepted entries
    int mark[kWave];              // run starting at each pair slot of the current round
};
template <int kGeo>
using SearchLds = SearchLdsT<geo_xyz(kGeo) ? 8 : 3>;

// LDS written by some lanes of a wavefront and read by others: the wavefront's
// LDS operations are executed in order, so it only takes a compiler barrier
// and the wait for outstanding LDS operations.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Issue priority of a wavefront through the phases of a layer step.  The
// prediction and the Kalman update are long runs of VALU work; the hit search
// and above all the beam selection spend most of their time waiting on LDS
// round trips and hit loads.  Raising the priority of the waiting phases lets
// a wavefront that comes out of a wait issue ahead of the wavefronts in their
// VALU runs (the SIMD picks the highest-priority ready wavefront), so its
// chain of waits ends sooner while the VALU runs fill the gaps.  The levels
// were chosen by timing the headline build; they change no result.
enum : int { kPrioVector = 0, kPrioWindow = 1, kPrioListing = 2, kPrioPairs = 1, kPrioSelect = 3 };
template <int kLevel>
__device__ __forceinline__ void wave_priority()
{
    __builtin_amdgcn_s_setprio(kLevel);
}

__device__ __forceinline__ int lanes_below(unsigned long long m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Inclusive prefix maximum over the wavefront of non-negative values, with
// DPP moves: within each row of 16 lanes by shifts of 1, 2, 4 and 8 lanes,
// then across rows by broadcasting lane 15 into rows 1 and 3 and lane 31
// into rows 2 and 3.  Lanes a move does not reach take 0, the identity.
__device__ __forceinline__ int wave_inclusive_max(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true));   // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true));   // row_shr:2
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true));   // row_shr:4
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true));   // row_shr:8
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, true));   // row_bcast:15 into rows 1, 3
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, true));   // row_bcast:31 into rows 2, 3
    return v;
}

template <int G, bool kStats, int kGeo>
struct WaveSearch {
    static constexpr bool kDisk = geo_disk(kGeo);
    static constexpr bool kXyz = geo_xyz(kGeo);
    static_assert(kAcc == 2 * kWave, "two accepted entries per lane");
    SearchLds<kGeo> &W;
    const float4 *bh;
    const Params &P;
    const int lane;
    Count &cnt;
    int n_runs = 0, n_pairs = 0, n_acc = 0;

    // Child key of accepted entry v and the seed group of its owner (the
    // owner's child hit count is the high half of its tally).
    __device__ __forceinline__ unsigned long long entry_key(const int2 v, int &grp) const
    {
        const int o = v.y & (kWave - 1);
        grp = o / G;
        return child_key(W.tally[o] >> 16, (unsigned)v.x, o - grp * G, (unsigned)v.y >> 6);
    }

    // Up to max_cands rounds over this lane's items (two adjacent slots of
    // the accepted list and one more key): round r takes the minimum key of
    // every seed group with LDS atomics, marks the item that holds it as
    // taken, and hands it to the group's lane of rank r (`mine`).  The items
    // of a group are distinct, so each round takes exactly one per group that
    // has any.  Items out of the round read a sink entry, so that the reads
    // of a round are issued together outside any branch; of two items of one
    // group in a lane only the smaller enters the round (the slots hold runs
    // of one candidate's pairs, so this halves the lanes that meet at one
    // address).  Program order suffices between the reads and writes of one
    // round: a wavefront's LDS instructions execute in order.  Which items are
    // live and which enter a round are kept as wavefront masks in scalar
    // registers, so that a round's bookkeeping is scalar work beside the
    // vector work of the other wavefronts.
    __device__ __forceinline__ void rounds(const unsigned long long (&key)[3], const int (&grp)[3], bool (&live)[3],
                                           bool (&taken)[3], unsigned long long &mine)
    {
        const int my_grp = lane / G, my_rank = lane - my_grp * G;
        mine = ~0ull;
        const unsigned long long L0i = __ballot(live[0]), L1i = __ballot(live[1]), L2i = __ballot(live[2]);
        unsigned long long L0 = L0i, L1 = L1i, L2 = L2i;
        // of slots 0 and 1 in one group, the larger waits while the smaller is live
        const bool same = grp[0] == grp[1];
        const unsigned long long Y0 = __ballot(same & (key[1] < key[0])), Y1 = __ballot(same & (key[0] < key[1]));
        for (int r = 0; r < P.max_cands; ++r) {
            if ((L0 | L1 | L2) == 0) break;
            const unsigned long long I0 = L0 & ~(Y0 & L1), I1 = L1 & ~(Y1 & L0), I2 = L2;
            const bool in0 = __builtin_amdgcn_inverse_ballot_w64(I0);
            const bool in1 = __builtin_amdgcn_inverse_ballot_w64(I1);
            const bool in2 = __builtin_amdgcn_inverse_ballot_w64(I2);
            const int a0 = in0 ? grp[0] : kWave, a1 = in1 ? grp[1] : kWave, a2 = in2 ? grp[2] : kWave;
            if (in0) atomicMin(&W.best[a0], key[0]);
            if (in1) atomicMin(&W.best[a1], key[1]);
            if (in2) atomicMin(&W.best[a2], key[2]);
            wave_lds_sync();
            const unsigned long long b0 = W.best[a0], b1 = W.best[a1], b2 = W.best[a2], bm = W.best[my_grp];
            L0 &= ~(__ballot(b0 == key[0]) & I0);
            L1 &= ~(__ballot(b1 == key[1]) & I1);
            L2 &= ~(__ballot(b2 == key[2]) & I2);
            mine = my_rank == r ? bm : mine;
            wave_lds_sync();
            if (my_rank == r) W.best[my_grp] = ~0ull;
            wave_lds_sync();
        }
        taken[0] |= __builtin_amdgcn_inverse_ballot_w64(L0i & ~L0);
        taken[1] |= __builtin_amdgcn_inverse_ballot_w64(L1i & ~L1);
        taken[2] |= __builtin_amdgcn_inverse_ballot_w64(L2i & ~L2);
        live[0] = __builtin_amdgcn_inverse_ballot_w64(L0);
        live[1] = __builtin_amdgcn_inverse_ballot_w64(L1);
        live[2] = __builtin_amdgcn_inverse_ballot_w64(L2);
    }

    // The accepted list is full: keep only its entries that are among the
    // max_cands best of their seed group so far (any other can no longer
    // make the beam), compacted to the front.
    __device__ __forceinline__ void prune()
    {
        wave_lds_sync();
        int2 v[2];
        unsigned long long key[3] = {~0ull, ~0ull, ~0ull};
        int grp[3] = {0, 0, 0};
        bool live[3] = {false, false, false}, taken[3] = {false, false, false};
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int e = 2 * lane + t;
            live[t] = e < n_acc;
            v[t] = live[t] ? W.acc[e] : make_int2(0, 0);
            if (live[t]) key[t] = entry_key(v[t], grp[t]);
        }
        unsigned long long mine;
        rounds(key, grp, live, taken, mine);
        const unsigned long long m0 = __ballot(taken[0]), m1 = __ballot(taken[1]);
        if (taken[0]) W.acc[lanes_below(m0)] = v[0];
        if (taken[1]) W.acc[__popcll(m0) + lanes_below(m1)] = v[1];
        n_acc = __popcll(m0) + __popcll(m1);
        wave_lds_sync();
    }

    // The next beam: the max_cands best children of every seed group among
    // its accepted entries and its candidates' own entries (`own_key`, ~0
    // for none; a hole or a stopped candidate).  Returns this lane's new
    // entry by its rank in the group (~0: none).
    __device__ __forceinline__ unsigned long long select(unsigned long long own_key)
    {
        wave_lds_sync();
        unsigned long long key[3] = {~0ull, ~0ull, own_key};
        int grp[3] = {0, 0, lane / G};
        bool live[3] = {false, false, own_key != ~0ull}, taken[3] = {false, false, false};
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int e = 2 * lane + t;
            live[t] = e < n_acc;
            if (live[t]) key[t] = entry_key(W.acc[e], grp[t]);
        }
        unsigned long long mine;
        rounds(key, grp, live, taken, mine);
        return mine;
    }

    // Pair slot t0 + lane of a round: its owner and hit (the load is left in
    // flight).  Runs starting in the round mark their slot; the other slots
    // continue the last run started before them.
    __device__ __forceinline__ bool fetch_pair(int t0, int &first, int &o, float4 &hv)
    {
        W.mark[lane] = -1;
        const int r = first + lane;
        const int start = r < n_runs ? W.run[r].y : 0x7FFFFFFF;
        const bool starts = start < t0 + kWave;
        if (starts) W.mark[start - t0] = r;
        const int prev = first - 1;
        first += __popcll(__ballot(starts));
        wave_lds_sync();
        // the last run starting at or before this slot: the marks rise with
        // the slot, so it is their prefix maximum
        const int last = wave_inclusive_max(W.mark[lane] + 1) - 1;
        const int rr = last >= 0 ? last : prev;
        const int pair = t0 + lane;
        const bool valid = pair < n_pairs;
        // every lane loads (a slot past the last pair, the first binned hit),
        // so that the load is issued and waited for outside any branch
        const int4 R = W.run[valid ? rr : 0];
        o = valid ? R.z : 0;
        hv = load_global(bh + (valid ? R.x + (pair - R.y) : 0));
        return valid;
    }

    // test one round's pairs (pair slot of this lane: valid, owner o, hit
    // hv) and append the accepted ones to the list
    __device__ __forceinline__ void test_round(const bool valid, const int o, const float4 hv)
    {
        bool ok = false;
        float tot = 0.f;
        const unsigned hid = (unsigned)__float_as_int(hv.w);   // every lane waits for its load here
        if (valid) {
            if constexpr (!kXyz) {
                const float4 a = W.own[0][o], b = W.own[1][o], c = W.own[2][o];
                const bool fwd = fmaf(a.x, hv.x, a.y * hv.y) > 0.f;
                if (kStats) {
                    cnt.scan++;
                    if (fabsf(hv.z - a.z) <= c.w && fabsf(fmaf(a.x, hv.y, -a.y * hv.x)) <= c.z && fwd)
                        cnt.chi2++;
                }
                const float c2 = kDisk ? hit_chi2_disk(a.x, a.y, b.x, b.y, b.z, hv.x, hv.y, hv.z, P.var_u, P.var_r)
                                       : hit_chi2(a.x, a.y, a.z, b.x, b.y, b.z, b.w, c.x, c.y, hv.x, hv.y, hv.z,
                                                  P.var_u, P.var_z);
                ok = fwd & (c2 < P.chi2_cut);
                tot = a.w + c2;
            } else {
                // two-step: the owner's prediction on the layer's average
                // surface, carried to this hit's own surface
                const float4 r0 = W.own[0][o], r1 = W.own[1][o], r2 = W.own[2][o];
                const bool fwd = fmaf(r0.x, hv.x, r0.y * hv.y) > 0.f;
                float c[21];
                c[0] = r2.w;
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    const float4 v = W.own[3 + i][o];
                    c[1 + 4 * i] = v.x;
                    c[2 + 4 * i] = v.y;
                    c[3 + 4 * i] = v.z;
                    c[4 + 4 * i] = v.w;
                }
                const float p[6] = {r0.x, r0.y, r0.z, r1.x, 0.f, 0.f};
                const Trig tg{r1.y, r1.z, r1.w, r2.x};
                const float rh = sqrtf(fmaf(hv.x, hv.x, hv.y * hv.y));
                const float irh = fast_rcp(rh);
                float np[6], F[6][6], sn, cn, cp[6];
                const bool reach = kDisk ? step_near_plane(p, tg, hv.z, P.w_per_qpt, np, F, sn, cn)
                                         : step_near_cyl(p, tg, rh, P.w_per_qpt, np, F, sn, cn);
                transport_pos<kDisk>(F, c, cp);
                const float ch = hv.x * irh, sh = hv.y * irh;
                const float c2 =
                    P.update3d ? hit_chi2_3d(np[0], np[1], np[2], cp[0], cp[1], cp[2], cp[3], cp[4], cp[5], hv.x,
                                             hv.y, hv.z, P.var_u, P.var_r, P.var_z)
                    : kDisk    ? hit_chi2_disk(np[0], np[1], cp[0], cp[1], cp[2], ch, sh, rh, P.var_u, P.var_r)
                               : hit_chi2(np[0], np[1], np[2], cp[0], cp[1], cp[2], cp[3], cp[4], cp[5], ch, sh,
                                          hv.z, P.var_u, P.var_z);
                if (kStats) {
                    cnt.scan++;
                    if (fwd && reach) cnt.chi2++;
                }
                ok = fwd & reach & (c2 < P.chi2_cut);
                tot = r0.w + c2;
            }
        }
        const unsigned long long am = __ballot(ok);
        const int n_new = __popcll(am);
        if (n_acc + n_new > kAcc) prune();   // leaves at most kWave entries
        if (ok) {
            W.acc[n_acc + lanes_below(am)] = make_int2(__float_as_int(tot), (int)((hid << 6) | (unsigned)o));
            atomicAdd(&W.tally[o], 1);
        }
        n_acc += n_new;
    }

    // evaluate every pair of the listed runs, one per lane and round; the hits
    // of the next round are loaded while this round's are tested.  Two rounds
    // per iteration, in alternating registers, so that the wait for a round's
    // hits falls after the next round's pair listing.
    __device__ __forceinline__ void evaluate()
    {
        if (n_pairs > 0) {
            wave_lds_sync();
            int first = 0;   // first run not yet started
            int oa, ob;
            float4 ha, hb;
            bool va = fetch_pair(0, first, oa, ha);
            for (int t0 = 0;; t0 += 2 * kWave) {
                const bool vb = fetch_pair(t0 + kWave, first, ob, hb);
                test_round(va, oa, ha);
                if (t0 + kWave >= n_pairs) break;
                va = fetch_pair(t0 + 2 * kWave, first, oa, ha);
                test_round(vb, ob, hb);
                if (t0 + 2 * kWave >= n_pairs) break;
            }
        }
        n_runs = 0;
        n_pairs = 0;
    }

    // list one run per lane (len 0: none)
    __device__ __forceinline__ void add_run(int beg, int len)
    {
        const unsigned long long m = __ballot(len > 0);
        const int n_new = __popcll(m);
        if (n_runs + n_new > kRuns || n_pairs >= (1 << 29)) evaluate();
        const int ex = wave_exclusive_sum(len, lane);
        if (len > 0) W.run[n_runs + lanes_below(m)] = make_int4(beg, n_pairs + ex, lane, 0);
        n_runs += n_new;
        n_pairs += __builtin_amdgcn_readlane(ex + len, kWave - 1);
    }
};

// Windowed search of layer L for the predicted state (pp, pc) of every lane
// with `predicted` set: the best K accepted hits of the lane in (lc, lid),
// sorted by accumulated chi2 then hit id; returns the lane's accepted count.
// All lanes of the wavefront must call it together.
// Half-widths of the window that holds every chi2 < cut hit of a surface,
// for a predicted position (x, y, z) with position covariance (cxx, cxy,
// cyy, czz): du along the layer, dz along the grid's second coordinate g2 (z,
// or r on a disk), and the bound x = du / r on the azimuth (inv_r: 1 / the
// cylinder's radius).
template <bool kDisk>
__device__ __forceinline__ void window_at(const Params &P, float x, float y, float z, float cxx, float cxy, float cyy,
                                          float czz, float inv_r, float scale, float &du, float &dz, float &g2,
                                          float &xr)
{
    {
        const float hd = 0.5f * (cxx - cyy);
        const float lmax = 0.5f * (cxx + cyy) + sqrtf(fmaf(hd, hd, cxy * cxy));
        if (!kDisk) {
            // the chi2 < cut ellipse lies inside |u| <= du, |dz| <= dz, since
            // S_uu(phi_h) <= lambda_max(C_xy) + V_u for every hit direction
            g2 = z;
            du = sqrtf(P.chi2_cut * (lmax + P.var_u)) * scale;
            dz = sqrtf(P.chi2_cut * (czz + P.var_z)) * scale;
            xr = du * inv_r;
        } else {
            // On a disk the position covariance has a radial part too.  Any
            // hit with chi2 < cut lies within d0 = sqrt(cut (lmax + max V))
            // of the predicted point, so its azimuth is within a0 = asin(d0 /
            // rp) of the prediction's.  The hit frame is the prediction's
            // (u_p, r_p) turned by that angle a, so sqrt(u_h^T C u_h) <=
            // sqrt(C_uu) + |a| sqrt(lmax) (likewise for r), which bounds
            // each residual separately: |rp sin a| <= du and
            // |r_h - rp cos a| <= dr.
            g2 = sqrtf(fmaf(x, x, y * y));
            const float irp = fast_rcp(g2);
            const float cp = x * irp, sp = y * irp;
            const float cuu = fmaf(sp * sp, cxx, fmaf(-2.f * sp * cp, cxy, cp * cp * cyy));
            const float crr = fmaf(cp * cp, cxx, fmaf(2.f * sp * cp, cxy, sp * sp * cyy));
            const float d0 = sqrtf(P.chi2_cut * (lmax + fmaxf(P.var_u, P.var_r))) * scale;
            const float x0 = d0 * irp;
            const float a0 = x0 >= 0.7f ? 0.5f * kPi : x0 * __builtin_amdgcn_rsqf(1.f - x0 * x0);
            const float sl = a0 * sqrtf(lmax);
            const float su = sqrtf(fmaxf(cuu, 0.f)) + sl, sr = sqrtf(fmaxf(crr, 0.f)) + sl;
            du = sqrtf(P.chi2_cut * fmaf(su, su, P.var_u)) * scale;
            // rp (1 - cos a) <= du^2 / rp for the low edge of the radius range
            dz = fmaf(du * du, irp, sqrtf(P.chi2_cut * fmaf(sr, sr, P.var_r)) * scale);
            xr = du * irp;
        }
    }
}

// |phi_h - phi| <= asin(x) <= x / sqrt(1 - x^2) for x = du / r
__device__ __forceinline__ float dphi_of(float xr)
{
    return (xr >= 0.7f || !(xr >= 0.f) ? 0.5f * kPi : xr * __builtin_amdgcn_rsqf(1.f - xr * xr)) + 1e-5f;
}

// Windowed search of layer L for the predicted state (pp, pc) of every lane
// with `predicted` set (summed chi2 `chi2`, `n_hits` hits so far): every
// accepted (candidate, hit) pair ends in the search's accepted list; returns
// the lane's accepted count.  All lanes of the wavefront must call it
// together.
template <int G, bool kStats, int kGeo>
__device__ __forceinline__ int search_layer(const float (&pp)[6], const float (&pc)[21], const Trig &tg, float chi2,
                                            int n_hits, bool predicted, int L, const LayerParam &lp, const Params &P,
                                            CEvent &E, int lane, WaveSearch<G, kStats, kGeo> &ws)
{
    SearchLds<kGeo> &W = ws.W;
    constexpr bool kDisk = geo_disk(kGeo), kXyz = geo_xyz(kGeo);
    const EvGrid gr = ev_grid(P, E);
    int n_rows = 0, izlo = 0, n_seg = 1, s0lo = 0, s0hi = -1, s1lo = 0, s1hi = -1;
    float du = 0.f, dz = 0.f, g2 = pp[2];
    if (predicted) {
        const float phipos = fast_atan2(pp[1], pp[0]);
        float lo, hi, g2lo, g2hi;   // azimuth offsets from phipos, second-coordinate range
        bool finite = isfinite(phipos);
        if constexpr (!kXyz) {
            float xr;
            window_at<kDisk>(P, pp[0], pp[1], pp[2], pc[sym(0, 0)], pc[sym(0, 1)], pc[sym(1, 1)], pc[sym(2, 2)],
                             lp.inv_r, P.win_scale, du, dz, g2, xr);
            hi = dphi_of(xr);
            lo = -hi;
            g2lo = g2 - dz;
            g2hi = g2 + dz;
        } else {
            // A thick layer's hits lie between two bounding surfaces: the
            // window is the union of the chi2 < cut windows at both (the
            // predicted point moves along the short arc between them and its
            // covariance changes quadratically with the step), widened by 10 %.
            lo = kInf;
            hi = -kInf;
            g2lo = kInf;
            g2hi = -kInf;
#pragma unroll
            for (int end = -1; end <= 1; end += 2) {
                const float where = (kDisk ? lp.zplane : lp.r) + (float)end * lp.half_thick;
                float np[6], F[6][6], sn, cn, cp[6];
                const bool reach = kDisk ? step_near_plane(pp, tg, where, P.w_per_qpt, np, F, sn, cn)
                                         : step_near_cyl(pp, tg, where, P.w_per_qpt, np, F, sn, cn);
                transport_pos<kDisk>(F, pc, cp);
                float due, dze, g2e, xre;
                window_at<kDisk>(P, np[0], np[1], np[2], cp[0], cp[1], cp[2], cp[5], fast_rcp(where),
                                 P.win_scale * 1.1f, due, dze, g2e, xre);
                const float off = wrap_pi(fast_atan2(np[1], np[0]) - phipos);
                const float dph = dphi_of(xre);
                lo = fminf(lo, off - dph);
                hi = fmaxf(hi, off + dph);
                g2lo = fminf(g2lo, g2e - dze);
                g2hi = fmaxf(g2hi, g2e + dze);
                finite = finite && reach;
            }
            if (!finite) {   // an edge out of reach: the whole layer
                finite = isfinite(phipos);
                lo = -kPi;
                hi = kPi;
                g2lo = -1e30f;
                g2hi = 1e30f;
            }
        }
        const int nphi = gr.bp;
        if (finite && isfinite(lo) && isfinite(hi) && !isnan(g2lo) && !isnan(g2hi)) {
            const float idphi = lp.inv_dphi * gr.sc, idz = lp.inv_dz * gr.sc;
            const int ilo = (int)floorf((phipos + lo + kPi) * idphi);
            const int ihi = (int)floorf((phipos + hi + kPi) * idphi);
            const float zlo = fmaxf((g2lo - 1e-4f - lp.grid_lo) * idz, -1.f);
            const float zhi = fminf((g2hi + 1e-4f - lp.grid_lo) * idz, (float)gr.bz);
            izlo = min(max((int)floorf(zlo), 0), gr.bz - 1);
            const int izhi = min(max((int)floorf(zhi), 0), gr.bz - 1);
            n_rows = izhi - izlo + 1;
            if (ihi - ilo + 1 >= nphi) {
                s0lo = 0;
                s0hi = nphi - 1;
            } else if (ilo < 0) {
                s0lo = ilo + nphi;
                s0hi = nphi - 1;
                s1lo = 0;
                s1hi = ihi;
                n_seg = 2;
            } else if (ihi >= nphi) {
                s0lo = ilo;
                s0hi = nphi - 1;
                s1lo = 0;
                s1hi = ihi - nphi;
                n_seg = 2;
            } else {
                s0lo = ilo;
                s0hi = ihi;
            }
        }
    }
    if constexpr (!kXyz) {
        W.own[0][lane] = make_float4(pp[0], pp[1], g2, chi2);
        W.own[1][lane] = make_float4(pc[sym(0, 0)], pc[sym(0, 1)], pc[sym(1, 1)], pc[sym(0, 2)]);
        W.own[2][lane] = make_float4(pc[sym(1, 2)], pc[sym(2, 2)], du, dz);
    } else {
        W.own[0][lane] = make_float4(pp[0], pp[1], pp[2], chi2);
        W.own[1][lane] = make_float4(pp[3], tg.sph, tg.cph, tg.sth);
        W.own[2][lane] = make_float4(tg.cth, pp[4], pp[5], pc[0]);
#pragma unroll
        for (int i = 0; i < 5; ++i)
            W.own[3 + i][lane] = make_float4(pc[1 + 4 * i], pc[2 + 4 * i], pc[3 + 4 * i], pc[4 + 4 * i]);
    }
    W.tally[lane] = (n_hits + 1) << 16;
    W.best[lane] = ~0ull;

    wave_priority<kPrioListing>();
    const int n_runs = n_rows * n_seg;
    const int *off = E.bin_off + L * bin_off_stride(gr.bp * gr.bz);
    // bin offsets of run q: [off[row + lo], off[row + hi + 1])
    auto run_bounds = [&](int q, int &b, int &e) {
        const int sg = n_seg == 2 ? (q & 1) : 0;
        const int row = (izlo + (n_seg == 2 ? q >> 1 : q)) * gr.bp;
        b = load_global(off + row + (sg ? s1lo : s0lo));
        e = load_global(off + row + (sg ? s1hi : s0hi) + 1);
    };
    int nb = 0, ne = 0;   // next run, loaded one iteration ahead
    if (n_runs > 0) run_bounds(0, nb, ne);
    for (int q = 0; __ballot(q < n_runs) != 0; ++q) {
        const int beg = nb, len = ne - nb;
        nb = ne = 0;
        if (q + 1 < n_runs) run_bounds(q + 1, nb, ne);
        ws.add_run(beg, len);
    }
    wave_priority<kPrioPairs>();
    ws.evaluate();
    wave_lds_sync();
    return W.tally[lane] & 0xFFFF;
}

__device__ __forceinline__ void init_lane(Lane &S, CEvent &E, const Params &P, int seed, bool first_slot)
{
    S.live = first_slot ? 1 : 0;
    S.stopped = 0;
    S.status = 0;
    S.n_holes = 0;
    S.chi2 = 0.f;
    S.n_hits = 0;
    S.tg = Trig{0.f, 1.f, 1.f, 0.f};
#pragma unroll
    for (int i = 0; i < 6; ++i) S.p[i] = 0.f;
#pragma unroll
    for (int i = 0; i < 21; ++i) S.c[i] = 0.f;
    if (!first_slot) return;
#pragma unroll
    for (int i = 0; i < 6; ++i) S.p[i] = load_global(E.seed_par + 6 * (size_t)seed + i);
#pragma unroll
    for (int i = 0; i < 21; ++i) S.c[i] = load_global(E.seed_cov + 21 * (size_t)seed + i);
    for (int L = 0; L < P.n_seed_layers; ++L) S.n_hits += load_global(E.seed_hits + (size_t)seed * P.n_seed_layers + L) >= 0;
    S.tg = trig_of(S.p);
}

// One building layer for every lane of a wavefront (Section 2: propagate the
// candidate to the next layer, collect compatible hits, branch; Section
// 3.2.1: re-rank and prune to max_cands per seed).
template <int G, bool kStats, int kGeo>
__device__ __forceinline__ void layer_step(Lane &S, const int L, const Params &P, CEvent &E,
                                           const int lane, const Hist &H, SearchLds<kGeo> &W, Count &cnt)
{
    constexpr bool kDisk = geo_disk(kGeo), kXyz = geo_xyz(kGeo);
    const int gbase = (lane / G) * G;
    const int slot = lane - gbase;
    const LayerParam lp = P.layer[L];
    const bool active = S.live && !S.stopped;

    // 1. scattering of the layer being left, propagation, transport.  The
    //    prediction replaces the state in place; a lane whose helix misses
    //    the layer keeps its state and stops.
    wave_priority<kPrioVector>();
    bool predicted = false;
    if (active) {
        float np[6], sn, cn;
        const bool ok = predict<kDisk>(S.p, S.tg, kDisk ? lp.zplane : lp.r, P.w_per_qpt, P.layer[L - 1].x0, P.mass2,
                                       np, sn, cn, S.c);
        if (kStats) cnt.prop++;
        if (ok) {
#pragma unroll
            for (int i = 0; i < 6; ++i) S.p[i] = np[i];
            S.tg.sph = sn;
            S.tg.cph = cn;
            predicted = true;
        } else {
            S.stopped = 1;
            S.status = 2;
        }
    }
    const float (&pp)[6] = S.p;
    const float (&pc)[21] = S.c;

    // 2. windowed hit search: every accepted hit child into the search's list
    wave_priority<kPrioWindow>();
    WaveSearch<G, kStats, kGeo> ws{W, E.binned, P, lane, cnt};
    const int nacc = search_layer<G, kStats, kGeo>(pp, pc, S.tg, S.chi2, S.n_hits, predicted, L, lp, P, E, lane, ws);
    if (kStats) cnt.acc += nacc;

    // 3. hole child, or stop on this surface (with the prediction as state)
    //    when neither a hit nor a hole is left
    const bool hole = predicted && (nacc == 0 || P.hole_always) && S.n_holes < P.max_holes;
    if (predicted && nacc == 0 && S.n_holes >= P.max_holes) {
        S.stopped = 1;
        S.status = 1;
    }
    const bool tail = S.live && (S.stopped || hole);

    // 4. keep the max_cands best children of the seed (accepted hits, and
    //    each candidate's hole or stop entry): the lane of rank r takes the
    //    r-th best key of its group
    wave_priority<kPrioSelect>();
    unsigned long long mine = ws.select(tail ? child_key(S.n_hits, __float_as_uint(S.chi2), slot, kHoleId) : ~0ull);
    if (slot >= P.max_cands || lane >= (kWave / G) * G) mine = ~0ull;

    // 5. each kept entry moves to the lane of its rank: fetch the parent's
    //    state and apply the Kalman update with the entry's hit
    wave_priority<kPrioVector>();
    const bool alive = mine != ~0ull;
    const int parent = alive ? key_parent(mine) : slot;
    const int src = alive ? gbase + parent : lane;
    const unsigned hid = key_hit(mine);
    const bool with_hit = alive && hid != kHoleId;
    float4 hv = make_float4(1.f, 0.f, 0.f, 0.f);
    if (with_hit) hv = load_global(E.hits + E.layer_off[L] + (int)hid);   // in flight during the shuffles
    if constexpr (!kXyz) {
#pragma unroll
        for (int i = 0; i < 6; ++i) S.p[i] = __shfl(S.p[i], src);
#pragma unroll
        for (int i = 0; i < 21; ++i) S.c[i] = __shfl(S.c[i], src);
        S.tg.sph = __shfl(S.tg.sph, src);
        S.tg.cph = __shfl(S.tg.cph, src);
        S.tg.sth = __shfl(S.tg.sth, src);
        S.tg.cth = __shfl(S.tg.cth, src);
    } else {
        // the whole prediction of every lane is still in the search LDS, so
        // no lane keeps its state in registers through the search
        const float4 r0 = W.own[0][src], r1 = W.own[1][src], r2 = W.own[2][src];
        S.p[0] = r0.x;
        S.p[1] = r0.y;
        S.p[2] = r0.z;
        S.p[3] = r1.x;
        S.p[4] = r2.y;
        S.p[5] = r2.z;
        S.tg = Trig{r1.y, r1.z, r1.w, r2.x};
        S.c[0] = r2.w;
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const float4 v = W.own[3 + i][src];
            S.c[1 + 4 * i] = v.x;
            S.c[2 + 4 * i] = v.y;
            S.c[3 + 4 * i] = v.z;
            S.c[4 + 4 * i] = v.w;
        }
    }
    const int p_holes = __shfl(S.n_holes, src);
    const int p_stopped = __shfl(S.stopped, src);
    const int p_status = __shfl(S.status, src);
    S.live = alive;
    if (!alive) return;
    S.n_hits = key_nhits(mine);
    S.chi2 = key_chi2(mine);
    S.n_holes = p_holes;
    S.stopped = p_stopped;
    S.status = p_status;
    if (with_hit) {
        if constexpr (!kXyz) {
            kf_update<kDisk>(S.p, S.c, S.tg, hv.x, hv.y, hv.z, P.var_u, kDisk ? P.var_r : P.var_z);
        } else {
            // second step to the hit's own surface, then the update there
            const float rh = sqrtf(fmaf(hv.x, hv.x, hv.y * hv.y));
            const float irh = fast_rcp(rh);
            float np[6], F[6][6], sn, cn;
            if (kDisk) step_near_plane(S.p, S.tg, hv.z, P.w_per_qpt, np, F, sn, cn);
            else step_near_cyl(S.p, S.tg, rh, P.w_per_qpt, np, F, sn, cn);
            transport<kDisk>(F, S.c);
#pragma unroll
            for (int i = 0; i < 6; ++i) S.p[i] = np[i];
            S.tg.sph = sn;
            S.tg.cph = cn;
            if (P.update3d) kf_update_3d<false>(S.p, S.c, S.tg, hv.x, hv.y, hv.z, P.var_u, P.var_r, P.var_z);
            else kf_update<kDisk>(S.p, S.c, S.tg, hv.x * irh, hv.y * irh, kDisk ? rh : hv.z, P.var_u,
                                  kDisk ? P.var_r : P.var_z);
        }
        if (kStats) cnt.upd++;
        H.put(L, lane, (int)hid, parent);
    } else {
        if (!p_stopped) S.n_holes += 1;
        H.put(L, lane, -1, parent);
    }
}

// One result row written by its own lane: eight 16-byte stores that fill its
// cache line.  `some` false: an empty row (zero state, counts and covariance).
__device__ __forceinline__ void store_record(float *rec, const float (&p)[6], const float (&c)[21], float chi2,
                                             int n_hits, int n_holes, int status, bool some)
{
    float w[kRecWords];
#pragma unroll
    for (int i = 0; i < 6; ++i) w[i] = some ? p[i] : 0.f;
#pragma unroll
    for (int i = 0; i < 21; ++i) w[kRecCov + i] = some ? c[i] : 0.f;
    w[kRecChi2] = some ? chi2 : 0.f;
    w[kRecHits] = __int_as_float(some ? n_hits : 0);
    w[kRecHoles] = __int_as_float(some ? n_holes : 0);
    w[kRecStatus] = __int_as_float(status);
    w[kRecWords - 1] = 0.f;
#pragma unroll
    for (int i = 0; i < kRecWords; i += 4)
        store_global(reinterpret_cast<float4 *>(rec + i), make_float4(w[i], w[i + 1], w[i + 2], w[i + 3]));
}

// Rank-0 candidate of each seed to the result rows, hit list unwound
// through the per-layer records.
template <int G>
__device__ __forceinline__ void finalize_lane(const Lane &S, const Params &P, CEvent &E, int lane,
                                              int seed, const Hist &H)
{
    const int gbase = (lane / G) * G;
    if (E.beam_rec && lane < (kWave / G) * G && seed < E.n_seeds && lane - gbase < P.max_cands) {
        // every rank of the final beam: rank r sits in lane gbase + r
        const int r = lane - gbase;
        const size_t b = (size_t)seed * P.max_cands + r;
        store_record(E.beam_rec + kRecWords * b, S.p, S.c, S.chi2, S.n_hits, S.n_holes, S.live ? S.status : -1,
                     S.live != 0);
        int *bh = E.beam_hits + b * P.n_layers;
        for (int L = 0; L < P.n_seed_layers; ++L)
            store_global(bh + L, S.live ? load_global(E.seed_hits + (size_t)seed * P.n_seed_layers + L) : -1);
        int cur = r;
        for (int L = P.n_layers - 1; L >= P.n_seed_layers; --L) {
            store_global(bh + L, S.live ? H.hit(L, gbase + cur) : -1);
            if (S.live) cur = H.parent(L, gbase + cur);
        }
    }
    if (lane != gbase || seed >= E.n_seeds) return;
    const size_t s = (size_t)seed;
    store_record(E.out_rec + kRecWords * s, S.p, S.c, S.chi2, S.n_hits, S.n_holes, S.status, true);
    int *oh = E.out_hits + s * P.n_layers;
    for (int L = 0; L < P.n_seed_layers; ++L) store_global(oh + L, load_global(E.seed_hits + s * P.n_seed_layers + L));
    int cur = 0;
    for (int L = P.n_layers - 1; L >= P.n_seed_layers; --L) {
        store_global(oh + L, H.hit(L, gbase + cur));
        cur = H.parent(L, gbase + cur);
    }
}

template <bool kStats>
__device__ __forceinline__ void flush_counts(const Count &cnt, CEvent &E, int lane)
{
    if (!kStats) return;
    unsigned long long v[5] = {cnt.prop, cnt.chi2, cnt.acc, cnt.upd, cnt.scan};
#pragma unroll
    for (int j = 0; j < 5; ++j) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) v[j] += shfl_xor_u64(v[j], o);
    }
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < 5; ++j) atomicAdd(&E.stats[j], v[j]);
    }
}

// LDS stride of a result row staged for 64 rows' contiguous way out: odd, so
// that the lanes' own rows fall on different banks.
constexpr int kRecLds = kRecWords + 1;

// ---------------------------------------------------------------------------
// Results to the caller: every field of the rows of several events widened to
// the ABI's types and written straight into page-locked host memory in one
// launch.  Bound by the host link (57 GB/s measured for one large copy): a
// copy per event and field instead leaves it idle between copies (57.6 MB of
// ten 20,000-track events, 80 copies: 1.83 ms; 165,000 rows of sixteen events
// in one launch: 0.85 ms, 55.8 GB/s).  A wavefront takes 64 rows: it reads
// them as one contiguous 8 KB run into LDS (row stride 33 words: no bank
// conflicts either way) and writes each field as one contiguous run, eight
// bytes a lane, so that the link carries whole 64-byte pieces whatever the
// field.  Up to 64 tiles are moved by four wavefronts each: one alone is held
// up by its own 40 stores (eight tiles 7.8 us, by four wavefronts 5.6).
// `t`: kWave * kRecLds words of the wavefront's own; it takes every `step`-th
// tile from `first` on.  kSplit > 1: of a block of kSplit wavefronts that move
// a tile together, the `part`-th.
template <int kSplit, class Args>
__device__ __forceinline__ void deliver_tiles(const Args &A, float *t, int first, int step, int lane, int part)
{
    static_assert(kSplit == 1 || kSplit == 4, "a wavefront, or four: state and counts, three thirds of the covariance");
    auto sync = [] {
        if constexpr (kSplit > 1) __syncthreads();
        else wave_lds_sync();
    };
    int j = 0;
    for (int tile = uniform(first); tile < A.n_tiles; tile += step) {
        while (j + 1 < A.n_jobs && A.job[j + 1].first_tile <= tile) ++j;
        const auto &J = A.job[j];
        const size_t r0 = (size_t)(tile - J.first_tile) * kDeliverTile;
        const int m = min(kDeliverTile, J.n - (int)r0);
        const float4 *src = reinterpret_cast<const float4 *>(J.rec + r0 * kRecWords);
        constexpr int kLoads = kRecWords / 4 / kSplit;
        float4 v[kLoads];
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const int w = (k * kSplit + part) * kWave + lane;
            v[k] = (w >> 3) < m ? load_global(src + w) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const int w = (k * kSplit + part) * kWave + lane;
            float *q = t + kRecLds * (w >> 3) + 4 * (w & 7);
            q[0] = v[k].x; q[1] = v[k].y; q[2] = v[k].z; q[3] = v[k].w;
        }
        sync();
        if (J.par && part == 0) {
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                const int w = k * kWave + lane, row = w / 6;
                if (row < m) store_global(J.par + r0 * 6 + w, (double)t[kRecLds * row + w - 6 * row]);
            }
        }
        if (J.cov && (kSplit == 1 || part > 0)) {
            constexpr int kStores = kSplit == 1 ? 21 : 7;
            const int k0 = kSplit == 1 ? 0 : (part - 1) * kStores;
#pragma unroll
            for (int k = 0; k < kStores; ++k) {
                const int w = (k0 + k) * kWave + lane, row = w / 21;
                if (row < m) store_global(J.cov + r0 * 21 + w, (double)t[kRecLds * row + kRecCov + w - 21 * row]);
            }
        }
        if (part == 0 && lane < m) {
            const float *row = t + kRecLds * lane;
            const size_t r = r0 + lane;
            const int nh = __float_as_int(row[kRecHits]), st = __float_as_int(row[kRecStatus]);
            if (J.chi2) store_global(J.chi2 + r, (double)row[kRecChi2]);
            if (J.n_hits) store_global(J.n_hits + r, nh);
            if (J.n_holes) store_global(J.n_holes + r, __float_as_int(row[kRecHoles]));
            // two measured coordinates per hit, minus the five track parameters
            if (J.ndof) store_global(J.ndof + r, st < 0 ? 0 : 2 * nh - 5);
            if (J.status) store_global(J.status + r, st);
        }
        if (J.hits_out) {
            const int n = m * A.n_layers;
            const int *src_h = J.hits + r0 * A.n_layers;
            for (int w = part * kWave + lane; w < n; w += kSplit * kWave)
                store_global(J.hits_out + r0 * A.n_layers + w, load_global(src_h + w));
        }
        sync();   // every row read before the next tile takes its place
    }
}

constexpr int kDeliverLds = kWave * kRecLds * (int)sizeof(float);   // per wavefront

template <int kJobs, int kSplit>
__global__ void __launch_bounds__(256) k_deliver(const DeliverArgsT<kJobs> A, const Stamp st)
{
    extern __shared__ int s_dyn[];
    stamp_start(st);
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    float *t = reinterpret_cast<float *>(s_dyn);
    if constexpr (kSplit > 1) {
        deliver_tiles<kSplit>(A, t, blockIdx.x, gridDim.x, lane, wave);
    } else {
        deliver_tiles<1>(A, t + wave * (kDeliverLds / (int)sizeof(float)), blockIdx.x * waves + wave,
                         gridDim.x * waves, lane, 0);
    }
}

// ---------------------------------------------------------------------------
// Dynamic LDS of the batched builder: the per-layer records of every wave
// (an int per lane and layer), then one SearchLds per wave.
__host__ __device__ constexpr int search_lds_offset(int waves, int n_layers)
{
    return waves * n_layers * kWave;   // in ints (a multiple of 64: 16-byte aligned)
}

// Batched builder.  Each wavefront takes work items (event, group of 64/G
// seeds) - from a device counter when persistent, else from its block index -
// and runs every building layer of its seeds with the state in registers.
// With `D` (page-locked; as 2.6 KB of arguments it made every launch 1.9 us
// later) one XCD's blocks, `deliver_blocks` of them, instead deliver the rows
// that the launch before built, and the other XCDs share the building: the
// host link works while the vector ALUs build, in one stream and with no
// event between.  One XCD fills the link (20,000 rows beside 42,000 seeds 119
// us, 102 the delivery alone), and its stores hold up only its own L2: spread
// over all XCDs the delivering wavefronts stalled every build's loads behind
// them (153 us, the sum of the two).
template <int G, bool kStats, int kGeo>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(geo_xyz(kGeo) ? 3 : 4))) k_build_batch(const Params P, const BatchArgs B, int persistent, const DeliverArgs *__restrict__ D, int deliver_blocks, const Stamp st)
{
    extern __shared__ int s_dyn[];
    stamp_start(st);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    const int W = blockDim.x >> 6;
    Hist H{s_dyn + wave * P.n_layers * kWave, kWave};
    SearchLds<kGeo> &SL = reinterpret_cast<SearchLds<kGeo> *>(s_dyn + search_lds_offset(W, P.n_layers))[wave];
    int item = B.first_item;
    if (deliver_blocks > 0) {
        // one XCD delivers, the others build
        const int x = blockIdx.x % kXcds, i = blockIdx.x / kXcds;
        if (x == 0) {
            typedef const __attribute__((address_space(4))) DeliverArgs CDeliver;
            if (i < deliver_blocks)
                deliver_tiles<1>(*(CDeliver *)D,
                                 reinterpret_cast<float *>(s_dyn) + wave * (kDeliverLds / (int)sizeof(float)),
                                 i * W + wave, deliver_blocks * W, lane, 0);
            return;
        }
        const int n = (B.end_item - B.first_item + W - 1) / W;   // building blocks
        const int q = n / (kXcds - 1), r = n % (kXcds - 1), y = x - 1;
        if (i >= q + (y < r ? 1 : 0)) return;
        item += (y * q + min(y, r) + i) * W + wave;
    } else {
        item += xcd_contiguous(blockIdx.x, gridDim.x) * W + wave;
    }
    for (;;) {
        if (persistent) {
            unsigned v = 0;
            if (lane == 0) v = atomicAdd(B.queue, 1u);
            item = (int)__shfl(v, 0);
        }
        item = uniform(item);
        if (item >= B.end_item) break;
        const int e = uniform(upper_bound_i32(B.item_prefix, B.n_events + 1, item) - 1);
        CEvent &E = event_desc(B.events, e);
        // the item's seeds, taken in azimuth order
        const int k = (item - B.item_prefix[e]) * B.seeds_per_item + lane / G;
        const bool valid = lane < B.seeds_per_item * G && k < E.n_seeds;
        const int seed = valid ? load_global(E.seed_order + k) : E.n_seeds;
        Lane S;
        init_lane(S, E, P, valid ? seed : 0, valid && lane % G == 0);
        Count cnt;
        for (int L = P.n_seed_layers; L < P.n_layers; ++L) layer_step<G, kStats, kGeo>(S, L, P, E, lane, H, SL, cnt);
        finalize_lane<G>(S, P, E, lane, valid ? seed : E.n_seeds, H);
        flush_counts<kStats>(cnt, E, lane);
        if (!persistent) break;
    }
}

// Per-layer builder: one event, one layer per launch, candidate state in
// device memory (structure of arrays, slot = seed * G + rank) between layers.
template <int G, bool kStats, int kGeo>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(geo_xyz(kGeo) ? 3 : 4))) k_build_layer(const Params P, const DevEvent *__restrict__ Ep, int L, int seeds_per_wave)
{
    CEvent &E = event_desc(Ep, 0);
    const int lane = threadIdx.x & (kWave - 1);
    const int item = uniform(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
    const int first = item * seeds_per_wave;
    if (first >= E.n_seeds) return;
    const int seed = first + lane / G;
    const bool valid = lane < seeds_per_wave * G && seed < E.n_seeds;
    const int ns = E.st_slots;
    const int slot = item * kWave + lane;
    Hist H{E.st_hist + item * kWave, ns};
    Lane S;
    if (L == P.n_seed_layers) {
        init_lane(S, E, P, valid ? seed : 0, valid && lane % G == 0);
    } else {
        // every lane's words in flight together, a dead one's (whatever its slot
        // holds) dropped after: loads that wait for `meta` made a layer of a
        // small event 0.8 us longer
        const int meta = load_global(E.st_meta + slot);
        const float chi2 = load_global(E.st_chi2 + slot);
        float p[6], c[21], tg[4];
#pragma unroll
        for (int i = 0; i < 6; ++i) p[i] = load_global(E.st_par + i * ns + slot);
#pragma unroll
        for (int i = 0; i < 21; ++i) c[i] = load_global(E.st_cov + i * ns + slot);
#pragma unroll
        for (int i = 0; i < 4; ++i) tg[i] = load_global(E.st_trig + i * ns + slot);
        S.live = meta & 1;
        S.stopped = (meta >> 1) & 1;
        S.status = (meta >> 2) & 3;
        S.n_hits = (meta >> 4) & 31;
        S.n_holes = (meta >> 9) & 15;
        S.chi2 = chi2;
#pragma unroll
        for (int i = 0; i < 6; ++i) S.p[i] = S.live ? p[i] : 0.f;
#pragma unroll
        for (int i = 0; i < 21; ++i) S.c[i] = S.live ? c[i] : 0.f;
        S.tg = S.live ? Trig{tg[0], tg[1], tg[2], tg[3]} : Trig{0.f, 1.f, 1.f, 0.f};
    }
    extern __shared__ int s_dyn[];
    SearchLds<kGeo> &SL = reinterpret_cast<SearchLds<kGeo> *>(s_dyn)[threadIdx.x >> 6];
    Count cnt;
    layer_step<G, kStats, kGeo>(S, L, P, E, lane, H, SL, cnt);
    if (L == P.n_layers - 1) {
        finalize_lane<G>(S, P, E, lane, valid ? seed : E.n_seeds, H);
    } else {
        store_global(E.st_meta + slot, S.live | (S.stopped << 1) | (S.status << 2) | (S.n_hits << 4) | (S.n_holes << 9));
        store_global(E.st_chi2 + slot, S.chi2);
        if (S.live) {
#pragma unroll
            for (int i = 0; i < 6; ++i) store_global(E.st_par + i * ns + slot, S.p[i]);
#pragma unroll
            for (int i = 0; i < 21; ++i) store_global(E.st_cov + i * ns + slot, S.c[i]);
            store_global(E.st_trig + 0 * ns + slot, S.tg.sph);
            store_global(E.st_trig + 1 * ns + slot, S.tg.cph);
            store_global(E.st_trig + 2 * ns + slot, S.tg.sth);
            store_global(E.st_trig + 3 * ns + slot, S.tg.cth);
        }
    }
    flush_counts<kStats>(cnt, E, lane);
}

// Updates of a fit taken in Joseph form: three hits (six measured
// coordinates) determine the five track parameters.
constexpr int kJosephUpdates = 3;

// ---------------------------------------------------------------------------
// KF fit over a fixed hit list: from the prior (p, c) on layer 0, for each
// layer the scattering of the previous one, propagation, transport, and the
// update with that layer's hit if it has one (hit_of(L) >= 0).  (op, oc) is
// the state after the last update.
template <int kGeo, class HitOf>
__device__ __forceinline__ void fit_track(const Params &P, CEvent &E, float (&p)[6], float (&c)[21],
                                          HitOf hit_of, float (&op)[6], float (&oc)[21], float &chi2, int &nupd,
                                          int &status)
{
#pragma unroll
    for (int i = 0; i < 6; ++i) op[i] = p[i];
#pragma unroll
    for (int i = 0; i < 21; ++i) oc[i] = c[i];
    chi2 = 0.f;
    nupd = 0;
    status = 0;
    // bit 2 of kGeo: the 3x3 measurement (fit kernels only; the build kernels
    // test it at run time)
    constexpr bool kDisk = geo_disk(kGeo), kXyz = geo_xyz(kGeo), kFit3d = (kGeo & 4) != 0;
    Trig tg = trig_of(p);
    if constexpr (!kXyz) {
        // Thin layers: the hit of layer L + 1 is loaded while layer L is
        // updated and layer L + 1 propagated to, by every lane (no hit: any
        // hit of the event, or the first word of its input block when it has
        // none), so that its latency hides behind that arithmetic.  Two
        // layers per iteration in alternating registers keep the wait for a
        // hit next to its use.
        const int nh1 = max(E.n_hits - 1, 0);
        auto hit_at = [&](int L, int h) { return load_global(E.hits + min(E.layer_off[L] + max(h, 0), nh1)); };
        auto step = [&](const int L, const int h, const float4 hv, int &h_next, float4 &hv_next) -> bool {
            const bool more = L + 1 < P.n_layers;
            h_next = more ? hit_of(L + 1) : -1;
            if (L > 0) {
                float np[6], sn, cn;
                if (!predict<kDisk>(p, tg, kDisk ? P.layer[L].zplane : P.layer[L].r, P.w_per_qpt,
                                    P.layer[L - 1].x0, P.mass2, np, sn, cn, c)) {
                    status = 2;
                    return false;
                }
                tg.sph = sn;
                tg.cph = cn;
#pragma unroll
                for (int i = 0; i < 6; ++i) p[i] = np[i];
            }
            if (more) hv_next = hit_at(L + 1, h_next);
            if (h >= 0) {
                // Joseph form for the first updates, as below
                if (nupd < kJosephUpdates) {
                    if (kFit3d) chi2 += kf_update_3d<true>(p, c, tg, hv.x, hv.y, hv.z, P.var_u, P.var_r, P.var_z);
                    else chi2 += kf_update_joseph<kDisk>(p, c, tg, hv.x, hv.y, hv.z, P.var_u, kDisk ? P.var_r : P.var_z);
                } else {
                    if (kFit3d) chi2 += kf_update_3d<false>(p, c, tg, hv.x, hv.y, hv.z, P.var_u, P.var_r, P.var_z);
                    else chi2 += kf_update<kDisk>(p, c, tg, hv.x, hv.y, hv.z, P.var_u, kDisk ? P.var_r : P.var_z);
                }
                ++nupd;
#pragma unroll
                for (int i = 0; i < 6; ++i) op[i] = p[i];
#pragma unroll
                for (int i = 0; i < 21; ++i) oc[i] = c[i];
            }
            return true;
        };
        int ha = hit_of(0), hb = -1;
        float4 va = hit_at(0, ha), vb = va;
        for (int L = 0; L < P.n_layers; L += 2) {
            if (!step(L, ha, va, hb, vb) || L + 1 >= P.n_layers) break;
            if (!step(L + 1, hb, vb, ha, va)) break;
        }
        return;
    }
    for (int L = 0; L < P.n_layers; ++L) {
        const int h = hit_of(L);
        float4 hv = make_float4(1.f, 0.f, 0.f, 0.f);
        float where = kDisk ? P.layer[L].zplane : P.layer[L].r;
        if constexpr (kXyz) {
            // the hit carries (x, y, z): its own surface is the target (the
            // two steps composed)
            if (h >= 0) {
                hv = load_global(E.hits + E.layer_off[L] + h);
                where = kDisk ? hv.z : sqrtf(fmaf(hv.x, hv.x, hv.y * hv.y));
            }
        }
        if (L > 0) {
            float np[6], sn, cn;
            if (!predict<kDisk>(p, tg, where, P.w_per_qpt, P.layer[L - 1].x0, P.mass2, np, sn, cn, c)) {
                status = 2;
                break;
            }
            tg.sph = sn;
            tg.cph = cn;
#pragma unroll
            for (int i = 0; i < 6; ++i) p[i] = np[i];
        }
        if (h >= 0) {
            float ch, sh, g2h;
            if constexpr (kXyz) {
                hv = load_global(E.hits + E.layer_off[L] + h);   // again: short live range across the step
                const float rh = sqrtf(fmaf(hv.x, hv.x, hv.y * hv.y));
                const float irh = fast_rcp(rh);
                ch = hv.x * irh;
                sh = hv.y * irh;
                g2h = kDisk ? rh : hv.z;
            } else {
                hv = load_global(E.hits + E.layer_off[L] + h);
                ch = hv.x;
                sh = hv.y;
                g2h = hv.z;
            }
            // A fit starts from a wide prior: until a few hits have pinned
            // the five parameters, C - K H C subtracts nearly equal numbers
            // and would lose FP32 digits, so those updates take the Joseph
            // form; after them the prediction is about as precise as a hit
            // and the plain form keeps its digits.
            if (nupd < kJosephUpdates) {
                if (kFit3d) chi2 += kf_update_3d<true>(p, c, tg, hv.x, hv.y, hv.z, P.var_u, P.var_r, P.var_z);
                else chi2 += kf_update_joseph<kDisk>(p, c, tg, ch, sh, g2h, P.var_u, kDisk ? P.var_r : P.var_z);
            } else {
                if (kFit3d) chi2 += kf_update_3d<false>(p, c, tg, hv.x, hv.y, hv.z, P.var_u, P.var_r, P.var_z);
                else chi2 += kf_update<kDisk>(p, c, tg, ch, sh, g2h, P.var_u, kDisk ? P.var_r : P.var_z);
            }
            ++nupd;
#pragma unroll
            for (int i = 0; i < 6; ++i) op[i] = p[i];
#pragma unroll
            for (int i = 0; i < 21; ++i) oc[i] = c[i];
        }
    }
}

// One track of a fit with known hits, prior read and results written per
// lane.
template <int kGeo>
__device__ __forceinline__ void fit_known(const Params &P, CEvent &E, const size_t t)
{
    float p[6], c[21], op[6], oc[21], chi2;
    int nupd, status;
#pragma unroll
    for (int i = 0; i < 6; ++i) p[i] = load_global(E.track_par + 6 * t + i);
#pragma unroll
    for (int i = 0; i < 21; ++i) c[i] = load_global(E.track_cov + 21 * t + i);
    fit_track<kGeo>(P, E, p, c, [&](int L) { return load_global(E.track_hits + t * P.n_layers + L); }, op, oc,
                    chi2, nupd, status);
    store_record(E.fit_rec + kRecWords * t, op, oc, chi2, nupd, P.n_layers - nupd, status, true);
}

// The result rows of a wavefront's 64 consecutive tracks through LDS to
// `out`, each store instruction one contiguous kilobyte.  `stage`: room for
// kWave * kRecLds words that no lane needs any more.
__device__ __forceinline__ void store_records(float *stage, float *out, int lane, const float (&p)[6],
                                              const float (&c)[21], float chi2, int nupd, int holes, int status)
{
    float *row = stage + kRecLds * lane;
#pragma unroll
    for (int i = 0; i < 6; ++i) row[i] = p[i];
#pragma unroll
    for (int i = 0; i < 21; ++i) row[kRecCov + i] = c[i];
    row[kRecChi2] = chi2;
    row[kRecHits] = __int_as_float(nupd);
    row[kRecHoles] = __int_as_float(holes);
    row[kRecStatus] = __int_as_float(status);
    row[kRecWords - 1] = 0.f;
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < kRecWords / 4; ++k) {
        const int w = k * kWave + lane;   // 16-byte piece of the 64 rows
        const float *q = stage + kRecLds * (w >> 3) + 4 * (w & 7);
        store_global(reinterpret_cast<float4 *>(out) + w, make_float4(q[0], q[1], q[2], q[3]));
    }
}

// Dynamic LDS of the fit kernel per wavefront: the 27 priors and the hit
// indices of 64 tracks, later their result rows.
__host__ __device__ constexpr int fit_lds_words(int n_layers)
{
    return kWave * (27 + n_layers > kRecLds ? 27 + n_layers : kRecLds);
}

// Fit with known hits: one lane per track.  A wavefront whose 64 tracks lie
// in one batch moves their priors, hit lists and results through LDS, so
// that every global access of those transfers is one contiguous run (the
// arrays are track-major: a lane's own words lie 24 to 84 bytes apart from
// its neighbour's); a wavefront across a batch boundary, or at the end of
// the grid, takes one pass per batch with per-lane accesses instead.
template <int kGeo>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(geo_xyz(kGeo) ? 3 : 4))) k_fit(const Params P, const BatchArgs B, const Stamp st)
{
    extern __shared__ int s_dyn[];
    stamp_start(st);
    const int lane = threadIdx.x & (kWave - 1);
    const int g0 = uniform(xcd_contiguous(blockIdx.x, gridDim.x) * blockDim.x + (threadIdx.x & ~(kWave - 1)));
    if (g0 >= B.total_tracks) return;
    const int g = g0 + lane;
    const int e0 = uniform(upper_bound_i32(B.track_prefix, B.n_events + 1, g0) - 1);
    if (g0 + kWave <= load_global(B.track_prefix + e0 + 1)) {
        CEvent &E = event_desc(B.events, e0);
        const size_t t0 = (size_t)(g0 - load_global(B.track_prefix + e0));
        const int nl = P.n_layers;
        float *sp = reinterpret_cast<float *>(s_dyn + (threadIdx.x >> 6) * fit_lds_words(nl));   // [64][6]
        float *sc = sp + 6 * kWave;                                                            // [64][21]
        int *sh = reinterpret_cast<int *>(sc + 21 * kWave);                                    // [64][nl]
        const float *gp = E.track_par + 6 * t0, *gc = E.track_cov + 21 * t0;
        const int *gh = E.track_hits + t0 * nl;
#pragma unroll
        for (int k = 0; k < 6; ++k) sp[k * kWave + lane] = load_global(gp + k * kWave + lane);
#pragma unroll
        for (int k = 0; k < 21; ++k) sc[k * kWave + lane] = load_global(gc + k * kWave + lane);
        for (int k = 0; k < nl; ++k) sh[k * kWave + lane] = load_global(gh + k * kWave + lane);
        wave_lds_sync();
        float p[6], c[21], op[6], oc[21], chi2;
        int nupd, status;
#pragma unroll
        for (int i = 0; i < 6; ++i) p[i] = sp[6 * lane + i];
#pragma unroll
        for (int i = 0; i < 21; ++i) c[i] = sc[21 * lane + i];
        fit_track<kGeo>(P, E, p, c, [&](int L) { return sh[nl * lane + L]; }, op, oc, chi2, nupd, status);
        wave_lds_sync();   // every prior and hit read before the results take their place
        store_records(sp, E.fit_rec + kRecWords * t0, lane, op, oc, chi2, nupd, nl - nupd, status);
        return;
    }
    if (g >= B.total_tracks) return;
    const int e_lane = upper_bound_i32(B.track_prefix, B.n_events + 1, g) - 1;
    // one pass per batch the wave's lanes cover (two where a batch boundary
    // falls inside the wave), each with a wave-uniform descriptor
    for (;;) {
        const int e = uniform(e_lane);
        if (e_lane != e) continue;
        CEvent &E = event_desc(B.events, e);
        fit_known<kGeo>(P, E, (size_t)(g - load_global(B.track_prefix + e)));
        break;
    }
}

// Prior of the final fit of a built track: the helix through its hits on
// layers 0, 1 and 2 (the transverse circle through the three points; z
// linear in the arc length), at the first hit, with a loose diagonal
// covariance in the frame (u, z, q/pT, phi, theta) of the layer tangent at
// that hit, (u, r, q/pT, phi, theta) on a disk: sigma = (1 cm, 10 cm,
// 1 / GeV, 0.1, 0.1).  FP32 from the event's packed hits; false without
// three usable points.
template <bool kDisk>
__device__ __forceinline__ bool final_fit_prior(CEvent &E, const Params &P, const int *hits, float (&p)[6],
                                                float (&c)[21])
{
    float q[3][3];
    for (int L = 0; L < 3; ++L) {
        const int h = hits[L];
        if (h < 0) return false;
        // the hit's position from its packed form: (x, y, z, -), or
        // (cos, sin, z, r) on a cylinder and (cos, sin, r, z) on a disk
        const float4 v = load_global(E.hits + E.layer_off[L] + h);
        if (geo_xyz(P.geo)) {
            q[L][0] = v.x;
            q[L][1] = v.y;
            q[L][2] = v.z;
        } else {
            const float r = kDisk ? v.z : v.w;
            q[L][0] = r * v.x;
            q[L][1] = r * v.y;
            q[L][2] = kDisk ? v.w : v.z;
        }
    }
    const float d1x = q[1][0] - q[0][0], d1y = q[1][1] - q[0][1];   // first to second
    const float d3x = q[2][0] - q[0][0], d3y = q[2][1] - q[0][1];   // first to third
    const float ex = q[2][0] - q[1][0], ey = q[2][1] - q[1][1];
    const float l1 = sqrtf(fmaf(d1x, d1x, d1y * d1y)), l3 = sqrtf(fmaf(d3x, d3x, d3y * d3y));
    const float l2 = sqrtf(fmaf(ex, ex, ey * ey));
    const float twice_area = fmaf(d1x, d3y, -d1y * d3x);
    if (!(l1 > 0.f && l2 > 0.f && l3 > 0.f) || twice_area == 0.f) return false;
    const float curv = 2.f * twice_area / (l1 * l2 * l3);           // > 0 turning counter-clockwise
    // tangent at the first point: the chord to the second point, turned back
    // by half the angle the arc between them sweeps
    const float half = asinf(fminf(1.f, fmaxf(-1.f, 0.5f * curv * l1)));
    const float phi = wrap_pi(atan2f(d1y, d1x) - half);
    const float u3 = 0.5f * curv * l3;
    const float arc3 = fabsf(u3) < 1e-4f ? l3 * fmaf(u3 * u3, 1.f / 6.f, 1.f)
                                         : 2.f * asinf(fminf(1.f, fmaxf(-1.f, u3))) / curv;
    const float theta = 0.5f * kPi - atanf((q[2][2] - q[0][2]) / arc3);
    p[0] = q[0][0];
    p[1] = q[0][1];
    p[2] = q[0][2];
    p[3] = curv / P.w_per_qpt;
    p[4] = phi;
    p[5] = theta;
    float sa, ca;
    sincosf(atan2f(q[0][1], q[0][0]), &sa, &ca);
#pragma unroll
    for (int i = 0; i < 21; ++i) c[i] = 0.f;
    if (!kDisk) {
        c[sym(0, 0)] = sa * sa;
        c[sym(0, 1)] = -sa * ca;
        c[sym(1, 1)] = ca * ca;
        c[sym(2, 2)] = 100.f;
    } else {
        c[sym(0, 0)] = fmaf(100.f * ca, ca, sa * sa);
        c[sym(0, 1)] = 99.f * sa * ca;
        c[sym(1, 1)] = fmaf(100.f * sa, sa, ca * ca);
    }
    c[sym(3, 3)] = 1.f;
    c[sym(4, 4)] = 0.01f;
    c[sym(5, 5)] = 0.01f;
    return true;
}

// Final fit of one built track, its hits from the build's output.
template <int kGeo>
__device__ __forceinline__ void refit_built(const Params &P, CEvent &E, const size_t t)
{
    const int *hits = E.out_hits + t * P.n_layers;
    float p[6], c[21], op[6], oc[21], chi2 = 0.f;
    int nupd = 0, status = 3;
    if (final_fit_prior<geo_disk(kGeo)>(E, P, hits, p, c))
        fit_track<kGeo>(P, E, p, c, [&](int L) { return load_global(hits + L); }, op, oc, chi2, nupd, status);
    else {
#pragma unroll
        for (int i = 0; i < 6; ++i) op[i] = 0.f;
#pragma unroll
        for (int i = 0; i < 21; ++i) oc[i] = 0.f;
    }
    const int holes = __float_as_int(load_global(E.out_rec + kRecWords * t + kRecHoles));
    store_record(E.rf_rec + kRecWords * t, op, oc, chi2, nupd, holes, status, true);
}

// Final fit of every built track of a batch (after the build): one lane per
// seed.  A wavefront whose 64 seeds lie in one event moves their hit lists in
// and their results out through LDS (as the fit does), so that each transfer
// is one contiguous run instead of 64 rows 40 to 168 bytes apart.
template <int kGeo>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(geo_xyz(kGeo) ? 3 : 4))) k_refit(const Params P, const BatchArgs B, const Stamp st)
{
    extern __shared__ int s_dyn[];
    stamp_start(st);
    const int lane = threadIdx.x & (kWave - 1);
    const int g0 = uniform(xcd_contiguous(blockIdx.x, gridDim.x) * blockDim.x + (threadIdx.x & ~(kWave - 1)));
    if (g0 >= B.total_seeds) return;
    const int g = g0 + lane;
    const int e0 = uniform(upper_bound_i32(B.seed_prefix, B.n_events + 1, g0) - 1);
    if (g0 + kWave <= load_global(B.seed_prefix + e0 + 1)) {
        CEvent &E = event_desc(B.events, e0);
        const size_t t0 = (size_t)(g0 - load_global(B.seed_prefix + e0));
        const int nl = P.n_layers;
        float *sp = reinterpret_cast<float *>(s_dyn + (threadIdx.x >> 6) * fit_lds_words(nl));   // [64][6]
        float *sc = sp + 6 * kWave;                                                            // [64][21]
        int *sh = reinterpret_cast<int *>(sc + 21 * kWave);                                    // [64][nl]
        const int *gh = E.out_hits + t0 * nl;
        for (int k = 0; k < nl; ++k) sh[k * kWave + lane] = load_global(gh + k * kWave + lane);
        wave_lds_sync();
        const int *hits = sh + nl * lane;
        int h3[3];
#pragma unroll
        for (int L = 0; L < 3; ++L) h3[L] = hits[L];
        float p[6], c[21], op[6], oc[21], chi2 = 0.f;
        int nupd = 0, status = 3;
        if (final_fit_prior<geo_disk(kGeo)>(E, P, h3, p, c))
            fit_track<kGeo>(P, E, p, c, [&](int L) { return hits[L]; }, op, oc, chi2, nupd, status);
        else {
#pragma unroll
            for (int i = 0; i < 6; ++i) op[i] = 0.f;
#pragma unroll
            for (int i = 0; i < 21; ++i) oc[i] = 0.f;
        }
        const int holes = __float_as_int(load_global(E.out_rec + kRecWords * (t0 + lane) + kRecHoles));
        wave_lds_sync();   // every hit read before the results take their place
        store_records(sp, E.rf_rec + kRecWords * t0, lane, op, oc, chi2, nupd, holes, status);
        return;
    }
    if (g >= B.total_seeds) return;
    const int e_lane = upper_bound_i32(B.seed_prefix, B.n_events + 1, g) - 1;
    // one pass per event the wave's lanes cover, as in k_fit
    for (;;) {
        const int e = uniform(e_lane);
        if (e_lane != e) continue;
        CEvent &E = event_desc(B.events, e);
        refit_built<kGeo>(P, E, (size_t)(g - load_global(B.seed_prefix + e)));
        break;
    }
}

// ---------------------------------------------------------------------------
// The no-allocation builder's batch descriptors: one fixed array in device
// memory per GPU, kept until the process ends.  Host code reaches it only
// through the address hipGetSymbolAddress returns for the current device.

static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];
static std::atomic<void *> g_scratch_addr[64];

hipError_t noalloc_scratch_init(int device)
{
    if (g_scratch_addr[device & 63].load()) return hipSuccess;
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_addr[device & 63].store(p);
    return hipSuccess;
}

void *noalloc_scratch(int device) { return g_scratch_addr[device & 63].load(); }

// ---------------------------------------------------------------------------
// launchers

static inline unsigned blocks_for(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

hipError_t launch_fill_i32(int *ptr, int value, int n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_fill_i32<<<blocks_for(n, 256), 256, 0, s>>>(ptr, value, n);
    return hipGetLastError();
}

hipError_t launch_stamp(const Stamp &st, hipStream_t s)
{
    if (!st.a) return hipSuccess;
    k_stamp<<<1, 1, 0, s>>>(st.a, st.b);
    return hipGetLastError();
}

hipError_t launch_mark(unsigned *flag, unsigned value, hipStream_t s)
{
    k_mark<<<1, 1, 0, s>>>(flag, value);
    return hipGetLastError();
}

hipError_t launch_copy(const void *src, void *dst, size_t bytes, hipStream_t s)
{
    const size_t n = bytes / 16;
    if (n == 0) return hipSuccess;
    const unsigned grid = (unsigned)std::min<size_t>((n + 255) / 256, 256 * 64);
    k_copy16<<<grid, 256, 0, s>>>(static_cast<const float4 *>(src), static_cast<float4 *>(dst), n);
    return hipGetLastError();
}

// A wavefront per tile while few tiles leave the link idle; from 256 tiles
// on, 256 wavefronts take tiles in turn: 64 MB of stores run at 55.2 GB/s from
// 64 blocks of 256 threads, 54.3 from 256.  Few jobs travel in a short
// argument list (2.6 KB of arguments make a launch 1.9 us later).
constexpr int kDeliverWaves = 256;
constexpr int kFewJobs = 2;

template <int kJobs>
static hipError_t launch_deliver_t(const DeliverArgsT<kJobs> &a, const Stamp &st, hipStream_t s)
{
    if (a.n_tiles <= kDeliverWaves / 4) k_deliver<kJobs, 4><<<a.n_tiles, 4 * kWave, kDeliverLds, s>>>(a, st);
    else if (a.n_tiles <= kDeliverWaves) k_deliver<kJobs, 1><<<a.n_tiles, kWave, kDeliverLds, s>>>(a, st);
    else k_deliver<kJobs, 1><<<kDeliverWaves / 4, 4 * kWave, 4 * kDeliverLds, s>>>(a, st);
    return hipGetLastError();
}

hipError_t launch_deliver(const DeliverArgs &a, hipStream_t s, const Stamp &st)
{
    if (a.n_tiles <= 0) return launch_stamp(st, s);
    if (a.n_jobs > kFewJobs) return launch_deliver_t(a, st, s);
    DeliverArgsT<kFewJobs> few;
    few.n_jobs = a.n_jobs;
    few.n_tiles = a.n_tiles;
    few.n_layers = a.n_layers;
    for (int j = 0; j < a.n_jobs; ++j) few.job[j] = a.job[j];
    return launch_deliver_t(few, st, s);
}

hipError_t launch_calib_fma(float *dst, int n_blocks, int iters, hipStream_t s)
{
    k_calib_fma<<<n_blocks, 256, 0, s>>>(dst, iters, 0.999999f, 1e-6f);
    return hipGetLastError();
}

int calib_fma_chains() { return kFmaChains; }

hipError_t launch_batch_zero(const BatchArgs &b, hipStream_t s)
{
    if (b.n_events <= 0) return hipSuccess;
    k_batch_zero<<<blocks_for(5 * b.n_events, 256), 256, 0, s>>>(b);
    return hipGetLastError();
}

static hipError_t launch_index_layer(const Params &p, const BatchArgs &b, const IndexExtent &x, int only,
                                     const Stamp &st, hipStream_t s)
{
    const unsigned blocks = (unsigned)(b.n_events * p.n_layers);
    const size_t lds = layer_block_lds(x.layer_hits, x.bins);
    if (!layer_block_fits(x.layer_hits, x.bins)) k_index_ranges<<<blocks, 1024, kLayerBlockLds, s>>>(p, b, only, st);
    else if (x.layer_hits <= 0xFFFF) k_index_layer<true><<<blocks, 1024, lds, s>>>(p, b, only, st);
    else k_index_layer<false><<<blocks, 1024, lds, s>>>(p, b, only, st);
    return hipGetLastError();
}

hipError_t launch_index(const Params &p, const BatchArgs &b, hipStream_t s, const Stamp &st)
{
    if (b.total_hits <= 0) return launch_stamp(st, s);
    const unsigned pairs = (unsigned)(b.n_events * p.n_layers);
    // One block per (event, layer) or the bucketed build, whichever is sooner
    // done.  Measured (us): a block takes 7 + 2.05 per 1,000 hits of the
    // fullest layer (650 hits 9, 3,900 14, 13,000 29, 65,000 104); the three
    // launches 14 + 0.0165 per 1,000 hits of the batch + 0.083 per (event,
    // layer) pair for blocks that have little to do (one event of 6,500 hits a
    // layer 17, of 13,000 19, of 65,000 31; 5, 7 and 10 events of 22,000 37,
    // 45 and 58, where blocks take 50, 52 and 57; 64 of 1,300 84 against 27).
    const double by_layer = 7.0 + 2.05e-3 * b.all.layer_hits;
    const double bucketed = 14.0 + 1.65e-5 * b.total_hits + 0.083 * pairs;
    if (b.layer_only.events == b.n_events || (by_layer < bucketed && layer_block_fits(b.all.layer_hits, b.all.bins)))
        return launch_index_layer(p, b, b.all, 0, st, s);
    const dim3 grid((unsigned)std::max(1, b.max_chunks), pairs);
    k_index_hist<<<grid, kBlockThreads, 0, s>>>(p, b, st);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    k_index_part<<<grid, kBlockThreads, 0, s>>>(p, b);
    err = hipGetLastError();
    if (err != hipSuccess) return err;
    k_index_place<<<dim3(kBuckets, pairs), kBlockThreads, sizeof(unsigned) << b.max_bucket_shift, s>>>(p, b);
    err = hipGetLastError();
    if (err != hipSuccess || b.layer_only.events == 0) return err;
    return launch_index_layer(p, b, b.layer_only, 1, Stamp{}, s);
}

size_t build_lds_bytes(int geo, int n_layers, int wpb)
{
    const size_t search = geo_xyz(geo) ? sizeof(SearchLds<2>) : sizeof(SearchLds<0>);
    return sizeof(int) * (size_t)search_lds_offset(wpb, n_layers) + (size_t)wpb * search;
}

// Wavefronts of a build launch that deliver: 16 / 64 / 256 of them took 126,
// 119 and 123 us for 20,000 rows beside a build, 436, 421 and 417 for 82,000.
constexpr int kOverlapWaves = 64;

template <int G, bool kStats>
static hipError_t launch_batch_t(const Params &p, const BatchArgs &b, int wpb, int persistent, int n_blocks,
                                 const DeliverArgs *d, hipStream_t s, const Stamp &st)
{
    const int dblocks = d && d->n_tiles > 0 ? std::max(1, kOverlapWaves / wpb) : 0;
    unsigned grid = persistent ? (unsigned)n_blocks : blocks_for(b.end_item - b.first_item, wpb);
    if (dblocks) grid = kXcds * std::max((unsigned)dblocks, (grid + kXcds - 2) / (kXcds - 1));
    if (grid == 0) return launch_stamp(st, s);
    const size_t hist = sizeof(int) * (size_t)search_lds_offset(wpb, p.n_layers);
    auto lds = [&](size_t search) { return std::max(hist + wpb * search, (size_t)(d ? wpb * kDeliverLds : 0)); };
    switch (p.geo) {
    case 0: k_build_batch<G, kStats, 0><<<grid, wpb * kWave, lds(sizeof(SearchLds<0>)), s>>>(p, b, persistent, d, dblocks, st); break;
    case 1: k_build_batch<G, kStats, 1><<<grid, wpb * kWave, lds(sizeof(SearchLds<1>)), s>>>(p, b, persistent, d, dblocks, st); break;
    case 2: k_build_batch<G, kStats, 2><<<grid, wpb * kWave, lds(sizeof(SearchLds<2>)), s>>>(p, b, persistent, d, dblocks, st); break;
    case 3: k_build_batch<G, kStats, 3><<<grid, wpb * kWave, lds(sizeof(SearchLds<3>)), s>>>(p, b, persistent, d, dblocks, st); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_build_batch(const Params &p, const BatchArgs &b, int G, int wpb, int persistent, int n_blocks,
                              bool stats, const DeliverArgs *d, hipStream_t s, const Stamp &st)
{
#define MKF_BATCH_CASE(g)                                                                            \
    case g: return stats ? launch_batch_t<g, true>(p, b, wpb, persistent, n_blocks, d, s, st)           \
                         : launch_batch_t<g, false>(p, b, wpb, persistent, n_blocks, d, s, st);
    switch (G) {
        MKF_BATCH_CASE(1)
        MKF_BATCH_CASE(2)
        MKF_BATCH_CASE(4)
        MKF_BATCH_CASE(6)
        MKF_BATCH_CASE(8)
    default: return hipErrorInvalidValue;
    }
#undef MKF_BATCH_CASE
}

template <int G, bool kStats>
static hipError_t launch_layer_t(const Params &p, const DevEvent *ev_dev, int n_seeds, int L, int spw,
                                 int wpb, hipStream_t s)
{
    const int items = (n_seeds + spw - 1) / spw;
    const unsigned grid = blocks_for(items, wpb);
    if (grid == 0) return hipSuccess;
    switch (p.geo) {
    case 0: k_build_layer<G, kStats, 0><<<grid, wpb * kWave, wpb * sizeof(SearchLds<0>), s>>>(p, ev_dev, L, spw); break;
    case 1: k_build_layer<G, kStats, 1><<<grid, wpb * kWave, wpb * sizeof(SearchLds<1>), s>>>(p, ev_dev, L, spw); break;
    case 2: k_build_layer<G, kStats, 2><<<grid, wpb * kWave, wpb * sizeof(SearchLds<2>), s>>>(p, ev_dev, L, spw); break;
    case 3: k_build_layer<G, kStats, 3><<<grid, wpb * kWave, wpb * sizeof(SearchLds<3>), s>>>(p, ev_dev, L, spw); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_build_layer(const Params &p, const DevEvent *ev_dev, const DevEvent &ev_host, int L, int G,
                              int spw, int wpb, bool stats, hipStream_t s)
{
    const int n = ev_host.n_seeds;
#define MKF_LAYER_CASE(g)                                                                            \
    case g: return stats ? launch_layer_t<g, true>(p, ev_dev, n, L, spw, wpb, s)                          \
                         : launch_layer_t<g, false>(p, ev_dev, n, L, spw, wpb, s);
    switch (G) {
        MKF_LAYER_CASE(1)
        MKF_LAYER_CASE(2)
        MKF_LAYER_CASE(4)
        MKF_LAYER_CASE(6)
        MKF_LAYER_CASE(8)
    default: return hipErrorInvalidValue;
    }
#undef MKF_LAYER_CASE
}

hipError_t launch_refit(const Params &p, const BatchArgs &b, hipStream_t s, const Stamp &st)
{
    if (b.total_seeds <= 0) return launch_stamp(st, s);
    const unsigned grid = blocks_for(b.total_seeds, 256);
    const size_t lds = 4 * sizeof(int) * (size_t)fit_lds_words(p.n_layers);
    switch (p.geo | (p.update3d ? 4 : 0)) {
    case 0: k_refit<0><<<grid, 256, lds, s>>>(p, b, st); break;
    case 1: k_refit<1><<<grid, 256, lds, s>>>(p, b, st); break;
    case 2: k_refit<2><<<grid, 256, lds, s>>>(p, b, st); break;
    case 3: k_refit<3><<<grid, 256, lds, s>>>(p, b, st); break;
    case 6: k_refit<6><<<grid, 256, lds, s>>>(p, b, st); break;
    case 7: k_refit<7><<<grid, 256, lds, s>>>(p, b, st); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_fit(const Params &p, const BatchArgs &b, hipStream_t s, const Stamp &st)
{
    if (b.total_tracks <= 0) return launch_stamp(st, s);
    const unsigned grid = blocks_for(b.total_tracks, 256);
    const size_t lds = 4 * sizeof(int) * (size_t)fit_lds_words(p.n_layers);
    switch (p.geo | (p.update3d ? 4 : 0)) {
    case 0: k_fit<0><<<grid, 256, lds, s>>>(p, b, st); break;
    case 1: k_fit<1><<<grid, 256, lds, s>>>(p, b, st); break;
    case 2: k_fit<2><<<grid, 256, lds, s>>>(p, b, st); break;
    case 3: k_fit<3><<<grid, 256, lds, s>>>(p, b, st); break;
    case 6: k_fit<6><<<grid, 256, lds, s>>>(p, b, st); break;
    case 7: k_fit<7><<<grid, 256, lds, s>>>(p, b, st); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace mkf
