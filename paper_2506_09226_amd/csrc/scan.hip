// Run offsets of the tiled scatters: a column-wise scan of per-tile counts.
#include <algorithm>

#include "gq_device.h"
#include "gq_internal.h"
#include "gq_ops.h"

// ---------------------------------------------------------------------------
// Run offsets from per-tile bucket counts in TILE-MAJOR layout (the counts of
// one tile are contiguous, so a histogram kernel writes them, and a scatter
// kernel reads its tile's P offsets, as one coalesced row):
//
//   off[t*P + b] = start[b] + sum_{t' < t} cnt[t'*P + b],
//   start[b]     = sum_{b' < b} total[b'],   start[P] = sum of all counts.
//
// Two small kernels, every access coalesced across buckets: per-chunk column
// sums, then one workgroup per chunk that sums all chunks' column sums (the
// bucket totals) and those before it, scans the totals over the buckets and
// writes its tiles' offsets.  A chunk is 32 tiles or as many as keep the
// chunks under 192, so what every workgroup reads again (192 sums a bucket,
// from L2) stays small.  Launches and dependent loads bound these kernels:
// with a scan of the sums and one of the totals as kernels of their own,
// 20M rows in 256 buckets took 355 us (350 now), a group-by of 5M rows 172.5
// (169.5), a pipeline of 1M rows 184 (180).  Up to 32 tiles take the second
// kernel alone.
// ---------------------------------------------------------------------------
namespace {

constexpr int TO_THREADS = 256;                     // of the chunk sums
constexpr int TO_OFF_THREADS = 1024;                // of the offsets
constexpr int TO_MAX_P = TO_OFF_THREADS;

// Column loops load TO_BATCH counts into registers before using them, so a
// thread keeps that many independent loads in flight.
constexpr int TO_BATCH = 32;
constexpr int TO_ONCE = 8;                          // tiles of a share that are held from one load
constexpr int TO_SUMS = 16;                         // chunk sums loaded together

int64_t to_chunk_tiles(int64_t ntiles)
{
    int64_t c = 32;
    while (c * 192 < ntiles) c *= 2;
    return c;
}

// Tiles that hold counts: those that the row count (the bound, or the device
// count within it) reaches; none of an empty input, whose one tile is not counted.
GQ_DEV int64_t to_live_tiles(int64_t ntiles, gq_tile_count live)
{
    int64_t n = live.n_bound;
    if (live.n_dev) {
        const int64_t d = *live.n_dev;
        n = d < 0 ? 0 : (d < n ? d : n);
    }
    const int64_t t = (n + live.tile_rows - 1) / live.tile_rows;
    return t < ntiles ? t : ntiles;
}

__global__ __launch_bounds__(TO_THREADS) void to_chunk_sum_kernel(const uint32_t *__restrict__ cnt, int64_t ntiles,
                                                                  int P, int64_t chunk, uint32_t *__restrict__ csum,
                                                                  gq_tile_count live)
{
    ntiles = to_live_tiles(ntiles, live);
    const int64_t c = blockIdx.x;
    const int b = blockIdx.y * TO_THREADS + threadIdx.x;
    if (b >= P) return;
    const int64_t t0 = c * chunk;
    const int64_t t1 = t0 + chunk < ntiles ? t0 + chunk : ntiles;
    uint32_t s = 0;
    for (int64_t t = t0; t < t1; t += TO_BATCH) {
        uint32_t x[TO_BATCH];
#pragma unroll
        for (int i = 0; i < TO_BATCH; ++i) x[i] = t + i < t1 ? cnt[(t + i) * P + b] : 0u;
#pragma unroll
        for (int i = 0; i < TO_BATCH; ++i) s += x[i];
    }
    csum[c * P + b] = s;
}

// Threads (g, b): column b, the g-th of 1024 >> lgp shares of the chunk sums
// and of the chunk's tiles (1 << lgp >= P columns).
__global__ __launch_bounds__(TO_OFF_THREADS) void to_offsets_kernel(uint32_t *__restrict__ cnt, int64_t ntiles, int P,
                                                                    int lgp, int64_t chunk, int nchunks,
                                                                    const uint32_t *__restrict__ csum,
                                                                    uint32_t *__restrict__ start,
                                                                    int64_t *__restrict__ start64, gq_tile_count live)
{
    __shared__ uint32_t s_pre[TO_OFF_THREADS], s_tot[TO_OFF_THREADS], s_sub[TO_OFF_THREADS];
    __shared__ uint32_t smem[TO_OFF_THREADS / 64];
    ntiles = to_live_tiles(ntiles, live);
    const int c = static_cast<int>(blockIdx.x);
    const int64_t t0 = c * chunk;
    if (c > 0 && t0 >= ntiles) return;               // no live tiles (chunk 0 also writes the starts)
    const int64_t t1 = t0 + chunk < ntiles ? t0 + chunk : ntiles;
    const int groups = TO_OFF_THREADS >> lgp;
    const int b = threadIdx.x & ((1 << lgp) - 1), g = threadIdx.x >> lgp;
    const int64_t per = (chunk + groups - 1) / groups;
    const int64_t a0 = t0 + g * per, a1 = a0 + per < t1 ? a0 + per : t1;
    // a share of few tiles is loaded once, together with the chunk sums
    const bool once = per <= TO_ONCE;
    uint32_t own[TO_ONCE];
#pragma unroll
    for (int i = 0; i < TO_ONCE; ++i) own[i] = (once && b < P && a0 + i < a1) ? cnt[(a0 + i) * P + b] : 0u;
    uint32_t sub = 0, pre = 0, tot = 0;
    if (b < P) {
        if (!once && (groups > 1 || nchunks == 1)) {  // counts of the tiles of this share
            for (int64_t t = a0; t < a1; t += TO_BATCH) {
                uint32_t x[TO_BATCH];
#pragma unroll
                for (int i = 0; i < TO_BATCH; ++i) x[i] = t + i < a1 ? cnt[(t + i) * P + b] : 0u;
#pragma unroll
                for (int i = 0; i < TO_BATCH; ++i) sub += x[i];
            }
        }
        if (nchunks > 1) {
            for (int d = g; d < nchunks; d += TO_SUMS * groups) {
                uint32_t x[TO_SUMS];
#pragma unroll
                for (int i = 0; i < TO_SUMS; ++i)
                    x[i] = d + i * groups < nchunks ? csum[static_cast<int64_t>(d + i * groups) * P + b] : 0u;
#pragma unroll
                for (int i = 0; i < TO_SUMS; ++i) {
                    tot += x[i];
                    pre += d + i * groups < c ? x[i] : 0u;
                }
            }
        }
    }
    if (once) {
#pragma unroll
        for (int i = 0; i < TO_ONCE; ++i) sub += own[i];
    }
    if (nchunks == 1) tot = sub;
    s_pre[threadIdx.x] = pre;
    s_tot[threadIdx.x] = tot;
    s_sub[threadIdx.x] = sub;
    __syncthreads();
    uint32_t before = 0, total = 0;
    if (g == 0) {                                    // this column over all shares
        for (int h = 0; h < groups; ++h) {
            before += s_pre[(h << lgp) | b];
            total += s_tot[(h << lgp) | b];
        }
    }
    uint32_t all;
    const uint32_t first = gq_block_exclusive_scan<TO_OFF_THREADS>(total, &all, smem);
    if (g == 0 && b < P) {
        s_tot[b] = first + before;
        if (c == 0) {
            start[b] = first;
            if (start64) start64[b] = static_cast<int64_t>(first);
        }
    }
    if (c == 0 && threadIdx.x == 0) {
        start[P] = all;
        if (start64) start64[P] = static_cast<int64_t>(all);
    }
    __syncthreads();
    if (b >= P) return;
    uint32_t run = s_tot[b];
    for (int h = 0; h < g; ++h) run += s_sub[(h << lgp) | b];
    if (once) {
#pragma unroll
        for (int i = 0; i < TO_ONCE; ++i) {
            if (a0 + i < a1) cnt[(a0 + i) * P + b] = run;
            run += own[i];
        }
        return;
    }
    for (int64_t t = a0; t < a1; t += TO_BATCH) {
        uint32_t x[TO_BATCH];
#pragma unroll
        for (int i = 0; i < TO_BATCH; ++i) x[i] = t + i < a1 ? cnt[(t + i) * P + b] : 0u;
#pragma unroll
        for (int i = 0; i < TO_BATCH; ++i) {
            if (t + i < a1) cnt[(t + i) * P + b] = run;
            run += x[i];
        }
    }
}

}  // namespace

// (The chunk count for up to ntiles tiles, as a bound that grows with ntiles.)
size_t gq_tile_offsets_workspace(int64_t ntiles, int P)
{
    gq_carver c(nullptr);
    const int64_t nchunks = std::min<int64_t>(ntiles / 32, 192) + 1;
    c.take<uint32_t>(static_cast<size_t>(nchunks * P));
    return c.bytes();
}

gq_status gq_tile_offsets(gq_ctx *ctx, uint32_t *cnt, int64_t ntiles, int P, uint32_t *start, void *ws,
                          hipStream_t s, const char *name, const gq_tile_count *live, int64_t *start64)
{
    const gq_tile_count lv = live ? *live : gq_tile_count{nullptr, ntiles, 1};
    if (live && live->tile_rows < 1) return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_tile_offsets: bad tile rows");
    if (P < 1 || P > TO_MAX_P || ntiles < 1) return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_tile_offsets: bad shape");
    gq_carver c(ws);
    const int64_t chunk = to_chunk_tiles(ntiles);
    const int64_t nchunks = (ntiles + chunk - 1) / chunk;
    uint32_t *csum = c.take<uint32_t>(static_cast<size_t>(nchunks * P));
    int lgp = 6;                                     // whole waves per share
    while ((1 << lgp) < P) ++lgp;
    if (nchunks > 1) {
        const dim3 grid(static_cast<uint32_t>(nchunks), static_cast<uint32_t>((P + TO_THREADS - 1) / TO_THREADS));
        GQ_TRY(gq_launch(ctx, name, to_chunk_sum_kernel, grid, dim3(TO_THREADS), 0, s,
                         static_cast<const uint32_t *>(cnt), ntiles, P, chunk, csum, lv));
    }
    return gq_launch(ctx, name, to_offsets_kernel, dim3(static_cast<uint32_t>(nchunks)), dim3(TO_OFF_THREADS), 0, s,
                     cnt, ntiles, P, lgp, chunk, static_cast<int>(nchunks), static_cast<const uint32_t *>(csum), start,
                     start64, lv);
}
