// Scan + filter: ordered stream compaction of a range predicate.
//
// One pass over the column.  A workgroup takes a unit of consecutive rows with
// one dequeue; each wave owns a contiguous stretch of the unit and tests it 64
// rows at a time, keeping the ballot of step i in lane i.  The unit's match
// count goes through a decoupled look-back over units, which gives its global
// offset; each wave then writes its matching row ids there, through an LDS stage
// of its own or, if most of its rows match, step by step at its offset plus the
// ballot's lane prefix.  Small inputs skip the look-back (filter_tiny_kernel).
#include <algorithm>
#include <limits>
#include <type_traits>

#include "gq_device.h"
#include "gq_internal.h"

// v_writelane_b32 (clang has no builtin for it): `old` with one lane's value
// replaced.  value and lane are the same in every lane.
extern "C" __device__ int gq_writelane(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

namespace {

// Bound by memory: 4 (or 8) bytes a row in, 4 bytes a match out.  1024-thread
// workgroups at 38 registers put 32 waves on a CU.  A unit is up to 32 steps
// of its 16 waves (32K rows): each unit costs a dequeue (atomics on one
// address take turns at about 20 ns) and a look-back that reads words other
// XCDs write; smaller inputs take fewer steps, for 128 to 256 units (3M rows:
// 14.6 us at 128 units, 20.5 at 600).  A step is a load, two instructions of
// test and two that put its ballot into lanes (with the ballot selected into
// its lane, and every step written by itself, 200M 4-byte rows took 214, 245,
// 265, 295 and 331 us at 0, 5, 30, 58 and 100% kept; so, 184, 198, 239, 289 and
// 325: 4.3 TB/s read with nothing kept, 4.9 TB/s read and written with all).
constexpr int FT_THREADS = 1024;
constexpr int FT_WAVES = FT_THREADS / 64;
constexpr int FT_MAX_STEPS = 32;                    // steps of a wave per unit (the ballots of 32 lanes)
constexpr int64_t FT_UNITS = 128;                   // units that smaller inputs are cut into
constexpr int64_t FT_MAX_SMALL_UNITS = 2 * FT_UNITS; // their most, just before the steps double

int ft_steps(int64_t n)                             // a power of two: a lane's rows in the stage lie in one word
{
    int steps = 1;
    while (steps < FT_MAX_STEPS && n >= 2 * steps * FT_THREADS * FT_UNITS) steps *= 2;
    return steps;
}

// A wave's matches go through LDS when the unit has FT_STAGE_STEPS steps or
// more (fewer write so little that the detour costs 0.3 us of 9) and three
// quarters or fewer of its rows match; the stage holds half of them (64 KB for
// the largest unit, two workgroups a CU).
constexpr int FT_STAGE_STEPS = 8;
__host__ __device__ constexpr int ft_stage(int steps) { return steps >= FT_STAGE_STEPS ? steps * 32 : 0; }

struct filter_ws {
    uint32_t *unit_ctr;
    uint64_t *status;
};

// The range test lo <= x < hi as one unsigned comparison in the column's type:
// x - base <= span, when any value of the type passes at all.
template <typename T>
struct ft_range {
    using U = std::make_unsigned_t<T>;
    U base, span;
    bool any;
    GQ_DEV ft_range(int64_t lo, int64_t hi)
    {
        const int64_t mn = std::numeric_limits<T>::min(), mx = std::numeric_limits<T>::max();
        const int64_t a = lo > mn ? lo : mn;
        const int64_t z = hi > mx ? mx : hi - 1;          // the last value that passes (hi > lo >= min: no wrap)
        any = hi > lo && a <= z;
        base = static_cast<U>(a);
        span = static_cast<U>(static_cast<U>(z) - base);
    }
    GQ_DEV bool test(T x) const { return any && static_cast<U>(static_cast<U>(x) - base) <= span; }
};

// A dequeue counter, then one look-back status word per unit; a workspace made
// for n rows serves every smaller call too.
filter_ws filter_layout(gq_carver &c, int64_t n)
{
    filter_ws w;
    const int64_t unit = static_cast<int64_t>(FT_THREADS) * ft_steps(n);
    const int64_t units = std::max((n + unit - 1) / unit, std::min((n + FT_THREADS - 1) / FT_THREADS, FT_MAX_SMALL_UNITS));
    w.unit_ctr = c.take<uint32_t>(64);
    w.status = c.take<uint64_t>(static_cast<size_t>(units > 0 ? units : 1));
    return w;
}

GQ_DEV int64_t ft_rows(int64_t bound, const int64_t *n_dev)
{
    if (!n_dev) return bound;
    const int64_t d = *n_dev;
    return d < bound ? (d > 0 ? d : 0) : bound;
}

// IN_PLACE: the output is the selection itself.  A unit's outputs lie at its own
// or earlier rows, and every earlier unit has read its rows before it publishes
// its count; so a unit keeps its row ids in LDS instead of reading them again.
template <typename T, bool HAS_SEL, bool IN_PLACE>
__global__ __launch_bounds__(FT_THREADS) void filter_kernel(const T *__restrict__ col,
                                                            const int32_t *__restrict__ sel_in,
                                                            int64_t n_bound, const int64_t *n_dev, int64_t lo,
                                                            int64_t hi, int steps, int32_t *__restrict__ out,
                                                            int64_t *n_out, uint32_t *unit_ctr, uint64_t *status)
{
    static_assert(HAS_SEL || !IN_PLACE, "without a selection there is nothing to overwrite");
    extern __shared__ int32_t held[];                       // the waves' stages (IN_PLACE: the unit's row ids)
    __shared__ uint32_t wcnt[FT_WAVES];
    __shared__ uint32_t s_unit;
    __shared__ uint64_t s_goff;
    const ft_range<T> range(lo, hi);
    const int64_t n = ft_rows(n_bound, n_dev);
    const int64_t unit = static_cast<int64_t>(FT_THREADS) * steps;
    const int64_t nunits = (n + unit - 1) / unit;
    if (static_cast<int64_t>(blockIdx.x) >= nunits) {       // as many workgroups take a unit as there are units
        if (blockIdx.x == 0 && threadIdx.x == 0) *n_out = 0;
        return;
    }
    if (threadIdx.x == 0) s_unit = atomicAdd(unit_ctr, 1u);
    __syncthreads();
    const uint32_t u = s_unit;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t row0 = static_cast<int64_t>(u) * unit + static_cast<int64_t>(wave) * steps * 64 + lane;
    constexpr int FT_BATCH = HAS_SEL ? 4 : 8;               // steps whose loads overlap (gathers: 64 us at 4, 85 at 8)
    uint32_t wlo = 0, whi = 0;                              // lane i: the matches of step i
    auto keep = [&](uint64_t b, int i) {
        wlo = static_cast<uint32_t>(gq_writelane(static_cast<int>(b), i, static_cast<int>(wlo)));
        whi = static_cast<uint32_t>(gq_writelane(static_cast<int>(b >> 32), i, static_cast<int>(whi)));
    };
    // a unit whose rows all exist goes without a bound test for each
    const bool full = !HAS_SEL && static_cast<int64_t>(u + 1) * unit <= n && steps % FT_BATCH == 0;
    for (int i0 = 0; full && i0 < steps; i0 += FT_BATCH) {
        const T *at = col + row0 + i0 * 64;
        T v[FT_BATCH];
#pragma unroll
        for (int c = 0; c < FT_BATCH; ++c) v[c] = __builtin_nontemporal_load(at + c * 64);
#pragma unroll
        for (int c = 0; c < FT_BATCH; ++c) keep(gq_ballot(range.test(v[c])), i0 + c);
    }
    for (int i0 = full ? steps : 0; i0 < steps; i0 += FT_BATCH) {
        T v[FT_BATCH];
#pragma unroll
        for (int c = 0; c < FT_BATCH; ++c) {
            const int64_t e = row0 + (i0 + c) * 64;
            v[c] = 0;
            if (i0 + c < steps && e < n) {
                if constexpr (HAS_SEL) {
                    const int32_t r = sel_in[e];
                    if (IN_PLACE) held[(wave * steps + i0 + c) * 64 + lane] = r;
                    v[c] = col[r];
                } else {
                    v[c] = __builtin_nontemporal_load(&col[e]);
                }
            }
        }
#pragma unroll
        for (int c = 0; c < FT_BATCH; ++c) {
            const int64_t e = row0 + (i0 + c) * 64;
            keep(gq_ballot(i0 + c < steps && e < n && range.test(v[c])), i0 + c);
        }
    }
    const uint32_t mine = static_cast<uint32_t>(__popc(wlo) + __popc(whi));
    const uint32_t incl = gq_wave_inclusive_scan(mine);
    if (lane == 63) wcnt[wave] = incl;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < FT_WAVES; ++w) {
        before += w < wave ? wcnt[w] : 0u;
        total += wcnt[w];
    }
    if (wave == 0) {
        const uint64_t g = gq_lookback(status, u, total);
        if (lane == 0) {
            s_goff = g;
            if (static_cast<int64_t>(u) == nunits - 1) *n_out = static_cast<int64_t>(g + total);
        }
    }
    __syncthreads();
    const uint32_t excl = before + incl - mine;             // lane i: matches of the unit before step i
    const int64_t goff = static_cast<int64_t>(s_goff);
    const uint32_t found = __builtin_amdgcn_readlane(incl, 63);
    if (!IN_PLACE && steps >= FT_STAGE_STEPS && found <= static_cast<uint32_t>(steps * 48)) {
        // The wave's matches through its LDS stage, so that they leave it 64 at a
        // time: lane l takes `per` consecutive rows, one match at a time; a wave
        // with more matches than the stage holds takes two rounds.
        const int cap = ft_stage(steps);
        int32_t *stage = held + wave * cap;
        const int per = found <= static_cast<uint32_t>(cap) ? steps : steps / 2;
        uint32_t done = 0;
        for (int r0 = 0; r0 < steps * 64; r0 += per * 64) {
            const int pos = r0 + lane * per, sh = pos & 31;
            const uint32_t lo32 = __shfl(wlo, pos >> 6, 64), hi32 = __shfl(whi, pos >> 6, 64);
            const uint32_t below = (1u << sh) - 1u;
            const bool upper = pos & 32;
            uint32_t bits = (upper ? hi32 : lo32) >> sh;
            if (per < 32) bits &= (1u << per) - 1u;
            uint32_t at = __shfl(incl - mine, pos >> 6, 64) - done +
                          (upper ? __popc(lo32) + __popc(hi32 & below) : __popc(lo32 & below));
            const int64_t first = row0 - lane + pos;
            while (bits) {
                const int64_t e = first + __builtin_ctz(bits);
                bits &= bits - 1;
                stage[at++] = HAS_SEL ? sel_in[e] : static_cast<int32_t>(e);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            // (the place after the last lane's matches: the count of this round)
            const uint32_t count = __builtin_amdgcn_readlane(at, 63);
            for (uint32_t q = lane; q < count; q += 64) out[goff + before + done + q] = stage[q];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            done += count;
        }
        return;
    }
    for (int i = 0; i < steps; ++i) {
        const uint32_t blo = __builtin_amdgcn_readlane(wlo, i), bhi = __builtin_amdgcn_readlane(whi, i);
        const uint64_t b = (static_cast<uint64_t>(bhi) << 32) | blo;
        const uint32_t pre = __builtin_amdgcn_readlane(excl, i);
        if ((b >> lane) & 1u) {
            const int64_t e = row0 + i * 64;
            out[goff + pre + gq_mbcnt(b)] =
                IN_PLACE ? held[(wave * steps + i) * 64 + lane] : HAS_SEL ? sel_in[e] : static_cast<int32_t>(e);
        }
    }
}

// Small inputs, bound by latency: one launch with no scratch to clear and no
// waiting (64K rows: 16.4 -> 5.7 us a call; with 4-byte loads 3 more).
// Workgroup t counts the matches of all rows before its own 1024 itself, so the
// line lies where the last one's reads take as long as the second launch and the
// look-back: one-launch and look-back form, us a call, 4-byte rows 5.7 and 8.9 at
// 64K, 7.3 and 8.9 at 128K, 9.6 and 9.7 at 192K; 8-byte rows 6.5 and 8.9 at 64K,
// 8.3 and 8.9 at 96K, 10.1 and 8.9 at 128K.  A selection's rows take two
// dependent loads, in no order: 6.0 and 8.9 at 8K, 7.3 and 8.8 at 16K, 8.9 and
// 8.9 at 20K, 13.5 and 8.9 at 32K.
constexpr int64_t FT_TINY_BYTES = 1 << 19;          // of the column
constexpr int64_t FT_TINY_SEL_ROWS = 1 << 14;

template <typename T, bool HAS_SEL>
__global__ __launch_bounds__(FT_THREADS) void filter_tiny_kernel(const T *__restrict__ col,
                                                                 const int32_t *__restrict__ sel_in,
                                                                 int64_t n_bound, const int64_t *n_dev, int64_t lo,
                                                                 int64_t hi, int vec, int32_t *__restrict__ out,
                                                                 int64_t *n_out)
{
    __shared__ uint32_t wprev[FT_WAVES], wcnt[FT_WAVES];
    const int64_t n = ft_rows(n_bound, n_dev);
    const int64_t base = static_cast<int64_t>(blockIdx.x) * FT_THREADS;
    if (base >= n) {
        if (blockIdx.x == 0 && threadIdx.x == 0) *n_out = 0;
        return;
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const ft_range<T> range(lo, hi);
    auto test = [&](int32_t r) { return range.test(col[r]); };
    const int32_t e = static_cast<int32_t>(base) + static_cast<int32_t>(threadIdx.x);
    const int32_t r = e < n ? (HAS_SEL ? sel_in[e] : e) : 0;
    uint32_t prev = 0;
    if (!HAS_SEL && vec) {                              // 16-byte loads (the column's start is 16-byte aligned)
        constexpr int PER = 16 / sizeof(T);
        constexpr int AHEAD = 8;
        typedef T vec_t __attribute__((ext_vector_type(PER)));
        const vec_t *cv = reinterpret_cast<const vec_t *>(col);
        const int32_t nv = static_cast<int32_t>(base) / PER;   // base is a multiple of 1024
        for (int32_t j0 = threadIdx.x; j0 < nv; j0 += FT_THREADS * AHEAD) {
            vec_t v[AHEAD];
#pragma unroll
            for (int c = 0; c < AHEAD; ++c) {
                const int32_t j = j0 + c * FT_THREADS;
                v[c] = cv[j < nv ? j : j0];
            }
#pragma unroll
            for (int c = 0; c < AHEAD; ++c) {
                uint32_t m = 0;
#pragma unroll
                for (int i = 0; i < PER; ++i) m += range.test(v[c][i]) ? 1u : 0u;
                prev += j0 + c * FT_THREADS < nv ? m : 0u;
            }
        }
    } else {
        constexpr int AHEAD = 16;
        for (int32_t j0 = threadIdx.x; j0 < base; j0 += FT_THREADS * AHEAD) {
#pragma unroll
            for (int c = 0; c < AHEAD; ++c) {
                const int32_t j = j0 + c * FT_THREADS;
                if (j < base) prev += test(HAS_SEL ? sel_in[j] : j) ? 1u : 0u;
            }
        }
    }
    const uint64_t b = gq_ballot(e < n && test(r));
    prev = gq_wave_sum(prev);
    if (lane == 0) {
        wprev[wave] = prev;
        wcnt[wave] = static_cast<uint32_t>(__popcll(b));
    }
    __syncthreads();
    uint32_t at = 0, total = 0;
#pragma unroll
    for (int w = 0; w < FT_WAVES; ++w) {
        at += wprev[w] + (w < wave ? wcnt[w] : 0u);
        total += wprev[w] + wcnt[w];
    }
    if ((b >> lane) & 1u) out[at + gq_mbcnt(b)] = r;
    if (base + FT_THREADS >= n && threadIdx.x == 0) *n_out = total;
}

template <typename T, bool S>
gq_status launch_filter(gq_ctx *ctx, const void *col, const int32_t *sel_in, int64_t n, const int64_t *n_dev,
                        int64_t lo, int64_t hi, int32_t *out, int64_t *n_out, void *scratch, hipStream_t s)
{
    const T *c = static_cast<const T *>(col);
    // (a count or a selection that is narrowed in place needs the look-back:
    // a unit writes after every earlier one has read its own)
    const bool in_place = S && out == sel_in;
    if (n <= (S ? FT_TINY_SEL_ROWS : FT_TINY_BYTES / int64_t(sizeof(T))) && n_out != n_dev && !in_place) {
        const uint32_t grid = static_cast<uint32_t>(n > 0 ? (n + FT_THREADS - 1) / FT_THREADS : 1);
        return gq_launch(ctx, "gq_filter", filter_tiny_kernel<T, S>, dim3(grid), dim3(FT_THREADS), 0, s, c, sel_in, n,
                         n_dev, lo, hi, reinterpret_cast<uintptr_t>(col) % 16 == 0 ? 1 : 0, out, n_out);
    }
    gq_carver cv(scratch);
    const filter_ws w = filter_layout(cv, n);
    GQ_TRY(gq_zero(ctx, scratch, cv.off / 4, s));     // unit counter + status words (a kernel: no memset node under capture)
    const int steps = ft_steps(n);
    const int64_t unit = static_cast<int64_t>(FT_THREADS) * steps;
    const dim3 grid(static_cast<uint32_t>(n > 0 ? (n + unit - 1) / unit : 1));
    auto launch = [&](auto kernel, int entries) {     // entries of LDS per wave
        return gq_launch(ctx, "gq_filter", kernel, grid, dim3(FT_THREADS),
                         static_cast<size_t>(FT_WAVES) * entries * sizeof(int32_t), s, c, sel_in, n, n_dev, lo, hi,
                         steps, out, n_out, w.unit_ctr, w.status);
    };
    if constexpr (S)
        if (in_place) return launch(filter_kernel<T, true, true>, steps * 64);
    return launch(filter_kernel<T, S, false>, ft_stage(steps));
}

gq_status run_filter(gq_ctx *ctx, const void *col, int dtype, const int32_t *sel_in, int64_t n, const int64_t *n_dev,
                     int64_t lo, int64_t hi, int32_t *out, int64_t *n_out, void *scratch, hipStream_t s)
{
    if (dtype == GQ_I32)
        return sel_in ? launch_filter<int32_t, true>(ctx, col, sel_in, n, n_dev, lo, hi, out, n_out, scratch, s)
                      : launch_filter<int32_t, false>(ctx, col, sel_in, n, n_dev, lo, hi, out, n_out, scratch, s);
    return sel_in ? launch_filter<int64_t, true>(ctx, col, sel_in, n, n_dev, lo, hi, out, n_out, scratch, s)
                  : launch_filter<int64_t, false>(ctx, col, sel_in, n, n_dev, lo, hi, out, n_out, scratch, s);
}

// Scratch of gq_filter_noalloc, one copy per GPU for the life of the
// process: the dequeue counter (64 words) and one look-back status word per
// unit, enough for the largest accepted input (GQ_MAX_ROWS rows: 65,536
// units), 512.25 KiB in all.
constexpr int64_t FT_SCRATCH_UNITS = (GQ_MAX_ROWS + FT_THREADS * FT_MAX_STEPS - 1) / (FT_THREADS * FT_MAX_STEPS);
constexpr size_t FT_SCRATCH_WORDS = 32 + static_cast<size_t>(FT_SCRATCH_UNITS);   // 8-byte words
__device__ __align__(256) uint64_t scratch[FT_SCRATCH_WORDS];

}  // namespace

// Device address of this library's filter scratch on the context's device
// (the device must be current).  Host code uses this address, never the
// array's name, which on the host is only a stand-in.
gq_status gq_filter_scratch_setup(gq_ctx *ctx)
{
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
        return gq_fail(ctx, GQ_ERR_HIP, "filter scratch address: %s", hipGetErrorString(e));
    ctx->filter_scratch = p;
    return GQ_OK;
}

extern "C" {

size_t gq_filter_workspace_bytes(int64_t n)
{
    if (n < 0) n = 0;
    gq_carver c(nullptr);
    filter_layout(c, n);
    return c.bytes();
}

gq_status gq_filter(gq_ctx *ctx, const void *col, int dtype, int64_t n, const int64_t *n_dev,
                    const int32_t *sel_in, int64_t lo, int64_t hi, int32_t *sel_out, int64_t *n_out_dev,
                    void *ws, size_t ws_bytes, gq_stream stream)
{
    if (!ctx) return GQ_ERR_INVALID_ARG;
    if ((!col && n > 0) || !sel_out || !n_out_dev)
        return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_filter: NULL column, output or count");
    if (n < 0 || n > GQ_MAX_ROWS) return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_filter: n=%lld out of range", (long long)n);
    if (dtype != GQ_I32 && dtype != GQ_I64) return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_filter: bad dtype %d", dtype);
    const size_t need = gq_filter_workspace_bytes(n);
    if (!ws || ws_bytes < need)
        return gq_fail(ctx, GQ_ERR_WORKSPACE, "gq_filter: workspace %zu < %zu bytes", ws_bytes, need);
    return run_filter(ctx, col, dtype, sel_in, n, n_dev, lo, hi, sel_out, n_out_dev, ws,
                      static_cast<hipStream_t>(stream));
}

gq_status gq_filter_noalloc(gq_ctx *ctx, const void *col, int dtype, int64_t n, const int64_t *n_dev,
                            const int32_t *sel_in, int64_t lo, int64_t hi, int32_t *sel_out, int64_t *n_out_dev,
                            gq_stream stream)
{
    if (!ctx) return GQ_ERR_INVALID_ARG;
    if ((!col && n > 0) || !sel_out || !n_out_dev)
        return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_filter_noalloc: NULL column, output or count");
    if (n < 0 || n > GQ_MAX_ROWS)
        return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_filter_noalloc: n=%lld outside [0, %lld]", (long long)n,
                       (long long)GQ_MAX_ROWS);
    if (dtype != GQ_I32 && dtype != GQ_I64)
        return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_filter_noalloc: bad dtype %d", dtype);
    if (!ctx->filter_scratch) return gq_fail(ctx, GQ_ERR_HIP, "gq_filter_noalloc: no scratch on this device");
    gq_carver need(nullptr);
    filter_layout(need, n);
    if (need.bytes() > FT_SCRATCH_WORDS * sizeof(uint64_t))
        return gq_fail(ctx, GQ_ERR_CAPACITY, "gq_filter_noalloc: %lld rows need %zu scratch bytes, more than %zu",
                       (long long)n, need.bytes(), FT_SCRATCH_WORDS * sizeof(uint64_t));
    return run_filter(ctx, col, dtype, sel_in, n, n_dev, lo, hi, sel_out, n_out_dev, ctx->filter_scratch,
                      static_cast<hipStream_t>(stream));
}

}  // extern "C"
