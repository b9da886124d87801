// Hash equi-join: open-addressing build and ordered probe.
//
// Table: a 256-byte header then 2^L slots of 16 bytes {int64 key, int32
// payload, int32 unused}; EMPTY key = INT64_MIN.  The home slot of a key is
// the TOP L bits of fmix64(key): the same hash bits that pick a key's radix
// partition, so a probe stream that was partitioned by that hash touches one
// contiguous slice of the table at a time.  Linear probing, wrapping.
//
// Build, tables of up to 8192 slots: one workgroup builds the table in LDS.
//
// Build, other small tables: a fill kernel writes header and EMPTY slots; an
// insert kernel claims slots with a 64-bit compare-and-swap in device memory and then
// stores the payload (the probe runs in a later kernel, so it sees the store).
//
// Build, large tables (device-memory CAS runs at only ~10 G/s on MI355X): the
// build rows are sorted by the region of their home slot, a region being
// 4096 consecutive slots: the partition operator by the top 8 hash bits,
// then, for more than 256 regions, one workgroup per bucket splitting it by
// the remaining region bits; one workgroup per region inserts its keys into an LDS copy of the
// region with LDS compare-and-swap and writes the region out linearly.  A key
// whose probe runs past its region's last slot goes to an overflow list and is
// inserted afterwards by device CAS from the first slot of the next region,
// which is exactly where linear probing would continue; the table is the same
// valid linear-probing table either way.
//
// Probe: a unit of probe rows is looked up with one 16-byte load per slot
// visited; matches become a bitmap (ballots), payloads wait in LDS, and after
// a block scan and a decoupled look-back over units each wave writes its
// matches at their place in probe order.
#include <algorithm>
#include <cstdlib>
#include <cstring>

#include "gq_device.h"
#include "gq_internal.h"
#include "gq_ops.h"

namespace {

constexpr uint64_t JT_MAGIC = 0x6a6f696e74626c31ull;   // "join tbl1"
constexpr int64_t JT_EMPTY = INT64_MIN;
constexpr size_t JT_HEADER = 256;

struct jt_header {
    uint64_t magic;
    uint32_t log2_slots;
    uint32_t unused;
    uint64_t slots;
};

struct alignas(16) jt_slot {
    int64_t key;
    int32_t payload;
    int32_t unused;
};

int jt_log2_slots(int64_t m, double lf)
{
    double want = static_cast<double>(m) / lf;
    int L = 6;
    while (L < 40 && static_cast<double>(1ull << L) < want) ++L;
    return L;
}

__global__ void jt_init_kernel(void *table, int log2_slots)
{
    const uint64_t slots = 1ull << log2_slots;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        jt_header *h = static_cast<jt_header *>(table);
        h->magic = JT_MAGIC;
        h->log2_slots = static_cast<uint32_t>(log2_slots);
        h->unused = 0;
        h->slots = slots;
    }
    jt_slot *s = reinterpret_cast<jt_slot *>(static_cast<char *>(table) + JT_HEADER);
    const uint64_t stride = static_cast<uint64_t>(gridDim.x) * blockDim.x;
    for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < slots; i += stride) {
        jt_slot e;
        e.key = JT_EMPTY;
        e.payload = 0;
        e.unused = 0;
        s[i] = e;
    }
}

// Keys beyond the region build's reach (too few, a selection or a device
// count), one per thread.  Walks on from the home slot look at JT_AHEAD slots
// in one trip (8: the same).  A build of up to JT_NEAR_KEYS keys is bound by the
// longest walk of any key, a chain of compare-and-swaps through the fabric (25
// slots and more in a table half full); most walks end within JT_NEAR slots of
// the home slot, which it tries one by one first.  A larger one is bound by the
// compare-and-swaps' number, of which looking first makes fewer.  One by one,
// looking from the home slot on, and from JT_NEAR on, us: 20K keys at load
// factor 0.25 8.6, 9.3 and 8.6, at 0.5 10.0, 11.0 and 9.9, 120K keys at 0.5
// 22.7, 20.6 and 19.9; 1.2M keys at 0.5 97, 78 and 97, 3M at 0.9 396, 213 and 281.
constexpr int JT_NEAR = 2;
constexpr int64_t JT_NEAR_KEYS = 1 << 18;
constexpr int JT_AHEAD = 4;

__global__ __launch_bounds__(256) void jt_insert_kernel(void *table, int log2_slots, const int64_t *__restrict__ key,
                                                        const int32_t *__restrict__ payload, int64_t m_bound,
                                                        const int64_t *n_dev, const int32_t *__restrict__ sel,
                                                        int near, uint32_t *status)
{
    int64_t m = m_bound;
    if (n_dev) {
        const int64_t d = *n_dev;
        m = d < m_bound ? (d > 0 ? d : 0) : m_bound;
    }
    jt_slot *slots = reinterpret_cast<jt_slot *>(static_cast<char *>(table) + JT_HEADER);
    const uint64_t mask = (1ull << log2_slots) - 1;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < m; i += stride) {
        const int64_t r = sel ? static_cast<int64_t>(sel[i]) : i;
        const int64_t k = key[r];
        const int32_t p = payload[r];
        if (k == JT_EMPTY) {
            gq_raise(status, GQ_ERR_INVALID_KEY);
            continue;
        }
        uint64_t s = gq_fmix64(static_cast<uint64_t>(k)) >> (64 - log2_slots);
        // the home slot and `near` on are tried at once; a walk on from there
        // reads JT_AHEAD slots together and tries those found empty
        const unsigned long long want = static_cast<unsigned long long>(k);
        const unsigned long long none = static_cast<unsigned long long>(JT_EMPTY);
        unsigned long long prev = atomicCAS(reinterpret_cast<unsigned long long *>(&slots[s].key), none, want);
        bool done = prev == none || prev == want;
        uint64_t probes = 0;
        for (int q = 0; q < near && !done; ++q) {
            s = (s + 1) & mask;
            ++probes;
            prev = atomicCAS(reinterpret_cast<unsigned long long *>(&slots[s].key), none, want);
            done = prev == none || prev == want;
        }
        while (!done && probes < mask) {
            unsigned long long w[JT_AHEAD];
#pragma unroll
            for (int i = 0; i < JT_AHEAD; ++i)
                w[i] = __hip_atomic_load(reinterpret_cast<unsigned long long *>(&slots[(s + 1 + i) & mask].key),
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            int at = JT_AHEAD;                       // the first slot that is empty or holds this key
#pragma unroll
            for (int i = JT_AHEAD - 1; i >= 0; --i)
                if (w[i] == none || w[i] == want) at = i;
            if (at == JT_AHEAD) {
                s = (s + JT_AHEAD) & mask;
                probes += JT_AHEAD;
                continue;
            }
            s = (s + 1 + at) & mask;
            probes += 1 + at;
            prev = atomicCAS(reinterpret_cast<unsigned long long *>(&slots[s].key), none, want);
            done = prev == none || prev == want;
        }
        if (!done) gq_raise(status, GQ_ERR_CAPACITY);
        else if (prev == want) gq_raise(status, GQ_ERR_DUPLICATE_KEY);
        else slots[s].payload = p;
    }
}

// Tables of at most JB_LDS_SLOTS slots, bound by latency: one workgroup builds
// the table in LDS and writes it out, in one launch with no device
// compare-and-swaps (4096 keys with a probe of 64K rows: 27.5 -> 24.7 us; 1000
// keys with 10K rows: 32.6 -> 20, of which the host's share is most).
constexpr int JB_LDS_SLOTS = 8192;                  // 96 KB of keys and payloads
constexpr int JB_THREADS = 1024;
constexpr int JB_BATCH = 4;                         // keys per thread loaded together

__global__ __launch_bounds__(JB_THREADS) void jt_lds_build_kernel(void *table, int log2_slots,
                                                                  const int64_t *__restrict__ key,
                                                                  const int32_t *__restrict__ payload, int64_t m_bound,
                                                                  const int64_t *n_dev, const int32_t *__restrict__ sel,
                                                                  uint32_t *status)
{
    extern __shared__ unsigned long long jb_keys[];
    const int slots = 1 << log2_slots;
    int32_t *jb_pay = reinterpret_cast<int32_t *>(jb_keys + slots);
    int64_t m = m_bound;
    if (n_dev) {
        const int64_t d = *n_dev;
        m = d < m_bound ? (d > 0 ? d : 0) : m_bound;
    }
    int64_t k[JB_BATCH];
    int32_t p[JB_BATCH];
    auto load = [&](int64_t i0) {
#pragma unroll
        for (int c = 0; c < JB_BATCH; ++c) {
            const int64_t i = i0 + c * JB_THREADS + threadIdx.x;
            k[c] = 0;
            p[c] = 0;
            if (i < m) {
                const int64_t r = sel ? static_cast<int64_t>(sel[i]) : i;
                k[c] = key[r];
                p[c] = payload[r];
            }
        }
    };
    load(0);
    for (int j = threadIdx.x; j < slots; j += JB_THREADS) {
        jb_keys[j] = static_cast<unsigned long long>(JT_EMPTY);
        jb_pay[j] = 0;
    }
    __syncthreads();
    for (int64_t i0 = 0; i0 < m; i0 += JB_THREADS * JB_BATCH) {
        if (i0 > 0) load(i0);
#pragma unroll
        for (int c = 0; c < JB_BATCH; ++c) {
            if (i0 + c * JB_THREADS + threadIdx.x >= m) continue;
            if (k[c] == JT_EMPTY) {
                gq_raise(status, GQ_ERR_INVALID_KEY);
                continue;
            }
            uint32_t s = static_cast<uint32_t>(gq_fmix64(static_cast<uint64_t>(k[c])) >> (64 - log2_slots));
            int probes = 0;
            for (; probes < slots; ++probes) {
                const unsigned long long prev = atomicCAS(&jb_keys[s], static_cast<unsigned long long>(JT_EMPTY),
                                                          static_cast<unsigned long long>(k[c]));
                if (prev == static_cast<unsigned long long>(JT_EMPTY)) {
                    jb_pay[s] = p[c];
                    break;
                }
                if (prev == static_cast<unsigned long long>(k[c])) {
                    gq_raise(status, GQ_ERR_DUPLICATE_KEY);
                    break;
                }
                s = (s + 1) & static_cast<uint32_t>(slots - 1);
            }
            if (probes == slots) gq_raise(status, GQ_ERR_CAPACITY);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        jt_header *h = static_cast<jt_header *>(table);
        h->magic = JT_MAGIC;
        h->log2_slots = static_cast<uint32_t>(log2_slots);
        h->unused = 0;
        h->slots = static_cast<uint64_t>(slots);
    }
    jt_slot *out = reinterpret_cast<jt_slot *>(static_cast<char *>(table) + JT_HEADER);
    for (int j = threadIdx.x; j < slots; j += JB_THREADS) {
        jt_slot e;
        e.key = static_cast<int64_t>(jb_keys[j]);
        e.payload = jb_pay[j];
        e.unused = 0;
        out[j] = e;
    }
}

constexpr int JR_BITS = 12;                         // 4096 slots per region (64 KiB)
constexpr int JR_SLOTS = 1 << JR_BITS;
constexpr int JR_MAX_REGION_BITS = 16;              // two 8-bit levels at most
constexpr int64_t JR_MIN_KEYS = 1 << 18;            // below this the CAS build is used

// Second level of the region sort.  The first level is a radix partition by
// the top JS_HIGH bits of the hash; workgroup b takes that partition's bucket
// b and splits it by the next g - JS_HIGH bits, so that the keys end up
// ordered by region (the top g bits) and roff[r] is the first key of region
// r.  It counts its bucket's sub-buckets first (one read of the keys), which
// gives both the region starts and the output cursors, then moves the bucket
// tile by tile: a tile's rows are grouped by sub-bucket in LDS and each group
// is written at its cursor as one run.  Rows keep no particular order inside
// a region; the region kernel's inserts do not depend on it.
constexpr int JS_HIGH = 8;                           // bits of the first level
constexpr int JS_THREADS = 1024;
constexpr int JS_ITEMS = 8;
constexpr int JS_TILE = JS_THREADS * JS_ITEMS;

GQ_DEV uint32_t js_sub(int64_t k, int g, uint32_t smask)
{
    return static_cast<uint32_t>(gq_fmix64(static_cast<uint64_t>(k)) >> (64 - g)) & smask;
}

__global__ __launch_bounds__(JS_THREADS) void jt_split_kernel(const int64_t *__restrict__ k1,
                                                              const int32_t *__restrict__ p1,
                                                              const int64_t *__restrict__ bstart, int64_t m, int g,
                                                              int64_t *__restrict__ k2, int32_t *__restrict__ p2,
                                                              int64_t *__restrict__ roff)
{
    __shared__ uint32_t cnt[1 << JS_HIGH];           // sub-bucket sizes, then a tile's counts
    __shared__ uint32_t tstart[1 << JS_HIGH];        // a tile's sub-bucket starts in the stage
    __shared__ int64_t cur[1 << JS_HIGH];            // output cursor of each sub-bucket
    __shared__ uint32_t scan_smem[JS_THREADS / 64];
    __shared__ uint8_t lsub[JS_TILE];
    __shared__ int64_t sk[JS_TILE];
    __shared__ int32_t sp[JS_TILE];
    const int sb = g - JS_HIGH;                      // 1..8 sub-bucket bits
    const uint32_t S = 1u << sb, smask = S - 1;
    const int tid = threadIdx.x;
    const int64_t b0 = bstart[blockIdx.x], b1 = bstart[blockIdx.x + 1];

    for (uint32_t i = tid; i < S; i += JS_THREADS) cnt[i] = 0;
    __syncthreads();
    for (int64_t i0 = b0; i0 < b1; i0 += 2 * JS_TILE) {
        int64_t kk[2 * JS_ITEMS];
#pragma unroll
        for (int c = 0; c < 2 * JS_ITEMS; ++c) {
            const int64_t e = i0 + c * JS_THREADS + tid;
            kk[c] = e < b1 ? k1[e] : 0;
        }
#pragma unroll
        for (int c = 0; c < 2 * JS_ITEMS; ++c)
            if (i0 + c * JS_THREADS + tid < b1) atomicAdd(&cnt[js_sub(kk[c], g, smask)], 1u);
    }
    __syncthreads();
    uint32_t total;
    const uint32_t excl = gq_block_exclusive_scan<JS_THREADS>(static_cast<uint32_t>(tid) < S ? cnt[tid] : 0u,
                                                              &total, scan_smem);
    if (static_cast<uint32_t>(tid) < S) {
        cur[tid] = b0 + excl;
        roff[(static_cast<int64_t>(blockIdx.x) << sb) + tid] = b0 + excl;
        cnt[tid] = 0;
    }
    if (blockIdx.x == gridDim.x - 1 && tid == 0) roff[static_cast<int64_t>(gridDim.x) << sb] = m;

    int64_t k[JS_ITEMS];
    int32_t p[JS_ITEMS];
    auto load_tile = [&](int64_t i0) {
#pragma unroll
        for (int c = 0; c < JS_ITEMS; ++c) {
            const int64_t e = i0 + c * JS_THREADS + tid;
            const bool v = e < b1;
            k[c] = v ? k1[e] : 0;
            p[c] = v ? p1[e] : 0;
        }
    };
    if (b0 < b1) load_tile(b0);
    __syncthreads();
    for (int64_t i0 = b0; i0 < b1; i0 += JS_TILE) {
        uint32_t l[JS_ITEMS], rank[JS_ITEMS];
#pragma unroll
        for (int c = 0; c < JS_ITEMS; ++c) {
            l[c] = js_sub(k[c], g, smask);
            if (i0 + c * JS_THREADS + tid < b1) rank[c] = atomicAdd(&cnt[l[c]], 1u);
        }
        gq_lds_barrier();
        uint32_t tot;
        const uint32_t st = gq_block_exclusive_scan_lds<JS_THREADS>(
            static_cast<uint32_t>(tid) < S ? cnt[tid] : 0u, &tot, scan_smem);
        if (static_cast<uint32_t>(tid) < S) tstart[tid] = st;
        gq_lds_barrier();
#pragma unroll
        for (int c = 0; c < JS_ITEMS; ++c) {
            if (i0 + c * JS_THREADS + tid < b1) {
                const uint32_t q = tstart[l[c]] + rank[c];
                sk[q] = k[c];
                sp[q] = p[c];
                lsub[q] = static_cast<uint8_t>(l[c]);
            }
        }
        const int64_t next = i0 + JS_TILE;
        if (next < b1) load_tile(next);              // in flight while this tile is written
        gq_lds_barrier();
        const uint32_t count = static_cast<uint32_t>(b1 - i0 < JS_TILE ? b1 - i0 : JS_TILE);
        for (uint32_t q = tid; q < count; q += JS_THREADS) {
            const uint32_t x = lsub[q];
            const int64_t dst = cur[x] + (q - tstart[x]);
            k2[dst] = sk[q];
            p2[dst] = sp[q];
        }
        gq_lds_barrier();
        if (static_cast<uint32_t>(tid) < S) {
            cur[tid] += cnt[tid];
            cnt[tid] = 0;
        }
        gq_lds_barrier();
    }
}

// A persistent grid walks the regions; the barriers between a region's phases
// order LDS only, so one region's table stores drain while the next region's
// keys load.  A thread's keys of a region (up to JR_BATCH, a region holding
// about 2048 * load factor keys) are loaded together, and the next region's
// are loaded before the current region is written out.
constexpr int JR_THREADS = 256;
constexpr int JR_BATCH = 8;                          // keys per thread loaded together

__global__ __launch_bounds__(JR_THREADS) void jt_region_kernel(void *table, int L, const int64_t *__restrict__ keys,
                                                               const int32_t *__restrict__ pay,
                                                               const int64_t *__restrict__ roff, int64_t nregions,
                                                               int64_t *__restrict__ ovf_key,
                                                               int32_t *__restrict__ ovf_pay, uint32_t *ovf_cnt,
                                                               int64_t ovf_cap, uint32_t *status)
{
    __shared__ unsigned long long sk[JR_SLOTS];
    __shared__ int32_t sp[JR_SLOTS];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        jt_header *h = static_cast<jt_header *>(table);
        h->magic = JT_MAGIC;
        h->log2_slots = static_cast<uint32_t>(L);
        h->unused = 0;
        h->slots = 1ull << L;
    }
    int64_t k[JR_BATCH];
    int32_t p[JR_BATCH];
    bool v[JR_BATCH];
    auto load_batch = [&](int64_t i0, int64_t end) {
#pragma unroll
        for (int c = 0; c < JR_BATCH; ++c) {
            const int64_t i = i0 + c * JR_THREADS + threadIdx.x;
            v[c] = i < end;
            k[c] = v[c] ? keys[i] : 0;
            p[c] = v[c] ? pay[i] : 0;
        }
    };
    int64_t region = blockIdx.x;
    int64_t r0 = 0, r1 = 0;
    if (region < nregions) {
        r0 = roff[region];
        r1 = roff[region + 1];
        load_batch(r0, r1);
    }
    for (; region < nregions; region += gridDim.x) {
        gq_lds_barrier();                             // the previous region is read out of LDS
        for (int j = threadIdx.x; j < JR_SLOTS; j += JR_THREADS) {
            sk[j] = static_cast<unsigned long long>(JT_EMPTY);
            sp[j] = 0;
        }
        gq_lds_barrier();
        for (int64_t i0 = r0;;) {
#pragma unroll
            for (int c = 0; c < JR_BATCH; ++c) {
                if (!v[c]) continue;
                if (k[c] == JT_EMPTY) {
                    gq_raise(status, GQ_ERR_INVALID_KEY);
                    continue;
                }
                uint32_t loc =
                    static_cast<uint32_t>(gq_fmix64(static_cast<uint64_t>(k[c])) >> (64 - L)) & (JR_SLOTS - 1);
                while (true) {
                    const unsigned long long prev = atomicCAS(&sk[loc], static_cast<unsigned long long>(JT_EMPTY),
                                                              static_cast<unsigned long long>(k[c]));
                    if (prev == static_cast<unsigned long long>(JT_EMPTY)) {
                        sp[loc] = p[c];
                        break;
                    }
                    if (prev == static_cast<unsigned long long>(k[c])) {
                        gq_raise(status, GQ_ERR_DUPLICATE_KEY);
                        break;
                    }
                    if (++loc == JR_SLOTS) {             // continue in the next region, later
                        const uint32_t idx = atomicAdd(ovf_cnt, 1u);
                        if (idx < ovf_cap) {
                            ovf_key[idx] = k[c];
                            ovf_pay[idx] = p[c];
                        } else {
                            gq_raise(status, GQ_ERR_CAPACITY);
                        }
                        break;
                    }
                }
            }
            i0 += JR_THREADS * JR_BATCH;
            if (i0 >= r1) break;
            load_batch(i0, r1);                          // a region with more keys than one batch
        }
        const int64_t next = region + gridDim.x;         // the next region's keys: in flight meanwhile
        if (next < nregions) {
            r0 = roff[next];
            r1 = roff[next + 1];
            load_batch(r0, r1);
        }
        gq_lds_barrier();
        jt_slot *slots = reinterpret_cast<jt_slot *>(static_cast<char *>(table) + JT_HEADER) +
                         (static_cast<uint64_t>(region) << JR_BITS);
        for (int j = threadIdx.x; j < JR_SLOTS; j += JR_THREADS) {
            jt_slot e;
            e.key = static_cast<int64_t>(sk[j]);
            e.payload = sp[j];
            e.unused = 0;
            slots[j] = e;
        }
    }
}

__global__ __launch_bounds__(256) void jt_overflow_kernel(void *table, int L, const int64_t *__restrict__ ovf_key,
                                                          const int32_t *__restrict__ ovf_pay,
                                                          const uint32_t *ovf_cnt, int64_t ovf_cap, uint32_t *status)
{
    const int64_t cnt = *ovf_cnt;
    const int64_t n = cnt < ovf_cap ? cnt : ovf_cap;
    jt_slot *slots = reinterpret_cast<jt_slot *>(static_cast<char *>(table) + JT_HEADER);
    const uint64_t mask = (1ull << L) - 1;
    const int g = L - JR_BITS;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t k = ovf_key[i];
        const uint64_t home_region = gq_fmix64(static_cast<uint64_t>(k)) >> (64 - g);
        uint64_t s = ((home_region + 1) << JR_BITS) & mask;
        uint64_t probes = 0;
        for (; probes <= mask; ++probes) {
            unsigned long long *kp = reinterpret_cast<unsigned long long *>(&slots[s].key);
            const unsigned long long prev =
                atomicCAS(kp, static_cast<unsigned long long>(JT_EMPTY), static_cast<unsigned long long>(k));
            if (prev == static_cast<unsigned long long>(JT_EMPTY)) {
                slots[s].payload = ovf_pay[i];
                break;
            }
            if (prev == static_cast<unsigned long long>(k)) {
                gq_raise(status, GQ_ERR_DUPLICATE_KEY);
                break;
            }
            s = (s + 1) & mask;
        }
        if (probes > mask) gq_raise(status, GQ_ERR_CAPACITY);
    }
}

int table_log2_from_bytes(size_t table_bytes)
{
    int L = 6;
    while (L < 40 && JT_HEADER + (size_t(2) << L) * sizeof(jt_slot) <= table_bytes) ++L;
    return L;
}

// Which build a call takes: "region" for large tables built from whole
// columns, "cas" otherwise.  GQ_JOIN_BUILD=cas|region forces one (testing).
bool use_region_build(int64_t m, int L, bool has_sel_or_count)
{
    const int g = L - JR_BITS;
    if (has_sel_or_count || g < 1 || g > JR_MAX_REGION_BITS) return false;
    const char *e = getenv("GQ_JOIN_BUILD");
    if (e && strcmp(e, "cas") == 0) return false;
    if (e && strcmp(e, "region") == 0) return true;
    return m >= JR_MIN_KEYS;
}

struct build_ws {
    int64_t *k1, *k2;
    int32_t *p1, *p2;
    int64_t *offsets;
    int64_t *roff;
    void *part_ws;
    int64_t *ovf_key;
    int32_t *ovf_pay;
    uint32_t *ovf_cnt;
    int64_t ovf_cap;
};

build_ws build_layout(gq_carver &c, int64_t m)
{
    build_ws w{};
    const size_t rows = static_cast<size_t>(m > 0 ? m : 1);
    w.ovf_cnt = c.take<uint32_t>(64);
    w.k1 = c.take<int64_t>(rows);
    w.k2 = c.take<int64_t>(rows);
    w.p1 = c.take<int32_t>(rows);
    w.p2 = c.take<int32_t>(rows);
    w.offsets = c.take<int64_t>(257);
    w.roff = c.take<int64_t>((size_t(1) << JR_MAX_REGION_BITS) + 1);
    w.part_ws = c.take<char>(gq_partition_bits_workspace(m, 8));
    w.ovf_cap = m / 8 + 1024;
    w.ovf_key = c.take<int64_t>(static_cast<size_t>(w.ovf_cap));
    w.ovf_pay = c.take<int32_t>(static_cast<size_t>(w.ovf_cap));
    return w;
}

gq_status region_build(gq_ctx *ctx, const int64_t *key, const int32_t *payload, int64_t m, void *table, int L,
                       void *ws, hipStream_t s)
{
    gq_carver c(ws);
    build_ws w = build_layout(c, m);
    const int g = L - JR_BITS;
    const int32_t pbytes = 4;
    static const gq_part_names nm{"gq_join_build_part_hist", "gq_join_build_part_scan", "gq_join_build_part_scatter"};
    GQ_TRY(gq_zero(ctx, w.ovf_cnt, 64, s));
    void *in[1] = {const_cast<int32_t *>(payload)};
    if (g <= JS_HIGH) {                             // one pass: its bucket starts are the region starts
        void *out[1] = {w.p2};
        GQ_TRY(gq_partition_bits(ctx, key, m, g, 64 - g, 1, in, &pbytes, w.k2, out, w.roff, w.part_ws, s, nm, 16));
    } else {                                        // the top JS_HIGH bits, then each bucket by the rest
        void *out[1] = {w.p1};
        GQ_TRY(gq_partition_bits(ctx, key, m, JS_HIGH, 64 - JS_HIGH, 1, in, &pbytes, w.k1, out, w.offsets, w.part_ws,
                                 s, nm, 16));
        GQ_TRY(gq_launch(ctx, "gq_join_build_split", jt_split_kernel, dim3(1u << JS_HIGH), dim3(JS_THREADS), 0, s,
                         static_cast<const int64_t *>(w.k1), static_cast<const int32_t *>(w.p1),
                         static_cast<const int64_t *>(w.offsets), m, g, w.k2, w.p2, w.roff));
    }
    const int64_t nregions = int64_t(1) << g;
    const uint32_t rgrid = static_cast<uint32_t>(std::min<int64_t>(nregions, int64_t(ctx->num_cus) * 3));
    GQ_TRY(gq_launch(ctx, "gq_join_build_regions", jt_region_kernel, dim3(rgrid), dim3(JR_THREADS), 0, s, table, L,
                     static_cast<const int64_t *>(w.k2), static_cast<const int32_t *>(w.p2),
                     static_cast<const int64_t *>(w.roff), nregions, w.ovf_key, w.ovf_pay, w.ovf_cnt, w.ovf_cap,
                     ctx->status_dev));
    return gq_launch(ctx, "gq_join_build_overflow", jt_overflow_kernel, dim3(64), dim3(256), 0, s, table, L,
                     static_cast<const int64_t *>(w.ovf_key), static_cast<const int32_t *>(w.ovf_pay),
                     static_cast<const uint32_t *>(w.ovf_cnt), w.ovf_cap, ctx->status_dev);
}

// Shape of the ordered probe.  A workgroup takes one unit of consecutive rows
// with one dequeue and one look-back; each wave owns a contiguous stretch of
// the unit and walks it 64 rows at a time, one row per lane: 32 waves per CU
// keep enough slot loads in flight, while more rows per lane in flight evict
// each other's lines from L2 before the next slot of a row is read (4 rows per
// lane 1.20, 2 rows 1.11, 1 row 1.09 ms on 50M probes of a 268 MB table).
//
// A large unit matters because each unit's look-back reads status words that
// other XCDs write, over the same path as the slot lines: with 4096-row units
// the same lookups took 1.29-1.50 ms.  16K rows (64 KB of LDS for their
// payloads, two workgroups per CU) are the most that keep 32 waves per CU.
// So 512 units run at a time, and a few more than that run a round of their
// own: calls of more than JP_ROUND_ROWS rows take the fewest steps that do in
// as many rounds (64K keys, units of 8 steps and so, us: 2.2M rows in 269 and
// 430 units 57 and 45, 4.3M in 525 and 467 100 and 69, 9M in 1075 and 977 158 and
// 135, 25M 374 and 333).  Below 1M rows half the chip's places are enough, a unit
// per CU (500K rows: 18.6 us in 245, 22 in 489; 1M in 489 and 245: 27 and 22).
// Up to JP_TINY_ROWS rows the chip is not full either way and a call is bound
// by one unit's chain of loads and the look-back: 512-row units (64K rows:
// 31 -> 12 us; 100K rows 18 us at 256 rows, 13 at 512 and at 1024).
constexpr int64_t JP_TINY_ROWS = 1 << 17;
constexpr int JP_AHEAD = 4;
constexpr int64_t JP_AHEAD_ROWS = 1 << 20;
constexpr int JP_THREADS = 1024;
constexpr int JP_TINY_THREADS = 512;
constexpr int JP_MAX_STEPS = 16;
constexpr int JP_SHORT_STEPS = 4;                   // with a unit per CU
constexpr int64_t JP_ROUND_ROWS = int64_t(512) * JP_THREADS;   // rows of a step of all resident units
struct jp_shape {
    int threads, steps;
    int64_t unit() const { return static_cast<int64_t>(threads) * steps; }
};

jp_shape jp_shape_of(int64_t n)
{
    if (n <= JP_TINY_ROWS) return {JP_TINY_THREADS, 1};
    const int64_t short_steps = (n + JP_ROUND_ROWS / 2 - 1) / (JP_ROUND_ROWS / 2);
    if (short_steps <= JP_SHORT_STEPS) return {JP_THREADS, static_cast<int>(short_steps)};
    const int64_t rounds = (n + JP_ROUND_ROWS * JP_MAX_STEPS - 1) / (JP_ROUND_ROWS * JP_MAX_STEPS);
    const int64_t steps = (n + JP_ROUND_ROWS * rounds - 1) / (JP_ROUND_ROWS * rounds);
    return {JP_THREADS, static_cast<int>(std::max<int64_t>(steps, JP_SHORT_STEPS))};
}

struct probe_ws {
    uint32_t *unit_ctr;
    uint64_t *status;
};

probe_ws probe_layout(gq_carver &c, int64_t n)
{
    probe_ws w;
    const int64_t rows = jp_shape_of(n).unit();
    int64_t units = (n + rows - 1) / rows;
    // a workspace made for n rows serves every smaller call too (the units of
    // a smaller call can be more: at most 512 a round, rounds of 8.4M rows)
    if (n > JP_TINY_ROWS) units = n / (JP_THREADS * JP_MAX_STEPS / 2) + 1024;
    w.unit_ctr = c.take<uint32_t>(64);
    w.status = c.take<uint64_t>(static_cast<size_t>(units > 0 ? units : 1));
    return w;
}

// Bound by the lines of the table: each probe moves a 128-byte line, and the
// chip moves about 55 G random lines/s from memory (a bare gather).  50M
// probes of a 6M-key table (268 MB): 1.49 -> 1.09 ms, 46 G probes/s with the
// 0.7 GB of keys and outputs streamed beside them.
//
// AHEAD: slots that a walk on from the home slot reads in one trip.  A call of
// few rows is one unit per workgroup and bound by its longest walks, a chain
// of trips to the L2; a call of many is bound by the lines themselves, and
// slots read too far cost more.  At 1 and at 4, us: 500K keys, 400K rows 19.5
// and 17.2, 2^20 rows 31.3 and 28.1, 1.5M 42.6 and 43.8, 3M 69 and 75; 50K keys,
// 200K rows 11.9 and 11.4, 2^20 22.1 and 21.5, 1.5M 32.6 and 34.5, 12M 159 and 173.
//
// IN_PLACE: prow_out is the selection itself.  A unit's outputs lie at its own
// or earlier rows, and every earlier unit has read its rows before it publishes
// its count; so a unit keeps its row ids in LDS instead of reading them again.
template <bool HAS_SEL, int THREADS, int AHEAD, bool IN_PLACE = false>
__global__ __launch_bounds__(THREADS) void jt_probe_kernel(const void *table, const int64_t *__restrict__ fk,
                                                           int64_t n_bound, const int64_t *n_dev,
                                                           const int32_t *__restrict__ sel, int steps,
                                                           int expect_log2, int32_t *__restrict__ prow_out,
                                                           int32_t *__restrict__ pay_out, int64_t *n_out,
                                                           uint32_t *unit_ctr, uint64_t *lb_status, uint32_t *status)
{
    constexpr int WAVES = THREADS / 64;
    constexpr int MAX_WORDS = WAVES * JP_MAX_STEPS;
    static_assert(MAX_WORDS <= THREADS, "one word per thread in the scan");
    static_assert(HAS_SEL || !IN_PLACE, "without a selection there is nothing to overwrite");
    extern __shared__ int32_t pay_lds[];              // payload of each row of the unit (then their row ids)
    int32_t *row_lds = pay_lds + THREADS * steps;     // IN_PLACE
    __shared__ uint64_t bits[MAX_WORDS];              // matches of the unit, one bit per row
    __shared__ uint32_t wpre[MAX_WORDS];              // matches before each word
    __shared__ uint32_t scan_smem[WAVES];
    __shared__ uint32_t s_unit;
    __shared__ uint64_t s_goff;

    int64_t n = n_bound;
    if (n_dev) {
        const int64_t d = *n_dev;
        n = d < n_bound ? (d > 0 ? d : 0) : n_bound;
    }
    if (threadIdx.x == 0) s_unit = atomicAdd(unit_ctr, 1u);
    __syncthreads();
    const uint32_t t = s_unit;
    const int L = static_cast<int>(static_cast<const jt_header *>(table)->log2_slots);
    if (expect_log2 != 0 && L != expect_log2) {       // the caller's table size is another: no output
        if (t == 0 && threadIdx.x == 0) {
            *n_out = 0;
            gq_raise(status, GQ_ERR_INVALID_ARG);
        }
        return;
    }
    const int64_t unit = static_cast<int64_t>(THREADS) * steps;
    const int64_t nunits = (n + unit - 1) / unit;
    if (static_cast<int64_t>(t) >= nunits) {
        if (t == 0 && threadIdx.x == 0) *n_out = 0;
        return;
    }
    const uint64_t mask = (1ull << L) - 1;
    const jt_slot *slots = reinterpret_cast<const jt_slot *>(static_cast<const char *>(table) + JT_HEADER);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int word0 = wave * steps;                   // the wave's first word
    const int64_t row0 = static_cast<int64_t>(t) * unit + static_cast<int64_t>(word0) * 64 + lane;

    // the key of the next step is loaded (and the selection of the one after)
    // while this step's slot is on its way: issued after the slot's load, which
    // is waited for first (loads return in order; issued before it, 1.18 ms)
    int32_t nr = 0;
    int64_t nk;
    auto load_row = [&](int i) {
        const int64_t e = row0 + i * 64;
        if (HAS_SEL) nr = (i < steps && e < n) ? sel[e] : 0;
    };
    auto load_key = [&](int i) {
        const int64_t e = row0 + i * 64;
        if (IN_PLACE && i < steps) row_lds[(word0 + i) * 64 + lane] = nr;
        nk = (i < steps && e < n) ? __builtin_nontemporal_load(&fk[HAS_SEL ? static_cast<int64_t>(nr) : e]) : JT_EMPTY;
    };
    load_row(0);
    load_key(0);
    load_row(1);
    for (int i = 0; i < steps; ++i) {
        const int64_t k = nk;
        uint64_t s = gq_fmix64(static_cast<uint64_t>(k)) >> (64 - L);
        int4 v{};
        if (k != JT_EMPTY) v = *reinterpret_cast<const int4 *>(&slots[s]);
        load_key(i + 1);
        load_row(i + 2);
        bool hit = false;
        int32_t pay = 0;
        if (k != JT_EMPTY) {                          // the marker is no key: it matches nothing
            const int64_t sk = (static_cast<int64_t>(static_cast<uint32_t>(v.y)) << 32) | static_cast<uint32_t>(v.x);
            hit = sk == k;
            if (hit) pay = v.z;
            bool done = hit || sk == JT_EMPTY;
            for (uint64_t probes = 0; !done && probes < mask; probes += AHEAD, s += AHEAD) {
                int4 u[AHEAD];
#pragma unroll
                for (int q = 0; q < AHEAD; ++q) u[q] = *reinterpret_cast<const int4 *>(&slots[(s + 1 + q) & mask]);
#pragma unroll
                for (int q = 0; q < AHEAD; ++q) {
                    const int64_t uk =
                        (static_cast<int64_t>(static_cast<uint32_t>(u[q].y)) << 32) | static_cast<uint32_t>(u[q].x);
                    if (!done && uk == k) {
                        hit = true;
                        pay = u[q].z;
                    }
                    done = done || uk == k || uk == JT_EMPTY;
                }
            }
        }
        const uint64_t b = gq_ballot(hit);
        if (lane == 0) bits[word0 + i] = b;
        pay_lds[(word0 + i) * 64 + lane] = pay;
    }
    __syncthreads();
    const int words = WAVES * steps;
    const uint32_t cnt = static_cast<int>(threadIdx.x) < words ? static_cast<uint32_t>(__popcll(bits[threadIdx.x])) : 0u;
    uint32_t total;
    const uint32_t pre = gq_block_exclusive_scan<THREADS>(cnt, &total, scan_smem);
    if (static_cast<int>(threadIdx.x) < words) wpre[threadIdx.x] = pre;
    if (wave == 0) {
        const uint64_t g = gq_lookback(lb_status, t, total);
        if (lane == 0) {
            s_goff = g;
            if (static_cast<int64_t>(t) == nunits - 1) *n_out = static_cast<int64_t>(g + total);
        }
    }
    __syncthreads();
    const int64_t goff = static_cast<int64_t>(s_goff);
    for (int i = 0; i < steps; ++i) {
        const uint64_t b = bits[word0 + i];
        if ((b >> lane) & 1u) {
            const int64_t o = goff + wpre[word0 + i] + gq_mbcnt(b);
            const int64_t e = row0 + i * 64;
            prow_out[o] = IN_PLACE ? row_lds[(word0 + i) * 64 + lane] : HAS_SEL ? sel[e] : static_cast<int32_t>(e);
            pay_out[o] = pay_lds[(word0 + i) * 64 + lane];
        }
    }
}

// Both probe entry points; expect_log2 != 0: the table must have that many
// slots (log2), checked on the device.
gq_status probe(const char *who, gq_ctx *ctx, const void *table, int expect_log2, const int64_t *fk, int64_t n,
                const int64_t *n_dev, const int32_t *sel, int32_t *prow_out, int32_t *payload_out, int64_t *n_out_dev,
                void *ws, size_t ws_bytes, gq_stream stream)
{
    if (!ctx) return GQ_ERR_INVALID_ARG;
    if (n < 0 || n > GQ_MAX_ROWS) return gq_fail(ctx, GQ_ERR_INVALID_ARG, "%s: n=%lld", who, (long long)n);
    if (!table || (!fk && n > 0) || !prow_out || !payload_out || !n_out_dev)
        return gq_fail(ctx, GQ_ERR_INVALID_ARG, "%s: NULL table, fk, output or count", who);
    const size_t need = gq_join_probe_workspace_bytes(n);
    if (!ws || ws_bytes < need)
        return gq_fail(ctx, GQ_ERR_WORKSPACE, "%s: workspace %zu < %zu bytes", who, ws_bytes, need);
    hipStream_t s = static_cast<hipStream_t>(stream);
    gq_carver c(ws);
    probe_ws w = probe_layout(c, n);
    GQ_TRY(gq_zero(ctx, ws, c.off / 4, s));
    const jp_shape sh = jp_shape_of(n);
    const int64_t unit = sh.unit();
    const uint32_t grid = static_cast<uint32_t>(n > 0 ? (n + unit - 1) / unit : 1);
    auto launch = [&](auto kernel, int held = 1) {   // held: 32-bit words kept per row
        return gq_launch(ctx, "gq_join_probe", kernel, dim3(grid), dim3(static_cast<uint32_t>(sh.threads)),
                         static_cast<size_t>(unit) * held * sizeof(int32_t), s, table, fk, n, n_dev, sel, sh.steps,
                         expect_log2, prow_out, payload_out, n_out_dev, w.unit_ctr, w.status, ctx->status_dev);
    };
    if (sel && prow_out == sel)                       // the selection is narrowed in place
        return sh.threads == JP_TINY_THREADS ? launch(jt_probe_kernel<true, JP_TINY_THREADS, JP_AHEAD, true>, 2)
                                             : launch(jt_probe_kernel<true, JP_THREADS, 1, true>, 2);
    if (sh.threads == JP_TINY_THREADS)
        return sel ? launch(jt_probe_kernel<true, JP_TINY_THREADS, JP_AHEAD>)
                   : launch(jt_probe_kernel<false, JP_TINY_THREADS, JP_AHEAD>);
    if (n <= JP_AHEAD_ROWS)
        return sel ? launch(jt_probe_kernel<true, JP_THREADS, JP_AHEAD>)
                   : launch(jt_probe_kernel<false, JP_THREADS, JP_AHEAD>);
    return sel ? launch(jt_probe_kernel<true, JP_THREADS, 1>) : launch(jt_probe_kernel<false, JP_THREADS, 1>);
}

}  // namespace

extern "C" {

size_t gq_join_table_bytes(int64_t m, double load_factor)
{
    if (m < 0 || !(load_factor > 0.0) || load_factor > 0.9) return 0;
    const int L = jt_log2_slots(m, load_factor);
    return JT_HEADER + (size_t(1) << L) * sizeof(jt_slot);
}

size_t gq_join_build_workspace_bytes(int64_t m, size_t table_bytes)
{
    if (m < 0) m = 0;
    const int L = table_log2_from_bytes(table_bytes);
    if (!use_region_build(m, L, false)) return 256;
    gq_carver c(nullptr);
    build_layout(c, m);
    return c.bytes();
}

gq_status gq_join_build(gq_ctx *ctx, const int64_t *key, const int32_t *payload, int64_t m, const int64_t *n_dev,
                        const int32_t *sel, void *table, size_t table_bytes, void *ws, size_t ws_bytes,
                        gq_stream stream)
{
    if (!ctx) return GQ_ERR_INVALID_ARG;
    if (m < 0 || m > GQ_MAX_ROWS) return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_join_build: m=%lld", (long long)m);
    if (!table || (m > 0 && (!key || !payload)))
        return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_join_build: NULL key, payload or table");
    if (reinterpret_cast<uintptr_t>(table) % 256 != 0)
        return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_join_build: table must be 256-byte aligned");
    if (table_bytes < JT_HEADER + 64 * sizeof(jt_slot))
        return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_join_build: table of %zu bytes is too small", table_bytes);
    const int L = table_log2_from_bytes(table_bytes);
    if (static_cast<double>(m) > 0.9 * static_cast<double>(1ull << L))
        return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_join_build: %lld keys exceed load factor 0.9 of %llu slots",
                       (long long)m, (unsigned long long)(1ull << L));
    const bool region = use_region_build(m, L, sel != nullptr || n_dev != nullptr);
    const size_t need = gq_join_build_workspace_bytes(m, table_bytes);
    if (region && (!ws || ws_bytes < need))
        return gq_fail(ctx, GQ_ERR_WORKSPACE, "gq_join_build: workspace %zu < %zu bytes", ws_bytes, need);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (region) return region_build(ctx, key, payload, m, table, L, ws, s);
    const uint64_t slots = 1ull << L;
    if (slots <= JB_LDS_SLOTS)
        return gq_launch(ctx, "gq_join_build_lds", jt_lds_build_kernel, dim3(1), dim3(JB_THREADS),
                         static_cast<size_t>(slots) * (sizeof(int64_t) + sizeof(int32_t)), s, table, L, key, payload, m,
                         n_dev, sel, ctx->status_dev);
    uint64_t blocks = (slots + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    GQ_TRY(gq_launch(ctx, "gq_join_build_init", jt_init_kernel, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, s, table,
                     L));
    if (m == 0) return GQ_OK;
    uint64_t ib = (static_cast<uint64_t>(m) + 255) / 256;
    if (ib > 65536) ib = 65536;
    return gq_launch(ctx, "gq_join_build_insert", jt_insert_kernel, dim3(static_cast<uint32_t>(ib)), dim3(256), 0, s, table,
                     L, key, payload, m, n_dev, sel, m <= JT_NEAR_KEYS ? JT_NEAR : 0, ctx->status_dev);
}

size_t gq_join_probe_workspace_bytes(int64_t n)
{
    if (n < 0) n = 0;
    gq_carver c(nullptr);
    probe_layout(c, n);
    return c.bytes();
}

gq_status gq_join_probe(gq_ctx *ctx, const void *table, const int64_t *fk, int64_t n, const int64_t *n_dev,
                        const int32_t *sel, int32_t *prow_out, int32_t *payload_out, int64_t *n_out_dev, void *ws,
                        size_t ws_bytes, gq_stream stream)
{
    return probe("gq_join_probe", ctx, table, 0, fk, n, n_dev, sel, prow_out, payload_out, n_out_dev, ws, ws_bytes,
                 stream);
}

size_t gq_join_probe_partitioned_workspace_bytes(int64_t n) { return gq_join_probe_workspace_bytes(n); }

// A probe stream in radix-partition order takes the same kernel: its units'
// slots then lie in one slice of the table (200M rows in 64 buckets against a
// 1 GiB table: 2.47 ms; splitting tiles by table region, probing the regions
// from LDS and restoring the order took 2.70 ms, and more on every smaller
// table, fan-out 4 to 8 bits and on skewed keys).
gq_status gq_join_probe_partitioned(gq_ctx *ctx, const void *table, size_t table_bytes, const int64_t *fk,
                                    int64_t n, const int64_t *n_dev, const int32_t *sel, int log2_fanout,
                                    int32_t *prow_out, int32_t *payload_out, int64_t *n_out_dev, void *ws,
                                    size_t ws_bytes, gq_stream stream)
{
    if (!ctx) return GQ_ERR_INVALID_ARG;
    if (table_bytes < JT_HEADER + 64 * sizeof(jt_slot))
        return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_join_probe_partitioned: table of %zu bytes is too small",
                       table_bytes);
    if (log2_fanout < 0 || log2_fanout > 16)
        return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_join_probe_partitioned: log2_fanout=%d", log2_fanout);
    // the size is checked for tables of 2^20 to 2^(log2_fanout + 20) slots
    const int L = table_log2_from_bytes(table_bytes);
    const bool check = L >= 20 && L - std::min(log2_fanout, 8) <= 20;
    return probe("gq_join_probe_partitioned", ctx, table, check ? L : 0, fk, n, n_dev, sel, prow_out, payload_out,
                 n_out_dev, ws, ws_bytes, stream);
}

}  // extern "C"
