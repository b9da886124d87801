// Top-k with ties broken by ascending row id.
//
// Every selected row gets a 96-bit order key (ok, rk): ok maps the int64 value
// to an unsigned word whose order is the requested order, and
// rk = 0x7fffffff - rowid ranks smaller row ids higher; the k entries with the
// largest keys are the answer.  Keys differ unless the selection names a row
// more than once: it then counts as often as it is named.
//
// Stage 1 (many workgroups, one pass over the data): each workgroup streams a
// contiguous chunk of the selection; rows whose key beats the workgroup's
// current threshold are appended to an LDS candidate buffer; when the buffer
// could overflow, a radix selection cuts it to the best k and raises the
// threshold to (the leading digits of) the k-th key.  The workgroup's best k
// go to a candidate array.  Row ids are loaded two steps ahead and values one
// step ahead, and the per-step barriers order LDS only, so the loads stay in
// flight.  Stage 2 merges the candidate lists with the same buffer loop:
// first groups of lists in parallel (one workgroup per group, each keeping its
// best k), then one workgroup over the group results, which sorts its best k
// (bitonic) and writes the answer.
#include "gq_device.h"
#include "gq_internal.h"

namespace {

constexpr int TK_THREADS = 512;
constexpr int TK_STEP_ITEMS = 4;
constexpr int TK_STEP = TK_THREADS * TK_STEP_ITEMS;  // rows per step
constexpr int TK_CAP = 4096;                          // LDS candidates
constexpr int TK_MAX_K = TK_CAP - TK_STEP;            // 2048
constexpr uint64_t TK_SIGN = 0x8000000000000000ull;
constexpr uint32_t TK_RANKED = 256;                   // keys of an answer that are ranked by counting
static_assert(TK_RANKED <= TK_THREADS, "one key per thread");

struct tk_entry {
    uint64_t ok;
    uint32_t rk;
};

GQ_DEV bool tk_better(uint64_t aok, uint32_t ark, uint64_t bok, uint32_t brk)
{
    return aok > bok || (aok == bok && ark > brk);
}

struct tk_lds {
    uint64_t ok[TK_CAP];
    uint32_t rk[TK_CAP];
    uint32_t count;
    uint64_t th_ok;
    uint32_t th_rk;
    uint32_t has_th;
    uint32_t hist[2][256];          // digit counts of the selection, two passes in turn
    uint64_t diff;                  // bits in which the entries' values differ
    uint32_t sel_bin, sel_need, sel_cnt;
    uint32_t scan[TK_THREADS / 64];
};

// Bitonic sort, best first, of the first `size` (power of two) entries.
// Stage (k, j) compares entries lo and lo + j, where lo is the i-th index
// with bit j clear: i with a zero inserted at bit position log2(j) (shifts
// and masks, no integer division).
GQ_DEV void tk_sort(tk_lds &L, int size)
{
    for (int k = 2; k <= size; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < size / 2; i += TK_THREADS) {
                const int lo = ((i & ~(j - 1)) << 1) | (i & (j - 1));
                const int hi = lo + j;
                const bool best_first = (lo & k) == 0;
                const uint64_t aok = L.ok[lo], bok = L.ok[hi];
                const uint32_t ark = L.rk[lo], brk = L.rk[hi];
                const bool swap = best_first ? tk_better(bok, brk, aok, ark) : tk_better(aok, ark, bok, brk);
                if (swap) {
                    L.ok[lo] = bok;
                    L.ok[hi] = aok;
                    L.rk[lo] = brk;
                    L.rk[hi] = ark;
                }
            }
            gq_lds_barrier();
        }
    }
}

// Sort the first L.count entries, best first.  Block-wide.
GQ_DEV void tk_sort_count(tk_lds &L)
{
    const int cnt = static_cast<int>(L.count);
    int size = 64;
    while (size < cnt) size <<= 1;
    for (int i = cnt + threadIdx.x; i < size; i += TK_THREADS) {
        L.ok[i] = 0;            // (0, 0) ranks below every real entry (rk >= 1)
        L.rk[i] = 0;
    }
    gq_lds_barrier();
    tk_sort(L, size);
}

// The leading digits of the need-th best of the buffer's entries (ok, rk hold
// this thread's, `valid` which of them exist; at least `need` exist), by radix
// selection over the 96-bit keys (ok, then rk), eight bits at a time.  A pass
// counts, among the entries that carry the digits chosen so far, how many take
// each value of the next digit; the chosen value is the one at which the count
// of better entries reaches the number still needed.  Once every entry
// carrying the chosen digits is needed, those entries and all better ones are
// exactly the best `need`: the entries whose digits under the masks are at
// least the prefix.  Entries of one row have equal keys: if the need-th best
// is one of several, every digit is chosen and the entries at or above the
// prefix are more than `need`.  The digits that all entries share are skipped:
// every add of such a pass would meet on one counter, and values far from 64
// bits wide (prices in cents) share most of theirs.  Block-wide.
constexpr int TK_PER = TK_CAP / TK_THREADS;           // buffer entries per thread

struct tk_prefix {
    uint64_t p_ok, m_ok;                              // chosen digits and their mask
    uint32_t p_rk, m_rk;
};

GQ_DEV tk_prefix tk_digits(tk_lds &L, const uint64_t (&ok)[TK_PER], const uint32_t (&rk)[TK_PER], uint32_t valid,
                           uint32_t need)
{
    const uint64_t ok0 = L.ok[0];
    uint64_t diff = 0;
#pragma unroll
    for (int i = 0; i < TK_PER; ++i) diff |= ((valid >> i) & 1u) ? ok[i] ^ ok0 : 0ull;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) diff |= __shfl_xor(diff, d, 64);
    if (threadIdx.x == 0) L.diff = 0;
    for (int i = threadIdx.x; i < 2 * 256; i += TK_THREADS) (&L.hist[0][0])[i] = 0;
    gq_lds_barrier();
    if (gq_lane() == 0 && diff) atomicOr(reinterpret_cast<unsigned long long *>(&L.diff), static_cast<unsigned long long>(diff));
    gq_lds_barrier();
    diff = L.diff;
    const int d0 = diff ? __builtin_clzll(diff) / 8 : 8;          // the first digit that differs
    tk_prefix x{0, 0, 0, 0};
    if (d0 > 0) {
        x.m_ok = d0 == 8 ? ~0ull : ~(~0ull >> (8 * d0));
        x.p_ok = ok0 & x.m_ok;
    }
    for (int d = d0; d < 12; ++d) {
        uint32_t *h = L.hist[d & 1];
        const int sh = d < 8 ? 56 - 8 * d : 24 - 8 * (d - 8);
#pragma unroll
        for (int i = 0; i < TK_PER; ++i) {
            if (((valid >> i) & 1u) && (ok[i] & x.m_ok) == x.p_ok && (rk[i] & x.m_rk) == x.p_rk) {
                const uint32_t dig = d < 8 ? static_cast<uint32_t>(ok[i] >> sh) & 255u : (rk[i] >> sh) & 255u;
                atomicAdd(&h[dig], 1u);
            }
        }
        if (d > d0)
            for (int i = threadIdx.x; i < 256; i += TK_THREADS) L.hist[(d + 1) & 1][i] = 0;
        gq_lds_barrier();
        if (threadIdx.x < 64) {                       // one wave finds the digit, from 255 down
            const uint32_t lane = threadIdx.x;
            uint32_t hb[4], sum = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                hb[j] = h[255 - 4 * lane - j];
                sum += hb[j];
            }
            const uint32_t incl = gq_wave_inclusive_scan(sum);
            uint32_t acc = incl - sum;
            if (acc < need && need <= incl) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (acc < need && need <= acc + hb[j]) {
                        L.sel_bin = 255 - 4 * lane - j;
                        L.sel_need = need - acc;
                        L.sel_cnt = hb[j];
                    }
                    acc += hb[j];
                }
            }
        }
        gq_lds_barrier();
        const uint32_t bin = L.sel_bin, c = L.sel_cnt;
        need = L.sel_need;
        if (d < 8) {
            x.p_ok |= static_cast<uint64_t>(bin) << sh;
            x.m_ok |= 255ull << sh;
        } else {
            x.p_rk |= bin << sh;
            x.m_rk |= 255u << sh;
        }
        if (c == need) break;                         // same in every thread
    }
    return x;
}

// This thread's entries of the buffer.
GQ_DEV uint32_t tk_entries(const tk_lds &L, uint64_t (&ok)[TK_PER], uint32_t (&rk)[TK_PER])
{
    const uint32_t cnt = L.count;
    uint32_t valid = 0;
#pragma unroll
    for (int i = 0; i < TK_PER; ++i) {
        const uint32_t e = threadIdx.x + i * TK_THREADS;
        const bool v = e < cnt;
        ok[i] = v ? L.ok[e] : 0;
        rk[i] = v ? L.rk[e] : 0;
        valid |= v ? (1u << i) : 0u;
    }
    return valid;
}

// Keep the best k entries of the buffer (in no particular order; never more
// than k, also where equal keys lie at the k-th place) and raise the threshold
// to the chosen digits followed by zero bits: no larger than the k-th best
// key, so no key that belongs in the best k is turned away later.
// Block-wide; L.count must be the same in every thread on entry.
GQ_DEV void tk_select(tk_lds &L, int k)
{
    if (L.count <= static_cast<uint32_t>(k)) return;
    uint64_t ok[TK_PER];
    uint32_t rk[TK_PER];
    const uint32_t valid = tk_entries(L, ok, rk);
    const tk_prefix x = tk_digits(L, ok, rk, valid, static_cast<uint32_t>(k));
    bool kp[TK_PER];
    uint32_t keep = 0;
#pragma unroll
    for (int i = 0; i < TK_PER; ++i) {
        const uint64_t a = ok[i] & x.m_ok;
        const uint32_t b = rk[i] & x.m_rk;
        kp[i] = ((valid >> i) & 1u) && (a > x.p_ok || (a == x.p_ok && b >= x.p_rk));
        keep += kp[i] ? 1u : 0u;
    }
    uint32_t total;
    uint32_t pos = gq_block_exclusive_scan_lds<TK_THREADS>(keep, &total, L.scan);
    // equal keys at the k-th place: those past the k best go behind them, where
    // the next candidates overwrite them
    const bool tie = total > static_cast<uint32_t>(k);
    if (__builtin_expect(tie, 0)) {
        uint32_t eq = 0, all;
#pragma unroll
        for (int i = 0; i < TK_PER; ++i) eq += kp[i] && ok[i] == x.p_ok && rk[i] == x.p_rk ? 1u : 0u;
        const uint32_t r = gq_block_exclusive_scan_lds<TK_THREADS>(eq, &all, L.scan);
        uint32_t better = pos - r, last = total - all + r;         // places of this thread's better and equal keys
#pragma unroll
        for (int i = 0; i < TK_PER; ++i) {
            if (kp[i]) {
                const bool e = ok[i] == x.p_ok && rk[i] == x.p_rk;
                const uint32_t at = e ? last++ : better++;
                L.ok[at] = ok[i];
                L.rk[at] = rk[i];
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < TK_PER; ++i) {
            if (kp[i]) {
                L.ok[pos] = ok[i];
                L.rk[pos] = rk[i];
                ++pos;
            }
        }
    }
    if (threadIdx.x == 0) {
        L.count = static_cast<uint32_t>(k);
        L.th_ok = x.p_ok;
        L.th_rk = x.p_rk;
        L.has_th = 1;
    }
    gq_lds_barrier();
}

GQ_DEV void tk_offer(tk_lds &L, bool valid, uint64_t ok, uint32_t rk, uint64_t th_ok, uint32_t th_rk, bool has_th)
{
    if (valid && (!has_th || tk_better(ok, rk, th_ok, th_rk))) {
        const uint32_t slot = atomicAdd(&L.count, 1u);
        L.ok[slot] = ok;
        L.rk[slot] = rk;
    }
}

GQ_DEV uint64_t tk_order(int64_t v, bool desc)
{
    const uint64_t u = static_cast<uint64_t>(v) ^ TK_SIGN;
    return desc ? u : ~u;
}

// Up to this k the merges take every candidate: recording and ranking the
// lists' bounds costs more than it saves (128 lists of 100 keys: 33 us in two
// merges, 39 us in one with bounds, and 5 us more in the scan).  At k = 1000
// and 512 lists the merges took 126 us without bounds and take 51 with them.
constexpr int TK_PLAIN_K = 256;

// Candidate lists: list i holds cnt[i] <= k keys from i * k, and a bound that
// at least `need` of them reach (0, 0 if it has fewer).
struct tk_lists {
    uint64_t *ok;
    uint32_t *rk;
    uint32_t *cnt;
    uint64_t *b_ok;
    uint32_t *b_rk;
};

// Keys per list whose bound is recorded: with `lists` of them, ceil(k / need)
// is about half the lists.
__host__ __device__ inline uint32_t tk_need(int k, int lists)
{
    if (k <= TK_PLAIN_K) return 0;
    const int x = (2 * k + lists - 1) / lists;
    return static_cast<uint32_t>(x < k ? x : k);
}

// The buffer's entries (at most k) as list blockIdx.x.
GQ_DEV void tk_write_list(tk_lds &L, int k, uint32_t need, const tk_lists &out)
{
    const uint32_t cnt = L.count;
    for (uint32_t i = threadIdx.x; i < cnt; i += TK_THREADS) {
        out.ok[static_cast<int64_t>(blockIdx.x) * k + i] = L.ok[i];
        out.rk[static_cast<int64_t>(blockIdx.x) * k + i] = L.rk[i];
    }
    tk_prefix x{0, 0, 0, 0};
    if (need != 0 && cnt >= need) {                                // same in every thread
        uint64_t ok[TK_PER];
        uint32_t rk[TK_PER];
        const uint32_t valid = tk_entries(L, ok, rk);
        x = tk_digits(L, ok, rk, valid, need);
    }
    if (threadIdx.x == 0) {
        out.cnt[blockIdx.x] = cnt;
        if (need != 0) {
            out.b_ok[blockIdx.x] = x.p_ok;
            out.b_rk[blockIdx.x] = x.p_rk;
        }
    }
}

__global__ __launch_bounds__(TK_THREADS) void topk_stage1_kernel(const int64_t *__restrict__ val,
                                                                 const int32_t *__restrict__ sel, int64_t n_bound,
                                                                 const int64_t *n_dev, int k, int desc,
                                                                 int64_t chunk, uint32_t need, tk_lists out)
{
    __shared__ tk_lds L;
    int64_t n = n_bound;
    if (n_dev) {
        const int64_t d = *n_dev;
        n = d < n_bound ? (d > 0 ? d : 0) : n_bound;
    }
    if (threadIdx.x == 0) {
        L.count = 0;
        L.has_th = 0;
        L.th_ok = 0;
        L.th_rk = 0;
    }
    gq_lds_barrier();
    // the chunk of each workgroup, from the device row count when there is one
    // (the host's chunk covers the bound and would leave workgroups idle)
    if (n_dev) {
        const int64_t per = (n + gridDim.x - 1) / gridDim.x;
        chunk = (per + TK_STEP - 1) / TK_STEP * TK_STEP;
        if (chunk < TK_STEP) chunk = TK_STEP;
    }
    const int64_t j0 = static_cast<int64_t>(blockIdx.x) * chunk;
    int64_t j1 = j0 + chunk;
    if (j1 > n) j1 = n;
    auto row_at = [&](int64_t j) -> int32_t {
        return j < j1 ? (sel ? __builtin_nontemporal_load(&sel[j]) : static_cast<int32_t>(j)) : 0;
    };
    // pipeline: r0/v0 = step s (offered now), r1/v1 = step s+1, r2 = step s+2
    int32_t r0[TK_STEP_ITEMS], r1[TK_STEP_ITEMS], r2[TK_STEP_ITEMS];
    int64_t v0[TK_STEP_ITEMS], v1[TK_STEP_ITEMS];
#pragma unroll
    for (int c = 0; c < TK_STEP_ITEMS; ++c) {
        r0[c] = row_at(j0 + c * TK_THREADS + threadIdx.x);
        r1[c] = row_at(j0 + TK_STEP + c * TK_THREADS + threadIdx.x);
    }
#pragma unroll
    for (int c = 0; c < TK_STEP_ITEMS; ++c) {
        const int64_t j = j0 + c * TK_THREADS + threadIdx.x;
        v0[c] = j < j1 ? __builtin_nontemporal_load(&val[r0[c]]) : 0;
    }
    for (int64_t s = j0; s < j1; s += TK_STEP) {
#pragma unroll
        for (int c = 0; c < TK_STEP_ITEMS; ++c) r2[c] = row_at(s + 2 * TK_STEP + c * TK_THREADS + threadIdx.x);
#pragma unroll
        for (int c = 0; c < TK_STEP_ITEMS; ++c) {
            const int64_t j = s + TK_STEP + c * TK_THREADS + threadIdx.x;
            v1[c] = j < j1 ? __builtin_nontemporal_load(&val[r1[c]]) : 0;
        }
        const uint64_t th_ok = L.th_ok;
        const uint32_t th_rk = L.th_rk;
        const bool has_th = L.has_th != 0;
#pragma unroll
        for (int c = 0; c < TK_STEP_ITEMS; ++c) {
            const int64_t j = s + c * TK_THREADS + threadIdx.x;
            tk_offer(L, j < j1, tk_order(v0[c], desc), 0x7fffffffu - static_cast<uint32_t>(r0[c]), th_ok, th_rk,
                     has_th);
        }
        gq_lds_barrier();
        const uint32_t cnt_now = L.count;      // same value in every thread
        gq_lds_barrier();
        if (cnt_now > static_cast<uint32_t>(TK_CAP - TK_STEP)) tk_select(L, k);
#pragma unroll
        for (int c = 0; c < TK_STEP_ITEMS; ++c) {
            r0[c] = r1[c];
            v0[c] = v1[c];
            r1[c] = r2[c];
        }
    }
    tk_select(L, k);
    tk_write_list(L, k, need, out);
}

// Merge lists [blockIdx.x * per, +per) of up to k keys each (in any order)
// into the best k; the last level (LAST) sorts them and writes the answer.
//
// First the lists' bounds give a key that the k-th best overall cannot be
// below: of all the level's lists, each has `need` keys at or above its
// bound, so the ceil(k / need)-th largest bound has k keys at or above it.
// With need about 2 k / lists that is near the median bound, and a list of
// rows in no particular order keeps about `need` of its k keys: the merge
// selects among about 2 k keys instead of lists * k.
template <bool LAST>
__global__ __launch_bounds__(TK_THREADS) void topk_merge_kernel(tk_lists in, int nlists, int per, int k,
                                                                uint32_t in_need, uint32_t need, tk_lists out,
                                                                int desc, int64_t *__restrict__ val_out,
                                                                int32_t *__restrict__ rowid_out, int64_t *n_out)
{
    __shared__ tk_lds L;
    __shared__ uint32_t pre[TK_THREADS];
    __shared__ uint32_t placed[TK_RANKED];                         // keys of the answer put at each place
    const int tid = threadIdx.x;
    if (LAST && tid < static_cast<int>(TK_RANKED)) placed[tid] = 0;
    const int b0 = static_cast<int>(blockIdx.x) * per;
    const int lists = nlists - b0 < per ? nlists - b0 : per;       // nlists <= TK_THREADS
    uint32_t total;
    pre[tid] = gq_block_exclusive_scan_lds<TK_THREADS>(tid < lists ? in.cnt[b0 + tid] : 0u, &total, L.scan);
    tk_prefix t{0, 0, 0, 0};
    if (in_need != 0) {
        // the bound of rank ceil(k / in_need) among all lists, its leading digits
        if (tid < nlists) {
            L.ok[tid] = in.b_ok[tid];
            L.rk[tid] = in.b_rk[tid];
        }
        if (tid == 0) L.count = static_cast<uint32_t>(nlists);
        gq_lds_barrier();
        uint64_t ok[TK_PER];
        uint32_t rk[TK_PER];
        const uint32_t valid = tk_entries(L, ok, rk);
        t = tk_digits(L, ok, rk, valid, (static_cast<uint32_t>(k) + in_need - 1) / in_need);
        gq_lds_barrier();
    }
    if (tid == 0) {
        L.count = 0;
        L.has_th = 0;
        L.th_ok = 0;
        L.th_rk = 0;
    }
    gq_lds_barrier();
    // the lists' keys as one sequence of `total`, a step ahead in flight
    uint64_t nok[TK_STEP_ITEMS];
    uint32_t nrk[TK_STEP_ITEMS];
    auto load = [&](uint32_t s) {
#pragma unroll
        for (int c = 0; c < TK_STEP_ITEMS; ++c) {
            const uint32_t j = s + c * TK_THREADS + tid;
            nok[c] = 0;
            nrk[c] = 0;                                            // (0, 0) is below every key
            if (j < total) {
                uint32_t w = 0;                                    // the last list with pre[w] <= j
#pragma unroll
                for (uint32_t d = TK_THREADS / 2; d; d >>= 1)
                    if (pre[w + d] <= j) w += d;
                const int64_t at = static_cast<int64_t>(b0 + static_cast<int>(w)) * k + (j - pre[w]);
                nok[c] = in.ok[at];
                nrk[c] = in.rk[at];
            }
        }
    };
    load(0);
    for (uint32_t s = 0; s < total; s += TK_STEP) {
        const uint64_t th_ok = L.th_ok;
        const uint32_t th_rk = L.th_rk;
        const bool has_th = L.has_th != 0;
#pragma unroll
        for (int c = 0; c < TK_STEP_ITEMS; ++c) {
            const bool in_reach = (nok[c] | nrk[c]) != 0 && !tk_better(t.p_ok, t.p_rk, nok[c], nrk[c]);
            tk_offer(L, in_reach, nok[c], nrk[c], th_ok, th_rk, has_th);
        }
        load(s + TK_STEP);
        gq_lds_barrier();
        const uint32_t cnt_now = L.count;      // same value in every thread
        gq_lds_barrier();
        if (cnt_now > static_cast<uint32_t>(TK_CAP - TK_STEP)) tk_select(L, k);
    }
    tk_select(L, k);
    if constexpr (!LAST) {
        tk_write_list(L, k, need, out);
    } else {
        const uint32_t cnt = L.count;                              // at most k
        auto put = [&](uint32_t at, uint64_t o, uint32_t r) {
            const uint64_t u = desc ? o : ~o;
            val_out[at] = static_cast<int64_t>(u ^ TK_SIGN);
            rowid_out[at] = static_cast<int32_t>(0x7fffffffu - r);
        };
        if (cnt <= TK_RANKED) {
            // a few keys: each thread counts those better than its own, with no
            // barrier in between, where a sort has one for each of its
            // log2(cnt)^2 / 2 stages (k = 100 of 3M rows 37.5 -> 34.2 us, k = 10
            // of 200K rows 21.9 -> 17.9); equal ones take the places from there on
            if (tid < static_cast<int>(cnt)) {
                const uint64_t o = L.ok[tid];
                const uint32_t r = L.rk[tid];
                uint32_t at = 0;
                for (uint32_t j = 0; j < cnt; ++j) at += tk_better(L.ok[j], L.rk[j], o, r) ? 1u : 0u;
                put(at + atomicAdd(&placed[at], 1u), o, r);
            }
        } else {
            tk_sort_count(L);                                      // the answer, best first
            for (uint32_t x = tid; x < cnt; x += TK_THREADS) put(x, L.ok[x], L.rk[x]);
        }
        if (tid == 0) *n_out = cnt;
    }
}

// Candidates that one workgroup merges alone, and lists per workgroup of a
// first merge level otherwise (k = 100, 128 lists: 33 us at 16, 36 at 32, 41 at
// 48).  Lists with bounds are merged in pairs where the bounds leave about 2 k
// keys (k = 1000 of 50M rows in no order: 158 us in pairs, 161 by three).  In a
// sorted column, or one with many ties, half the lists or all of them pass the
// bound, and the last merge, alone on the chip, walks their keys; so a group
// takes as many lists as leave it TK_LAST_MERGE of them at most (50M rows, in
// pairs and in such groups, us: the 1000 largest values of a rising column 1131
// and 936, its 1000 smallest 252 and 214, 2048 of equal values 456 and 282).
int64_t tk_one_merge(int k) { return k <= TK_PLAIN_K ? 8192 : 32768; }
constexpr int64_t TK_LAST_MERGE = 3 << 16;
int tk_merge_per(int64_t lists, int k)
{
    if (k <= TK_PLAIN_K) return 16;
    const int64_t per = (lists * k + TK_LAST_MERGE - 1) / TK_LAST_MERGE;
    return per > 2 ? static_cast<int>(per) : 2;
}
constexpr int TK_MAX_LISTS = 512;                     // two scan workgroups per CU
static_assert(TK_MAX_LISTS <= TK_THREADS, "a merge holds one list per thread");

struct tk_ws {
    tk_lists first, second;
    int blocks, groups, per;            // lists, groups of `per` lists in the first merge level (0: one merge)
    int64_t chunk;
};

tk_lists tk_take_lists(gq_carver &c, int64_t lists, int k)
{
    tk_lists l;
    l.ok = c.take<uint64_t>(static_cast<size_t>(lists) * k);
    l.rk = c.take<uint32_t>(static_cast<size_t>(lists) * k);
    l.cnt = c.take<uint32_t>(static_cast<size_t>(lists));
    l.b_ok = c.take<uint64_t>(static_cast<size_t>(lists));
    l.b_rk = c.take<uint32_t>(static_cast<size_t>(lists));
    return l;
}

tk_ws tk_layout(gq_carver &c, int64_t n, int k)
{
    tk_ws w;
    // at least 2 steps per block: a small scan is a chain of steps, and the
    // merge takes more lists more easily (1M rows, k = 100: 166 us for the
    // pipeline around it at 2, 174 at 4, 168 at 1; 3M rows 37 at 2, 41 at 4)
    int64_t blocks = (n + 2 * TK_STEP - 1) / (2 * TK_STEP);
    if (blocks > TK_MAX_LISTS) blocks = TK_MAX_LISTS;          // two 512-thread workgroups fit a CU (95 VGPRs)
    if (blocks < 1) blocks = 1;
    int64_t chunk = (n + blocks - 1) / blocks;
    chunk = ((chunk + TK_STEP - 1) / TK_STEP) * TK_STEP;
    if (chunk < TK_STEP) chunk = TK_STEP;
    w.blocks = static_cast<int>(blocks);
    w.per = tk_merge_per(blocks, k);
    w.groups = blocks * k > tk_one_merge(k) ? static_cast<int>((blocks + w.per - 1) / w.per) : 0;
    w.chunk = chunk;
    w.first = tk_take_lists(c, blocks, k);
    // (room for the groups of the fewest lists, so that the size grows with n)
    const int fewest = tk_merge_per(1, k);
    if (w.groups > 0) w.second = tk_take_lists(c, (blocks + fewest - 1) / fewest, k);
    return w;
}

}  // namespace

extern "C" {

size_t gq_topk_workspace_bytes(int64_t n, int k)
{
    if (n < 0) n = 0;
    if (k < 1) k = 1;
    gq_carver c(nullptr);
    tk_layout(c, n, k);
    if (k <= TK_PLAIN_K) return c.bytes();
    // a workspace made for k keys serves smaller answers too (above TK_PLAIN_K
    // more candidates are merged at once, without lists of a second level)
    gq_carver p(nullptr);
    tk_layout(p, n, TK_PLAIN_K);
    return c.bytes() > p.bytes() ? c.bytes() : p.bytes();
}

gq_status gq_topk(gq_ctx *ctx, const int64_t *val, const int32_t *sel, int64_t n, const int64_t *n_dev, int k,
                  int descending, int64_t *val_out, int32_t *rowid_out, int64_t *n_out_dev, void *ws,
                  size_t ws_bytes, gq_stream stream)
{
    if (!ctx) return GQ_ERR_INVALID_ARG;
    if (n < 0 || n > GQ_MAX_ROWS) return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_topk: n=%lld", (long long)n);
    if (k < 1) return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_topk: k=%d", k);
    if (k > TK_MAX_K) return gq_fail(ctx, GQ_ERR_UNSUPPORTED, "gq_topk: k=%d > %d", k, TK_MAX_K);
    if ((!val && n > 0) || !val_out || !rowid_out || !n_out_dev)
        return gq_fail(ctx, GQ_ERR_INVALID_ARG, "gq_topk: NULL value, output or count");
    const size_t need = gq_topk_workspace_bytes(n, k);
    if (!ws || ws_bytes < need)
        return gq_fail(ctx, GQ_ERR_WORKSPACE, "gq_topk: workspace %zu < %zu bytes", ws_bytes, need);
    hipStream_t s = static_cast<hipStream_t>(stream);
    gq_carver c(ws);
    tk_ws w = tk_layout(c, n, k);
    const int d = descending ? 1 : 0;
    const uint32_t need1 = tk_need(k, w.blocks);
    GQ_TRY(gq_launch(ctx, "gq_topk_local", topk_stage1_kernel, dim3(static_cast<uint32_t>(w.blocks)),
                     dim3(TK_THREADS), 0, s, val, sel, n, n_dev, k, d, w.chunk, need1, w.first));
    if (w.groups == 0)
        return gq_launch(ctx, "gq_topk_merge", topk_merge_kernel<true>, dim3(1), dim3(TK_THREADS), 0, s, w.first,
                         w.blocks, w.blocks, k, need1, 0u, tk_lists{}, d, val_out, rowid_out, n_out_dev);
    const uint32_t need2 = tk_need(k, w.groups);
    GQ_TRY(gq_launch(ctx, "gq_topk_merge", topk_merge_kernel<false>, dim3(static_cast<uint32_t>(w.groups)),
                     dim3(TK_THREADS), 0, s, w.first, w.blocks, w.per, k, need1, need2, w.second, d, val_out,
                     rowid_out, n_out_dev));
    return gq_launch(ctx, "gq_topk_merge", topk_merge_kernel<true>, dim3(1), dim3(TK_THREADS), 0, s, w.second,
                     w.groups, w.groups, k, need2, 0u, tk_lists{}, d, val_out, rowid_out, n_out_dev);
}

}  // extern "C"
