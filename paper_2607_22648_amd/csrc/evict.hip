// Frequency-based leaf eviction (PTStore Section 4.1, "Access
// pattern-aware eviction policy": frequency over recency, GDSF adapted to
// shared prefixes).
//
// Every access of a block adds 1 to its frequency F and sets its priority
// H = L + F, L being the store's clock. An insert that needs more new blocks
// than the never-used ids left evicts the difference, each time taking a
// block with no resident child that the batch did not match, the one with
// the lowest H, then the deepest, then the smallest id, and raising L to its
// H. Taken one at a time that is a sequential walk; it has a parallel form:
//
//   a child is never accessed without its parent and the clock only grows,
//   so H(child) <= H(parent), and with depth as the second key the child
//   ranks strictly before its parent in the order (H, deeper first, id).
//   The blocks the batch did not match include every descendant of each of
//   them. Hence the lowest-ranked of them always has no resident child, and
//   the one-at-a-time walk takes exactly the first `want` of them in that
//   order.
//
// So the victims are the `want` smallest keys (H, depth descending, id)
// among the unmatched blocks, found by a radix select. A range pass first
// takes the minimum and maximum of each field over the candidates; the key
// then keeps only the bits in which candidates can differ,
//   (H - Hmin) | (depth_max - depth) | (id - id_min),
// left-aligned in 128 bits (typically some 40 bits wide). Digit passes over
// all candidates, each a 2048-bin histogram of the next 11 bits among the
// keys that agree with the threshold found so far, whose last workgroup to
// finish picks the digit; once few candidates agree in the digits found,
// they are listed, and the last workgroup finds the remaining digits over
// the list alone. Then the victims are marked in a bit mask, their index
// slots become tombstones, L takes their largest H, and a scan lists them by
// ascending id, the order in which their ids are reused. When deleted slots
// have piled up, the index is cleared instead and publish enters the
// surviving blocks again.
//
// The work of a search is small (16 bytes per candidate and pass); what it
// costs is launches. Eight here, where the twelve digit passes, the scan,
// the list and two rebuild steps had made seventeen. A store of up to 16,384
// blocks runs none of this: see evict_small.hpp.
#include "kernels.hpp"
#include "evict_small.hpp"

namespace ptsd {
namespace {

constexpr int kThreads = 256;

typedef unsigned __int128 u128;

// Is `id` ranked by the running search? (sel_lo_id <= id < sel_hi_id holds.)
__device__ inline bool sel_candidate(const EvictView& ev, const DevState* st, int64_t id) {
    return st->sel_hot || ev.prot[id] != (int32_t)st->ev_epoch;
}

// The candidate's compressed key, left-aligned in 128 bits (state written by
// the range pass). Eviction: (H - Hmin, depth_max - depth, id - id_min), the
// smallest go. Hot set: (Hmax - H, id - id_min), the smallest stay.
__device__ inline u128 sel_key(const EvictView& ev, const DevState* st, int64_t id) {
    const bool hot = st->sel_hot != 0;
    const u128 p = (u128)(hot ? st->sel_pbase - ev.prio[id] : ev.prio[id] - st->sel_pbase);
    const u128 d = hot ? (u128)0 : (u128)(st->sel_dmax - (uint64_t)ev.depth[id]);
    const u128 i = (u128)((uint64_t)id - st->sel_imin);
    const unsigned wd = st->sel_wd, wi = st->sel_wi, w = st->sel_w;
    const u128 c = (p << (wd + wi)) | (d << wi) | i;
    return w == 0 ? (u128)0 : c << (128u - w);
}

__device__ inline unsigned long long lanes_below(int lane) {
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

template <typename T, typename Op>
__device__ inline T wave_reduce(T v, Op op, int lane) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v = op(v, (T)shfl_u64((uint64_t)v, lane ^ d));
    return v;
}

// Ranges of H, depth and id over the candidates, their number, and from them
// the key layout. Also clears the digit histograms. Each workgroup writes its
// own partial (no shared-address atomics); the last one to finish combines
// them. Serves both searches (eviction and hot set, see sel_key); an
// eviction's victims are counted here, so that whether the index is rebuilt
// is known before they are marked.
__global__ __launch_bounds__(kThreads) void k_sel_range(EvictView ev, DevState* st, int64_t capacity,
                                                        uint64_t slots_n) {
    if (st->ev_want == 0) return;  // uniform over the grid
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < (int64_t)kSelPasses * kSelBins;
         i += (int64_t)gridDim.x * kThreads)
        ev.hist[i] = 0;
    const int64_t lo_id = (int64_t)st->sel_lo_id, hi_id = (int64_t)st->sel_hi_id;
    // [0] min H, [1] -max H, [2] min depth, [3] -max depth, [4] min id, [5] -max id: all minima
    uint64_t v[6] = {~0ull, ~0ull, ~0ull, ~0ull, ~0ull, ~0ull};
    uint64_t n = 0;
    for (int64_t id = lo_id + (int64_t)blockIdx.x * kThreads + threadIdx.x; id < hi_id;
         id += (int64_t)gridDim.x * kThreads) {
        if (!sel_candidate(ev, st, id)) continue;
        const uint64_t x[6] = {ev.prio[id], ~ev.prio[id], (uint64_t)ev.depth[id], ~(uint64_t)ev.depth[id],
                               (uint64_t)id, ~(uint64_t)id};
#pragma unroll
        for (int k = 0; k < 6; ++k) v[k] = x[k] < v[k] ? x[k] : v[k];
        ++n;
    }
    auto mn = [](uint64_t a, uint64_t b) { return a < b ? a : b; };
    auto sum = [](uint64_t a, uint64_t b) { return a + b; };
    __shared__ uint64_t red[kThreads / kWave][8];
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = wave_reduce(v[k], mn, lane);
    n = wave_reduce(n, sum, lane);
    if (lane == 0) {
        for (int k = 0; k < 6; ++k) red[wv][k] = v[k];
        red[wv][6] = n;
    }
    __syncthreads();
    if (threadIdx.x < 7) {
        const int k = threadIdx.x;
        uint64_t a = red[0][k];
        for (int w = 1; w < kThreads / kWave; ++w) a = k < 6 ? mn(a, red[w][k]) : a + red[w][k];
        ev.part[(int64_t)blockIdx.x * 8 + k] = a;
    }
    __shared__ int last;
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(&st->sel_range_done, 1u) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    __threadfence();
    // last workgroup: combine the partials (one wave per field)
    __shared__ uint64_t tot[8];
    for (int k = wv; k < 7; k += kThreads / kWave) {
        uint64_t a = k < 6 ? ~0ull : 0ull;
        for (int64_t g = lane; g < gridDim.x; g += kWave) {
            const uint64_t x = __hip_atomic_load(&ev.part[g * 8 + k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            a = k < 6 ? mn(a, x) : a + x;
        }
        a = k < 6 ? wave_reduce(a, mn, lane) : wave_reduce(a, sum, lane);
        if (lane == 0) tot[k] = a;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    if (!st->sel_hot)
        evict_account(st, capacity, slots_n, tot[6] < st->ev_want ? tot[6] : st->ev_want);
    if (tot[6] <= st->ev_want) {  // every candidate goes
        st->ev_all = 1;
        return;
    }
    const uint64_t pmin = tot[0], pmax = ~tot[1], dmin = tot[2], dmax = ~tot[3], imin = tot[4],
                   imax = ~tot[5];
    const bool hot = st->sel_hot != 0;
    const unsigned wp = bit_width(pmax - pmin), wd = hot ? 0u : bit_width(dmax - dmin),
                   wi = bit_width(imax - imin);
    st->sel_pbase = hot ? pmax : pmin;
    st->sel_dmax = dmax;
    st->sel_imin = imin;
    st->sel_wd = wd;
    st->sel_wi = wi;
    st->sel_w = wp + wd + wi;  // <= 64 + 31 + 31
    st->sel_npass = (wp + wd + wi + kSelBits - 1) / kSelBits;
}

// One digit pass of the threshold search. Past the second, it runs only while
// more candidates agree with the threshold than one workgroup should list: a
// block with far more accesses than the others widens H by twenty bits or
// more, all of them equal among the candidates that matter, so that how many
// digits it takes to tell those apart is not known beforehand. Evicting 256
// of 1,048,576 blocks, one of them with 2*10^7 accesses: 225 us in the
// eviction's kernels; 272 with three passes, 4,500 with two, 245 with twelve
// that all run. A pass that exits costs 1.7 us.
__global__ __launch_bounds__(kThreads) void k_sel_pass(EvictView ev, DevState* st, int pass) {
    // uniform: the last workgroup changes these when all have read them
    if (st->ev_want == 0 || st->ev_all || (unsigned)pass >= st->sel_npass) return;
    if (pass > 1 && st->sel_bin <= kSelListMax) return;
    __shared__ unsigned int h[kSelBins];
    __shared__ unsigned int part[kThreads];
    __shared__ int last;
    const int t = threadIdx.x;
    for (int b = t; b < kSelBins; b += kThreads) h[b] = 0;
    __syncthreads();
    const int64_t lo_id = (int64_t)st->sel_lo_id, hi_id = (int64_t)st->sel_hi_id;
    const u128 thr = ((u128)st->sel_hi << 64) | (u128)st->sel_lo;
    const int hi_bit = 128 - kSelBits * pass;          // digit = key bits [lo_bit, hi_bit)
    const int lo_bit = hi_bit - kSelBits > 0 ? hi_bit - kSelBits : 0;
    const unsigned dmask = (1u << (hi_bit - lo_bit)) - 1u;
    for (int64_t id = lo_id + (int64_t)blockIdx.x * kThreads + t; id < hi_id;
         id += (int64_t)gridDim.x * kThreads) {
        if (!sel_candidate(ev, st, id)) continue;
        const u128 k = sel_key(ev, st, id);
        if (pass > 0 && (k >> hi_bit) != (thr >> hi_bit)) continue;
        atomicAdd(&h[(unsigned)(k >> lo_bit) & dmask], 1u);
    }
    __syncthreads();
    uint32_t* gh = ev.hist + pass * kSelBins;
    for (int b = t; b < kSelBins; b += kThreads)
        if (h[b]) atomicAdd(&gh[b], h[b]);
    __threadfence();
    __syncthreads();
    if (t == 0) last = atomicAdd(&st->sel_done[pass], 1u) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    __threadfence();
    // last workgroup: the digit whose bin holds the need-th smallest key
    constexpr int kPer = kSelBins / kThreads;
    unsigned own = 0;
    for (int j = 0; j < kPer; ++j) {
        h[t * kPer + j] = __hip_atomic_load(&gh[t * kPer + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        own += h[t * kPer + j];
    }
    part[t] = own;
    __syncthreads();
    for (int d = 1; d < kThreads; d <<= 1) {  // inclusive scan of the per-thread sums
        const unsigned v = t >= d ? part[t - d] : 0u;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    const uint64_t need = st->sel_need;
    const uint64_t before = part[t] - own;
    if (before < need && need <= part[t]) {  // exactly one thread
        uint64_t cum = before;
        int j = 0;
        for (; j < kPer - 1; ++j) {
            if (cum + h[t * kPer + j] >= need) break;
            cum += h[t * kPer + j];
        }
        const unsigned digit = (unsigned)(t * kPer + j);
        const u128 nt = thr | ((u128)digit << lo_bit);
        st->sel_need = need - cum;
        st->sel_known = (unsigned)pass + 1;
        st->sel_bin = h[digit];
        st->sel_hi = (uint64_t)(nt >> 64);
        st->sel_lo = (uint64_t)nt;
    }
}

// The digits past those of the passes: the candidates that agree with the
// threshold so far are listed (their ids, in the array the victims come into
// later), and the last workgroup finds the rest over the list by itself. The
// list has at most kSelListMax entries unless all kSelPasses passes ran and
// left more, in keys alike in their first 44 bits.
constexpr int kFinishThreads = 1024;

__global__ __launch_bounds__(kFinishThreads) void k_sel_finish(EvictView ev, DevState* st) {
    if (st->ev_want == 0 || st->ev_all || st->sel_npass <= st->sel_known) return;  // uniform
    __shared__ uint32_t h[kSelBins];
    __shared__ uint32_t wsum[kFinishThreads / kWave], found[2];
    __shared__ int last;
    const int t = threadIdx.x, lane = t & (kWave - 1);
    const int64_t lo_id = (int64_t)st->sel_lo_id, hi_id = (int64_t)st->sel_hi_id;
    u128 thr = ((u128)st->sel_hi << 64) | (u128)st->sel_lo;
    const int known = (int)st->sel_known;
    const int open = 128 - kSelBits * known;  // key bits not yet found
    for (int64_t base = lo_id + (int64_t)blockIdx.x * kFinishThreads; base < hi_id;
         base += (int64_t)gridDim.x * kFinishThreads) {
        const int64_t id = base + t;
        const bool in = id < hi_id && sel_candidate(ev, st, id) &&
                        (sel_key(ev, st, id) >> open) == (thr >> open);
        const unsigned long long mask = ballot64(in);
        unsigned at = 0;
        if (lane == 0 && mask) at = atomicAdd(&st->sel_list, (unsigned)__popcll(mask));
        at = (unsigned)__shfl((int)at, 0, kWave);
        if (in) ev.victims[at + __popcll(mask & lanes_below(lane))] = (int32_t)id;
    }
    __threadfence();
    __syncthreads();
    if (t == 0) last = atomicAdd(&st->sel_done[kSelPasses], 1u) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    __threadfence();
    const unsigned n = __hip_atomic_load(&st->sel_list, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t need = (uint32_t)st->sel_need;
    h[2 * t] = h[2 * t + 1] = 0;
    __syncthreads();
    for (int pass = known; pass < (int)st->sel_npass; ++pass) {
        const int hi_bit = 128 - kSelBits * pass;
        const int lo_bit = hi_bit - kSelBits > 0 ? hi_bit - kSelBits : 0;
        const unsigned dmask = (1u << (hi_bit - lo_bit)) - 1u;
        for (unsigned i = t; i < n; i += kFinishThreads) {
            const int32_t id = __hip_atomic_load(&ev.victims[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const u128 k = sel_key(ev, st, id);
            if ((k >> hi_bit) == (thr >> hi_bit)) atomicAdd(&h[(unsigned)(k >> lo_bit) & dmask], 1u);
        }
        uint32_t before;
        const unsigned digit = small_digit(h, wsum, found, need, &before);
        thr |= (u128)digit << lo_bit;
        need -= before;
    }
    if (t == 0) {
        st->sel_hi = (uint64_t)(thr >> 64);
        st->sel_lo = (uint64_t)thr;
    }
}

// Marks the victims (one bit per id), takes them out of the index and raises
// the clock to their largest priority. An index to be rebuilt is cleared
// instead.
__global__ __launch_bounds__(kThreads) void k_ev_mark(EvictView ev, DevState* st, Slot* slots,
                                                      uint64_t slots_n) {
    if (st->ev_want == 0) return;
    const int lane = threadIdx.x & (kWave - 1);
    const bool all = st->ev_all != 0, rebuild = st->ev_rebuild != 0;
    const u128 thr = ((u128)st->sel_hi << 64) | (u128)st->sel_lo;
    const int64_t old = (int64_t)st->insert_old_count;
    const int64_t span = ev.words * kWave;
    const int32_t epoch = (int32_t)st->ev_epoch;
    uint64_t maxp = 0;
    for (int64_t base = (int64_t)blockIdx.x * kThreads; base < span; base += (int64_t)gridDim.x * kThreads) {
        const int64_t id = base + threadIdx.x;
        bool sel = false;
        if (id < old && ev.prot[id] != epoch) {
            sel = all || sel_key(ev, st, id) <= thr;
            if (sel) {
                const uint64_t hp = ev.prio[id];
                maxp = hp > maxp ? hp : maxp;
                drop_victim(ev, st, slots, id, rebuild);
            }
        }
        const unsigned long long mask = ballot64(sel);
        if (lane == 0 && id / kWave < ev.words) ev.wmask[id / kWave] = mask;
    }
    if (rebuild)
        for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < slots_n;
             i += (uint64_t)gridDim.x * kThreads)
            slots[i] = empty_slot();
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const uint64_t o = shfl_u64(maxp, lane ^ d);
        maxp = o > maxp ? o : maxp;
    }
    if (lane == 0 && maxp) atomicMax(&st->clock, (unsigned long long)maxp);
}

// One workgroup: lists the victims by ascending id, from the bit mask in
// tiles of 1024 x 4 words.
constexpr int kListPer = 4;

__global__ __launch_bounds__(1024) void k_ev_list(EvictView ev, DevState* st) {
    if (st->ev_want == 0) return;
    __shared__ uint32_t wsum[1024 / kWave];
    const int t = threadIdx.x, lane = t & (kWave - 1), wv = t / kWave;
    uint32_t carry = 0;
    for (int64_t base = 0; base < ev.words; base += 1024 * kListPer) {
        const int64_t w0 = base + t * kListPer;
        uint64_t m[kListPer];
        uint32_t s = 0;
#pragma unroll
        for (int k = 0; k < kListPer; ++k) {
            m[k] = w0 + k < ev.words ? ev.wmask[w0 + k] : 0ull;
            s += (uint32_t)__popcll(m[k]);
        }
        uint32_t x = s;
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, d, kWave);
            if (lane >= d) x += y;
        }
        if (lane == kWave - 1) wsum[wv] = x;
        __syncthreads();
        uint32_t at = carry + x - s;
        for (int w = 0; w < 1024 / kWave; ++w) {
            const uint32_t ws = wsum[w];
            if (w < wv) at += ws;
            carry += ws;
        }
#pragma unroll
        for (int k = 0; k < kListPer; ++k)
            for (uint64_t b = m[k]; b; b &= b - 1)
                ev.victims[at++] = (int32_t)((w0 + k) * kWave + __ffsll((long long)b) - 1);
        __syncthreads();  // wsum is written again by the next tile
    }
}

// ---------------------------------------------------------------------------
// Replication of the hot set (Section 4.1, "Replication of popular
// prefixes"): the replica slots hold the `replicas` host-tier blocks with the
// highest H. The same threshold search ranks the host tier by (H descending,
// id); blocks that left the set free their slots, blocks that entered it are
// paired, in ascending id order, with the free slots in ascending order and
// copied in.
// ---------------------------------------------------------------------------

__global__ void k_rep_setup(DevState* st, TierView tier) {
    const int t = threadIdx.x;
    if (t < kSelDone) st->sel_done[t] = 0;
    if (t != 0) return;
    st->sel_list = 0;
    st->sel_known = 0;
    st->sel_bin = 0;
    const uint64_t count = st->count;
    st->sel_hot = 1;
    st->sel_lo_id = (uint64_t)tier.owned;
    st->sel_hi_id = count > (uint64_t)tier.owned ? count : (uint64_t)tier.owned;
    st->ev_want = (uint64_t)tier.replicas;
    st->ev_all = 0;
    st->sel_range_done = 0;
    st->sel_npass = 0;
    st->sel_hi = 0;
    st->sel_lo = 0;
    st->sel_need = (uint64_t)tier.replicas;
    st->rep_new = 0;
}

// Host-tier blocks that left the hot set give up their slot; those that
// entered it get a bit in enter_mask.
__global__ __launch_bounds__(kThreads) void k_rep_diff(EvictView ev, DevState* st) {
    const TierView& t = ev.tier;
    const int lane = threadIdx.x & (kWave - 1);
    const bool all = st->ev_all != 0;
    const u128 thr = ((u128)st->sel_hi << 64) | (u128)st->sel_lo;
    const int64_t hi_id = (int64_t)st->sel_hi_id;
    const int64_t span = ((t.host_blocks + kWave - 1) / kWave) * kWave;
    unsigned long long dropped = 0;
    for (int64_t h = (int64_t)blockIdx.x * kThreads + threadIdx.x; h - threadIdx.x < span;
         h += (int64_t)gridDim.x * kThreads) {
        const int64_t id = t.owned + h;
        bool hot = false, have = false;
        if (h < t.host_blocks) {
            hot = id < hi_id && (all || sel_key(ev, st, id) <= thr);
            const int32_t slot = t.rep_of[h];
            have = slot >= 0;
            if (have && !hot) {
                t.rep_of[h] = -1;
                t.rep_id[slot] = -1;
                ++dropped;
            }
        }
        const unsigned long long mask = ballot64(hot && !have);
        if (lane == 0 && h / kWave < span / kWave) t.enter_mask[h / kWave] = mask;
    }
    dropped = wave_reduce(dropped, [](uint64_t a, uint64_t b) { return a + b; }, lane);
    if (lane == 0 && dropped) atomicSub(&st->rep_count, dropped);
}

// Exclusive scan over the block (blockDim.x = 1024) of one value per thread;
// returns this thread's offset, *total the sum.
__device__ inline uint32_t block_scan(uint32_t v, uint32_t* part, uint32_t* total) {
    const int t = threadIdx.x, nt = blockDim.x;
    part[t] = v;
    __syncthreads();
    for (int d = 1; d < nt; d <<= 1) {
        const uint32_t x = t >= d ? part[t - d] : 0u;
        __syncthreads();
        part[t] += x;
        __syncthreads();
    }
    const uint32_t incl = part[t];
    *total = part[nt - 1];
    __syncthreads();
    return incl - v;
}

// One workgroup: lists the free slots and the entering blocks in ascending
// order, pairs them and writes the copies to make.
__global__ __launch_bounds__(1024) void k_rep_assign(EvictView ev, DevState* st) {
    const TierView& t = ev.tier;
    __shared__ uint32_t part[1024];
    const int tid = threadIdx.x, nt = blockDim.x;
    uint32_t nfree = 0;
    for (int64_t base = 0; base < t.replicas; base += nt) {
        const int64_t slot = base + tid;
        const uint32_t f = slot < t.replicas && t.rep_id[slot] < 0 ? 1u : 0u;
        uint32_t tot;
        const uint32_t off = block_scan(f, part, &tot);
        if (f) t.free_list[nfree + off] = (int32_t)slot;
        nfree += tot;
    }
    const int64_t words = (t.host_blocks + kWave - 1) / kWave;
    uint32_t nenter = 0;
    for (int64_t base = 0; base < words; base += nt) {
        const int64_t w = base + tid;
        const uint64_t mask = w < words ? t.enter_mask[w] : 0ull;
        uint32_t tot;
        uint32_t off = block_scan((uint32_t)__popcll(mask), part, &tot);
        for (uint64_t m = mask; m; m &= m - 1) {  // the hot set never exceeds the slots
            const int b = __ffsll((long long)m) - 1;
            const uint32_t k = nenter + off++;
            if (k < nfree) t.enter_list[k] = (int32_t)(w * kWave + b);
        }
        nenter += tot;
    }
    if (nenter > nfree) nenter = nfree;
    __syncthreads();
    for (uint32_t k = tid; k < nenter; k += nt) {
        const int32_t h = t.enter_list[k], slot = t.free_list[k];
        t.rep_of[h] = slot;
        t.rep_id[slot] = h;
        Pair p;
        p.row = (int32_t)(t.dev_rows + h);   // host-tier home
        p.cb = (int32_t)(t.owned + slot);    // device replica row
        t.copies[k] = p;
    }
    if (tid == 0) {
        st->rep_new = nenter;
        st->rep_count += nenter;
        st->rep_copies += nenter;
    }
}

unsigned grid_for(int64_t n, int64_t cap_groups) {
    int64_t g = (n + kThreads - 1) / kThreads;
    if (g > cap_groups) g = cap_groups;
    if (g < 1) g = 1;
    return (unsigned)g;
}

}  // namespace

namespace {
// The threshold search over `n` ids at most (the range is in the state).
hipError_t launch_search(const EvictView& ev, DevState* st, int64_t n, int64_t capacity,
                         uint64_t slots_n, hipStream_t s) {
    hipError_t e;
    // about four candidates per thread: few workgroups add to the same bins
    const unsigned g = grid_for((n + 3) / 4, kSelGroups);
    hipLaunchKernelGGL(k_sel_range, dim3(g), dim3(kThreads), 0, s, ev, st, capacity, slots_n);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (int p = 0; p < kSelPasses; ++p) {
        hipLaunchKernelGGL(k_sel_pass, dim3(g), dim3(kThreads), 0, s, ev, st, p);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_sel_finish, dim3((g + 3) / 4), dim3(kFinishThreads), 0, s, ev, st);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_evict(const IndexView& ix, const InsertTarget& tgt, const EvictView& ev,
                        hipStream_t s) {
    hipError_t e = launch_search(ev, ix.state, tgt.capacity, tgt.capacity, ix.slot_mask + 1, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_ev_mark, dim3(grid_for(ev.words * kWave, 2048)), dim3(kThreads), 0, s, ev,
                       ix.state, tgt.slots, ix.slot_mask + 1);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_ev_list, dim3(1), dim3(1024), 0, s, ev, ix.state);
    return hipGetLastError();
}

hipError_t launch_replicate(const IndexView& ix, const EvictView& ev, const CopyPlan& p,
                            hipStream_t s) {
    hipError_t e;
    const TierView& t = ev.tier;
    hipLaunchKernelGGL(k_rep_setup, dim3(1), dim3(64), 0, s, ix.state, t);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = launch_search(ev, ix.state, t.host_blocks, 0, 0, s)) != hipSuccess) return e;
    const unsigned gw = grid_for(((t.host_blocks + kWave - 1) / kWave) * kWave, 2048);
    hipLaunchKernelGGL(k_rep_diff, dim3(gw), dim3(kThreads), 0, s, ev, ix.state);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_rep_assign, dim3(1), dim3(1024), 0, s, ev, ix.state);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return launch_copy_rows(p, t.copies, &ix.state->rep_new, t.replicas, s);
}

}  // namespace ptsd
