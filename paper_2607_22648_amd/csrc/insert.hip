// Deduplicating insert (PTStore Sections 1 and 4: a store keeps only the
// increment beyond the longest common prefix, so stored prefixes grow
// without redundancy like a trie; the new object appends ids for its
// increment, Section 4.1).
//
// The result equals inserting the requests one after another: a missing
// block becomes a new node whose id is the next free one in (request, block)
// order, and a block already created by an earlier request of the batch is
// reused. The GPU gets there without serialising requests or blocks:
//
//   match      match every request against the store as it was (m0, ids) and
//              write the chained keys of all its blocks (the key of block b is
//              a function of the whole prefix up to b). Each missing block
//              b >= m0 claims or joins the batch-table entry named by (key,
//              depth) and records in it the smallest request that needs it;
//              the block that claims an entry also records its depth there
//              (lookup.hip, kInsert)
//   verify     lane per block: the entry must hold the block's depth (else
//              blocks of two depths, possibly of one request, share it), and
//              the entry's smallest request o must hold the same prefix. It
//              does if block b's tokens are equal and either b is both
//              requests' first missing block under the same stored parent, or
//              both requests' blocks b-1 sit in the same entry (by induction,
//              equal prefixes). Any failure -- a collision of names between
//              different prefixes -- raises a flag. The same pass notes every
//              block's owner, the first (smallest r) request to need it, and
//              counts each request's own
//   rank       one workgroup. Only when the flag is up it first redoes the
//              claim exactly: the table is cleared and rebuilt one block after
//              another per request, each block named by (entry of its parent,
//              its tokens); slower, same result. Then the exclusive scan of
//              the counts gives every request its first rank; the store count
//              advances, clipped at capacity
//   publish    lane per block: id, created, m_out, block metadata, index slot;
//              empties the batch-table entries the batch used
//
// Ranks need no per-block pass: whoever needs a block also needs its parent,
// so the blocks a request is the first to need are its last cnt[r] ones, and
// its block b has rank start[r] + b with start[r] = (scan of the counts) -
// (its first such block). The new id is old count + rank; ids at or beyond
// capacity are refused (children rank after parents, so what is refused is
// always a suffix of a path).
//
// Ids come from a scan, never from an atomic counter, so they are
// deterministic and equal the sequential ones.
//
// What bounds a call is the number of dependent launches, about 4.6 us each
// for batches of up to a few hundred requests, not the work in them. Hence
// four kernels (without eviction, or with a small store's, all of whose
// eviction runs inside rank), where lookup, key hashing, two table clears,
// claim, exact claim, verify, count, scan, assign, publish and touch had
// been launches of their own; each wave has one 64-block window of one
// request, so that a request of many windows is not walked by one wave. The
// claim can run inside the match because the batch table is empty whenever
// an insert begins: publish leaves it so.
//
// With eviction on, verify also marks the blocks the batch matched
// (protected), rank computes how many blocks must be evicted and frees them
// (a small store; a larger one in the kernels of evict.hip between rank and
// publish), publish hands out never-used ids and then the freed ones, may
// take a deleted index slot, and accesses the resident paths.
#include "kernels.hpp"
#include "evict_small.hpp"

namespace ptsd {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr uint32_t kStoreLabel = 0x80000000u;  // parent label of a stored block: bit 31 | (id + 1)

// A block's tokens move four at a time where the block size allows it
// (stored rows then start on 16 bytes), sixteen in flight: a token per step,
// each waiting for the one before, had been half of publish.
__device__ inline bool same_tokens(const int32_t* __restrict__ a, const int32_t* __restrict__ b, int bt) {
    if ((bt & 3) == 0) {
        bool eq = true;
        for (int i = 0; i < bt / 4; i += 4) {
            int4 u[4], w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {  // past the end: the last piece again
                u[j] = load_tokens4(a + 4 * min(i + j, bt / 4 - 1));
                w[j] = load_tokens4(b + 4 * min(i + j, bt / 4 - 1));
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                eq &= (u[j].x == w[j].x) & (u[j].y == w[j].y) & (u[j].z == w[j].z) & (u[j].w == w[j].w);
        }
        return eq;
    }
    for (int i = 0; i < bt; ++i)
        if (a[i] != b[i]) return false;
    return true;
}

// dst: a stored row
__device__ inline void copy_tokens(int32_t* __restrict__ dst, const int32_t* __restrict__ src, int bt) {
    if ((bt & 3) == 0) {
        for (int i = 0; i < bt / 4; i += 4) {
            int4 u[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) u[j] = load_tokens4(src + 4 * min(i + j, bt / 4 - 1));
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (i + j < bt / 4) reinterpret_cast<int4*>(dst)[i + j] = u[j];
        }
        return;
    }
    for (int i = 0; i < bt; ++i) dst[i] = src[i];
}

struct InsertArgs {
    IndexView ix;
    InsertTarget tgt;
    EvictView ev;
    Batch bat;
    InsertScratch sc;
    int32_t* m_out;
    int32_t* ids;
    uint8_t* created;
};

__device__ inline void count_cas(const InsertArgs& a, unsigned long long cas,
                                 unsigned long long fails, int lane) {
    if (!a.ix.counters) return;
    CounterSlot* cs = counter_slot(a.ix.state);
    wave_count(&cs->cas_attempts, cas, lane);
    wave_count(&cs->cas_failures, fails, lane);
}

// Windows of 64 blocks a request has room for.
__host__ __device__ inline int64_t windows(int32_t max_blocks) { return (max_blocks + kWave - 1) / kWave; }

// One wave per (request, window).
struct WaveOf {
    int64_t r;
    int32_t b, w;  // this lane's block, the window
    int lane;
    bool any;      // the request exists
};
__device__ inline WaveOf wave_of(const Batch& bat) {
    WaveOf v;
    v.lane = threadIdx.x & (kWave - 1);
    const int64_t nw = windows(bat.max_blocks);
    const int64_t i = (int64_t)blockIdx.x * kWaves + threadIdx.x / kWave;
    v.r = i / nw;
    v.w = (int32_t)(i - v.r * nw);
    v.b = v.w * kWave + v.lane;
    v.any = v.r < bat.R;
    return v;
}

__global__ __launch_bounds__(kThreads) void k_verify(InsertArgs a) {
    const WaveOf v = wave_of(a.bat);
    if (!v.any) return;
    const int bt = a.ix.block_tokens;
    const int64_t maxb = a.bat.max_blocks, r = v.r;
    const int32_t b = v.b, m0 = a.sc.m0[r], n = a.sc.nblk[r];
    if (a.ev.on && b < m0)  // a block this request matched: not evicted by this insert
        a.ev.prot[a.ids[r * maxb + b]] = (int32_t)a.ix.state->ev_epoch;
    if (v.w * kWave + kWave <= m0 || v.w * kWave >= n) return;  // no new block in the window
    const BatchEntry* __restrict__ tab = a.sc.table;
    bool ok = true, own = false;
    if (b >= m0 && b < n) {
        const int32_t label = a.sc.label[r * maxb + b];
        const BatchEntry te = tab[label];
        const int64_t o = te.owner;
        own = o == r;
        a.sc.owner[r * maxb + b] = te.owner;  // for publish, which empties the table
        ok = te.depth == b;  // else the entry was claimed at another depth
        if (ok && !own) {
            const int32_t om0 = a.sc.m0[o];
            ok = b < a.sc.nblk[o] && b >= om0 &&
                 same_tokens(a.bat.tokens + a.bat.offsets[o] + (int64_t)b * bt,
                             a.bat.tokens + a.bat.offsets[r] + (int64_t)b * bt, bt);
            if (ok) {
                if (b == m0)
                    ok = om0 == b && (b == 0 || a.ids[o * maxb + b - 1] == a.ids[r * maxb + b - 1]);
                else
                    ok = om0 <= b - 1 && a.sc.label[o * maxb + b - 1] == a.sc.label[r * maxb + b - 1];
            }
        }
    }
    if (!ok) *a.sc.collision = 1;
    const int c = __popcll(ballot64(own));
    if (v.lane == 0 && c) atomicAdd(&a.sc.cnt[r], c);
}

__device__ inline BatchEntry empty_entry() {
    BatchEntry e;
    e.word = kEmptyKey;
    e.owner = kNoOwner;
    e.depth = -1;
    return e;
}

// The exact claim, by one workgroup: one block after another per request
// (runs only on a collision). Labels, owners and counts are made anew. The
// entries and counts are changed by device-scope atomics, so what an earlier
// plain read left in the compute unit's cache is dropped between the steps.
__device__ inline void claim_exact(const InsertArgs& a) {
    const int t = threadIdx.x, nt = blockDim.x;
    const int bt = a.ix.block_tokens;
    const int64_t maxb = a.bat.max_blocks;
    BatchEntry* __restrict__ tab = a.sc.table;
    const HashTables* __restrict__ ht = a.ix.ht;
    if (t == 0) atomicAdd(&a.ix.state->insert_fallbacks, 1ull);
    for (uint64_t i = t; i <= a.sc.table_mask; i += nt) tab[i] = empty_entry();
    for (int64_t r = t; r < a.bat.R; r += nt) a.sc.cnt[r] = 0;
    __threadfence();
    __syncthreads();
    for (int64_t r = t; r < a.bat.R; r += nt) {
        const int32_t n = a.sc.nblk[r], m0 = a.sc.m0[r];
        const int64_t o0 = a.bat.offsets[r];
        uint32_t plabel = m0 == 0 ? kStoreLabel : (kStoreLabel | (uint32_t)(a.ids[r * maxb + m0 - 1] + 1));
        for (int32_t b = m0; b < n; ++b) {
            const uint64_t ik = index_key(a.sc.keys[r * maxb + b], *ht);
            const uint32_t tpos = (uint32_t)(o0 + (int64_t)b * bt);
            const unsigned long long word = ((unsigned long long)plabel << 32) | tpos;
            uint64_t pos = slot_of(ik, ~ht->slot_seed, a.sc.table_mask);
            while (true) {
                const unsigned long long prev = atomicCAS(&tab[pos].word, kEmptyKey, word);
                if (prev == kEmptyKey) break;
                if ((uint32_t)(prev >> 32) == plabel &&
                    same_tokens(a.bat.tokens + (uint32_t)prev, a.bat.tokens + tpos, bt))
                    break;
                pos = (pos + 1) & a.sc.table_mask;
            }
            atomicMin(&tab[pos].owner, (int32_t)r);
            a.sc.label[r * maxb + b] = (int32_t)pos;
            plabel = (uint32_t)pos;
        }
    }
    __threadfence();
    __syncthreads();
    for (int64_t r = t; r < a.bat.R; r += nt) {
        int32_t c = 0;
        for (int32_t b = a.sc.m0[r]; b < a.sc.nblk[r]; ++b) {
            const int32_t o = __hip_atomic_load(&tab[a.sc.label[r * maxb + b]].owner, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
            a.sc.owner[r * maxb + b] = o;
            c += o == (int32_t)r;
        }
        a.sc.cnt[r] = c;
    }
    __threadfence();
    __syncthreads();
}

// One workgroup: every request's start rank and the store count. The
// requests go in tiles of 1024 x 4, four neighbouring counts per thread, as
// in the copies' list; a batch has at most 2^29 blocks, so every sum fits in
// 32 bits. A small store's eviction follows in the same workgroup.
constexpr int kRankThreads = 1024;
constexpr int kRankPer = 4;

template <bool EVICT_SMALL>
__global__ __launch_bounds__(kRankThreads) void k_rank(InsertArgs a) {
    __shared__ uint32_t wsum[kRankThreads / kWave];
    DevState* st = a.ix.state;
    const int R = a.bat.R;
    const int t = threadIdx.x, lane = t & (kWave - 1), wv = t / kWave;
    // every load that does not wait for another goes out together: the flag,
    // the state, the first tile's counts and a small store's blocks
    const unsigned int collision = *a.sc.collision;
    const long long old = (long long)st->count;
    const int32_t epoch = EVICT_SMALL ? (int32_t)st->ev_epoch : 0;
    const unsigned long long tombstones = EVICT_SMALL ? st->tombstones : 0ull;
    uint32_t v[kRankPer], n[kRankPer];
    auto load_counts = [&](int i0) {
#pragma unroll
        for (int k = 0; k < kRankPer; ++k) {
            v[k] = i0 + k < R ? (uint32_t)a.sc.cnt[i0 + k] : 0u;
            n[k] = i0 + k < R ? (uint32_t)a.sc.nblk[i0 + k] : 0u;
        }
    };
    load_counts(t * kRankPer);
    SmallBlocks blocks;
    if (EVICT_SMALL) load_blocks(a.ev, a.tgt.capacity, &blocks);
    if (collision) {  // uniform
        claim_exact(a);
        load_counts(t * kRankPer);
    }
    uint32_t carry = 0;
    for (int base = 0; base < R; base += kRankThreads * kRankPer) {
        const int i0 = base + t * kRankPer;
        if (base) load_counts(i0);
        uint32_t s = 0;
#pragma unroll
        for (int k = 0; k < kRankPer; ++k) s += v[k];
        const uint32_t x = wave_scan_add(s);
        if (lane == kWave - 1) wsum[wv] = x;
        __syncthreads();
        uint32_t total;
        uint32_t run = carry + waves_before(wsum, wv, &total) + x - s;
        carry += total;
#pragma unroll
        for (int k = 0; k < kRankPer; ++k) {
            if (i0 + k < R) a.sc.start[i0 + k] = (int32_t)(run - (n[k] - v[k]));
            run += v[k];
        }
        __syncthreads();  // wsum is written again by the next tile
    }
    const long long total = carry;
    const long long cap = a.tgt.capacity;
    const long long want = total - (cap - old);  // ids the batch needs beyond the never-used ones
    __syncthreads();                             // every wave has read the count
    if (t == 0) {
        st->insert_old_count = (unsigned long long)old;
        st->insert_full = 0;
        if (want > 0 && !a.ev.on) {  // with eviction: decided once victims are known
            st->full_events += 1;
            st->insert_full = 1;
        }
        st->count = (unsigned long long)(want > 0 ? cap : old + total);
        if (a.ev.on) {
            st->ev_new = (unsigned long long)total;
            st->ev_want = want > 0 ? (unsigned long long)want : 0ull;
            st->ev_all = 0;
            st->ev_nv = 0;
            st->ev_rebuild = 0;
            st->sel_range_done = 0;
            st->sel_list = 0;
            st->sel_known = 0;
            st->sel_bin = 0;
            for (int k = 0; k < kSelDone; ++k) st->sel_done[k] = 0;
            st->sel_npass = 0;
            st->sel_hot = 0;
            st->sel_lo_id = 0;
            st->sel_hi_id = (unsigned long long)old;
            st->sel_hi = 0;
            st->sel_lo = 0;
            st->sel_need = st->ev_want;
        }
    }
    if (!EVICT_SMALL || want <= 0) return;  // uniform
    __syncthreads();  // the state above is read below
    evict_small(a.ev, st, a.tgt.slots, a.ix.slot_mask + 1, a.tgt.capacity, old, want, epoch,
                tombstones, blocks);
}

// Re-enters into the index, cleared by the eviction, every block that
// survived it; the batch's new blocks are entered at the same time (each by
// its own compare-and-swap on an empty slot, in any order).
__device__ inline void reenter_survivors(const InsertArgs& a) {
    const int64_t old = (int64_t)a.ix.state->insert_old_count;
    for (int64_t id = (int64_t)blockIdx.x * kThreads + threadIdx.x; id < old;
         id += (int64_t)gridDim.x * kThreads) {
        if ((a.ev.wmask[id / kWave] >> (id & (kWave - 1))) & 1ull) continue;  // evicted
        const uint64_t ik = a.ev.nkey[id];
        uint64_t pos = slot_of(ik, a.ix.ht->slot_seed, a.ix.slot_mask);
        // at most half the slots hold blocks, so an empty one is always found
        for (uint64_t step = 0; step <= a.ix.slot_mask; ++step) {
            const unsigned long long prev =
                atomicCAS(reinterpret_cast<unsigned long long*>(&a.tgt.slots[pos].key), kEmptyKey,
                          (unsigned long long)ik);
            if (prev == kEmptyKey) {
                a.tgt.slots[pos].id = (int32_t)id;
                a.tgt.slots[pos].parent = a.tgt.parent[id];
                a.ev.spos[id] = (uint32_t)pos;
                break;
            }
            pos = (pos + 1) & a.ix.slot_mask;
        }
    }
}

// The id of a new block at depth b that `owner` is the first to need: -1 if
// it is refused.
__device__ inline int32_t new_id(const InsertArgs& a, int32_t owner, int32_t b, long long old,
                                 long long fresh, long long nv) {
    const long long k = (long long)a.sc.start[owner] + b;  // rank among the batch's new blocks
    if (k < fresh) return (int32_t)(old + k);
    return k - fresh < nv ? a.ev.victims[k - fresh] : -1;
}

__global__ __launch_bounds__(kThreads) void k_publish(InsertArgs a) {
    const WaveOf v = wave_of(a.bat);
    if (a.ev.on && a.ix.state->ev_rebuild) reenter_survivors(a);
    if (!v.any) return;
    const int bt = a.ix.block_tokens;
    const int64_t maxb = a.bat.max_blocks, r = v.r;
    const int32_t b = v.b, m0 = a.sc.m0[r], n = a.sc.nblk[r];
    const HashTables* __restrict__ ht = a.ix.ht;
    int32_t* __restrict__ row = a.ids + r * maxb;
    uint8_t* __restrict__ crow = a.created + r * maxb;
    if (b < maxb && (b < m0 || b >= n)) crow[b] = 0;
    if (m0 == n && b == 0) a.m_out[r] = n;
    const uint64_t clock = a.ev.on ? a.ix.state->clock : 0;
    const long long old = (long long)a.ix.state->insert_old_count;
    const long long fresh = a.tgt.capacity - old;                     // never-used ids
    const long long nv = a.ev.on ? (long long)a.ix.state->ev_nv : 0;  // freed ids
    unsigned long long cas = 0, fails = 0, tombs_taken = 0;
    const bool is_new = b >= m0 && b < n;
    int32_t id = -1, owner = -1;
    if (is_new) {
        owner = a.sc.owner[r * maxb + b];
        a.sc.table[a.sc.label[r * maxb + b]] = empty_entry();  // nothing reads it any more
        id = new_id(a, owner, b, old, fresh, nv);
    } else if (a.ev.on && b < m0) id = row[b];
    int32_t parent = __shfl_up(id, 1, kWave);
    if (is_new) {
        if (b == m0)
            parent = m0 == 0 ? -1 : row[m0 - 1];
        else if (v.lane == 0)
            parent = new_id(a, a.sc.owner[r * maxb + b - 1], b - 1, old, fresh, nv);
        // refusals are a suffix of the request: one lane holds the cut
        if (id < 0 && (b == m0 || parent >= 0)) a.m_out[r] = b;
        if (id >= 0 && b == n - 1) a.m_out[r] = n;
        const bool mine = id >= 0 && owner == (int32_t)r;
        row[b] = id;
        crow[b] = mine ? 1 : 0;
        if (mine) {
            a.tgt.parent[id] = parent;
            copy_tokens(a.tgt.tokens + (int64_t)id * bt, a.bat.tokens + a.bat.offsets[r] + (int64_t)b * bt, bt);
            const uint64_t ik = index_key(a.sc.keys[r * maxb + b], *ht);
            uint64_t pos = slot_of(ik, ht->slot_seed, a.ix.slot_mask);
            Slot* slots = a.tgt.slots;
            // at most half the slots hold blocks and at most a quarter are
            // deleted, so a free slot is always found
            for (uint64_t step = 0; step <= a.ix.slot_mask; ++step) {
                unsigned long long* kp = reinterpret_cast<unsigned long long*>(&slots[pos].key);
                unsigned long long prev = atomicCAS(kp, kEmptyKey, (unsigned long long)ik);
                ++cas;
                bool got = prev == kEmptyKey;
                if (!got && a.ev.on && prev == kTombKey) {
                    prev = atomicCAS(kp, kTombKey, (unsigned long long)ik);
                    ++cas;
                    got = prev == kTombKey;
                    tombs_taken += got ? 1 : 0;
                }
                if (got) {
                    slots[pos].id = id;
                    slots[pos].parent = parent;
                    break;
                }
                ++fails;
                pos = (pos + 1) & a.ix.slot_mask;
            }
            if (a.ev.on) {
                a.ev.depth[id] = b;
                a.ev.prot[id] = 0;
                a.ev.nkey[id] = ik;
                a.ev.spos[id] = (uint32_t)pos;
            }
        }
    }
    // every block of the resident path counts one access (an id that held no
    // block had F = H = 0)
    if (a.ev.on && id >= 0) {
        const uint64_t f = atomicAdd((unsigned long long*)&a.ev.freq[id], 1ull) + 1ull;
        atomicMax((unsigned long long*)&a.ev.prio[id], (unsigned long long)(clock + f));
    }
    count_cas(a, cas, fails, v.lane);
    if (a.ev.on) wave_sub(&a.ix.state->tombstones, tombs_taken, v.lane);
}

}  // namespace

namespace {
size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

__global__ void k_empty_batch(BatchEntry* t, uint64_t n) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        t[i] = empty_entry();
}
}  // namespace

uint64_t insert_table_entries(int32_t R, int32_t max_blocks) {
    const uint64_t rb = (uint64_t)R * (uint64_t)max_blocks;
    uint64_t t = 64;
    while (t < 2 * rb) t <<= 1;
    return t;
}

size_t insert_scratch_bytes(int32_t R, int32_t max_blocks, uint64_t table_cap) {
    const size_t rb = (size_t)R * (size_t)max_blocks;
    return up256(table_cap * sizeof(BatchEntry)) + up256(rb * 8) + 2 * up256(rb * 4) +
           4 * up256((size_t)R * 4) + 256;
}

void insert_scratch_carve(void* base, int32_t R, int32_t max_blocks, uint64_t table_cap,
                          InsertScratch* out) {
    const size_t rb = (size_t)R * (size_t)max_blocks;
    uint8_t* p = static_cast<uint8_t*>(base);
    auto take = [&](size_t bytes) {
        uint8_t* q = p;
        p += up256(bytes);
        return q;
    };
    out->table = reinterpret_cast<BatchEntry*>(take(table_cap * sizeof(BatchEntry)));
    out->table_mask = insert_table_entries(R, max_blocks) - 1;
    out->keys = reinterpret_cast<uint64_t*>(take(rb * 8));
    out->label = reinterpret_cast<int32_t*>(take(rb * 4));
    out->owner = reinterpret_cast<int32_t*>(take(rb * 4));
    out->m0 = reinterpret_cast<int32_t*>(take((size_t)R * 4));
    out->nblk = reinterpret_cast<int32_t*>(take((size_t)R * 4));
    out->cnt = reinterpret_cast<int32_t*>(take((size_t)R * 4));
    out->start = reinterpret_cast<int32_t*>(take((size_t)R * 4));
    out->collision = reinterpret_cast<unsigned int*>(p);
}

hipError_t launch_empty_batch(void* table, uint64_t entries, hipStream_t s) {
    uint64_t g = (entries + 255) / 256;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_empty_batch, dim3((unsigned)g), dim3(256), 0, s, static_cast<BatchEntry*>(table),
                       entries);
    return hipGetLastError();
}

namespace {
// Workgroups of a kernel with one wave per (request, window).
unsigned window_grid(const Batch& b) {
    return (unsigned)(((int64_t)b.R * windows(b.max_blocks) + kWaves - 1) / kWaves);
}
}  // namespace

hipError_t launch_insert_match(const IndexView& ix, const InsertTarget& tgt, const EvictView& ev,
                               const Batch& b, const InsertScratch& sc, int32_t* m_out, int32_t* ids,
                               uint8_t* created, hipStream_t s) {
    hipError_t e;
    IndexView quiet = ix;  // the insert's own match is not an access
    quiet.freq = nullptr;
    quiet.prio = nullptr;
    const InsertMatch im{sc.keys, sc.label, sc.nblk, sc.cnt, sc.table, sc.table_mask, sc.collision, ev.on};
    if ((e = launch_match(quiet, b, sc.m0, ids, im, s)) != hipSuccess) return e;
    InsertArgs a{quiet, tgt, ev, b, sc, m_out, ids, created};
    const unsigned wgrid = window_grid(b);
    hipLaunchKernelGGL(k_verify, dim3(wgrid), dim3(kThreads), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (ev.on && evicts_in_rank(tgt.capacity, ix.slot_mask + 1))
        hipLaunchKernelGGL(k_rank<true>, dim3(1), dim3(kRankThreads), 0, s, a);
    else
        hipLaunchKernelGGL(k_rank<false>, dim3(1), dim3(kRankThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_insert_commit(const IndexView& ix, const InsertTarget& tgt, const EvictView& ev,
                                const Batch& b, const InsertScratch& sc, int32_t* m_out, int32_t* ids,
                                uint8_t* created, hipStream_t s) {
    IndexView quiet = ix;
    quiet.freq = nullptr;
    quiet.prio = nullptr;
    InsertArgs a{quiet, tgt, ev, b, sc, m_out, ids, created};
    // a rebuild of the index enters every surviving block, however small the
    // batch: about four a thread, on at most as many workgroups as a selection
    // (an insert of one request that rebuilds 131,072 blocks: 137 us; on the
    // batch's one workgroup 2,160, without a rebuild 114)
    unsigned g = window_grid(b);
    if (ev.on) {
        const int64_t whole = (tgt.capacity + 4 * kThreads - 1) / (4 * kThreads);
        const unsigned most = (unsigned)(whole < kSelGroups ? whole : kSelGroups);
        if (g < most) g = most;
    }
    hipLaunchKernelGGL(k_publish, dim3(g), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace ptsd
