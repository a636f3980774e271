// Eviction of a small store, inside the insert's rank kernel (insert.hip),
// and what it shares with the kernels of a larger one (evict.hip, which
// states the order of the victims and why a selection by rank is the
// one-at-a-time walk).
#pragma once

#include "kernels.hpp"

namespace ptsd {

__device__ inline unsigned bit_width(uint64_t x) { return x ? 64u - (unsigned)__clzll((long long)x) : 0u; }

// A victim leaves the index (unless it is being cleared anyway) and the
// replica map; its access counts start again from zero for the id's next
// block.
__device__ inline void drop_victim(const EvictView& ev, DevState* st, Slot* slots, int64_t id,
                                   bool rebuild) {
    if (!rebuild) slots[ev.spos[id]].key = kTombKey;
    ev.freq[id] = 0;
    ev.prio[id] = 0;
    if (ev.tier.rep_of && id >= ev.tier.owned) {  // its replica goes too
        const int64_t h = id - ev.tier.owned;
        const int32_t slot = ev.tier.rep_of[h];
        if (slot >= 0) {
            ev.tier.rep_of[h] = -1;
            ev.tier.rep_id[slot] = -1;
            atomicSub(&st->rep_count, 1ull);
        }
    }
}

// Does an eviction of nv blocks leave deleted slots in more than a quarter of
// the index? Then it is rebuilt.
__device__ inline bool rebuilds(unsigned long long tombstones, unsigned long long nv, uint64_t slots_n) {
    return (tombstones + nv) * 4 > slots_n;
}

// What an eviction of nv blocks does to the store's counters (one thread).
__device__ inline void evict_account(DevState* st, int64_t capacity, uint64_t slots_n,
                                     unsigned long long nv) {
    const unsigned long long fresh = (unsigned long long)capacity - st->insert_old_count;
    const bool rebuild = rebuilds(st->tombstones, nv, slots_n);
    st->ev_nv = nv;
    st->evictions += nv;
    if (st->ev_new > fresh + nv) {
        st->full_events += 1;
        st->insert_full = 1;
    }
    st->rebuilds += rebuild ? 1 : 0;
    st->tombstones = rebuild ? 0ull : st->tombstones + nv;
    st->ev_rebuild = rebuild ? 1 : 0;
}

__device__ inline Slot empty_slot() {
    Slot z;
    z.key = kEmptyKey;
    z.id = -1;
    z.parent = -1;
    return z;
}

// A store of at most kSmallEvictMax blocks evicts in one workgroup of 1024
// threads, 16 blocks each, their priorities and depths in registers: one
// pass over memory and a few LDS digit passes of about 1 us, where the
// kernels for larger stores cost a launch each. An insert of 128 chat turns
// and its scatter into a full store takes 55 us with 5,120 blocks and 63 with
// 16,336; by the kernels of evict.hip 99 and 98. Past 16 blocks a thread the
// registers run out, and one compute unit's bandwidth (about 0.1 TB/s) starts
// to show. It shows in the index too, which a rebuild clears: with 16,000
// blocks an insert of 14,400 takes 78 us here, 95 when it rebuilds an index of
// 2^18 slots, 177 with 2^20 and 506 with 2^22; by the kernels of evict.hip 92
// and 92 to 104. So a store that was given more than 2^18 slots (eight times
// what 16,384 blocks get by default) takes those.
constexpr int kSmallEvictPer = 16;
constexpr int kSmallEvictThreads = 1024;
static_assert(kSmallEvictMax == (int64_t)kSmallEvictPer * kSmallEvictThreads, "blocks of the workgroup");

// The digit of a 2048-bin histogram whose bin holds the need-th smallest key
// (need >= 1, at most the keys counted); *before: keys in smaller bins. All
// 1024 threads call it; the histogram is zero again afterwards.
__device__ inline unsigned small_digit(uint32_t* h, uint32_t* wsum, uint32_t* found, uint32_t need,
                                       uint32_t* before) {
    const int t = threadIdx.x, lane = t & (kWave - 1), wv = t / kWave;
    __syncthreads();
    const uint32_t c0 = h[2 * t], c1 = h[2 * t + 1];
    h[2 * t] = h[2 * t + 1] = 0;
    const uint32_t x = wave_scan_add(c0 + c1);
    if (lane == kWave - 1) wsum[wv] = x;
    __syncthreads();
    uint32_t total;
    const uint32_t below = waves_before(wsum, wv, &total) + x - c0 - c1;
    if (below < need && need <= below + c0 + c1) {  // exactly one thread
        const bool second = below + c0 < need;
        found[0] = 2u * (unsigned)t + (second ? 1u : 0u);
        found[1] = below + (second ? c0 : 0u);
    }
    __syncthreads();
    *before = found[1];
    return found[0];
}

// The blocks of a small store, kSmallEvictPer a thread: block k * 1024 + t.
struct SmallBlocks {
    uint64_t p[kSmallEvictPer];  // priority H
    uint32_t d[kSmallEvictPer];  // depth
    int32_t pr[kSmallEvictPer];  // protection mark
};

// Issued before the rank kernel's scan, so that the two wait together. The
// tests of k here and below are uniform: a store of 5,000 blocks runs 5 of
// the 16 steps.
__device__ inline void load_blocks(const EvictView& ev, int64_t capacity, SmallBlocks* x) {
    const int t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < kSmallEvictPer; ++k) {
        x->p[k] = 0;
        x->d[k] = 0;
        x->pr[k] = 0;
        if (k * kSmallEvictThreads >= capacity) continue;
        const int64_t id = min((int64_t)(k * kSmallEvictThreads + t), capacity - 1);
        x->p[k] = ev.prio[id];
        x->d[k] = (uint32_t)ev.depth[id];
        x->pr[k] = ev.prot[id];
    }
}

// Evicts for a batch that needs `want` > 0 ids beyond the never-used ones
// (`old` blocks stored before it): the victims' list, bit mask, counters and
// clock as the larger stores' kernels leave them. The digits run over the
// bits in which candidates differ at all (the OR and AND of their keys).
__device__ inline void evict_small(const EvictView& ev, DevState* st, Slot* slots, uint64_t slots_n,
                                   int64_t capacity, long long old, long long want, int32_t epoch,
                                   unsigned long long tombstones, SmallBlocks& x) {
    constexpr int E = kSmallEvictPer, NT = kSmallEvictThreads, NW = NT / kWave;
    static_assert(kSelBins == 2 * NT, "two histogram bins per thread");
    static_assert(NW == 16, "per-wave values are combined in rows of 16 lanes");
    __shared__ uint32_t hist[kSelBins];
    __shared__ uint32_t wsum[NW], found[2], cnt[E * NW], tcnt[E * NW];
    __shared__ uint32_t red[8][NW];
    __shared__ uint16_t list[kSmallEvictMax];
    const int t = threadIdx.x, lane = t & (kWave - 1), wv = t / kWave;
    uint64_t(&p)[E] = x.p;
    uint32_t(&d)[E] = x.d;
    hist[2 * t] = hist[2 * t + 1] = 0;
    uint32_t cand = 0;  // bit k: block k * NT + t may be evicted
    uint64_t por = 0, pand = ~0ull;
    uint32_t dor = 0, dand = ~0u;
#pragma unroll
    for (int k = 0; k < E; ++k) {
        if (k * NT >= old) continue;
        d[k] = ~d[k];  // deeper is smaller
        if (k * NT + t < old && x.pr[k] != epoch) {
            cand |= 1u << k;
            por |= p[k];
            pand &= p[k];
            dor |= d[k];
            dand &= d[k];
        }
    }
    auto op_or = [](uint32_t a, uint32_t b) { return a | b; };
    auto op_and = [](uint32_t a, uint32_t b) { return a & b; };
    auto op_add = [](uint32_t a, uint32_t b) { return a + b; };
    {
        const uint32_t v0 = wave_scan((uint32_t)por, 0u, op_or);
        const uint32_t v1 = wave_scan((uint32_t)(por >> 32), 0u, op_or);
        const uint32_t v2 = wave_scan(dor, 0u, op_or);
        const uint32_t v3 = wave_scan((uint32_t)pand, ~0u, op_and);
        const uint32_t v4 = wave_scan((uint32_t)(pand >> 32), ~0u, op_and);
        const uint32_t v5 = wave_scan(dand, ~0u, op_and);
        const uint32_t v6 = wave_scan_add((uint32_t)__popc(cand));
        if (lane == kWave - 1) {
            red[0][wv] = v0;
            red[1][wv] = v1;
            red[2][wv] = v2;
            red[3][wv] = v3;
            red[4][wv] = v4;
            red[5][wv] = v5;
            red[6][wv] = v6;
        }
    }
    __syncthreads();
    const int l = lane & 15;
    const uint32_t por0 = read_lane(row_scan(red[0][l], 0u, op_or), 15);
    const uint32_t por1 = read_lane(row_scan(red[1][l], 0u, op_or), 15);
    dor = read_lane(row_scan(red[2][l], 0u, op_or), 15);
    const uint32_t pand0 = read_lane(row_scan(red[3][l], ~0u, op_and), 15);
    const uint32_t pand1 = read_lane(row_scan(red[4][l], ~0u, op_and), 15);
    dand = read_lane(row_scan(red[5][l], ~0u, op_and), 15);
    const uint32_t nc = read_lane(row_scan(red[6][l], 0u, op_add), 15);
    por = (uint64_t)por1 << 32 | por0;
    pand = (uint64_t)pand1 << 32 | pand0;
    const bool all = (long long)nc <= want;
    const unsigned long long nv = all ? nc : (unsigned long long)want;
    const bool rebuild = rebuilds(tombstones, nv, slots_n);
    // Threshold of the want smallest (H, deeper first, id): digits of H, then
    // of the depth among the blocks of exactly that H; of the blocks that tie
    // in both, the first ones by id go.
    uint32_t need = (uint32_t)want;
    uint64_t t1 = all ? ~0ull : 0;
    uint32_t t2 = all ? ~0u : 0;
    if (!all) {
        int hi = (int)bit_width(por ^ pand);
        t1 = hi >= 64 ? 0ull : pand >> hi << hi;  // the bits all candidates share
        while (hi > 0) {
            const int lo = hi > kSelBits ? hi - kSelBits : 0;
            const unsigned dm = (1u << (hi - lo)) - 1u;
#pragma unroll
            for (int k = 0; k < E; ++k)
                if (k * NT < old && ((cand >> k) & 1u) && (hi >= 64 || (p[k] >> hi) == (t1 >> hi)))
                    atomicAdd(&hist[(unsigned)(p[k] >> lo) & dm], 1u);
            uint32_t before;
            t1 |= (uint64_t)small_digit(hist, wsum, found, need, &before) << lo;
            need -= before;
            hi = lo;
        }
        hi = (int)bit_width(dor ^ dand);
        t2 = hi >= 32 ? 0u : dand >> hi << hi;
        while (hi > 0) {
            const int lo = hi > kSelBits ? hi - kSelBits : 0;
            const unsigned dm = (1u << (hi - lo)) - 1u;
#pragma unroll
            for (int k = 0; k < E; ++k)
                if (k * NT < old && ((cand >> k) & 1u) && p[k] == t1 &&
                    (hi >= 32 || (d[k] >> hi) == (t2 >> hi)))
                    atomicAdd(&hist[(d[k] >> lo) & dm], 1u);
            uint32_t before;
            t2 |= small_digit(hist, wsum, found, need, &before) << lo;
            need -= before;
            hi = lo;
        }
    }
    // the victims: per 64 blocks how many go for certain and how many tie
    uint32_t sure = 0, tie = 0;
    uint64_t maxp = 0;
#pragma unroll
    for (int k = 0; k < E; ++k) {
        if (k * NT >= old) {
            if (lane == 0) cnt[k * NW + wv] = tcnt[k * NW + wv] = 0;
            continue;
        }
        const bool c = (cand >> k) & 1u;
        const bool eq = c && !all && p[k] == t1 && d[k] == t2;
        const bool lt = c && (all || p[k] < t1 || (p[k] == t1 && d[k] < t2));
        sure |= lt ? 1u << k : 0u;
        tie |= eq ? 1u << k : 0u;
        if (all && c && p[k] > maxp) maxp = p[k];
        const uint32_t ns = (uint32_t)__popcll(ballot64(lt));
        const uint32_t nt = (uint32_t)__popcll(ballot64(eq));
        if (lane == 0) {
            cnt[k * NW + wv] = ns;
            tcnt[k * NW + wv] = nt;
        }
    }
    // the largest H that goes: the threshold's, or, of all, the largest
    if (!all)
        maxp = t == 0 ? t1 : 0ull;
    if (maxp) atomicMax(&st->clock, (unsigned long long)maxp);
    __syncthreads();
    if (wv == 0) {  // exclusive scans, four counts a lane: of the ties, then of all that go
        static_assert(E * NW == 4 * kWave, "four counts per lane");
        uint32_t c[4], tc[4], s = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            tc[j] = tcnt[4 * lane + j];
            c[j] = cnt[4 * lane + j];
            s += tc[j];
        }
        uint32_t run = wave_scan_add(s) - s;
        s = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {  // ties that go: the first `need` of them
            const uint32_t take = run >= need ? 0u : (need - run < tc[j] ? need - run : tc[j]);
            run += tc[j];
            tcnt[4 * lane + j] = take;
            c[j] += take;
            s += c[j];
        }
        run = wave_scan_add(s) - s;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            cnt[4 * lane + j] = run;
            run += c[j];
        }
    }
    __syncthreads();
    const unsigned long long below = lane == 0 ? 0ull : ~0ull >> (64 - lane);
#pragma unroll
    for (int k = 0; k < E; ++k) {
        if (k * NT >= old) continue;
        const unsigned long long ties = ballot64((tie >> k) & 1u);
        const bool go = ((sure >> k) & 1u) ||
                        (((tie >> k) & 1u) && (uint32_t)__popcll(ties & below) < tcnt[k * NW + wv]);
        const unsigned long long mask = ballot64(go);
        if (lane == 0 && k * NW + wv < ev.words) ev.wmask[k * NW + wv] = mask;
        if (go) list[cnt[k * NW + wv] + __popcll(mask & below)] = (uint16_t)(k * NT + t);
    }
    __syncthreads();
    for (uint32_t i = t; i < (uint32_t)nv; i += NT) {
        const int32_t id = list[i];
        ev.victims[i] = id;
        drop_victim(ev, st, slots, id, rebuild);
    }
    if (rebuild)  // the survivors are entered again by publish
        for (uint64_t i = t; i < slots_n; i += NT) slots[i] = empty_slot();
    if (t == 0) evict_account(st, capacity, slots_n, nv);
}

}  // namespace ptsd
