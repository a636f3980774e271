// Batched longest-common-prefix lookup (PTStore Section 4.1, the LCP query:
// the longest prefix of a request that is stored, and the ids along it).
//
// One wavefront per request, lane j owns block w0+j of a 64-block window:
//   1. the wave copies the window's tokens into LDS with coalesced loads and
//      each lane hashes its block from there;
//   2. a wave prefix scan chains the hashes into per-block prefix keys;
//   3. each lane probes the open-addressing index for its key up to the
//      first key hit; the hits' stored tokens are compared by four lanes per
//      row, and a lane whose hit holds other tokens probes on, so it accepts
//      the first slot whose stored block has the same tokens;
//   4. the candidate of lane j must have as parent the id accepted by lane
//      j-1 (the root, -1, for block 0; the slot carries the parent id, so this
//      costs no extra load); a ballot finds the first lane that
//      fails, which is the end of the match. If that lane did find a block
//      with the right tokens but the wrong parent (two prefixes whose keys
//      collide), it keeps probing for one with the right parent before the
//      window is decided, so the answer never depends on the hash.
// Windows are walked in order and the walk stops at the first miss; for
// requests with room for more than one window, k_lookup_wide gives each
// window of a round its own wave instead.
// With eviction on, every matched block counts one access: its frequency F
// grows by one and its priority becomes max(H, L + F), which is L + F for
// the final F whatever order the atomics land in.
//
// An insert's match is the same walk (kInsert): it also writes every block's
// chained key, going on to hash the windows past the first miss, and claims
// the batch-table entries of the blocks past the match (see insert.hip).
#include "kernels.hpp"

namespace ptsd {
namespace {

constexpr int kThreads = 256;
constexpr int kWavesPerGroup = kThreads / kWave;

// Makes a wave's LDS writes visible to its other lanes and keeps the
// compiler from moving LDS accesses across this point. A wave's LDS
// operations are performed in the order it issues them, so no other wave
// takes part.
__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// All four bits of each 4-bit group of b set -> one bit per group (16 bits).
__device__ inline uint64_t quads_all(uint64_t b) {
    uint64_t t = b & (b >> 1);
    t = t & (t >> 2) & 0x1111111111111111ull;
    t = (t | (t >> 3)) & 0x0303030303030303ull;
    t = (t | (t >> 6)) & 0x000F000F000F000Full;
    t = (t | (t >> 12)) & 0x000000FF000000FFull;
    return (t | (t >> 24)) & 0xFFFFull;
}

constexpr int kQuads = 4;  // 16-byte pieces of a block of 16 tokens

// A window of up to 64 blocks of 16 tokens of one request, staged in the
// wave's own LDS area. The request is read with coalesced 16-byte loads
// (consecutive lanes, consecutive bytes: a 4 KiB window costs 64 requests to
// the L2 instead of 256 when each lane read its own block), and each lane
// then hashes and compares its block from LDS. Stored rows are compared four
// lanes to a row, so one load instruction reads 16 whole 64-byte rows.
struct Window16 {
    int4* sh;  // [kWave][kQuads], this wave's area
    int lane;

    // area: the workgroup's LDS, kWave * kQuads int4 per wave
    __device__ inline void init(int4* area, int wave, int l) {
        sh = area + wave * (kWave * kQuads);
        lane = l;
    }

    // n > 0. All of a lane's loads are issued before any is waited for:
    // pieces past the window's end re-read the last piece of the request's
    // blocks and land in LDS rows no lane reads. A window past the request's
    // end (uniform) has no lane that reads any.
    __device__ inline void stage(const int32_t* __restrict__ seq, int w0, int n, int) {
        if (w0 >= n) return;
        wave_lds_sync();  // the previous window's reads are issued
        const int nq = (n - w0 < kWave ? n - w0 : kWave) * kQuads;
        const int32_t* base = seq + (int64_t)w0 * 16;
        const int q0 = lane, q1 = kWave + lane, q2 = 2 * kWave + lane, q3 = 3 * kWave + lane;
        const int4 v0 = load_tokens4(base + 4 * (q0 < nq ? q0 : nq - 1));
        const int4 v1 = load_tokens4(base + 4 * (q1 < nq ? q1 : nq - 1));
        const int4 v2 = load_tokens4(base + 4 * (q2 < nq ? q2 : nq - 1));
        const int4 v3 = load_tokens4(base + 4 * (q3 < nq ? q3 : nq - 1));
        sh[q0] = v0;
        sh[q1] = v1;
        sh[q2] = v2;
        sh[q3] = v3;
        wave_lds_sync();
    }
    // streamed from LDS a piece at a time (four tokens live, not sixteen)
    __device__ inline uint64_t hash(bool active, uint64_t seed, int) const {
        if (!active) return 0;
        uint64_t h = content_hash_init(seed, 16);
#pragma unroll
        for (int i = 0; i < kQuads; ++i) {
            const int4 v = sh[lane * kQuads + i];
            h = content_hash_pair(h, v.x, v.y, 4 * i);
            h = content_hash_pair(h, v.z, v.w, 4 * i + 2);
        }
        return content_hash_final(h);
    }
    // This lane's block against one stored row (64-byte aligned). Only the
    // rare paths (a key hit with other tokens, a key collision between
    // prefixes) compare one lane at a time, so this takes one piece per step
    // to keep the kernel's register count down.
    __device__ inline bool equals(const int32_t* __restrict__ s, int) const {
        bool eq = true;
#pragma unroll 1
        for (int i = 0; i < kQuads; ++i) {
            const int4 v = *reinterpret_cast<const int4*>(s + 4 * i);
            const int4 w = sh[lane * kQuads + i];
            eq &= (v.x == w.x) & (v.y == w.y) & (v.z == w.z) & (v.w == w.w);
        }
        return eq;
    }
    // Token check of every lane's candidate (-1: none); called by the whole
    // wave. Returns whether this lane's candidate row holds its tokens. The
    // four row loads are issued together; a lane of a block without a
    // candidate reads row 0 (always allocated) and ignores it.
    __device__ inline bool verify(const int32_t* __restrict__ tokens, int32_t cand, int) const {
        constexpr int G = kWave / 16;
        int32_t id[G];
        int4 v[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            id[g] = __shfl(cand, g * 16 + (lane >> 2), kWave);
            const int64_t row = id[g] >= 0 ? id[g] : 0;
            v[g] = *reinterpret_cast<const int4*>(tokens + row * 16 + 4 * (lane & 3));
        }
        uint64_t ok = 0;  // bit j: block j's candidate row holds block j's tokens
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int4 w = sh[(g * 16 + (lane >> 2)) * kQuads + (lane & 3)];
            const bool eq = (id[g] >= 0) & (v[g].x == w.x) & (v[g].y == w.y) & (v[g].z == w.z) &
                            (v[g].w == w.w);
            ok |= quads_all(ballot64(eq)) << (16 * g);
        }
        return (ok >> lane) & 1;
    }
};

// A window of blocks of another multiple of four tokens (which: through_lds).
// Its tokens pass through the wave's LDS area sixteen a block at a time: four
// lanes read 64 neighbouring bytes of a row, every lane hashes its own block's part from
// LDS, and the next part's loads are under way meanwhile. The token check
// reads the window and the stored rows again by whole lines, lane p of the
// window's 16-byte pieces on the piece's row. Reading and comparing its own
// block a token at a time, every lane had waited for memory about once per
// token: the query of 96 ragged requests of up to 16,384 tokens in blocks of
// 32 takes 24.4 us that way and 12.6 this way (calls back to back).
struct WindowQuads {
    int4* sh;  // [kWave][kQuads], this wave's area
    const int32_t* base;
    int4 v[kQuads];  // the next part of the window on its way to LDS
    int lane, rows;  // rows: blocks from the window's first to the request's end, at most kWave

    __device__ inline void init(int4* area, int wave, int l) {
        sh = area + wave * (kWave * kQuads);
        lane = l;
    }
    __device__ inline void load_part(int part, int bt) {
        const int col = min(kQuads * part + (lane & 3), bt / 4 - 1);
#pragma unroll
        for (int g = 0; g < kQuads; ++g)
            v[g] = load_tokens4(base + min(g * 16 + (lane >> 2), rows - 1) * bt + 4 * col);
    }
    // n > 0
    __device__ inline void stage(const int32_t* __restrict__ seq, int w0, int n, int bt) {
        base = seq + (int64_t)w0 * bt;
        rows = min(n - w0, kWave);
        if (rows > 0) load_part(0, bt);
    }
    // called by the whole wave; a window past the request's end (uniform) has
    // nothing to hash: inserts of 4,096 requests of 4 blocks of 32 tokens with
    // room for 2,048 take 229 us, 271 when such windows were hashed
    __device__ inline uint64_t hash(bool active, uint64_t seed, int bt) {
        if (rows <= 0) return 0;
        uint64_t h = content_hash_init(seed, bt);
        const int parts = (bt / 4 + kQuads - 1) / kQuads;
        for (int part = 0; part < parts; ++part) {
            wave_lds_sync();  // the previous part's reads are issued
#pragma unroll
            for (int g = 0; g < kQuads; ++g) sh[g * kWave + lane] = v[g];
            wave_lds_sync();
            if (part + 1 < parts) load_part(part + 1, bt);
            const int end = min(bt / 4 - part * kQuads, kQuads);
#pragma unroll
            for (int i = 0; i < kQuads; ++i)
                if (i < end) {
                    const int4 x = sh[lane * kQuads + i];
                    const int at = 4 * (part * kQuads + i);
                    h = content_hash_pair(h, x.x, x.y, at);
                    h = content_hash_pair(h, x.z, x.w, at + 2);
                }
        }
        return active ? content_hash_final(h) : 0;
    }
    // This lane's block against one stored row (16-byte aligned).
    __device__ inline bool equals(const int32_t* __restrict__ s, int bt) const {
        bool eq = true;
        for (int i = 0; i < bt; i += 4) {
            const int4 a = *reinterpret_cast<const int4*>(s + i);
            const int4 w = load_tokens4(base + lane * bt + i);
            eq &= (a.x == w.x) & (a.y == w.y) & (a.z == w.z) & (a.w == w.w);
        }
        return eq;
    }
    // Token check of every lane's candidate (-1: none); called by the whole
    // wave. A lane that finds a difference clears the row's word in LDS.
    __device__ inline bool verify(const int32_t* __restrict__ tokens, int32_t cand, int bt) const {
        if (!ballot64(cand >= 0)) return false;  // uniform; a candidate means rows > 0
        int32_t* same = reinterpret_cast<int32_t*>(sh);
        wave_lds_sync();  // the hash's reads are issued
        same[lane] = 1;
        wave_lds_sync();
        const int q = bt / 4;
        const unsigned inv = (65536u + (unsigned)q - 1u) / (unsigned)q;  // p / q for p < 1024, q <= 16
        for (int i0 = 0; i0 < q; i0 += kQuads) {
            int32_t row[kQuads], id[kQuads];
            int4 a[kQuads], w[kQuads];
#pragma unroll
            for (int j = 0; j < kQuads; ++j) {
                const int p = min(i0 + j, q - 1) * kWave + lane;  // past the end: the last again
                row[j] = (int32_t)(((unsigned)p * inv) >> 16);
                const int col = p - row[j] * q;
                id[j] = __shfl(cand, row[j], kWave);
                const int64_t stored = id[j] >= 0 ? id[j] : 0;
                a[j] = *reinterpret_cast<const int4*>(tokens + stored * bt + 4 * col);
                w[j] = load_tokens4(base + min(row[j], rows - 1) * bt + 4 * col);
            }
#pragma unroll
            for (int j = 0; j < kQuads; ++j)
                if ((id[j] >= 0) & !((a[j].x == w[j].x) & (a[j].y == w[j].y) & (a[j].z == w[j].z) &
                                     (a[j].w == w[j].w)))
                    same[row[j]] = 0;
        }
        wave_lds_sync();
        return cand >= 0 && same[lane] != 0;
    }
};

// Any block size: each lane reads its own block from the request.
struct WindowAny {
    const int32_t* p;  // this lane's block (meaningful for lanes inside the request)
    int lane;

    __device__ inline void init(int4*, int, int l) { lane = l; }

    __device__ inline void stage(const int32_t* __restrict__ seq, int w0, int, int bt) {
        p = seq + (int64_t)(w0 + lane) * bt;
    }
    __device__ inline uint64_t hash(bool active, uint64_t seed, int bt) const {
        return active ? content_hash_mem(p, bt, seed) : 0;
    }
    __device__ inline bool equals(const int32_t* __restrict__ s, int bt) const {
        for (int i = 0; i < bt; ++i)
            if (s[i] != p[i]) return false;
        return true;
    }
    __device__ inline bool verify(const int32_t* __restrict__ tokens, int32_t cand, int bt) const {
        return cand >= 0 && equals(tokens + (int64_t)cand * bt, bt);
    }
};

// The window type for a block size: 16, any multiple of 4 (kFours) or any at
// all (0).
constexpr int kFours = 4;
template <int BT>
struct WindowOf {
    static_assert(BT == 0, "block sizes: 16, a multiple of 4, or any");
    typedef WindowAny type;
};
template <>
struct WindowOf<kFours> {
    typedef WindowQuads type;
};
template <>
struct WindowOf<16> {
    typedef Window16 type;
};

// First slot along the probe sequence from `pos` that holds `ikey`, its
// tokens not yet compared; -1 at the first empty slot. *pos_out is the slot
// and *parent_out the block's parent id.
__device__ inline int32_t probe_key(const IndexView& ix, uint64_t ikey, uint64_t pos, uint64_t* pos_out,
                                    int32_t* parent_out, unsigned* probes) {
    while (true) {
        const Slot s = load_slot(ix.slots + pos);
        ++*probes;
        if (s.key == kEmptyKey) {
            *pos_out = pos;
            return -1;
        }
        if (s.key == ikey) {
            *pos_out = pos;
            *parent_out = s.parent;
            return s.id;
        }
        pos = (pos + 1) & ix.slot_mask;
    }
}

// Linear probing from `pos` for a slot holding `ikey` whose block has the
// lane's tokens (and, if need_parent, parent id `want_parent`), comparing as
// it goes. Returns the block id or -1 at the first empty slot.
template <class Win>
__device__ inline int32_t probe(const IndexView& ix, uint64_t ikey, uint64_t pos, const Win& win,
                                bool need_parent, int32_t want_parent, uint64_t* pos_out,
                                int32_t* parent_out, unsigned* probes, unsigned* cmps) {
    const int bt = ix.block_tokens;
    while (true) {
        const Slot s = load_slot(ix.slots + pos);
        ++*probes;
        if (s.key == kEmptyKey) {
            *pos_out = pos;
            return -1;
        }
        if (s.key == ikey && (!need_parent || s.parent == want_parent)) {
            ++*cmps;
            if (win.equals(ix.tokens + (int64_t)s.id * bt, bt)) {
                *pos_out = pos;
                *parent_out = s.parent;
                return s.id;
            }
        }
        pos = (pos + 1) & ix.slot_mask;
    }
}

// Every lane's first block along its key's probe sequence that holds its
// tokens (-1: none); called by the whole wave. All lanes find their first
// key hit, the hits' tokens are compared together, and a lane whose hit
// holds other tokens (a content-hash collision) probes on alone.
template <class Win>
__device__ inline int32_t find_block(const IndexView& ix, const Win& win, bool active, uint64_t ik,
                                     uint64_t slot_seed, uint64_t* pos, int32_t* par, unsigned* probes,
                                     unsigned* cmps) {
    int32_t cand = -1;
    if (active) {
        cand = probe_key(ix, ik, slot_of(ik, slot_seed, ix.slot_mask), pos, par, probes);
        if (cand >= 0) ++*cmps;
    }
    const bool same = win.verify(ix.tokens, cand, ix.block_tokens);
    if (cand >= 0 && !same)
        cand = probe(ix, ik, (*pos + 1) & ix.slot_mask, win, false, 0, pos, par, probes, cmps);
    return cand;
}

// Request bounds; a malformed request is empty and counted.
__device__ inline int32_t request_blocks(const Batch& b, int64_t r, int bt, int lane,
                                         DevState* st, int64_t* o0) {
    int64_t a = b.offsets[r], e = b.offsets[r + 1];
    if (a < 0 || e < a || e > b.n_tokens) {
        if (lane == 0) atomicAdd(&st->bad_entries, 1ull);
        *o0 = 0;
        return 0;
    }
    *o0 = a;
    int64_t n = (e - a) / bt;
    return (int32_t)(n < b.max_blocks ? n : b.max_blocks);
}

// What a walk does besides matching: variants of their own, so that the
// plain lookup keeps its register count.
enum Mode {
    kPlain,   // nothing
    kTouch,   // count accesses (eviction on)
    kInsert,  // an insert's match: keys of every block, claims of the new ones
};

// The collision flag down, and the eviction epoch advanced, so that a
// replayed capture marks its own matches.
__device__ inline void insert_setup(const InsertMatch& im, DevState* st) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *im.collision = 0;
        if (im.ev_on) {  // protection marks are compared with it; 0 marks nothing
            const unsigned long long e = st->ev_epoch + 1;
            st->ev_epoch = e >= 0x7FFFFFFFull ? 1ull : e;
        }
    }
}

// Request r's new block b, index key ik, claims or joins the batch-table
// entry of its name. The table holds at least twice as many entries as the
// batch has blocks.
__device__ inline void claim(const InsertMatch& im, int64_t at, int64_t r, int32_t b, uint64_t ik,
                             uint64_t slot_seed, uint32_t weak_tag, unsigned* cas, unsigned* fails) {
    const unsigned long long tag = batch_tag(ik, b, slot_seed, weak_tag);
    uint64_t pos = tag & im.table_mask;
    while (true) {
        const unsigned long long prev = atomicCAS(&im.table[pos].word, kEmptyKey, tag);
        ++*cas;
        if (prev == kEmptyKey) {
            im.table[pos].depth = b;  // read by verify, a kernel later
            break;
        }
        if (prev == tag) break;
        ++*fails;
        pos = (pos + 1) & im.table_mask;
    }
    atomicMin(&im.table[pos].owner, (int32_t)r);
    im.label[at] = (int32_t)pos;
}

template <int BT, int MODE>
__global__ __launch_bounds__(kThreads) void k_lookup(IndexView ix, Batch bat, int32_t* __restrict__ m_out,
                                                     int32_t* __restrict__ ids_out, InsertMatch im) {
    constexpr bool TOUCH = MODE == kTouch;
    if (MODE == kInsert) insert_setup(im, ix.state);
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t r = (int64_t)blockIdx.x * kWavesPerGroup + (threadIdx.x / kWave);
    if (r >= bat.R) return;  // uniform per wave
    const int bt = BT == 16 ? 16 : ix.block_tokens;
    const ChainConsts cc = chain_consts(ix.ht, lane);
    int64_t o0;
    const int32_t n = request_blocks(bat, r, bt, lane, ix.state, &o0);
    const int32_t* __restrict__ seq = bat.tokens + o0;
    int32_t* __restrict__ row = ids_out + r * bat.max_blocks;
    __shared__ int4 sh_tok[BT ? kThreads * kQuads : 1];
    typename WindowOf<BT>::type win;
    win.init(sh_tok, threadIdx.x / kWave, lane);

    const uint64_t clock = TOUCH ? ix.state->clock : 0;
    uint64_t carry_key = cc.root_key;
    int32_t carry_id = -1;  // the root
    int32_t m = 0;
    unsigned probes = 0, cmps = 0, cas = 0, fails = 0;
    const uint32_t weak_tag = MODE == kInsert ? ix.ht->weak_tag : 0;
    int w0 = 0;
    bool done = false;
    for (; w0 < n && !done; w0 += kWave) {
        const int b = w0 + lane;
        const bool active = b < n;
        win.stage(seq, w0, n, bt);
        const uint64_t c = win.hash(active, cc.content_seed, bt);
        const uint64_t k = window_chain(c, carry_key, cc, lane);
        if (MODE == kInsert && active) im.keys[r * bat.max_blocks + b] = k;  // one window: see launch_lookup
        const uint64_t ik = index_key(k, cc);
        int32_t cpar = -2;
        uint64_t pos = 0;
        int32_t cand = find_block(ix, win, active, ik, cc.slot_seed, &pos, &cpar, &probes, &cmps);
        int first_bad = kWave;
        while (true) {
            int32_t prev = __shfl_up(cand, 1, kWave);
            if (lane == 0) prev = carry_id;
            const int32_t par = cand >= 0 ? cpar : -2;
            const bool ok = active && cand >= 0 && par == prev;
            const unsigned long long bad = ballot64(!ok);
            if (bad == 0) break;
            const int f = __ffsll((long long)bad) - 1;
            const int retry = __shfl((active && cand >= 0 && par != prev) ? 1 : 0, f, kWave);
            if (!retry) {
                first_bad = f;
                break;
            }
            // keys of two different prefixes collided: lane f looks further
            // along its probe sequence for the block with the right parent
            if (lane == f)
                cand = probe(ix, ik, (pos + 1) & ix.slot_mask, win, true, prev, &pos, &cpar,
                             &probes, &cmps);
        }
        if (MODE == kInsert && active && lane >= first_bad)
            claim(im, r * bat.max_blocks + b, r, b, ik, cc.slot_seed, weak_tag, &cas, &fails);
        if (active) row[b] = lane < first_bad ? cand : -1;
        if (TOUCH && active && lane < first_bad) {
            const uint64_t f = atomicAdd((unsigned long long*)&ix.freq[cand], 1ull) + 1ull;
            atomicMax((unsigned long long*)&ix.prio[cand], (unsigned long long)(clock + f));
        }
        if (first_bad < kWave) {
            m = w0 + first_bad;
            done = true;
        } else {
            m = w0 + kWave;
            carry_id = __shfl(cand, kWave - 1, kWave);
            carry_key = shfl_u64(k, kWave - 1);
        }
    }
    const int fill_from = w0 < n ? w0 : n;
    for (int b = fill_from + lane; b < bat.max_blocks; b += kWave) row[b] = -1;
    if (lane == 0) {
        m_out[r] = m;
        if (MODE == kInsert) {
            im.nblk[r] = n;
            im.cnt[r] = 0;
        }
    }
    if (ix.counters) {
        CounterSlot* cs = counter_slot(ix.state);
        wave_count(&cs->probes, probes, lane);
        wave_count(&cs->token_compares, cmps, lane);
        if (MODE == kInsert) {
            wave_count(&cs->cas_attempts, cas, lane);
            wave_count(&cs->cas_failures, fails, lane);
        }
    }
}

// Long requests: one workgroup of W waves per request, each wave on its
// own window, W windows per round instead of one after another. Within a
// round each wave scans its window's key chain from a zero carry; the affine
// chain makes window w's carry P^64 * (carry of window w-1) + (its offset),
// folded over the round's earlier windows from LDS, so every lane then has
// its key and probes at once. A position's parent check needs the candidate
// of the position before it, across a wave boundary through LDS. The round's
// first failing position decides; only when it found the right tokens under
// another parent (a key collision) does that lane probe on, and the round is
// checked again.
template <int BT, int MODE, int W>
__global__ __launch_bounds__(W * kWave) void k_lookup_wide(IndexView ix, Batch bat,
                                                           int32_t* __restrict__ m_out,
                                                           int32_t* __restrict__ ids_out, InsertMatch im) {
    constexpr bool TOUCH = MODE == kTouch;
    if (MODE == kInsert) insert_setup(im, ix.state);
    __shared__ uint64_t sh_off[W];   // each window's chain offset (zero carry)
    __shared__ int32_t sh_last[W];   // candidate of each window's last lane
    __shared__ int32_t sh_fail[W];   // first failing lane per window (kWave: none)
    __shared__ int32_t sh_retry[W];  // 1: that lane found the tokens under another parent
    __shared__ uint64_t sh_klast;    // key of the round's last position
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = threadIdx.x / kWave;
    const int64_t r = blockIdx.x;
    if (r >= bat.R) return;  // uniform over the workgroup
    const int bt = BT == 16 ? 16 : ix.block_tokens;
    const ChainConsts cc = chain_consts(ix.ht, lane);
    int64_t o0;
    const int32_t n = request_blocks(bat, r, bt, wv == 0 ? lane : 1, ix.state, &o0);
    const int32_t* __restrict__ seq = bat.tokens + o0;
    int32_t* __restrict__ row = ids_out + r * bat.max_blocks;
    const uint64_t clock = TOUCH ? ix.state->clock : 0;
    const uint64_t p64 = ix.ht->pow_lane[kWave - 1];  // P^64
    __shared__ int4 sh_tok[BT ? W * kWave * kQuads : 1];
    typename WindowOf<BT>::type win;
    win.init(sh_tok, wv, lane);
    uint64_t carry_key = cc.root_key;
    int32_t carry_id = -1;  // the root
    int32_t m = n;
    unsigned probes = 0, cmps = 0, cas = 0, fails = 0;
    const uint32_t weak_tag = MODE == kInsert ? ix.ht->weak_tag : 0;
    int r0 = 0;  // first block of the round
    for (; r0 < n; r0 += W * kWave) {
        const int b = r0 + wv * kWave + lane;
        const bool active = b < n;
        win.stage(seq, r0 + wv * kWave, n, bt);
        const uint64_t c = win.hash(active, cc.content_seed, bt);
        const uint64_t sl = window_chain(c, 0, cc, lane);  // zero-carry chain
        if (lane == kWave - 1) sh_off[wv] = sl;
        __syncthreads();
        uint64_t carry = carry_key;
        for (int i = 0; i < wv; ++i) carry = addmod61(mulmod61(p64, carry), sh_off[i]);
        const uint64_t k = addmod61(mulmod61(cc.lane_pow, carry), sl);
        if (MODE == kInsert && active) im.keys[r * bat.max_blocks + b] = k;
        const uint64_t ik = index_key(k, cc);
        int32_t cpar = -2;
        uint64_t pos = 0;
        int32_t cand = find_block(ix, win, active, ik, cc.slot_seed, &pos, &cpar, &probes, &cmps);
        if (wv == W - 1 && lane == kWave - 1) sh_klast = k;
        int fail = W * kWave;  // first failing position of the round, relative to r0
        while (true) {
            if (lane == kWave - 1) sh_last[wv] = cand;
            __syncthreads();
            int32_t prev = __shfl_up(cand, 1, kWave);
            if (lane == 0) prev = wv == 0 ? carry_id : sh_last[wv - 1];
            const int32_t par = cand >= 0 ? cpar : -2;
            const bool ok = active && cand >= 0 && par == prev;
            const unsigned long long bad = ballot64(!ok);
            const int f = bad ? __ffsll((long long)bad) - 1 : kWave;
            const int rt = f < kWave ? __shfl((active && cand >= 0 && par != prev) ? 1 : 0, f, kWave) : 0;
            if (lane == 0) {
                sh_fail[wv] = f;
                sh_retry[wv] = rt;
            }
            __syncthreads();
            int fw = -1;
            for (int i = 0; i < W; ++i)
                if (sh_fail[i] < kWave) {
                    fw = i;
                    break;
                }
            const int fl = fw >= 0 ? sh_fail[fw] : kWave;
            const bool again = fw >= 0 && sh_retry[fw];
            fail = fw >= 0 ? fw * kWave + fl : W * kWave;  // anew in each check: a retry may clear it
            __syncthreads();  // every wave has read the round's flags
            if (!again) break;
            // keys of two different prefixes collided: that lane looks
            // further along its probe sequence for the block with the
            // right parent, then the round is checked again
            if (wv == fw && lane == fl)
                cand = probe(ix, ik, (pos + 1) & ix.slot_mask, win, true, prev, &pos, &cpar,
                             &probes, &cmps);
        }
        const int rel = wv * kWave + lane;
        if (MODE == kInsert && active && rel >= fail)
            claim(im, r * bat.max_blocks + b, r, b, ik, cc.slot_seed, weak_tag, &cas, &fails);
        if (active) row[b] = rel < fail ? cand : -1;
        if (TOUCH && active && rel < fail) {
            const uint64_t fq = atomicAdd((unsigned long long*)&ix.freq[cand], 1ull) + 1ull;
            atomicMax((unsigned long long*)&ix.prio[cand], (unsigned long long)(clock + fq));
        }
        if (fail < W * kWave) {
            m = r0 + fail < n ? r0 + fail : n;
            r0 += W * kWave;
            if (MODE == kInsert) carry_key = sh_klast;  // the last round's writes: a barrier ago
            break;
        }
        carry_key = sh_klast;
        carry_id = sh_last[W - 1];
        __syncthreads();  // sh_klast and sh_last read before the next round writes them
    }
    const int fill_from = r0 < n ? r0 : n;
    for (int b = fill_from + (int)threadIdx.x; b < bat.max_blocks; b += W * kWave) row[b] = -1;
    if (threadIdx.x == 0) {
        m_out[r] = m;
        if (MODE == kInsert) {
            im.nblk[r] = n;
            im.cnt[r] = 0;
        }
    }
    if (MODE == kInsert) {  // keys of the rounds past the miss: no probing
        for (; r0 < n; r0 += W * kWave) {
            const int b = r0 + wv * kWave + lane;
            __syncthreads();  // the round before has read sh_off and sh_klast
            win.stage(seq, r0 + wv * kWave, n, bt);
            const uint64_t c = win.hash(b < n, cc.content_seed, bt);
            const uint64_t sl = window_chain(c, 0, cc, lane);
            if (lane == kWave - 1) sh_off[wv] = sl;
            __syncthreads();
            uint64_t carry = carry_key;
            for (int i = 0; i < wv; ++i) carry = addmod61(mulmod61(p64, carry), sh_off[i]);
            const uint64_t k = addmod61(mulmod61(cc.lane_pow, carry), sl);
            if (b < n) {
                im.keys[r * bat.max_blocks + b] = k;
                claim(im, r * bat.max_blocks + b, r, b, index_key(k, cc), cc.slot_seed, weak_tag, &cas, &fails);
            }
            if (wv == W - 1 && lane == kWave - 1) sh_klast = k;
            __syncthreads();
            carry_key = sh_klast;
        }
    }
    if (ix.counters) {
        CounterSlot* cs = counter_slot(ix.state);
        wave_count(&cs->probes, probes, lane);
        wave_count(&cs->token_compares, cmps, lane);
        if (MODE == kInsert) {
            wave_count(&cs->cas_attempts, cas, lane);
            wave_count(&cs->cas_failures, fails, lane);
        }
    }
}

}  // namespace

namespace {
// Whether windows of a multiple of four tokens pass through LDS (WindowQuads)
// or each lane reads its own block. LDS costs half of the waves a compute unit
// can hold and the same work for 64 rows however few a request has; it saves
// a lane its trips to memory, one to two per token. With at most 192 tokens a
// request and more of them than the device then holds waves (4,096), or with
// blocks of four, there is less to save: 8,192 requests of 16 blocks of 8
// tokens take 14.8 us through LDS and 14.1 without (none stored: 12.3 and
// 11.0), of 4 blocks of 20 17.6 and 15.3, of 16 blocks of 4 13.8 and 10.8.
// Past the line LDS wins: 16 blocks of 20 20.2 and 24.4, of 32 22.4 and 47.6;
// 2,048 requests of 64 blocks of 8 7.8 and 10.4.
bool through_lds(const IndexView& ix, const Batch& b) {
    const int32_t bt = ix.block_tokens;
    if (bt % 4 != 0 || bt == 4) return false;
    return b.R <= 4096 || (int64_t)bt * b.max_blocks > 192;
}

template <int MODE, int W>
void launch_wide(const IndexView& ix, const Batch& b, int32_t* m, int32_t* ids, const InsertMatch& im,
                 hipStream_t s) {
    const dim3 grid((unsigned)b.R), block(W * kWave);
    if (ix.block_tokens == 16)
        hipLaunchKernelGGL((k_lookup_wide<16, MODE, W>), grid, block, 0, s, ix, b, m, ids, im);
    else if (through_lds(ix, b))
        hipLaunchKernelGGL((k_lookup_wide<kFours, MODE, W>), grid, block, 0, s, ix, b, m, ids, im);
    else
        hipLaunchKernelGGL((k_lookup_wide<0, MODE, W>), grid, block, 0, s, ix, b, m, ids, im);
}

template <int MODE>
hipError_t launch(const IndexView& ix, const Batch& b, int32_t* m, int32_t* ids, const InsertMatch& im,
                  hipStream_t s) {
    // requests of more than one window: a workgroup per request, windows in
    // parallel (4 waves up to 256 blocks, 8 up to 512, 16 beyond)
    if (b.max_blocks > kWave) {
        if (b.max_blocks <= 4 * kWave)
            launch_wide<MODE, 4>(ix, b, m, ids, im, s);
        else if (b.max_blocks <= 8 * kWave)
            launch_wide<MODE, 8>(ix, b, m, ids, im, s);
        else
            launch_wide<MODE, 16>(ix, b, m, ids, im, s);
        return hipGetLastError();
    }
    const unsigned grid = (unsigned)((b.R + kWavesPerGroup - 1) / kWavesPerGroup);
    if (ix.block_tokens == 16)
        hipLaunchKernelGGL((k_lookup<16, MODE>), dim3(grid), dim3(kThreads), 0, s, ix, b, m, ids, im);
    else if (through_lds(ix, b))
        hipLaunchKernelGGL((k_lookup<kFours, MODE>), dim3(grid), dim3(kThreads), 0, s, ix, b, m, ids, im);
    else
        hipLaunchKernelGGL((k_lookup<0, MODE>), dim3(grid), dim3(kThreads), 0, s, ix, b, m, ids, im);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_lookup(const IndexView& ix, const Batch& b, int32_t* m, int32_t* ids, hipStream_t s) {
    const InsertMatch none{};
    return ix.freq ? launch<kTouch>(ix, b, m, ids, none, s) : launch<kPlain>(ix, b, m, ids, none, s);
}

hipError_t launch_match(const IndexView& ix, const Batch& b, int32_t* m, int32_t* ids,
                        const InsertMatch& im, hipStream_t s) {
    return launch<kInsert>(ix, b, m, ids, im, s);
}

}  // namespace ptsd
