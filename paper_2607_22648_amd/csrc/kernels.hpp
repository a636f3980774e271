// Launch interface between the host runtime (api.hip) and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_common.hpp"

namespace ptsd {

// View of the store used by the lookup kernels (read-only but for the
// access counts).
struct IndexView {
    const Slot* slots;
    uint64_t slot_mask;
    const int32_t* parent;   // [capacity]
    const int32_t* tokens;   // [capacity][block_tokens]
    const HashTables* ht;
    DevState* state;
    uint64_t* freq;          // [capacity] access counts, or null: no accounting
    uint64_t* prio;          // [capacity] priorities H = L + F
    int32_t block_tokens;
    int32_t counters;        // 1: count probes and comparisons
};

// One block to move: physical row (see TierView) <-> cache block cb.
struct Pair {
    int32_t row;
    int32_t cb;
};

// Where block bytes live. Physical rows 0 .. dev_rows-1 are rows of the
// device pool (rows below `owned` are the home of ids below `owned`, the
// rest are replica slots); rows dev_rows + j are rows of the pinned host
// tier, the home of id owned + j.
struct TierView {
    uint8_t* host;        // host tier base (device-accessible), null if none
    int64_t owned;        // ids below live in device memory
    int64_t dev_rows;     // device pool rows: owned + replica slots
    int64_t host_blocks;
    int32_t* rep_of;      // [host_blocks] replica slot or -1; null without replicas
    int32_t* rep_id;      // [replicas] host-tier index (id - owned) held, or -1
    int64_t replicas;
    uint64_t* enter_mask; // [ceil(host_blocks / 64)] blocks entering the hot set
    int32_t* free_list;   // [replicas] free slots, ascending (replicate scratch)
    int32_t* enter_list;  // [replicas] entering host-tier indices, ascending
    Pair* copies;         // [replicas] {host row, replica row} to copy
};

// Most workgroups of a selection pass.
constexpr int kSelGroups = 256;

// Per-block eviction state and the scratch of the victim selection
// (allocated with the store when eviction is on).
struct EvictView {
    uint64_t* freq;     // [capacity] F, 0 for an id that holds no block
    uint64_t* prio;     // [capacity] H, likewise
    int32_t* prot;      // [capacity] last insert epoch (DevState::ev_epoch) whose batch
                        // matched the block
    int32_t* depth;     // [capacity] 0 for a child of the root
    uint64_t* nkey;     // [capacity] index key, to rebuild the index
    uint32_t* spos;     // [capacity] index slot, to delete the entry
    uint64_t* wmask;    // [words] victims of the running insert, one bit per id
    int32_t* victims;   // [capacity] freed ids, ascending (before that, the search's list)
    uint32_t* hist;     // [kSelPasses][kSelBins] digit histograms
    uint64_t* part;     // [kSelGroups][8] per-workgroup partials of the range pass
    int64_t words;      // ceil(capacity / 64)
    int32_t on;         // 0: eviction disabled, nothing here is touched
    TierView tier;      // an evicted host-tier block loses its replica
};

struct Batch {
    const int32_t* tokens;
    const int64_t* offsets;
    int64_t n_tokens;
    int32_t R;
    int32_t max_blocks;
};

// An entry of an insert's batch table, which names the batch's new blocks.
// Empty entries hold kEmptyKey, kNoOwner and any depth.
struct alignas(16) BatchEntry {
    unsigned long long word;  // claim: tag of (key, depth); exact: (parent label << 32) | token position
    int32_t owner;            // smallest request that needs this block
    int32_t depth;            // depth of the claiming block (exact claim: -1)
};
constexpr int32_t kNoOwner = 0x7FFFFFFF;

// lookup.hip
hipError_t launch_lookup(const IndexView& ix, const Batch& b, int32_t* m, int32_t* ids,
                         hipStream_t s);
// An insert's match: the lookup (not an access), and what the insert's later
// kernels need of it.
struct InsertMatch {
    uint64_t* keys;           // [R][max_blocks] out: chained key of every whole block
    int32_t* label;           // [R][max_blocks] out: batch-table entry of each new block
    int32_t* nblk;            // [R] out: blocks of each request (0 for a malformed one)
    int32_t* cnt;             // [R] out: zeroed
    BatchEntry* table;        // the batch table, empty; the new blocks claim their entries
    uint64_t table_mask;
    unsigned int* collision;  // lowered
    int32_t ev_on;            // 1: advance the eviction epoch
};
hipError_t launch_match(const IndexView& ix, const Batch& b, int32_t* m, int32_t* ids,
                        const InsertMatch& im, hipStream_t s);

// copy.hip
struct CopyPlan {
    uint8_t* pool;
    int64_t block_bytes;
    int64_t chunk_bytes;
    int32_t chunks_per_block;  // 2 * layers
    int32_t chunks_per_group;  // chunks one copy unit moves
    int32_t threads;           // workgroup size of the copy kernel
    int32_t gather_threads;    // the same of a gather
    int32_t grid;              // workgroups of the copy kernel, 0 = chosen per call
    int32_t gather_grid;       // most workgroups of a gather (one per unit below that)
    int32_t loop_grid;         // workgroups of a looping (sparse) copy
    int32_t host_grid;         // workgroups that loop over host-tier rows
    DevState* state;
    TierView tier;
    // per-layer slab sizes (null when every layer has chunk_bytes): the
    // device table lbase[l] = 2 * (sum of the slab sizes of layers 0..l-1),
    // L + 1 entries, and the host's copy of it
    const int64_t* lbase;
    const int64_t* lbase_host;
};

// Most layers a store with per-layer slab sizes may have.
constexpr int kMaxVarLayers = 1024;


// A block a gather reads once, and the cache blocks it writes it to:
// dests[base .. base + n), 1 <= n <= kSliceDests. 16-byte aligned, so that a
// kernel reads one with a single load.
struct alignas(16) Slice {
    int32_t row;
    int32_t base;
    int32_t n;
    int32_t pad;
};
constexpr int kSliceDests = 64;  // one per lane of a wave

// Descriptor list of one gather / scatter call: the blocks whose row is in
// device memory first (*total of them), then those whose row is in the host
// tier (*total_h), each part in (request, block) order. A gather turns it
// into slices: each distinct row once, with the cache blocks that need it
// (device-row slices from 0, host-row slices from *total, in the order of
// the first request that needs the row). The row table groups the list's
// entries by row; it sits at the start of the scratch, table_cap slots that
// every call leaves empty, and a call uses its first table_mask + 1.
struct CopyScratch {
    unsigned long long* tkey;    // [table_cap] (row + 1) << 32 | entries so far; 0: empty
    int32_t* tbase;              // [table_cap] where the row's cache blocks start in dests
    uint64_t table_mask;
    Pair* pairs;                 // [R * max_blocks]
    Slice* slices;               // [R * max_blocks]
    int32_t* dests;              // [R * max_blocks]
    int32_t* pslot;              // [R * max_blocks] table slot of each list entry
    int32_t* prank;              // [R * max_blocks] its place among the row's cache blocks
    int32_t* row_cnt;            // [R] device-row blocks of each request
    int32_t* row_cnt_h;          // [R] host-row blocks of each request
    int64_t* row_base;           // [R] exclusive scan of row_cnt
    int64_t* row_base_h;         // [R] exclusive scan of row_cnt_h
    unsigned long long* total;   // device-row pairs
    unsigned long long* total_h; // host-row pairs (after the device-row ones)
    unsigned long long* nslices;   // device-row slices
    unsigned long long* nslices_h; // host-row slices (from slices + *total)
    unsigned long long* ndests;    // cache blocks of device-row slices handed out
    unsigned long long* ndests_h;  // the same for host-row slices (from dests + *total)
};
// Row-table slots a call needs (a power of two >= 2 R max_blocks, at least
// 64), and the scratch bytes of a call after a table region of table_cap
// slots; the carve lays a call out in such a scratch.
uint64_t copy_table_slots(int32_t R, int32_t max_blocks);
size_t copy_scratch_bytes(int32_t R, int32_t max_blocks, uint64_t table_cap);
void copy_scratch_carve(void* base, int32_t R, int32_t max_blocks, uint64_t table_cap,
                        CopyScratch* out);
// Empty row table: zeroes the first `bytes` of a new scratch.
hipError_t launch_zero(void* p, size_t bytes, hipStream_t s);

hipError_t launch_gather_select(const CopyPlan& p, const CopyScratch& sc, const int32_t* ids,
                                const int32_t* m, const int32_t* block_table, int32_t R,
                                int32_t max_blocks, int64_t cache_blocks, hipStream_t s);
hipError_t launch_scatter_select(const CopyPlan& p, const CopyScratch& sc, const int32_t* ids,
                                 const uint8_t* created, const int32_t* block_table, int32_t R,
                                 int32_t max_blocks, int64_t cache_blocks, hipStream_t s);
// Copies of layers l0 .. l1-1 of the listed blocks.
hipError_t launch_gather_copy(const CopyPlan& p, const CopyScratch& sc, uint8_t* cache,
                              int64_t cache_blocks, int32_t R, int32_t max_blocks, int32_t l0,
                              int32_t l1, hipStream_t s);
// A gather of one request into device rows without a list: select and copy in
// one launch, for a call that does not keep its list (no host tier only).
inline bool gathers_without_list(const CopyPlan& p, int32_t R) {
    return R == 1 && p.tier.host_blocks == 0;
}
hipError_t launch_gather_one(const CopyPlan& p, const int32_t* ids, const int32_t* m,
                             const int32_t* block_table, int32_t max_blocks, uint8_t* cache,
                             int64_t cache_blocks, int32_t l0, int32_t l1, hipStream_t s);
hipError_t launch_scatter_copy(const CopyPlan& p, const CopyScratch& sc, const uint8_t* cache,
                               int64_t cache_blocks, int32_t R, int32_t max_blocks, int32_t l0,
                               int32_t l1, hipStream_t s);
// Whole-block copies between rows: pairs[k] = {source row, destination row}.
hipError_t launch_copy_rows(const CopyPlan& p, const Pair* pairs, const unsigned long long* total,
                            int64_t max_pairs, hipStream_t s);

// insert.hip
// The batch table sits at the start of the scratch, table_cap entries that
// every insert leaves empty; a call uses its first table_mask + 1.
struct InsertScratch {
    BatchEntry* table;
    uint64_t table_mask;
    uint64_t* keys;       // [R][max_blocks]
    int32_t* m0;          // [R] match length before the insert
    int32_t* nblk;        // [R] blocks of each request
    int32_t* label;       // [R][max_blocks] batch-table slot of each new block
    int32_t* cnt;         // [R] blocks each request is the first to need (its last ones)
    int32_t* start;       // [R] rank of its block b among the batch's new blocks is start + b
    int32_t* owner;       // [R][max_blocks] smallest request that needs each new block
    unsigned int* collision;  // set when the fast claim must be redone exactly
};
// Batch-table entries a call needs, and the scratch bytes of a call after a
// table of table_cap entries; the carve lays a call out in such a scratch.
uint64_t insert_table_entries(int32_t R, int32_t max_blocks);
size_t insert_scratch_bytes(int32_t R, int32_t max_blocks, uint64_t table_cap);
void insert_scratch_carve(void* base, int32_t R, int32_t max_blocks, uint64_t table_cap,
                          InsertScratch* out);
// Empty batch table in a new scratch.
hipError_t launch_empty_batch(void* table, uint64_t entries, hipStream_t s);

struct InsertTarget {
    Slot* slots;
    int32_t* parent;
    int32_t* tokens;
    int64_t capacity;
};
// An insert is enqueued in three parts: match (lookup .. ranks), then, with
// eviction on, launch_evict, then commit (publish and accesses).
hipError_t launch_insert_match(const IndexView& ix, const InsertTarget& tgt, const EvictView& ev,
                               const Batch& b, const InsertScratch& sc, int32_t* m_out, int32_t* ids,
                               uint8_t* created, hipStream_t s);
hipError_t launch_insert_commit(const IndexView& ix, const InsertTarget& tgt, const EvictView& ev,
                                const Batch& b, const InsertScratch& sc, int32_t* m_out, int32_t* ids,
                                uint8_t* created, hipStream_t s);

// A store of at most this many blocks and index slots evicts inside the
// insert's match part (why the lines lie there: evict_small.hpp).
constexpr int64_t kSmallEvictMax = 16384;
constexpr uint64_t kSmallEvictSlots = 1ull << 18;
inline bool evicts_in_rank(int64_t capacity, uint64_t slots_n) {
    return capacity <= kSmallEvictMax && slots_n <= kSmallEvictSlots;
}

// evict.hip: victim selection and index maintenance of an insert into a larger
// store (between its match and its commit).
hipError_t launch_evict(const IndexView& ix, const InsertTarget& tgt, const EvictView& ev,
                        hipStream_t s);

// evict.hip: make the replica slots hold the hot set of the host tier.
hipError_t launch_replicate(const IndexView& ix, const EvictView& ev, const CopyPlan& p,
                            hipStream_t s);

// api.hip helpers
hipError_t launch_fill_slots(Slot* slots, int64_t n, hipStream_t s);

}  // namespace ptsd
