// Host-side launchers of the HIP kernels (internal to libhookcc).
#pragma once

#include "common.hpp"

namespace hookcc {

// pi[v] = v for v < n; resets the control block.  (Fig. 4, first step.)
// With u non-null, ctrl->windowed or ctrl->scattered says whether consecutive
// entries of the list touch nearby ids.
hipError_t launch_init(int32_t* pi, int32_t n, Ctrl* ctrl, hipStream_t s, const int32_t* u = nullptr,
                       const int32_t* v = nullptr, int64_t m = 0);

// Atomic-Hook (Fig. 3) of entries [begin, end).  When `bits` is non-null the
// giant-component filter is applied (only if ctrl->filter_on is set);
// `halve` adds path halving to the climb; `sym` hooks only entries with
// u <= v (valid when every pair is present in both orientations).
hipError_t launch_ahook(const int32_t* u, const int32_t* v, int64_t begin, int64_t end,
                        int32_t* pi, int32_t n, Ctrl* ctrl, const uint32_t* bits, int block,
                        int ept, bool coherent, bool halve, bool sym, hipStream_t s);

// Atomic-Hook of entries [begin, end), two entries per thread, no filter (short
// segments).
hipError_t launch_ahook_short(const int32_t* u, const int32_t* v, int64_t begin, int64_t end,
                              int32_t* pi, int32_t n, Ctrl* ctrl, bool halve, bool sym,
                              hipStream_t s);
// One atomic-free Hook (Fig. 2) pass over entries [0, m), which are hooked
// again later.  No range check.  Does nothing when `gate` is non-null and
// *gate <= limit.
hipError_t launch_hook_prefix(const int32_t* u, const int32_t* v, int64_t m, int32_t* pi, int32_t n,
                              hipStream_t s, const uint32_t* gate = nullptr, uint32_t limit = 0);

// Where a call's last launch copies the control block for the host (pinned
// memory); nothing is copied when host is null.
struct Post {
    const Ctrl* ctrl = nullptr;
    Ctrl* host = nullptr;
};

// Multi-Jump (Fig. 3) over all n vertices.  `coherent` selects agent-scope
// tree loads and stores (see common.hpp).
hipError_t launch_mj(int32_t* pi, int32_t n, bool coherent, hipStream_t s, Post post = {});

// Multi-Jump for deep trees: pointer jumping within blocks of consecutive
// vertices in LDS, then a climb across blocks (the plain Multi-Jump for
// n < 2^22).  Postcondition as launch_mj: every tree is a star.
hipError_t launch_mj_deep(int32_t* pi, int32_t n, hipStream_t s);
// Multi-Jump with interleaved climbs (atomic-free path); does nothing when
// `gate` is non-null and *gate <= limit.  `settle`: every vertex is stored
// (after a pass of racing workgroup-scope stores); launch_mj_deep always does.
hipError_t launch_mj1(int32_t* pi, int32_t n, const uint32_t* gate, hipStream_t s, bool settle,
                      uint32_t limit = 0, Post post = {});

// Giant-component sample: label of the component that holds the most of
// 1,024 edge endpoints drawn across entries [0, m); sets ctrl->giant and
// ctrl->filter_on.  `again`: only when the filter is not on yet.
hipError_t launch_sample_giant(const int32_t* u, int64_t m, const int32_t* pi, int32_t n,
                               Ctrl* ctrl, hipStream_t s, bool again = false);

// bits[v] = (pi[v] == pi[ctrl->giant]) for v < n (stars required); no-op
// unless ctrl->filter_on.
hipError_t launch_bitmap(const int32_t* pi, int32_t n, Ctrl* ctrl, uint32_t* bits, hipStream_t s);
// Multi-Jump, then (when ctrl->filter_on) the giant bitmap and, when hot_tags
// is non-null, the cached words of the hot-word table, or when vtab is
// non-null, the bits of the vertex table, in one pass.
hipError_t launch_mj_bitmap(int32_t* pi, int32_t n, Ctrl* ctrl, uint32_t* bits,
                            const uint32_t* hot_tags, uint32_t* hot_vals, int slots, uint8_t* vtab,
                            hipStream_t s);

// Atomic-free Hook (Fig. 2) of round `round` (1-based).  Round 1 reads the
// input entries [0, m) and checks ranges; later rounds read the frontier of
// root pairs written by the previous round's compaction (size in ctrl->count).
hipError_t launch_hook_plain(int round, const int32_t* u, const int32_t* v, int64_t m,
                             const int2* f0, const int2* f1, int32_t* pi, int32_t n, Ctrl* ctrl,
                             int block, int ept, int grid_cap, hipStream_t s);

// Window round of the hybrid plan: an atomic-free Hook round over all m
// entries in which each workgroup first joins its chunk of entries inside an
// LDS window of consecutive vertices (see kernels_batch.hip).  Range-checks
// the entries.  Leaves pi a forest (not of stars).  `prefix` > 0: where
// ctrl->scattered is set, the atomic-free round over entries [0, prefix)
// instead (pi the identity, no range check).
hipError_t launch_hook_window(const int32_t* u, const int32_t* v, int64_t m, int32_t* pi,
                              int32_t n, Ctrl* ctrl, uint32_t far_limit, hipStream_t s,
                              int64_t prefix = 0);
int32_t window_slots(int64_t m);  // ids that a window of that round holds
// Atomic-Hook with path halving of the *count root pairs of a frontier.
hipError_t launch_ahook_pairs(const int2* fr, const uint32_t* count, int64_t cap, int32_t* pi,
                              bool halve, int grid_cap, hipStream_t s);

// Atomic-Hook of entries [begin, end) with each workgroup's active roots joined
// in LDS first; pi a forest of stars with few roots left.  Gate as above.
// `all` > end: entries [begin, all) when ctrl->windowed is set.
hipError_t launch_hook_contract(const int32_t* u, const int32_t* v, int64_t begin, int64_t end,
                                int32_t* pi, int32_t n, Ctrl* ctrl, bool halve, hipStream_t s,
                                const uint32_t* gate = nullptr, uint32_t limit = 0, int64_t all = 0);

// Frontier compaction after the Compress of round `round`: keeps the entries
// whose endpoints still have different roots, written as root pairs to f0 or
// f1 (capacity cap), size accumulated in ctrl->count[round & 1].
// tau: frontier rewrite threshold in thousandths (0xffffffff = every round).
// Does nothing when `skip` is non-null and *skip > limit.
hipError_t launch_compact(int round, const int32_t* u, const int32_t* v, int64_t m, int2* f0,
                          int2* f1, int64_t cap, const int32_t* pi, int32_t n, Ctrl* ctrl,
                          uint32_t tau, int block, int ept, int grid_cap, hipStream_t s,
                          const uint32_t* skip = nullptr, uint32_t limit = 0);

// Fig. 1 as a host loop: a Hook pass over all m entries that sets
// ctrl->hook_changed when an entry's parents differ, and one level of Jump
// (Fig. 2) over all vertices that sets ctrl->jump_changed when it moves a
// pointer.
hipError_t launch_hook_flag(const int32_t* u, const int32_t* v, int64_t m, int32_t* pi, int32_t n,
                            Ctrl* ctrl, int block, int ept, hipStream_t s);
hipError_t launch_jump(int32_t* pi, int32_t n, Ctrl* ctrl, hipStream_t s);

// Hot-word LDS cache of the giant bitmap (kernels_hot.hip): `slots`
// direct-mapped slots (16384 or 32768); tags[t] = k means slot t caches bitmap
// word k * slots + t.  Global tag/value arrays hold kHotSlotsMax words.
constexpr int kHotSlotsMax = 32768;
// Vertex table: kVertSets sets of kVertWays one-byte slots; slot 2s + w holds
// the tag k of the vertex k * kVertSets + s (k < kVertTagNone; kVertTagNone
// marks an empty slot).  In device memory: the tags (kVertSlots bytes), then
// one member flag per slot (kVertSlots bytes; 1 = in the giant component).
constexpr int kVertSets = 5 << 14;  // 81,920
constexpr int kVertWays = 2;
constexpr int kVertSlots = kVertSets * kVertWays;  // 163,840 bytes = all 160 KiB of LDS
constexpr uint32_t kVertTagNone = 255;
// Selection sample: up to kVertRuns runs of 64 entries, kVRunsPerPart runs per
// workgroup part; sets grouped in kVBuckets buckets of kVBucketSets.
constexpr int64_t kVertRuns = int64_t(1) << 15;
constexpr int kVRunsPerPart = 128;       // runs of one part
constexpr int kVRunsPerPartShort = 32;   // where that gives at most kVPartsMax parts
constexpr int kVPartsMax = (int)(kVertRuns / kVRunsPerPart);
constexpr int kVPartCap = kVRunsPerPart * 64 * 2;  // endpoints of one part
constexpr int kVBucketSets = 64;
constexpr int kVBuckets = kVertSets / kVBucketSets;
// Scratch words used by launch_hot_vprepare.
constexpr int64_t kVertScratchWords = (int64_t)kVPartsMax * kVPartCap + 2LL * kVPartsMax * kVBuckets;
// For every set, the kVertWays most sampled vertices (scratch:
// kVertScratchWords words); member flags are cleared (launch_mj_bitmap fills
// them).
hipError_t launch_hot_vprepare(const int32_t* u, const int32_t* v, int64_t m, int32_t n,
                               uint32_t* scratch, uint8_t* table, hipStream_t s);
// Filtered Atomic-Hook of entries [begin, end), membership tests answered in
// LDS from the bitmap (n <= kLdsPartMaxN; all of it up to kLdsBitsMaxN, then
// its first kLdsBitsMaxN vertices) or from the vertex table.
constexpr int kLdsBytes = 160 * 1024;
constexpr int32_t kLdsBitsMaxN = kLdsBytes * 8;  // 1,310,720
constexpr int32_t kLdsPartMaxN = 2 * kLdsBitsMaxN;
hipError_t launch_filter_bits(const int32_t* u, const int32_t* v, int64_t begin, int64_t end,
                              int32_t* pi, int32_t n, Ctrl* ctrl, const uint32_t* bits, bool halve,
                              bool sym, hipStream_t s);
hipError_t launch_filter_vertex(const int32_t* u, const int32_t* v, int64_t begin, int64_t end,
                                int32_t* pi, int32_t n, Ctrl* ctrl, const uint32_t* bits,
                                const uint8_t* table, bool halve, bool sym, hipStream_t s);
// Counts sampled endpoints per bitmap word (counts: ceil(n/32) words of
// scratch) and picks the hottest word for every slot.
hipError_t launch_hot_prepare(const int32_t* u, const int32_t* v, int64_t m, int32_t n,
                              uint32_t* counts, uint32_t* tags, int slots, hipStream_t s);
// vals[t] = bits[tags[t] * slots + t]; no-op unless ctrl->filter_on.
hipError_t launch_hot_values(const uint32_t* bits, const uint32_t* tags, uint32_t* vals,
                             const Ctrl* ctrl, int slots, hipStream_t s);
// Filtered Atomic-Hook of entries [begin, end) answering bit tests from the
// LDS copy of (tags, vals) when possible (persistent, one workgroup per CU).
hipError_t launch_ahook_hot(const int32_t* u, const int32_t* v, int64_t begin, int64_t end,
                            int32_t* pi, int32_t n, Ctrl* ctrl, const uint32_t* bits,
                            const uint32_t* tags, const uint32_t* vals, int ept, int slots,
                            bool halve, bool sym, hipStream_t s);

// CSR adjacency (kernels_csr.hip): Atomic-Hook of entries [begin, end) of
// col[], the first endpoint of entry i being its row; `bits` non-null applies
// the giant filter; `sym` hooks only col > row.
hipError_t launch_ahook_csr(const int64_t* row_ptr, const int32_t* col, int32_t n, int64_t begin,
                            int64_t end, int32_t* pi, Ctrl* ctrl, const uint32_t* bits, bool sym,
                            bool halve, hipStream_t s);
// CSR by tiles of kCsrTile entries: the check of row_ptr, the initial tree,
// the row of each tile's first entry (tile_row: tiles + 1 words) and, with su
// non-null, one pair (su[r], sv[r]) per row (see k_csr_prep).
constexpr int kCsrTile = 1024;
constexpr int32_t kCsrLdsBitsMaxN = (kLdsBytes - kCsrTile * 2 * 16) * 8;
hipError_t launch_csr_prep(const int64_t* row_ptr, const int32_t* col, int32_t n, int64_t m,
                           Ctrl* ctrl, int32_t* pi, int32_t* tile_row, int32_t* su, int32_t* sv,
                           hipStream_t s);
// eu[i] = row of entry i.
hipError_t launch_csr_expand(const int64_t* row_ptr, const int32_t* tile_row, int32_t n, int64_t m,
                             int32_t* eu, hipStream_t s);
// Filtered Atomic-Hook of all entries (unfiltered when ctrl->filter_on is 0).
hipError_t launch_csr_filter(const int64_t* row_ptr, const int32_t* col, int32_t n, int64_t m,
                             const int32_t* tile_row, int32_t* pi, Ctrl* ctrl,
                             const uint32_t* bits, bool halve, bool sym, hipStream_t s);
// Sets the range bit unless row_ptr[0] == 0, row_ptr[n] == m and row_ptr is
// non-decreasing.
hipError_t launch_csr_check(const int64_t* row_ptr, int32_t n, int64_t m, Ctrl* ctrl,
                            hipStream_t s);

// Streaming and gather probes used to measure the memory ceilings.
hipError_t launch_probe_stream(const int32_t* u, const int32_t* v, int64_t m, uint32_t* sink,
                               hipStream_t s);
hipError_t launch_probe_gather(const int32_t* u, const int32_t* v, int64_t m, const int32_t* table,
                               int32_t n, uint32_t* sink, hipStream_t s);
// Stream + one agent-scope compare-and-swap per entry on table[u] (table
// must hold table[x] = x; it is left unchanged): succeeding or failing form.
hipError_t launch_probe_cas(const int32_t* u, const int32_t* v, int64_t m, int32_t* table,
                            int32_t n, bool fail, uint32_t* sink, hipStream_t s);
// Memory-model probe (modes 7-9, see kernels_probe.hip): t is int32[128].
hipError_t launch_probe_mm(int mode, int32_t* t, hipStream_t s);
hipError_t launch_probe_bitgather(const int32_t* u, const int32_t* v, int64_t m,
                                  const uint32_t* bits, int32_t n, int variant, uint32_t* sink,
                                  hipStream_t s);

// Batched solve: one workgroup per graph, tree array in LDS, graphs taken
// from device work queues in the order of `descs`; `cus` = CU count, and
// each CU runs as many `block`-thread workgroups as the LDS allows.
// `heads` points at the queues' counters, kQueueBytes of zeroed device memory.
constexpr int kQueues = 8;
constexpr int kQueueStride = 32;  // words between two counters (a cache line each)
constexpr size_t kQueueBytes = sizeof(uint32_t) * kQueues * kQueueStride;
hipError_t prepare_batch_lds();  // once per process, before the first launch
hipError_t launch_batch_lds(const GraphDesc* descs, int32_t count, int32_t max_n, uint32_t* heads,
                            int32_t* status, bool halve, int cus, hipStream_t s, int block);

// A batch by its offsets (vo, eo: int64[count + 1], device or pinned host
// memory) and packed arrays.
struct BatchSrc {
    const int64_t* vo;
    const int64_t* eo;
    const int32_t* u;
    const int32_t* v;
    int32_t* out;
    int32_t max_n;
    int32_t seg_cap;
};
// Batched solve straight from the offsets, in the given order, without a
// preparation launch; status[0 .. 2] as for launch_batch_lds and
// launch_batch_prep.
hipError_t launch_batch_direct(const BatchSrc& src, int32_t count, int32_t* status, bool halve,
                               int cus, hipStream_t s, int block);

// Whether a batch is solved without preparation launches.
bool batch_direct(int32_t count, int32_t max_n, int block, int cus);
// Workgroup size of the LDS solver for a launch of `count` graphs of at most
// max_n vertices.
int batch_block(int32_t count, int32_t max_n);
// Segment caps that stand for the default: lds_auto_segments per graph, of many
// graphs and of at most kFewGraphs.
constexpr int32_t kSegAuto = -1;
constexpr int32_t kSegAutoFew = -2;
constexpr int32_t kFewGraphs = 256;
// Segments of one LDS-solved graph.  A second one (a Multi-Jump half-way)
// costs two barriers and a pass over the vertices and shortens the climbs of
// the second half: it pays for large dense graphs only (alone, n = 1,000,
// m = 65,536 30.0 against 33.5 us; n = 8,192, m = 131,072 46.0 against 54.0;
// n = 8,192, m = 32,768 28.5 against 28.1).  Of 10,000 graphs of average
// degree up to 16 none gets a second one (868 us; two where m / n >= 4 886,
// two where m / n >= 1.5 925 us).  Where every graph has a CU of its own, the
// longer climbs are not hidden by other graphs' work, and it pays from four
// entries per vertex on (100 graphs, n = 60,000, m = 240,000 155 against 168 us;
// n = 20,000, m = 80,000 57 against 58; but 400 of the latter 103 against 98).
__host__ __device__ inline int32_t lds_auto_segments(int64_t m, int64_t n, bool few) {
    return (m > 32768 && m / 8 > n) || (few && m > 65536 && m / 4 >= n) ? 2 : 1;
}

// One graph of at most 32,768 vertices solved by one workgroup in LDS
// (prepare_batch_lds first); *status (device or pinned host) = kStatusRange,
// or *prior (0 when null).
hipError_t launch_single_lds(const GraphDesc& d, const int32_t* prior, int32_t* status, bool halve,
                             hipStream_t s);

// Descriptors of a batch with device offsets, largest first (two launches,
// one thread per graph, with a scan launch between them above 32,768
// graphs); `rows` is scratch of (ceil(B / 1024) + 1) x 256 int32.
// Clears the queue counters; status[1] / status[2] get kStatusBadGraph /
// kStatusRange for invalid graphs (status may be pinned host memory).
hipError_t launch_batch_prep(const int64_t* vo, const int64_t* eo, int32_t B, const int32_t* u,
                             const int32_t* v, int32_t* out, int32_t max_n, int32_t seg_cap,
                             GraphDesc* descs, int32_t* rows, uint32_t* heads, int32_t* status,
                             hipStream_t s);

// Zeroes `words` 32-bit words with a kernel (graph-capture friendly).
hipError_t launch_zero(void* p, int64_t words, hipStream_t s);

int device_cu_count();

}  // namespace hookcc
