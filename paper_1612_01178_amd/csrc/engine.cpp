// Host engine of libhookcc (the C ABI wrappers are in capi.cpp).
//
// The engine turns a call into a plan (hook variant, segment bounds, filter,
// tiling), takes device scratch from a per-(device, stream) cache, enqueues
// the kernel sequence on the caller's stream, and ends with one stream
// synchronisation plus a 256-byte read of the device control block (status
// bits and statistics).  No step of the solve runs on the host.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "engine.hpp"

namespace hookcc {

namespace {
thread_local std::string t_err;
}  // namespace

int32_t fail(int32_t code, const std::string& msg) {
    t_err = msg;
    return code;
}

const char* last_error() { return t_err.c_str(); }

namespace {

#define HIPCHK(expr)                                                                       \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess)                                                              \
            return fail(e_ == hipErrorOutOfMemory ? CC_ERR_NOMEM : CC_ERR_HIP,             \
                        std::string(#expr) + ": " + hipGetErrorString(e_));                \
    } while (0)

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Size class of a work amount w: 4 * floor(log2 w) + the two bits below the
// leading one (0..255; larger w, larger class).
int size_class(uint64_t w) {
    w |= 1;
    const int lg = 63 - __builtin_clzll(w);
    const int frac = lg >= 2 ? (int)((w >> (lg - 2)) & 3) : (int)((w << (2 - lg)) & 3);
    return lg * 4 + frac;
}

// ---------------------------------------------------------------------- plans
// round(m / n), at least 1, for m >= 0 and n > 0, without overflow.
int64_t round_ratio(int64_t m, int64_t n) {
    return std::max<int64_t>(1, m / n + ((m % n) * 2 >= n ? 1 : 0));
}

// First entry of segment i of S over m entries: floor(m * i / S) rounded down
// to a multiple of 4 (keeps 16-byte loads aligned); 128-bit product, so any
// m >= 0 works.
int64_t segment_start(int64_t m, int64_t i, int64_t S) {
    return (int64_t)(((__int128)m * i) / S) & ~int64_t(3);
}

// The automatic filtered plan starts with kPrefixRounds atomic-free rounds
// over the first n entries and a contracting hook of the same entries up to
// kPrefixMaxN vertices, and with an Atomic-Hook of the first n / 16 entries
// above (R-MAT 18, m = 2.6 M: 98 against 106 us; R-MAT 20, m = 2^24: 202
// against 197; R-MAT 21, m = 50 M: 515 against 481; uniform n = 262,144,
// m = 2^22: 182 against 191).  Rounds alone leave fragments that then meet
// in the filtered launches, thousands of entries on a few roots (R-MAT 18
// 170 us, uniform n = 65,536 743 us).  The launches after the rounds take
// kPrefixStart * n entries and then kPrefixGrowth times more each.
//
// A list whose consecutive entries touch nearby ids (the init kernel looks at
// 256 places of it) has no giant in that part, and hooking the rest entry by
// entry is bound by the compare-and-swaps on few roots (2,000 cliques of 60: 238
// us; band of 2^18 vertices, m = 4.2 M: 447).  The first round then is a window
// round over the whole list, the contracting hook takes the whole list too, and
// the launches after it find nothing to do (115 and 100 us; R-MAT 18 pays 3 to 5
// us for the look and the gates).
//
// The Atomic-Hook of the first n / 16 entries runs two entries per thread up
// to kShortMaxN vertices, 8 per thread above, where more climbs at once
// contend for the hubs (R-MAT 20 197 against 229 us, 22 667 and 670, 23
// 1,348 against 1,325, 24 3,313 against 3,257).
constexpr int32_t kShortMaxN = 1 << 22;
constexpr int32_t kPrefixMaxN = 1 << 19;
constexpr int kPrefixRounds = 3;
constexpr int64_t kPrefixStart = 2;
constexpr int64_t kPrefixGrowth = 8;

// End of the launch of that rest which starts at `from`.
int64_t prefix_end(int64_t from, int64_t take, int64_t m) {
    const int64_t to = std::min<int64_t>(m, (from + take) & ~int64_t(3));
    return m - to < take / 2 ? m : to;
}

// Hybrid plan (see enqueue_hybrid).
constexpr int kHybridRounds = 2;
constexpr int32_t kHybridRoundsMaxN = 1 << 20;
constexpr int64_t kHybridLong = int64_t(1) << 22;

struct Plan {
    int hook = CC_HOOK_ATOMIC;  // resolved variant: CC_HOOK_ATOMIC, CC_HOOK_PLAIN or CC_HOOK_HYBRID
    int segments = 1;
    int filter = CC_FILTER_OFF;
    int filter_after = 1;
    int block = 256;
    int ept = 8;
    int64_t max_rounds = 0;
    int rounds_per_check = 4;
    bool profile = false;
    int host_loop = CC_HOST_LOOP_OFF;
    bool coherent = false;
    bool hot = false;  // hot-word LDS cache of the giant bitmap
    int hot_slots = 32768;
    bool halve = true;  // path halving in the Atomic-Hook climb
    bool symmetric = false;  // caller promises both orientations of every pair
    bool graph = false;      // capture the launch sequence in a hipGraph and replay it
    bool no_sync = false;    // enqueue only; status read later by cc_stream_status
    uint32_t tau = 0xffffffffu;  // atomic-free Hook: frontier rewrite threshold (1/1000)
    bool lds_single = false;     // one workgroup solves the whole graph in LDS
    bool lds_bits = false;       // hot: the giant bitmap in LDS
    bool table_room = false;     // the workspace has the vertex table's room all the same
    bool auto_filter = false;    // the filtered schedule of the automatic choice
    bool prefix = false;         // auto_filter: atomic-free rounds over a prefix come first
    bool frontier = false;       // hybrid: the entries left are compacted into pairs
};

// Small lists that the automatic choice gives to one LDS workgroup.  The
// launch costs ~4 us plus ~0.5 us per 1,000 vertices (init, Multi-Jump,
// labels: up to 32,768 vertices, where the slots are 32 bits wide) and
// ~0.22 us per 1,000 entries, against ~70 us for the atomic-free rounds' 14
// commands whatever the size (C call, median: n = 1,000, m = 4,000 17 against
// 68 us; n = 8,192, m = 65,536 34 against 80; n = 32,768, m = 65,536 50
// against 85; n = 65,536, m = 131,072 111 against 76).
bool fits_lds_single(int64_t n, int64_t m) {
    return n > 0 && n <= 32768 && m <= 131072 - 2 * n;
}

// Hook variants an input form supports: pair lists all of them; CSR input and
// the large graphs of a list the Atomic-Hook and the hybrid plan; edges that
// are uploaded in chunks the Atomic-Hook only.
enum PlanInput { kInputPairs, kInputCsr, kInputGraphList, kInputAtomicOnly };

int32_t make_plan(int32_t n, int64_t m, const cc_options* o, Plan& p,
                  PlanInput input = kInputPairs) {
    const bool allow_plain = input == kInputPairs;
    const bool allow_hybrid = input != kInputAtomicOnly;
    cc_options d;
    std::memset(&d, 0, sizeof d);
    d.filter = CC_FILTER_AUTO;
    const cc_options& op = o ? *o : d;
    if (op.reserved[0] != 0) return fail(CC_ERR_ARG, "cc_options.reserved must be zero");
    if (op.graph != 0 && op.graph != 1) return fail(CC_ERR_ARG, "cc_options.graph must be 0 or 1");
    p.graph = op.graph == 1;
    if (op.no_sync != 0 && op.no_sync != 1)
        return fail(CC_ERR_ARG, "cc_options.no_sync must be 0 or 1");
    p.no_sync = op.no_sync == 1;
    if (op.compact_threshold < 0 || op.compact_threshold > 1000)
        return fail(CC_ERR_ARG, "cc_options.compact_threshold must be in [0, 1000]");
    p.tau = op.compact_threshold ? (uint32_t)op.compact_threshold : 0xffffffffu;
    if (op.symmetric != 0 && op.symmetric != 1)
        return fail(CC_ERR_ARG, "cc_options.symmetric must be 0 or 1");
    p.symmetric = op.symmetric == 1;
    if (op.hot_cache < CC_HOT_AUTO || op.hot_cache > CC_HOT_VERTEX)
        return fail(CC_ERR_ARG, "unknown cc_options.hot_cache");
    // Hot cache: the whole bitmap where it fits the LDS (n <= 1,310,720), its
    // first 1,310,720 vertices where that is half of them at least (R-MAT 21,
    // m = 50 M: 495 us against 526 with the vertex table; uniform n = 2^21,
    // m = 33 M: 766 and 854; but R-MAT 22: 742 and 633, and above, where few
    // vertices are in the first part, R-MAT 23: 1,511 and 1,119), then the
    // vertex table where every id fits its tags (n <= 255 *
    // 81,920; R-MAT 24: 3.9 ms against 4.52 with 32,768 word slots), else the
    // word table.
    const bool vert = op.hot_cache == CC_HOT_VERTEX ||
                      (op.hot_cache == CC_HOT_AUTO && n <= (int64_t)kVertTagNone * kVertSets);
    p.lds_bits = op.hot_cache == CC_HOT_AUTO && n <= kLdsPartMaxN;
    // a call that asks for the filter itself has been told the table's size
    p.table_room = op.filter == CC_FILTER_GIANT;
    p.hot_slots = op.hot_cache == CC_HOT_ON ? 16384 : vert ? kVertSlots : 32768;
    if (op.path_halving < CC_HALVE_AUTO || op.path_halving > CC_HALVE_OFF)
        return fail(CC_ERR_ARG, "unknown cc_options.path_halving");
    p.halve = op.path_halving != CC_HALVE_OFF;
    if (op.coherent_loads != 0 && op.coherent_loads != 1)
        return fail(CC_ERR_ARG, "cc_options.coherent_loads must be 0 or 1");
    p.coherent = op.coherent_loads == 1;
    if (op.hook != CC_HOOK_AUTO && op.hook != CC_HOOK_ATOMIC && op.hook != CC_HOOK_PLAIN &&
        op.hook != CC_HOOK_HYBRID)
        return fail(CC_ERR_ARG, "unknown cc_options.hook");
    if (op.segments < 0) return fail(CC_ERR_ARG, "cc_options.segments < 0");
    // Average-degree heuristic (Section 3.B, Fig. 4): s = 2|E|/|V|, read as
    // s = (entries passed) / n -- the average degree when the list holds both
    // orientations of every edge, half of it when each edge is listed once
    // (the library cannot tell the two apart).
    const int64_t s_paper = n > 0 ? std::min<int64_t>(int64_t(1) << 20, round_ratio(m, n)) : 1;
    // Automatic variant (measured on gfx950): on dense lists (average degree
    // >= 8, m >= 2^21) the filtered Atomic-Hook wins (one pass over the entries,
    // most of them reduced to two bitmap tests; R-MAT 24 3.2 ms against 38 ms
    // for the atomic-free rounds; R-MAT 18, m = 2.6 M 98 us against 113 for the
    // hybrid plan, R-MAT 17, m = 2^20 83 against 75); on all other lists the
    // hybrid plan (percolated 4096^2 grid 0.32 ms against 1.07 Atomic-Hook and
    // 0.99 atomic-free rounds; 1237 x 1001 grid 83 us against 186 atomic-free
    // rounds; R-MAT 20, m = 2^22 262 us; uniform n = 65,536, m = 524,672 60
    // against 85), unless the call sets an option of the rounds.  CSR input
    // likewise, without rounds; its filtered plan finds the giant with two
    // neighbours per row and wins from 2^20 entries (R-MAT 16, m = 1.4 M: 71 us
    // against 112 hybrid; R-MAT 15, m = 0.8 M: 86 against 88; R-MAT 13,
    // m = 0.6 M: 97 against 85).
    const bool large = m >= (int64_t(1) << 22);
    const bool dense_large = m >= int64_t(1) << (input == kInputCsr ? 20 : 21) &&
                             n > 0 && m >= 8 * (int64_t)n;
    // A call that sets an option of the rounds gets them where it always did.
    const bool rounds_asked = op.max_rounds != 0 || op.rounds_per_check != 0 || op.compact_threshold != 0;
    // So does a CSR call that sets an option of the segments.
    const bool segments_asked = op.segments != 0 || op.filter_after != 0 || op.filter != CC_FILTER_AUTO;
    bool auto_filtered = false;
    if (op.hook == CC_HOOK_AUTO) {
        if (allow_plain && op.symmetric == 0 && rounds_asked && !large && op.no_sync == 0) {
            p.hook = CC_HOOK_PLAIN;
        } else if (!allow_hybrid || (allow_plain && op.symmetric == 1) || dense_large ||
                   (input == kInputCsr && segments_asked && !large) ||
                   (input == kInputGraphList && m >= (int64_t(1) << 32))) {
            p.hook = CC_HOOK_ATOMIC;
            auto_filtered = dense_large && op.filter != CC_FILTER_OFF;
        } else {
            p.hook = CC_HOOK_HYBRID;
        }
        p.lds_single = fits_lds_single(n, m) &&
                       (allow_plain ? op.symmetric == 0 && !rounds_asked
                                    : input == kInputCsr && !segments_asked);
        if (p.lds_single) p.hook = allow_plain && op.no_sync == 0 ? CC_HOOK_PLAIN : CC_HOOK_HYBRID;
    } else {
        p.hook = op.hook;
    }
    // the scratch of a graph in a list does not grow with its entries
    p.frontier = p.hook == CC_HOOK_HYBRID && m >= kHybridLong && input != kInputGraphList;
    if ((!allow_plain && p.hook == CC_HOOK_PLAIN) || (!allow_hybrid && p.hook == CC_HOOK_HYBRID))
        return fail(CC_ERR_ARG, "the atomic-free Hook is not available here");
    int64_t s = op.segments;
    // The filtered plan hooks its first segment unfiltered, and that launch
    // is the costliest per entry (hub roots contended before any giant
    // exists): a first segment of ~n/16 entries (R-MAT 24: 3.80 ms against
    // 3.86 at n/8 and 3.98 at n/4).
    if (s == 0) s = auto_filtered ? 16 * s_paper : s_paper;
    const int64_t smax = std::max<int64_t>(1, m / 4 + (m % 4 != 0));
    s = std::max<int64_t>(1, std::min<int64_t>(s, smax));
    s = std::min<int64_t>(s, 1 << 20);
    p.segments = (int)s;
    if (op.filter < CC_FILTER_OFF || op.filter > CC_FILTER_AUTO)
        return fail(CC_ERR_ARG, "unknown cc_options.filter");
    if (op.filter_after < 0) return fail(CC_ERR_ARG, "cc_options.filter_after < 0");
    p.filter_after = op.filter_after ? op.filter_after : 1;
    if (p.hook != CC_HOOK_ATOMIC) {
        p.filter = CC_FILTER_OFF;
    } else if (op.hook == CC_HOOK_AUTO && op.filter == CC_FILTER_AUTO) {
        p.filter = auto_filtered ? CC_FILTER_GIANT : CC_FILTER_OFF;
    } else if (op.filter == CC_FILTER_AUTO) {
        // A giant component is near-certain at average degree >= 3.5, and the
        // sample + bitmap cost only pays off on large edge lists.
        p.filter = (p.segments >= 4 && m >= (int64_t(1) << 22)) ? CC_FILTER_GIANT : CC_FILTER_OFF;
    } else {
        p.filter = op.filter;
    }
    if (p.filter == CC_FILTER_GIANT && p.filter_after >= p.segments) p.filter = CC_FILTER_OFF;
    p.hot = p.filter == CC_FILTER_GIANT && op.hot_cache != CC_HOT_OFF && !p.coherent;
    p.auto_filter = auto_filtered && p.filter == CC_FILTER_GIANT && p.hot && op.segments == 0 &&
                    op.filter_after == 0 && op.block == 0 && op.edges_per_thread == 0;
    p.prefix = p.auto_filter && n <= kPrefixMaxN;
    if (op.block != 0) {
        if (op.block < 64 || op.block > 1024 || op.block % 64)
            return fail(CC_ERR_ARG, "cc_options.block must be a multiple of 64 in [64, 1024]");
        p.block = op.block;
    } else if (auto_filtered) {
        p.block = 512;  // first (unfiltered) segment: R-MAT 24 3.78 ms against 3.80 at 256
    }
    // Tile: 16 entries per thread for the plain Atomic-Hook (measured best on
    // sparse lists, e.g. the percolated grid), 8 where the filter runs.
    p.ept = (p.filter == CC_FILTER_GIANT || p.hook != CC_HOOK_ATOMIC) ? 8 : 16;
    // The hybrid plan's atomic-free round over the whole list runs best in
    // large tiles (percolated 4096^2 grid: 0.73 ms at 1024 threads x 16
    // entries against 0.83 ms at 256 x 8).
    if (p.hook == CC_HOOK_HYBRID) {
        p.ept = 16;
        if (op.block == 0) p.block = 1024;
    }
    if (op.edges_per_thread != 0) {
        if (op.edges_per_thread != 4 && op.edges_per_thread != 8 && op.edges_per_thread != 16)
            return fail(CC_ERR_ARG, "cc_options.edges_per_thread must be 4, 8 or 16");
        p.ept = op.edges_per_thread;
    }
    if (op.max_rounds < 0) return fail(CC_ERR_ARG, "cc_options.max_rounds < 0");
    p.max_rounds = op.max_rounds ? op.max_rounds : (int64_t)n + 1;
    if (op.rounds_per_check < 0) return fail(CC_ERR_ARG, "cc_options.rounds_per_check < 0");
    p.rounds_per_check = op.rounds_per_check ? op.rounds_per_check : 4;
    if (op.profile != 0 && op.profile != 1) return fail(CC_ERR_ARG, "cc_options.profile must be 0 or 1");
    p.profile = op.profile == 1;
    if (op.host_loop < CC_HOST_LOOP_OFF || op.host_loop > CC_HOST_LOOP_MULTIJUMP)
        return fail(CC_ERR_ARG, "unknown cc_options.host_loop");
    if (op.host_loop != CC_HOST_LOOP_OFF && op.hook != CC_HOOK_PLAIN)
        return fail(CC_ERR_ARG, "cc_options.host_loop needs hook = CC_HOOK_PLAIN");
    p.host_loop = op.host_loop;
    if (p.symmetric && p.hook != CC_HOOK_ATOMIC && !(input == kInputCsr && p.hook == CC_HOOK_HYBRID))
        return fail(CC_ERR_ARG, "cc_options.symmetric needs the Atomic-Hook");
    if ((p.hook == CC_HOOK_PLAIN || p.hook == CC_HOOK_HYBRID) && m >= (int64_t(1) << 32))
        return fail(CC_ERR_ARG, "atomic-free Hook supports m < 2^32 entries");
    if (p.no_sync && ((p.hook != CC_HOOK_ATOMIC && p.hook != CC_HOOK_HYBRID) || p.profile))
        return fail(CC_ERR_ARG,
                    "cc_options.no_sync needs the Atomic-Hook (the atomic-free Hook reads the "
                    "device convergence word from the host) and profile = 0");
    return CC_OK;
}

// Workspace: [Ctrl 256 B][giant bitmap][frontier 0][frontier 1]
struct Layout {
    size_t bits = 0, f0 = 0, f1 = 0, total = 0;
    size_t hot_counts = 0, hot_tags = 0, hot_vals = 0;
    int64_t cap = 0;
};

Layout layout(int32_t n, int64_t m, const Plan& p) {
    Layout L;
    size_t off = 256;
    if (p.lds_single) {  // the status word only
        L.total = off;
        return L;
    }
    if (p.hook == CC_HOOK_ATOMIC && p.filter == CC_FILTER_GIANT) {
        L.bits = off;
        off += align256(((size_t)n + 31) / 32 * 4);
        if (p.hot && p.lds_bits && !p.table_room) {  // nothing but the bitmap
        } else if (p.hot && p.hot_slots == kVertSlots) {  // selection scratch, byte table
            L.hot_counts = off;
            off += align256((size_t)kVertScratchWords * 4);
            L.hot_tags = L.hot_vals = off;  // tags, then member flags
            off += align256((size_t)kVertSlots * 2);
        } else if (p.hot) {
            L.hot_counts = off;
            off += align256(((size_t)n + 31) / 32 * 4);
            L.hot_tags = off;
            off += align256((size_t)kHotSlotsMax * 4);
            L.hot_vals = off;
            off += align256((size_t)kHotSlotsMax * 4);
        }
    }
    if (p.hook == CC_HOOK_PLAIN && p.host_loop == CC_HOST_LOOP_OFF) {
        L.cap = m;
        L.f0 = off;
        off += align256((size_t)m * 8);
        L.f1 = off;
        off += align256((size_t)m * 8);
    }
    if (p.frontier) {  // written once
        L.cap = m;
        L.f0 = L.f1 = off;
        off += align256((size_t)m * 8);
    }
    L.total = off;
    return L;
}

// ---------------------------------------------------------------------- workspace cache
struct PoolEntry {
    std::mutex mu;  // held for the whole duration of a call using this entry
    void* dev = nullptr;
    size_t bytes = 0;
    Ctrl* host_ctrl = nullptr;  // pinned, host_ctrl_count control blocks
    int64_t host_ctrl_count = 0;
    void* host_stage = nullptr; // pinned staging for batch descriptors
    size_t stage_bytes = 0;
    hipStream_t copy_stream = nullptr;  // host-to-device staging of streamed solves
    hipEvent_t copied[2] = {nullptr, nullptr};
    int32_t* batch_status = nullptr;  // pinned: the LDS batch launch's status word
    hipEvent_t consumed[2] = {nullptr, nullptr};
    // status word of the last no-sync call (pinned) and the event after its copy
    int32_t* async_slot = nullptr;
    hipEvent_t async_done = nullptr;
    bool async_called = false;
    // captured launch sequences of recent calls, most recent last
    struct Captured {
        uint64_t key;
        hipGraph_t graph;
        hipGraphExec_t exec;
    };
    std::vector<Captured> graphs;
};

// Waits for the work of earlier no-sync calls on this entry's stream (before
// a buffer or a graph that work may still use is freed).
void drain_async(PoolEntry* e) {
    if (e->async_called && e->async_done) (void)hipEventSynchronize(e->async_done);
}

void drop_graphs(PoolEntry* e) {
    if (!e->graphs.empty()) drain_async(e);
    for (auto& c : e->graphs) {
        (void)hipGraphExecDestroy(c.exec);
        (void)hipGraphDestroy(c.graph);
    }
    e->graphs.clear();
}

// FNV-1a over the bytes that determine a launch sequence.
struct KeyHash {
    uint64_t h = 1469598103934665603ULL;
    template <class T>
    KeyHash& add(const T& x) {
        const unsigned char* p = reinterpret_cast<const unsigned char*>(&x);
        for (size_t i = 0; i < sizeof(T); ++i) h = (h ^ p[i]) * 1099511628211ULL;
        return *this;
    }
};

std::mutex g_pool_mu;
std::map<std::pair<int, hipStream_t>, std::unique_ptr<PoolEntry>> g_pool;

PoolEntry* pool_entry(hipStream_t s) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = -1;
    std::lock_guard<std::mutex> g(g_pool_mu);
    auto& e = g_pool[{dev, s}];
    if (!e) e.reset(new PoolEntry());
    return e.get();
}

int32_t ensure_dev(PoolEntry* e, size_t bytes) {
    if (e->bytes >= bytes && e->dev) return CC_OK;
    drop_graphs(e);  // captured graphs point into the old buffer
    drain_async(e);
    if (e->dev) {
        HIPCHK(hipFree(e->dev));
        e->dev = nullptr;
        e->bytes = 0;
    }
    size_t want = std::max<size_t>(bytes, 1 << 20);
    HIPCHK(hipMalloc(&e->dev, want));
    e->bytes = want;
    return CC_OK;
}

int32_t ensure_host(PoolEntry* e, int64_t count = 1) {
    if (e->host_ctrl && e->host_ctrl_count >= count) return CC_OK;
    drop_graphs(e);  // captured launches post to the old blocks
    if (e->host_ctrl) {
        HIPCHK(hipHostFree(e->host_ctrl));
        e->host_ctrl = nullptr;
        e->host_ctrl_count = 0;
    }
    const int64_t want = std::max<int64_t>(count, 16);
    HIPCHK(hipHostMalloc((void**)&e->host_ctrl, sizeof(Ctrl) * want, hipHostMallocDefault));
    e->host_ctrl_count = want;
    return CC_OK;
}

int32_t ensure_stage(PoolEntry* e, size_t bytes) {
    if (e->stage_bytes >= bytes && e->host_stage) return CC_OK;
    drop_graphs(e);  // captured copies read from the old staging buffer
    if (e->host_stage) {
        HIPCHK(hipHostFree(e->host_stage));
        e->host_stage = nullptr;
        e->stage_bytes = 0;
    }
    size_t want = std::max<size_t>(bytes, 1 << 16);
    HIPCHK(hipHostMalloc(&e->host_stage, want, hipHostMallocDefault));
    e->stage_bytes = want;
    return CC_OK;
}

// ---------------------------------------------------------------------- profiling
struct Timer {
    bool on = false;
    hipStream_t s = nullptr;
    struct Ev {
        hipEvent_t a, b;
        int phase;
    };
    std::vector<Ev> evs;
    ~Timer() {
        for (auto& e : evs) {
            (void)hipEventDestroy(e.a);
            (void)hipEventDestroy(e.b);
        }
    }
    hipError_t begin(int phase) {
        if (!on) return hipSuccess;
        Ev e;
        e.phase = phase;
        hipError_t r = hipEventCreate(&e.a);
        if (r != hipSuccess) return r;
        r = hipEventCreate(&e.b);
        if (r != hipSuccess) return r;
        evs.push_back(e);
        return hipEventRecord(e.a, s);
    }
    hipError_t end() {
        if (!on) return hipSuccess;
        return hipEventRecord(evs.back().b, s);
    }
    void collect(cc_stats* st) {
        if (!on || !st) return;
        float t[3] = {0, 0, 0};
        for (auto& e : evs) {
            float ms = 0;
            if (hipEventElapsedTime(&ms, e.a, e.b) == hipSuccess) t[e.phase] += ms;
        }
        st->hook_ms = t[0];
        st->compress_ms = t[1];
        st->other_ms = t[2];
    }
};
enum { kPhaseHook = 0, kPhaseCompress = 1, kPhaseOther = 2 };

#define TIMED(phase, expr)                 \
    do {                                   \
        HIPCHK(tm.begin(phase));           \
        HIPCHK(expr);                      \
        HIPCHK(tm.end());                  \
    } while (0)

// Runs `enqueue` on s through a cached hipGraph keyed by `key`: the first
// call with a key captures the launch sequence, later calls replay it.  Up
// to 8 graphs are kept per pool entry.  Needs a stream other than the null
// stream (the legacy null stream cannot be captured).
template <class F>
int32_t run_graph(PoolEntry* pe, uint64_t key, hipStream_t s, F&& enqueue) {
    PoolEntry::Captured* hit = nullptr;
    for (auto& c : pe->graphs)
        if (c.key == key) hit = &c;
    if (!hit) {
        HIPCHK(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
        int32_t rc = enqueue();
        hipGraph_t g = nullptr;
        hipError_t e = hipStreamEndCapture(s, &g);
        if (rc != CC_OK) {
            if (g) (void)hipGraphDestroy(g);
            return rc;
        }
        if (e != hipSuccess) return fail(CC_ERR_HIP, std::string("graph capture: ") + hipGetErrorString(e));
        hipGraphExec_t x = nullptr;
        e = hipGraphInstantiate(&x, g, nullptr, nullptr, 0);
        if (e != hipSuccess) {
            (void)hipGraphDestroy(g);
            return fail(CC_ERR_HIP, std::string("graph instantiate: ") + hipGetErrorString(e));
        }
        if (pe->graphs.size() >= 8) {
            drain_async(pe);
            (void)hipGraphExecDestroy(pe->graphs.front().exec);
            (void)hipGraphDestroy(pe->graphs.front().graph);
            pe->graphs.erase(pe->graphs.begin());
        }
        pe->graphs.push_back({key, g, x});
        hit = &pe->graphs.back();
    }
    HIPCHK(hipGraphLaunch(hit->exec, s));
    return CC_OK;
}

// ---------------------------------------------------------------------- single solve
// Waits for the call's work.  The control block reaches hctrl by a copy unless
// the last launch has posted it there.
int32_t finish(hipStream_t s, const Ctrl* dctrl, Ctrl* hctrl, cc_stats* st, bool posted = false) {
    if (!posted) HIPCHK(hipMemcpyAsync(hctrl, dctrl, sizeof(Ctrl), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if (st) st->host_syncs += 1;
    return CC_OK;
}

// No-sync end of a call: the status word is copied to the entry's pinned slot
// and an event recorded after it; cc_stream_status reads both later.
int32_t post_async(PoolEntry* e, hipStream_t s, const Ctrl* dctrl) {
    if (!e->async_slot) HIPCHK(hipHostMalloc((void**)&e->async_slot, 256, hipHostMallocDefault));
    if (!e->async_done) HIPCHK(hipEventCreateWithFlags(&e->async_done, hipEventDisableTiming));
    HIPCHK(hipMemcpyAsync(e->async_slot, &dctrl->status, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    HIPCHK(hipEventRecord(e->async_done, s));
    e->async_called = true;
    return CC_OK;
}


// Giant-filter buffers of one solve (null when the plan does not use them).
struct FilterBufs {
    uint32_t* bits = nullptr;
    uint32_t* hot_counts = nullptr;
    uint32_t* hot_tags = nullptr;
    uint32_t* hot_vals = nullptr;
    uint8_t* vtab = nullptr;  // vertex table (then hot_tags and hot_vals stay null)
};

FilterBufs filter_bufs(char* base, const Layout& L) {
    FilterBufs f;
    if (L.bits) f.bits = reinterpret_cast<uint32_t*>(base + L.bits);
    if (L.hot_counts && L.hot_tags == L.hot_vals) {
        f.hot_counts = reinterpret_cast<uint32_t*>(base + L.hot_counts);
        f.vtab = reinterpret_cast<uint8_t*>(base + L.hot_tags);
    } else if (L.hot_counts) {
        f.hot_counts = reinterpret_cast<uint32_t*>(base + L.hot_counts);
        f.hot_tags = reinterpret_cast<uint32_t*>(base + L.hot_tags);
        f.hot_vals = reinterpret_cast<uint32_t*>(base + L.hot_vals);
    }
    return f;
}

// Growth factor of the super-segments hooked after the giant filter is on:
// with the filter, later segments hook few edges, so they are taken in
// launches of 2, 8, 32, ... segments (from kSuperStart times the unfiltered
// prefix; each launch followed by a Multi-Jump and a bitmap refresh).
// Measured on R-MAT 24 (s = 512, from 1 segment): x2 3.81 ms, x4 3.76 ms,
// x8 3.88 ms -- fewer refreshes against a staler bitmap.
constexpr int64_t kSuperGrowth = 4;
// Segments of the first filtered launch, as a multiple of the unfiltered
// prefix (filter_after segments): R-MAT 24 (s = 512, launches of 2, 8, 32,
// 128 and 341 segments) 3.58 ms against 3.63 ms for 1, 3.64 for 4 and 3.61
// for 8; the same graph as CSR 4.74 against 4.76 ms for 1.
constexpr int64_t kSuperStart = 2;

// Enqueues the Atomic-Hook solve (Fig. 4) of one graph on s; no
// synchronisation.  `ctrl` is the graph's control block, posted to `host`
// (nullable) by the last launch.
int32_t enqueue_atomic(int32_t n, const int32_t* u, const int32_t* v, int64_t m, int32_t* pi,
                       const Plan& p, Ctrl* ctrl, const FilterBufs& fb, hipStream_t s, Timer& tm,
                       cc_stats* st, Ctrl* host) {
    uint32_t* bits = fb.bits;
    const bool hot = p.hot && fb.hot_tags != nullptr;
    const bool lds_bits = p.hot && p.lds_bits;
    const bool vhot = p.hot && !lds_bits && fb.vtab != nullptr;
    const int S = p.segments;
    auto bound = [&](int64_t i) -> int64_t {
        if (i >= S) return m;
        return segment_start(m, i, S);
    };
    int hooks = 0, jumps = 0;
    const Post post = {ctrl, host};
    if (p.prefix)
        TIMED(kPhaseOther, launch_init(pi, n, ctrl, s, u, v, m));
    else
        TIMED(kPhaseOther, launch_init(pi, n, ctrl, s));
    if (p.filter != CC_FILTER_GIANT) {
        // Fig. 4: for each segment, Atomic-Hook the segment, then Multi-Jump all of V.
        for (int i = 0; i < S; ++i) {
            TIMED(kPhaseHook, launch_ahook(u, v, bound(i), bound(i + 1), pi, n, ctrl, nullptr,
                                           p.block, p.ept, p.coherent, p.halve, p.symmetric, s));
            TIMED(kPhaseCompress, launch_mj(pi, n, p.coherent, s, i + 1 == S ? post : Post{}));
            ++hooks;
            ++jumps;
        }
    } else {
        const int fa = p.filter_after;
        // The part of the list that finds the giant.
        const int64_t prefix = std::min<int64_t>(m, n) & ~int64_t(3);
        // Where consecutive entries touch nearby ids, that part holds none, and
        // one window round and a contracting hook of all entries solve the list;
        // the launches after them find ctrl->windowed set.
        const uint32_t* scattered = &ctrl->scattered;
        for (int i = 0; p.prefix && i <= kPrefixRounds; ++i) {
            if (i == 0)
                TIMED(kPhaseHook, launch_hook_window(u, v, m, pi, n, ctrl, 0, s, prefix));
            else if (i < kPrefixRounds)
                TIMED(kPhaseHook, launch_hook_prefix(u, v, prefix, pi, n, s, scattered));
            else
                TIMED(kPhaseHook, launch_hook_contract(u, v, 0, prefix, pi, n, ctrl, p.halve, s, nullptr, 0, m));
            TIMED(kPhaseCompress, launch_mj1(pi, n, i == 0 || i == kPrefixRounds ? nullptr : scattered, s,
                                             i < kPrefixRounds));
            ++hooks;
            ++jumps;
        }
        for (int i = 0; !p.prefix && i < fa; ++i) {
            if (p.auto_filter && n <= kShortMaxN)
                TIMED(kPhaseHook, launch_ahook_short(u, v, bound(i), bound(i + 1), pi, n, ctrl,
                                                     p.halve, p.symmetric, s));
            else
                TIMED(kPhaseHook, launch_ahook(u, v, bound(i), bound(i + 1), pi, n, ctrl, nullptr,
                                               p.block, p.ept, p.coherent, p.halve, p.symmetric, s));
            TIMED(kPhaseCompress, launch_mj(pi, n, p.coherent, s));
            ++hooks;
            ++jumps;
        }
        if (vhot) TIMED(kPhaseOther, launch_hot_vprepare(u, v, m, n, fb.hot_counts, fb.vtab, s));
        TIMED(kPhaseOther, launch_sample_giant(u, m, pi, n, ctrl, s));
        if (vhot)  // the bitmap and the table's member flags
            TIMED(kPhaseOther, launch_mj_bitmap(pi, n, ctrl, bits, nullptr, nullptr, 0, fb.vtab, s));
        else
            TIMED(kPhaseOther, launch_bitmap(pi, n, ctrl, bits, s));
        if (hot) {
            TIMED(kPhaseOther, launch_hot_prepare(u, v, m, n, fb.hot_counts, fb.hot_tags,
                                                  p.hot_slots, s));
            TIMED(kPhaseOther, launch_hot_values(bits, fb.hot_tags, fb.hot_vals, ctrl,
                                                 p.hot_slots, s));
        }
        // The rest of the list in super-segments that grow by kSuperGrowth,
        // each followed by a Compress and a bitmap refresh.
        int64_t g = fa, step = kSuperStart * fa;                  // in segments
        int again = 0;
        int64_t from = p.prefix ? prefix : bound(fa), take = kPrefixStart * (int64_t)n;  // in entries
        while (from < m) {
            int64_t to;
            if (p.prefix) {
                to = prefix_end(from, take, m);
                take *= kPrefixGrowth;
            } else {
                g = std::min<int64_t>(S, g + step);
                to = bound(g);
                step *= kSuperGrowth;
            }
            if (lds_bits)
                TIMED(kPhaseHook, launch_filter_bits(u, v, from, to, pi, n, ctrl, bits, p.halve,
                                                     p.symmetric, s));
            else if (hot)
                TIMED(kPhaseHook, launch_ahook_hot(u, v, from, to, pi, n, ctrl, bits,
                                                   fb.hot_tags, fb.hot_vals, p.ept, p.hot_slots,
                                                   p.halve, p.symmetric, s));
            else if (vhot)
                TIMED(kPhaseHook, launch_filter_vertex(u, v, from, to, pi, n, ctrl, bits, fb.vtab,
                                                       p.halve, p.symmetric, s));
            else
                TIMED(kPhaseHook, launch_ahook(u, v, from, to, pi, n, ctrl, bits,
                                               p.block, p.ept, p.coherent, p.halve, p.symmetric, s));
            // A giant that the first part was too short for (uniform random
            // lists need ~n / 2 entries) is looked for again after the next two.
            if (p.auto_filter && to < m && ++again <= 2)
                TIMED(kPhaseOther, launch_sample_giant(u, m, pi, n, ctrl, s, true));
            if (to < m && !p.coherent) {
                // Compress, bitmap refresh and hot-word refresh in one pass
                TIMED(kPhaseCompress, launch_mj_bitmap(pi, n, ctrl, bits, hot ? fb.hot_tags : nullptr,
                                                       fb.hot_vals, p.hot_slots,
                                                       vhot ? fb.vtab : nullptr, s));
            } else {
                TIMED(kPhaseCompress, launch_mj(pi, n, p.coherent, s, to < m ? Post{} : post));
                if (to < m) TIMED(kPhaseOther, launch_bitmap(pi, n, ctrl, bits, s));
            }
            ++hooks;
            ++jumps;
            from = to;
        }
    }
    if (st) {
        st->hook_launches += hooks;
        st->compress_launches += jumps;
    }
    return CC_OK;
}

// Hybrid plan: one atomic-free Hook round (Fig. 2) over all entries, in
// which each workgroup first joins its chunk of entries in an LDS window
// (launch_hook_window), then a pass over all entries that hooks the ones
// still active for good (Fig. 3), and a final Multi-Jump.  A fixed launch
// sequence without a host read; what depends on the input is decided on the
// device by win_far, which exceeds far_limit when more than a quarter of the
// entries (or a whole chunk) were hooked outside the windows.
//
// Short lists: Multi-Jump, and where there is no locality up to kHybridRounds more
// atomic-free rounds (each round leaves about a sixteenth of the roots, so
// that the last pass joins few; up to kHybridRoundsMaxN vertices, above which
// a round's gathers cost more than the compare-and-swaps it saves), then the
// contracting hook over all entries.  Long lists with locality instead
// compact the entries whose parents differ into pairs and hook those: an
// entry with equal parents is inside one tree, a kept pair is a valid climb
// start, and few entries are left, so no Multi-Jump runs first (4096^2 grid:
// 318 us against 352 with the contracting hook).
int32_t enqueue_hybrid(int32_t n, const int32_t* u, const int32_t* v, int64_t m, int32_t* pi,
                       const Plan& p, char* ws, const Layout& L, hipStream_t s, Timer& tm,
                       cc_stats* st, Ctrl* host, bool init = true) {
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws);
    const int grid_cap = device_cu_count() * 8;
    const uint32_t far_limit = (uint32_t)(m / 8);  // win_far counts pairs of entries
    const uint32_t* far = &ctrl->win_far;
    const bool longer = p.frontier;
    // Uniform lists of fewer entries than vertices have no large component; on
    // denser lists one round more leaves few enough roots (uniform, one and two
    // rounds: n = 300,000, m = 1.95 M 131 and 147 us, n = 100,000, m = 750,000 82
    // and 87, but n = 200,000, m = 1.1 M 119 and 112, n = 100,000, m = 300,000 82
    // and 69; R-MAT 18, m = 1.7 M 108 and 126), and on long ones a second round's
    // gathers cost more than it saves (n = 2^20, m = 4.4 M 357 and 393, none 404;
    // R-MAT 20, m = 5.2 M 288 and 340).
    const int rounds = n > kHybridRoundsMaxN || 10 * m < 11 * (int64_t)n ? 0
                       : longer || m >= 6 * (int64_t)n                   ? 1
                                                                         : kHybridRounds;
    if (init) TIMED(kPhaseOther, launch_init(pi, n, ctrl, s));
    TIMED(kPhaseHook, launch_hook_window(u, v, m, pi, n, ctrl, far_limit, s));
    TIMED(kPhaseCompress, launch_mj1(pi, n, longer ? far : nullptr, s, true, far_limit));
    for (int r = 0; r < rounds; ++r) {
        TIMED(kPhaseHook, launch_hook_prefix(u, v, m, pi, n, s, far, far_limit));
        TIMED(kPhaseCompress, launch_mj1(pi, n, far, s, true, far_limit));
    }
    if (longer) {
        int2* F = reinterpret_cast<int2*>(ws + L.f0);
        // one workgroup per tile: 2,048 of them striding over 4096^2's 5,733 end
        // unevenly (56.0 us, 54.5 now)
        TIMED(kPhaseHook, launch_compact(1, u, v, m, F, F, L.cap, pi, n, ctrl, 0xffffffffu, p.block,
                                         p.ept, INT_MAX, s, far, far_limit));
        TIMED(kPhaseHook, launch_ahook_pairs(F, &ctrl->count[1], L.cap, pi, p.halve, grid_cap, s));
    }
    TIMED(kPhaseHook, launch_hook_contract(u, v, 0, m, pi, n, ctrl, p.halve, s,
                                           longer ? far : nullptr, far_limit));
    TIMED(kPhaseCompress, launch_mj1(pi, n, nullptr, s, false, 0, Post{ctrl, host}));
    if (st) {
        st->hook_launches += 2 + rounds + (longer ? 2 : 0);
        st->compress_launches += 2 + rounds;
    }
    return CC_OK;
}

// The atomic-free Hook in blocks of K = rounds_per_check rounds, the host
// reading the control block after each block.  With `graph`, each block's
// launches (block b: rounds bK+1 .. bK+K; block 0 also the init) are
// captured once per (arrays, sizes, plan, b) and replayed.
int32_t solve_plain(int32_t n, const int32_t* u, const int32_t* v, int64_t m, int32_t* pi,
                    const Plan& p, char* ws, const Layout& L, hipStream_t s, PoolEntry* pe,
                    Ctrl* hctrl, bool use_graph, Timer& tm, cc_stats* st, int64_t* rounds_run) {
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws);
    int2* F0 = reinterpret_cast<int2*>(ws + L.f0);
    int2* F1 = reinterpret_cast<int2*>(ws + L.f1);
    const int grid_cap = device_cu_count() * 8;
    const int K = p.rounds_per_check;
    auto enqueue_block = [&](int64_t b) -> int32_t {
        if (b == 0) TIMED(kPhaseOther, launch_init(pi, n, ctrl, s));
        for (int k = 0; k < K; ++k) {
            const int64_t r = b * K + k + 1;
            // sources and sizes are chosen on the device (round_src); the
            // grid covers the capacity and loops over what is there
            const int64_t work = (r == 1) ? m : L.cap;
            TIMED(kPhaseHook, launch_hook_plain((int)r, u, v, work, F0, F1, pi, n, ctrl, p.block,
                                                p.ept, grid_cap, s));
            if (r == 1)  // the round leaves chains
                TIMED(kPhaseCompress, launch_mj_deep(pi, n, s));
            else
                TIMED(kPhaseCompress, launch_mj1(pi, n, &ctrl->count[(r - 1) & 1], s, true));
            TIMED(kPhaseHook, launch_compact((int)r, u, v, work, F0, F1, L.cap, pi, n, ctrl,
                                             p.tau, p.block, p.ept, grid_cap, s));
        }
        return CC_OK;
    };
    int64_t r = 0;
    int hooks = 0, jumps = 0;
    for (int64_t b = 0;; ++b) {
        int32_t rc;
        if (use_graph) {
            KeyHash k;
            k.add(n).add(m).add(u).add(v).add(pi).add(ws).add(s).add(p.block).add(p.ept)
                .add(p.tau).add(K).add(b);
            rc = run_graph(pe, k.h, s, [&]() { return enqueue_block(b); });
        } else {
            rc = enqueue_block(b);
        }
        if (rc != CC_OK) return rc;
        r += K;
        hooks += 2 * K;
        jumps += K;
        rc = finish(s, ctrl, hctrl, st);
        if (rc != CC_OK) return rc;
        if (hctrl->status) break;  // reported by the caller
        if (hctrl->count[r & 1] == 0) break;
        if (r >= p.max_rounds) {
            *rounds_run = r;
            if (st) {
                st->hook_launches += hooks;
                st->compress_launches += jumps;
            }
            return fail(CC_ERR_NOCONVERGE, "atomic-free Hook did not converge within max_rounds");
        }
    }
    *rounds_run = r;
    if (st) {
        st->hook_launches += hooks;
        st->compress_launches += jumps;
    }
    return CC_OK;
}

// Fig. 1 exactly as the paper's baseline runs it: every Hook pass covers all
// entries, and the host reads a device "changed" flag after every launch
// (the CPU-GPU round trips that Section 1 sets out to remove).  Compress is
// either repeated single-level Jump launches (Fig. 2) or one Multi-Jump.
int32_t solve_host_loop(int32_t n, const int32_t* u, const int32_t* v, int64_t m, int32_t* pi,
                        const Plan& p, char* ws, hipStream_t s, Ctrl* hctrl, Timer& tm,
                        cc_stats* st) {
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws);
    TIMED(kPhaseOther, launch_init(pi, n, ctrl, s));
    int64_t rounds = 0;
    int hooks = 0, jumps = 0;
    while (true) {
        ++rounds;
        HIPCHK(hipMemsetAsync(&ctrl->hook_changed, 0, 4, s));
        TIMED(kPhaseHook, launch_hook_flag(u, v, m, pi, n, ctrl, p.block, p.ept, s));
        ++hooks;
        int32_t rc = finish(s, ctrl, hctrl, st);
        if (rc != CC_OK) return rc;
        if (hctrl->status) break;
        const bool hooked = hctrl->hook_changed != 0;
        if (p.host_loop == CC_HOST_LOOP_MULTIJUMP) {
            TIMED(kPhaseCompress, launch_mj1(pi, n, nullptr, s, true));
            ++jumps;
        } else {
            while (true) {
                HIPCHK(hipMemsetAsync(&ctrl->jump_changed, 0, 4, s));
                TIMED(kPhaseCompress, launch_jump(pi, n, ctrl, s));
                ++jumps;
                rc = finish(s, ctrl, hctrl, st);
                if (rc != CC_OK) return rc;
                if (!hctrl->jump_changed) break;
            }
        }
        if (!hooked) break;
        if (rounds >= p.max_rounds) {
            if (st) {
                st->rounds = (int32_t)rounds;
                st->hook_launches += hooks;
                st->compress_launches += jumps;
            }
            return fail(CC_ERR_NOCONVERGE, "Hook did not converge within max_rounds");
        }
    }
    int32_t rc = finish(s, ctrl, hctrl, st);
    if (rc != CC_OK) return rc;
    if (st) {
        st->rounds = (int32_t)rounds;
        st->hook_launches += hooks;
        st->compress_launches += jumps;
    }
    return CC_OK;
}

int32_t check_args(int32_t n, const int32_t* u, const int32_t* v, int64_t m, const int32_t* out) {
    if (n < 0) return fail(CC_ERR_ARG, "n < 0");
    if (m < 0) return fail(CC_ERR_ARG, "m < 0");
    if (m > 0 && (!u || !v)) return fail(CC_ERR_ARG, "null edge array with m > 0");
    if (n > 0 && !out) return fail(CC_ERR_ARG, "null out_label with n > 0");
    return CC_OK;
}


// Enqueues the solve of one graph with plan p on s into the workspace ws
// (laid out by L) and waits for it; `hctrl` receives the control block.
// `pe` (nullable) supplies the captured launch sequences of p.graph and the
// status slot of p.no_sync; without it neither is used (the caller has
// rejected both).
int32_t run_solve(int32_t n, const int32_t* u, const int32_t* v, int64_t m, int32_t* out,
                  const Plan& p, const Layout& L, char* ws, Ctrl* hctrl, PoolEntry* pe,
                  hipStream_t s, cc_stats* st) {
    int32_t rc = CC_OK;
    Timer tm;
    tm.on = p.profile;
    tm.s = s;
    int64_t rounds = 0;
    const bool use_graph = p.graph && s != nullptr && !p.profile && pe != nullptr;
    if (p.lds_single) {
        // one launch, which reports the status straight to pinned host memory
        // where the call waits for it
        HIPCHK(prepare_batch_lds());
        const GraphDesc d = {u, v, out, m, n, lds_auto_segments(m, n, true)};
        Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws);
        const bool direct = pe && !p.no_sync;
        TIMED(kPhaseHook, launch_single_lds(d, nullptr, direct ? &hctrl->status : &ctrl->status, p.halve, s));
        if (st) st->hook_launches = 1;
        if (p.no_sync && pe) return post_async(pe, s, ctrl);
        if (!direct)
            HIPCHK(hipMemcpyAsync(&hctrl->status, &ctrl->status, 4, hipMemcpyDeviceToHost, s));
        HIPCHK(hipStreamSynchronize(s));
        tm.collect(st);
        if (st) {
            st->host_syncs = 1;
            st->rounds = 1;
        }
        const int32_t status = *(volatile int32_t*)&hctrl->status;
        if (status & kStatusRange) return fail(CC_ERR_RANGE, "edge endpoint outside [0, n)");
        return CC_OK;
    }
    if (p.hook == CC_HOOK_ATOMIC || p.hook == CC_HOOK_HYBRID) {
        // fixed launch sequences: no host read until the end
        // (the pool's control blocks are pinned: the last launch posts there)
        Ctrl* host = pe && !p.no_sync ? hctrl : nullptr;
        auto enqueue = [&](cc_stats* sx) {
            if (p.hook == CC_HOOK_HYBRID)
                return enqueue_hybrid(n, u, v, m, out, p, ws, L, s, tm, sx, host);
            return enqueue_atomic(n, u, v, m, out, p, reinterpret_cast<Ctrl*>(ws),
                                  filter_bufs(ws, L), s, tm, sx, host);
        };
        if (use_graph) {
            KeyHash k;
            k.add(n).add(m).add(u).add(v).add(out).add(ws).add(s).add(host).add(p.hook).add(p.segments)
                .add(p.filter).add(p.filter_after).add(p.block).add(p.ept).add(p.coherent)
                .add(p.hot).add(p.hot_slots).add(p.lds_bits).add(p.auto_filter).add(p.prefix).add(p.halve)
                .add(p.symmetric);
            rc = run_graph(pe, k.h, s, [&]() { return enqueue(st); });
        } else {
            rc = enqueue(st);
        }
        if (rc == CC_OK && p.no_sync && pe) {
            rc = post_async(pe, s, reinterpret_cast<const Ctrl*>(ws));
            if (st) st->giant_label = -1;  // not known without a synchronisation
            return rc;
        }
        if (rc == CC_OK) rc = finish(s, reinterpret_cast<Ctrl*>(ws), hctrl, st, host != nullptr);
    } else if (p.host_loop != CC_HOST_LOOP_OFF) {
        rc = solve_host_loop(n, u, v, m, out, p, ws, s, hctrl, tm, st);
    } else {
        rc = solve_plain(n, u, v, m, out, p, ws, L, s, pe, hctrl, use_graph, tm, st, &rounds);
    }
    if (rc != CC_OK && rc != CC_ERR_NOCONVERGE) return rc;
    const Ctrl& c = *hctrl;
    tm.collect(st);
    if (st) {
        st->filter_used = (p.filter == CC_FILTER_GIANT && c.filter_on) ? 1 : 0;
        st->giant_label = st->filter_used ? c.giant : -1;
        if (p.hook == CC_HOOK_PLAIN && p.host_loop == CC_HOST_LOOP_OFF) {
            st->rounds = c.rounds;
            st->active_edges = c.active_round1;
        }
    }
    if (c.status & kStatusRange) return fail(CC_ERR_RANGE, "edge endpoint outside [0, n)");
    if (c.status & kStatusOverflow) return fail(CC_ERR_NOMEM, "frontier capacity exceeded");
    return rc;
}

void init_stats(cc_stats* st, const Plan& p, int32_t n, int64_t m) {
    if (!st) return;
    std::memset(st, 0, sizeof *st);
    st->hook = p.hook;
    st->segments = p.hook == CC_HOOK_ATOMIC ? p.segments : 0;
    if (p.prefix) {  // the launches that the rest of the list is taken in
        st->segments = 0;
        for (int64_t from = std::min<int64_t>(m, n) & ~int64_t(3), take = kPrefixStart * (int64_t)n; from < m;
             take *= kPrefixGrowth) {
            from = prefix_end(from, take, m);
            ++st->segments;
        }
    }
    st->giant_label = -1;
}

}  // namespace

int32_t labels_impl(int32_t n, const int32_t* u, const int32_t* v, int64_t m, int32_t* out,
                    const cc_options* opts, void* workspace, size_t ws_bytes, hipStream_t s,
                    cc_stats* st) {
    int32_t rc = check_args(n, u, v, m, out);
    if (rc != CC_OK) return rc;
    Plan p;
    rc = make_plan(n, m, opts, p);
    if (rc != CC_OK) return rc;
    init_stats(st, p, n, m);
    if (n == 0) {
        if (m > 0) return fail(CC_ERR_RANGE, "edge endpoint outside [0, n) (n == 0)");
        return CC_OK;
    }
    const Layout L = layout(n, m, p);
    PoolEntry* pe = pool_entry(s);
    std::lock_guard<std::mutex> lk(pe->mu);
    rc = ensure_host(pe);
    if (rc != CC_OK) return rc;
    char* ws;
    if (workspace) {
        if (ws_bytes < L.total) return fail(CC_ERR_NOMEM, "workspace smaller than cc_workspace_bytes()");
        if ((uintptr_t)workspace & 255) return fail(CC_ERR_ARG, "workspace must be 256-byte aligned");
        ws = static_cast<char*>(workspace);
    } else {
        rc = ensure_dev(pe, L.total);
        if (rc != CC_OK) return rc;
        ws = static_cast<char*>(pe->dev);
    }
    return run_solve(n, u, v, m, out, p, L, ws, pe->host_ctrl, pe, s, st);
}

// ---------------------------------------------------------------------- no-allocation solve
// cc_labels_noalloc: the solve of cc_labels_ex with its workspace taken from
// a fixed device array instead of the pool or the caller, for callers that
// must not allocate.  One array per device (each GPU the library runs on
// holds its own copy until the process ends); host code reaches it only
// through the address hipGetSymbolAddress returns for the current device.
namespace {

static __device__ __align__(256) char scratch[CC_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu[kMaxDevices];   // one call at a time per device
char* g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch`, guarded as above

}  // namespace

int32_t labels_noalloc_impl(int32_t n, const int32_t* u, const int32_t* v, int64_t m,
                            int32_t* out, const cc_options* opts, hipStream_t s, cc_stats* st) {
    int32_t rc = check_args(n, u, v, m, out);
    if (rc != CC_OK) return rc;
    if (opts && (opts->graph != 0 || opts->no_sync != 0 || opts->profile != 0))
        return fail(CC_ERR_ARG, "cc_labels_noalloc: graph, no_sync and profile must be 0");
    Plan p;
    rc = make_plan(n, m, opts, p);
    if (rc != CC_OK) return rc;
    Layout L = layout(n, m, p);
    if (L.total > (size_t)CC_NOALLOC_SCRATCH_BYTES && (!opts || opts->hook == CC_HOOK_AUTO)) {
        // the automatic choice falls back to plans whose workspace fits: the
        // Atomic-Hook (no frontier), then without the giant filter (256 bytes)
        cc_options o;
        if (opts) o = *opts;
        else cc_options_init(&o);
        o.hook = CC_HOOK_ATOMIC;
        rc = make_plan(n, m, &o, p);
        if (rc != CC_OK) return rc;
        L = layout(n, m, p);
        if (L.total > (size_t)CC_NOALLOC_SCRATCH_BYTES) {
            o.filter = CC_FILTER_OFF;
            rc = make_plan(n, m, &o, p);
            if (rc != CC_OK) return rc;
            L = layout(n, m, p);
        }
    }
    if (L.total > (size_t)CC_NOALLOC_SCRATCH_BYTES)
        return fail(CC_ERR_NOMEM, "cc_labels_noalloc: the plan needs " + std::to_string(L.total) +
                                      " bytes of workspace; the fixed buffer holds " +
                                      std::to_string((size_t)CC_NOALLOC_SCRATCH_BYTES) +
                                      " (use cc_labels_ex, or the automatic hook)");
    init_stats(st, p, n, m);
    if (n == 0) {
        if (m > 0) return fail(CC_ERR_RANGE, "edge endpoint outside [0, n) (n == 0)");
        return CC_OK;
    }
    int dev = 0;
    HIPCHK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(CC_ERR_ARG, "device index out of range");
    std::lock_guard<std::mutex> lk(g_scratch_mu[dev]);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        HIPCHK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr || ((uintptr_t)ptr & 255))
            return fail(CC_ERR_HIP, "cc_labels_noalloc: unusable address of the fixed buffer");
        g_scratch_ptr[dev] = static_cast<char*>(ptr);
    }
    // every kernel of the solve writes the workspace words it reads (the
    // control block is reset by the init kernel), so the previous call's
    // contents need no clearing
    Ctrl hctrl;
    return run_solve(n, u, v, m, out, p, L, g_scratch_ptr[dev], &hctrl, nullptr, s, st);
}

// ---------------------------------------------------------------------- streamed solve
// Edges in host memory, larger than one wants to (or can) hold in HBM.  The
// Atomic-Hook reads every entry exactly once, so the list is cut into chunks
// that are copied host-to-device on a copy stream into two staging buffers
// (double buffering: chunk i+1 is copied while chunk i is hooked) and hooked
// on the caller's stream, each chunk followed by a Multi-Jump (Fig. 4 with one
// segment per chunk).  With the giant filter, the first chunk's Compress is
// followed by the sample and the bitmap, which later chunks use and which is
// rebuilt after each chunk's Compress.  Only pi, the bitmap and the staging
// buffers (2 x 2 x chunk x 4 bytes) occupy device memory.
int32_t stream_impl(int32_t n, const int32_t* hu, const int32_t* hv, int64_t m, int32_t* out,
                    int64_t chunk, const cc_options* opts, hipStream_t s, cc_stats* st) {
    int32_t rc = check_args(n, hu, hv, m, out);
    if (rc != CC_OK) return rc;
    if (chunk < 0) return fail(CC_ERR_ARG, "chunk_entries < 0");
    if (chunk == 0) chunk = int64_t(1) << 24;
    chunk = std::max<int64_t>(4, chunk & ~int64_t(3));
    if (opts && opts->hook == CC_HOOK_PLAIN)
        return fail(CC_ERR_ARG, "streamed solves use the Atomic-Hook (each entry is read once)");
    if (opts && opts->no_sync)
        return fail(CC_ERR_ARG, "cc_options.no_sync is for cc_labels_ex and cc_labels_csr only");
    Plan p;
    rc = make_plan(n, m, opts, p, kInputAtomicOnly);
    if (rc != CC_OK) return rc;
    // Giant filter: as asked, or (auto) for dense lists that span several chunks.
    const int32_t fopt = opts ? opts->filter : CC_FILTER_AUTO;
    const bool filter = fopt == CC_FILTER_GIANT ||
                        (fopt == CC_FILTER_AUTO && m >= 8 * (int64_t)n && m > chunk);
    if (st) {
        std::memset(st, 0, sizeof *st);
        st->hook = CC_HOOK_ATOMIC;
        st->giant_label = -1;
    }
    if (n == 0) {
        if (m > 0) return fail(CC_ERR_RANGE, "edge endpoint outside [0, n) (n == 0)");
        return CC_OK;
    }
    const int64_t chunks = std::max<int64_t>(1, (m + chunk - 1) / chunk);
    const size_t bits_bytes = filter ? align256(((size_t)n + 31) / 32 * 4) : 0;
    const size_t stage = align256((size_t)chunk * 4);
    const size_t total = 256 + bits_bytes + 4 * stage;
    PoolEntry* pe = pool_entry(s);
    std::lock_guard<std::mutex> lk(pe->mu);
    rc = ensure_host(pe);
    if (rc != CC_OK) return rc;
    rc = ensure_dev(pe, total);
    if (rc != CC_OK) return rc;
    if (!pe->copy_stream) HIPCHK(hipStreamCreateWithFlags(&pe->copy_stream, hipStreamNonBlocking));
    for (int i = 0; i < 2; ++i) {
        if (!pe->copied[i]) HIPCHK(hipEventCreateWithFlags(&pe->copied[i], hipEventDisableTiming));
        if (!pe->consumed[i]) HIPCHK(hipEventCreateWithFlags(&pe->consumed[i], hipEventDisableTiming));
    }
    char* ws = static_cast<char*>(pe->dev);
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws);
    uint32_t* bits = filter ? reinterpret_cast<uint32_t*>(ws + 256) : nullptr;
    int32_t* su[2] = {reinterpret_cast<int32_t*>(ws + 256 + bits_bytes),
                      reinterpret_cast<int32_t*>(ws + 256 + bits_bytes + stage)};
    int32_t* sv[2] = {reinterpret_cast<int32_t*>(ws + 256 + bits_bytes + 2 * stage),
                      reinterpret_cast<int32_t*>(ws + 256 + bits_bytes + 3 * stage)};
    hipStream_t cs = pe->copy_stream;
    HIPCHK(launch_init(out, n, ctrl, s));
    // The copy stream must not overwrite a staging buffer before the solve
    // stream is done with it, nor start before init is queued (ordering only).
    HIPCHK(hipEventRecord(pe->consumed[0], s));
    HIPCHK(hipEventRecord(pe->consumed[1], s));
    int hooks = 0, jumps = 0;
    for (int64_t i = 0; i < chunks; ++i) {
        const int b = (int)(i & 1);
        const int64_t e0 = i * chunk, len = std::min<int64_t>(chunk, m - e0);
        HIPCHK(hipStreamWaitEvent(cs, pe->consumed[b], 0));
        if (len > 0) {
            HIPCHK(hipMemcpyAsync(su[b], hu + e0, (size_t)len * 4, hipMemcpyHostToDevice, cs));
            HIPCHK(hipMemcpyAsync(sv[b], hv + e0, (size_t)len * 4, hipMemcpyHostToDevice, cs));
        }
        HIPCHK(hipEventRecord(pe->copied[b], cs));
        HIPCHK(hipStreamWaitEvent(s, pe->copied[b], 0));
        const bool filtered = filter && i > 0;
        HIPCHK(launch_ahook(su[b], sv[b], 0, len, out, n, ctrl, filtered ? bits : nullptr, p.block,
                            p.ept, p.coherent, p.halve, p.symmetric, s));
        HIPCHK(launch_mj(out, n, p.coherent, s));
        ++hooks;
        ++jumps;
        if (filter && i == 0) HIPCHK(launch_sample_giant(su[b], len, out, n, ctrl, s));
        if (filter && i + 1 < chunks) HIPCHK(launch_bitmap(out, n, ctrl, bits, s));
        HIPCHK(hipEventRecord(pe->consumed[b], s));
    }
    rc = finish(s, ctrl, pe->host_ctrl, st);
    if (rc != CC_OK) return rc;
    if (st) {
        st->segments = (int32_t)chunks;
        st->hook_launches = hooks;
        st->compress_launches = jumps;
        st->filter_used = (filter && pe->host_ctrl->filter_on) ? 1 : 0;
        st->giant_label = st->filter_used ? pe->host_ctrl->giant : -1;
    }
    if (pe->host_ctrl->status & kStatusRange) return fail(CC_ERR_RANGE, "edge endpoint outside [0, n)");
    return CC_OK;
}

// ---------------------------------------------------------------------- CSR input
// The first endpoint of an entry is its row.  The hybrid plan writes the row
// of every entry once (4 bytes per entry written and read) and is then the
// pair-list plan; a second set of kernels that find rows on the fly was slower
// (2048^2 grid: 346 us, 200 now) and only went beyond 2^22 entries (50 x 4,000
// grid: 354, 75 now).
//
// The automatic filtered plan hooks two neighbours of every row first: the
// first one in the initial tree, the last one by an atomic-free round and a
// contracting hook.  That finds the giant whatever the order of the rows (of
// R-MAT 20's 646,362 vertices with an edge all but 200 or so are in it), so
// one filtered pass over all entries follows: R-MAT 20, 2^25 entries 147 us
// against 466 for growing segments of rows, whose first ones contend for the
// hubs; a split pass with a bitmap refresh in between 193.
//
// The smallest lists are solved by one workgroup in LDS.  With options of its own
// (segments, filter_after, filter) the Atomic-Hook runs segments of the col[]
// array, each followed by a Multi-Jump; with the giant filter the growing
// super-segments of enqueue_atomic.
int32_t csr_impl(int32_t n, const int64_t* row_ptr, const int32_t* col, int64_t m, int32_t* out,
                 const cc_options* opts, hipStream_t s, cc_stats* st) {
    if (n < 0 || m < 0) return fail(CC_ERR_ARG, "n < 0 or m < 0");
    if (!row_ptr) return fail(CC_ERR_ARG, "null row_ptr");
    if (m > 0 && !col) return fail(CC_ERR_ARG, "null col with m > 0");
    if (n > 0 && !out) return fail(CC_ERR_ARG, "null out_label with n > 0");
    if (opts && opts->hook == CC_HOOK_PLAIN)
        return fail(CC_ERR_ARG, "CSR input uses the Atomic-Hook or the hybrid plan");
    Plan p;
    int32_t rc = make_plan(n, m, opts, p, kInputCsr);
    if (rc != CC_OK) return rc;
    if (st) {
        std::memset(st, 0, sizeof *st);
        st->hook = p.hook;
        st->giant_label = -1;
    }
    if (n == 0) {
        if (m > 0) return fail(CC_ERR_RANGE, "entries in a graph with no vertices");
        return CC_OK;
    }
    PoolEntry* pe = pool_entry(s);
    std::lock_guard<std::mutex> lk(pe->mu);
    rc = ensure_host(pe);
    if (rc != CC_OK) return rc;
    bool tiled = p.hook == CC_HOOK_HYBRID || p.auto_filter;
    // Workspace: [control block, bitmap or hybrid frontier][first row of each
    // tile][row of each entry (hybrid) or the sampled pairs (filtered plan)]
    const Layout L = layout(n, m, p);
    const size_t bits_bytes = align256(((size_t)n + 31) / 32 * 4);
    const size_t base = p.hook == CC_HOOK_HYBRID ? L.total : 256 + bits_bytes;
    const size_t tile_bytes = align256(((size_t)m / kCsrTile + 2) * 4);
    const size_t row_bytes = align256((p.hook == CC_HOOK_HYBRID ? (size_t)m : (size_t)n) * 4);
    if (tiled) {
        const size_t need = base + tile_bytes + (p.auto_filter ? 2 : 1) * row_bytes;
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (pe->bytes < need && hipStreamIsCapturing(s, &cap) != hipSuccess) {
            (void)hipGetLastError();
            cap = hipStreamCaptureStatusNone;
        }
        const bool capturing = cap != hipStreamCaptureStatusNone;
        rc = capturing ? fail(CC_ERR_NOMEM, "no memory for the plan inside a stream capture")
                       : ensure_dev(pe, need);
        if (rc != CC_OK) {
            // No memory for it, or none to be had inside a capture: an explicit
            // plan is refused; the automatic one falls back to the filtered
            // segments, which need the bitmap, or to unfiltered ones, which
            // need the control block only (R-MAT 20, 2^25 entries, inside a
            // capture: 457 us, 969 unfiltered).
            (void)hipGetLastError();
            if (opts && opts->hook != CC_HOOK_AUTO) return rc;
            tiled = false;
            const bool fits = capturing ? pe->bytes >= 256 + bits_bytes
                                        : ensure_dev(pe, 256 + bits_bytes) == CC_OK;
            (void)hipGetLastError();
            p.lds_single = false;
            if (!p.auto_filter || !fits) {
                p.filter = CC_FILTER_OFF;
                p.segments = (int)std::min<int64_t>(std::min<int64_t>(1 << 20, round_ratio(m, n)), m / 4 + 1);
            }
            p.auto_filter = false;
            p.hook = CC_HOOK_ATOMIC;
        }
    }
    const bool filter = p.filter == CC_FILTER_GIANT;
    rc = ensure_dev(pe, 256 + (filter ? bits_bytes : 0));
    if (rc != CC_OK) return rc;
    if (st) {
        st->hook = p.hook;
        st->segments = p.hook != CC_HOOK_ATOMIC ? 0 : p.auto_filter ? 1 : p.segments;
    }
    char* ws = static_cast<char*>(pe->dev);
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws);
    uint32_t* bits = filter ? reinterpret_cast<uint32_t*>(ws + 256) : nullptr;
    int32_t* tile_row = tiled ? reinterpret_cast<int32_t*>(ws + base) : nullptr;
    int32_t* rows = tiled ? reinterpret_cast<int32_t*>(ws + base + tile_bytes) : nullptr;
    const int S = p.segments;
    auto bound = [&](int64_t i) -> int64_t { return i >= S ? m : segment_start(m, i, S); };
    Timer tm;
    tm.on = p.profile;
    tm.s = s;
    const Post post = {ctrl, p.no_sync ? nullptr : pe->host_ctrl};
    int hooks = 0, jumps = 0;
    if (tiled) {
        TIMED(kPhaseOther, launch_init(out, 1, ctrl, s));
    } else {
        TIMED(kPhaseOther, launch_init(out, n, ctrl, s));
        TIMED(kPhaseOther, launch_csr_check(row_ptr, n, m, ctrl, s));
    }
    if (p.lds_single) {
        // The rows of all entries, then one workgroup in LDS: three launches
        // against the hybrid plan's ten (path of 30 vertices 35 us against 84,
        // of 5,000 63 against 171, star of 20,000 44 against 96; 7 n entries
        // of 20,000 vertices 95 against 89).
        TIMED(kPhaseOther, launch_csr_prep(row_ptr, col, n, m, ctrl, out, tile_row, nullptr, nullptr, s));
        TIMED(kPhaseOther, launch_csr_expand(row_ptr, tile_row, n, m, rows, s));
        HIPCHK(prepare_batch_lds());
        const GraphDesc d = {rows, col, out, m, n, lds_auto_segments(m, n, true)};
        TIMED(kPhaseHook, launch_single_lds(d, &ctrl->status, p.no_sync ? &ctrl->status : &pe->host_ctrl->status,
                                            p.halve, s));
        hooks = 1;
    } else if (p.hook == CC_HOOK_HYBRID) {
        TIMED(kPhaseOther, launch_csr_prep(row_ptr, col, n, m, ctrl, out, tile_row, nullptr, nullptr, s));
        TIMED(kPhaseOther, launch_csr_expand(row_ptr, tile_row, n, m, rows, s));
        cc_stats counts = {};
        rc = enqueue_hybrid(n, rows, col, m, out, p, ws, L, s, tm, &counts, post.host, /*init=*/false);
        if (rc != CC_OK) return rc;
        hooks = counts.hook_launches;
        jumps = counts.compress_launches;
    } else if (p.auto_filter) {
        int32_t* sv = rows + row_bytes / 4;
        TIMED(kPhaseOther, launch_csr_prep(row_ptr, col, n, m, ctrl, out, tile_row, rows, sv, s));
        TIMED(kPhaseCompress, launch_mj_deep(out, n, s));
        TIMED(kPhaseHook, launch_hook_prefix(rows, sv, n, out, n, s));
        TIMED(kPhaseCompress, launch_mj1(out, n, nullptr, s, true));
        TIMED(kPhaseHook, launch_hook_contract(rows, sv, 0, n, out, n, ctrl, p.halve, s));
        TIMED(kPhaseCompress, launch_mj1(out, n, nullptr, s, false));
        TIMED(kPhaseOther, launch_sample_giant(col, m, out, n, ctrl, s));
        TIMED(kPhaseOther, launch_bitmap(out, n, ctrl, bits, s));
        TIMED(kPhaseHook, launch_csr_filter(row_ptr, col, n, m, tile_row, out, ctrl, bits, p.halve,
                                            p.symmetric, s));
        TIMED(kPhaseCompress, launch_mj(out, n, false, s, post));
        hooks = 3;
        jumps = 4;
    } else if (!filter) {
        for (int i = 0; i < S; ++i) {
            TIMED(kPhaseHook, launch_ahook_csr(row_ptr, col, n, bound(i), bound(i + 1), out, ctrl,
                                               nullptr, p.symmetric, p.halve, s));
            TIMED(kPhaseCompress, launch_mj(out, n, false, s, i + 1 == S ? post : Post{}));
            ++hooks;
            ++jumps;
        }
    } else {
        const int fa = p.filter_after;
        for (int i = 0; i < fa; ++i) {
            TIMED(kPhaseHook, launch_ahook_csr(row_ptr, col, n, bound(i), bound(i + 1), out, ctrl,
                                               nullptr, p.symmetric, p.halve, s));
            TIMED(kPhaseCompress, launch_mj(out, n, false, s));
            ++hooks;
            ++jumps;
        }
        // endpoints sampled from col[] (the second endpoints of the entries)
        TIMED(kPhaseOther, launch_sample_giant(col, m, out, n, ctrl, s));
        TIMED(kPhaseOther, launch_bitmap(out, n, ctrl, bits, s));
        int64_t g = fa, step = kSuperStart * fa;
        while (g < S) {
            const int64_t h = std::min<int64_t>(S, g + step);
            TIMED(kPhaseHook, launch_ahook_csr(row_ptr, col, n, bound(g), bound(h), out, ctrl, bits,
                                               p.symmetric, p.halve, s));
            TIMED(kPhaseCompress, launch_mj(out, n, false, s, h < S ? Post{} : post));
            ++hooks;
            ++jumps;
            if (h < S) TIMED(kPhaseOther, launch_bitmap(out, n, ctrl, bits, s));
            g = h;
            step *= kSuperGrowth;
        }
    }
    if (p.no_sync) {
        if (st) {
            st->hook_launches = hooks;
            st->compress_launches = jumps;
        }
        return post_async(pe, s, ctrl);
    }
    rc = finish(s, ctrl, pe->host_ctrl, st, true);
    if (rc != CC_OK) return rc;
    tm.collect(st);
    if (st) {
        st->hook_launches = hooks;
        st->compress_launches = jumps;
        st->filter_used = (filter && pe->host_ctrl->filter_on) ? 1 : 0;
        st->giant_label = st->filter_used ? pe->host_ctrl->giant : -1;
    }
    if (pe->host_ctrl->status & kStatusRange)
        return fail(CC_ERR_RANGE, "column id outside [0, n) or malformed row_ptr");
    return CC_OK;
}

size_t workspace_bytes_impl(int32_t n, int64_t m, const cc_options* opts) {
    if (n < 0 || m < 0) return 0;
    Plan p;
    if (make_plan(n, m, opts, p) != CC_OK) return 0;
    return layout(n, m, p).total;
}

// ---------------------------------------------------------------------- graph lists
// Segments of an LDS-solved graph: min(cap, round(m / n)) (at least 1), or
// round(m / n) for cap 0, the default rule for kSegAuto*; small caps by
// comparison, without a division.
int32_t lds_segments(int64_t m, int64_t n, int32_t cap) {
    if (cap < 0) return lds_auto_segments(m, n, cap == kSegAutoFew);
    if (cap > 0 && cap <= 16 && m < (int64_t(1) << 61)) {
        int32_t k = cap;  // round(m / n) >= k  <=>  2m >= (2k - 1) n
        while (k > 1 && 2 * m < (2 * (int64_t)k - 1) * n) --k;
        return k;
    }
    const int32_t r = (int32_t)std::min<int64_t>(int64_t(1) << 20, round_ratio(m, n));
    return cap > 0 ? std::min(r, cap) : r;
}

// How many of the LDS graphs, largest first, a list's solve gives to the
// device-memory path instead.  One workgroup takes ~0.28 us per 1,000 entries
// (n = 65,536, m = 1.3 M: 384 us), and a few graphs with many entries keep the
// launch from ending while the other CUs idle; the device-memory path takes
// them one after the other, ~80 us each.  The count with the least sum of both
// (at most 16 graphs of kListAloneM entries and more).
template <class GraphAt>
int32_t alone_count(const std::vector<int32_t>& small, GraphAt&& graph_at) {
    constexpr double kUsPerEntry = 2.8e-4, kDeviceUs = 80.0;
    if (small.empty() || graph_at(small[0]).m < kListAloneM) return 0;
    double rest = 0;
    for (int32_t g : small) rest += kUsPerEntry / 256 * (double)graph_at(g).m;
    int32_t best = 0;
    double least = 1e30, device = 0;
    for (int32_t k = 0; k <= 16; ++k) {
        const double next = k < (int32_t)small.size() ? kUsPerEntry * (double)graph_at(small[k]).m : 0;
        const double cost = device + std::max(next, rest);
        if (cost < least) {
            least = cost;
            best = k;
        }
        if (k == (int32_t)small.size() || graph_at(small[k]).m < kListAloneM) break;
        device += kDeviceUs;
        rest -= next / 256;
    }
    return best;
}

// The graph-list solve over any graph accessor: graph_at(g) returns graph g
// as a cc_graph (the caller's array, or one computed from batch offsets, so a
// batch never materialises a list).  Small graphs (n <= CC_BATCH_LDS_MAX_N)
// go to one persistent LDS launch whose workgroups take them largest first;
// every larger graph, and the few that alone would prolong that launch
// (alone_count), get a device-memory solve with its own control block: the
// filtered plan where dense, else the hybrid plan without its frontier (R-MAT
// 17, m = 1.05 M: 8 Atomic-Hook segments before).  Everything is enqueued on `s`; the call ends with one
// synchronisation, after which the LDS launch's pinned status word and the
// large graphs' control blocks (posted by their last launches) are read.
template <class GraphAt>
int32_t list_core(int32_t count, GraphAt&& graph_at, const cc_options* opts, hipStream_t s,
                  cc_stats* st, void* workspace, size_t ws_bytes, size_t* ws_needed) {
    if (ws_needed) *ws_needed = 0;
    if (count < 0) return fail(CC_ERR_ARG, "graph count < 0");
    if (opts && opts->no_sync)
        return fail(CC_ERR_ARG, "cc_options.no_sync is for cc_labels_ex and cc_labels_csr only");
    // Per-graph segment count of the LDS solver: min(S, round(m/n)) for a
    // cap S > 0.  Default (S = 0): one or two by lds_auto_segments with path
    // halving in the LDS climb (the default), the paper's round(m/n) (no cap)
    // with halving off.
    const int32_t ph = opts ? opts->path_halving : CC_HALVE_AUTO;
    if (ph < CC_HALVE_AUTO || ph > CC_HALVE_OFF) return fail(CC_ERR_ARG, "unknown cc_options.path_halving");
    const bool lds_halve = ph != CC_HALVE_OFF;
    int32_t seg_cap = opts ? opts->segments : 0;
    if (seg_cap < 0) return fail(CC_ERR_ARG, "cc_options.segments < 0");
    // workgroup size of the LDS solver (0 = by the graphs' sizes)
    int32_t lds_block = opts ? opts->block : 0;
    if (lds_block != 0 && (lds_block < 64 || lds_block > 1024 || lds_block % 64))
        return fail(CC_ERR_ARG, "cc_options.block must be a multiple of 64 in [64, 1024]");
    if (seg_cap == 0 && lds_halve) seg_cap = count <= kFewGraphs ? kSegAutoFew : kSegAuto;
    if (st) {
        std::memset(st, 0, sizeof *st);
        st->giant_label = -1;
    }
    if (count == 0) return CC_OK;
    // host scratch kept per thread: a call allocates nothing once warm
    static thread_local std::vector<int32_t> small, large, sorted;
    static thread_local std::vector<uint8_t> cls;
    small.clear();
    large.clear();
    small.reserve((size_t)count);
    cls.resize((size_t)count);
    int64_t start[257] = {0};
    int64_t maxn_small = 0;
    for (int32_t g = 0; g < count; ++g) {
        const cc_graph G = graph_at(g);
        if (G.reserved != 0) return fail(CC_ERR_ARG, "cc_graph.reserved must be zero");
        if (G.n < 0 || G.m < 0) return fail(CC_ERR_ARG, "graph with n < 0 or m < 0");
        if (G.m > 0 && (!G.edges_u || !G.edges_v)) return fail(CC_ERR_ARG, "null edge array");
        if (G.n > 0 && !G.out_label) return fail(CC_ERR_ARG, "null out_label");
        if (G.n == 0) {
            if (G.m > 0) return fail(CC_ERR_RANGE, "edge endpoint outside [0, n) (empty graph)");
            continue;
        }
        if (G.n <= CC_BATCH_LDS_MAX_N) {
            const uint8_t c = (uint8_t)(255 - size_class((uint64_t)G.m + (uint64_t)G.n));
            cls[small.size()] = c;
            ++start[c + 1];
            small.push_back(g);
            maxn_small = std::max<int64_t>(maxn_small, G.n);
        } else {
            large.push_back(g);
        }
    }
    // Largest first (longest-processing-time order): the queue's tail holds
    // the small graphs, which even out the workgroups' finishing times.  An
    // O(count) counting sort on a size class (four classes per power of two
    // of m + n) gives that order; a comparison sort of 10,000 graphs costs
    // about a millisecond of host time, more than a third of the solve.
    {
        const size_t k = small.size();
        for (int c = 0; c < 256; ++c) start[c + 1] += start[c];
        sorted.resize(k);
        for (size_t i = 0; i < k; ++i) sorted[start[cls[i]]++] = small[i];
        small.swap(sorted);
    }
    // The workspace of a solve that gives the first `moved` of the small graphs
    // to the device-memory path: the LDS launch's queue counters, its
    // descriptors right after (one copy from the staging buffer uploads both
    // and clears the counters), then the large graphs' control blocks and
    // their regions.
    const int32_t nl0 = (int32_t)large.size();
    const bool by_rule = ph == CC_HALVE_AUTO && lds_block == 0 && (!opts || opts->segments == 0);
    int32_t moved = by_rule ? alone_count(small, graph_at) : 0;
    int32_t ns, nl;
    std::vector<Plan> plans;
    std::vector<size_t> region_off;
    std::vector<Layout> layouts;
    const size_t desc_off = kQueueBytes;
    size_t desc_bytes, lctrl_off, off;
    while (true) {
        ns = (int32_t)small.size() - moved;
        nl = nl0 + moved;
        large.insert(large.end(), small.begin(), small.begin() + moved);
        plans.assign(nl, Plan());
        region_off.assign(nl, 0);
        layouts.assign(nl, Layout());
        desc_bytes = align256((size_t)ns * sizeof(GraphDesc));
        lctrl_off = desc_off + desc_bytes;
        off = lctrl_off + align256((size_t)nl * sizeof(Ctrl));
        for (int32_t i = 0; i < nl; ++i) {
            const cc_graph G = graph_at(large[i]);
            int32_t rc = make_plan(G.n, G.m, nullptr, plans[i], kInputGraphList);
            if (rc != CC_OK) return rc;
            layouts[i] = layout(G.n, G.m, plans[i]);  // its control block is lctrls[i] instead
            region_off[i] = off;
            off += align256(layouts[i].total);
        }
        if (moved == 0 || !workspace || ws_bytes >= off) break;
        large.resize(nl0);  // a workspace sized for the LDS launch alone
        moved = 0;
    }
    if (moved) {
        small.erase(small.begin(), small.begin() + moved);
        maxn_small = 0;
        for (int32_t g : small) maxn_small = std::max<int64_t>(maxn_small, graph_at(g).n);
    }
    if (lds_block == 0) lds_block = batch_block(ns, (int32_t)maxn_small);
    if (ws_needed) {  // size query only
        *ws_needed = off;
        return CC_OK;
    }
    if (workspace) {
        if (ws_bytes < off) return fail(CC_ERR_NOMEM, "graph-list workspace too small");
        if ((uintptr_t)workspace & 255) return fail(CC_ERR_ARG, "workspace must be 256-byte aligned");
    }
    if (ns > 0) HIPCHK(prepare_batch_lds());
    PoolEntry* pe = pool_entry(s);
    std::lock_guard<std::mutex> lk(pe->mu);
    int32_t rc = ensure_host(pe, std::max(1, nl));
    if (rc != CC_OK) return rc;
    if (!pe->batch_status)
        HIPCHK(hipHostMalloc((void**)&pe->batch_status, 256, hipHostMallocDefault));
    if (!workspace) {
        rc = ensure_dev(pe, off);
        if (rc != CC_OK) return rc;
    }
    if (ns > 0) {
        rc = ensure_stage(pe, desc_off + desc_bytes);
        if (rc != CC_OK) return rc;
    }
    char* ws = workspace ? static_cast<char*>(workspace) : static_cast<char*>(pe->dev);
    uint32_t* heads = reinterpret_cast<uint32_t*>(ws);        // the LDS launch's queues
    Ctrl* lctrls = reinterpret_cast<Ctrl*>(ws + lctrl_off);   // the large graphs'
    // The LDS launch reports a bad endpoint in a pinned host word, so a call
    // without large graphs needs no copy back before its synchronisation.
    *pe->batch_status = 0;
    if (ns > 0) {
        std::memset(pe->host_stage, 0, desc_off);  // the cleared queue counters
        GraphDesc* hd = reinterpret_cast<GraphDesc*>(static_cast<char*>(pe->host_stage) + desc_off);
        for (int32_t i = 0; i < ns; ++i) {
            const cc_graph G = graph_at(small[i]);
            GraphDesc& d = hd[i];
            d.u = G.edges_u;
            d.v = G.edges_v;
            d.out = G.out_label;
            d.m = G.m;
            d.n = G.n;
            // average-degree segmentation per graph (Section 3.B), capped
            d.segments = lds_segments(G.m, G.n, seg_cap);
        }
    }
    // The launch sequence: clear the LDS solver's queue counters, upload the
    // descriptors, one persistent LDS launch, then every large graph's solve.
    Timer tm;
    auto enqueue = [&]() -> int32_t {
        if (ns > 0) {
            HIPCHK(hipMemcpyAsync(ws, pe->host_stage, desc_off + desc_bytes, hipMemcpyHostToDevice, s));
            HIPCHK(launch_batch_lds(reinterpret_cast<GraphDesc*>(ws + desc_off), ns,
                                    (int32_t)maxn_small, heads, pe->batch_status,
                                    lds_halve, device_cu_count(), s, lds_block));
        }
        for (int32_t i = 0; i < nl; ++i) {
            const cc_graph G = graph_at(large[i]);
            int32_t r2 = plans[i].hook == CC_HOOK_HYBRID
                             ? enqueue_hybrid(G.n, G.edges_u, G.edges_v, G.m, G.out_label, plans[i],
                                              reinterpret_cast<char*>(&lctrls[i]), layouts[i], s, tm,
                                              nullptr, &pe->host_ctrl[i])
                             : enqueue_atomic(G.n, G.edges_u, G.edges_v, G.m, G.out_label, plans[i],
                                              &lctrls[i], filter_bufs(ws + region_off[i], layouts[i]),
                                              s, tm, nullptr, &pe->host_ctrl[i]);
            if (r2 != CC_OK) return r2;
        }
        return CC_OK;
    };
    const bool use_graph = opts && opts->graph == 1 && s != nullptr;
    if (use_graph) {
        KeyHash k;
        // The LDS graphs' descriptors are not part of the key: the captured
        // copy node re-reads the pinned staging buffer, rewritten above, at
        // every replay.  Only what the capture bakes in is: sizes, pointers,
        // the LDS launch shape, and each large graph's arrays and plan.
        k.add(count).add(ws).add(s).add(pe->host_stage).add(pe->host_ctrl).add(seg_cap).add(lds_halve)
            .add(maxn_small).add(ns).add(nl).add(lds_block);
        for (int32_t i = 0; i < nl; ++i) {
            const cc_graph G = graph_at(large[i]);
            k.add(G.edges_u).add(G.edges_v).add(G.out_label).add(G.m).add(G.n);
        }
        rc = run_graph(pe, k.h, s, enqueue);
    } else {
        rc = enqueue();
    }
    if (rc != CC_OK) return rc;
    if (st) st->hook_launches += (ns > 0 ? 1 : 0);
    HIPCHK(hipStreamSynchronize(s));
    if (st) st->host_syncs += 1;
    bool bad = (*(volatile int32_t*)pe->batch_status & kStatusRange) != 0;
    for (int32_t i = 0; i < nl; ++i) bad |= (pe->host_ctrl[i].status & kStatusRange) != 0;
    if (bad) return fail(CC_ERR_RANGE, "edge endpoint outside [0, n_g)");
    return CC_OK;
}

int32_t list_impl(int32_t count, const cc_graph* graphs, const cc_options* opts, hipStream_t s,
                  cc_stats* st, void* workspace, size_t ws_bytes, size_t* ws_needed) {
    if (count > 0 && !graphs) {
        if (ws_needed) *ws_needed = 0;
        return fail(CC_ERR_ARG, "null graph list");
    }
    return list_core(count, [graphs](int32_t g) { return graphs[g]; }, opts, s, st, workspace,
                     ws_bytes, ws_needed);
}

int32_t batch_lds_impl(int32_t B, const int64_t* vo, const int64_t* eo, const int64_t* hvo,
                       const int64_t* heo, const int32_t* u, const int32_t* v, int32_t* out,
                       int32_t max_n, const cc_options* opts, hipStream_t s, cc_stats* st);

int32_t batch_impl(int32_t B, const int64_t* vo, const int64_t* eo, const int32_t* u,
                   const int32_t* v, int32_t* out, const cc_options* opts, hipStream_t s,
                   cc_stats* st) {
    if (B < 0) return fail(CC_ERR_ARG, "num_graphs < 0");
    if (opts && opts->no_sync)
        return fail(CC_ERR_ARG, "cc_options.no_sync is for cc_labels_ex and cc_labels_csr only");
    if (B == 0) {
        if (st) {
            std::memset(st, 0, sizeof *st);
            st->giant_label = -1;
        }
        return CC_OK;
    }
    if (!vo || !eo) return fail(CC_ERR_ARG, "null offsets");
    if (vo[0] != 0 || eo[0] != 0) return fail(CC_ERR_ARG, "offsets must start at 0");
    int64_t max_n = 0;
    for (int32_t g = 0; g < B; ++g) {
        const int64_t nv = vo[g + 1] - vo[g], ne = eo[g + 1] - eo[g];
        if (nv < 0 || ne < 0) return fail(CC_ERR_ARG, "offsets must be non-decreasing");
        if (nv > INT32_MAX) return fail(CC_ERR_ARG, "graph with 2^31 or more vertices");
        max_n = std::max(max_n, nv);
    }
    if (eo[B] > 0 && (!u || !v)) return fail(CC_ERR_ARG, "null edge array");
    if (vo[B] > 0 && !out) return fail(CC_ERR_ARG, "null out_label");
    // Every graph LDS-sized: the offsets are copied to the device as they are
    // and the graphs ordered and described there (the device-offset path),
    // which costs less host time than building the descriptors here.
    if (max_n <= CC_BATCH_LDS_MAX_N)
        return batch_lds_impl(B, nullptr, nullptr, vo, eo, u, v, out,
                              (int32_t)std::max<int64_t>(1, max_n), opts, s, st);
    // graph g straight from the offsets: no list of B graphs is built
    auto graph_at = [=](int32_t g) {
        cc_graph G;
        const int64_t ne = eo[g + 1] - eo[g];
        G.edges_u = ne ? u + eo[g] : nullptr;
        G.edges_v = ne ? v + eo[g] : nullptr;
        G.out_label = out ? out + vo[g] : nullptr;
        G.m = ne;
        G.n = (int32_t)(vo[g + 1] - vo[g]);
        G.reserved = 0;
        return G;
    };
    return list_core(B, graph_at, opts, s, st, nullptr, 0, nullptr);
}

// Device offsets: the preparation workgroup builds the descriptors and the
// largest-first order on the device (no host pass over the graphs), then the
// persistent LDS launch solves them; one synchronisation.
// The LDS batch with offsets in device memory (vo, eo), or in host memory
// (hvo, heo non-null: copied through the pinned staging buffer into the
// workspace first, one copy per call).
// Host offsets of up to this many graphs are read by the solving launch from
// the pinned staging buffer, larger batches copy them first (one launch for
// graphs of up to 256 vertices, against a copy and the launch: 2,000 graphs
// 32.4 against 35.4 us, 8,000 graphs 55.5 against 50.8 us).
constexpr int32_t kZeroCopyGraphs = 4096;

int32_t batch_lds_impl(int32_t B, const int64_t* vo, const int64_t* eo, const int64_t* hvo,
                       const int64_t* heo, const int32_t* u, const int32_t* v, int32_t* out,
                       int32_t max_n, const cc_options* opts, hipStream_t s, cc_stats* st) {
    if (B < 0) return fail(CC_ERR_ARG, "num_graphs < 0");
    if (opts && opts->no_sync)
        return fail(CC_ERR_ARG, "cc_options.no_sync is for cc_labels_ex and cc_labels_csr only");
    const int32_t ph = opts ? opts->path_halving : CC_HALVE_AUTO;
    if (ph < CC_HALVE_AUTO || ph > CC_HALVE_OFF) return fail(CC_ERR_ARG, "unknown cc_options.path_halving");
    const bool lds_halve = ph != CC_HALVE_OFF;
    int32_t seg_cap = opts ? opts->segments : 0;
    if (seg_cap < 0) return fail(CC_ERR_ARG, "cc_options.segments < 0");
    if (seg_cap == 0 && lds_halve) seg_cap = B <= kFewGraphs ? kSegAutoFew : kSegAuto;
    int32_t lds_block = opts ? opts->block : 0;
    if (lds_block != 0 && (lds_block < 64 || lds_block > 1024 || lds_block % 64))
        return fail(CC_ERR_ARG, "cc_options.block must be a multiple of 64 in [64, 1024]");
    if (max_n < 1 || max_n > CC_BATCH_LDS_MAX_N)
        return fail(CC_ERR_ARG, "max_n must be in [1, CC_BATCH_LDS_MAX_N]");
    if (st) {
        std::memset(st, 0, sizeof *st);
        st->giant_label = -1;
    }
    if (B == 0) return CC_OK;
    // null edge or label arrays are allowed for graphs without entries /
    // vertices; the preparation launch checks that on the device
    const bool staged = hvo && heo;
    if (!staged && (!vo || !eo)) return fail(CC_ERR_ARG, "null offsets");
    if (lds_block == 0) lds_block = batch_block(B, max_n);
    const bool direct = batch_direct(B, max_n, lds_block, device_cu_count());
    const bool zero_copy = direct && staged && B <= kZeroCopyGraphs;
    if ((size_t)B > (SIZE_MAX - kQueueBytes) / sizeof(GraphDesc)) return fail(CC_ERR_ARG, "too many graphs");
    const size_t desc_off = kQueueBytes;
    const size_t rows_off = desc_off + align256((size_t)B * sizeof(GraphDesc));
    const size_t off_bytes = align256(((size_t)B + 1) * 8);  // one offset array
    const size_t offs_off = rows_off + align256((((size_t)B + 1023) / 1024 + 1) * 256 * 4);
    const size_t total = offs_off + (staged && !zero_copy ? 2 * off_bytes : 0);
    HIPCHK(prepare_batch_lds());
    PoolEntry* pe = pool_entry(s);
    std::lock_guard<std::mutex> lk(pe->mu);
    int32_t rc = ensure_dev(pe, total);
    if (rc != CC_OK) return rc;
    if (staged) {
        rc = ensure_stage(pe, 2 * off_bytes);
        if (rc != CC_OK) return rc;
        std::memcpy(pe->host_stage, hvo, ((size_t)B + 1) * 8);
        std::memcpy(static_cast<char*>(pe->host_stage) + off_bytes, heo, ((size_t)B + 1) * 8);
    }
    if (!pe->batch_status)
        HIPCHK(hipHostMalloc((void**)&pe->batch_status, 256, hipHostMallocDefault));
    pe->batch_status[0] = pe->batch_status[1] = pe->batch_status[2] = 0;
    char* ws = static_cast<char*>(pe->dev);
    if (staged) {
        const char* at = zero_copy ? static_cast<const char*>(pe->host_stage) : ws + offs_off;
        vo = reinterpret_cast<const int64_t*>(at);
        eo = reinterpret_cast<const int64_t*>(at + off_bytes);
    }
    uint32_t* heads = reinterpret_cast<uint32_t*>(ws);
    GraphDesc* descs = reinterpret_cast<GraphDesc*>(ws + desc_off);
    int32_t* rows = reinterpret_cast<int32_t*>(ws + rows_off);
    auto enqueue = [&]() -> int32_t {
        if (staged && !zero_copy)
            HIPCHK(hipMemcpyAsync(ws + offs_off, pe->host_stage, 2 * off_bytes,
                                  hipMemcpyHostToDevice, s));
        if (direct) {
            const BatchSrc src = {vo, eo, u, v, out, max_n, seg_cap};
            HIPCHK(launch_batch_direct(src, B, pe->batch_status, lds_halve, device_cu_count(), s,
                                       lds_block));
            return CC_OK;
        }
        HIPCHK(launch_batch_prep(vo, eo, B, u, v, out, max_n, seg_cap, descs, rows, heads,
                                 pe->batch_status, s));
        HIPCHK(launch_batch_lds(descs, B, max_n, heads, pe->batch_status, lds_halve,
                                device_cu_count(), s, lds_block));
        return CC_OK;
    };
    if (opts && opts->graph == 1 && s != nullptr) {
        KeyHash k;
        // staged offsets: the captured copy re-reads the staging buffer,
        // rewritten above, at every replay
        k.add(uint64_t(0xba7c4de71ce)).add(B).add(vo).add(eo).add(u).add(v).add(out).add(max_n)
            .add(seg_cap).add(lds_halve).add(lds_block).add(ws).add(s).add(staged)
            .add(pe->host_stage);
        rc = run_graph(pe, k.h, s, enqueue);
    } else {
        rc = enqueue();
    }
    if (rc != CC_OK) return rc;
    if (st) st->hook_launches += 1;
    HIPCHK(hipStreamSynchronize(s));
    if (st) st->host_syncs += 1;
    const int32_t prep = *(volatile int32_t*)(pe->batch_status + 1) |
                         *(volatile int32_t*)(pe->batch_status + 2);
    const int32_t solve = *(volatile int32_t*)pe->batch_status;
    if (prep & kStatusBadGraph)
        return fail(CC_ERR_ARG, "batch offsets must start at 0, be non-decreasing and give "
                                "every graph at most max_n vertices");
    if ((prep | solve) & kStatusRange) return fail(CC_ERR_RANGE, "edge endpoint outside [0, n_g)");
    return CC_OK;
}

int32_t batch_device_impl(int32_t B, const int64_t* vo, const int64_t* eo, const int32_t* u,
                          const int32_t* v, int32_t* out, int32_t max_n, const cc_options* opts,
                          hipStream_t s, cc_stats* st) {
    return batch_lds_impl(B, vo, eo, nullptr, nullptr, u, v, out, max_n, opts, s, st);
}

// ---------------------------------------------------------------------- probes, release
int32_t probe_impl(int32_t mode, const int32_t* u, const int32_t* v, int64_t m, const void* table,
                   int32_t n, hipStream_t s) {
    if (m < 0 || mode < 0 || mode > 11) return fail(CC_ERR_ARG, "bad probe arguments");
    if (mode >= 7) {  // memory-model probe: table is int32[128], edges unused
        if (!table || n < 128) return fail(CC_ERR_ARG, "memory-model probe needs a 128-word table");
        HIPCHK(launch_probe_mm(mode, static_cast<int32_t*>(const_cast<void*>(table)), s));
        return CC_OK;
    }
    if (m > 0 && (!u || !v)) return fail(CC_ERR_ARG, "null edge array");
    if (mode > 0 && (!table || n <= 0)) return fail(CC_ERR_ARG, "probe table required");
    if (((uintptr_t)u & 15) || ((uintptr_t)v & 15))
        return fail(CC_ERR_ARG, "probe edge arrays must be 16-byte aligned");
    PoolEntry* pe = pool_entry(s);
    std::lock_guard<std::mutex> lk(pe->mu);
    int32_t rc = ensure_dev(pe, 256);
    if (rc != CC_OK) return rc;
    uint32_t* sink = static_cast<uint32_t*>(pe->dev);
    if (mode == 0)
        HIPCHK(launch_probe_stream(u, v, m, sink, s));
    else if (mode == 1)
        HIPCHK(launch_probe_gather(u, v, m, static_cast<const int32_t*>(table), n, sink, s));
    else if (mode >= 5)
        HIPCHK(launch_probe_cas(u, v, m, static_cast<int32_t*>(const_cast<void*>(table)), n,
                                mode == 6, sink, s));
    else
        HIPCHK(launch_probe_bitgather(u, v, m, static_cast<const uint32_t*>(table), n, mode - 2,
                                      sink, s));
    return CC_OK;
}

void release_impl() {
    std::lock_guard<std::mutex> g(g_pool_mu);
    for (auto& kv : g_pool) {
        PoolEntry* e = kv.second.get();
        std::lock_guard<std::mutex> lk(e->mu);
        drain_async(e);
        drop_graphs(e);
        if (e->async_done) (void)hipEventDestroy(e->async_done);
        if (e->async_slot) (void)hipHostFree(e->async_slot);
        e->async_done = nullptr;
        e->async_slot = nullptr;
        e->async_called = false;
        for (int i = 0; i < 2; ++i) {
            if (e->copied[i]) (void)hipEventDestroy(e->copied[i]);
            if (e->consumed[i]) (void)hipEventDestroy(e->consumed[i]);
            e->copied[i] = e->consumed[i] = nullptr;
        }
        if (e->copy_stream) (void)hipStreamDestroy(e->copy_stream);
        e->copy_stream = nullptr;
        if (e->dev) (void)hipFree(e->dev);
        if (e->host_ctrl) (void)hipHostFree(e->host_ctrl);
        if (e->host_stage) (void)hipHostFree(e->host_stage);
        if (e->batch_status) (void)hipHostFree(e->batch_status);
        e->batch_status = nullptr;
        e->dev = nullptr;
        e->host_ctrl = nullptr;
        e->host_stage = nullptr;
        e->bytes = e->stage_bytes = 0;
        e->host_ctrl_count = 0;
    }
    g_pool.clear();
}

int32_t stream_status_impl(hipStream_t s) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = -1;
    PoolEntry* e = nullptr;
    {
        std::lock_guard<std::mutex> g(g_pool_mu);
        auto it = g_pool.find({dev, s});
        if (it != g_pool.end()) e = it->second.get();
    }
    if (!e) return fail(CC_ERR_ARG, "no no-sync call on this stream and device");
    std::lock_guard<std::mutex> lk(e->mu);
    if (!e->async_called) return fail(CC_ERR_ARG, "no no-sync call on this stream and device");
    const hipError_t q = hipEventQuery(e->async_done);
    if (q == hipErrorNotReady) return CC_PENDING;
    if (q != hipSuccess) return fail(CC_ERR_HIP, std::string("hipEventQuery: ") + hipGetErrorString(q));
    const int32_t status = *reinterpret_cast<volatile int32_t*>(e->async_slot);
    if (status & kStatusRange) return fail(CC_ERR_RANGE, "edge endpoint outside [0, n)");
    if (status & kStatusOverflow) return fail(CC_ERR_NOMEM, "frontier capacity exceeded");
    return CC_OK;
}

}  // namespace hookcc
