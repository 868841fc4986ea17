// Batched solve of many small graphs in one persistent launch (CDNA4).
//
// Persistent workgroups (1024 threads, 16 waves, by default; as many per CU as
// the LDS of the launch's largest graph allows) take graphs from device
// work queues (atomic counters over descriptors ordered largest first, by
// the host or, for offsets in device memory, by the preparation launches
// below) and solve each one entirely in LDS: the graph's tree array pi lives in LDS as
// local ids, 32-bit for n <= 32768 and 16-bit up to 65536 (at most 128 KiB of
// the 160 KiB LDS), the edge entries are streamed once from HBM, and the
// labels are written once.
// Per graph the schedule is the paper's adaptive one (Fig. 4): for each of
// the graph's s edge segments, Atomic-Hook the segment, then Multi-Jump all
// its vertices, with a workgroup barrier between phases.
#include "kernels.hpp"

namespace hookcc {

constexpr int kBatchEPT = 8;  // edge entries per thread per step
// Fourth word of a raw buffer resource on gfx9-family GPUs (32-bit data
// format, no swizzle) and the non-temporal cache policy of a buffer load.
constexpr int32_t kBufferRsrcWord3 = 0x00020000;
constexpr int32_t kBufferNonTemporal = 2;

// 16-bit compare-and-swap in LDS, built on the 32-bit CAS of the containing
// word: succeeds iff slot `idx` holds `expected`; returns the value found.
// The other half-word may change concurrently; the loop then retries with
// the fresh word, so only a change of this half-word can make it fail.
__device__ __forceinline__ uint32_t lds_cas16(uint16_t* spi, uint32_t idx, uint32_t expected,
                                              uint32_t desired) {
    uint32_t* w = reinterpret_cast<uint32_t*>(spi) + (idx >> 1);
    const uint32_t sh = (idx & 1) * 16;
    uint32_t old = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    while (true) {
        const uint32_t cur = (old >> sh) & 0xffffu;
        if (cur != expected) return cur;
        const uint32_t nw = (old & ~(0xffffu << sh)) | (desired << sh);
        const uint32_t prev = atomicCAS(w, old, nw);
        if (prev == old) return expected;
        old = prev;
    }
}

// The graph's arrays come from a descriptor in memory, so the compiler cannot
// tell their address space; they are global memory, and saying so gives
// global (not flat) loads and stores.
typedef __attribute__((address_space(1))) const int32_t g_cint;
typedef __attribute__((address_space(1))) int32_t g_int;

// Slots of the tree array in LDS.  Graphs of at most kWideMaxN vertices keep
// 32-bit slots (4n bytes <= 128 KiB) and hook with the native 32-bit LDS
// compare-and-swap; larger ones keep 16-bit slots (2n bytes) and hook with
// lds_cas16 on the containing word.
constexpr uint32_t kWideMaxN = 32768;

// Relaxed workgroup-scope atomics, not volatile accesses: the compiler keeps
// every access (other threads change pi concurrently) and still sees that
// the pointer is in LDS, so these are ds_read / ds_write -- a volatile access
// through the pointer became a flat access, which also waits on the
// outstanding global loads of the software pipeline.
template <typename T>
__device__ __forceinline__ uint32_t lds_ld(T* spi, uint32_t idx) {
    return __hip_atomic_load(spi + idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T>
__device__ __forceinline__ void lds_st(T* spi, uint32_t idx, uint32_t x) {
    __hip_atomic_store(spi + idx, (T)x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Compare-and-swap of slot idx from `expected` to `desired`; returns the value
// found (== expected on success).
__device__ __forceinline__ uint32_t lds_cas(uint32_t* spi, uint32_t idx, uint32_t expected,
                                            uint32_t desired) {
    __hip_atomic_compare_exchange_strong(spi + idx, &expected, desired, __ATOMIC_RELAXED,
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return expected;
}
__device__ __forceinline__ uint32_t lds_cas(uint16_t* spi, uint32_t idx, uint32_t expected,
                                            uint32_t desired) {
    return lds_cas16(spi, idx, expected, desired);
}

// Atomic-Hook in LDS (Fig. 3, top), same steps as the device-memory kernel;
// with `halve`, a passed non-root H whose grandparent differs from its
// parent is re-pointed at the grandparent (path halving).  The re-point of a
// non-root never meets a successful CAS on its own slot (that needs a root),
// and with 16-bit slots it cannot be lost to, nor undo, a concurrent CAS on
// the other half of its 32-bit word: that CAS compares the whole word, so it
// fails and retries if the store landed between its read and its swap.  In
// LDS the store costs one write, and the shallower trees let a graph run
// with fewer segments (fewer Multi-Jump passes over its vertices).
template <typename T>
__device__ __forceinline__ void lds_atomic_hook(T* spi, uint32_t pu, uint32_t pv, bool halve) {
    // One exit, at the loop's head, and no branch inside (halve is uniform):
    // after a successful CAS both ends are set to L, which ends the loop; the
    // two loads and the store of that last pass are wasted but cheaper than
    // the exec-mask bookkeeping of a second exit.
    while (pu != pv) {
        const uint32_t H = pu > pv ? pu : pv;
        const uint32_t L = pu > pv ? pv : pu;
        const uint32_t found = lds_cas(spi, H, H, L);
        const uint32_t gu = lds_ld(spi, found);
        const uint32_t gv = lds_ld(spi, L);
        // H is no root now (it was none or the CAS made it a child of L), so
        // no CAS can succeed on its slot and every value stored there is one
        // of its ancestors: gu (found's parent, found itself, or L after a
        // successful CAS) is one, whichever halving store lands last.
        if (halve) lds_st(spi, H, gu);
        const bool hooked = found == H;
        pu = hooked ? L : gu;
        pv = hooked ? L : gv;
    }
}

// The roots p1, p2 of vertices x and y (a root is its own), their climbs
// interleaved; a finished climb stays on its root, whose parent is itself.
// A climb of more than kDeepLdsSteps steps stores where it has got to at
// every further step, so that the vertices of a chain shorten it for each
// other (a path of 2^15 vertices, whose climbs otherwise walk up to 2^15 levels
// in each of 16 passes: 17.8 -> 0.12 ms; from the 9th step on, trees of a few
// dozen levels lost up to 15 %).  The first three steps are not counted: most
// climbs end there (10,000 graphs: 873 us, 883 counting from the first; 4096^2
// grid 327 and 335).
constexpr int kDeepLdsSteps = 64;

template <typename T>
__device__ __forceinline__ void lds_climb(T* spi, uint32_t x, uint32_t y, uint32_t& p1,
                                          uint32_t& p2) {
    p1 = lds_ld(spi, x);
    p2 = lds_ld(spi, y);
    uint32_t g1 = lds_ld(spi, p1), g2 = lds_ld(spi, p2);
    auto under_way = [&] { return g1 != p1 || g2 != p2; };
    auto step = [&] {
        p1 = g1;
        p2 = g2;
        g1 = lds_ld(spi, p1);
        g2 = lds_ld(spi, p2);
    };
    if (!under_way()) return;
    step();
    if (!under_way()) return;
    step();
    if (!under_way()) return;
    step();
    int k = 3;
    while (under_way()) {
        if (++k > kDeepLdsSteps) {
            lds_st(spi, x, g1);
            lds_st(spi, y, g2);
        }
        step();
    }
}

// Entries [base, base + step) of the edge arrays, clipped at `end`: lane
// tid loads entries base + tid + j * blockDim.x into a[j], b[j] (0 past
// `end`).  Each array is read through a raw buffer resource whose size is
// the step's entries inside [base, end), so no load is issued past `end`;
// the byte offsets are per lane and the same at every step.
template <int EPT = kBatchEPT>
__device__ __forceinline__ void edge_step_loads(g_cint* du, g_cint* dv, int64_t base, int64_t end,
                                                int64_t step, int32_t* a, int32_t* b) {
    const int64_t rem = end - base < step ? end - base : step;
    const int32_t bytes = rem > 0 ? (int32_t)(rem * 4) : 0;
    const __amdgpu_buffer_rsrc_t ru =
        __builtin_amdgcn_make_buffer_rsrc((void*)(du + base), 0, bytes, kBufferRsrcWord3);
    const __amdgpu_buffer_rsrc_t rv =
        __builtin_amdgcn_make_buffer_rsrc((void*)(dv + base), 0, bytes, kBufferRsrcWord3);
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
        const int32_t off = (int32_t)((threadIdx.x + j * blockDim.x) * 4);
        a[j] = __builtin_amdgcn_raw_buffer_load_b32(ru, off, 0, kBufferNonTemporal);
        b[j] = __builtin_amdgcn_raw_buffer_load_b32(rv, off, 0, kBufferNonTemporal);
    }
}

// One graph by the whole workgroup (called by every thread): init, then per
// segment Atomic-Hook of its entries and Multi-Jump of its vertices; the last
// Multi-Jump writes the labels instead of storing the roots in LDS.  Sets
// `bad` on an endpoint outside [0, n).  Returns without a final barrier: the
// caller's next barrier separates the label reads from the next graph's init.
template <typename T>
__device__ __forceinline__ void solve_graph(T* spi, const GraphDesc& d, bool halve, bool& bad) {
    const uint32_t tid = threadIdx.x;
    const uint32_t nthr = blockDim.x;
    const uint32_t n = (uint32_t)d.n;
    g_cint* du = (g_cint*)d.u;
    g_cint* dv = (g_cint*)d.v;
    g_int* dout = (g_int*)d.out;
    const int32_t s = d.segments > 0 ? d.segments : 1;
    const int64_t step = (int64_t)nthr * kBatchEPT;
    int32_t a[kBatchEPT], b[kBatchEPT], na[kBatchEPT], nb[kBatchEPT];
    // the first segment's first loads go out before the init, so that their
    // latency overlaps it and its barrier
    edge_step_loads(du, dv, 0, d.m / s, step, a, b);
    for (uint32_t x = tid; x < n; x += nthr) lds_st(spi, x, x);
    __syncthreads();
    for (int32_t seg = 0; seg < s; ++seg) {
        const int64_t b0 = d.m * seg / s, b1 = d.m * (seg + 1) / s;
        // kBatchEPT entries per thread per step, all loads issued before
        // any hook, and the next step's loads issued before this step's
        // hooks (software pipelining), so the edge stream's latency
        // overlaps the LDS work.  The loads go through buffer resources
        // that cover exactly the step's entries: the per-lane byte offsets
        // are the same at every step, and a load past the segment's end
        // returns 0 without touching memory.  No branch surrounds a load or
        // a hook: such an entry, and one out of range, becomes the pair
        // (0, 0), whose hook does nothing -- divergent branches would cost
        // more scalar exec-mask instructions than the work they skip.
        if (b1 > b0) {
            int64_t base = b0;
            if (seg > 0) edge_step_loads(du, dv, base, b1, step, a, b);
            for (; base < b1; base += step) {
                edge_step_loads(du, dv, base + step, b1, step, na, nb);
#pragma unroll
                for (int j = 0; j < kBatchEPT; ++j) {
                    const bool ok = max((uint32_t)a[j], (uint32_t)b[j]) < n;
                    bad |= !ok;
                    const uint32_t x = ok ? (uint32_t)a[j] : 0u;
                    const uint32_t y = ok ? (uint32_t)b[j] : 0u;
                    lds_atomic_hook(spi, lds_ld(spi, x), lds_ld(spi, y), halve);
                }
#pragma unroll
                for (int j = 0; j < kBatchEPT; ++j) {
                    a[j] = na[j];
                    b[j] = nb[j];
                }
            }
        }
        __syncthreads();
        // Multi-Jump (Fig. 3, bottom) over the graph's vertices, low ids first.
        // Each vertex climbs to its root and stores it (a root stores
        // itself); no hook runs in this phase, so only the stores of other
        // climbers race with it, and each stores an ancestor.  After the last
        // segment the root is the label: it goes to global memory only.
        // Two vertices per thread and pass.
        const bool last = seg + 1 == s;
        for (uint32_t x = tid; x < n; x += 2 * nthr) {
            const uint32_t y = x + nthr;
            const bool has_y = y < n;
            uint32_t p1, p2;
            lds_climb(spi, x, has_y ? y : x, p1, p2);
            if (last) {
                dout[x] = (int32_t)p1;
                if (has_y) dout[y] = (int32_t)p2;
            } else {
                lds_st(spi, x, p1);
                if (has_y) lds_st(spi, y, p2);
            }
        }
        if (!last) __syncthreads();
    }
}

// Workgroup b takes graph b first and then draws from work queue b mod
// kQueues, which holds every kQueues-th of the graphs past the first
// gridDim.x, in order.  A single counter served one draw in ~13 ns and every
// workgroup drew its first graph from it, so 2,000 graphs of at most 64
// vertices took 60 us at 512 workgroups and 146 us at 8,192 (20,000 graphs:
// 270 us), whatever their size.
template <bool HALVE>
__global__ __launch_bounds__(1024) void k_batch_lds(const GraphDesc* __restrict__ descs,
                                                    int32_t count, uint32_t* heads,
                                                    int32_t* status) {
    constexpr bool halve = HALVE;  // a compile-time constant: no branch in the hook loop
    extern __shared__ uint16_t spi[];
    __shared__ uint32_t next;
    bool bad = false;
    const uint32_t q = blockIdx.x % kQueues;
    const uint32_t k0 = (gridDim.x - q + kQueues - 1) / kQueues;  // first position of queue q past the grid
    const bool more = (uint32_t)count > gridDim.x;
    uint32_t idx = blockIdx.x;
    while (idx < (uint32_t)count) {
        const GraphDesc d = descs[idx];
        // The next position is fetched while this graph is solved, so the
        // queue's latency is paid once per workgroup, not once per graph.
        // Thread 0 writes `next` again only after the barriers inside
        // solve_graph, which every thread passes after reading it.
        uint32_t pre = 0;
        if (more && threadIdx.x == 0) pre = atomicAdd(heads + q * kQueueStride, 1u);
        if ((uint32_t)d.n <= kWideMaxN)
            solve_graph(reinterpret_cast<uint32_t*>(spi), d, halve, bad);
        else
            solve_graph(spi, d, halve, bad);
        if (!more) break;
        if (threadIdx.x == 0) next = q + kQueues * (k0 + pre);
        __syncthreads();
        idx = next;
    }
    // status may be host memory: a plain store (every writer stores the same
    // bit) visible to the host once the launch has completed
    if (bad) __hip_atomic_store(status, kStatusRange, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One small graph, given by value, by one workgroup.  *status (device or pinned
// host memory) receives kStatusRange, or what *prior says.
template <bool HALVE>
__global__ __launch_bounds__(1024) void k_single_lds(GraphDesc d, const int32_t* prior, int32_t* status) {
    extern __shared__ uint16_t spi[];
    bool bad = false;
    solve_graph(reinterpret_cast<uint32_t*>(spi), d, HALVE, bad);
    const int any = __syncthreads_or(bad);
    if (threadIdx.x == 0)
        __hip_atomic_store(status, any ? kStatusRange : prior ? *prior : 0, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------
// Preparation of a batch whose offsets are in device memory, in two launches
// of one thread per graph: every graph is checked and given its size class
// of m + n (four classes per power of two, the order the host-offset call
// builds); the graphs are placed largest class first (a counting sort) and
// their descriptors written for k_batch_lds.  A graph whose offsets are
// invalid (not starting at 0, decreasing, more than max_n vertices) or that
// has entries but no vertex gets an empty descriptor (nothing is read or
// written for it); status[1] / status[2] (host memory) then receive
// kStatusBadGraph / kStatusRange.  The queue counters are cleared for the
// solve.

__device__ __forceinline__ int batch_size_class(uint64_t w) {
    w |= 1;
    const int lg = 63 - __clzll((long long)w);
    const int frac = lg >= 2 ? (int)((w >> (lg - 2)) & 3) : (int)((w << (2 - lg)) & 3);
    return lg * 4 + frac;
}

// min(cap, round(m / n)), at least 1 (cap 0: round(m / n) up to 2^20;
// negative: the default rule)
__device__ __forceinline__ int32_t batch_segments(int64_t m, int64_t n, int32_t cap) {
    if (cap < 0) return lds_auto_segments(m, n, cap == kSegAutoFew);
    if (cap > 0 && cap <= 16 && m < (int64_t(1) << 61)) {
        int32_t k = cap;
        while (k > 1 && 2 * m < (2 * (int64_t)k - 1) * n) --k;
        return k;
    }
    int64_t r = m / n + ((m % n) * 2 >= n ? 1 : 0);
    r = r < 1 ? 1 : (r > (int64_t(1) << 20) ? (int64_t(1) << 20) : r);
    return cap > 0 && r > cap ? cap : (int32_t)r;
}

constexpr int kPrepGraphs = 1024;  // graphs per preparation workgroup, one per thread

struct PrepGraph {
    int64_t v0, n, e0, m;
    int32_t cls;   // position class: 0 = largest
    int32_t flag;  // 0, kStatusBadGraph or kStatusRange
};

__device__ __forceinline__ PrepGraph prep_graph(const int64_t* vo, const int64_t* eo, int32_t g,
                                                int32_t max_n, bool edges, bool labels) {
    PrepGraph p;
    p.v0 = vo[g];
    p.e0 = eo[g];
    p.n = vo[g + 1] - p.v0;
    p.m = eo[g + 1] - p.e0;
    p.flag = 0;
    // (edges / labels: whether those arrays were given; a null one may only
    // belong to graphs that have no entries / no vertices)
    if ((g == 0 && (p.v0 != 0 || p.e0 != 0)) || p.n < 0 || p.m < 0 || p.n > max_n ||
        (p.m > 0 && !edges) || (p.n > 0 && !labels))
        p.flag = kStatusBadGraph;
    else if (p.n == 0 && p.m > 0)
        p.flag = kStatusRange;
    if (p.flag) p.n = p.m = 0;
    p.cls = 255 - batch_size_class((uint64_t)p.m + (uint64_t)p.n);
    return p;
}

// The batch without preparation: workgroup b takes graphs b, b + gridDim.x,
// ... in the given order and reads each one's offsets itself (from pinned
// host memory when the offsets are there).  For small graphs the order does
// not matter (no graph takes much longer than another), and the call is one
// launch instead of three and a copy.  Invalid graphs are skipped and
// reported as by the preparation launches.
template <bool HALVE>
__global__ __launch_bounds__(1024) void k_batch_direct(BatchSrc src, int32_t count,
                                                       int32_t* status) {
    extern __shared__ uint16_t spi[];
    bool bad = false;
    int32_t flags = 0;
    for (int64_t g = blockIdx.x; g < count; g += gridDim.x) {
        const PrepGraph p = prep_graph(src.vo, src.eo, (int32_t)g, src.max_n, src.u && src.v,
                                       src.out != nullptr);
        flags |= p.flag;
        GraphDesc d;
        d.u = src.u + p.e0;
        d.v = src.v + p.e0;
        d.out = src.out + p.v0;
        d.m = p.m;
        d.n = (int32_t)p.n;
        d.segments = p.n > 0 ? batch_segments(p.m, p.n, src.seg_cap) : 1;
        solve_graph(reinterpret_cast<uint32_t*>(spi), d, HALVE, bad);
        __syncthreads();  // the label reads before the next graph's init
    }
    if (bad) __hip_atomic_store(status, kStatusRange, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (threadIdx.x == 0 && (flags & kStatusBadGraph))
        __hip_atomic_store(status + 1, kStatusBadGraph, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (threadIdx.x == 0 && (flags & kStatusRange))
        __hip_atomic_store(status + 2, kStatusRange, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Step 1 (one thread per graph, kPrepGraphs per workgroup): each workgroup
// counts its graphs per class into its row of `rows` (W x 256).
__global__ __launch_bounds__(1024) void k_batch_prep_count(const int64_t* __restrict__ vo,
                                                           const int64_t* __restrict__ eo,
                                                           int32_t B, int32_t max_n, bool edges,
                                                           bool labels, int32_t* __restrict__ rows,
                                                           uint32_t* __restrict__ heads) {
    __shared__ int32_t hist[256];
    const int32_t tid = threadIdx.x;
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    const int32_t g = blockIdx.x * kPrepGraphs + tid;
    if (g < B) atomicAdd(&hist[prep_graph(vo, eo, g, max_n, edges, labels).cls], 1);
    __syncthreads();
    if (tid < 256) rows[blockIdx.x * 256 + tid] = hist[tid];
    if (blockIdx.x == 0 && tid < kQueues * kQueueStride) heads[tid] = 0;
}

// Up to this many preparation workgroups, each placing workgroup sums the
// rows of all of them itself (W x 256 loads each); above it a scan launch
// turns the rows into prefix sums first, so that the work stays linear in B.
constexpr int32_t kPrepLoopMaxW = 32;

// Step 1b (only when W > kPrepLoopMaxW; one workgroup per class c): column c
// of `rows` becomes the exclusive prefix sums over the workgroups (row w: the
// graphs of class c in workgroups before w), and totals[c] its sum.  Thread t
// takes a run of consecutive rows.
__global__ __launch_bounds__(1024) void k_batch_prep_scan(int32_t* __restrict__ rows, int32_t W,
                                                          int32_t* __restrict__ totals) {
    __shared__ int32_t wsum[16];
    const int32_t c = blockIdx.x, tid = threadIdx.x;
    const int32_t lane = tid & 63, wave = tid >> 6;
    const int32_t per = (W + 1023) / 1024;
    const int32_t w0 = min(W, tid * per), w1 = min(W, w0 + per);
    int32_t sum = 0;
    for (int32_t w = w0; w < w1; ++w) sum += rows[(int64_t)w * 256 + c];
    int32_t incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t t = __shfl_up(incl, d, 64);
        if (lane >= d) incl += t;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int32_t at = incl - sum, all = 0;
    for (int32_t i = 0; i < 16; ++i) {
        at += i < wave ? wsum[i] : 0;
        all += wsum[i];
    }
    for (int32_t w = w0; w < w1; ++w) {
        const int32_t r = rows[(int64_t)w * 256 + c];
        rows[(int64_t)w * 256 + c] = at;
        at += r;
    }
    if (tid == 0) totals[c] = all;
}

// Step 2: each workgroup finds where its graphs of each class go (all
// earlier classes of every workgroup, then this class of the earlier
// workgroups) and writes their descriptors there.  `totals` null: `rows`
// holds the per-workgroup counts; else the scanned rows and the totals.
__global__ __launch_bounds__(1024) void k_batch_prep_place(
    const int64_t* __restrict__ vo, const int64_t* __restrict__ eo, int32_t B, const int32_t* u,
    const int32_t* v, int32_t* out, int32_t max_n, int32_t seg_cap,
    const int32_t* __restrict__ rows, const int32_t* __restrict__ totals, int32_t W,
    GraphDesc* __restrict__ descs, int32_t* status) {
    __shared__ int32_t base[256];
    __shared__ int32_t flags;
    const int32_t tid = threadIdx.x;
    int32_t total = 0, before = 0;
    if (tid < 256 && totals) {
        total = totals[tid];
        before = rows[(int64_t)blockIdx.x * 256 + tid];
    } else if (tid < 256) {
        for (int32_t w = 0; w < W; ++w) {
            const int32_t r = rows[w * 256 + tid];
            total += r;
            before += w < (int32_t)blockIdx.x ? r : 0;
        }
    }
    if (tid == 0) flags = 0;
    __shared__ int32_t tot[256];
    if (tid < 256) tot[tid] = total;
    __syncthreads();
    if (tid < 64) {
        // exclusive scan of the 256 class totals: 4 per lane, then across the wave
        const int32_t c0 = tot[4 * tid], c1 = tot[4 * tid + 1], c2 = tot[4 * tid + 2],
                      c3 = tot[4 * tid + 3];
        const int32_t sum = c0 + c1 + c2 + c3;
        int32_t inc = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t t = __shfl_up(inc, d, 64);
            if (tid >= d) inc += t;
        }
        const int32_t ex = inc - sum;
        tot[4 * tid] = ex;
        tot[4 * tid + 1] = ex + c0;
        tot[4 * tid + 2] = ex + c0 + c1;
        tot[4 * tid + 3] = ex + c0 + c1 + c2;
    }
    __syncthreads();
    if (tid < 256) base[tid] = tot[tid] + before;
    __syncthreads();
    const int32_t g = blockIdx.x * kPrepGraphs + tid;
    if (g < B) {
        const PrepGraph p = prep_graph(vo, eo, g, max_n, u && v, out != nullptr);
        const int32_t pos = atomicAdd(&base[p.cls], 1);
        GraphDesc d;
        d.u = u + p.e0;
        d.v = v + p.e0;
        d.out = out + p.v0;
        d.m = p.m;
        d.n = (int32_t)p.n;
        d.segments = p.n > 0 ? batch_segments(p.m, p.n, seg_cap) : 1;
        descs[pos] = d;
        if (p.flag) atomicOr(&flags, p.flag);
    }
    __syncthreads();
    // one word per kind of fault, so that plain stores of different
    // workgroups never overwrite each other's bits
    if (tid == 0 && (flags & kStatusBadGraph))
        __hip_atomic_store(status + 1, kStatusBadGraph, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (tid == 0 && (flags & kStatusRange))
        __hip_atomic_store(status + 2, kStatusRange, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t launch_batch_prep(const int64_t* vo, const int64_t* eo, int32_t B, const int32_t* u,
                             const int32_t* v, int32_t* out, int32_t max_n, int32_t seg_cap,
                             GraphDesc* descs, int32_t* rows, uint32_t* heads, int32_t* status,
                             hipStream_t s) {
    if (B <= 0) return hipSuccess;
    const int32_t W = (int32_t)(((int64_t)B + kPrepGraphs - 1) / kPrepGraphs);
    k_batch_prep_count<<<W, kPrepGraphs, 0, s>>>(vo, eo, B, max_n, u && v, out != nullptr, rows,
                                                 heads);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    int32_t* totals = nullptr;
    if (W > kPrepLoopMaxW) {
        totals = rows + (int64_t)W * 256;
        k_batch_prep_scan<<<256, 1024, 0, s>>>(rows, W, totals);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    k_batch_prep_place<<<W, kPrepGraphs, 0, s>>>(vo, eo, B, u, v, out, max_n, seg_cap, rows, totals,
                                                 W, descs, status);
    return hipGetLastError();
}

// Window round of the hybrid plan (an atomic-free Hook round, Fig. 2, with
// the Hook of each workgroup's chunk done in LDS; beyond the paper).
// Workgroup w takes entries [w * chunk, (w + 1) * chunk) and a window of
// `slots` consecutive vertices starting at the smallest endpoint among the
// chunk's first blockDim.x entries.  Entries with both endpoints in the window
// are joined completely in LDS (Atomic-Hook with path halving on 16-bit local
// ids, then a Multi-Jump over the window); every other entry gets the
// device-memory atomic-free Hook (pi[max] = min of the endpoints' current
// parents).  Then each window vertex that is not its local root is pointed at
// it.  The number of entries hooked outside the windows is added to
// ctrl->win_far, in pairs.
//
// A chunk of whose first entries fewer than three eighths lie in its window
// has no locality; it is hooked without a window, each entry pointing its
// larger endpoint at the smaller one (their own parents at the init; nothing
// is loaded), and raises ctrl->win_far above far_limit, so that the caller
// treats the list as one without locality.
//
// Every value written to pi names a vertex of the slot's own component below
// the slot (a local root, or the smaller of two vertices joined by an entry),
// so pi stays a forest of subsets of components with pi[x] <= x.  Stores of
// different workgroups to one slot overwrite each other, which can split a
// chunk's local component into several trees; the pass that follows over all
// entries joins them.  The window stores are of agent scope (see settling in
// common.hpp; the slots are hardly contended, the cost is nil); those of
// chunks without locality are not, and a settling Multi-Jump follows them.
// On inputs whose consecutive entries touch nearby ids (a row-major lattice)
// nearly every entry is joined in LDS and few survive the round.
//
// Sizes by list length (window_shape below): a chunk of a percolated lattice
// spans ~0.8 ids per entry plus a row; long lists take the largest chunks of
// which two workgroups fit a CU (80 KiB of LDS), shorter ones smaller chunks,
// so that every CU has one.
constexpr int kWinEPT = 4;  // entries per thread per step (registers: two workgroups per CU)

__global__ __launch_bounds__(1024) void k_hook_window(const int32_t* __restrict__ eu,
                                                      const int32_t* __restrict__ ev, int64_t m,
                                                      int32_t* pi, int32_t n, Ctrl* ctrl,
                                                      int32_t chunk, uint32_t slots,
                                                      int32_t segments, uint32_t far_limit,
                                                      int64_t prefix) {
    extern __shared__ uint16_t spi[];
    __shared__ int32_t wave_min[16];
    const uint32_t tid = threadIdx.x, nthr = blockDim.x;
    if (prefix > 0 && ctrl->scattered) {
        const int64_t e = (int64_t)blockIdx.x * nthr + tid;
        for (int64_t i = e; i < prefix; i += (int64_t)gridDim.x * nthr) {
            const int32_t x = __builtin_nontemporal_load(eu + i), y = __builtin_nontemporal_load(ev + i);
            if (x != y && max((uint32_t)x, (uint32_t)y) < (uint32_t)n) st_rlx(pi + max(x, y), min(x, y));
        }
        return;
    }
    const uint32_t lane = tid & 63, wave = tid >> 6, waves = nthr >> 6;
    const int64_t c0 = (int64_t)blockIdx.x * chunk;
    const int64_t c1 = min(m, c0 + chunk);
    const int64_t step = (int64_t)nthr * kWinEPT;
    g_cint* gu = (g_cint*)eu;
    g_cint* gv = (g_cint*)ev;
    int32_t a[kWinEPT], b[kWinEPT], na[kWinEPT], nb[kWinEPT];
    // the window starts at the smallest endpoint among the first blockDim.x
    // entries; the LDS is set while they are loaded
    const int64_t first_end = c0 + (c1 - c0) / segments;
    edge_step_loads<kWinEPT>(gu, gv, c0, first_end, step, a, b);
    uint32_t* w32 = reinterpret_cast<uint32_t*>(spi);
    for (uint32_t w = tid; w < slots / 2; w += nthr) w32[w] = ((2 * w + 1) << 16) | (2 * w);
    const bool first = c0 + tid < first_end && max((uint32_t)a[0], (uint32_t)b[0]) < (uint32_t)n;
    int32_t lo = first ? min(a[0], b[0]) : INT32_MAX;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) lo = min(lo, __shfl_xor(lo, d, 64));
    if (lane == 0) wave_min[wave] = lo;
    __syncthreads();
    int32_t base = wave_min[0];
    for (uint32_t i = 1; i < waves; ++i) base = min(base, wave_min[i]);
    if (base == INT32_MAX) base = 0;
    // window vertices: [base, base + span)
    const uint32_t span = (uint32_t)min<int64_t>((int64_t)slots, (int64_t)n - base);
    bool bad = false;
    const int near = __syncthreads_count(first && (uint32_t)max(a[0], b[0]) - (uint32_t)base < span);
    if (8 * near < 3 * (int)min(first_end - c0, (int64_t)nthr)) {
        for (int64_t sb = c0; sb < c1; sb += step) {
            if (sb > c0 || segments > 1) edge_step_loads<kWinEPT>(gu, gv, sb, c1, step, a, b);
#pragma unroll
            for (int j = 0; j < kWinEPT; ++j) {
                const bool ok = max((uint32_t)a[j], (uint32_t)b[j]) < (uint32_t)n;
                bad |= !ok;
                if (ok && a[j] != b[j]) st_rlx(pi + max(a[j], b[j]), min(a[j], b[j]));
            }
        }
        // a plain store: additions by other workgroups only raise it
        if (tid == 0)
            __hip_atomic_store(&ctrl->win_far, far_limit + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (bad) atomicOr(&ctrl->status, kStatusRange);
        return;
    }
    uint32_t far = 0;  // entries hooked outside the window
    // The chunk in `segments` segments, each followed by a Multi-Jump over
    // the window (the schedule of Fig. 4 inside the chunk) so that later
    // climbs start from stars.  kWinEPT entries per thread per step,
    // consecutive threads on consecutive entries (coalesced, through buffer
    // resources as in the batched solver), the next step's loads issued
    // before this step's hooks.  An entry past the segment's end reads as
    // (0, 0); no branch surrounds the LDS hook, which is given (0, 0) -- a
    // no-op -- for every entry that is not inside the window.
    for (int seg = 0; seg < segments; ++seg) {
        const int64_t s0 = c0 + (c1 - c0) * seg / segments;
        const int64_t s1 = c0 + (c1 - c0) * (seg + 1) / segments;
        if (seg > 0) edge_step_loads<kWinEPT>(gu, gv, s0, s1, step, a, b);
        for (int64_t sb = s0; sb < s1; sb += step) {
            edge_step_loads<kWinEPT>(gu, gv, sb + step, s1, step, na, nb);
            const uint32_t rem = (uint32_t)min(s1 - sb, (int64_t)step);
#pragma unroll
            for (int j = 0; j < kWinEPT; ++j) {
                const bool in = tid + j * nthr < rem;
                const uint32_t x = (uint32_t)a[j], y = (uint32_t)b[j];
                const bool ok = max(x, y) < (uint32_t)n;
                bad |= in && !ok;
                const uint32_t la = x - (uint32_t)base, lb = y - (uint32_t)base;
                const bool win = ok && la < span && lb < span;
                lds_atomic_hook(spi, lds_ld(spi, win ? la : 0u), lds_ld(spi, win ? lb : 0u), true);
                if (in && ok && !win) {
                    ++far;
                    const int32_t pa = ld_rlx(pi + x), pb = ld_rlx(pi + y);
                    if (pa != pb) st_tree<true>(pi + max(pa, pb), min(pa, pb));
                }
            }
#pragma unroll
            for (int j = 0; j < kWinEPT; ++j) {
                a[j] = na[j];
                b[j] = nb[j];
            }
        }
        __syncthreads();
        // Multi-Jump over the window: each vertex climbs to its local root
        // and stores it once; after the last segment the local roots of the
        // non-roots go to pi (two vertices per thread and pass, their climbs interleaved)
        const bool last = seg + 1 == segments;
        for (uint32_t x = tid; x < span; x += 2 * nthr) {
            const uint32_t y = x + nthr;
            const bool has_y = y < span;
            uint32_t p1, p2;
            lds_climb(spi, x, has_y ? y : x, p1, p2);
            if (!last) {
                lds_st(spi, x, p1);
                if (has_y) lds_st(spi, y, p2);
            } else {
                if (p1 != x) st_tree<true>(pi + base + (int32_t)x, base + (int32_t)p1);
                if (has_y && p2 != y) st_tree<true>(pi + base + (int32_t)y, base + (int32_t)p2);
            }
        }
        __syncthreads();
    }
    // the workgroup's count of entries hooked outside its window
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) far += __shfl_xor(far, d, 64);
    if (lane == 0 && far) atomicAdd(&ctrl->win_far, (far + 1) / 2);
    if (bad) atomicOr(&ctrl->status, kStatusRange);
}

// Chunk and window sizes for m entries (whole solve, us; percolated lattices):
// 4096^2, 23 M entries 318 (49,152-entry chunks) and 328 (24,576); 2048^2,
// 5.9 M 170 and 131; 1237 x 1001, 1.7 M 96 (24,576) and 83 (8,192); 300^2,
// 126,000 41 (4,096).
struct WindowShape {
    int32_t chunk, segments;
    uint32_t slots;
};
static WindowShape window_shape(int64_t m) {
    if (m >= 8 << 20) return {49152, 2, 40960};
    if (m >= 3 << 20) return {24576, 2, 24576};
    if (m >= 1 << 20) return {8192, 2, 12288};
    return {4096, 1, 8192};
}

int32_t window_slots(int64_t m) { return (int32_t)window_shape(m).slots; }

hipError_t launch_hook_window(const int32_t* u, const int32_t* v, int64_t m, int32_t* pi,
                              int32_t n, Ctrl* ctrl, uint32_t far_limit, hipStream_t s,
                              int64_t prefix) {
    if (m <= 0) return hipSuccess;
    static hipError_t once = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hook_window),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 40960 * 2);
    if (once != hipSuccess) return once;
    const WindowShape w = window_shape(m);
    const int64_t grid = (m + w.chunk - 1) / w.chunk;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    k_hook_window<<<(int)grid, 1024, w.slots * 2, s>>>(u, v, m, pi, n, ctrl, w.chunk, w.slots,
                                                       w.segments, far_limit, prefix);
    return hipGetLastError();
}

hipError_t prepare_batch_lds() {
    // Allows up to 128 KiB of dynamic LDS; set once, outside any capture.
    static hipError_t once = [] {
        const void* fn[] = {reinterpret_cast<const void*>(&k_batch_lds<true>),
                            reinterpret_cast<const void*>(&k_batch_lds<false>),
                            reinterpret_cast<const void*>(&k_batch_direct<true>),
                            reinterpret_cast<const void*>(&k_batch_direct<false>),
                            reinterpret_cast<const void*>(&k_single_lds<true>),
                            reinterpret_cast<const void*>(&k_single_lds<false>)};
        for (const void* f : fn) {
            const hipError_t e =
                hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 65536 * 2);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }();
    return once;
}

// LDS bytes of the tree array of a graph of at most n vertices: 32-bit slots
// up to kWideMaxN vertices, 16-bit above.
static size_t lds_tree_bytes(int32_t n) {
    return (uint32_t)n <= kWideMaxN ? (size_t)n * 4 : (size_t)kWideMaxN * 4;
}

hipError_t launch_single_lds(const GraphDesc& d, const int32_t* prior, int32_t* status, bool halve,
                             hipStream_t s) {
    if (d.n < 1 || (uint32_t)d.n > kWideMaxN) return hipErrorInvalidValue;
    if (halve)
        k_single_lds<true><<<1, 1024, lds_tree_bytes(d.n), s>>>(d, prior, status);
    else
        k_single_lds<false><<<1, 1024, lds_tree_bytes(d.n), s>>>(d, prior, status);
    return hipGetLastError();
}

// Workgroups of a persistent LDS launch that fit on the CUs at once (LDS, with
// a margin for the kernel's own static LDS, and thread limits, at most 32
// waves per CU).
static int64_t batch_resident(int32_t max_n, int block, int cus) {
    const size_t lds = lds_tree_bytes(max_n);
    const size_t per_cu = std::min<size_t>((size_t)(160 * 1024) / (lds + 256), (size_t)(2048 / block));
    return cus * (int64_t)std::max<size_t>(1, per_cu);
}

// A small graph does not fill 1024 threads, and smaller workgroups keep more
// graphs in flight; a few graphs are solved faster by large ones.  Per call,
// device offsets, at 128 / 256 / 512 / 1024 threads (us): 20,000 graphs of
// up to 256 vertices 75 / 76 / 99 / 167; 8,000 of up to 1,024 vertices 61 /
// 60 / 69 / 98, 20 of them 33 / 30 / 29 / 29; 8,000 of up to 4,096 vertices
// 85 / 73 / 82 / 110, 2,000 of them 65 / 50 / 47 / 50, 200 of them 53 / 40 /
// 35 / 33; 2,000 of up to 8,192 vertices 109 / 75 / 61 / 62.
int batch_block(int32_t count, int32_t max_n) {
    if (count <= 512) return max_n <= 1024 ? 512 : 1024;
    if (max_n <= 256) return 128;
    if (max_n <= 1024) return 256;
    if (max_n <= 4096) return count > 4096 ? 256 : 512;
    return max_n <= 8192 ? 512 : 1024;
}

// The order of the graphs only matters when workgroups take several each, and
// hardly for the smallest ones: otherwise the preparation launches are left
// out (200 graphs of up to 4,096 vertices 28.6 against 33.3 us, 2,000 of up
// to 1,024 vertices 32.8 against 36.0; where it matters: 8,000 of up to 4,096
// vertices 102 against 82; 100,000 of up to 256 vertices 175 against 219).
bool batch_direct(int32_t count, int32_t max_n, int block, int cus) {
    return max_n <= 256 || ((uint32_t)max_n <= kWideMaxN && count <= batch_resident(max_n, block, cus));
}

hipError_t launch_batch_lds(const GraphDesc* descs, int32_t count, int32_t max_n, uint32_t* heads,
                            int32_t* status, bool halve, int cus, hipStream_t s, int block) {
    if (count <= 0) return hipSuccess;
    if (max_n < 1 || max_n > 65536) return hipErrorInvalidValue;
    if (block < 64 || block > 1024 || block % 64) return hipErrorInvalidValue;
    const size_t lds = lds_tree_bytes(max_n);
    const int grid = (int)std::min<int64_t>(count, batch_resident(max_n, block, cus));
    if (halve)
        k_batch_lds<true><<<grid, block, lds, s>>>(descs, count, heads, status);
    else
        k_batch_lds<false><<<grid, block, lds, s>>>(descs, count, heads, status);
    return hipGetLastError();
}

hipError_t launch_batch_direct(const BatchSrc& src, int32_t count, int32_t* status, bool halve,
                               int cus, hipStream_t s, int block) {
    if (count <= 0) return hipSuccess;
    if (src.max_n < 1 || (uint32_t)src.max_n > kWideMaxN) return hipErrorInvalidValue;
    if (block < 64 || block > 1024 || block % 64) return hipErrorInvalidValue;
    const size_t lds = lds_tree_bytes(src.max_n);
    const int grid = (int)std::min<int64_t>(count, batch_resident(src.max_n, block, cus));
    if (halve)
        k_batch_direct<true><<<grid, block, lds, s>>>(src, count, status);
    else
        k_batch_direct<false><<<grid, block, lds, s>>>(src, count, status);
    return hipGetLastError();
}

}  // namespace hookcc
