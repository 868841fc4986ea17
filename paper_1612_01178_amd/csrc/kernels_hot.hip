// Hot-word LDS cache for the giant-component filter (CDNA4).
//
// The filtered Atomic-Hook tests two bits of the giant bitmap (n/8 bytes,
// L2-resident) per edge entry; on skewed graphs those random L2 accesses,
// not the edge stream, bound the pass.  Endpoint frequencies are very
// skewed, so a small set of bitmap words takes a large share of the tests.
// This file keeps the hottest words in LDS:
//
//   k_hot_count   counts sampled endpoint occurrences per bitmap word
//   k_hot_select  for every LDS slot t (of `slots`, 16384 or 32768), picks the
//                 hottest word w = k * slots + t (direct-mapped; ties -> smallest k)
//   k_hot_values  copies the chosen words' current bits (after each bitmap build)
//   k_ahook_hot   the filtered Atomic-Hook, persistent: each workgroup loads
//                 the (tag, word) table into LDS once and answers a bit test
//                 from LDS when the word is cached, else from the bitmap
//
// The table holds copies of bitmap words taken after the bitmap was built,
// so a cached answer is exactly the bitmap's answer; the filter's exactness
// argument is unchanged.
//
// Vertex table (kVertSets two-way sets of one-byte slots, all 160 KiB of
// LDS): a hot vertex shares its bitmap word with 31 mostly cold ones, so word
// slots spend most of their bits on vertices that are rarely tested.  Set s
// caches up to two vertices v = k * kVertSets + s by their tags k; the LDS
// copy keeps a tag only while its vertex is in the giant component (else the
// slot reads as empty), so a tag match answers the test with 1 and anything
// else goes to the bitmap.  Membership only grows (trees only merge), and the
// hot vertices of a graph with a giant component are nearly all in it.
// Five times the hot vertices of the word table in the same LDS (R-MAT 24:
// 56 % of the bit tests answered in LDS, against 35 % for 32,768 word slots).
// Chosen from sampled endpoints (k_vsample, k_vselect); the fused
// Multi-Jump/bitmap pass refreshes the member flags in device memory with
// byte stores, each flag written only by its own vertex.
#include "kernels.hpp"
#include "pair_queue.hpp"

namespace hookcc {

typedef int32_t v4i __attribute__((ext_vector_type(4)));

constexpr uint32_t kHotNone = 0xffffffffu;

__global__ __launch_bounds__(256) void k_hot_zero(uint32_t* __restrict__ p, int64_t words) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// Sample i reads entry floor(i * m / S) and counts the words of both ends.
__global__ __launch_bounds__(256) void k_hot_count(const int32_t* __restrict__ eu,
                                                   const int32_t* __restrict__ ev, int64_t m,
                                                   int32_t n, int64_t S, uint32_t* counts) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= S) return;
    const int64_t e = i * m / S;
    const uint32_t a = (uint32_t)eu[e], b = (uint32_t)ev[e];
    if (a < (uint32_t)n) atomicAdd(counts + (a >> 5), 1u);
    if (b < (uint32_t)n) atomicAdd(counts + (b >> 5), 1u);
}

__global__ __launch_bounds__(256) void k_hot_select(const uint32_t* __restrict__ counts, int64_t nw,
                                                    uint32_t* __restrict__ tags, int slots) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= slots) return;
    uint32_t best_k = kHotNone, best_c = 0;
    for (int64_t w = t, k = 0; w < nw; w += slots, ++k) {
        const uint32_t c = counts[w];
        if (best_k == kHotNone || c > best_c) {
            best_k = (uint32_t)k;
            best_c = c;
        }
    }
    tags[t] = best_k;
}

__global__ __launch_bounds__(256) void k_hot_values(const uint32_t* __restrict__ bits,
                                                    const uint32_t* __restrict__ tags,
                                                    uint32_t* __restrict__ vals, const Ctrl* ctrl,
                                                    int slots) {
    if (!ctrl->filter_on) return;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= slots) return;
    const uint32_t k = tags[t];
    vals[t] = (k == kHotNone) ? 0u : bits[(int64_t)k * slots + t];
}

// Vertex table selection, without global atomics (random atomics over a
// per-vertex count array run at about 2 x 10^10/s here, 0.2 ms for 2^22
// endpoints).  Sampled entries: up to kVertRuns runs of 64 consecutive
// entries spread evenly over the list.  Endpoints x < n with tag
// x / kVertSets < kVertTagNone are candidates; bucket(x) is the range of
// kVBucketSets sets that holds set x mod kVertSets.
//   k_vsample  workgroup g takes its part of the runs, histograms its
//              candidates by bucket in LDS, scans, and writes them grouped by
//              bucket into its own part of `region`, with the per-bucket
//              counts and offsets (cnt, off: [part][bucket]).
//   k_vselect  workgroup b gathers bucket b from every part, counts every
//              (set, tag) pair in LDS, and gives each set the kVertWays tags
//              with the largest counts (ties -> smaller tag).
// Entry of sample s: lane s % 64 of run s / 64, which starts at about
// (s / 64) * (m - 64) / runs (step = (m - 64) / runs; m >= 64).
__device__ __forceinline__ int64_t vsample_entry(int64_t s, int64_t m, double step) {
    const int64_t r0 = (int64_t)((double)(s >> 6) * step);
    return min(r0, m - 64) + (s & 63);
}

__device__ __forceinline__ bool vcandidate(uint32_t x, int32_t n) {
    return x < (uint32_t)n && x / kVertSets < kVertTagNone;
}

__device__ __forceinline__ uint32_t vbucket(uint32_t x) {
    return (x % kVertSets) / kVBucketSets;
}

// Exclusive scan of one value per thread over a 256-thread workgroup;
// returns this thread's base (the sum of the values of lower threads).
__device__ __forceinline__ uint32_t block_scan(uint32_t pair, uint32_t* wsum) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t incl = pair;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    uint32_t base = 0;
    for (int i = 0; i < w; ++i) base += wsum[i];
    return base + incl - pair;
}

template <int RUNS>  // of one part
__global__ __launch_bounds__(256) void k_vsample(const int32_t* __restrict__ eu,
                                                 const int32_t* __restrict__ ev, int64_t m,
                                                 int32_t n, int64_t runs, double step,
                                                 uint32_t* __restrict__ region,
                                                 uint32_t* __restrict__ cnt,
                                                 uint32_t* __restrict__ off) {
    constexpr int kVPerThread = RUNS * 64 / 256;  // sampled entries per thread
    constexpr int kPer = (kVBuckets + 255) / 256;  // buckets per thread in the scan
    __shared__ uint32_t hist[256 * kPer];
    __shared__ uint32_t cur[256 * kPer];
    __shared__ uint32_t wsum[4];
    __shared__ uint32_t stage[RUNS * 64 * 2];  // the part, grouped by bucket
    const int g = blockIdx.x;
    const int tid = threadIdx.x;
#pragma unroll
    for (int q = 0; q < kPer; ++q) hist[kPer * tid + q] = 0;
    // this thread's samples, all loads issued before any is used
    const int64_t s0 = (int64_t)g * RUNS * 64;
    const int64_t s1 = min(runs, (int64_t)(g + 1) * RUNS) * 64;
    uint32_t x[kVPerThread], y[kVPerThread];
#pragma unroll
    for (int i = 0; i < kVPerThread; ++i) {
        const int64_t s = s0 + tid + (int64_t)i * 256;
        const int64_t e = s < s1 ? vsample_entry(s, m, step) : 0;
        x[i] = s < s1 ? (uint32_t)eu[e] : 0xffffffffu;
        y[i] = s < s1 ? (uint32_t)ev[e] : 0xffffffffu;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kVPerThread; ++i) {
        if (vcandidate(x[i], n)) atomicAdd(&hist[vbucket(x[i])], 1u);
        if (vcandidate(y[i], n)) atomicAdd(&hist[vbucket(y[i])], 1u);
    }
    __syncthreads();
    // exclusive scan: thread tid owns buckets kPer * tid .. kPer * tid + kPer - 1
    uint32_t own = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) own += hist[kPer * tid + q];
    uint32_t at = block_scan(own, wsum);
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int bk = kPer * tid + q;
        const uint32_t h = hist[bk];
        cur[bk] = at;
        if (bk < kVBuckets) {
            cnt[(int64_t)g * kVBuckets + bk] = h;
            off[(int64_t)g * kVBuckets + bk] = at;
        }
        at += h;
    }
    const uint32_t total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kVPerThread; ++i) {
        if (vcandidate(x[i], n)) stage[atomicAdd(&cur[vbucket(x[i])], 1u)] = x[i];
        if (vcandidate(y[i], n)) stage[atomicAdd(&cur[vbucket(y[i])], 1u)] = y[i];
    }
    __syncthreads();
    uint32_t* part = region + (int64_t)g * kVPartCap;
    for (uint32_t i = tid; i < total; i += 256) part[i] = stage[i];
}

__global__ __launch_bounds__(256) void k_vselect(const uint32_t* __restrict__ region,
                                                 const uint32_t* __restrict__ cnt,
                                                 const uint32_t* __restrict__ off, int parts,
                                                 int32_t n, uint8_t* __restrict__ tags) {
    constexpr int kTags = (int)kVertTagNone;  // candidate tags 0 .. kTags - 1
    // 16-bit counters, two per word (counter i in half i & 1 of word i / 2);
    // at most 65,535 endpoints of a bucket are counted, so none overflows
    __shared__ uint32_t c[kVBucketSets * kTags / 2 + 1];
    __shared__ uint32_t start[kVPartsMax + 1];  // first flat index of each part's piece
    __shared__ uint32_t src0[kVPartsMax];       // its offset in region
    __shared__ uint32_t wsum[4];
    static_assert(kVPartsMax == 256 && kVBucketSets <= 256, "one part per thread");
    const int b = blockIdx.x;
    const int tid = threadIdx.x;
    // the bucket's piece of every part, flattened: piece of part g holds the
    // flat indices [start[g], start[g + 1])
    const uint32_t k = tid < parts ? cnt[(int64_t)tid * kVBuckets + b] : 0u;
    src0[tid] = tid < parts ? (uint32_t)(tid * kVPartCap) + off[(int64_t)tid * kVBuckets + b] : 0u;
    for (int i = tid; i < kVBucketSets * kTags / 2 + 1; i += 256) c[i] = 0;
    const uint32_t st = block_scan(k, wsum);
    start[tid] = st;
    if (tid == 255) start[256] = st + k;
    __syncthreads();
    const uint32_t total = min(start[256], 65535u);
    constexpr int kUnroll = 8;  // independent gathers in flight per thread
    for (uint32_t j0 = 0; j0 < total; j0 += 256 * kUnroll) {
        uint32_t xs[kUnroll];
#pragma unroll
        for (int q = 0; q < kUnroll; ++q) {
            const uint32_t j = j0 + q * 256 + tid;
            // the last part g with start[g] <= j (start[0] = 0; parts past
            // the last non-empty piece start at total > j)
            uint32_t g = 0;
#pragma unroll
            for (uint32_t d = kVPartsMax / 2; d >= 1; d >>= 1)
                if (start[g + d] <= j) g += d;
            const uint32_t at = j < total ? src0[g] + (j - start[g]) : 0u;  // 0: in bounds
            xs[q] = j < total ? region[at] : 0xffffffffu;
        }
#pragma unroll
        for (int q = 0; q < kUnroll; ++q) {
            if (xs[q] == 0xffffffffu) continue;
            const uint32_t i = (xs[q] % kVertSets % kVBucketSets) * kTags + xs[q] / kVertSets;
            atomicAdd(&c[i >> 1], 1u << (16 * (i & 1)));
        }
    }
    __syncthreads();
    // the two largest counts of set s (ties -> smaller tag); tags of vertices
    // past n are not candidates.  Threads 4i .. 4i + 3 scan a quarter of set
    // i's tags each, then merge their top two in two butterfly steps.
    static_assert(4 * kVBucketSets == 256 && kVertWays == 2, "four threads per set, two ways");
    constexpr int kQuarter = (kTags + 3) / 4;
    const int set = tid >> 2, part = tid & 3;
    const int64_t s = (int64_t)b * kVBucketSets + set;
    const int64_t tags_n = (int64_t)n > s ? ((int64_t)n - s + kVertSets - 1) / kVertSets : 0;
    const int q0 = part * kQuarter;
    const int q1 = (int)min<int64_t>(tags_n, min(kTags, (part + 1) * kQuarter));
    uint32_t k1 = kVertTagNone, c1 = 0, k2 = kVertTagNone, c2 = 0;
#pragma unroll 8
    for (int q = q0; q < q1; ++q) {
        const uint32_t i = set * kTags + q;
        const uint32_t cc = c[i >> 1] >> (16 * (i & 1)) & 0xffffu;
        if (k1 == kVertTagNone || cc > c1) {
            k2 = k1;
            c2 = c1;
            k1 = (uint32_t)q;
            c1 = cc;
        } else if (k2 == kVertTagNone || cc > c2) {
            k2 = (uint32_t)q;
            c2 = cc;
        }
    }
    // merge with the partner's list: the order is count descending, then tag
    // ascending (the same in every thread, so all four end with one result)
    auto before = [](uint32_t ka, uint32_t ca, uint32_t kb, uint32_t cb) {
        return ka != kVertTagNone && (kb == kVertTagNone || ca > cb || (ca == cb && ka < kb));
    };
#pragma unroll
    for (int d = 1; d <= 2; d <<= 1) {
        const uint32_t o1 = __shfl_xor(k1, d, 64), p1 = __shfl_xor(c1, d, 64);
        const uint32_t o2 = __shfl_xor(k2, d, 64), p2 = __shfl_xor(c2, d, 64);
        if (before(k1, c1, o1, p1)) {
            if (!before(k2, c2, o1, p1)) {
                k2 = o1;
                c2 = p1;
            }
        } else {
            if (!before(k1, c1, o2, p2)) {
                k2 = o2;
                c2 = p2;
            } else {
                k2 = k1;
                c2 = c1;
            }
            k1 = o1;
            c1 = p1;
        }
    }
    if (part == 0) {
        tags[2 * s] = (uint8_t)k1;
        tags[2 * s + 1] = (uint8_t)k2;
        tags[kVertSlots + 2 * s] = tags[kVertSlots + 2 * s + 1] = 0;  // member flags
    }
}

template <int EPT>
__device__ __forceinline__ void load_tile(const int32_t* __restrict__ p, int64_t e0,
                                          int64_t stride, int64_t end, bool vec,
                                          int32_t (&x)[EPT]) {
#pragma unroll
    for (int k = 0; k < EPT / 4; ++k) {
        const int64_t e = e0 + k * stride;
        if (vec && e + 3 < end) {
            v4i q = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p + e));
            x[4 * k + 0] = q.x;
            x[4 * k + 1] = q.y;
            x[4 * k + 2] = q.z;
            x[4 * k + 3] = q.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                x[4 * k + j] = (e + j < end) ? __builtin_nontemporal_load(p + e + j) : 0;
        }
    }
}

// Atomic-Hook climb (Fig. 3, top), cached loads; see atomic_hook in
// kernels_core.hip for the argument.
__device__ __forceinline__ void hot_climb(int32_t* pi, int32_t pu, int32_t pv, bool halve) {
    uint32_t step = 0;
    while (pu != pv) {
        const int32_t H = pu > pv ? pu : pv;
        const int32_t L = pu > pv ? pv : pu;
        int32_t found = ld_tree<false>(pi + H);
        if (found == H) {
            found = cas_root(pi + H, H, L);
            if (found == H) return;
        }
        pu = ld_tree<false>(pi + found);
        pv = ld_tree<false>(pi + L);
        if (halve && pu != found && step++ % kHalveEveryFiltered == 0)
            halve_to(pi + H, pu);  // path halving
    }
}

// SLOTS slots with tags of type TagT (16384 x uint16 = 96 KiB of LDS with the
// words, or 32768 x uint8 = 160 KiB); a tag equal to TagT's maximum marks an
// empty slot (also used for a word index too large for the tag type).
template <int EPT, int SLOTS, typename TagT>
__global__ __launch_bounds__(1024) void k_ahook_hot(const int32_t* __restrict__ eu,
                                                    const int32_t* __restrict__ ev, int64_t begin,
                                                    int64_t end, bool vec, int32_t* pi, int32_t n,
                                                    Ctrl* ctrl, const uint32_t* __restrict__ bits,
                                                    const uint32_t* __restrict__ gtags,
                                                    const uint32_t* __restrict__ gvals, bool halve,
                                                    bool sym) {
    constexpr uint32_t kEmpty = (uint32_t)(TagT)(~(TagT)0);
    __shared__ TagT ltag[SLOTS];
    __shared__ uint32_t lval[SLOTS];
    const bool filter = ctrl->filter_on != 0;
    const int32_t g = ctrl->giant;
    if (filter) {
        for (uint32_t t = threadIdx.x; t < (uint32_t)SLOTS; t += blockDim.x) {
            const uint32_t k = gtags[t];
            ltag[t] = (TagT)((k == kHotNone || k >= kEmpty) ? kEmpty : k);
            lval[t] = gvals[t];
        }
        __syncthreads();
    }
    const int64_t stride = (int64_t)blockDim.x * 4;
    const int64_t tile = (int64_t)blockDim.x * EPT;
    bool bad = false;
    for (int64_t t0 = begin + (int64_t)blockIdx.x * tile; t0 < end; t0 += (int64_t)gridDim.x * tile) {
        const int64_t e0 = t0 + (int64_t)threadIdx.x * 4;
        int32_t a[EPT], b[EPT];
        load_tile<EPT>(eu, e0, stride, end, vec, a);
        load_tile<EPT>(ev, e0, stride, end, vec, b);
        uint32_t act = 0;
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const bool in = (uint32_t)a[j] < (uint32_t)n && (uint32_t)b[j] < (uint32_t)n;
            bad |= !in;
            if (in && a[j] != b[j] && !(sym && a[j] > b[j])) act |= 1u << j;
        }
        int32_t pa[EPT], pb[EPT];
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            if (!(act >> j & 1)) continue;
            uint32_t ba = 0, bb = 0;
            if (filter) {
                const uint32_t wa = (uint32_t)a[j] >> 5, wb = (uint32_t)b[j] >> 5;
                const uint32_t sa = wa & (SLOTS - 1), sb = wb & (SLOTS - 1);
                const uint32_t ka = wa / SLOTS, kb = wb / SLOTS;
                // ka == kEmpty can never be cached (it is the empty marker).
                // Two separate (relaxed atomic) loads, the LDS one
                // unconditional: plain loads here are merged into one load
                // from a selected address, which is a flat load that also
                // waits on the LDS traffic.
                const bool hita = ka < kEmpty && (uint32_t)ltag[sa] == ka;
                const bool hitb = kb < kEmpty && (uint32_t)ltag[sb] == kb;
                uint32_t worda = __hip_atomic_load(lval + sa, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                uint32_t wordb = __hip_atomic_load(lval + sb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (!hita) worda = __hip_atomic_load(bits + wa, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (!hitb) wordb = __hip_atomic_load(bits + wb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                ba = worda >> (a[j] & 31) & 1;
                bb = wordb >> (b[j] & 31) & 1;
            }
            if (ba & bb) {
                act &= ~(1u << j);
            } else {
                pa[j] = ba ? g : ld_tree<false>(pi + a[j]);
                pb[j] = bb ? g : ld_tree<false>(pi + b[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < EPT; ++j)
            if (act >> j & 1) hot_climb(pi, pa[j], pb[j], halve);
    }
    if (bad) atomicOr(&ctrl->status, kStatusRange);
}

hipError_t launch_hot_prepare(const int32_t* u, const int32_t* v, int64_t m, int32_t n,
                              uint32_t* counts, uint32_t* tags, int slots, hipStream_t s) {
    if (slots != 16384 && slots != 32768) return hipErrorInvalidValue;
    const int64_t nw = ((int64_t)n + 31) / 32;
    k_hot_zero<<<1024, 256, 0, s>>>(counts, nw);
    const int64_t S = std::min<int64_t>(m, int64_t(1) << 19);
    if (S > 0) k_hot_count<<<(int)((S + 255) / 256), 256, 0, s>>>(u, v, m, n, S, counts);
    k_hot_select<<<slots / 256, 256, 0, s>>>(counts, nw, tags, slots);
    return hipGetLastError();
}

hipError_t launch_hot_values(const uint32_t* bits, const uint32_t* tags, uint32_t* vals,
                             const Ctrl* ctrl, int slots, hipStream_t s) {
    if (slots != 16384 && slots != 32768) return hipErrorInvalidValue;
    k_hot_values<<<slots / 256, 256, 0, s>>>(bits, tags, vals, ctrl, slots);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------- filtered hook
// Entries [t0, t0 + blockDim.x * EPT) of one edge array, 0 past `end`: groups
// of four consecutive ones per lane, or single ones (EPT < 4).
template <int EPT>
__device__ __forceinline__ void load_step(const int32_t* __restrict__ p, int64_t t0, int64_t end,
                                          bool vec, int32_t (&x)[EPT]) {
    if constexpr (EPT >= 4) {
        load_tile<EPT>(p, t0 + (int64_t)threadIdx.x * 4, (int64_t)blockDim.x * 4, end, vec, x);
    } else {
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const int64_t e = t0 + (int64_t)j * blockDim.x + threadIdx.x;
            x[j] = e < end ? __builtin_nontemporal_load(p + e) : 0;
        }
    }
}

// Filtered Atomic-Hook of entries [begin, end), persistent.  A membership
// test is answered in LDS:
//   kFilterBits    the whole giant bitmap (n <= kLdsBitsMaxN).  The pass is
//                  then bound by the edge stream and by the climbs of the
//                  entries it keeps (R-MAT 20, 2^24 entries: 413 us with the
//                  vertex table and climbs in place, 194 us);
//   kFilterVertex  the vertex table (a slot's tag kept only while its member
//                  flag is set): 1 when set x mod kVertSets holds the tag
//                  x / kVertSets, else the bitmap in device memory decides.
//                  Bound by the address and L2 rate of those tests (R-MAT 24
//                  3.46 ms with the kept entries hooked in place, 3.24 with
//                  the queue, 3.12 with the queue passed by where all entries
//                  of a wave's step are inside the giant);
//   kFilterPart    the bitmap of the first kLdsBitsMaxN vertices; the others'
//                  tests go to device memory (R-MAT 21, 50 M entries: 526 us
//                  with the vertex table, 481).
// Only lanes whose test is not answered in LDS load: a load of a fixed word by
// the other lanes costs more than the branch (R-MAT 24 3.50 ms).
enum { kFilterBits = 0, kFilterVertex = 1, kFilterPart = 2 };

template <int EPT, int MODE>
__global__ __launch_bounds__(1024) void k_filter(const int32_t* __restrict__ eu,
                                                 const int32_t* __restrict__ ev, int64_t begin,
                                                 int64_t end, bool vec, int32_t* pi, int32_t n,
                                                 Ctrl* ctrl, const uint32_t* __restrict__ bits,
                                                 const uint8_t* __restrict__ gtab, bool halve,
                                                 bool sym) {
    extern __shared__ uint32_t lds[];
    if (ctrl->windowed) return;  // nothing is left to hook
    const bool filter = ctrl->filter_on != 0;
    const int32_t g = ctrl->giant;
    if (filter) {
        if (MODE != kFilterVertex) {
            const uint32_t words = ((uint32_t)min(n, kLdsBitsMaxN) + 31) / 32;
            for (uint32_t i = threadIdx.x * 4; i < words; i += blockDim.x * 4) {
                if (i + 3 < words) {
                    *reinterpret_cast<v4i*>(lds + i) = *reinterpret_cast<const v4i*>(bits + i);
                } else {
                    for (uint32_t k = i; k < words; ++k) lds[k] = bits[k];
                }
            }
        } else {
            // tag | 0xff per byte whose member flag (0 or 1) is 0: bytes of
            // (0x01010101 - flags) are 1 - flag, times 0xff without carries
            const v4i* tg = reinterpret_cast<const v4i*>(gtab);
            const v4i* fl = reinterpret_cast<const v4i*>(gtab + kVertSlots);
            v4i* dst = reinterpret_cast<v4i*>(lds);
            for (uint32_t i = threadIdx.x; i < (uint32_t)(kVertSlots / 16); i += blockDim.x) {
                const v4i t = tg[i], f = fl[i];
                v4i o;
                o.x = (int32_t)((uint32_t)t.x | (0x01010101u - (uint32_t)f.x) * 0xffu);
                o.y = (int32_t)((uint32_t)t.y | (0x01010101u - (uint32_t)f.y) * 0xffu);
                o.z = (int32_t)((uint32_t)t.z | (0x01010101u - (uint32_t)f.z) * 0xffu);
                o.w = (int32_t)((uint32_t)t.w | (0x01010101u - (uint32_t)f.w) * 0xffu);
                dst[i] = o;
            }
        }
        __syncthreads();
    }
    const uint16_t* lset = reinterpret_cast<const uint16_t*>(lds);
    const int64_t tile = (int64_t)blockDim.x * EPT;
    uint32_t top = 0;  // largest endpoint seen
    PairQueue q;
    for (int64_t t0 = begin + (int64_t)blockIdx.x * tile; t0 < end; t0 += (int64_t)gridDim.x * tile) {
        int32_t a[EPT], b[EPT];
        load_step<EPT>(eu, t0, end, vec, a);
        load_step<EPT>(ev, t0, end, vec, b);
        // bit j of ma, mb: entry j's first, second endpoint is in the giant.
        // An endpoint out of range is tested as n - 1; `top` reports it.
        uint32_t ma = 0, mb = 0;
        if (filter) {
            uint32_t wa[EPT], wb[EPT];
#pragma unroll
            for (int j = 0; j < EPT; ++j) {
                const uint32_t xa = min((uint32_t)a[j], (uint32_t)n - 1), xb = min((uint32_t)b[j], (uint32_t)n - 1);
                if (MODE == kFilterBits) {
                    wa[j] = lds[xa >> 5] >> (xa & 31);
                    wb[j] = lds[xb >> 5] >> (xb & 31);
                } else if (MODE == kFilterPart) {
                    const bool hita = xa < (uint32_t)kLdsBitsMaxN, hitb = xb < (uint32_t)kLdsBitsMaxN;
                    wa[j] = lds[hita ? xa >> 5 : 0u];
                    wb[j] = lds[hitb ? xb >> 5 : 0u];
                    if (!hita) wa[j] = bits[xa >> 5];
                    if (!hitb) wb[j] = bits[xb >> 5];
                    wa[j] >>= xa & 31;
                    wb[j] >>= xb & 31;
                } else {
                    // a tag of kVertTagNone (the empty marker) or more never hits
                    const uint32_t sa = lset[xa % kVertSets], sb = lset[xb % kVertSets];
                    const uint32_t ka = xa / kVertSets, kb = xb / kVertSets;
                    const bool hita = ka < kVertTagNone && ((sa & 0xffu) == ka || (sa >> 8) == ka);
                    const bool hitb = kb < kVertTagNone && ((sb & 0xffu) == kb || (sb >> 8) == kb);
                    wa[j] = wb[j] = 1;
                    if (!hita) wa[j] = bits[xa >> 5] >> (xa & 31);
                    if (!hitb) wb[j] = bits[xb >> 5] >> (xb & 31);
                }
            }
#pragma unroll
            for (int j = 0; j < EPT; ++j) {
                ma |= (wa[j] & 1) << j;
                mb |= (wb[j] & 1) << j;
            }
        }
        // Nearly every step is inside the giant altogether.
        constexpr uint32_t kAll = (1u << EPT) - 1;
#pragma unroll
        for (int j = 0; j < EPT; ++j) top = max(top, max((uint32_t)a[j], (uint32_t)b[j]));
        if (!__any((ma & mb) != kAll)) continue;
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const uint32_t ba = ma >> j & 1, bb = mb >> j & 1;
            const bool in = max((uint32_t)a[j], (uint32_t)b[j]) < (uint32_t)n;
            const bool keep = in && a[j] != b[j] && !(ba & bb) && !(sym && a[j] > b[j]);
            // an endpoint in the giant starts its climb at the giant's root
            q.push(keep, ba ? g : a[j], bb ? g : b[j], pi, halve);
        }
    }
    q.flush(pi, halve);
    if (top >= (uint32_t)n) atomicOr(&ctrl->status, kStatusRange);
}

hipError_t launch_hot_vprepare(const int32_t* u, const int32_t* v, int64_t m, int32_t n,
                               uint32_t* scratch, uint8_t* table, hipStream_t s) {
    uint32_t* region = scratch;
    uint32_t* cnt = region + (int64_t)kVPartsMax * kVPartCap;
    uint32_t* off = cnt + kVPartsMax * kVBuckets;
    // one run of 64 in 8,192 entries, at most kVertRuns (R-MAT 21, 50 M
    // entries: selection 59 us with 2^15 runs, 24 us with 6,144)
    const int64_t want = std::max<int64_t>(64, std::min<int64_t>(kVertRuns, m / 8192));
    const int64_t runs = m >= 64 ? std::min<int64_t>(want, m / 64) : 0;
    const bool few = runs <= (int64_t)kVPartsMax * kVRunsPerPartShort;
    const int per = few ? kVRunsPerPartShort : kVRunsPerPart;
    const int parts = (int)((runs + per - 1) / per);
    const double step = runs > 0 ? (double)(m - 64) / (double)runs : 0.0;
    if (parts > 0 && few)
        k_vsample<kVRunsPerPartShort><<<parts, 256, 0, s>>>(u, v, m, n, runs, step, region, cnt, off);
    else if (parts > 0)
        k_vsample<kVRunsPerPart><<<parts, 256, 0, s>>>(u, v, m, n, runs, step, region, cnt, off);
    k_vselect<<<kVBuckets, 256, 0, s>>>(region, cnt, off, parts, n, table);  // tags
    return hipGetLastError();
}

template <int MODE>
static hipError_t filter_dispatch(const int32_t* u, const int32_t* v, int64_t begin, int64_t end,
                                  int32_t* pi, int32_t n, Ctrl* ctrl, const uint32_t* bits,
                                  const uint8_t* table, bool halve, bool sym, hipStream_t s) {
    if (end <= begin) return hipSuccess;
    static hipError_t once = [] {
        const void* fn[] = {reinterpret_cast<const void*>(&k_filter<1, MODE>),
                            reinterpret_cast<const void*>(&k_filter<2, MODE>),
                            reinterpret_cast<const void*>(&k_filter<4, MODE>),
                            reinterpret_cast<const void*>(&k_filter<8, MODE>)};
        for (const void* f : fn) {
            const hipError_t e =
                hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }();
    if (once != hipSuccess) return once;
    const int block = 1024;
    const size_t lds = MODE == kFilterBits ? ((size_t)n + 127) / 128 * 16 : MODE == kFilterPart ? (size_t)kLdsBytes : (size_t)kVertSlots;
    if (lds > (size_t)kLdsBytes) return hipErrorInvalidValue;
    // workgroups that are resident at once: two per CU where the LDS allows
    const int64_t cap = (int64_t)device_cu_count() * (2 * lds <= (size_t)kLdsBytes ? 2 : 1);
    // 8 entries per thread; with the bitmap in LDS fewer where that leaves
    // CUs without a tile: a short segment is bound by the chain of climbs of
    // each wave (R-MAT 18, 2^19 entries: 42 us at 8 entries, 64 CUs).  On the
    // larger graphs of the vertex table the first segments' climbs contend for
    // the hubs, and more of them at once are slower (R-MAT 23, 2^20 entries:
    // 91 us at 2 entries, 256 CUs, 47 us at 8, 128 CUs).
    int ept = 8;
    while (MODE == kFilterBits && ept > 1 && end - begin < cap * block * ept) ept /= 2;
    const int64_t tiles = (end - begin + (int64_t)block * ept - 1) / ((int64_t)block * ept);
    const int grid = (int)std::min<int64_t>(tiles, cap);
    const bool vec = (((uintptr_t)(u + begin) | (uintptr_t)(v + begin)) & 15) == 0;
    switch (ept) {
        case 1: k_filter<1, MODE><<<grid, block, lds, s>>>(u, v, begin, end, vec, pi, n, ctrl, bits, table, halve, sym); break;
        case 2: k_filter<2, MODE><<<grid, block, lds, s>>>(u, v, begin, end, vec, pi, n, ctrl, bits, table, halve, sym); break;
        case 4: k_filter<4, MODE><<<grid, block, lds, s>>>(u, v, begin, end, vec, pi, n, ctrl, bits, table, halve, sym); break;
        default: k_filter<8, MODE><<<grid, block, lds, s>>>(u, v, begin, end, vec, pi, n, ctrl, bits, table, halve, sym); break;
    }
    return hipGetLastError();
}

hipError_t launch_filter_bits(const int32_t* u, const int32_t* v, int64_t begin, int64_t end,
                              int32_t* pi, int32_t n, Ctrl* ctrl, const uint32_t* bits, bool halve,
                              bool sym, hipStream_t s) {
    if (n > kLdsBitsMaxN)
        return filter_dispatch<kFilterPart>(u, v, begin, end, pi, n, ctrl, bits, nullptr, halve, sym, s);
    return filter_dispatch<kFilterBits>(u, v, begin, end, pi, n, ctrl, bits, nullptr, halve, sym, s);
}

hipError_t launch_filter_vertex(const int32_t* u, const int32_t* v, int64_t begin, int64_t end,
                                int32_t* pi, int32_t n, Ctrl* ctrl, const uint32_t* bits,
                                const uint8_t* table, bool halve, bool sym, hipStream_t s) {
    return filter_dispatch<kFilterVertex>(u, v, begin, end, pi, n, ctrl, bits, table, halve, sym, s);
}

template <int SLOTS, typename TagT>
static hipError_t ahook_hot_ept(int ept, int grid, int block, hipStream_t s, const int32_t* u,
                                const int32_t* v, int64_t begin, int64_t end, bool vec, int32_t* pi,
                                int32_t n, Ctrl* ctrl, const uint32_t* bits, const uint32_t* tags,
                                const uint32_t* vals, bool halve, bool sym) {
    switch (ept) {
        case 4: k_ahook_hot<4, SLOTS, TagT><<<grid, block, 0, s>>>(u, v, begin, end, vec, pi, n, ctrl, bits, tags, vals, halve, sym); break;
        case 8:
        case 16:  // the 16-entry tile does not fit the registers next to the LDS table; run 8
            k_ahook_hot<8, SLOTS, TagT><<<grid, block, 0, s>>>(u, v, begin, end, vec, pi, n, ctrl, bits, tags, vals, halve, sym); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_ahook_hot(const int32_t* u, const int32_t* v, int64_t begin, int64_t end,
                            int32_t* pi, int32_t n, Ctrl* ctrl, const uint32_t* bits,
                            const uint32_t* tags, const uint32_t* vals, int ept, int slots,
                            bool halve, bool sym, hipStream_t s) {
    if (end <= begin) return hipSuccess;
    const int block = 1024;
    const int64_t tile = (int64_t)block * ept;
    const int64_t tiles = (end - begin + tile - 1) / tile;
    const int64_t cap = (int64_t)device_cu_count();  // one 1024-thread workgroup per CU (LDS)
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(tiles, cap));
    const bool vec = (((uintptr_t)(u + begin) | (uintptr_t)(v + begin)) & 15) == 0;
    if (slots == 16384)
        return ahook_hot_ept<16384, uint16_t>(ept, grid, block, s, u, v, begin, end, vec, pi, n,
                                              ctrl, bits, tags, vals, halve, sym);
    if (slots == 32768)
        return ahook_hot_ept<32768, uint8_t>(ept, grid, block, s, u, v, begin, end, vec, pi, n,
                                             ctrl, bits, tags, vals, halve, sym);
    return hipErrorInvalidValue;
}

}  // namespace hookcc
