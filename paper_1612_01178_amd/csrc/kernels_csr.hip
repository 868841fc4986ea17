// Atomic-Hook over a CSR adjacency (row_ptr[n+1], col[m]): entry i of row r
// is the pair (r, col[i]).  The paper's hook works on any subsets of E
// (Fig. 4), so the solve is the same as for pair lists; only the way an
// entry's first endpoint is found differs.  The automatic plans use the
// kernels by tiles further down; k_ahook_csr serves calls that set segments or
// the filter's options themselves, or that ask for the Atomic-Hook, and those for
// which the other plans' scratch cannot be had.
//
// k_ahook_csr finds rows on the fly.  Each workgroup takes a tile of
// consecutive entries and finds the rows spanning it (row_ptr is int64 and
// non-decreasing) with a 32-ary search per tile end, both run at once by the
// first wave (half a wave each): 5 dependent rounds of loads for 16M rows
// instead of the 24 of a binary search, which at one tile per 2,048 entries
// otherwise dominate the pass.  The tile then loads that window of row_ptr
// into LDS, and every thread finds the row of its first entry by a binary
// search in LDS, advancing linearly for its following entries.  A tile whose
// window exceeds the LDS budget (many empty rows) searches row_ptr in device
// memory instead.
//
// With the giant filter, the row's bit is tested once per group of four
// consecutive entries (they nearly always share the row) instead of once
// per entry: on a skewed CSR graph the per-entry cost drops to one bit test.
// `sym`: the adjacency is symmetric (every pair stored in both rows), so
// only the entries with col > row are hooked: the copy of each pair kept is
// the one in the smaller endpoint's row, so the first segments (the first
// rows) already join the low ids to the whole graph and the giant component
// forms before the filter samples for it.  Keeping col < row instead hooks
// only pairs inside the row prefix seen so far, and the filter finds no
// giant until late.
#include "kernels.hpp"
#include "pair_queue.hpp"

namespace hookcc {

constexpr int kCsrWindow = 4096;  // rows of row_ptr held in LDS per tile

// Largest r in [0, n - 1] with rp[r] <= e, by lanes [half*32, half*32 + 32)
// of the calling wave (every lane of the wave must call it; each half-wave
// searches for its own e).  Each round, the half-wave's lanes probe 32
// evenly spaced rows of the current interval, and the interval shrinks to
// the gap after the last probe that is still <= e.
__device__ __forceinline__ int64_t upper_row32(const int64_t* __restrict__ rp, int32_t n, int64_t e) {
    const int lane = threadIdx.x & 63;
    const int sub = lane & 31;
    const int half = lane >> 5;
    int64_t lo = 0, hi = (int64_t)n - 1;  // answer in [lo, hi]; rp[0] <= e assumed
    while (true) {
        const int64_t span = hi - lo + 1;
        const bool last = span <= 32;
        // probe k (1..32) of this half-wave
        const int64_t probe = last ? lo + sub : lo + (span * (sub + 1)) / 33;
        const bool ok = probe <= hi && rp[probe] <= e;
        const uint64_t mk = __ballot(ok);
        const uint32_t mine = (uint32_t)(mk >> (32 * half));
        // rp is non-decreasing, so the probes that pass form a prefix
        const int cnt = __popc(mine);
        if (last) return lo + cnt - 1 < lo ? lo : lo + cnt - 1;
        // probes p_1 < ... < p_32; the answer lies in [p_cnt, p_{cnt+1} - 1]
        const int64_t nlo = cnt ? lo + (span * cnt) / 33 : lo;
        const int64_t nhi = cnt < 32 ? lo + (span * (cnt + 1)) / 33 - 1 : hi;
        lo = nlo;
        hi = nhi < lo ? lo : nhi;
    }
}

__device__ __forceinline__ int64_t upper_row(const int64_t* __restrict__ rp, int64_t lo, int64_t hi,
                                             int64_t e) {
    // largest r in [lo, hi] with rp[r] <= e (rp[lo] <= e assumed)
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (rp[mid] <= e) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

template <int EPT>
__global__ __launch_bounds__(512) void k_ahook_csr(const int64_t* __restrict__ row_ptr,
                                                   const int32_t* __restrict__ col, int32_t n,
                                                   int64_t begin, int64_t end, int32_t* pi,
                                                   Ctrl* ctrl, const uint32_t* __restrict__ bits,
                                                   bool filter, bool sym, bool halve) {
    __shared__ int64_t win[kCsrWindow + 1];
    __shared__ int64_t r_lo_sh, r_hi_sh;
    const int64_t tile = (int64_t)blockDim.x * EPT;
    const int64_t t0 = begin + (int64_t)blockIdx.x * tile;
    const int64_t t1 = min(end, t0 + tile);  // exclusive
    if (threadIdx.x < 64) {
        // half-wave 0 finds the row of t0, half-wave 1 the row of t1 - 1
        const int64_t r = upper_row32(row_ptr, n, threadIdx.x < 32 ? t0 : t1 - 1);
        if (threadIdx.x == 0) r_lo_sh = r;
        if (threadIdx.x == 32) r_hi_sh = r;
    }
    __syncthreads();
    const int64_t r_lo = r_lo_sh;
    const int64_t r_hi = r_hi_sh < r_lo ? r_lo : r_hi_sh;  // only a malformed row_ptr inverts them
    const bool in_lds = r_hi - r_lo + 1 <= kCsrWindow;
    if (in_lds)
        for (int64_t r = r_lo + threadIdx.x; r <= r_hi + 1; r += blockDim.x) win[r - r_lo] = row_ptr[r];
    __syncthreads();
    const bool use_filter = filter && ctrl->filter_on;
    const int32_t g = use_filter ? ctrl->giant : 0;
    bool bad = false;
#pragma unroll
    for (int k = 0; k < EPT / 4; ++k) {
        const int64_t e0 = t0 + (int64_t)k * blockDim.x * 4 + (int64_t)threadIdx.x * 4;
        if (e0 >= t1) continue;
        // row of e0, then of the next three entries
        int64_t r;
        if (in_lds) {
            int64_t lo = 0, hi = r_hi - r_lo;
            while (lo < hi) {
                const int64_t mid = (lo + hi + 1) >> 1;
                if (win[mid] <= e0) lo = mid;
                else hi = mid - 1;
            }
            r = r_lo + lo;
        } else {
            r = upper_row(row_ptr, r_lo, r_hi, e0);
        }
        int32_t a[4], b[4];
        uint32_t act = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t e = e0 + j;
            if (e >= t1) {
                a[j] = b[j] = 0;
                continue;
            }
            // advance to the row that owns e (rows may be empty); stays
            // inside the window even if row_ptr is malformed.  Two loops,
            // not one with a select between the LDS and the global row_ptr,
            // which would become flat loads.
            if (in_lds) {
                while (r < r_hi && win[r + 1 - r_lo] <= e) ++r;
            } else {
                while (r < (int64_t)n - 1 && row_ptr[r + 1] <= e) ++r;
            }
            a[j] = (int32_t)r;
            b[j] = __builtin_nontemporal_load(col + e);
            const bool in = (uint32_t)b[j] < (uint32_t)n;
            bad |= !in;
            if (in && a[j] != b[j] && !(sym && b[j] < a[j])) act |= 1u << j;
        }
        if (!act) continue;
        int32_t pa[4], pb[4];
        uint32_t inga = 0, ingb = 0;
        if (use_filter) {
            // the row's bit once per group (the group spans at most a few rows)
            const uint32_t ra = (uint32_t)a[0];
            const uint32_t ba0 = bits[ra >> 5] >> (ra & 31) & 1;
            uint32_t wb[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) wb[j] = bits[(act >> j & 1) ? ((uint32_t)b[j] >> 5) : 0u];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t x = (uint32_t)a[j];
                const uint32_t bax = (x == ra) ? ba0 : (bits[x >> 5] >> (x & 31) & 1);
                inga |= bax << j;
                ingb |= (wb[j] >> ((uint32_t)b[j] & 31) & 1u) << j;
            }
            act &= ~(inga & ingb);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool na = (act >> j & 1) && !(inga >> j & 1);
            const bool nb = (act >> j & 1) && !(ingb >> j & 1);
            const int32_t xa = ld_tree<false>(pi + (na ? a[j] : 0));
            const int32_t xb = ld_tree<false>(pi + (nb ? b[j] : 0));
            pa[j] = na ? xa : g;
            pb[j] = nb ? xb : g;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (!(act >> j & 1)) continue;
            int32_t pu = pa[j], pv = pb[j];
            uint32_t step = 0;
            // Atomic-Hook climb (Fig. 3, top) with optional path halving; see
            // atomic_hook in kernels_core.hip for why it is correct and finite.
            while (pu != pv) {
                const int32_t H = pu > pv ? pu : pv;
                const int32_t L = pu > pv ? pv : pu;
                int32_t found = ld_tree<false>(pi + H);
                if (found == H) {
                    found = cas_root(pi + H, H, L);
                    if (found == H) break;
                }
                pu = ld_tree<false>(pi + found);
                pv = ld_tree<false>(pi + L);
                if (halve && pu != found && step++ % kHalveEveryFiltered == 0)
                    halve_to(pi + H, pu);
            }
        }
    }
    if (bad) atomicOr(&ctrl->status, kStatusRange);
}

// ----------------------------------------------------------------------------- preparation
// The first launch of the plans that go by tiles of kCsrTile entries.  The
// first workgroups take one row per thread: the check of row_ptr, the initial
// tree and, with SAMPLE, the pair (su[r], sv[r]) = (r, last neighbour) (r
// itself where there is none or it is out of range).  The tree starts as
// singletons, with SAMPLE as pi[r] = min(r, first neighbour): one round of the
// atomic-free Hook in which every vertex is written by its own thread, so
// nothing races.  First and last neighbours of adjacent rows share their
// cache lines.  The other workgroups find the row that owns the first entry
// of each tile, half a wave per tile.
template <bool SAMPLE>
__global__ __launch_bounds__(256) void k_csr_prep(const int64_t* __restrict__ row_ptr,
                                                  const int32_t* __restrict__ col, int32_t n,
                                                  int64_t m, int row_blocks, int64_t tiles, Ctrl* ctrl,
                                                  int32_t* __restrict__ pi, int32_t* __restrict__ tile_row,
                                                  int32_t* __restrict__ su, int32_t* __restrict__ sv) {
    if ((int)blockIdx.x >= row_blocks) {
        const int64_t t = ((int64_t)blockIdx.x - row_blocks) * 8 + (threadIdx.x >> 5);
        const int64_t r = upper_row32(row_ptr, n, min(t, tiles - 1) * kCsrTile);
        if ((threadIdx.x & 31) == 0 && t < tiles) tile_row[t] = (int32_t)r;
        return;
    }
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const int64_t s = row_ptr[r], e = row_ptr[r + 1];
    if (e < s || (r == 0 && s != 0) || (r == n - 1 && e != m)) atomicOr(&ctrl->status, kStatusRange);
    int32_t first = (int32_t)r, last = (int32_t)r;
    if (SAMPLE && s >= 0 && s < e && e <= m) {
        first = col[s];
        last = col[e - 1];
        if ((uint32_t)first >= (uint32_t)n) first = (int32_t)r;
        if ((uint32_t)last >= (uint32_t)n) last = (int32_t)r;
    }
    pi[r] = min((int32_t)r, first);
    if (SAMPLE) {
        su[r] = (int32_t)r;
        sv[r] = last;
    }
    if (r == n - 1) tile_row[tiles] = n - 1;
}

hipError_t launch_csr_prep(const int64_t* row_ptr, const int32_t* col, int32_t n, int64_t m,
                           Ctrl* ctrl, int32_t* pi, int32_t* tile_row, int32_t* su, int32_t* sv,
                           hipStream_t s) {
    const int row_blocks = (int)(((int64_t)n + 255) / 256);
    const int64_t tiles = (m + kCsrTile - 1) / kCsrTile;
    const int64_t grid = row_blocks + (tiles + 7) / 8;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    if (su)
        k_csr_prep<true><<<(int)grid, 256, 0, s>>>(row_ptr, col, n, m, row_blocks, tiles, ctrl, pi, tile_row, su, sv);
    else
        k_csr_prep<false><<<(int)grid, 256, 0, s>>>(row_ptr, col, n, m, row_blocks, tiles, ctrl, pi, tile_row, su, sv);
    return hipGetLastError();
}

// Row of tile t's first entry, inside [0, n) whatever row_ptr holds.
__device__ __forceinline__ int32_t tile_first_row(const int32_t* tile_row, int64_t t, int32_t n) {
    return min(max(tile_row[t], 0), n - 1);
}

// Rows that a tile walks through.
constexpr int64_t kCsrMaxSpan = 8 * kCsrTile;

// The rows of all entries (eu[i] = row of entry i), so that the pair-list
// plans can run on (eu, col): one workgroup per tile marks the starts of its
// rows in LDS (the last row starting at a position wins: the ones before it
// are empty) and fills the positions between them by a running maximum.  A
// tile that spans more than kCsrMaxSpan rows, nearly all of them empty,
// searches the row of each entry instead.  Bound by the 4 bytes written per
// entry (2048^2 grid, 11.7 M entries: 18 us).
__global__ __launch_bounds__(256) void k_csr_expand(const int64_t* __restrict__ row_ptr,
                                                    const int32_t* __restrict__ tile_row, int32_t n,
                                                    int64_t m, int32_t* __restrict__ eu) {
    constexpr int kPer = kCsrTile / 256;
    __shared__ int32_t head[kCsrTile];
    __shared__ int32_t wave_max[4];
    const int tid = threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.x * kCsrTile;
    const int cnt = (int)min((int64_t)kCsrTile, m - t0);
    const int32_t lo = tile_first_row(tile_row, blockIdx.x, n);
    const int32_t hi = tile_first_row(tile_row, (int64_t)blockIdx.x + 1, n);
    if ((int64_t)hi - lo > kCsrMaxSpan) {
        for (int i = tid; i < cnt; i += 256) eu[t0 + i] = (int32_t)upper_row(row_ptr, lo, hi, t0 + i);
        return;
    }
    for (int i = tid; i < kCsrTile; i += 256) head[i] = lo;
    __syncthreads();
    for (int64_t r = (int64_t)lo + 1 + tid; r <= hi; r += 256) {
        const int64_t at = row_ptr[r] - t0;
        if (at >= 0 && at < cnt) atomicMax(&head[at], (int32_t)r);
    }
    __syncthreads();
    int32_t x[kPer];
    int32_t run = lo;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        run = max(run, head[tid * kPer + k]);
        x[k] = run;
    }
    // exclusive running maximum over the threads before this one
    int32_t incl = run;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t y = __shfl_up(incl, d, 64);
        if ((tid & 63) >= d) incl = max(incl, y);
    }
    if ((tid & 63) == 63) wave_max[tid >> 6] = incl;
    int32_t before = __shfl_up(incl, 1, 64);
    if ((tid & 63) == 0) before = lo;
    __syncthreads();
    for (int w = 0; w < (tid >> 6); ++w) before = max(before, wave_max[w]);
#pragma unroll
    for (int k = 0; k < kPer; ++k) head[tid * kPer + k] = max(x[k], before);
    __syncthreads();
    for (int i = tid; i < cnt; i += 256) eu[t0 + i] = head[i];
}

hipError_t launch_csr_expand(const int64_t* row_ptr, const int32_t* tile_row, int32_t n, int64_t m,
                             int32_t* eu, hipStream_t s) {
    if (m <= 0) return hipSuccess;
    const int64_t tiles = (m + kCsrTile - 1) / kCsrTile;
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    k_csr_expand<<<(int)tiles, 256, 0, s>>>(row_ptr, tile_row, n, m, eu);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------- filtered pass
// Filtered Atomic-Hook of the entries of a CSR adjacency, after a giant
// component has been found and marked in `bits`.  An entry whose column is in
// the giant needs hooking only if its row is not, and rows outside the giant
// are few, so entries do not look up their rows.  Each wave takes tiles of its
// own, without a barrier:
//   1. each row outside the giant writes its number in the tile to the LDS
//      slots of its entries: short rows by one lane, long ones by the wave
//      (skipped where there is none, the usual case);
//   2. each entry reads its slot: a number there is its row, none means a row
//      in the giant.  What is not inside the giant goes to the wave's queue.
// Without a giant (filter off) every row counts as outside it.  A tile that
// spans more than kCsrMaxSpan rows searches row_ptr per entry instead.
// Persistent.  ALL (n <= kCsrLdsBitsMaxN): the whole bitmap is in LDS and the
// pass streams 4 bytes per entry and 8 per row, bound by instruction issue
// (R-MAT 20, 2^25 entries: 36.5 us, 3.7 TB/s; with tiles of 4,096 entries per
// workgroup and two barriers each 68; the growing segments with a row search
// per tile took 387).  Else the first kCsrLdsBitsMaxN vertices' bits are, and
// the other tests go to the L2, whose request rate bounds them (solves, without
// any bits in LDS and now: R-MAT 21, 6 * 10^7 entries 374 and 285 us; R-MAT 22,
// 10^8 entries 790 and 715; R-MAT 24, 3.2 * 10^8 entries 2,033 and 1,957).
constexpr int kCsrShortRow = 32;
constexpr int kCsrFilterThreads = 1024;
constexpr int kCsrEPT = kCsrTile / 64;
static_assert(kCsrMaxSpan < 65535, "rows of a tile are numbered in 16 bits");

typedef int32_t v4i __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

template <bool ALL, bool VEC>
__global__ __launch_bounds__(kCsrFilterThreads) void k_csr_filter(
    const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col, int32_t n, int64_t m,
    const int32_t* __restrict__ tile_row, int32_t* pi, Ctrl* ctrl,
    const uint32_t* __restrict__ bits, bool halve, bool sym) {
    extern __shared__ uint32_t lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    // per entry of the wave's tile: 1 + its row's number in the tile, 0 = a row of the giant
    uint16_t* owner = reinterpret_cast<uint16_t*>(lds) + (tid >> 6) * kCsrTile;
    uint32_t* lbits = lds + kCsrTile / 2 * (kCsrFilterThreads / 64);  // the bitmap's first part
    const uint32_t on_mask = ctrl->filter_on != 0 ? ~0u : 0u;
    const int32_t g = ctrl->giant;
#pragma unroll
    for (int k = 0; k < kCsrEPT / 4; ++k) *reinterpret_cast<v2u*>(owner + 256 * k + 4 * lane) = v2u{0, 0};
    if (on_mask) {
        const uint32_t words = ((uint32_t)min(n, kCsrLdsBitsMaxN) + 31) / 32;
#pragma unroll 4
        for (uint32_t i = tid * 4; i + 3 < words; i += kCsrFilterThreads * 4)
            *reinterpret_cast<v4i*>(lbits + i) = *reinterpret_cast<const v4i*>(bits + i);
        if (tid < (int)(words & 3)) lbits[(words & ~3u) + tid] = bits[(words & ~3u) + tid];
    }
    __syncthreads();
    auto word_of = [&](uint32_t x) -> uint32_t {
        if (ALL) return lbits[x >> 5];
        const bool near = x < (uint32_t)kCsrLdsBitsMaxN;
        uint32_t w = lbits[near ? x >> 5 : 0u];
        if (!near) w = bits[x >> 5];
        return w;
    };
    auto in_giant = [&](uint32_t x) -> bool {  // x < n
        return (word_of(x & on_mask) & on_mask) >> (x & 31) & 1;
    };
    const int64_t tiles = (m + kCsrTile - 1) / kCsrTile;
    bool bad = false;
    uint32_t top = 0;  // largest column seen
    PairQueue q;
    // Loaded ahead: a tile's rows by two tiles, its entries and row bounds (one
    // row per lane) by one.  Two register sets take turns (a copy from one to
    // the other would wait for the loads in flight), and the loads are
    // unconditional, at clamped addresses: after a branch around a load the
    // waits would cover every load before it.
    struct Tile {
        int32_t c[kCsrEPT];
        int32_t rows;  // even lanes: the first row, odd lanes: the next tile's
        int64_t s, e;
    };
    const int64_t stride = (int64_t)gridDim.x * (kCsrFilterThreads / 64);
    auto row_in = [&](int32_t r) { return min(max(r, 0), n - 1); };  // whatever row_ptr holds
    auto fetch_rows = [&](int64_t t, Tile& x) { x.rows = tile_row[min(t + (lane & 1), tiles)]; };
    auto fetch = [&](int64_t t, Tile& x) {
#pragma unroll
        for (int k = 0; k < kCsrEPT / 4; ++k) {
            const int64_t e = t * kCsrTile + 256 * k + 4 * lane;
            if (VEC) {
                const v4i q4 = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(col + min(e, (m - 4) & ~int64_t(3))));
                x.c[4 * k + 0] = q4.x;
                x.c[4 * k + 1] = q4.y;
                x.c[4 * k + 2] = q4.z;
                x.c[4 * k + 3] = q4.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) x.c[4 * k + j] = __builtin_nontemporal_load(col + min(e + j, m - 1));
            }
        }
    };
    auto bounds = [&](Tile& x) {
        const int32_t r = min(row_in(__builtin_amdgcn_readlane(x.rows, 0)), n - 1 - min(lane, n - 1)) + min(lane, n - 1);
        x.s = row_ptr[r];
        x.e = row_ptr[r + 1];
    };
    auto step = [&](int64_t t, Tile& x, Tile& x1) {
        if (t >= tiles) return;
        const int64_t t0 = t * kCsrTile;
        const int cnt = (int)min((int64_t)kCsrTile, m - t0);
        const int32_t lo = row_in(__builtin_amdgcn_readlane(x.rows, 0));
        const int32_t hi = max(lo, row_in(__builtin_amdgcn_readlane(x.rows, 1)));
        if (VEC && t == tiles - 1 && (m & 3)) {  // the last entries, which no 16-byte load holds
#pragma unroll
            for (int i = 0; i < kCsrEPT; ++i) x.c[i] = col[min(t0 + 256 * (i >> 2) + 4 * lane + (i & 3), m - 1)];
        }
        bounds(x1);
        fetch_rows(t + 2 * stride, x);
        fetch(t + stride, x1);
        if (hi - lo > kCsrMaxSpan) {  // mostly empty rows: each entry looks up its own
#pragma nounroll
            for (int i = lane; i < kCsrTile; i += 64) {
                const int32_t y = col[t0 + min(i, cnt - 1)], r = (int32_t)upper_row(row_ptr, lo, hi, t0 + min(i, cnt - 1));
                const bool in = (uint32_t)y < (uint32_t)n;
                bad |= !in;
                const bool gx = in_giant((uint32_t)r), gy = in_giant(in ? (uint32_t)y : 0u);
                q.push(i < cnt && in && r != y && !(gx && gy) && !(sym && y < r), gx ? g : r, gy ? g : y, pi, halve);
            }
            return;
        }
        // the row's entries inside the tile: [from, from + len)
        auto clip = [&](int64_t at) { return (int)min(max(at - t0, (int64_t)0), (int64_t)cnt); };
        auto mark = [&](int r0, int from, int len) {  // rows lo + r0 + lane; whole waves
            const bool brief = len <= kCsrShortRow;
            if (brief)
                for (int k = from; k < from + len; ++k) owner[k] = (uint16_t)(r0 + lane + 1);
            for (uint64_t wide = __ballot(!brief); wide; wide &= wide - 1) {
                const int src = __ffsll((long long)wide) - 1;
                const int rf = __builtin_amdgcn_readlane(from, src), rl = __builtin_amdgcn_readlane(len, src);
                for (int k = lane; k < rl; k += 64) owner[rf + k] = (uint16_t)(r0 + src + 1);
            }
        };
        const int32_t r = lo + min(lane, hi - lo);
        const int from = clip(x.s);
        int len = max(0, clip(x.e) - from);
        if (lane > hi - lo || in_giant((uint32_t)r)) len = 0;
        // rows outside the giant, or a part of a tile
        const bool some = __any(len > 0) || hi - lo >= 64 || on_mask == 0 || cnt < kCsrTile;
        if (some) {
            mark(0, from, len);
            for (int r0 = 64; r0 <= hi - lo; r0 += 256) {
                int64_t s[4], e[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int32_t rr = lo + min(r0 + 64 * i + lane, hi - lo);
                    s[i] = row_ptr[rr];
                    e[i] = row_ptr[rr + 1];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int rr = r0 + 64 * i + lane;
                    const int f = clip(s[i]);
                    const bool out = rr <= hi - lo && !in_giant((uint32_t)(lo + min(rr, hi - lo)));
                    mark(r0 + 64 * i, f, out ? max(0, clip(e[i]) - f) : 0);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int k = 0; k < kCsrEPT / 4; ++k) {
            if (!some) {  // the usual case: entries of the giant's rows, all inside it
                uint32_t inside = 1;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t y = min((uint32_t)x.c[4 * k + j], (uint32_t)n - 1);
                    top = max(top, (uint32_t)x.c[4 * k + j]);
                    inside &= word_of(y) >> (y & 31);
                }
                if (!__any(inside == 0)) continue;
            }
            int32_t a[4], b[4];
            bool keep[4];
            v2u own = {0, 0};
            if (some) {
                own = *reinterpret_cast<const v2u*>(owner + 256 * k + 4 * lane);
                *reinterpret_cast<v2u*>(owner + 256 * k + 4 * lane) = v2u{0, 0};
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int32_t y = x.c[4 * k + j];
                const bool on = 256 * k + 4 * lane + j < cnt, in = (uint32_t)y < (uint32_t)n;
                bad |= on && !in;
                const bool gy = in_giant(in ? (uint32_t)y : 0u);
                int32_t r = (int32_t)((j & 2 ? own.y : own.x) >> (16 * (j & 1)) & 0xffff);
                const bool gx = r == 0;
                r += lo - 1;
                a[j] = gx ? g : r;
                b[j] = gy ? g : y;
                // without a giant only entries outside a malformed row_ptr have no row
                keep[j] = on && in && a[j] != b[j] && (gx ? on_mask != 0 : !sym || y > r);
            }
            if (!__any(keep[0] || keep[1] || keep[2] || keep[3])) continue;
#pragma nounroll
            for (int j = 0; j < 4; ++j)
                q.push(j == 0 ? keep[0] : j == 1 ? keep[1] : j == 2 ? keep[2] : keep[3],
                       j == 0 ? a[0] : j == 1 ? a[1] : j == 2 ? a[2] : a[3],
                       j == 0 ? b[0] : j == 1 ? b[1] : j == 2 ? b[2] : b[3], pi, halve);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    const int64_t first = (int64_t)blockIdx.x * (kCsrFilterThreads / 64) + (tid >> 6);
    Tile x0, x1;
    fetch_rows(first, x0);
    fetch_rows(first + stride, x1);
    bounds(x0);
    // these arrive before the loads of entries go out, as in the loop
    asm volatile("" : "+v"(x0.s), "+v"(x0.e), "+v"(x1.rows));
    fetch(first, x0);
    for (int64_t t = first; t < tiles; t += 2 * stride) {
        step(t, x0, x1);
        step(t + stride, x1, x0);
    }
    q.flush(pi, halve);
    if (bad || top >= (uint32_t)n) atomicOr(&ctrl->status, kStatusRange);
}

hipError_t launch_csr_filter(const int64_t* row_ptr, const int32_t* col, int32_t n, int64_t m,
                             const int32_t* tile_row, int32_t* pi, Ctrl* ctrl, const uint32_t* bits,
                             bool halve, bool sym, hipStream_t s) {
    if (m <= 0 || n <= 0) return hipSuccess;
    auto allow = [](const void* f) {
        return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    };
    static const hipError_t once[4] = {allow(reinterpret_cast<const void*>(&k_csr_filter<true, false>)),
                                       allow(reinterpret_cast<const void*>(&k_csr_filter<true, true>)),
                                       allow(reinterpret_cast<const void*>(&k_csr_filter<false, false>)),
                                       allow(reinterpret_cast<const void*>(&k_csr_filter<false, true>))};
    for (hipError_t e : once)
        if (e != hipSuccess) return e;
    constexpr int kWaves = kCsrFilterThreads / 64;
    const bool all = n <= kCsrLdsBitsMaxN;
    const size_t lds = kCsrTile * 2 * kWaves + ((size_t)std::min(n, kCsrLdsBitsMaxN) + 127) / 128 * 16;
    const int64_t tiles = (m + kCsrTile - 1) / kCsrTile;
    const int64_t cap = (int64_t)device_cu_count() * (2 * lds <= (size_t)kLdsBytes ? 2 : 1);
    const int grid = (int)std::min<int64_t>((tiles + kWaves - 1) / kWaves, cap);
    const bool vec = ((uintptr_t)col & 15) == 0 && m >= 4;
    const auto kernel = all ? (vec ? &k_csr_filter<true, true> : &k_csr_filter<true, false>)
                            : (vec ? &k_csr_filter<false, true> : &k_csr_filter<false, false>);
    kernel<<<grid, kCsrFilterThreads, lds, s>>>(row_ptr, col, n, m, tile_row, pi, ctrl, bits, halve, sym);
    return hipGetLastError();
}

// Entry-count check of a CSR adjacency: status bit kStatusRange when
// row_ptr is not non-decreasing from 0 to m (done on the device, one pass).
__global__ __launch_bounds__(256) void k_csr_check(const int64_t* __restrict__ row_ptr, int32_t n,
                                                   int64_t m, Ctrl* ctrl) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r > n) return;
    bool bad = false;
    if (r == 0) bad = row_ptr[0] != 0;
    if (r == n) bad = row_ptr[n] != m;
    if (r < n) bad = bad || row_ptr[r + 1] < row_ptr[r];
    if (bad) atomicOr(&ctrl->status, kStatusRange);
}

hipError_t launch_csr_check(const int64_t* row_ptr, int32_t n, int64_t m, Ctrl* ctrl,
                            hipStream_t s) {
    const int grid = (int)(((int64_t)n + 1 + 255) / 256);
    k_csr_check<<<grid, 256, 0, s>>>(row_ptr, n, m, ctrl);
    return hipGetLastError();
}

hipError_t launch_ahook_csr(const int64_t* row_ptr, const int32_t* col, int32_t n, int64_t begin,
                            int64_t end, int32_t* pi, Ctrl* ctrl, const uint32_t* bits, bool sym,
                            bool halve, hipStream_t s) {
    if (end <= begin || n <= 0) return hipSuccess;
    // 512 threads x 8 entries per tile: measured on R-MAT 24 (2^29 entries)
    // 4.97 ms against 5.86 (256 x 8), 5.49 (256 x 16), 5.13 (1024 x 8)
    constexpr int EPT = 8;
    constexpr int kBlock = 512;
    const int64_t tile = kBlock * EPT;
    const int64_t grid64 = (end - begin + tile - 1) / tile;
    if (grid64 > 0x7fffffff) return hipErrorInvalidValue;
    k_ahook_csr<EPT><<<(int)grid64, kBlock, 0, s>>>(row_ptr, col, n, begin, end, pi, ctrl, bits,
                                                    bits != nullptr, sym, halve);
    return hipGetLastError();
}

}  // namespace hookcc
