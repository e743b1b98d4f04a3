// Steps a3-a5 with one host synchronisation: the octree, its monopole
// moments, the DFS preorder with subtree "skip" links, the particle groups
// and their bounding boxes, all derived from the sorted Morton keys.
//
// Let delta(s) be the number of leading 3-bit digits that keys s-1 and s
// share (-1 for s = 0).  The cell of level L holding particle s starts at s
// iff delta(s) < L, and ends before the next index e with delta(e) < L.  It
// holds at least W particles iff some run of W consecutive particles that
// contains s lies inside it, i.e. iff delta >= L over that run's interior.
// So the deepest level whose cell holding s has more than k particles is
//   lambda_k(s) = max over runs [t, t + k] containing s of min delta(t+1 .. t+k)
// (-1 if there is no such run), a max of mins over runs of at most 65
// particles, taken per particle from an LDS tile.  From it:
//   - s lies in the leaf of level leaf(s) = min(21, max(1, lambda_{n_leaf}(s) + 1))
//     (a cell is split iff it holds more than n_leaf particles; the root
//     always);
//   - the cells starting at s are the levels delta(s)+1 .. leaf(s), a chain
//     in which each is the first child of the one before: their preorder
//     numbers are start(s) + L - delta(s) - 1, start the exclusive scan of
//     the chain lengths, so the whole preorder follows from one scan;
//   - s lies in the group candidate of level max(1, lambda_{n_group}(s) + 1)
//     (lambda = 21: a level-21 cell with more than n_group particles, cut
//     into chunks of n_group); whether a candidate starts a group follows
//     from its left siblings, found by 64-lane scans of delta in LDS.
// Each level's cells also get consecutive slots ordered by first particle
// (per-block counts, scanned per level), so that a cell's children are one
// contiguous run of the next level's slots; counts, moments and skip links
// then follow bottom-up, one launch per level, sized from the level totals
// read at the one synchronisation.
//
// Compiled with -ffp-contract=off: the group boxes feed the list decisions,
// which must be the literal FP64 expressions.
#include <string>
#include <type_traits>

#include "common.h"
#include "walks.h"

namespace srf {
namespace {

constexpr int kLvThreads = 256;
constexpr int kLvTile = 1024;                      // particles per block
constexpr int kPer = kLvTile / kLvThreads;
constexpr int kHalo = 64;                          // runs hold at most 65 particles
constexpr int kLvRuns = kLvTile + kHalo;           // run starts
constexpr int kLog = 7;                            // range tables for lengths 1..64
constexpr int kLeft = 512;                         // left reach of the sibling scans (7 siblings of <= 64, + 64)
constexpr int kScanSpan = kLeft + kLvTile + kHalo; // deltas of the sibling scans

__device__ __forceinline__ int shared_digits(uint64_t a, uint64_t b) {
    const uint64_t x = a ^ b;   // keys use the low 63 bits
    return x ? (__clzll(x) - 1) / 3 : kMaxLevel;
}

__device__ __forceinline__ int floor_log2(int v) { return 31 - __clz(v); }

// First index in [lo, s] whose key equals keys[s] (sorted keys).
__device__ __forceinline__ int64_t first_equal(const uint64_t* __restrict__ keys, int64_t lo, int64_t s) {
    const uint64_t k = keys[s];
    int64_t hi = s;
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if (keys[mid] < k) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Whether the candidate of level lv >= 2 at index js of the deltas mn[0]
// starts a group (see k_levels).  It holds at most n_group particles, so its
// end is within reach; its left siblings before the closing one span at most 7
// x 64 particles, inside the left reach.
__device__ __forceinline__ bool starts_group(const int8_t (*mn)[kScanSpan], int js, int lv, int n_group) {
    int end = js + 1;
#pragma unroll
    for (int k = kLog - 1; k >= 0; --k)
        if (end + (1 << k) <= kScanSpan && mn[k][end] >= lv) end += 1 << k;
    const int own = end - js;
    uint64_t sizes = 0;   // the siblings' sizes, nearest first, 8 bits each
    int ns = 0, pos = js;
    while (ns < 7 && mn[0][pos] >= lv - 1) {   // pos is not the parent's first index
        int at = pos;   // all deltas of [at, pos) are >= lv
#pragma unroll
        for (int k = kLog - 1; k >= 0; --k)
            if (at >= (1 << k) && mn[k][at - (1 << k)] >= lv) at -= 1 << k;
        const int c = pos - at + 1;   // the sibling starts at at - 1
        if (at == 0 || c > n_group) break;
        sizes |= (uint64_t)c << (8 * ns++);
        pos -= c;
    }
    int run = 0;   // the run that is open before the candidate
    for (int k = ns - 1; k >= 0; --k) {
        const int c = (int)((sizes >> (8 * k)) & 0xffu);
        run = run > 0 && run + c <= n_group ? run + c : c;
    }
    return !(run > 0 && run + own <= n_group);
}

// Per particle: delta, leaf level, the chain length of the cells starting
// there and the group-start mark; per block and level the number of cells
// (blk[L * nblocks + block]), and per block the sums of the chain lengths
// and of the marks (rows kLevels and kLevels + 1 of blk).
//
// Group starts.  A candidate (level >= 1, at most n_group particles, parent
// the root or holding more than n_group) starts a group under the root, and
// under any other parent unless the greedy run of the candidate siblings
// before it (octant order, closed by a sibling with more than n_group
// particles or by an overflow) takes it in.  Under a parent of level >= 1 the
// candidate's end and its left siblings' starts are each the nearest index
// after (before) a position with delta below the candidate's level, found in
// seven steps down the range table of minima; a sibling whose start is more
// than n_group away closes the run.  Each lane looks up its own candidate:
// with the wave scanning 64 deltas for one candidate after another this took
// most of a tile's time (44 us at 4096 particles, now 31 with 256 threads and
// 15 with 1024).
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_levels(int64_t n, const uint64_t* __restrict__ keys, int n_leaf,
                                                       int n_group, int64_t nblocks, int8_t* __restrict__ delta,
                                                       int8_t* __restrict__ leaflv, int32_t* __restrict__ chain,
                                                       int32_t* __restrict__ mark, int32_t* __restrict__ blk) {
    constexpr int PER = kLvTile / THREADS;
    __shared__ int8_t mn[kLog][kScanSpan]; // mn[k][j] = min delta over [j, j + 2^k), j from b0 - kLeft on
    __shared__ int8_t mx[kLog][kLvRuns];   // mx[k][j] = max run minimum over run starts [j, j + 2^k)
    const int8_t* dl = mn[0];              // the deltas themselves
    __shared__ unsigned lh[kLevels + 2];   // cells per level; the tile's chain and mark sums
    const int64_t b0 = blockIdx.x * (int64_t)kLvTile;
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < kLevels + 2) lh[tid] = 0;
    for (int j = tid; j < kScanSpan; j += THREADS) {
        const int64_t i = b0 - kLeft + j;
        int d = -1;
        if (i >= 1 && i < n) d = shared_digits(keys[i - 1], keys[i]);
        mn[0][j] = (int8_t)d;
    }
    __syncthreads();
    for (int k = 1; k < kLog; ++k) {
        const int h = 1 << (k - 1);
        for (int j = tid; j < kScanSpan; j += THREADS) {
            // entries whose range runs past the span are never queried
            const int a = mn[k - 1][j], b = j + h < kScanSpan ? mn[k - 1][j + h] : a;
            mn[k][j] = (int8_t)(a < b ? a : b);
        }
        __syncthreads();
    }
    int lam[2][PER];
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const int W = (w == 0 ? n_leaf : n_group) + 1;   // run length, 2..65
        const int kq = floor_log2(W - 1);
        // minimum of delta over the interior of the run starting at each t
        for (int j = tid; j < kLvRuns; j += THREADS) {
            const int64_t t = b0 - kHalo + j;
            int v = -1;
            if (t >= 0 && t + W - 1 <= n - 1) {
                const int jm = j + kLeft - kHalo;
                const int a = mn[kq][jm + 1], b = mn[kq][jm + W - (1 << kq)];
                v = a < b ? a : b;
            }
            mx[0][j] = (int8_t)v;
        }
        __syncthreads();
        const int kr = floor_log2(W);
        for (int k = 1; k <= kr; ++k) {
            const int h = 1 << (k - 1);
            for (int j = tid; j < kLvRuns; j += THREADS) {
                const int a = mx[k - 1][j], b = j + h < kLvRuns ? mx[k - 1][j + h] : a;
                mx[k][j] = (int8_t)(a > b ? a : b);
            }
            __syncthreads();
        }
        // maximum over the runs [s - W + 1, s] that contain s
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int js = kHalo + tid + q * THREADS;
            const int a = mx[kr][js - W + 1], b = mx[kr][js - (1 << kr) + 1];
            lam[w][q] = a > b ? a : b;
        }
        __syncthreads();
    }
    int32_t csum = 0, msum = 0;   // this thread's chain lengths and group marks
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int64_t s = b0 + tid + q * THREADS;   // a wave holds 64 consecutive particles
        const bool on = s < n;
        const int js = kLeft + tid + q * THREADS;  // index of s in dl
        const int d = dl[js];
        int ll = lam[0][q] + 1;
        ll = ll < 1 ? 1 : (ll > kMaxLevel ? kMaxLevel : ll);
        const int lg = lam[1][q];
        const int kap = lg + 1 > 1 ? lg + 1 : 1;
        int m = 0;
        if (on) {
            delta[s] = (int8_t)d;
            leaflv[s] = (int8_t)ll;
            chain[s] = ll > d ? ll - d : 0;
            csum += ll > d ? ll - d : 0;
            for (int L = d + 1; L <= ll; ++L) atomicAdd(&lh[L], 1u);
            if (lg >= kMaxLevel) {
                m = ((s - first_equal(keys, 0, s)) % n_group) == 0;   // chunks of a level-21 cell
            } else if (d < kap) {
                m = kap == 1 || starts_group(mn, js, kap, n_group);
            }
        }
        if (on) mark[s] = m;
        msum += on ? m : 0;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        csum += __shfl_xor(csum, o, 64);
        msum += __shfl_xor(msum, o, 64);
    }
    if (lane == 0) {
        atomicAdd(&lh[kLevels], (unsigned)csum);
        atomicAdd(&lh[kLevels + 1], (unsigned)msum);
    }
    __syncthreads();
    if (tid < kLevels + 2) blk[(int64_t)tid * nblocks + blockIdx.x] = (int32_t)lh[tid];
}

// In place, over the tiles of k_levels: the exclusive scans of the chain
// lengths (the preorder number of each chain's first cell) and of the group
// marks (the group number of each group start), each tile starting from its
// scanned sum (rows kLevels and kLevels + 1 of blk); each group start also
// goes to its group's place in gfirst.  Thread t takes the tile's entries 4t ..
// 4t + 3.
__global__ __launch_bounds__(kLvThreads) void k_scan_tiles(int64_t n, int64_t nblocks, int32_t* __restrict__ chain,
                                                           const int32_t* __restrict__ mark,
                                                           const int32_t* __restrict__ blk,
                                                           int32_t* __restrict__ gfirst,
                                                           const int32_t* __restrict__ stat,
                                                           int32_t* __restrict__ host_stat) {
    static_assert(kPer == 4, "four entries per thread");
    __shared__ int32_t wsum[kLvThreads / 64][2];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    if (blockIdx.x == 0 && tid < kStatWords) host_stat[tid] = stat[tid];   // read at the build's synchronisation
    const int64_t s0 = blockIdx.x * (int64_t)kLvTile + kPer * tid;
    int32_t c[kPer], m[kPer];
    if (s0 + kPer <= n) {
        const int4 cv = *reinterpret_cast<const int4*>(chain + s0);
        const int4 mv = *reinterpret_cast<const int4*>(mark + s0);
        c[0] = cv.x, c[1] = cv.y, c[2] = cv.z, c[3] = cv.w;
        m[0] = mv.x, m[1] = mv.y, m[2] = mv.z, m[3] = mv.w;
    } else {
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            c[k] = s0 + k < n ? chain[s0 + k] : 0;
            m[k] = s0 + k < n ? mark[s0 + k] : 0;
        }
    }
    const int32_t cs = c[0] + c[1] + c[2] + c[3], ms = m[0] + m[1] + m[2] + m[3];
    int32_t ci = cs, mi = ms;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t u = __shfl_up(ci, o, 64), v = __shfl_up(mi, o, 64);
        if (lane >= o) {
            ci += u;
            mi += v;
        }
    }
    if (lane == 63) {
        wsum[wid][0] = ci;
        wsum[wid][1] = mi;
    }
    __syncthreads();
    int32_t co = blk[(int64_t)kLevels * nblocks + blockIdx.x] + ci - cs;
    int32_t mo = blk[(int64_t)(kLevels + 1) * nblocks + blockIdx.x] + mi - ms;
#pragma unroll
    for (int w = 0; w < kLvThreads / 64; ++w) {
        if (w < wid) {
            co += wsum[w][0];
            mo += wsum[w][1];
        }
    }
    int32_t cx[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        cx[k] = co;
        if (m[k]) gfirst[mo] = (int32_t)(s0 + k);
        co += c[k];
        mo += m[k];
    }
    if (s0 + kPer <= n) {
        *reinterpret_cast<int4*>(chain + s0) = make_int4(cx[0], cx[1], cx[2], cx[3]);
    } else {
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            if (s0 + k < n) chain[s0 + k] = cx[k];
        }
    }
}

// Exclusive scan of one level's per-block cell counts (block = level), in
// place; the level's total goes to tot.  Rows kLevels and kLevels + 1 (the
// tiles' chain and mark sums) are scanned the same way.
__global__ __launch_bounds__(256) void k_level_scan(int64_t nblocks, int32_t* __restrict__ blk,
                                                    int32_t* __restrict__ tot) {
    constexpr int kItems = 4;
    __shared__ int32_t wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    int32_t* row = blk + (int64_t)blockIdx.x * nblocks;
    int32_t carry = 0;
    for (int64_t c0 = 0; c0 < nblocks; c0 += 256 * kItems) {
        const int64_t j = c0 + (int64_t)tid * kItems;
        int32_t v[kItems];
        int32_t s = 0;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            v[k] = j + k < nblocks ? row[j + k] : 0;
            s += v[k];
        }
        int32_t incl = s;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t u = __shfl_up(incl, o, 64);
            if (lane >= o) incl += u;
        }
        if (lane == 63) wsum[wid] = incl;
        __syncthreads();
        int32_t off = carry + incl - s, total = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            off += w < wid ? wsum[w] : 0;
            total += wsum[w];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            if (j + k < nblocks) row[j + k] = off;
            off += v[k];
        }
        carry += total;
    }
    if (tid == 0) tot[blockIdx.x] = carry;
}

__device__ __forceinline__ uint32_t compact3(uint64_t v) {
    v &= 0x1249249249249249ull;
    v = (v ^ (v >> 2)) & 0x10c30c30c30c30c3ull;
    v = (v ^ (v >> 4)) & 0x100f00f00f00f00full;
    v = (v ^ (v >> 8)) & 0x1f0000ff0000ffull;
    v = (v ^ (v >> 16)) & 0x1f00000000ffffull;
    v = (v ^ (v >> 32)) & 0x1fffffull;
    return (uint32_t)v;
}

struct LevelBase {
    int32_t off[kLevels + 1];   // first slot of each level; off[kLevels] = number of cells
};

// The cells starting at each particle (same tiling as k_levels): their
// level slot (level base + the block's offset + the rank among the block's
// cells of that level, by first particle) and, in preorder, their geometry,
// first index and key prefix; per slot the first particle, the preorder
// number and the slot of the first child (-1 for a leaf).
constexpr int kWords = kLvTile / 32;

__global__ __launch_bounds__(kLvThreads) void k_cells(int64_t n, int64_t nblocks, const uint64_t* __restrict__ keys,
                                                      const int8_t* __restrict__ delta,
                                                      const int8_t* __restrict__ leaflv,
                                                      const int32_t* __restrict__ start, LevelBase base,
                                                      const int32_t* __restrict__ blk, NodeGeo* __restrict__ geo,
                                                      int32_t* __restrict__ pfirst, uint64_t* __restrict__ prefix,
                                                      int32_t* __restrict__ sfirst, int32_t* __restrict__ spre,
                                                      int32_t* __restrict__ schild) {
    __shared__ uint32_t msk[kLevels][kWords];
    __shared__ int32_t wpre[kLevels][kWords];
    const int tid = threadIdx.x;
    const int64_t b0 = blockIdx.x * (int64_t)kLvTile;
    for (int q = tid; q < kLevels * kWords; q += kLvThreads) (&msk[0][0])[q] = 0u;
    __syncthreads();
    int d[kPer], ll[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int p = tid + q * kLvThreads;
        const int64_t s = b0 + p;
        d[q] = 0;
        ll[q] = 0;
        if (s < n) {
            d[q] = delta[s];
            ll[q] = leaflv[s];
            for (int L = d[q] + 1; L <= ll[q]; ++L) atomicOr(&msk[L][p >> 5], 1u << (p & 31));
        }
    }
    __syncthreads();
    if (tid < kLevels) {
        int32_t acc = 0;
        for (int w = 0; w < kWords; ++w) {
            wpre[tid][w] = acc;
            acc += __popc(msk[tid][w]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int p = tid + q * kLvThreads;
        const int64_t s = b0 + p;
        if (s >= n || ll[q] <= d[q]) continue;
        const int32_t st = start[s];
        const uint64_t k = keys[s];
        const uint32_t below = (1u << (p & 31)) - 1u;
        int32_t slot_next = -1;
        for (int L = ll[q]; L >= d[q] + 1; --L) {   // deepest first: each cell's first child is the one before
            const int32_t rank = wpre[L][p >> 5] + __popc(msk[L][p >> 5] & below);
            const int32_t slot = base.off[L] + blk[(int64_t)L * nblocks + blockIdx.x] + rank;
            const int32_t pre = st + (L - d[q] - 1);
            sfirst[slot] = (int32_t)s;
            spre[slot] = pre;
            schild[slot] = slot_next;
            slot_next = slot;
            const uint64_t pf = L == 0 ? 0ull : k >> (3 * (kMaxLevel - L));
            NodeGeo g;
            g.ix = compact3(pf >> 2);
            g.iy = compact3(pf >> 1);
            g.iz = compact3(pf);
            g.level_leaf = (uint32_t)L | (L == ll[q] ? 0x100u : 0u);
            geo[pre] = g;
            pfirst[pre] = (int32_t)s;
            prefix[pre] = pf;
        }
    }
}

// The walk records of a cell (see common.h).
__device__ __forceinline__ uint2 walk_record(const NodeGeo& g, int32_t count, int32_t skip) {
    const uint32_t lv = g.level_leaf & 0xffu;
    const uint32_t leaf = (g.level_leaf >> 8) & 1u;
    const uint32_t oct = ((g.ix & 1u) << 2) | ((g.iy & 1u) << 1) | (g.iz & 1u);
    const uint32_t cnt = count < (int32_t)kWalkCountMax ? (uint32_t)count : kWalkCountMax;
    return make_uint2(lv | (leaf << 5) | (oct << 6) | (cnt << 9), (uint32_t)skip);
}

__device__ __forceinline__ uint4 slot_record(const NodeGeo& g, uint32_t a, int kids) {
    return make_uint4(g.ix | ((a & 0x7ffu) << 21), g.iy | (((a >> 11) & 0x7ffu) << 21),
                      g.iz | (((a >> 22) & 0x3ffu) << 21), (g.level_leaf & 0xffu) | ((uint32_t)kids << 5));
}

// One level, deepest first, 4 lanes per cell.  A leaf's particles run to
// the first particle of the next cell in preorder; an inner cell's children
// are the next level's slots from its first child on, while their first
// particle lies before the first particle of the next slot of this level.
// Sums and counts are kept per slot; count, skip link and monopole go to
// the cell's preorder record, the children get their parent, and the cell
// its walk records (the one in preorder by k_pack where the tree is large).
constexpr int kMomLanes = 4;

struct MomentArgs {
    int64_t n, nn;
    const int32_t *sfirst, *spre, *schild, *pfirst, *start;
    const double *px, *py, *pz, *pm;
    int32_t* scount;
    double *sM, *sX, *sY, *sZ;
    NodeRange* rng;
    double *oM, *oX, *oY, *oZ;
    int32_t* leaf_of;
    const NodeGeo* geo;
    uint2* pack;
    uint4* srec;
};

// Cell i of the slots [lo, hi): a leaf, or an inner cell of the level [lo, hi),
// whose children lie before next_hi; those that `CELLS` leaves out are passed
// by.
enum Cells { kLeaves = 1, kInner = 2, kAllCells = kLeaves | kInner };

template <int CELLS>
__device__ __forceinline__ void moments_cell(const MomentArgs& a, int64_t i, int32_t lo, int32_t hi, int32_t next_hi) {
    const int j = threadIdx.x & (kMomLanes - 1);
    const int64_t c = i < hi ? i : lo;
    const int32_t f = a.sfirst[c], pre = a.spre[c], ch = a.schild[c];
    const bool on = i < hi && (CELLS == kAllCells || (ch < 0) == (CELLS == kLeaves)), leaf = ch < 0;
    double sm = 0, sx = 0, sy = 0, sz = 0;
    int64_t cnt = 0;
    int kids = 0;
    if ((CELLS & kLeaves) && on && leaf) {
        const int64_t e = pre + 1 < a.nn ? a.pfirst[pre + 1] : a.n;
        for (int64_t s = f + j; s < e; s += kMomLanes) {
            const double mm = a.pm[s];
            sm += mm;
            sx += mm * a.px[s];
            sy += mm * a.py[s];
            sz += mm * a.pz[s];
            a.leaf_of[s] = pre;
        }
        cnt = j == 0 ? e - f : 0;
    }
    if ((CELLS & kInner) && on && !leaf) {
        const int64_t lim = c + 1 < hi ? a.sfirst[c + 1] : a.n;   // first particle of the next cell of this level
        // a cell has at most eight children: two for each lane, loaded together
        int32_t qf[2], qn[2], qp[2];
        double v[2][4];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int32_t q = ch + j + k * kMomLanes < next_hi ? ch + j + k * kMomLanes : next_hi - 1;
            qf[k] = ch + j + k * kMomLanes < next_hi ? a.sfirst[q] : INT32_MAX;
            qn[k] = a.scount[q];
            qp[k] = a.spre[q];
            v[k][0] = a.sM[q];
            v[k][1] = a.sX[q];
            v[k][2] = a.sY[q];
            v[k][3] = a.sZ[q];
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (qf[k] >= lim) continue;
            sm += v[k][0];
            sx += v[k][1];
            sy += v[k][2];
            sz += v[k][3];
            cnt += qn[k];
            ++kids;
            a.rng[qp[k]].parent = pre;
        }
    }
#pragma unroll
    for (int o = kMomLanes / 2; o >= 1; o >>= 1) {
        sm += __shfl_xor(sm, o, kMomLanes);
        sx += __shfl_xor(sx, o, kMomLanes);
        sy += __shfl_xor(sy, o, kMomLanes);
        sz += __shfl_xor(sz, o, kMomLanes);
        cnt += __shfl_xor(cnt, o, kMomLanes);
        kids += __shfl_xor(kids, o, kMomLanes);
    }
    if (on && j == 0) {
        a.scount[c] = (int32_t)cnt;
        a.sM[c] = sm;
        a.sX[c] = sx;
        a.sY[c] = sy;
        a.sZ[c] = sz;
        const int64_t e = f + cnt;
        a.rng[pre].first = f;
        a.rng[pre].count = (int32_t)cnt;
        const int32_t skip = e < a.n ? a.start[e] : (int32_t)a.nn;
        a.rng[pre].skip = skip;
        NodeGeo g;
        if (CELLS != kAllCells || a.srec) g = a.geo[pre];
        if (CELLS != kAllCells) a.pack[pre] = walk_record(g, (int32_t)cnt, skip);
        if (a.srec) a.srec[c] = slot_record(g, leaf ? (uint32_t)cnt : (uint32_t)ch, kids);
        if (pre == 0) a.rng[pre].parent = -1;
        a.oM[pre] = sm;
        a.oX[pre] = sx / sm;
        a.oY[pre] = sy / sm;
        a.oZ[pre] = sz / sm;
    }
}

// The walk records of a large tree's cells, in order.
__global__ __launch_bounds__(256) void k_pack(MomentArgs a) {
    const int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (c < a.nn) a.pack[c] = walk_record(a.geo[c], a.rng[c].count, a.rng[c].skip);
}

template <int CELLS>
__global__ __launch_bounds__(256) void k_moments(MomentArgs a, int32_t lo, int32_t hi, int32_t next_hi) {
    moments_cell<CELLS>(a, lo + blockIdx.x * (int64_t)(256 / kMomLanes) + threadIdx.x / kMomLanes, lo, hi, next_hi);
}

// Several levels of at most kFewCells cells each, deepest first, by one block:
// the first levels and, in a clustered set, the last ones, each of which was a
// launch of its own with a few waves.
constexpr int kMomBlock = 1024;
constexpr int32_t kFewCells = 1024;
// In trees of at most this many cells the leaves, most of the cells and of the
// time, come before the levels in one launch, so that a level waits only for
// its children's sums (10007 clustered particles: 52 us with the leaves among
// the levels, 33 us).  In larger ones the chip is full either way, and the
// records, which lie in preorder, are written line by line by a level that has
// both its kinds of cells at hand, the walk records by a kernel of their own.
// tree_build with the leaves before / among the levels, us: uniform particles,
// 262144 with 75000 cells 172 / 185, with 386000 242 / 239, 10^6 with 1.5e6
// 525 / 491, 8e6 with 1.2e7 3350 / 2750; clustered, 2^20 with 3e5 345 / 345, 8e6
// with 1.1e7 3400 / 2810.
constexpr int64_t kLeavesFirst = 3 << 17;
template <int CELLS>
__global__ __launch_bounds__(kMomBlock) void k_moments_few(MomentArgs a, LevelBase base, int deepest, int top) {
    for (int L = deepest; L >= top; --L) {
        const int32_t lo = base.off[L], hi = base.off[L + 1], next_hi = L < kMaxLevel ? base.off[L + 2] : hi;
        for (int64_t i = lo; i < hi; i += kMomBlock / kMomLanes)
            moments_cell<CELLS>(a, i + threadIdx.x / kMomLanes, lo, hi, next_hi);
        __syncthreads();   // the level's sums are read by the next one's cells
    }
}

// A refitted tree (the structure held, the particles moved), one level,
// deepest first, 4 lanes per cell.  A leaf takes its particles at their
// periodic images nearest its dyadic centre; an inner cell takes its
// children's sums and boxes, each child moved as a whole by the whole
// number of box lengths that brings its box centre nearest the cell's
// centre.  The box is the min and max of those images per axis; the sums
// give the monopole.  Slot sums and boxes (sbox: lo xyz, hi xyz per slot)
// feed the next level up; monopoles and boxes go to the preorder records.
__global__ __launch_bounds__(256) void k_refit_level(int32_t lo, int32_t hi, int32_t next_hi, int64_t n,
                                                     const int32_t* __restrict__ sfirst,
                                                     const int32_t* __restrict__ spre,
                                                     const int32_t* __restrict__ schild,
                                                     const NodeGeo* __restrict__ geo,
                                                     const NodeRange* __restrict__ rng, const double* __restrict__ px,
                                                     const double* __restrict__ py, const double* __restrict__ pz,
                                                     const double* __restrict__ pm, double* __restrict__ sM,
                                                     double* __restrict__ sX, double* __restrict__ sY,
                                                     double* __restrict__ sZ, double* __restrict__ sbox,
                                                     double* __restrict__ oM, double* __restrict__ oX,
                                                     double* __restrict__ oY, double* __restrict__ oZ,
                                                     double* __restrict__ clo, double* __restrict__ chi) {
    const int64_t i = lo + blockIdx.x * (int64_t)(256 / kMomLanes) + threadIdx.x / kMomLanes;
    const int j = threadIdx.x & (kMomLanes - 1);
    const bool on = i < hi;
    const int64_t c = on ? i : lo;
    const int32_t f = sfirst[c], pre = spre[c], ch = schild[c];
    const NodeGeo g = geo[pre];
    const int lv = (int)(g.level_leaf & 0xffu);
    const double cref[3] = {ldexp((double)g.ix + 0.5, -lv), ldexp((double)g.iy + 0.5, -lv),
                            ldexp((double)g.iz + 0.5, -lv)};
    double sm = 0, sv[3] = {0, 0, 0}, bl[3], bh[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        bl[a] = INFINITY;
        bh[a] = -INFINITY;
    }
    if (on) {
        if (ch < 0) {
            const int64_t e = f + (int64_t)rng[pre].count;
            for (int64_t s = f + j; s < e; s += kMomLanes) {
                const double mm = pm[s];
                const double u[3] = {px[s], py[s], pz[s]};
                sm += mm;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const double v = u[a] - rint(u[a] - cref[a]);
                    sv[a] += mm * v;
                    bl[a] = v < bl[a] ? v : bl[a];
                    bh[a] = v > bh[a] ? v : bh[a];
                }
            }
        } else {
            const int64_t lim = c + 1 < hi ? sfirst[c + 1] : n;
            for (int64_t q = ch + j; q < next_hi && sfirst[q] < lim; q += kMomLanes) {
                const double mq = sM[q];
                const double sq[3] = {sX[q], sY[q], sZ[q]};
                sm += mq;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const double l = sbox[q * 6 + a], h = sbox[q * 6 + 3 + a];
                    const double sh = rint((l + h) * 0.5 - cref[a]);
                    const double vl = l - sh, vh = h - sh;
                    bl[a] = vl < bl[a] ? vl : bl[a];
                    bh[a] = vh > bh[a] ? vh : bh[a];
                    sv[a] += sq[a] - sh * mq;
                }
            }
        }
    }
#pragma unroll
    for (int o = kMomLanes / 2; o >= 1; o >>= 1) {
        sm += __shfl_xor(sm, o, kMomLanes);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            sv[a] += __shfl_xor(sv[a], o, kMomLanes);
            const double l = __shfl_xor(bl[a], o, kMomLanes), h = __shfl_xor(bh[a], o, kMomLanes);
            bl[a] = l < bl[a] ? l : bl[a];
            bh[a] = h > bh[a] ? h : bh[a];
        }
    }
    if (on && j == 0) {
        sM[c] = sm;
        sX[c] = sv[0];
        sY[c] = sv[1];
        sZ[c] = sv[2];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            sbox[c * 6 + a] = bl[a];
            sbox[c * 6 + 3 + a] = bh[a];
            clo[(int64_t)pre * 3 + a] = bl[a];
            chi[(int64_t)pre * 3 + a] = bh[a];
        }
        oM[pre] = sm;
        oX[pre] = sv[0] / sm;
        oY[pre] = sv[1] / sm;
        oZ[pre] = sv[2] / sm;
    }
}

// A cell's 16-byte packed record.
__device__ __forceinline__ uint4 pack16(const NodeGeo& g, const NodeRange& r) {
    const uint32_t sk = (uint32_t)r.skip;
    const uint32_t lv = g.level_leaf & 0xffu;
    const bool leaf = (g.level_leaf >> 8) & 1u;
    uint4 pk;
    pk.x = g.ix | ((sk & 0x7ffu) << 21);
    pk.y = g.iy | (((sk >> 11) & 0x7ffu) << 21);
    pk.z = g.iz | (((sk >> 22) & 0x3ffu) << 21);
    pk.w = lv | (leaf ? 0x20u : 0u) | ((uint32_t)(r.count < (int32_t)kPackCountMax ? r.count : (int32_t)kPackCountMax) << 6);
    return pk;
}

// The walk record of each cell of a refitted tree (preorder): the packed
// record, and the box rounded outward to multiples of q = 2^-(level + 10),
// K = floor(lo / q) and ceil(hi / q) (exact), stored as offsets from the
// centre's multiple ic * 1024 + 512 when both fit 16 bits.
__global__ void k_refit_pack(int64_t nn, const NodeGeo* __restrict__ geo, const NodeRange* __restrict__ rng,
                             const double* __restrict__ clo, const double* __restrict__ chi,
                             RefitCell* __restrict__ out) {
    const int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (c >= nn) return;
    const NodeGeo g = geo[c];
    const int e = (int)(g.level_leaf & 0xffu) + kRefitShift;
    const uint32_t ic[3] = {g.ix, g.iy, g.iz};
    RefitCell r;
    r.pk = pack16(g, rng[c]);
    bool ok = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int64_t kc = (int64_t)ic[a] * (1 << kRefitShift) + (1 << (kRefitShift - 1));
        const int64_t kl = (int64_t)floor(ldexp(clo[c * 3 + a], e)) - kc;
        const int64_t kh = (int64_t)ceil(ldexp(chi[c * 3 + a], e)) - kc;
        ok = ok && kl >= -kRefitMaxOff && kh <= kRefitMaxOff;
        r.b[a] = (int32_t)(((uint32_t)(uint16_t)(int16_t)kl) | ((uint32_t)(uint16_t)(int16_t)kh << 16));
    }
    r.b[3] = ok ? 1 : 0;
    out[c] = r;
}

// Tight boxes: 16 lanes per group, lane j taking the group's particles
// j, j + 16, ... (min and max are exact in any order).  In a refitted tree
// (REFIT) each position is first moved to its periodic image nearest the
// group's first particle; in a fresh one the groups' firsts and counts are
// taken from `starts` (each group's first particle, in order).
constexpr int kBoxLanes = 16;

template <bool REFIT>
__global__ __launch_bounds__(256) void k_group_bbox(int64_t ng, int64_t n, const int32_t* __restrict__ starts,
                                                    int32_t* __restrict__ gfirst, int32_t* __restrict__ gcount, const double* __restrict__ px,
                                                    const double* __restrict__ py, const double* __restrict__ pz,
                                                    double* __restrict__ lo, double* __restrict__ hi) {
    const int64_t g = blockIdx.x * (int64_t)(256 / kBoxLanes) + threadIdx.x / kBoxLanes;
    const int j = threadIdx.x & (kBoxLanes - 1);
    double a[3], b[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        a[k] = INFINITY;
        b[k] = -INFINITY;
    }
    if (g < ng) {
        int32_t f, cnt;
        if (REFIT) {
            f = gfirst[g];
            cnt = gcount[g];
        } else {
            f = starts[g];
            cnt = (g + 1 < ng ? starts[g + 1] : (int32_t)n) - f;
            if (j == 0) {
                gfirst[g] = f;
                gcount[g] = cnt;
            }
        }
        const double r[3] = {px[f], py[f], pz[f]};
        for (int32_t q = j; q < cnt; q += kBoxLanes) {
            double v[3] = {px[f + q], py[f + q], pz[f + q]};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                if (REFIT) v[k] = v[k] - rint(v[k] - r[k]);
                a[k] = v[k] < a[k] ? v[k] : a[k];
                b[k] = v[k] > b[k] ? v[k] : b[k];
            }
        }
    }
#pragma unroll
    for (int o = kBoxLanes / 2; o >= 1; o >>= 1) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double u = __shfl_xor(a[k], o, kBoxLanes);
            const double w = __shfl_xor(b[k], o, kBoxLanes);
            a[k] = u < a[k] ? u : a[k];
            b[k] = w > b[k] ? w : b[k];
        }
    }
    if (g < ng && j == 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            lo[g * 3 + k] = a[k];
            hi[g * 3 + k] = b[k];
        }
    }
}

}  // namespace

bool build_cells_and_groups(Tree& t, int32_t* d_stat, hipStream_t st) {
    const int64_t n = t.n;
    const int64_t nblocks = (n + kLvTile - 1) / kLvTile;
    HostSlot slot(st);
    // per-particle levels, chain lengths and group starts; per-block cell counts
    DevBuf<int8_t> delta(n, st), leaflv(n, st);
    DevBuf<int32_t> start(n, st), mark(n, st), starts(n, st), blk((kLevels + 2) * nblocks, st);
    auto levels = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)nblocks), dim3(threads), 0, st, n, t.keys.get(), t.n_leaf, t.n_group,
                           nblocks, delta.get(), leaflv.get(), start.get(), mark.get(), blk.get());
    };
    // a particle per thread where the tiles do not fill the chip (the kernel
    // is then one tile's latency: 34 us with 256 threads, 14 with 1024, at
    // 131071 particles); four where they do, beside the gather on the second
    // stream (278 against 720 us at 1.3e7)
    if (nblocks <= 512) levels(k_levels<1024>, 1024);
    else levels(k_levels<256>, 256);
    SRF_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_level_scan, dim3(kLevels + 2), dim3(256), 0, st, nblocks, blk.get(), d_stat + kStatTotals);
    SRF_HIP(hipGetLastError());
    // preorder number of each chain's first cell, first particle of each group
    hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)nblocks), dim3(kLvThreads), 0, st, n, nblocks, start.get(),
                       mark.get(), blk.get(), starts.get(), d_stat, slot.device<int32_t>());
    SRF_HIP(hipGetLastError());
    // the one synchronisation: sizes and the device's check of the inputs
    const int32_t* hs = slot.wait<int32_t>();
    // the cells below read the sorted positions, gathered on the second stream
    if (t.gathered) SRF_HIP(hipStreamWaitEvent(st, t.gathered, 0));
    if (hs[kStatFlag] & 1) fail(SRF_EDOMAIN, "non-finite particle position");
    if (hs[kStatFlag] & 2) fail(SRF_EDOMAIN, "particle mass not finite and > 0");
    if (hs[kStatFlag] & 8) return false;   // the order is incomplete (see build_sorted)
    // (a level holds fewer than 2^31 cells: its per-block counts are exact
    // int32 sums of counts below n; the total is checked here)
    LevelBase base;
    int64_t acc = 0;
    int max_level = 0;
    for (int L = 0; L < kLevels; ++L) {
        base.off[L] = (int32_t)(acc < INT32_MAX ? acc : INT32_MAX);
        acc += hs[kStatTotals + L];
        if (hs[kStatTotals + L] > 0) max_level = L;
    }
    if (acc > (int64_t)INT32_MAX - 1)
        fail(SRF_EINVAL, "the tree would hold " + std::to_string(acc) + " cells, past 32-bit cell indices");
    base.off[kLevels] = (int32_t)acc;
    const int64_t nn = acc, ng = hs[kStatTotals + kLevels + 1];
    t.n_nodes = nn;
    t.n_groups = ng;
    t.max_level = max_level;

    // cells: slots and geometry, then counts, moments and links bottom-up
    t.geo.alloc(nn, st);
    t.range.alloc(nn, st);
    t.pack.alloc(nn, st);
    t.prefix.alloc(nn, st);
    t.nM.alloc(nn, st);
    t.nX.alloc(nn, st);
    t.nY.alloc(nn, st);
    t.nZ.alloc(nn, st);
    t.leaf_of.alloc(n, st);
    t.sfirst.alloc(nn, st);
    t.spre.alloc(nn, st);
    t.schild.alloc(nn, st);
    if (may_wave_walk(n, ng, t.n_leaf, max_level) && nn < kWaveWalkCells) t.srec.alloc(nn, st);
    for (int L = 0; L <= kLevels; ++L) t.level_off[L] = base.off[L];
    int32_t* sfirst = t.sfirst.get();
    int32_t* spre = t.spre.get();
    int32_t* schild = t.schild.get();
    DevBuf<int32_t> pfirst(nn, st), scount(nn, st);
    DevBuf<double> sM(nn, st), sX(nn, st), sY(nn, st), sZ(nn, st);
    // the groups' kernel runs beside the cells on the second stream where the
    // gather did; a small tree's would end before the events are recorded
    const bool two = t.gathered != nullptr;
    hipStream_t aux = two ? aux_stream() : st;
    if (two) {
        SRF_HIP(hipEventCreateWithFlags(&t.sized, hipEventDisableTiming));
        SRF_HIP(hipEventCreateWithFlags(&t.grouped, hipEventDisableTiming));
        SRF_HIP(hipEventRecord(t.sized, st));
    }

    hipLaunchKernelGGL(k_cells, dim3((unsigned)nblocks), dim3(kLvThreads), 0, st, n, nblocks, t.keys.get(),
                       delta.get(), leaflv.get(), start.get(), base, blk.get(), t.geo.get(), pfirst.get(),
                       t.prefix.get(), sfirst, spre, schild);
    SRF_HIP(hipGetLastError());
    const MomentArgs ma{n, nn, sfirst, spre, schild, pfirst.get(), start.get(), t.px.get(), t.py.get(), t.pz.get(),
                        t.pm.get(), scount.get(), sM.get(), sX.get(), sY.get(), sZ.get(), t.range.get(), t.nM.get(),
                        t.nX.get(), t.nY.get(), t.nZ.get(), t.leaf_of.get(), t.geo.get(), t.pack.get(), t.srec.get()};
    auto cells_of = [&](int L) { return base.off[L + 1] - base.off[L]; };
    // levels `deepest` and up, bottom-up
    auto levels_up = [&](auto cells, int deepest) {
        constexpr int CELLS = decltype(cells)::value;
        for (int L = deepest; L >= 0; --L) {
            int top = L;   // levels L down to top in one launch
            while (cells_of(L) <= kFewCells && top > 0 && cells_of(top - 1) <= kFewCells) --top;
            if (cells_of(L) <= kFewCells) {
                hipLaunchKernelGGL(k_moments_few<CELLS>, dim3(1), dim3(kMomBlock), 0, st, ma, base, L, top);
                L = top;
            } else {
                const int32_t lo = base.off[L], hi = base.off[L + 1];
                hipLaunchKernelGGL(k_moments<CELLS>, dim3(grid_for(hi - lo, 256 / kMomLanes, 1 << 30)), dim3(256), 0, st,
                                   ma, lo, hi, L < kMaxLevel ? base.off[L + 2] : hi);
            }
            SRF_HIP(hipGetLastError());
        }
    };
    if (nn <= kLeavesFirst) {   // the leaves of every level at once, then the inner cells (the deepest level has none)
        hipLaunchKernelGGL(k_moments<kLeaves>, dim3(grid_for(nn, 256 / kMomLanes, 1 << 30)), dim3(256), 0, st, ma, 0,
                           (int32_t)nn, (int32_t)nn);
        SRF_HIP(hipGetLastError());
        levels_up(std::integral_constant<int, kInner>{}, max_level - 1);
    } else {
        levels_up(std::integral_constant<int, kAllCells>{}, max_level);
        hipLaunchKernelGGL(k_pack, dim3(grid_for(nn, 256, 1 << 30)), dim3(256), 0, st, ma);
        SRF_HIP(hipGetLastError());
    }

    // groups (from their first particles and the sorted positions alone),
    // queued after the cells, which are the longer chain
    t.gfirst.alloc(ng, st);
    t.gcount.alloc(ng, st);
    t.glo.alloc(ng * 3, st);
    t.ghi.alloc(ng * 3, st);
    // on every way out (an error included) `grouped` marks all the work
    // queued on the second stream, and the build's stream waits for it
    // before the starts are freed (declared after them, so destroyed first)
    struct JoinAtExit {
        hipStream_t st, aux;
        hipEvent_t e;
        ~JoinAtExit() {
            if (!e) return;
            (void)hipEventRecord(e, aux);
            (void)hipStreamWaitEvent(st, e, 0);
        }
    } join{st, aux, t.grouped};
    if (two) SRF_HIP(hipStreamWaitEvent(aux, t.sized, 0));
    hipLaunchKernelGGL(k_group_bbox<false>, dim3(grid_for(ng, 256 / kBoxLanes, 1 << 30)), dim3(256), 0, aux, ng, n,
                       starts.get(), t.gfirst.get(), t.gcount.get(), t.px.get(), t.py.get(), t.pz.get(), t.glo.get(),
                       t.ghi.get());
    SRF_HIP(hipGetLastError());
    return true;
}

void refit_cells_and_groups(Tree& t, hipStream_t st) {
    const int64_t n = t.n, nn = t.n_nodes, ng = t.n_groups;
    if (!t.clo.get()) {
        t.clo.alloc(nn * 3, st);
        t.chi.alloc(nn * 3, st);
    }
    DevBuf<double> sM(nn, st), sX(nn, st), sY(nn, st), sZ(nn, st), sbox(nn * 6, st);
    for (int L = t.max_level; L >= 0; --L) {
        const int32_t lo = t.level_off[L], hi = t.level_off[L + 1];
        if (hi <= lo) continue;
        const int32_t next_hi = L < kMaxLevel ? t.level_off[L + 2] : hi;
        hipLaunchKernelGGL(k_refit_level, dim3(grid_for(hi - lo, 256 / kMomLanes, 1 << 30)), dim3(256), 0, st, lo,
                           hi, next_hi, n, t.sfirst.get(), t.spre.get(), t.schild.get(), t.geo.get(), t.range.get(),
                           t.px.get(), t.py.get(), t.pz.get(), t.pm.get(), sM.get(), sX.get(), sY.get(), sZ.get(),
                           sbox.get(), t.nM.get(), t.nX.get(), t.nY.get(), t.nZ.get(), t.clo.get(), t.chi.get());
        SRF_HIP(hipGetLastError());
    }
    if (!t.rpack.get()) t.rpack.alloc(nn, st);
    hipLaunchKernelGGL(k_refit_pack, dim3(grid_for(nn, 256, 1 << 30)), dim3(256), 0, st, nn, t.geo.get(),
                       t.range.get(), t.clo.get(), t.chi.get(), t.rpack.get());
    SRF_HIP(hipGetLastError());
    if (ng > 0) {
        hipLaunchKernelGGL(k_group_bbox<true>, dim3(grid_for(ng, 256 / kBoxLanes, 1 << 30)), dim3(256), 0, st, ng, n,
                           (const int32_t*)nullptr, t.gfirst.get(), t.gcount.get(), t.px.get(), t.py.get(),
                           t.pz.get(), t.glo.get(), t.ghi.get());
        SRF_HIP(hipGetLastError());
    }
}

}  // namespace srf
