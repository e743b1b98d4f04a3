// Step a6: per-group interaction lists (Barnes' modified traversal with the
// cutoff pruning of the short-range part).
//
// A walk decides for each group which cells are pruned, accepted or opened and
// which leaves remain, counts the entries, and stores one item per leaf or
// accepted cell, in DFS order, in the group's slot of a scratch array.  A scan
// places the lists, and an expansion pass writes the entries (a leaf's
// particles ascending, cells in preorder) with one wave per group, so that the
// list memory is written in whole lines.
//
// Usually one wave walks for each group, with a stack in LDS (k_walk).  Large
// trees with short lists, and those where some group fits neither its slot nor
// the stack, are walked by one thread per group (k_lists; walks.h has the rule)
// without a stack, over the preorder cell array: a cell that is pruned, accepted
// or a leaf is left through its skip link, any other cell is opened by stepping
// to the next preorder index (its first child).  When a list does not fit the
// slot of that walk, a second one stores every group's items compactly.
//
// Compiled with -ffp-contract=off: the decisions are the literal FP64
// expressions, evaluated in this order:
//   per axis t = |cen_c - cen_g|, t = min(t, 1 - t), e = max(0, t - (half + h_g))
//   d2 = (e_x e_x + e_y e_y) + e_z e_z
//   prune  iff d2(half = side/2) >= r_cut * r_cut
//   accept iff side * side < (theta * theta) * d2(half = 0)
// with cen_c the cell's geometric centre, or for the acceptance test of the
// centre-of-mass criterion its centre of mass.  A refitted tree measures
// each cell by the box [lo, hi] of its particles instead, every bound
// rounded outward to a multiple of 2^-(level + 10) (a cell whose bounds do
// not fit 16-bit offsets from its centre is never pruned or accepted):
//   cen_c = (lo + hi) * 0.5, half = (hi - lo) * 0.5 per axis,
//   per axis t = cen_c - cen_g, t = |t - rint(t)|, e = max(0, t - (half + h_g))
//   d2 as above; prune iff d2 >= r_cut * r_cut,
//   accept iff s * s < (theta * theta) * d2(half = 0, cen_c or the centre of mass),
// s the larger of the cell's dyadic side and the box's longest side
// (2 max(half)), so that a cell holding a member of the group is never
// accepted, however small its box.  For a fresh tree the walk first takes
// the two tests in FP32 with an error margin, and evaluates the FP64
// expressions only for the few cells whose FP32 values lie within the
// margin of a threshold (classify32 below): the decisions, and so the
// lists, are those of the FP64 expressions.
#include <type_traits>

#include "common.h"
#include "walks.h"

namespace srf {
namespace {

struct Frame {
    double cg[3], hg[3];
};

__device__ __forceinline__ Frame group_frame(const double* __restrict__ lo, const double* __restrict__ hi, int64_t g) {
    Frame f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double l = lo[g * 3 + a], h = hi[g * 3 + a];
        f.cg[a] = (l + h) * 0.5;
        f.hg[a] = (h - l) * 0.5;
    }
    return f;
}

__device__ __forceinline__ double axis_gap(double cen, double cg, double half) {
    double t = fabs(cen - cg);
    double t2 = 1.0 - t;
    t = t2 < t ? t2 : t;
    double r = t - half;
    return r > 0.0 ? r : 0.0;
}

// Decoded cell: exact centre and side.
struct Cell {
    double c[3], side, hs;
    int level, leaf;
    uint32_t count;
    int64_t skip;
};

// The cell of an 8-byte walk record, its coordinates found from those of
// the cell visited before (w): the new cell's parent is that cell or one of
// its ancestors, at level k.level - 1, whose coordinates are w's shifted
// down by the levels between; the cell's own low bits are `oct`.
struct WalkPos {
    uint32_t ix = 0, iy = 0, iz = 0;
    int level = -1;
};

__device__ __forceinline__ Cell decode_walk(const uint2 r, WalkPos& w) {
    Cell k;
    k.level = (int)(r.x & 31u);
    k.leaf = (int)((r.x >> 5) & 1u);
    const uint32_t oct = (r.x >> 6) & 7u;
    k.count = r.x >> 9;
    k.skip = (int64_t)r.y;
    const int sh = w.level + 1 - k.level;
    w.ix = ((w.ix >> sh) << 1) | (oct >> 2);
    w.iy = ((w.iy >> sh) << 1) | ((oct >> 1) & 1u);
    w.iz = ((w.iz >> sh) << 1) | (oct & 1u);
    w.level = k.level;
    return k;
}

// The exact centre and side of the cell last decoded into w.
__device__ __forceinline__ void cell_geometry(Cell& k, const WalkPos& w) {
    k.side = ldexp(1.0, -k.level);
    k.hs = k.side * 0.5;
    k.c[0] = ldexp((double)w.ix + 0.5, -k.level);
    k.c[1] = ldexp((double)w.iy + 0.5, -k.level);
    k.c[2] = ldexp((double)w.iz + 0.5, -k.level);
}

__device__ __forceinline__ Cell decode(const uint4 r) {
    Cell k;
    k.level = (int)(r.w & 31u);
    k.leaf = (int)((r.w >> 5) & 1u);
    k.count = r.w >> 6;
    k.skip = (int64_t)((r.x >> 21) | ((r.y >> 21) << 11) | ((r.z >> 21) << 22));
    k.side = ldexp(1.0, -k.level);
    k.hs = k.side * 0.5;
    k.c[0] = ldexp((double)(r.x & 0x1fffffu) + 0.5, -k.level);
    k.c[1] = ldexp((double)(r.y & 0x1fffffu) + 0.5, -k.level);
    k.c[2] = ldexp((double)(r.z & 0x1fffffu) + 0.5, -k.level);
    return k;
}

// 0: pruned, 1: accepted as a monopole, 2: leaf (expand), 3: open.  `mc`
// is the point the acceptance test measures to (the geometric centre, or
// the centre of mass with the centre-of-mass criterion).
__device__ __forceinline__ int classify(const Cell& k, const double* mc, const Frame& f, double rc2, double th2) {
    double ex = axis_gap(k.c[0], f.cg[0], k.hs + f.hg[0]);
    double ey = axis_gap(k.c[1], f.cg[1], k.hs + f.hg[1]);
    double ez = axis_gap(k.c[2], f.cg[2], k.hs + f.hg[2]);
    double D2 = (ex * ex + ey * ey) + ez * ez;
    if (D2 >= rc2) return 0;
    ex = axis_gap(mc[0], f.cg[0], f.hg[0]);
    ey = axis_gap(mc[1], f.cg[1], f.hg[1]);
    ez = axis_gap(mc[2], f.cg[2], f.hg[2]);
    double d2 = (ex * ex + ey * ey) + ez * ez;
    if (k.side * k.side < th2 * d2) return 1;
    return k.leaf ? 2 : 3;
}

// A first look in FP32 at the same two tests.  Every quantity before the
// squares is within 4e-7 of its exact value (the centres are exact in FP32,
// the group's centre and half sizes are rounded once, and each of the four
// operations per axis rounds a value below 1), so a squared distance D2 is
// within 1.4e-6 sqrt(D2) + 2.4e-7 D2 + 1e-12 of its exact value; FP64 is
// within 1e-15.  A test is decided here only when the FP32 value clears its
// threshold X by more than b(X) = 2.5e-6 sqrt(X) + 2e-6 X + 1e-12, which
// exceeds both errors together, so that the FP64 expressions would decide
// the same way; otherwise (-1) they are evaluated.
struct Frame32 {
    float cg[3], hg[3];
};

__device__ __forceinline__ float axis_gap32(float cen, float cg, float half) {
    float t = fabsf(cen - cg);
    const float t2 = 1.0f - t;
    t = t2 < t ? t2 : t;
    const float r = t - half;
    return r > 0.0f ? r : 0.0f;
}

// rc_hi / rc_lo: r_cut^2 +- b(r_cut^2); inv_th: 1 / theta.
__device__ __forceinline__ int classify32(int level, int leaf, const float* c, const float* mc, const Frame32& f,
                                          float rc_hi, float rc_lo, float inv_th) {
    const float side = __int_as_float((127 - level) << 23);   // 2^-level, exact
    const float hs = side * 0.5f;
    float ex = axis_gap32(c[0], f.cg[0], hs + f.hg[0]);
    float ey = axis_gap32(c[1], f.cg[1], hs + f.hg[1]);
    float ez = axis_gap32(c[2], f.cg[2], hs + f.hg[2]);
    const float D2 = (ex * ex + ey * ey) + ez * ez;
    if (D2 >= rc_hi) return 0;
    if (!(D2 < rc_lo)) return -1;
    ex = axis_gap32(mc[0], f.cg[0], f.hg[0]);
    ey = axis_gap32(mc[1], f.cg[1], f.hg[1]);
    ez = axis_gap32(mc[2], f.cg[2], f.hg[2]);
    const float d2 = (ex * ex + ey * ey) + ez * ez;
    const float sx = side * inv_th, X = sx * sx;   // accept iff d2 > side^2 / theta^2
    const float b = 2.5e-6f * sx + 2e-6f * X + 1e-12f;
    if (d2 > X + b) return 1;
    if (!(d2 < X - b)) return -1;
    return leaf ? 2 : 3;
}

struct Bounds32 {
    float rc_hi, rc_lo, inv_th;
};

__device__ __forceinline__ Bounds32 bounds32(double rc2, double th2) {
    const float rc2f = (float)rc2;
    const float bp = 2.5e-6f * sqrtf(rc2f) + 2e-6f * rc2f + 1e-12f;
    return {rc2f + bp, rc2f - bp, th2 > 0.0 ? (float)(1.0 / sqrt(th2)) : INFINITY};
}

__device__ __forceinline__ double refit_axis_gap(double cen, double cg, double half) {
    double t = cen - cg;
    t = fabs(t - rint(t));
    double r = t - half;
    return r > 0.0 ? r : 0.0;
}

// The rounded box of a refitted cell: bound K q with K the stored offset
// plus the centre's multiple ic * 1024 + 512 (exact in FP64).
__device__ __forceinline__ void refit_box(const RefitCell& r, const Cell& k, double* bl, double* bh) {
    const uint32_t ic[3] = {r.pk.x & 0x1fffffu, r.pk.y & 0x1fffffu, r.pk.z & 0x1fffffu};
    const int e = k.level + kRefitShift;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int64_t kc = (int64_t)ic[a] * (1 << kRefitShift) + (1 << (kRefitShift - 1));
        const int32_t lo = (int32_t)(int16_t)(r.b[a] & 0xffff), hi = r.b[a] >> 16;
        bl[a] = ldexp((double)(kc + lo), -e);
        bh[a] = ldexp((double)(kc + hi), -e);
    }
}

// The same classification for a cell of a refitted tree with box [bl, bh].
__device__ __forceinline__ int classify_refit(const Cell& k, const double* bl, const double* bh, const double* mc,
                                              bool com, const Frame& f, double rc2, double th2) {
    double cen[3], half[3], hmax = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        cen[a] = (bl[a] + bh[a]) * 0.5;
        half[a] = (bh[a] - bl[a]) * 0.5;
        hmax = half[a] > hmax ? half[a] : hmax;
    }
    double side = hmax + hmax;
    side = k.side > side ? k.side : side;
    double ex = refit_axis_gap(cen[0], f.cg[0], half[0] + f.hg[0]);
    double ey = refit_axis_gap(cen[1], f.cg[1], half[1] + f.hg[1]);
    double ez = refit_axis_gap(cen[2], f.cg[2], half[2] + f.hg[2]);
    double D2 = (ex * ex + ey * ey) + ez * ez;
    if (D2 >= rc2) return 0;
    const double* m = com ? mc : cen;
    ex = refit_axis_gap(m[0], f.cg[0], 0.0 + f.hg[0]);
    ey = refit_axis_gap(m[1], f.cg[1], 0.0 + f.hg[1]);
    ez = refit_axis_gap(m[2], f.cg[2], 0.0 + f.hg[2]);
    double d2 = (ex * ex + ey * ey) + ez * ez;
    if (side * side < th2 * d2) return 1;
    return k.leaf ? 2 : 3;
}

// The class of the cell of a slot record (its preorder id `pre`), by the
// tests of k_lists: FP32 first for a built tree, its rounded box for a
// refitted one.
template <bool COM, bool REFIT>
__device__ __forceinline__ int classify_slot(const uint4& r, int level, bool leaf, int32_t pre,
                                             const double* __restrict__ nX, const double* __restrict__ nY,
                                             const double* __restrict__ nZ, const RefitCell* __restrict__ rpack,
                                             const Frame& f, const Frame32& f32, const Bounds32& b32, double rc2,
                                             double th2) {
    const uint32_t ix = r.x & 0x1fffffu, iy = r.y & 0x1fffffu, iz = r.z & 0x1fffffu;
    Cell k;
    k.level = level;
    k.leaf = leaf;
    double com[3] = {0.0, 0.0, 0.0};
    if (COM) {
        com[0] = nX[pre];
        com[1] = nY[pre];
        com[2] = nZ[pre];
    }
    WalkPos w;
    w.ix = ix;
    w.iy = iy;
    w.iz = iz;
    if (REFIT) {
        RefitCell rc;
        rc.pk = r;
        const int4 b = *reinterpret_cast<const int4*>(rpack[pre].b);
        rc.b[0] = b.x;
        rc.b[1] = b.y;
        rc.b[2] = b.z;
        rc.b[3] = b.w;
        if (!(rc.b[3] & 1)) return leaf ? 2 : 3;
        k.side = ldexp(1.0, -level);
        double bl[3], bh[3];
        refit_box(rc, k, bl, bh);
        return classify_refit(k, bl, bh, com, COM, f, rc2, th2);
    }
    // (i + 1/2) 2^-level: exact in FP32 (i < 2^21)
    const float side32 = __int_as_float((127 - level) << 23), hs32 = side32 * 0.5f;
    const float c32[3] = {__fmaf_rn((float)ix, side32, hs32), __fmaf_rn((float)iy, side32, hs32),
                          __fmaf_rn((float)iz, side32, hs32)};
    const float m32[3] = {COM ? (float)com[0] : c32[0], COM ? (float)com[1] : c32[1], COM ? (float)com[2] : c32[2]};
    const int cls = classify32(level, leaf, c32, m32, f32, b32.rc_hi, b32.rc_lo, b32.inv_th);
    if (cls >= 0) return cls;
    cell_geometry(k, w);
    return classify(k, COM ? com : k.c, f, rc2, th2);
}

// Items of one group pass through a 16-slot LDS buffer of the thread and go
// to memory as aligned 64-byte chunks (the partial chunks at the two ends of
// a group's items are written item by item), so that the item array is
// written in whole lines rather than by scattered 4-byte stores.
constexpr int kWc = 16;          // items per chunk
constexpr int kWcStride = 17;    // LDS slots per thread (padding against bank conflicts)

struct ItemWriter {
    int32_t* buf;      // this thread's LDS slots
    int32_t* dst;      // the item array
    int64_t start;     // index of the group's first item
    int64_t pos;       // index of the next item
    int64_t end;       // capacity limit: items at or past `end` are counted, not stored
    __device__ __forceinline__ void put(int32_t v) {
        if (pos < end) buf[pos & (kWc - 1)] = v;
        ++pos;
        if ((pos & (kWc - 1)) == 0 && pos <= end) {
            const int64_t c0 = pos - kWc;
            if (c0 >= start) {
                int4* d = reinterpret_cast<int4*>(dst + c0);
#pragma unroll
                for (int k = 0; k < kWc / 4; ++k) d[k] = make_int4(buf[4 * k], buf[4 * k + 1], buf[4 * k + 2], buf[4 * k + 3]);
            } else {
                for (int64_t k = start; k < pos; ++k) dst[k] = buf[k & (kWc - 1)];
            }
        }
    }
    __device__ __forceinline__ void finish() {
        if (pos > end) return;
        int64_t k = pos & ~(int64_t)(kWc - 1);
        if (k < start) k = start;
        for (; k < pos; ++k) dst[k] = buf[k & (kWc - 1)];
    }
};

// One thread walks the cell array once for G consecutive groups.  A cell
// is visited while at least one of them opened its parent; mask[L] (G bits
// per level, packed in one 64-bit word) holds the groups that opened the
// visited cell's parent at level L - 1.
//
// The counting walk (WRITE = false) sizes each group's list and also stores
// its items into a slot of kSlot items per group (items past the slot are
// counted in totals[3], and the lists are then rebuilt with WRITE = true:
// a second walk that stores the items of every group compactly at ioff).
constexpr int64_t kSlot = 2048;
// The totals (particle entries, cell entries, interactions, groups that did
// not fit) are kept in kTotals rows of four, block b adding to row b mod
// kTotals, and summed at the end: one row for all groups made the waves'
// walk wait for its atomics (34 ns a group, 1.9 ms at 51000 groups).
constexpr int kTotals = 256;
constexpr int kListThreads = 64;   // one wave per block (128 and 256 measured slower)

template <int G, bool WRITE, bool COM, bool REFIT>
__global__ __launch_bounds__(kListThreads) void k_lists(int64_t ng, const double* __restrict__ glo,
                                               const double* __restrict__ ghi, const int32_t* __restrict__ gcount,
                                               const uint2* __restrict__ pack, const NodeRange* __restrict__ rng,
                                               const double* __restrict__ nX, const double* __restrict__ nY,
                                               const double* __restrict__ nZ,
                                               const RefitCell* __restrict__ rpack, int64_t nn, double rc2, double th2, int64_t* __restrict__ cnt,
                                               int64_t* __restrict__ icnt, unsigned long long* __restrict__ totals,
                                               const int64_t* __restrict__ ioff, int32_t* __restrict__ items) {
    static_assert(G * kLevels <= 64, "level masks must fit one word");
    const int64_t t = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const int64_t g0 = t * G;
    __shared__ int32_t wbuf[kListThreads * G * kWcStride];
    Frame f[G];
    int64_t np[G], nc[G], w[G];
    ItemWriter out[G];
    uint64_t valid = 0;
#pragma unroll
    for (int q = 0; q < G; ++q) {
        np[q] = nc[q] = w[q] = 0;
        const int64_t g = g0 + q < ng ? g0 + q : ng - 1;
        f[q] = group_frame(glo, ghi, g);
        if (g0 + q < ng) valid |= 1ull << q;
        out[q].buf = wbuf + (threadIdx.x * G + q) * kWcStride;
        out[q].dst = items;
        out[q].start = out[q].pos = WRITE ? ioff[g] : g * kSlot;
        out[q].end = WRITE ? INT64_MAX : g * kSlot + kSlot;
    }
    Frame32 f32[G];
#pragma unroll
    for (int q = 0; q < G; ++q)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            f32[q].cg[a] = (float)f[q].cg[a];
            f32[q].hg[a] = (float)f[q].hg[a];
        }
    const Bounds32 b32 = bounds32(rc2, th2);
    const uint64_t full = (1ull << G) - 1ull;
    uint64_t masks = valid;  // level 0
    int64_t i = valid ? 0 : nn;
    WalkPos wpos;
    while (i < nn) {
        RefitCell rc;
        if (REFIT) rc = rpack[i];
        Cell k = REFIT ? decode(rc.pk) : decode_walk(pack[i], wpos);
        const uint64_t act = (masks >> (k.level * G)) & full;
        uint64_t open = 0;
        if (act) {
            float c32[3] = {0.0f, 0.0f, 0.0f}, mc32[3] = {0.0f, 0.0f, 0.0f};
            double com[3] = {0.0, 0.0, 0.0};
            if (!REFIT) {
                const float side32 = __int_as_float((127 - k.level) << 23);
                const float hs32 = side32 * 0.5f;
                // (i + 1/2) 2^-level: exact in FP32 (i < 2^21)
                c32[0] = __fmaf_rn((float)wpos.ix, side32, hs32);
                c32[1] = __fmaf_rn((float)wpos.iy, side32, hs32);
                c32[2] = __fmaf_rn((float)wpos.iz, side32, hs32);
                mc32[0] = c32[0];
                mc32[1] = c32[1];
                mc32[2] = c32[2];
            }
            if (COM) {
                com[0] = nX[i];
                com[1] = nY[i];
                com[2] = nZ[i];
                mc32[0] = (float)com[0];
                mc32[1] = (float)com[1];
                mc32[2] = (float)com[2];
            }
            bool geom = REFIT;   // FP64 geometry computed (a refitted cell's comes with its record)
            double mcen[3] = {0.0, 0.0, 0.0};
            if (REFIT) {
                mcen[0] = COM ? com[0] : k.c[0];
                mcen[1] = COM ? com[1] : k.c[1];
                mcen[2] = COM ? com[2] : k.c[2];
            }
            double bl[3] = {0, 0, 0}, bh[3] = {0, 0, 0};
            bool bounded = true;
            if (REFIT) {
                bounded = rc.b[3] & 1;
                refit_box(rc, k, bl, bh);
            }
#pragma unroll
            for (int q = 0; q < G; ++q) {
                if (!((act >> q) & 1ull)) continue;
                int cls;
                if (REFIT) {
                    cls = bounded ? classify_refit(k, bl, bh, mcen, COM, f[q], rc2, th2) : (k.leaf ? 2 : 3);
                } else {
                    cls = classify32(k.level, k.leaf, c32, mc32, f32[q], b32.rc_hi, b32.rc_lo, b32.inv_th);
                    if (cls < 0) {
                        if (!geom) {
                            cell_geometry(k, wpos);
                            mcen[0] = COM ? com[0] : k.c[0];
                            mcen[1] = COM ? com[1] : k.c[1];
                            mcen[2] = COM ? com[2] : k.c[2];
                            geom = true;
                        }
                        cls = classify(k, mcen, f[q], rc2, th2);
                    }
                }
                if (cls == 3) {
                    open |= 1ull << q;
                } else if (cls == 1) {
                    out[q].put(-(int32_t)i - 1);
                    if (!WRITE) ++nc[q];
                } else if (cls == 2) {
                    out[q].put((int32_t)i);
                    if (!WRITE) {
                        uint32_t m = k.count;
                        if (m == (REFIT ? kPackCountMax : kWalkCountMax)) m = (uint32_t)rng[i].count;
                        np[q] += m;
                        ++w[q];
                    }
                }
            }
        }
        if (open) {
            const int sh = (k.level + 1) * G;
            masks = (masks & ~(full << sh)) | (open << sh);
            ++i;
        } else {
            i = k.skip;
        }
    }
#pragma unroll
    for (int q = 0; q < G; ++q)
        if ((valid >> q) & 1ull) out[q].finish();
    if (WRITE) return;
    unsigned long long a = 0, b = 0, c = 0, d = 0;
#pragma unroll
    for (int q = 0; q < G; ++q) {
        if (!((valid >> q) & 1ull)) continue;
        cnt[g0 + q] = np[q] + nc[q];
        icnt[g0 + q] = w[q] + nc[q];   // leaves + accepted cells
        a += (unsigned long long)np[q];
        b += (unsigned long long)nc[q];
        c += (unsigned long long)gcount[g0 + q] * (unsigned long long)(np[q] + nc[q]);
        d += (w[q] + nc[q] > kSlot) ? 1ull : 0ull;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        a += __shfl_xor(a, o, 64);
        b += __shfl_xor(b, o, 64);
        c += __shfl_xor(c, o, 64);
        d += __shfl_xor(d, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        totals += 4 * (blockIdx.x & (kTotals - 1));
        atomicAdd(&totals[0], a);
        atomicAdd(&totals[1], b);
        atomicAdd(&totals[2], c);
        if (d) atomicAdd(&totals[3], d);
    }
}

// The same lists from one wave per group (where walks.h says so).  The wave
// keeps the cells its group still has to
// look at on a stack in LDS, as level slots; it takes up to 64 of them at a
// time, one per lane, and pushes the children of those it opens (they are
// one run of the next level's slots, so their records are read side by
// side).  Items go to the group's slot as they are found, and are put in
// preorder at the end by a bitonic sort in registers: the order in which the
// thread's walk finds them.
//
// A thread's walk is a chain of dependent loads, one per visited cell: about
// 1.1 ms for a clustered set of any size below 10^6 particles, with a wave
// for 64 groups and most of the chip idle.  Here the chain is one load per 64
// cells, and the waves are 64 times as many; but it issues more instructions
// per group (idle lanes in the top levels, the sort).
// k_lists against k_walk, us: 160 / 11 at 4096 uniform particles (96 groups),
// 1117 / 49 at 131071 clustered ones (3050), 1564 / 383 at 2^21 (51000), 744
// / 184 at 2^21 on the Zel'dovich lattice (33000), 1594 / 1317 at 1.3e7
// clustered (316000, 14 levels); refitted trees at 2^21: 933 / 290.
// In trees of at most kWideGroups groups a slot holds kWideSlot items (a group
// of a void beside clumps of a 2 x 10^5 particle set has 2100), and a group of
// more than kWaveItems leaves them unsorted for k_sort_wide, whose registers
// would cost this kernel its occupancy; they are counted in the low half of
// totals[3].  A group that fits neither its slot nor the stack is counted in
// the high half and leaves its list empty; the thread's walk then does the
// whole tree.  Such a group also sets *gave_up, and the waves that start after
// it leave at once: their lists would be thrown away (make_lists with
// single-particle leaves, where groups in clusters do not fit, threads alone /
// with a whole walk before / with one given up, us: 8453 / 9150 / 8690 for 4.1e6
// clustered particles, 9468 / 11173 / 9641 for 8e6).
constexpr int kWaveStack = 1536;   // 6 KB of LDS
constexpr int kWaveItems = 2048;   // what the sort takes
constexpr int64_t kWideSlot = 4096;
constexpr int64_t kWideGroups = 1 << 16;   // 1 GB of slots
constexpr unsigned long long kUnsorted = 1ull, kOverflow = 1ull << 32;
static_assert(kWaveItems == kSlot, "a narrow slot's items are sorted where they are found");

// The value of lane ^ M.
template <int M>
__device__ __forceinline__ int lane_xor(int x) {
    if (M == 1) return __builtin_amdgcn_mov_dpp(x, 0xb1, 0xf, 0xf, true);    // quad_perm:[1,0,3,2]
    if (M == 2) return __builtin_amdgcn_mov_dpp(x, 0x4e, 0xf, 0xf, true);    // quad_perm:[2,3,0,1]
    if (M == 8) return __builtin_amdgcn_mov_dpp(x, 0x128, 0xf, 0xf, true);   // row_ror:8
    if (M == 32) return __shfl_xor(x, 32, 64);
    return __builtin_amdgcn_ds_swizzle(x, (M << 10) | 0x1f);
}

template <int R, int K, int M>
__device__ __forceinline__ void bitonic_step(int (&v)[R], int lane) {
    // element e = lane R + r; ascending where bit K of e is clear
    if constexpr (M >= R) {
        const bool low = ((lane & (M / R)) == 0) == ((lane & (K / R)) == 0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int o = lane_xor<M / R>(v[r]);
            const int mn = v[r] < o ? v[r] : o, mx = v[r] < o ? o : v[r];
            v[r] = low ? mn : mx;
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r & M) continue;
            const bool up = K >= R ? (lane & (K / R)) == 0 : (r & K) == 0;
            const int x = v[r], y = v[r | M];
            const int mn = x < y ? x : y, mx = x < y ? y : x;
            v[r] = up ? mn : mx;
            v[r | M] = up ? mx : mn;
        }
    }
    if constexpr (M > 1) bitonic_step<R, K, M / 2>(v, lane);
}

template <int R, int K>
__device__ __forceinline__ void bitonic_merge(int (&v)[R], int lane) {
    bitonic_step<R, K, K / 2>(v, lane);
    if constexpr (K < 64 * R) bitonic_merge<R, 2 * K>(v, lane);
}

// n <= 64 R item keys (2 preorder + accepted) at out sorted, and left there as
// items.
template <int R>
__device__ __forceinline__ void sort_items(int n, int lane, int32_t* out) {
    int v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = r * 64 + lane < n ? out[r * 64 + lane] : INT32_MAX;
    bitonic_merge<R, 2>(v, lane);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int32_t c = v[r] >> 1;
        if (lane * R + r < n) out[lane * R + r] = (v[r] & 1) ? -c - 1 : c;
    }
}

template <bool COM, bool REFIT>
__global__ __launch_bounds__(64) void k_walk(int64_t ng, const double* __restrict__ glo,
                                             const double* __restrict__ ghi, const int32_t* __restrict__ gcount,
                                             const uint4* __restrict__ srec, const int32_t* __restrict__ spre,
                                             const double* __restrict__ nX, const double* __restrict__ nY,
                                             const double* __restrict__ nZ, const RefitCell* __restrict__ rpack,
                                             double rc2, double th2, int64_t* __restrict__ cnt,
                                             int64_t* __restrict__ icnt, unsigned long long* __restrict__ totals,
                                             int32_t* __restrict__ items, int64_t slot) {
    __shared__ int32_t stack[kWaveStack];   // filled from the back
    const int lane = threadIdx.x;
    const int64_t g = xcd_block(blockIdx.x, gridDim.x);
    const Frame f = group_frame(glo, ghi, g);
    Frame32 f32;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        f32.cg[a] = (float)f.cg[a];
        f32.hg[a] = (float)f.hg[a];
    }
    const Bounds32 b32 = bounds32(rc2, th2);
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    unsigned long long* gave_up = totals + 4 * kTotals;
    totals += 4 * (blockIdx.x & (kTotals - 1));
    if (__hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
        if (lane == 0) cnt[g] = icnt[g] = 0;
        return;
    }
    int32_t* out = items + g * slot;
    int ni = 0, top = kWaveStack - 1;   // the stack is stack[top, kWaveStack)
    uint32_t np = 0, nc = 0;
    if (lane == 0) stack[top] = 0;   // the root is slot 0
    __syncthreads();
    while (top < kWaveStack) {
        const bool on = top + lane < kWaveStack;
        int cls = 0, kids = 0;
        int32_t pre = 0;
        uint32_t a = 0;
        if (on) {
            const int32_t c = stack[top + lane];
            const uint4 r = srec[c];
            pre = spre[c];
            const int level = (int)(r.w & 31u);
            kids = (int)(r.w >> 5);
            a = (r.x >> 21) | ((r.y >> 21) << 11) | ((r.z >> 21) << 22);
            cls = classify_slot<COM, REFIT>(r, level, kids == 0, pre, nX, nY, nZ, rpack, f, f32, b32, rc2, th2);
        }
        top = top + 64 < kWaveStack ? top + 64 : kWaveStack;
        const bool item = cls == 1 || cls == 2;
        const uint64_t mi = __ballot(item);
        if (cls != 3) kids = 0;
        const int incl = wave_scan(kids);
        const int push = __builtin_amdgcn_readlane(incl, 63), found = __popcll(mi);
        if (ni + found > slot || push > top) {
            if (lane == 0) {
                cnt[g] = icnt[g] = 0;
                atomicAdd(&totals[3], kOverflow);
                __hip_atomic_store(gave_up, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            return;
        }
        __syncthreads();   // the stack's entries are read before they are overwritten
        if (item) out[ni + __popcll(mi & lt)] = 2 * pre + (cls == 1 ? 1 : 0);
        if (cls == 1) ++nc;
        if (cls == 2) np += a;
        ni += found;
        top -= push;
        int32_t* d = stack + top + incl - kids;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (k < kids) d[k] = (int32_t)a + k;
        __syncthreads();
    }
    __threadfence_block();   // the keys are read back by other lanes
    if (ni <= 256) sort_items<4>(ni, lane, out);
    else if (ni <= 512) sort_items<8>(ni, lane, out);
    else if (ni <= 1024) sort_items<16>(ni, lane, out);
    else if (ni <= kWaveItems) sort_items<32>(ni, lane, out);
    else if (lane == 0) atomicAdd(&totals[3], kUnsorted);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        np += __shfl_xor(np, o, 64);
        nc += __shfl_xor(nc, o, 64);
    }
    if (lane == 0) {
        cnt[g] = (int64_t)np + nc;
        icnt[g] = ni;
        atomicAdd(&totals[0], (unsigned long long)np);
        atomicAdd(&totals[1], (unsigned long long)nc);
        atomicAdd(&totals[2], (unsigned long long)gcount[g] * ((unsigned long long)np + nc));
    }
}

__global__ __launch_bounds__(64) void k_sort_wide(const int64_t* __restrict__ icnt, int32_t* __restrict__ items) {
    const int64_t n = icnt[blockIdx.x];
    if (n > kWaveItems) sort_items<64>((int)n, threadIdx.x, items + blockIdx.x * kWideSlot);
}

// One block: the totals' rows summed into *host (pinned memory), and, with ng
// > 0, the exclusive scan of the ng list lengths in place with the total at
// the end, four lengths a thread at a time.
constexpr int kScanBlock = 1024;
constexpr int64_t kScanGroups = 16384;   // one block's scan is shorter than the general one's three launches

__global__ __launch_bounds__(kScanBlock) void k_list_totals(int64_t ng, int64_t* __restrict__ off,
                                                            const unsigned long long* __restrict__ totals,
                                                            unsigned long long* __restrict__ host) {
    __shared__ unsigned long long part[4][kTotals / 64];
    __shared__ int64_t wsum[kScanBlock / 64];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    if (tid < kTotals) {
        unsigned long long v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = totals[4 * tid + k];
            for (int o = 32; o >= 1; o >>= 1) v[k] += __shfl_xor(v[k], o, 64);
            if (lane == 0) part[k][wid] = v[k];
        }
    }
    __syncthreads();
    if (tid < 4) {
        unsigned long long v = 0;
        for (int w = 0; w < kTotals / 64; ++w) v += part[tid][w];
        host[tid] = v;
    }
    int64_t carry = 0;
    for (int64_t c0 = 0; c0 < ng; c0 += 4 * kScanBlock) {
        const int64_t j = c0 + 4 * (int64_t)tid;
        int64_t v[4], sum = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = j + k < ng ? off[j + k] : 0;
            sum += v[k];
        }
        int64_t incl = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t u = __shfl_up(incl, o, 64);
            if (lane >= o) incl += u;
        }
        if (lane == 63) wsum[wid] = incl;
        __syncthreads();
        int64_t at = carry + incl - sum;
#pragma unroll
        for (int w = 0; w < kScanBlock / 64; ++w) {
            at += w < wid ? wsum[w] : 0;
            carry += wsum[w];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (j + k < ng) off[j + k] = at;
            at += v[k];
        }
    }
    if (tid == 0 && ng > 0) off[ng] = carry;
}

// Expansion: one wave per group turns its items into entries.  A leaf item
// stands for its particles first..first+count-1, a cell item for itself.
// Items are taken kExpandItems at a time: each lane loads four of them, the
// next batch's four while it places these, and the four items' ranges (all
// of a batch's range loads in flight together), a scan of the item sizes
// places each item, and the entries are written
// either through an LDS buffer (each lane writes its own items' entries,
// then the wave copies the buffer out, 64 consecutive entries per store) or,
// when the batch's entries exceed the buffer, directly, lane k writing
// entries k, k + 64, ... and finding its item by binary search over the
// scan.
// Items of group g: icnt[g] of them from g * slot when slot > 0, else
// [ioff[g], ioff[g + 1]).
constexpr int kExpandBuf = 1024;
constexpr int kExpandPer = 4;                   // items per lane per batch
constexpr int kExpandItems = 64 * kExpandPer;   // items per batch

__global__ __launch_bounds__(64) void k_expand(int64_t ng, int64_t slot, const int64_t* __restrict__ icnt,
                                               const int64_t* __restrict__ ioff, const int32_t* __restrict__ items,
                                               const NodeRange* __restrict__ rng, const int64_t* __restrict__ off,
                                               int32_t* __restrict__ ent) {
    __shared__ int32_t s_end[kExpandItems], s_first[kExpandItems];
    __shared__ int32_t s_ent[kExpandBuf];
    const int64_t g = xcd_block(blockIdx.x, gridDim.x);
    if (g >= ng) return;
    const int lane = threadIdx.x;
    const int64_t i0 = slot > 0 ? g * slot : ioff[g];
    const int64_t i1 = slot > 0 ? i0 + icnt[g] : ioff[g + 1];
    int32_t* dst = ent + off[g];
    // item q = 64 k + lane of the batch at c0
    int32_t v[kExpandPer];
#pragma unroll
    for (int k = 0; k < kExpandPer; ++k) {
        const int64_t ii = i0 + 64 * k + lane;
        v[k] = ii < i1 ? items[ii] : INT32_MIN;
    }
    for (int64_t c0 = i0; c0 < i1; c0 += kExpandItems) {
        // every lane loads a range (a cell item or an empty place that of
        // cell 0, unused), so that no branch separates the batch's loads
        int32_t rf[kExpandPer], rc[kExpandPer], vn[kExpandPer], first[kExpandPer], n[kExpandPer];
#pragma unroll
        for (int k = 0; k < kExpandPer; ++k) {
            const NodeRange& r = rng[v[k] >= 0 ? v[k] : 0];
            rf[k] = r.first;
            rc[k] = r.count;
        }
#pragma unroll
        for (int k = 0; k < kExpandPer; ++k) {
            const int64_t ii = c0 + kExpandItems + 64 * k + lane;
            vn[k] = ii < i1 ? items[ii] : INT32_MIN;
        }
#pragma unroll
        for (int k = 0; k < kExpandPer; ++k) {
            first[k] = v[k] >= 0 ? rf[k] : v[k];
            n[k] = v[k] >= 0 ? rc[k] : (v[k] == INT32_MIN ? 0 : 1);
        }
        uint64_t leafmask[kExpandPer];
        int carry = 0;
        int incl[kExpandPer];
#pragma unroll
        for (int k = 0; k < kExpandPer; ++k) {
            int x = n[k];
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int u = __shfl_up(x, o, 64);
                if (lane >= o) x += u;
            }
            incl[k] = x + carry;
            carry += __shfl(x, 63, 64);
            leafmask[k] = __ballot(v[k] >= 0 && n[k] > 0);
        }
        const int total = carry;
        if (total <= kExpandBuf) {
            // a leaf's entries are first, first + 1, ...; a cell's only
            // entry is its code
#pragma unroll
            for (int k = 0; k < kExpandPer; ++k) {
                const int b = incl[k] - n[k];
                if (v[k] >= 0) {
                    for (int q = 0; q < n[k]; ++q) s_ent[b + q] = first[k] + q;
                } else if (n[k] > 0) {
                    s_ent[b] = first[k];
                }
            }
            __syncthreads();
            for (int k = lane; k < total; k += 64) dst[k] = s_ent[k];
            __syncthreads();
        } else {
#pragma unroll
            for (int k = 0; k < kExpandPer; ++k) {
                s_end[64 * k + lane] = incl[k];
                s_first[64 * k + lane] = v[k] >= 0 ? first[k] - (incl[k] - n[k]) : first[k];
            }
            __syncthreads();
            for (int e = lane; e < total; e += 64) {
                // first item whose end exceeds e
                int lo = 0;
#pragma unroll
                for (int step = kExpandItems / 2; step >= 1; step >>= 1)
                    if (s_end[lo + step - 1] <= e) lo += step;
                const int32_t f = s_first[lo];
                dst[e] = ((leafmask[lo >> 6] >> (lo & 63)) & 1ull) ? f + e : f;
            }
            __syncthreads();
        }
        dst += total;
#pragma unroll
        for (int k = 0; k < kExpandPer; ++k) v[k] = vn[k];
    }
}

constexpr int kGroupsPerThread = 1;

}  // namespace

void build_lists(const Tree& t, Lists& l, hipStream_t st) {
    const int64_t ng = t.n_groups;
    const double rc2 = l.r_cut * l.r_cut;
    const double th2 = l.theta * l.theta;
    l.n_groups = ng;
    l.off.alloc(ng + 1, st);
    DevBuf<int64_t> icnt(ng + 1, st);
    int32_t cells[kLevels];
    for (int L = 0; L < kLevels; ++L) cells[L] = t.level_off[L + 1] - t.level_off[L];
    const bool waves = ng > 0 && t.srec.get() && wave_walk(t.n, ng, cells, t.max_level, l.r_cut, l.theta);
    const int64_t slot_items = waves && ng <= kWideGroups ? kWideSlot : kSlot;
    DevBuf<int32_t> slots(ng > 0 ? ng * slot_items : 1, st);
    DevBuf<unsigned long long> totals(4 * kTotals + 1, st);   // the rows, and whether the waves gave up
    const int B = kListThreads;
    constexpr int G = kGroupsPerThread;
    const int64_t nthreads = (ng + G - 1) / G;
    const dim3 grid(grid_for(nthreads, B, 1 << 30)), block(B);
    const bool com = l.mac == SRF_MAC_COM;
    // the walk for this tree: geometric or refitted cells, either criterion
    auto walk = [&](auto kernel, int64_t* cnt, int64_t* ic, unsigned long long* tot, const int64_t* ioff,
                    int32_t* out) {
        hipLaunchKernelGGL(kernel, grid, block, 0, st, ng, t.glo.get(), t.ghi.get(), t.gcount.get(), t.pack.get(),
                           t.range.get(), t.nX.get(), t.nY.get(), t.nZ.get(), t.rpack.get(), t.n_nodes,
                           rc2, th2, cnt, ic, tot, ioff, out);
    };
    auto walk_all = [&](auto write, int64_t* cnt, int64_t* ic, unsigned long long* tot, const int64_t* ioff,
                        int32_t* out) {
        constexpr bool W = decltype(write)::value;
        if (t.refit) {
            if (com) walk(k_lists<G, W, true, true>, cnt, ic, tot, ioff, out);
            else walk(k_lists<G, W, false, true>, cnt, ic, tot, ioff, out);
        } else {
            if (com) walk(k_lists<G, W, true, false>, cnt, ic, tot, ioff, out);
            else walk(k_lists<G, W, false, false>, cnt, ic, tot, ioff, out);
        }
    };
    auto wave_walk = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)ng), dim3(64), 0, st, ng, t.glo.get(), t.ghi.get(), t.gcount.get(),
                           t.srec.get(), t.spre.get(), t.nX.get(), t.nY.get(), t.nZ.get(), t.rpack.get(), rc2, th2,
                           l.off.get(), icnt.get(), totals.get(), slots.get(), slot_items);
    };
    // sizes and items: by waves, and by threads when the tree is past the
    // waves' range or some group's list does not fit a wave's buffer
    HostSlot slot(st);
    const unsigned long long* h = nullptr;
    auto count = [&](bool by_waves) {
        fill_u64(totals.get(), 0ull, 4 * kTotals + 1, st);
        if (!by_waves)
            walk_all(std::false_type{}, l.off.get(), icnt.get(), totals.get(), (const int64_t*)nullptr, slots.get());
        else if (t.refit)
            com ? wave_walk(k_walk<true, true>) : wave_walk(k_walk<false, true>);
        else
            com ? wave_walk(k_walk<true, false>) : wave_walk(k_walk<false, false>);
        SRF_HIP(hipGetLastError());
        const bool one = ng <= kScanGroups;
        if (!one) exclusive_scan_i64(l.off.get(), ng, true, st);
        hipLaunchKernelGGL(k_list_totals, dim3(1), dim3(kScanBlock), 0, st, one ? ng : 0, l.off.get(), totals.get(),
                           slot.device<unsigned long long>());
        SRF_HIP(hipGetLastError());
        h = slot.wait<unsigned long long>();
    };
    count(waves);
    int64_t slot_now = slot_items;
    if (waves && h[3] >= kOverflow) {
        count(false);
        slot_now = kSlot;
    }
    l.n_particle_entries = (int64_t)h[0];
    l.n_node_entries = (int64_t)h[1];
    l.n_entries = (int64_t)(h[0] + h[1]);
    l.interactions = (int64_t)h[2];
    l.ent.alloc(l.n_entries > 0 ? l.n_entries : 1, st);
    if (ng == 0) return;
    if (h[3] == 0 || slot_now == kWideSlot) {
        // every group's items fit its slot
        if (h[3] != 0) {
            hipLaunchKernelGGL(k_sort_wide, dim3((unsigned)ng), dim3(64), 0, st, icnt.get(), slots.get());
            SRF_HIP(hipGetLastError());
        }
        hipLaunchKernelGGL(k_expand, dim3((unsigned)ng), dim3(64), 0, st, ng, slot_now, icnt.get(),
                           (const int64_t*)nullptr, slots.get(), t.range.get(), l.off.get(), l.ent.get());
        SRF_HIP(hipGetLastError());
        return;
    }
    // some group has more items than a slot holds: walk again and store
    // every group's items compactly
    slots.reset();
    exclusive_scan_i64(icnt.get(), ng, true, st);
    int64_t n_items = 0;
    SRF_HIP(hipMemcpyAsync(&n_items, icnt.get() + ng, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    SRF_HIP(hipStreamSynchronize(st));
    DevBuf<int32_t> items(n_items > 0 ? n_items : 1, st);
    walk_all(std::true_type{}, (int64_t*)nullptr, (int64_t*)nullptr, (unsigned long long*)nullptr,
             (const int64_t*)icnt.get(), items.get());
    SRF_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_expand, dim3((unsigned)ng), dim3(64), 0, st, ng, (int64_t)0, (const int64_t*)nullptr,
                       icnt.get(), items.get(), t.range.get(), l.off.get(), l.ent.get());
    SRF_HIP(hipGetLastError());
}

}  // namespace srf
