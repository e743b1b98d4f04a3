// Long-range (PM) half of the TreePM force split on one GPU (Sec. 2 split,
// PM steps of Sec. 2.2, "Relay Mesh Method"), in FP64 on a periodic n^3 mesh with points at
// x = i/n:
//   1. TSC assignment of the sorted particles to 27 mesh points each,
//   2. 3-D FFT (Stockham, one pass per axis, lines staged in LDS),
//   3. multiplication by the Green's function
//        -4 pi G S(k)^2 / (k^2 W(k)^2),  S(k) = 12 (2 - 2 cos u - u sin u)/u^4,
//        u = |k| r_cut / 2 (the S2 cloud of the split),
//        W(k) = prod_axes sinc(k_a / 2n)^3 (the TSC window, deconvolved for
//        assignment and interpolation), zero at k = 0,
//   4. inverse FFT, 5. accelerations on the mesh by fourth-order central
//   differences, 6. TSC interpolation back to the particles.
#include <cmath>

#include "common.h"

namespace srf {
namespace {

// TSC stencil along one axis: nearest mesh point i0 = floor(u + 1/2) and
// weights of i0-1, i0, i0+1 for u = x n.
struct Tsc {
    int i0;
    double w[3];
};

__device__ __forceinline__ Tsc tsc(double x, int n) {
    const double u = x * n;
    const double c = floor(u + 0.5);
    const double d = u - c;
    Tsc t;
    t.i0 = (int)c;
    t.w[0] = 0.5 * (0.5 - d) * (0.5 - d);
    t.w[1] = 0.75 - d * d;
    t.w[2] = 0.5 * (0.5 + d) * (0.5 + d);
    return t;
}

__device__ __forceinline__ int wrap_i(int i, int n) { return i & (n - 1); }   // n is a power of two

// TSC weights of one coordinate u = x n on the four mesh points c - 1 .. c + 2,
// c = floor(u): those of tsc() on the three points about floor(u + 1/2), which
// is c or c + 1, and zero on the fourth.
__device__ __forceinline__ int tsc4(double u, double (&w)[4]) {
    const double c = floor(u), i0 = floor(u + 0.5);
    const double d = u - i0;
    const double a = 0.5 * (0.5 - d) * (0.5 - d), b = 0.75 - d * d, e = 0.5 * (0.5 + d) * (0.5 + d);
    const bool up = i0 > c;
    w[0] = up ? 0.0 : a;
    w[1] = up ? a : b;
    w[2] = up ? b : e;
    w[3] = up ? e : 0.0;
    return (int)c;
}

// The box of mesh points of a run of consecutive particles: wave w of a
// workgroup finds that of the w-th part of the workgroup's particles, and the
// workgroup then takes the parts in pieces, as many at a time as have a
// common box of at most `most` points.  (The Morton order jumps at the faces
// of its cubes: one box for all of them would often be too large.)
struct MeshBox {
    int lo[3], hi[3];
    __device__ __forceinline__ int64_t points(int reach) const {
        return (int64_t)(hi[0] - lo[0] + reach) * (hi[1] - lo[1] + reach) * (hi[2] - lo[2] + reach);
    }
};

// `shift`: 0 for the cells floor(u), 1/2 for the nearest points.
__device__ __forceinline__ MeshBox wave_box(int64_t s0, int64_t s1, const double* __restrict__ px,
                                            const double* __restrict__ py, const double* __restrict__ pz, int n,
                                            double shift) {
    MeshBox b;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        b.lo[a] = INT32_MAX;
        b.hi[a] = INT32_MIN;
    }
    for (int64_t s = s0 + (threadIdx.x & 63); s < s1; s += 64) {
        const double u[3] = {px[s] * n, py[s] * n, pz[s] * n};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int c = (int)floor(u[a] + shift);
            b.lo[a] = min(b.lo[a], c);
            b.hi[a] = max(b.hi[a], c);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
        for (int o = 32; o >= 1; o >>= 1) {
            b.lo[a] = min(b.lo[a], __shfl_xor(b.lo[a], o, 64));
            b.hi[a] = max(b.hi[a], __shfl_xor(b.hi[a], o, 64));
        }
    return b;
}

// The piece from part `part` on: returns its end and its box (one of more
// than `most` points where the parts do not fit).
__device__ __forceinline__ int next_piece(const MeshBox* parts, int part, int n_parts, int reach, int most,
                                          MeshBox& box) {
    box = parts[part];
    int end = part + 1;
    if (box.points(reach) > most) {   // too large by itself: with the parts after it that are, too
        while (end < n_parts && parts[end].points(reach) > most) ++end;
        return end;
    }
    for (; end < n_parts; ++end) {
        MeshBox u;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            u.lo[a] = min(box.lo[a], parts[end].lo[a]);
            u.hi[a] = max(box.hi[a], parts[end].hi[a]);
        }
        if (u.points(reach) > most) break;
        box = u;
    }
    return end;
}

// 1. density (mass per unit volume) on the mesh.
// The particles come in Morton order, so those of one mesh cell (a cube of the
// octree, n being a power of two) follow each other, and together touch the
// 4 x 4 x 4 points about the cell.  Their contributions are a contraction over
// the particles p of the run,
//   rho[a][b][c] = sum_p (m wx[a] wy[b])_p wz[c]_p,
// which a wave takes four particles at a time with the FP64 matrix
// instruction of four 4 x 4 x 4 blocks (block a, row b, column c, depth p),
// from weights its lanes have computed, one particle each, and left in LDS.
// A lane ends with one point's sum.  A workgroup takes kChunk particles in
// pieces whose box of mesh points fits kBoxMax points, adds the runs' sums to
// the box in LDS and the box to the mesh with one global atomic per touched
// point; where even one part's box does not fit, or the particles are few and
// spread, the runs' sums go to the mesh directly.
//   With each particle's 27 products added to the box by LDS atomics, which
// serialise over the particles of a cell, and one box per workgroup, which half
// the workgroups' particles did not fit, the kernel took 1.97 ms for 2^24
// particles on 128^3 points; with the matrix instruction 1.45 ms, and with the
// pieces 0.42 ms (58 us for 2^21 on 64^3, from 298).  Reading the particles
// takes 0.1 ms; the rest is the runs' sums, one LDS atomic a lane each.
constexpr int kAssignWaves = 8;
constexpr int kAssignThreads = 64 * kAssignWaves;
// Particles per workgroup: kChunk, halved down to 64 a wave while that leaves
// fewer than kBlocks workgroups (50653 particles on 32^3: the call 215 us with
// 4096 a workgroup, 106 us with 512).
constexpr int kChunk = 4096;
constexpr int kBlocks = 512;
// With fewer than kFewToAssign particles half the CUs or more are idle, and what
// counts is the time of one workgroup: up to eight boxes cleared and written
// one after the other, where particles that moved since their tree was made
// spread the parts.  A workgroup then takes a box only if one holds all its
// particles.  The call, with the pieces' boxes and so: uniform, moved by 3 cells
// of the mesh, 10000 on 16^3 196 us and 118, 40000 on 32^3 209 and 127; in mesh
// order 127 and 112; 65000 moved on 32^3 209 and 137.  Clusters keep their box:
// 65000 with a spread of 0.01 on 16^3 90 us, 106 without any.  From 80000 on,
// boxes gain or cost little in order (200000 on 64^3 157 us, 204 without).
constexpr int64_t kFewToAssign = 1 << 16;
constexpr int kBoxMax = 3328;   // FP64 values in LDS (two workgroups per CU)
constexpr int kWtRow = 68;      // 64 particles, padded: a block's reads fall on distinct banks

__global__ __launch_bounds__(kAssignThreads) void k_tsc_assign(int64_t np, const double* __restrict__ px,
                                                               const double* __restrict__ py,
                                                               const double* __restrict__ pz,
                                                               const double* __restrict__ pm, int n, int chunk,
                                                               int most, double* __restrict__ mesh) {
    __shared__ double sum_at[kBoxMax];
    __shared__ MeshBox parts[kAssignWaves];
    __shared__ double wts[kAssignWaves][3][4][kWtRow];   // per wave: axis (x times the mass), point, particle
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t c0 = (int64_t)blockIdx.x * chunk, c1 = c0 + chunk < np ? c0 + chunk : np;
    const int per = chunk / kAssignWaves;   // particles per part
    const double q = (double)n * n * n;
    const int64_t nn = n;
    const int64_t p0 = c0 + wave * per;
    if (p0 < c1) {
        const MeshBox b = wave_box(p0, p0 + per < c1 ? p0 + per : c1, px, py, pz, n, 0.0);
        if (lane == 0) parts[wave] = b;
    }
    const int n_parts = (int)((c1 - c0 + per - 1) / per);
    // this lane's place in the matrix blocks: depth, block, row or column
    const int kp = lane >> 4, ka = (lane >> 2) & 3, kb = lane & 3;
    const double* wx = wts[wave][0][ka] + kp;
    const double* wy = wts[wave][1][kb] + kp;
    const double* wz = wts[wave][2][kb] + kp;
    __syncthreads();
    for (int part = 0; part < n_parts;) {
        MeshBox box;
        int end = next_piece(parts, part, n_parts, 4, most, box);
        const bool spread = np < kFewToAssign && end < n_parts;   // seen at the first piece
        if (spread) end = n_parts;
        const int64_t s0 = c0 + part * per;
        const int cnt = (int)((c0 + end * per < c1 ? c0 + end * per : c1) - s0);
        part = end;
        const int bd1 = box.hi[1] - box.lo[1] + 4, bd2 = box.hi[2] - box.lo[2] + 4;
        const int64_t vol = box.points(4);
        const bool boxed = vol <= most && !spread;
        double* my_sum = sum_at + (ka * bd1 + kp) * bd2 + kb;
        if (boxed) {
            __syncthreads();   // the last piece's box has been read
            for (int k = tid; k < vol; k += kAssignThreads) sum_at[k] = 0.0;
            __syncthreads();
        }
        for (int k0 = 64 * wave; k0 < cnt; k0 += kAssignThreads) {
            const bool on = k0 + lane < cnt;
            const int64_t s = s0 + k0 + (on ? lane : 0);
            double w[4];
            const double mq = on ? pm[s] * q : 0.0;
            const int cx = tsc4(px[s] * n, w);
#pragma unroll
            for (int j = 0; j < 4; ++j) wts[wave][0][j][lane] = mq * w[j];
            const int cy = tsc4(py[s] * n, w);
#pragma unroll
            for (int j = 0; j < 4; ++j) wts[wave][1][j][lane] = w[j];
            const int cz = tsc4(pz[s] * n, w);
#pragma unroll
            for (int j = 0; j < 4; ++j) wts[wave][2][j][lane] = w[j];
            const int cell = (cx << 20) | (cy << 10) | cz;   // n <= 1024
            // lanes that start a run of one cell
            const int before = __shfl_up(cell, 1, 64);
            const int m = cnt - k0 < 64 ? cnt - k0 : 64;
            uint64_t starts = __ballot(lane < m && (lane == 0 || cell != before));
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            while (starts) {
                const int r0 = __ffsll((unsigned long long)starts) - 1;
                starts &= starts - 1;
                const int r1 = starts ? __ffsll((unsigned long long)starts) - 1 : m;
                const int rc = __builtin_amdgcn_readlane(cell, r0);
                const int rx = rc >> 20, ry = (rc >> 10) & 1023, rz = rc & 1023;
                double sum = 0.0;
                for (int p0 = r0; p0 < r1; p0 += 4) {
                    const bool in = kp < r1 - p0;
                    const double A = wx[p0] * wy[p0];
                    sum = __builtin_amdgcn_mfma_f64_4x4x4f64(in ? A : 0.0, in ? wz[p0] : 0.0, sum, 0, 0, 0);
                }
                // sum of point row kp, block ka, column kb of the 4 x 4 x 4 about the cell
                if (boxed) {
                    const int at = ((rx - box.lo[0]) * bd1 + (ry - box.lo[1])) * bd2 + (rz - box.lo[2]);
                    atomicAdd(my_sum + at, sum);
                } else if (sum != 0.0) {
                    const int64_t g = ((int64_t)wrap_i(rx - 1 + ka, n) * nn + wrap_i(ry - 1 + kp, n)) * nn +
                                      wrap_i(rz - 1 + kb, n);
                    unsafeAtomicAdd(mesh + g, sum);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        if (!boxed) continue;
        __syncthreads();
        for (int k = tid; k < vol; k += kAssignThreads) {
            const double v = sum_at[k];
            if (v == 0.0) continue;
            const int iz = k % bd2, iy = (k / bd2) % bd1, ix = k / (bd2 * bd1);
            const int64_t g = ((int64_t)wrap_i(box.lo[0] - 1 + ix, n) * nn + wrap_i(box.lo[1] - 1 + iy, n)) * nn +
                              wrap_i(box.lo[2] - 1 + iz, n);
            unsafeAtomicAdd(mesh + g, v);
        }
    }
}

__device__ __forceinline__ double wavenumber(int i, int n) {
    return 2.0 * M_PI * (double)(i < n / 2 ? i : i - n);
}

__device__ __forceinline__ double sinc(double v) { return v == 0.0 ? 1.0 : sin(v) / v; }

// Transform of the unit-mass S2 cloud at u = k r_cut / 2; Taylor series
// below u = 1/2, where the closed form's O(1) terms cancel to O(u^4).
__device__ __forceinline__ double s2_shape(double u) {
    if (u < 0.5) {
        const double v = u * u;
        return 1.0 + v * (-1.0 / 15.0 + v * (1.0 / 560.0 + v * (-1.0 / 37800.0 + v / 3991680.0)));
    }
    double s, c;
    sincos(u, &s, &c);
    return 12.0 * (2.0 - 2.0 * c - u * s) / (u * u * u * u);
}

// 2. and 4. FFT passes: length-n transforms of all n^2 lines along one axis.
// A workgroup stages kBn / n lines in LDS (consecutive in the contiguous mesh
// index, so that loads and stores are coalesced), runs radix-4 Stockham stages
// there (one of radix 2 first where log2(n) is odd; half the stages, LDS
// traffic and barriers of radix 2 alone), and writes back in place.
// axis 2 (contiguous): line L starts at L n, element stride 1;
// axis 1: line L = (x, z) starts at x n^2 + z, stride n;
// axis 0: line L = (y, z) starts at L, stride n^2.
// The first pass (axis 2) reads the real density.  The pass over axis 0 is
// the middle one: it transforms, multiplies the spectrum by the Green's
// function / n^3 (step 3; the inverse FFT is unnormalised) and transforms
// back, which saves a pass and the Green's function's own over the mesh.
// Each workgroup makes its own table of twiddles, so that no launch is
// needed for them.
//   Two buffers of 32 KB allowed two workgroups a CU, and the passes waited
// for memory: 31-35 us each at 128^3 in radix 2 or 4, 18-19 us in place (35 us
// the middle one), 109 us in all against 228 for six passes, the Green's
// function and the table of twiddles.
constexpr int kFftThreads = 256;
constexpr int kBn = 2048;   // complex values staged per workgroup

enum FftPass { kForward, kForwardReal, kInverse, kGreen };

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// The stages over the lines in buf, in place: a thread holds its butterflies'
// values in registers while the workgroup has read all and written none, so
// that a workgroup needs one buffer and four fit a CU.  tw[j] =
// exp(-2 pi i j / n) for j < 3 n / 4.
template <bool INV>
__device__ void fft_stages(double2* buf, int n, int log2n, const double2* tw) {
    int m = 1;
    if (log2n & 1) {
        constexpr int kPer = kBn / 2 / kFftThreads;
        const int log2h = log2n - 1, half = n / 2;
        double2 u[kPer], v[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int t = threadIdx.x + i * kFftThreads;
            const double2* p = buf + (t >> log2h) * n + (t & (half - 1));
            u[i] = p[0];
            v[i] = p[half];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int t = threadIdx.x + i * kFftThreads;
            double2* o = buf + (t >> log2h) * n + 2 * (t & (half - 1));
            o[0] = make_double2(u[i].x + v[i].x, u[i].y + v[i].y);
            o[1] = make_double2(u[i].x - v[i].x, u[i].y - v[i].y);
        }
        __syncthreads();
        m = 2;
    }
    constexpr int kPer = kBn / 4 / kFftThreads;
    const int log2q = log2n - 2, quarter = n / 4;
    for (; m < n; m *= 4) {
        const int step = quarter / m;
        double2 x[kPer][4];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int t = threadIdx.x + i * kFftThreads;
            const double2* p = buf + (t >> log2q) * n + (t & (quarter - 1));
#pragma unroll
            for (int r = 0; r < 4; ++r) x[i][r] = p[r * quarter];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int t = threadIdx.x + i * kFftThreads;
            const int q = t & (quarter - 1), k = q & (m - 1);
            double2 w1 = tw[k * step], w2 = tw[2 * k * step], w3 = tw[3 * k * step];
            if (INV) {
                w1.y = -w1.y;
                w2.y = -w2.y;
                w3.y = -w3.y;
            }
            const double2 x0 = x[i][0], x1 = cmul(x[i][1], w1), x2 = cmul(x[i][2], w2), x3 = cmul(x[i][3], w3);
            const double2 a = make_double2(x0.x + x2.x, x0.y + x2.y), c = make_double2(x0.x - x2.x, x0.y - x2.y);
            const double2 e = make_double2(x1.x + x3.x, x1.y + x3.y), f = make_double2(x1.x - x3.x, x1.y - x3.y);
            // -i f forward, +i f inverse
            const double2 g = INV ? make_double2(-f.y, f.x) : make_double2(f.y, -f.x);
            double2* o = buf + (t >> log2q) * n + 4 * q - 3 * k;
            o[0] = make_double2(a.x + e.x, a.y + e.y);
            o[m] = make_double2(c.x + g.x, c.y + g.y);
            o[2 * m] = make_double2(a.x - e.x, a.y - e.y);
            o[3 * m] = make_double2(c.x - g.x, c.y - g.y);
        }
        __syncthreads();
    }
}

// LDS: the lines, the twiddles, and for kGreen the window sinc(k_i / 2n).
inline size_t fft_shared_bytes(int n) { return sizeof(double2) * (kBn + n / 4 * 3) + sizeof(double) * n; }

template <FftPass PASS>
__global__ __launch_bounds__(kFftThreads) void k_fft_axis(double2* __restrict__ mesh,
                                                           const double* __restrict__ density, int n, int log2n,
                                                           int axis, double r_cut, double G) {
    extern __shared__ double2 buf[];
    double2* tw = buf + kBn;
    double* win = reinterpret_cast<double*>(tw + n / 4 * 3);
    const int log2b = 31 - __clz(kBn) - log2n, B = 1 << log2b;   // lines per workgroup
    const int64_t nn = n;
    const int64_t L0 = (int64_t)blockIdx.x * B;
    // line b of the workgroup occupies [b n, b n + n) in LDS; element idx of
    // the workgroup is read and written by the thread idx mod kFftThreads
    auto place = [&](int idx, int& b, int64_t& at) -> int {
        int j;
        if (axis == 2) {
            b = idx >> log2n;
            j = idx & (n - 1);
        } else {
            j = idx >> log2b;
            b = idx & (B - 1);
        }
        const int64_t L = L0 + b;
        at = axis == 2 ? L * nn + j : (axis == 1 ? (L >> log2n) * nn * nn + (L & (n - 1)) + j * nn : L + j * nn * nn);
        return j;
    };
    for (int idx = threadIdx.x; idx < kBn; idx += kFftThreads) {
        int b;
        int64_t at;
        const int j = place(idx, b, at);
        buf[b * n + j] = PASS == kForwardReal ? make_double2(density[at], 0.0) : mesh[at];
    }
    for (int j = threadIdx.x; j < n / 4 * 3; j += kFftThreads) {
        double s, c;
        sincospi(-2.0 * j / n, &s, &c);
        tw[j] = make_double2(c, s);
    }
    if (PASS == kGreen)
        for (int j = threadIdx.x; j < n; j += kFftThreads) win[j] = sinc(wavenumber(j, n) * (0.5 / n));
    __syncthreads();
    fft_stages<PASS == kInverse>(buf, n, log2n, tw);
    if (PASS == kGreen) {
        const double scale = -4.0 * M_PI * G / ((double)n * n * n);
        for (int idx = threadIdx.x; idx < kBn; idx += kFftThreads) {
            const int b = idx >> log2n, ix = idx & (n - 1);
            const int64_t L = L0 + b;
            const int iy = (int)(L >> log2n), iz = (int)(L & (n - 1));
            const double kx = wavenumber(ix, n), ky = wavenumber(iy, n), kz = wavenumber(iz, n);
            const double k2 = kx * kx + ky * ky + kz * kz;
            const double w1 = win[ix] * win[iy] * win[iz], W = w1 * w1 * w1;
            const double S = s2_shape(sqrt(k2) * r_cut * 0.5);
            const double g = k2 > 0.0 ? scale * S * S / (k2 * W * W) : 0.0;
            buf[idx] = make_double2(buf[idx].x * g, buf[idx].y * g);
        }
        __syncthreads();
        fft_stages<true>(buf, n, log2n, tw);
    }
    for (int idx = threadIdx.x; idx < kBn; idx += kFftThreads) {
        int b;
        int64_t at;
        const int j = place(idx, b, at);
        mesh[at] = buf[b * n + j];
    }
}

// 5. a = -grad phi, fourth-order central differences, from the real parts;
// the three components of a mesh point side by side (x, y, z, unused), so
// that the interpolation reads one 32-byte record per stencil point
__global__ void k_fd4(const double2* __restrict__ phi, int n, double4* __restrict__ acc) {
    const int64_t nn = n;
    const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (idx >= nn * nn * nn) return;
    const int iz = (int)(idx % nn), iy = (int)((idx / nn) % nn), ix = (int)(idx / (nn * nn));
    auto at = [&](int x, int y, int z) -> double {
        x = (x + n) % n;
        y = (y + n) % n;
        z = (z + n) % n;
        return phi[((int64_t)x * nn + y) * nn + z].x;
    };
    const double c1 = 2.0 / 3.0 * n, c2 = 1.0 / 12.0 * n;
    double4 a;
    a.x = -(c1 * (at(ix + 1, iy, iz) - at(ix - 1, iy, iz)) - c2 * (at(ix + 2, iy, iz) - at(ix - 2, iy, iz)));
    a.y = -(c1 * (at(ix, iy + 1, iz) - at(ix, iy - 1, iz)) - c2 * (at(ix, iy + 2, iz) - at(ix, iy - 2, iz)));
    a.z = -(c1 * (at(ix, iy, iz + 1) - at(ix, iy, iz - 1)) - c2 * (at(ix, iy, iz + 2) - at(ix, iy, iz - 2)));
    a.w = 0.0;
    acc[idx] = a;
}

// 6. TSC interpolation at the sorted particles; output in input order.  A
// workgroup takes kInterp consecutive particles, in pieces as the assignment
// does, and copies the box of mesh points they touch to LDS, when it fits, one
// array per component, so that a
// particle's 27 records come from there and not through the vector cache,
// whose rate bound the kernel: 0.96 -> 0.49 ms for 2^24 particles on 128^3
// points, 125 -> 67 us for 2^21 on 64^3.
constexpr int kInterpThreads = 256;
constexpr int kInterp = 2048;      // particles per workgroup, halved for few particles as the assignment's
constexpr int kInterpBox = 1664;   // points: 39 KB of LDS, four workgroups per CU

__global__ __launch_bounds__(kInterpThreads) void k_tsc_interp(int64_t np, const double* __restrict__ px,
                                                               const double* __restrict__ py,
                                                               const double* __restrict__ pz,
                                                               const int32_t* __restrict__ perm, int n, int chunk,
                                                               const double4* __restrict__ acc,
                                                               double* __restrict__ ax, double* __restrict__ ay,
                                                               double* __restrict__ az, int64_t os) {
    __shared__ double fld[3][kInterpBox];
    __shared__ MeshBox parts[kInterpThreads / 64];
    const int tid = threadIdx.x, wave = tid >> 6;
    const int64_t c0 = (int64_t)blockIdx.x * chunk, c1 = c0 + chunk < np ? c0 + chunk : np;
    const int per = chunk / (kInterpThreads / 64);
    const int64_t nn = n;
    const int64_t p0 = c0 + wave * per;
    if (p0 < c1) {
        const MeshBox b = wave_box(p0, p0 + per < c1 ? p0 + per : c1, px, py, pz, n, 0.5);
        if ((tid & 63) == 0) parts[wave] = b;
    }
    const int n_parts = (int)((c1 - c0 + per - 1) / per);
    __syncthreads();
    for (int part = 0; part < n_parts;) {
        MeshBox box;
        const int end = next_piece(parts, part, n_parts, 3, kInterpBox, box);
        const int64_t s0 = c0 + part * per;
        const int cnt = (int)((c0 + end * per < c1 ? c0 + end * per : c1) - s0);
        part = end;
        const int bd1 = box.hi[1] - box.lo[1] + 3, bd2 = box.hi[2] - box.lo[2] + 3;
        const int64_t vol = box.points(3);
        const bool boxed = vol <= kInterpBox;
        if (boxed) {
            __syncthreads();   // the last piece's box has been read
            for (int k = tid; k < vol; k += kInterpThreads) {
                const int iz = k % bd2, iy = (k / bd2) % bd1, ix = k / (bd2 * bd1);
                const int64_t g = ((int64_t)wrap_i(box.lo[0] - 1 + ix, n) * nn + wrap_i(box.lo[1] - 1 + iy, n)) * nn +
                                  wrap_i(box.lo[2] - 1 + iz, n);
                const double4 m = acc[g];
                fld[0][k] = m.x;
                fld[1][k] = m.y;
                fld[2][k] = m.z;
            }
            __syncthreads();
        }
        for (int k = tid; k < cnt; k += kInterpThreads) {
            const int64_t s = s0 + k;
            const Tsc a = tsc(px[s], n), b = tsc(py[s], n), c = tsc(pz[s], n);
            double fx = 0, fy = 0, fz = 0;
            if (boxed) {
                const int at = ((a.i0 - box.lo[0]) * bd1 + (b.i0 - box.lo[1])) * bd2 + (c.i0 - box.lo[2]);
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        const double wij = a.w[i] * b.w[j];
                        const int row = at + (i * bd1 + j) * bd2;
#pragma unroll
                        for (int e = 0; e < 3; ++e) {
                            const double w = wij * c.w[e];
                            fx += w * fld[0][row + e];
                            fy += w * fld[1][row + e];
                            fz += w * fld[2][row + e];
                        }
                    }
            } else {
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        const double wij = a.w[i] * b.w[j];
                        const int64_t row = ((int64_t)wrap_i(a.i0 - 1 + i, n) * nn + wrap_i(b.i0 - 1 + j, n)) * nn;
#pragma unroll
                        for (int e = 0; e < 3; ++e) {
                            const double w = wij * c.w[e];
                            const double4 m = acc[row + wrap_i(c.i0 - 1 + e, n)];
                            fx += w * m.x;
                            fy += w * m.y;
                            fz += w * m.z;
                        }
                    }
            }
            const int64_t o = (int64_t)perm[s] * os;
            ax[o] = fx;
            ay[o] = fy;
            az[o] = fz;
        }
    }
}

}  // namespace

void launch_pm(const Tree& t, double G, double r_cut, int n, double* ax, double* ay, double* az, int64_t os,
               hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
    const int64_t np = t.n;
    const int64_t cells = (int64_t)n * n * n;
    DevBuf<double2> mesh(cells, st);
    DevBuf<double4> acc(cells, st);
    double* density = reinterpret_cast<double*>(acc.get());   // until the first FFT pass has read it
    if (ev0) SRF_HIP(hipEventRecord(ev0, st));
    fill_f64(density, 0.0, cells, st);
    auto blocks = [&](int chunk) { return (unsigned)((np + chunk - 1) / chunk); };
    int chunk = kChunk, ichunk = kInterp;
    while (chunk > kAssignThreads && blocks(chunk) < kBlocks) chunk /= 2;
    while (ichunk > kInterpThreads && blocks(ichunk) < 2 * kBlocks) ichunk /= 2;
    // with fewer than a particle to two points a box has more points than its
    // particles touch, and few particles fit one: no boxes then (30007
    // particles on 64^3: the call 120 us, with boxes 210; on 16^3 68 and 70)
    const int most = 2 * np < cells ? 0 : kBoxMax;
    hipLaunchKernelGGL(k_tsc_assign, dim3(blocks(chunk)), dim3(kAssignThreads), 0, st, np, t.px.get(), t.py.get(),
                       t.pz.get(), t.pm.get(), n, chunk, most, density);
    SRF_HIP(hipGetLastError());
    int log2n = 0;
    while ((1 << log2n) < n) ++log2n;
    auto pass = [&](auto kernel, int axis) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)(cells / kBn)), dim3(kFftThreads), fft_shared_bytes(n), st,
                           mesh.get(),
                           (const double*)density, n, log2n, axis, r_cut, G);
        SRF_HIP(hipGetLastError());
    };
    pass(k_fft_axis<kForwardReal>, 2);
    pass(k_fft_axis<kForward>, 1);
    pass(k_fft_axis<kGreen>, 0);
    pass(k_fft_axis<kInverse>, 1);
    pass(k_fft_axis<kInverse>, 2);
    hipLaunchKernelGGL(k_fd4, dim3(grid_for(cells, 256, 1 << 30)), dim3(256), 0, st, mesh.get(), n, acc.get());
    SRF_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_tsc_interp, dim3(blocks(ichunk)), dim3(kInterpThreads), 0, st, np, t.px.get(), t.py.get(),
                       t.pz.get(), t.perm.get(), n, ichunk, acc.get(), ax, ay, az, os);
    SRF_HIP(hipGetLastError());
    if (ev1) SRF_HIP(hipEventRecord(ev1, st));
}

}  // namespace srf
