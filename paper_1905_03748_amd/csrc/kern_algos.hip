// Device-resident iterative algorithms built on the operators: CGLS (FP64 inner products and
// residual recurrence, scalars kept in device memory so an iteration never waits on the host),
// OS-SART (SART with one angle per update when block = 1) and TV steepest descent.  Reductions use a fixed partition
// (DOT_BLOCKS contiguous ranges, fixed wave/block trees, fixed final sum), so results are bitwise
// repeatable regardless of what else shares the device.
#include <algorithm>
#include <cfloat>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <type_traits>
#include <utility>

#include "dev_common.hpp"

namespace ct {

namespace {

constexpr int DOT_BLOCKS = 1024;
constexpr int DOT_THREADS = 256;
constexpr int EW_THREADS = 256;

inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

inline unsigned ew_grid(int64_t n) {
    int64_t g = (n + EW_THREADS - 1) / EW_THREADS;
    if (g > 65536 * 16) g = 65536 * 16;
    if (g < 1) g = 1;
    return (unsigned)g;
}

template <typename T>
__global__ __launch_bounds__(DOT_THREADS) void k_dot_partial(const T *__restrict__ a, const T *__restrict__ b, int64_t n,
                                                             double *__restrict__ partials) {
    __shared__ double lds[DOT_THREADS / 64];
    const int64_t chunk = (n + gridDim.x - 1) / gridDim.x;
    const int64_t lo = (int64_t)blockIdx.x * chunk;
    const int64_t hi = lo + chunk < n ? lo + chunk : n;
    double s = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += blockDim.x) s += to_d(a[i]) * to_d(b[i]);
    s = block_sum(s, lds);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

__global__ __launch_bounds__(DOT_THREADS) void k_sum_partials(const double *__restrict__ partials, int n,
                                                              double *__restrict__ out) {
    __shared__ double lds[DOT_THREADS / 64];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) s += partials[i];
    s = block_sum(s, lds);
    if (threadIdx.x == 0) *out = s;
}

template <typename TS, typename TD>
__global__ void k_convert(const TS *__restrict__ s, TD *__restrict__ d, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        d[i] = from_d<TD>(to_d(s[i]));
}

// r (FP32) = b - r, b in its storage type
template <typename T>
__global__ void k_rsub_from(const T *__restrict__ b, float *__restrict__ r, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        r[i] = ldf(b, i) - r[i];
}

// y (storage type) += sign * scal[idx] * x (FP32)
template <typename T>
__global__ void k_axpy_mixed(T *__restrict__ y, const float *__restrict__ x, const double *__restrict__ scal, int idx,
                             float sign, int64_t n) {
    const float a = sign * (float)scal[idx];
    if (a == 0.0f) return;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = from_f<T>(fmaf(a, x[i], ldf(y, i)));
}

template <typename T>
__global__ void k_copy(const T *__restrict__ s, T *__restrict__ d, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        d[i] = s[i];
}

// y += sign * scal[idx] * x
template <typename T>
__global__ void k_axpy_s(T *__restrict__ y, const T *__restrict__ x, const double *__restrict__ scal, int idx,
                         float sign, int64_t n) {
    const float a = sign * (float)scal[idx];
    if (a == 0.0f) return;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = from_f<T>(fmaf(a, ldf(x, i), ldf(y, i)));
}

// p = s + scal[idx] * p
template <typename T>
__global__ void k_xpby_s(T *__restrict__ p, const T *__restrict__ s, const double *__restrict__ scal, int idx,
                         int64_t n) {
    const float bta = (float)scal[idx];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = from_f<T>(fmaf(bta, ldf(p, i), ldf(s, i)));
}

// CGLS scalar slots
enum { S_GAMMA = 0, S_DELTA = 1, S_ALPHA = 2, S_BETA = 3, S_RHO = 4, S_STOP = 5, S_TMP = 6, S_COUNT = 8 };

__global__ void k_cgls_start(double *scal, double *resid) {
    scal[S_STOP] = 0.0;
    scal[S_ALPHA] = 0.0;
    scal[S_BETA] = 0.0;
    if (resid) resid[0] = sqrt(fmax(scal[S_RHO], 0.0));
}

__global__ void k_cgls_alpha(double *scal, double *resid, int k) {
    const double delta = scal[S_DELTA];
    if (scal[S_STOP] != 0.0 || delta == 0.0) {
        scal[S_STOP] = 1.0;
        scal[S_ALPHA] = 0.0;
    } else {
        const double alpha = scal[S_GAMMA] / delta;
        scal[S_ALPHA] = alpha;
        scal[S_RHO] = scal[S_RHO] - alpha * scal[S_GAMMA];
    }
    if (resid) resid[k + 1] = sqrt(fmax(scal[S_RHO], 0.0));
}

__global__ void k_cgls_beta(double *scal) {
    const double gnew = scal[S_TMP];
    if (scal[S_STOP] != 0.0) {
        scal[S_BETA] = 0.0;
        return;
    }
    scal[S_BETA] = scal[S_GAMMA] != 0.0 ? gnew / scal[S_GAMMA] : 0.0;
    scal[S_GAMMA] = gnew;
}

// SART residual for one angle: r = (b - r) / chord where chord > thr, else 0 (b in its storage type)
template <typename TP>
__global__ void k_sart_resid(const TP *__restrict__ b, const float *__restrict__ chord, float *__restrict__ r,
                             float thr, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float c = chord[i];
        r[i] = c > thr ? (to_f(b[i]) - r[i]) / c : 0.0f;
    }
}

// The same residual written transposed, rT[u][v], through 32 x 32 LDS tiles; blockIdx.z is the
// angle within the subset (each array advances by one projection per angle)
template <typename TP>
__global__ __launch_bounds__(256) void k_sart_resid_t(const TP *__restrict__ b, const float *__restrict__ chord,
                                                      const float *__restrict__ r, float *__restrict__ rT, float thr,
                                                      int nu, int nv) {
    __shared__ float tile[32][33];
    const int u0 = blockIdx.x * 32, v0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int64_t po = (int64_t)blockIdx.z * nu * nv;
    b += po;
    chord += po;
    r += po;
    rT += po;
#pragma unroll
    for (int k = 0; k < 32; k += 8) {
        const int u = u0 + tx, v = v0 + ty + k;
        if (u < nu && v < nv) {
            const int64_t i = (int64_t)v * nu + u;
            const float c = chord[i];
            tile[ty + k][tx] = c > thr ? (to_f(b[i]) - r[i]) / c : 0.0f;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 32; k += 8) {
        const int v = v0 + tx, u = u0 + ty + k;
        if (u < nu && v < nv) rT[(int64_t)u * nv + v] = tile[tx][ty + k];
    }
}

// TV_eps gradient with forward differences, unit spacing, zero difference at the last index:
//   g = p_x(i - 1) - p_x + p_y(j - 1) - p_y + p_z(k - 1) - p_z,  p = D x / sqrt(|D x|^2 + eps).
// Slices kg0 .. kg0 + nk - 1 of the volume (nz slices in all); x holds slices from kx0 on (at least
// z - 1 .. z + 1 where they exist).  A whole resident volume has kx0 = kg0 = 0.
//
// A step needs ||g|| before it can move x, so it makes two passes, each forming g from x in registers:
// k_tv_norm sums g^2 (reads x), k_tv_apply writes x - a g to another array (reads x, writes it): 12 bytes
// of memory traffic per voxel and step, where a stored gradient took 24 (write g, read it for the norm,
// read g and x, write x).  Each thread walks a run of slices of one (i, j) column: a voxel's gradient reads
// seven positions of its own slice and three of the next, so the thread loads the seven positions of
// each slice once, a slice ahead of their use, and carries them up the column, with p_z of the slice below.
// Positions past an edge of the volume read the edge voxel, so their differences are zero without a test.
// The reciprocal square roots are the hardware's (1 ulp; a square root and a division each took about 25
// instructions, four pairs per voxel): s >= eps, so a normal eps keeps them from denormal arguments, and
// TINY serves an eps below FLT_MIN (and slices of 2^32 pixels, with 64-bit offsets).  Bound: HBM and the
// address unit (7 loads of 4.7 cycles per wave and slice) about evenly.
// Five steps at 512^3 (with the copy of the image): 5.85 -> 2.75 ms (2.90 before the loads ran ahead).
constexpr int TV_TY = 8;               // rows of a tile (waves of a block); a tile is 64 columns wide
constexpr int TV_THREADS = 64 * TV_TY;
struct TvPlane {
    float c, e, n, w, wn, s, se;  // (i, j), (i + 1, j), (i, j + 1), (i - 1, j), (i - 1, j + 1), (i, j - 1), (i + 1, j - 1)
};
struct TvArgs {
    int nx, ny, nz;
    float eps;
    int64_t kx0, kg0, nk;
    int zr;               // slices of a run
    unsigned bx, by, bz;  // tiles along each axis
    int by_xcd;           // an eighth of the tiles, in order, per XCD
};
// Tile t in launch order (workgroups are dealt to the 8 XCDs in turn) as its place in the image.
__device__ __forceinline__ unsigned tv_tile(const TvArgs &A, unsigned t) {
    const unsigned e = A.bx * A.by * A.bz / 8;
    return A.by_xcd && t < 8 * e ? (t % 8) * e + t / 8 : t;
}
template <bool TINY>
__device__ __forceinline__ float tv_rsqrt(float s) {
    return TINY ? 1.0f / sqrtf(s) : __builtin_amdgcn_rsqf(s);
}
// visit(offset in x, x, g) for every voxel of the thread's run in the tile
template <bool TINY, typename F>
__device__ __forceinline__ void tv_walk(const float *__restrict__ x, const TvArgs &A, unsigned t, F visit) {
    const unsigned tx = t % A.bx, ty = t / A.bx % A.by, tz = t / (A.bx * A.by);
    const int i = (int)tx * 64 + ((int)threadIdx.x & 63);
    const int j = (int)ty * TV_TY + ((int)threadIdx.x >> 6);
    if (i >= A.nx || j >= A.ny) return;
    const int64_t sz = (int64_t)A.nx * A.ny;
    // offsets of the seven positions in a slice (32-bit from a wave-uniform slice base)
    using O = typename std::conditional<TINY, int64_t, uint32_t>::type;
    const O oc = (O)j * A.nx + i, oe = oc + (i < A.nx - 1 ? 1 : 0), ow = oc - (i > 0 ? 1 : 0);
    const O up = j < A.ny - 1 ? A.nx : 0, dn = j > 0 ? A.nx : 0;
    const O on = oc + up, own = ow + up, os = oc - dn, ose = oe - dn;
    const int64_t r0 = (int64_t)tz * A.zr, r1 = min(r0 + (int64_t)A.zr, A.nk);
    const int64_t k0 = A.kg0 + r0;
    const float *p = x + (k0 - A.kx0) * sz;  // slice of row r
    auto plane = [&](const float *q) { return TvPlane{q[oc], q[oe], q[on], q[ow], q[own], q[os], q[ose]}; };
    const int64_t top = min(r1, (int64_t)A.nz - 1 - A.kg0);  // rows below it have a slice above in the volume
    TvPlane pc = plane(p), pn = r0 < top ? plane(p + sz) : pc;
    float pz = 0.0f;  // p_z of the slice below
    if (k0 > 0) {
        const float *q = p - sz;
        const float c = q[oc], dx = q[oe] - c, dy = q[on] - c, dz = pc.c - c;
        pz = dz * tv_rsqrt<TINY>(fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, A.eps))));
    }
#pragma unroll 1
    for (int64_t r = r0; r < r1; ++r, p += sz) {
        // the slice above the next one is loaded while this one is worked on
        TvPlane pf = pn;
        if (r + 1 < top) pf = plane(p + 2 * sz);
        const float c = pc.c;
        const float dx = pc.e - c, dy = pc.n - c, dz = pn.c - c;
        const float q = tv_rsqrt<TINY>(fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, A.eps))));
        const float wx = c - pc.w, wy = pc.wn - pc.w, wz = pn.w - pc.w;
        const float qw = tv_rsqrt<TINY>(fmaf(wx, wx, fmaf(wy, wy, fmaf(wz, wz, A.eps))));
        const float sx = pc.se - pc.s, sy = c - pc.s, sz_ = pn.s - pc.s;
        const float qs = tv_rsqrt<TINY>(fmaf(sx, sx, fmaf(sy, sy, fmaf(sz_, sz_, A.eps))));
        const float g = fmaf(-(dx + dy + dz), q, fmaf(wx, qw, fmaf(sy, qs, pz)));
        visit((p - x) + oc, c, g);
        pz = dz * q;
        pc = pn;
        pn = pf;
    }
}

// Partial sums of g^2 (and, XX, of x^2) over the tiles, FP64: block b takes tiles b, b + gridDim.x, ...
// and writes partials[b] (and partials[DOT_BLOCKS + b]).  COPY also writes x to y.
template <bool TINY, bool XX, bool COPY>
__global__ __launch_bounds__(TV_THREADS) void k_tv_norm(const float *__restrict__ x, TvArgs A, float *__restrict__ y,
                                                        double *__restrict__ partials) {
    __shared__ double lds[TV_TY];
    double gg = 0.0, xx = 0.0;
    const unsigned n = A.bx * A.by * A.bz;
    for (unsigned t = blockIdx.x; t < n; t += gridDim.x)
        tv_walk<TINY>(x, A, tv_tile(A, t), [&](int64_t o, float c, float g) {
            gg = fma((double)g, (double)g, gg);
            if (XX) xx = fma((double)c, (double)c, xx);
            if (COPY) y[o] = c;
        });
    gg = block_sum(gg, lds);
    if (threadIdx.x == 0) partials[blockIdx.x] = gg;
    if (XX) {
        xx = block_sum(xx, lds);
        if (threadIdx.x == 0) partials[DOT_BLOCKS + blockIdx.x] = xx;
    }
}

// TV scalars: [0] = ||x_in||^2, [1] = alpha, [2] = ||g||^2
// The partial sums of k_tv_norm in a fixed order; with XX also alpha = lambda ||x_in||
template <bool XX>
__global__ __launch_bounds__(DOT_THREADS) void k_tv_sum(const double *__restrict__ partials, int n,
                                                        double *__restrict__ scal, double lambda) {
    __shared__ double lds[DOT_THREADS / 64];
    double gg = 0.0, xx = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        gg += partials[i];
        if (XX) xx += partials[DOT_BLOCKS + i];
    }
    gg = block_sum(gg, lds);
    if (XX) xx = block_sum(xx, lds);
    if (threadIdx.x == 0) {
        scal[2] = gg;
        if (XX) {
            scal[0] = xx;
            scal[1] = lambda * sqrt(xx);
        }
    }
}

// y = x - alpha g / ||g|| over the slices of A (x as it is when ||g|| is not positive); y holds slices
// from ky0 on
template <bool TINY>
__global__ __launch_bounds__(TV_THREADS) void k_tv_apply(const float *__restrict__ x, float *__restrict__ y, TvArgs A,
                                                         int64_t ky0, const double *__restrict__ scal) {
    const double ng2 = scal[2];
    const bool go = ng2 > 0.0;
    const float a = go ? (float)(scal[1] / sqrt(ng2)) : 0.0f;
    float *yo = y - (ky0 - A.kx0) * ((int64_t)A.nx * A.ny);
    tv_walk<TINY>(x, A, tv_tile(A, (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x),
                  [&](int64_t o, float c, float g) { yo[o] = go ? fmaf(-a, g, c) : c; });
}

TvArgs tv_args(int nx, int ny, int nz, double eps, int64_t kx0, int64_t kg0, int64_t nk) {
    TvArgs A;
    A.nx = nx;
    A.ny = ny;
    A.nz = nz;
    A.eps = (float)eps;
    A.kx0 = kx0;
    A.kg0 = kg0;
    A.nk = nk;
    A.bx = (unsigned)((nx + 63) / 64);
    A.by = (unsigned)((ny + TV_TY - 1) / TV_TY);
    // a run's first slice costs 1.4 of the others, so runs are as long as still leaves 1024 blocks of 8
    // waves (a full chip): 512^3 with runs of 32 / 16 / 8 / 4 slices 2.95 / 3.07 / 3.23 / 3.67 ms (5
    // steps), 256^3 0.40 / 0.41 / 0.39 / 0.43, 101 x 97 x 90 0.148 / 0.105 / 0.094 / 0.088 (4 steps)
    A.zr = 32;
    while (A.zr > 4 && (int64_t)A.bx * A.by * ((nk + A.zr - 1) / A.zr) < 1024) A.zr /= 2;
    A.bz = (unsigned)((nk + A.zr - 1) / A.zr);
    // images that the 256 MB last-level cache holds: neighbouring tiles on one XCD read their shared rows
    // from its L2 (256^3 0.39 -> 0.33 ms, 301 x 290 x 277 0.69 -> 0.64); larger ones stream better from all
    // XCDs at once (512^3 2.74 against 2.82 ms)
    A.by_xcd = (int64_t)nx * ny * nz <= (int64_t(64) << 20);
    return A;
}
bool tv_tiny(const TvArgs &A) { return !(A.eps >= FLT_MIN) || (int64_t)A.nx * A.ny >= (int64_t(1) << 32); }

// ||g||^2 of slices kg0 .. kg0 + nk - 1 into scal[2]; xx: also their ||x||^2 into scal[0] and
// alpha = lambda ||x|| into scal[1]; copy (with xx): x to y.  partials: 2 DOT_BLOCKS doubles.
ct_status launch_tv_norm(const float *x, const TvArgs &A, bool xx, float *y, double *partials, double *scal, double lambda,
                         hipStream_t st) {
    const int64_t tiles = (int64_t)A.bx * A.by * A.bz;
    if (tiles > 0x7fffffff) return fail(CT_ERR_ARG, "TV: the image is too large");
    const unsigned nb = (unsigned)std::min<int64_t>(tiles, DOT_BLOCKS);
#define CT_TV_N(TI, XX_, CO) \
    hipLaunchKernelGGL((k_tv_norm<TI, XX_, CO>), dim3(nb), dim3(TV_THREADS), 0, st, x, A, y, partials)
    if (tv_tiny(A)) {
        if (xx && y) CT_TV_N(true, true, true);
        else if (xx) CT_TV_N(true, true, false);
        else CT_TV_N(true, false, false);
    } else {
        if (xx && y) CT_TV_N(false, true, true);
        else if (xx) CT_TV_N(false, true, false);
        else CT_TV_N(false, false, false);
    }
#undef CT_TV_N
    CT_HIP(hipGetLastError());
    if (xx) hipLaunchKernelGGL((k_tv_sum<true>), dim3(1), dim3(DOT_THREADS), 0, st, partials, (int)nb, scal, lambda);
    else hipLaunchKernelGGL((k_tv_sum<false>), dim3(1), dim3(DOT_THREADS), 0, st, partials, (int)nb, scal, lambda);
    CT_HIP(hipGetLastError());
    return CT_OK;
}

ct_status launch_tv_apply(const float *x, float *y, const TvArgs &A, int64_t ky0, const double *scal, hipStream_t st) {
    const dim3 grid(A.bx, A.by, A.bz);
    if (tv_tiny(A)) hipLaunchKernelGGL((k_tv_apply<true>), grid, dim3(TV_THREADS), 0, st, x, y, A, ky0, scal);
    else hipLaunchKernelGGL((k_tv_apply<false>), grid, dim3(TV_THREADS), 0, st, x, y, A, ky0, scal);
    CT_HIP(hipGetLastError());
    return CT_OK;
}

// ROF model by Chambolle's projection.  The dual field p = (px, py, pz) holds one FP32 volume per
// axis.  Divergence, minus the adjoint of the forward-difference gradient: along each axis
// p_i - p_{i-1} inside, p_0 at the first index, -p_{n-2} at the last, 0 for an axis of one voxel.
__device__ __forceinline__ float rof_div(const float *__restrict__ px, const float *__restrict__ py,
                                         const float *__restrict__ pz, int i, int j, int k, int nx, int ny, int nz,
                                         int64_t o, int64_t sy, int64_t sz) {
    float d = 0.0f;
    if (nz > 1) d += k == 0 ? pz[o] : (k == nz - 1 ? -pz[o - sz] : pz[o] - pz[o - sz]);
    if (ny > 1) d += j == 0 ? py[o] : (j == ny - 1 ? -py[o - sy] : py[o] - py[o - sy]);
    if (nx > 1) d += i == 0 ? px[o] : (i == nx - 1 ? -px[o - 1] : px[o] - px[o - 1]);
    return d;
}

// The iteration's arithmetic, shared by the one-pass and two-pass kernels (explicit FMAs, so that both
// round alike): w from div p, the step's denominator 1 + tau |grad w|, and a component's new value.
__device__ __forceinline__ float rof_w(float div, float f, float inv_lam) { return fmaf(-f, inv_lam, div); }
__device__ __forceinline__ float rof_den(float gx, float gy, float gz, float tau) {
    return fmaf(tau, sqrtf(fmaf(gz, gz, fmaf(gy, gy, gx * gx))), 1.0f);
}
__device__ __forceinline__ float rof_p(float p, float g, float tau, float den) { return fmaf(tau, g, p) / den; }

// w = div p - f / lam
__global__ __launch_bounds__(256) void k_rof_w(const float *__restrict__ f, const float *__restrict__ px,
                                               const float *__restrict__ py, const float *__restrict__ pz,
                                               float *__restrict__ w, int nx, int ny, int nz, float inv_lam) {
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);
    const int j = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int k = blockIdx.z;
    if (i >= nx || j >= ny) return;
    const int64_t sy = nx, sz = (int64_t)nx * ny;
    const int64_t o = k * sz + (int64_t)j * sy + i;
    w[o] = rof_w(rof_div(px, py, pz, i, j, k, nx, ny, nz, o, sy, sz), f[o], inv_lam);
}

// p <- (p + tau grad w) / (1 + tau |grad w|), forward differences, zero at the last index
__global__ __launch_bounds__(256) void k_rof_p(const float *__restrict__ w, float *__restrict__ px,
                                               float *__restrict__ py, float *__restrict__ pz, int nx, int ny, int nz,
                                               float tau) {
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);
    const int j = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int k = blockIdx.z;
    if (i >= nx || j >= ny) return;
    const int64_t sy = nx, sz = (int64_t)nx * ny;
    const int64_t o = k * sz + (int64_t)j * sy + i;
    const float wc = w[o];
    const float gx = i < nx - 1 ? w[o + 1] - wc : 0.0f;
    const float gy = j < ny - 1 ? w[o + sy] - wc : 0.0f;
    const float gz = k < nz - 1 ? w[o + sz] - wc : 0.0f;
    const float den = rof_den(gx, gy, gz, tau);
    px[o] = rof_p(px[o], gx, tau, den);
    py[o] = rof_p(py[o], gy, tau, den);
    pz[o] = rof_p(pz[o], gz, tau, den);
}

// One whole iteration, p into q (another dual field; a voxel's step reads its neighbours' old p), without
// storing w: 28 bytes of memory traffic per voxel where the two passes take 48.  A thread walks a run of
// slices of its (i, j) column and needs w at the voxel, at its right neighbour, at the row above and at
// the slice above.  w of the slice above becomes the next slice's own; the right neighbour's comes from
// the next lane (the last lane forms it itself); the row above's is formed again (its loads are the next
// wave's, in L1).  So a slice takes 11 loads (4.7 address-unit cycles each, a quarter of the time its
// 28 bytes take from HBM) and no LDS or barrier.  FIRST: p = 0 is not read.  The arithmetic is that of the
// two passes, bit for bit.  Bound: HBM.  512^3, 10 iterations 20.1 -> 10.7 ms (3.8 TB/s of the 28 bytes);
// 301 x 277 x 193, 20 iterations 4.87 -> 3.04 ms.
constexpr int ROF_TY = 4;
struct RofArgs {
    const float *f, *px, *py, *pz;
    float *qx, *qy, *qz;
    int nx, ny, nz, zr;
    float inv_lam, tau;
};
template <bool FIRST>
__global__ __launch_bounds__(64 * ROF_TY) void k_rof_step(RofArgs A) {
    const int lane = threadIdx.x & 63;
    const int iu = blockIdx.x * 64 + lane, i = min(iu, A.nx - 1);  // lanes past the row repeat its last voxel
    const int j = blockIdx.y * ROF_TY + (threadIdx.x >> 6);
    if (j >= A.ny) return;
    const int64_t sy = A.nx, sz = (int64_t)A.nx * A.ny;
    const int k0 = blockIdx.z * A.zr, k1 = min(k0 + A.zr, A.nz);
    const bool hx = i < A.nx - 1, hy = j < A.ny - 1, lx = i > 0, ly = j > 0;
    const int64_t ow = lx ? -1 : 0, os = ly ? -sy : 0, on = hy ? sy : 0, oe = hx ? 1 : 0;
    // w at offset o whose x, y and z components of p are (x, y, z) there and (xm, ym, zm) one voxel below
    // along each axis; h / l: it is not the last / first voxel of the axis
    auto w_of = [&](float f, float x, float xm, bool h_x, bool l_x, float y, float ym, bool h_y, bool l_y, float z,
                    float zm, bool h_z, bool l_z) {
        float d = (h_z ? z : 0.0f) - (l_z ? zm : 0.0f);
        d += (h_y ? y : 0.0f) - (l_y ? ym : 0.0f);
        d += (h_x ? x : 0.0f) - (l_x ? xm : 0.0f);
        return rof_w(d, f, A.inv_lam);
    };
    auto ld = [&](const float *a, int64_t o) { return FIRST ? 0.0f : a[o]; };
    int64_t o = (int64_t)k0 * sz + (int64_t)j * sy + i;
    const int64_t od = k0 > 0 ? -sz : 0;
    const bool edge = lane == 63 && hx;  // forms its right neighbour's w itself
    const bool hx2 = i + 1 < A.nx - 1, hy2 = j + 1 < A.ny - 1;
    // the slice's own p, and p_z of the slice below at the row above and (last lane) at the right neighbour
    float x = ld(A.px, o), y = ld(A.py, o), z = ld(A.pz, o);
    float w = w_of(A.f[o], x, ld(A.px, o + ow), hx, lx, y, ld(A.py, o + os), hy, ly, z, ld(A.pz, o + od),
                   k0 < A.nz - 1, k0 > 0);
    float znm = ld(A.pz, o + on + od), zem = edge ? ld(A.pz, o + oe + od) : 0.0f;
    for (int k = k0; k < k1; ++k, o += sz) {
        const bool hz = k < A.nz - 1, lz = k > 0;
        // the slice above
        float xu = 0.0f, yu = 0.0f, zu = 0.0f, wu = 0.0f;
        if (hz) {
            const int64_t u = o + sz;
            xu = ld(A.px, u);
            yu = ld(A.py, u);
            zu = ld(A.pz, u);
            wu = w_of(A.f[u], xu, ld(A.px, u + ow), hx, lx, yu, ld(A.py, u + os), hy, ly, zu, z, k + 1 < A.nz - 1, true);
        }
        // the row above
        const int64_t n = o + on;
        const float zn = ld(A.pz, n);
        const float wn = w_of(A.f[n], ld(A.px, n), ld(A.px, n + ow), hx, lx, ld(A.py, n), y, hy2, true, zn, znm, hz, lz);
        znm = zn;
        // the right neighbour
        float we = __shfl_down(w, 1, 64);
        if (edge) {
            const int64_t e = o + oe;
            const float ze = ld(A.pz, e);
            we = w_of(A.f[e], ld(A.px, e), x, hx2, true, ld(A.py, e), ld(A.py, e + os), hy, ly, ze, zem, hz, lz);
            zem = ze;
        }
        const float gx = hx ? we - w : 0.0f, gy = hy ? wn - w : 0.0f, gz = hz ? wu - w : 0.0f;
        const float den = rof_den(gx, gy, gz, A.tau);
        if (iu < A.nx) {
            A.qx[o] = rof_p(x, gx, A.tau, den);
            A.qy[o] = rof_p(y, gy, A.tau, den);
            A.qz[o] = rof_p(z, gz, A.tau, den);
        }
        x = xu;
        y = yu;
        z = zu;
        w = wu;
    }
}

// u = f - lam div p, in place over f (each voxel reads only its own f)
__global__ __launch_bounds__(256) void k_rof_u(float *__restrict__ x, const float *__restrict__ px,
                                               const float *__restrict__ py, const float *__restrict__ pz, int nx,
                                               int ny, int nz, float lam) {
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);
    const int j = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int k = blockIdx.z;
    if (i >= nx || j >= ny) return;
    const int64_t sy = nx, sz = (int64_t)nx * ny;
    const int64_t o = k * sz + (int64_t)j * sy + i;
    x[o] = fmaf(-lam, rof_div(px, py, pz, i, j, k, nx, ny, nz, o, sy, sz), x[o]);
}

__global__ void k_fill_zero(float *__restrict__ p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0f;
}

struct Workspace {
    char *base = nullptr;
    bool owned = false;
    hipStream_t st = nullptr;
    size_t off = 0;
    void *take(size_t bytes) {
        void *p = base + off;
        off += align256(bytes);
        return p;
    }
    ct_status acquire(void *user, size_t bytes, hipStream_t s) {
        st = s;
        if (user) {
            base = (char *)user;
            return CT_OK;
        }
        CT_HIP(CT_MALLOC_ASYNC((void **)&base, bytes ? bytes : 256, s));
        owned = true;
        return CT_OK;
    }
    ~Workspace() {
        if (owned && base) (void)hipFreeAsync(base, st);
    }
};

}  // namespace

size_t dot_partials_count() { return DOT_BLOCKS; }

ct_status dot_f64(const void *a, const void *b, ct_dtype t, int64_t n, double *out, double *partials, hipStream_t st) {
    Workspace ws;
    if (!partials) {
        ct_status s = ws.acquire(nullptr, DOT_BLOCKS * sizeof(double), st);
        if (s != CT_OK) return s;
        partials = (double *)ws.take(DOT_BLOCKS * sizeof(double));
    }
    CT_DISPATCH1_ANY(t, T,
                     hipLaunchKernelGGL((k_dot_partial<T>), dim3(DOT_BLOCKS), dim3(DOT_THREADS), 0, st, (const T *)a,
                                        (const T *)b, n, partials));
    CT_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(DOT_THREADS), 0, st, partials, DOT_BLOCKS, out);
    CT_HIP(hipGetLastError());
    return CT_OK;
}

ct_status convert(const void *src, ct_dtype s_t, void *dst, ct_dtype d_t, int64_t n, hipStream_t st) {
    if (n == 0) return CT_OK;
    CT_DISPATCH1_ANY(s_t, TS,
                     CT_DISPATCH1_ANY(d_t, TD,
                                      hipLaunchKernelGGL((k_convert<TS, TD>), dim3(ew_grid(n)), dim3(EW_THREADS), 0, st,
                                                         (const TS *)src, (TD *)dst, n)));
    CT_HIP(hipGetLastError());
    return CT_OK;
}

// ---------------------------------------------------------------------------------------------
// CGLS

// The recurrence vectors r, q (projection-shaped) and s, p (volume-shaped) are FP32 whatever the
// storage of x and b: CGLS search directions are unnormalised (A p grows like the operator norm
// squared times the data), which overflows FP16's range on realistic problems.
// r, q (projections), s, p (volumes), partials and scalars, the Siddon column copy of the volume
// being projected, and the exact adjoint's transposed projection copy: no allocation per iteration
size_t cgls_workspace(const ct_plan *p, ct_dtype, ct_dtype) {
    const ct_geometry &g = p->g;
    const size_t nv = (size_t)g.nVoxel[0] * g.nVoxel[1] * g.nVoxel[2];
    const size_t np = (size_t)g.nDetector[0] * g.nDetector[1] * p->angles.size();
    return 2 * align256(nv * 4) + 2 * align256(np * 4) + align256(DOT_BLOCKS * 8) + align256(S_COUNT * 8) +
           align256(zcol_bytes(g, 4)) + align256(p->angles.size() * adj_chunk_bytes_per_angle(g));
}

ct_status cgls_run(ct_plan *p, const void *b, ct_dtype pt, void *x, ct_dtype vt, int32_t niter, double *resid,
                   void *work, hipStream_t st) {
    const ct_geometry &g = p->g;
    const int64_t nv = g.nVoxel[0] * g.nVoxel[1] * g.nVoxel[2];
    const int64_t na = (int64_t)p->angles.size();
    const int64_t np = g.nDetector[0] * g.nDetector[1] * na;
    Workspace ws;
    ct_status s = ws.acquire(work, cgls_workspace(p, vt, pt), st);
    if (s != CT_OK) return s;
    float *r = (float *)ws.take(np * 4);
    float *q = (float *)ws.take(np * 4);
    float *sv = (float *)ws.take(nv * 4);
    float *pv = (float *)ws.take(nv * 4);
    double *parts = (double *)ws.take(DOT_BLOCKS * 8);
    double *scal = (double *)ws.take(S_COUNT * 8);
    void *vz = zcol_base(ws.take(zcol_bytes(g, 4)), 4);
    const size_t qbytes = (size_t)na * adj_chunk_bytes_per_angle(g);
    void *yq = ws.take(qbytes);
    const Slab full = full_slab(g);
    Slab single = full;  // the adjoint's, voxels taken one by one
    single.pairs = false;
    const bool col = zcol_ok(p, 0, na);
#define CK(e)                          \
    do {                               \
        ct_status s_ = (e);            \
        if (s_ != CT_OK) return s_;    \
    } while (0)
    // A v through the column copy in the workspace (refreshed from v first)
    auto fwd = [&](const void *v, ct_dtype t, float *out) -> ct_status {
        if (col) {
            ct_status s_ = launch_zcols(v, t, vz, g.nVoxel[0], g.nVoxel[1], g.nVoxel[2], st);
            if (s_ != CT_OK) return s_;
        }
        return launch_forward(p, CT_SIDDON, v, t, out, CT_F32, 0, 0, na, full, st, col ? vz : nullptr);
    };
    // r = b - A x ; s = A^T r ; p = s ; gamma = <s,s> ; rho = <r,r>
    CK(fwd(x, vt, r));
    CT_DISPATCH1(pt, T, hipLaunchKernelGGL((k_rsub_from<T>), dim3(ew_grid(np)), dim3(EW_THREADS), 0, st, (const T *)b, r, np));
    CT_HIP(hipGetLastError());
    CK(launch_backproject(p, CT_BP_ADJOINT, r, CT_F32, sv, CT_F32, 0, 0, na, single, st, yq, qbytes));
    hipLaunchKernelGGL((k_copy<float>), dim3(ew_grid(nv)), dim3(EW_THREADS), 0, st, (const float *)sv, pv, nv);
    CT_HIP(hipGetLastError());
    CK(dot_f64(sv, sv, CT_F32, nv, scal + S_GAMMA, parts, st));
    CK(dot_f64(r, r, CT_F32, np, scal + S_RHO, parts, st));
    hipLaunchKernelGGL(k_cgls_start, dim3(1), dim3(1), 0, st, scal, resid);
    CT_HIP(hipGetLastError());
    for (int32_t k = 0; k < niter; ++k) {
        // q = A p ; delta = <q,q> ; alpha = gamma / delta
        CK(fwd(pv, CT_F32, q));
        CK(dot_f64(q, q, CT_F32, np, scal + S_DELTA, parts, st));
        hipLaunchKernelGGL(k_cgls_alpha, dim3(1), dim3(1), 0, st, scal, resid, k);
        CT_HIP(hipGetLastError());
        // x += alpha p (x in its storage type) ; r -= alpha q
        CT_DISPATCH1(vt, T, hipLaunchKernelGGL((k_axpy_mixed<T>), dim3(ew_grid(nv)), dim3(EW_THREADS), 0, st, (T *)x,
                                               (const float *)pv, scal, (int)S_ALPHA, 1.0f, nv));
        hipLaunchKernelGGL((k_axpy_s<float>), dim3(ew_grid(np)), dim3(EW_THREADS), 0, st, r, (const float *)q, scal,
                           (int)S_ALPHA, -1.0f, np);
        CT_HIP(hipGetLastError());
        // s = A^T r ; gamma' = <s,s> ; beta = gamma'/gamma ; p = s + beta p
        CK(launch_backproject(p, CT_BP_ADJOINT, r, CT_F32, sv, CT_F32, 0, 0, na, single, st, yq, qbytes));
        CK(dot_f64(sv, sv, CT_F32, nv, scal + S_TMP, parts, st));
        hipLaunchKernelGGL(k_cgls_beta, dim3(1), dim3(1), 0, st, scal);
        CT_HIP(hipGetLastError());
        hipLaunchKernelGGL((k_xpby_s<float>), dim3(ew_grid(nv)), dim3(EW_THREADS), 0, st, pv, (const float *)sv, scal,
                           (int)S_BETA, nv);
        CT_HIP(hipGetLastError());
    }
    return CT_OK;
}

// ---------------------------------------------------------------------------------------------
// SART

// chords of every ray, one subset's residuals (and their transposes), and a column-major copy of x
// that the sweep projects from and updates in place (x is restored from it at the end)
size_t sart_workspace(const ct_plan *p, int32_t block) {
    const ct_geometry &g = p->g;
    const size_t pix = (size_t)g.nDetector[0] * g.nDetector[1];
    const size_t nb = (size_t)std::max<int32_t>(block, 1);
    return align256(pix * p->angles.size() * 4) + 2 * align256(pix * nb * 4) + align256(zcol_bytes(g, 4));
}

// OS-SART: the angles in natural order, cut into consecutive subsets of `block` (the last one may be
// shorter); each subset projects, forms its weighted residuals and makes one update (block = 1 is
// SART)
ct_status sart_run(ct_plan *p, const void *b, ct_dtype pt, void *x, ct_dtype vt, int32_t niter, double lambda,
                   int32_t block, void *work, hipStream_t st) {
    const ct_geometry &g = p->g;
    const int64_t na = (int64_t)p->angles.size();
    const int64_t pix = g.nDetector[0] * g.nDetector[1];
    const int64_t nvox = g.nVoxel[0] * g.nVoxel[1] * g.nVoxel[2];
    const size_t pe = dtype_size(pt);
    Workspace ws;
    ct_status s = ws.acquire(work, sart_workspace(p, block), st);
    if (s != CT_OK) return s;
    float *chord = (float *)ws.take(pix * na * 4);
    float *r = (float *)ws.take(pix * block * 4);
    float *rT = (float *)ws.take(pix * block * 4);
    float *xz = (float *)zcol_base(ws.take(zcol_bytes(g, 4)), 4);
    const float thr = (float)(1e-2 * std::fmin(g.dVoxel[0], std::fmin(g.dVoxel[1], g.dVoxel[2])));
    const int nu = (int)g.nDetector[0], nv = (int)g.nDetector[1];
    CK(launch_ray_chord(p, chord, 0, na, st));
    Slab full = full_slab(g);
    full.own_angles = true;  // (a sweep always projects the same subsets)
    // the sweep updates an FP32 image: the column-major copy, or (other geometries) x itself when
    // it is stored in FP32, else an FP32 copy of it; a 16-bit x is rounded once, at the end
    // the column-major sweep's update kernel is written for a circular orbit; plans of views update
    // x through the per-view kernel
    if (zcol_ok(p, 0, na) && !p->views) {
        CK(launch_zcols_f32(x, vt, xz, g.nVoxel[0], g.nVoxel[1], g.nVoxel[2], st));
        for (int32_t it = 0; it < niter; ++it) {
            for (int64_t t0 = 0; t0 < na; t0 += block) {
                const int64_t t1 = std::min<int64_t>(na, t0 + block);
                CK(launch_forward(p, CT_SIDDON, xz, CT_F32, r, CT_F32, 0, t0, t1, full, st, xz));
                const dim3 tg((unsigned)((nu + 31) / 32), (unsigned)((nv + 31) / 32), (unsigned)(t1 - t0));
                const void *bt = (const char *)b + t0 * pix * pe;
                CT_DISPATCH1(pt, TP,
                             hipLaunchKernelGGL((k_sart_resid_t<TP>), tg, dim3(256), 0, st, (const TP *)bt,
                                                chord + t0 * pix, (const float *)r, rT, thr, nu, nv));
                CT_HIP(hipGetLastError());
                CK(launch_sart_update_col(p, rT, xz, t0, t1, (float)lambda, st));
            }
        }
        CK(launch_zcols_inv_f32(xz, x, vt, g.nVoxel[0], g.nVoxel[1], g.nVoxel[2], st));
        return CT_OK;
    }
    float *xf = (float *)x;
    if (vt != CT_F32) {
        xf = xz;
        CK(convert(x, vt, xf, CT_F32, nvox, st));
    }
    for (int32_t it = 0; it < niter; ++it) {
        for (int64_t t0 = 0; t0 < na; t0 += block) {
            const int64_t t1 = std::min<int64_t>(na, t0 + block);
            CK(launch_forward(p, CT_SIDDON, xf, CT_F32, r, CT_F32, 0, t0, t1, full, st));
            const void *bt = (const char *)b + t0 * pix * pe;
            CT_DISPATCH1(pt, TP,
                         hipLaunchKernelGGL((k_sart_resid<TP>), dim3(ew_grid((t1 - t0) * pix)), dim3(EW_THREADS), 0, st,
                                            (const TP *)bt, chord + t0 * pix, r, thr, (t1 - t0) * pix));
            CT_HIP(hipGetLastError());
            CK(launch_sart_update(p, r, xf, t0, t1, (float)lambda, st));
        }
    }
    if (vt != CT_F32) CK(convert(xf, CT_F32, x, vt, nvox, st));
    return CT_OK;
}

// ---------------------------------------------------------------------------------------------
// TV steepest descent

size_t tv_workspace(const ct_geometry &g, ct_dtype vt) {
    const size_t nv = (size_t)g.nVoxel[0] * g.nVoxel[1] * g.nVoxel[2];
    // a 16-bit image is stepped in an FP32 copy
    return align256(nv * 4) * (vt == CT_F32 ? 1 : 2) + align256(2 * DOT_BLOCKS * 8) + align256(4 * 8);
}

ct_status tv_run(const ct_geometry &g, void *xs, ct_dtype vt, int32_t nsteps, double lambda, double eps, void *work,
                 hipStream_t st) {
    const int nx = (int)g.nVoxel[0], ny = (int)g.nVoxel[1], nz = (int)g.nVoxel[2];
    const int64_t nv = (int64_t)nx * ny * nz;
    Workspace ws;
    ct_status s = ws.acquire(work, tv_workspace(g, vt), st);
    if (s != CT_OK) return s;
    float *buf = (float *)ws.take(nv * 4);
    double *parts = (double *)ws.take(2 * DOT_BLOCKS * 8);
    double *scal = (double *)ws.take(4 * 8);
    float *x = (float *)xs;
    if (vt != CT_F32) {
        x = (float *)ws.take(nv * 4);
        CK(convert(xs, vt, x, CT_F32, nv, st));
    }
    if (nsteps <= 0) return CT_OK;
    const TvArgs A = tv_args(nx, ny, nz, eps, 0, 0, nz);
    // the steps alternate between the two arrays; with an odd number of them on an FP32 image the first
    // norm pass copies x, so that the last step writes the caller's array
    const bool copy = vt == CT_F32 && (nsteps & 1);
    float *src = copy ? buf : x, *dst = copy ? x : buf;
    for (int32_t k = 0; k < nsteps; ++k) {
        if (k == 0) CK(launch_tv_norm(x, A, true, copy ? buf : nullptr, parts, scal, lambda, st));
        else CK(launch_tv_norm(src, A, false, nullptr, parts, scal, lambda, st));
        CK(launch_tv_apply(src, dst, A, 0, scal, st));
        std::swap(src, dst);
    }
    if (vt != CT_F32) CK(convert(src, CT_F32, xs, vt, nv, st));
    return CT_OK;
#undef CK
}


// ---------------------------------------------------------------------------------------------
// ROF model (Chambolle's projection)

namespace {
// Whether an iteration runs in one pass between two dual fields (workspace: six volumes) or in two
// passes over one (four: px, py, pz, w).  The one-pass form takes half the time; above 16 GiB per volume
// its two more volumes would be what no longer fits a 288 GB device, so the four-volume form stays there,
// where the library's own allocation of six fails, and for callers' buffers that hold four.
bool rof_one_pass(const ct_geometry &g) {
    return (uint64_t)g.nVoxel[0] * g.nVoxel[1] * g.nVoxel[2] <= (uint64_t(4) << 30);
}
size_t rof_volumes(const ct_geometry &g, int n) {
    return (size_t)n * align256((size_t)g.nVoxel[0] * g.nVoxel[1] * g.nVoxel[2] * 4);
}
}  // namespace

size_t rof_workspace(const ct_geometry &g) { return rof_volumes(g, 4); }

ct_status rof_run(const ct_geometry &g, void *x, int32_t niter, double lambda, double tau, void *work, size_t work_bytes,
                  hipStream_t st) {
    const int nx = (int)g.nVoxel[0], ny = (int)g.nVoxel[1], nz = (int)g.nVoxel[2];
    const int64_t nv = (int64_t)nx * ny * nz;
    if (niter == 0) return CT_OK;  // u = f
    bool one = rof_one_pass(g) && (!work || work_bytes >= rof_volumes(g, 6));
    Workspace ws;
    ct_status s = ws.acquire(work, rof_volumes(g, one ? 6 : 4), st);
    if (s == CT_ERR_OOM && one) {
        (void)hipGetLastError();
        one = false;
        s = ws.acquire(nullptr, rof_volumes(g, 4), st);
    }
    if (s != CT_OK) return s;
    float *p[3], *q[3];
    for (auto &v : p) v = (float *)ws.take(nv * 4);
    const dim3 grid((nx + 63) / 64, (ny + 3) / 4, nz);
    if (one) {
        for (auto &v : q) v = (float *)ws.take(nv * 4);
        // runs of 8 slices, 4 where those would leave fewer than 2048 blocks of 4 waves (longer ones read
        // less twice but keep fewer rows of one slice in flight: 301 x 277 x 193, 20 iterations, runs of
        // 8 / 16 / 32 slices 3.04 / 3.14 / 3.35 ms; 512^3, 10 iterations, 10.70 / 10.83 / 10.84 ms)
        const int zr = (int64_t)grid.x * grid.y * ((nz + 7) / 8) < 2048 ? 4 : 8;
        const dim3 rgrid(grid.x, (ny + ROF_TY - 1) / ROF_TY, (nz + zr - 1) / zr);
        for (int32_t it = 0; it < niter; ++it) {
            const RofArgs A{(const float *)x, p[0], p[1], p[2], q[0], q[1], q[2], nx, ny, nz, zr,
                            (float)(1.0 / lambda), (float)tau};
            if (it == 0) hipLaunchKernelGGL((k_rof_step<true>), rgrid, dim3(64 * ROF_TY), 0, st, A);
            else hipLaunchKernelGGL((k_rof_step<false>), rgrid, dim3(64 * ROF_TY), 0, st, A);
            CT_HIP(hipGetLastError());
            std::swap(p, q);
        }
    } else {
        float *w = (float *)ws.take(nv * 4);
        for (auto &v : p) hipLaunchKernelGGL(k_fill_zero, dim3(ew_grid(nv)), dim3(EW_THREADS), 0, st, v, nv);
        CT_HIP(hipGetLastError());
        for (int32_t it = 0; it < niter; ++it) {
            hipLaunchKernelGGL(k_rof_w, grid, dim3(256), 0, st, (const float *)x, p[0], p[1], p[2], w, nx, ny, nz,
                               (float)(1.0 / lambda));
            hipLaunchKernelGGL(k_rof_p, grid, dim3(256), 0, st, (const float *)w, p[0], p[1], p[2], nx, ny, nz,
                               (float)tau);
            CT_HIP(hipGetLastError());
        }
    }
    hipLaunchKernelGGL(k_rof_u, grid, dim3(256), 0, st, (float *)x, p[0], p[1], p[2], nx, ny, nz, (float)lambda);
    CT_HIP(hipGetLastError());
    return CT_OK;
}

// ---------------------------------------------------------------------------------------------
// TV steepest descent out of core: the image in host memory, slabs of axial slices under a device
// memory cap.  The gradient at slice z needs slices z - 1 .. z + 1, so each slab is uploaded with a
// halo slice on either side.  A step is two passes over the slabs: the first sums ||g||^2 (and,
// at the first step, ||x_in||^2) slab by slab in FP64, in slab order; the second recomputes each
// slab's gradient and applies x -= alpha g / ||g||.  In the second pass the slab below has already
// been updated, so its last slice is kept on the device as it was before that update and replaces
// the uploaded lower halo: every gradient of a step sees the image from before the step.

namespace {

constexpr uint64_t TV_RESERVE = 64ull << 20;

struct DevMem {
    void *p = nullptr;
    ~DevMem() {
        if (p) (void)hipFree(p);
    }
};

// CT_OOC_VERBOSE=1 reports each finished pass on stderr (long out-of-core runs)
bool tv_verbose() {
    static const bool v = [] {
        const char *e = std::getenv("CT_OOC_VERBOSE");
        return e && e[0] && e[0] != '0';
    }();
    return v;
}

struct OwnStream {
    hipStream_t s = nullptr;
    ~OwnStream() {
        if (s) (void)hipStreamDestroy(s);
    }
};

}  // namespace

__global__ void k_scale_entry(double *p, double f) { *p *= f; }

ct_status tv_host_run_halo(const ct_geometry &g, float *hx, int32_t nsteps, double lambda, double eps, int32_t depth,
                           uint64_t cap, ct_ooc_stats *stats);

ct_status tv_host_run(const ct_geometry &g, float *hx, int32_t nsteps, double lambda, double eps, int32_t depth,
                      uint64_t cap, ct_ooc_stats *stats) {
    if (depth > 0) return tv_host_run_halo(g, hx, nsteps, lambda, eps, depth, cap, stats);
    const auto t_start = std::chrono::steady_clock::now();
    const int nx = (int)g.nVoxel[0], ny = (int)g.nVoxel[1];
    const int64_t nz = g.nVoxel[2];
    const int64_t slice = (int64_t)nx * ny;
    const uint64_t sb = (uint64_t)slice * sizeof(float);
    const uint64_t fixed = TV_RESERVE + align256(DOT_BLOCKS * 8) + align256(4 * 8);
    // device: the slab with two halo slices, its updated slices, one saved slice
    if (cap <= fixed || (cap - fixed) / sb < 5)
        return fail(CT_ERR_CAP, "device memory cap is below one slab slice plus halos and buffers");
    int64_t h = (int64_t)(((cap - fixed) / sb - 3) / 2);
    h = std::max<int64_t>(1, std::min<int64_t>(h, nz));
    const int64_t nsp = (nz + h - 1) / h;
    h = (nz + nsp - 1) / nsp;
    ct_ooc_stats st;
    std::memset(&st, 0, sizeof(st));
    st.n_slabs = (int32_t)nsp;
    st.slab_slices = (int32_t)h;
    OwnStream S;
    CT_HIP(hipStreamCreateWithFlags(&S.s, hipStreamNonBlocking));
    DevMem xb, gb, saved, parts, scal;
    CT_HIP(CT_MALLOC(&xb.p, (size_t)(h + 2) * sb));
    CT_HIP(CT_MALLOC(&gb.p, (size_t)h * sb));
    CT_HIP(CT_MALLOC(&saved.p, (size_t)sb));
    CT_HIP(CT_MALLOC(&parts.p, 2 * DOT_BLOCKS * 8));
    CT_HIP(CT_MALLOC(&scal.p, 4 * 8));
    float *xbuf = (float *)xb.p, *gbuf = (float *)gb.p;
    double *dscal = (double *)scal.p;
    const hipStream_t s = S.s;
    auto bounds = [&](int64_t n, int64_t &o0, int64_t &o1, int64_t &m0, int64_t &m1) {
        o0 = n * h;
        o1 = std::min(nz, o0 + h);
        m0 = std::max<int64_t>(0, o0 - 1);
        m1 = std::min(nz, o1 + 1);
    };
    // ||g||^2 (and, first step, ||x||^2) of the slab's own slices
    auto norms = [&](int64_t m0, int64_t o0, int64_t o1, bool with_x, double (&out)[3]) -> ct_status {
        ct_status e = launch_tv_norm(xbuf, tv_args(nx, ny, (int)nz, eps, m0, o0, o1 - o0), with_x, nullptr,
                                     (double *)parts.p, dscal, lambda, s);
        if (e != CT_OK) return e;
        CT_HIP(hipMemcpyAsync(out, dscal, sizeof(out), hipMemcpyDeviceToHost, s));
        CT_HIP(hipStreamSynchronize(s));
        return CT_OK;
    };
    double alpha = 0.0;
    ct_status e = CT_OK;
    for (int32_t step = 0; step < nsteps; ++step) {
        double gg = 0.0, xx = 0.0;
        for (int64_t n = 0; n < nsp; ++n) {  // pass 1: norms
            int64_t o0, o1, m0, m1;
            bounds(n, o0, o1, m0, m1);
            CT_HIP(hipMemcpyAsync(xbuf, hx + m0 * slice, (size_t)(m1 - m0) * sb, hipMemcpyHostToDevice, s));
            st.bytes_h2d += (double)(m1 - m0) * sb;
            double d[3] = {0.0, 0.0, 0.0};
            if ((e = norms(m0, o0, o1, step == 0, d)) != CT_OK) return e;
            gg += d[2];
            if (step == 0) xx += d[0];
        }
        if (step == 0) alpha = lambda * std::sqrt(xx);
        if (tv_verbose()) {
            std::fprintf(stderr, "[ct ooc tv] step %d: norms done at %.1f s\n", step + 1,
                         std::chrono::duration<double>(std::chrono::steady_clock::now() - t_start).count());
            std::fflush(stderr);
        }
        const double hs[4] = {xx, alpha, gg, 0.0};
        CT_HIP(hipMemcpyAsync(dscal, hs, sizeof(hs), hipMemcpyHostToDevice, s));
        for (int64_t n = 0; n < nsp; ++n) {  // pass 2: update
            int64_t o0, o1, m0, m1;
            bounds(n, o0, o1, m0, m1);
            CT_HIP(hipMemcpyAsync(xbuf, hx + m0 * slice, (size_t)(m1 - m0) * sb, hipMemcpyHostToDevice, s));
            st.bytes_h2d += (double)(m1 - m0) * sb;
            if (n > 0) CT_HIP(hipMemcpyAsync(xbuf, saved.p, (size_t)sb, hipMemcpyDeviceToDevice, s));
            if (n + 1 < nsp)
                CT_HIP(hipMemcpyAsync(saved.p, xbuf + (o1 - 1 - m0) * slice, (size_t)sb, hipMemcpyDeviceToDevice, s));
            const int64_t nown = (o1 - o0) * slice;
            if ((e = launch_tv_apply(xbuf, gbuf, tv_args(nx, ny, (int)nz, eps, m0, o0, o1 - o0), o0, dscal, s)) !=
                CT_OK)
                return e;
            CT_HIP(hipMemcpyAsync(hx + o0 * slice, gbuf, (size_t)nown * 4, hipMemcpyDeviceToHost, s));
            CT_HIP(hipStreamSynchronize(s));
            st.bytes_d2h += (double)nown * 4;
        }
        if (tv_verbose()) {
            std::fprintf(stderr, "[ct ooc tv] step %d: update done at %.1f s\n", step + 1,
                         std::chrono::duration<double>(std::chrono::steady_clock::now() - t_start).count());
            std::fflush(stderr);
        }
    }
    CT_HIP(hipStreamSynchronize(s));
    st.t_total_s = std::chrono::duration<double>(std::chrono::steady_clock::now() - t_start).count();
    if (stats) *stats = st;
    return CT_OK;
}


// The splitting of Section 2.3: each slab carries `depth` halo slices of its neighbours on either
// side and takes up to `depth` steps on its own copy before the slabs exchange anything.  A halo
// slice stops being exact one step after its outer neighbour, so the gradient is computed on a
// region that shrinks by a slice per step at each inner boundary and always covers the slab's own
// slices.  Each step's ||g||^2 is the slab's own sum scaled by (image slices / slab slices), the
// uniform-distribution estimate, so no norm is exchanged; alpha = lambda ||x_in|| comes from one
// pass over the whole image first.  In a round every slab starts from the image as it stood at the
// round's start: the lower halo is a device copy of the slices below, taken before their update.
ct_status tv_host_run_halo(const ct_geometry &g, float *hx, int32_t nsteps, double lambda, double eps, int32_t depth,
                           uint64_t cap, ct_ooc_stats *stats) {
    const auto t_start = std::chrono::steady_clock::now();
    const int nx = (int)g.nVoxel[0], ny = (int)g.nVoxel[1];
    const int64_t nz = g.nVoxel[2];
    const int64_t d = depth;
    const int64_t slice = (int64_t)nx * ny;
    const uint64_t sb = (uint64_t)slice * sizeof(float);
    const uint64_t fixed = TV_RESERVE + align256(DOT_BLOCKS * 8) + align256(4 * 8);
    // device: the slab with its halos twice (the steps alternate), `depth` saved slices
    if (cap <= fixed || (cap - fixed) / sb < (uint64_t)(5 * d + 2))
        return fail(CT_ERR_CAP, "device memory cap is below one slab slice plus halos and buffers");
    int64_t h = (int64_t)(((cap - fixed) / sb - 5 * d) / 2);
    h = std::max<int64_t>(1, std::min<int64_t>(h, nz));
    const int64_t nsp = (nz + h - 1) / h;
    h = (nz + nsp - 1) / nsp;
    ct_ooc_stats st;
    std::memset(&st, 0, sizeof(st));
    st.n_slabs = (int32_t)nsp;
    st.slab_slices = (int32_t)h;
    OwnStream S;
    CT_HIP(hipStreamCreateWithFlags(&S.s, hipStreamNonBlocking));
    DevMem xb, gb, saved, parts, scal;
    CT_HIP(CT_MALLOC(&xb.p, (size_t)(h + 2 * d) * sb));
    CT_HIP(CT_MALLOC(&gb.p, (size_t)(h + 2 * d) * sb));
    CT_HIP(CT_MALLOC(&saved.p, (size_t)d * sb));
    CT_HIP(CT_MALLOC(&parts.p, 2 * DOT_BLOCKS * 8));
    CT_HIP(CT_MALLOC(&scal.p, 4 * 8));
    float *xbuf = (float *)xb.p, *gbuf = (float *)gb.p, *sbuf = (float *)saved.p;
    double *dscal = (double *)scal.p;
    const hipStream_t s = S.s;
    ct_status e = CT_OK;
    // alpha from ||x_in||, summed slab by slab in FP64
    double xx = 0.0;
    for (int64_t n = 0; n < nsp; ++n) {
        const int64_t o0 = n * h, o1 = std::min(nz, o0 + h);
        CT_HIP(hipMemcpyAsync(xbuf, hx + o0 * slice, (size_t)(o1 - o0) * sb, hipMemcpyHostToDevice, s));
        st.bytes_h2d += (double)(o1 - o0) * sb;
        if ((e = dot_f64(xbuf, xbuf, CT_F32, (o1 - o0) * slice, dscal + 3, (double *)parts.p, s)) != CT_OK) return e;
        double v = 0.0;
        CT_HIP(hipMemcpyAsync(&v, dscal + 3, 8, hipMemcpyDeviceToHost, s));
        CT_HIP(hipStreamSynchronize(s));
        xx += v;
    }
    const double hs[4] = {xx, lambda * std::sqrt(xx), 0.0, 0.0};
    CT_HIP(hipMemcpyAsync(dscal, hs, sizeof(hs), hipMemcpyHostToDevice, s));
    CT_HIP(hipStreamSynchronize(s));
    for (int32_t done = 0; done < nsteps;) {
        const int64_t k = std::min<int64_t>(d, nsteps - done);
        for (int64_t n = 0; n < nsp; ++n) {
            const int64_t o0 = n * h, o1 = std::min(nz, o0 + h);
            const int64_t m0 = std::max<int64_t>(0, o0 - d), m1 = std::min(nz, o1 + d);
            CT_HIP(hipMemcpyAsync(xbuf + (o0 - m0) * slice, hx + o0 * slice, (size_t)(m1 - o0) * sb,
                                  hipMemcpyHostToDevice, s));
            st.bytes_h2d += (double)(m1 - o0) * sb;
            if (o0 > m0) CT_HIP(hipMemcpyAsync(xbuf, sbuf, (size_t)(o0 - m0) * sb, hipMemcpyDeviceToDevice, s));
            if (n + 1 < nsp) {  // the next slab's lower halo, as it stands at the round's start
                const int64_t n0 = std::max<int64_t>(0, o1 - d);
                CT_HIP(hipMemcpyAsync(sbuf, xbuf + (n0 - m0) * slice, (size_t)(o1 - n0) * sb, hipMemcpyDeviceToDevice,
                                      s));
            }
            const int64_t nown = (o1 - o0) * slice;
            float *cur = xbuf, *next = gbuf;
            for (int64_t i = 0; i < k; ++i) {
                const int64_t r0 = m0 == 0 ? 0 : m0 + i + 1, r1 = m1 == nz ? nz : m1 - i - 1;
                if ((e = launch_tv_norm(cur, tv_args(nx, ny, (int)nz, eps, m0, o0, o1 - o0), false, nullptr,
                                        (double *)parts.p, dscal, lambda, s)) != CT_OK)
                    return e;
                hipLaunchKernelGGL(k_scale_entry, dim3(1), dim3(1), 0, s, dscal + 2, (double)nz / (double)(o1 - o0));
                CT_HIP(hipGetLastError());
                // the slices a later step still reads lie in [r0, r1)
                if ((e = launch_tv_apply(cur, next, tv_args(nx, ny, (int)nz, eps, m0, r0, r1 - r0), m0, dscal, s)) !=
                    CT_OK)
                    return e;
                std::swap(cur, next);
            }
            CT_HIP(hipMemcpyAsync(hx + o0 * slice, cur + (o0 - m0) * slice, (size_t)nown * 4, hipMemcpyDeviceToHost,
                                  s));
            CT_HIP(hipStreamSynchronize(s));
            st.bytes_d2h += (double)nown * 4;
        }
        done += (int32_t)k;
        if (tv_verbose()) {
            std::fprintf(stderr, "[ct ooc tv] %d of %d steps done at %.1f s\n", done, nsteps,
                         std::chrono::duration<double>(std::chrono::steady_clock::now() - t_start).count());
            std::fflush(stderr);
        }
    }
    st.t_total_s = std::chrono::duration<double>(std::chrono::steady_clock::now() - t_start).count();
    if (stats) *stats = st;
    return CT_OK;
}

// The ROF iteration of rof_run on an image in host memory (Section 2.3: the minimiser holds five
// image copies, f, the dual field p and w, and its image splits stream through host memory).  The
// dual field lives in the caller's host workspace (three images).  Rounds of up to `depth`
// iterations: each slab uploads f and p over its slices with `depth` halo slices below and
// depth + 1 above, iterates on its copy with the copy's ends treated as the image's ends, and writes
// back its own slices of p.  A wrong end value spoils one more slice per iteration (two at the upper
// end in the first, where the forward difference reads the slice above), so the own slices equal
// the whole-image iteration bit for bit: the step needs no sum over the image.  In a round every
// slab starts from the state at the round's start: its lower halo is a device copy of the slices
// below, taken before their update.  A last pass forms u = f - lam div p slab by slab.
size_t rof_host_workspace(const ct_geometry &g) {
    return (size_t)3 * g.nVoxel[0] * g.nVoxel[1] * g.nVoxel[2] * sizeof(float);
}

ct_status rof_host_run(const ct_geometry &g, float *hx, int32_t niter, double lambda, double tau, int32_t depth,
                       float *hp, uint64_t cap, ct_ooc_stats *stats) {
    const auto t_start = std::chrono::steady_clock::now();
    const int nx = (int)g.nVoxel[0], ny = (int)g.nVoxel[1];
    const int64_t nz = g.nVoxel[2];
    const int64_t d = depth;
    const int64_t slice = (int64_t)nx * ny;
    const int64_t nvox = slice * nz;
    const uint64_t sb = (uint64_t)slice * sizeof(float);
    // device: f, px, py, pz and w over the slab with its halos, and the next slab's lower halo of p
    const uint64_t avail = cap > TV_RESERVE ? (cap - TV_RESERVE) / sb : 0;
    if (avail < (uint64_t)(5 * (2 * d + 2) + 3 * d))
        return fail(CT_ERR_CAP, "device memory cap is below one slab slice plus halos and buffers");
    int64_t h = (int64_t)((avail - 3 * d) / 5) - 2 * d - 1;
    h = std::max<int64_t>(1, std::min<int64_t>(h, nz));
    const int64_t nsp = (nz + h - 1) / h;
    h = (nz + nsp - 1) / nsp;
    const int64_t L = std::min<int64_t>(nz, h + 2 * d + 1);  // slices of the largest copy
    ct_ooc_stats st;
    std::memset(&st, 0, sizeof(st));
    st.n_slabs = (int32_t)nsp;
    st.slab_slices = (int32_t)h;
    OwnStream S;
    CT_HIP(hipStreamCreateWithFlags(&S.s, hipStreamNonBlocking));
    DevMem fm, pm[3], wm, sm;
    CT_HIP(CT_MALLOC(&fm.p, (size_t)L * sb));
    for (auto &b : pm) CT_HIP(CT_MALLOC(&b.p, (size_t)L * sb));
    CT_HIP(CT_MALLOC(&wm.p, (size_t)L * sb));
    CT_HIP(CT_MALLOC(&sm.p, (size_t)3 * d * sb));
    float *fb = (float *)fm.p, *wb = (float *)wm.p, *sv = (float *)sm.p;
    float *pb[3] = {(float *)pm[0].p, (float *)pm[1].p, (float *)pm[2].p};
    const hipStream_t s = S.s;
    auto up = [&](float *dst, const float *src, int64_t n_sl) -> ct_status {
        if (n_sl <= 0) return CT_OK;
        CT_HIP(hipMemcpyAsync(dst, src, (size_t)n_sl * sb, hipMemcpyHostToDevice, s));
        st.bytes_h2d += (double)n_sl * sb;
        return CT_OK;
    };
    auto down = [&](float *dst, const float *src, int64_t n_sl) -> ct_status {
        CT_HIP(hipMemcpyAsync(dst, src, (size_t)n_sl * sb, hipMemcpyDeviceToHost, s));
        st.bytes_d2h += (double)n_sl * sb;
        return CT_OK;
    };
    ct_status e = CT_OK;
    bool first = true;
    for (int32_t done = 0; done < niter;) {
        const int64_t k = std::min<int64_t>(d, niter - done);
        for (int64_t n = 0; n < nsp; ++n) {
            const int64_t o0 = n * h, o1 = std::min(nz, o0 + h);
            const int64_t m0 = std::max<int64_t>(0, o0 - d), m1 = std::min(nz, o1 + d + 1), len = m1 - m0;
            if ((e = up(fb, hx + m0 * slice, len)) != CT_OK) return e;
            for (int c = 0; c < 3; ++c) {
                if (first) {  // p = 0 at the start
                    hipLaunchKernelGGL(k_fill_zero, dim3(ew_grid(len * slice)), dim3(EW_THREADS), 0, s, pb[c], len * slice);
                    CT_HIP(hipGetLastError());
                } else {
                    if ((e = up(pb[c] + (o0 - m0) * slice, hp + c * nvox + o0 * slice, m1 - o0)) != CT_OK) return e;
                    if (o0 > m0)
                        CT_HIP(hipMemcpyAsync(pb[c], sv + c * d * slice, (size_t)(o0 - m0) * sb, hipMemcpyDeviceToDevice, s));
                }
                if (n + 1 < nsp) {  // the next slab's lower halo, as it stands at the round's start
                    const int64_t n0 = std::max<int64_t>(0, o1 - d);
                    CT_HIP(hipMemcpyAsync(sv + c * d * slice, pb[c] + (n0 - m0) * slice, (size_t)(o1 - n0) * sb,
                                          hipMemcpyDeviceToDevice, s));
                }
            }
            const dim3 grid((nx + 63) / 64, (ny + 3) / 4, (unsigned)len);
            for (int64_t i = 0; i < k; ++i) {
                hipLaunchKernelGGL(k_rof_w, grid, dim3(256), 0, s, (const float *)fb, pb[0], pb[1], pb[2], wb, nx, ny,
                                   (int)len, (float)(1.0 / lambda));
                hipLaunchKernelGGL(k_rof_p, grid, dim3(256), 0, s, (const float *)wb, pb[0], pb[1], pb[2], nx, ny,
                                   (int)len, (float)tau);
                CT_HIP(hipGetLastError());
            }
            for (int c = 0; c < 3; ++c)
                if ((e = down(hp + c * nvox + o0 * slice, pb[c] + (o0 - m0) * slice, o1 - o0)) != CT_OK) return e;
            CT_HIP(hipStreamSynchronize(s));
        }
        first = false;
        done += (int32_t)k;
        if (tv_verbose()) {
            std::fprintf(stderr, "[ct ooc rof] %d of %d iterations done at %.1f s\n", done, niter,
                         std::chrono::duration<double>(std::chrono::steady_clock::now() - t_start).count());
            std::fflush(stderr);
        }
    }
    // u = f - lam div p: the divergence at a slice reads p there and one slice below, and is the
    // interior form only below the copy's top, so each slab takes one slice either side
    for (int64_t n = 0; n < nsp; ++n) {
        const int64_t o0 = n * h, o1 = std::min(nz, o0 + h);
        const int64_t m0 = std::max<int64_t>(0, o0 - 1), m1 = std::min(nz, o1 + 1), len = m1 - m0;
        if ((e = up(fb, hx + m0 * slice, len)) != CT_OK) return e;
        for (int c = 0; c < 3; ++c) {
            if (niter == 0) {
                hipLaunchKernelGGL(k_fill_zero, dim3(ew_grid(len * slice)), dim3(EW_THREADS), 0, s, pb[c], len * slice);
                CT_HIP(hipGetLastError());
            } else if ((e = up(pb[c], hp + c * nvox + m0 * slice, len)) != CT_OK) {
                return e;
            }
        }
        const dim3 grid((nx + 63) / 64, (ny + 3) / 4, (unsigned)len);
        hipLaunchKernelGGL(k_rof_u, grid, dim3(256), 0, s, fb, pb[0], pb[1], pb[2], nx, ny, (int)len, (float)lambda);
        CT_HIP(hipGetLastError());
        if ((e = down(hx + o0 * slice, fb + (o0 - m0) * slice, o1 - o0)) != CT_OK) return e;
        CT_HIP(hipStreamSynchronize(s));
    }
    st.t_total_s = std::chrono::duration<double>(std::chrono::steady_clock::now() - t_start).count();
    if (stats) *stats = st;
    return CT_OK;
}

}  // namespace ct
