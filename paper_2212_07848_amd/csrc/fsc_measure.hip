// fsc_measure.hip -- density gathers, FP64 state reductions, and the
// structure-factor pipeline S(k) = <|dn(k)|^2> / N of Lulli et al.
// (arXiv:2212.07848, the quantity compared with Eq. 16): real transforms of the
// gathered density, line by line in LDS, and binning of the last transform
// where it lies, with FP64 accumulation.
#include <algorithm>
#include <cmath>
#include <utility>
#include <vector>

#include "fsc_internal.h"

namespace fsc {

template <typename real>
struct cplx {
    real re, im;
};

// ---------------------------------------------------------------------------
// Density gather: the streamed state at x is f_i(x) = f*_i(x - c_i) of the
// stored post-collision buffer; dn = sum_i df_i.  One block = 256 x-values
// of one (y, z) row.
// ---------------------------------------------------------------------------
template <class L, typename real>
__device__ inline void gather_node(const real *src, const Geometry &g, int x, int y, int z,
                                   real (&f)[L::Q]) {
    const int xm = x == 0 ? g.nx - 1 : x - 1, xp = x + 1 == g.nx ? 0 : x + 1;
    const int ym = y == 0 ? g.ny - 1 : y - 1, yp = y + 1 == g.ny ? 0 : y + 1;
    const int zm = z == 0 ? g.nz - 1 : z - 1, zp = z + 1 == g.nz ? 0 : z + 1;
#pragma unroll
    for (int i = 0; i < L::Q; ++i) {
        const int cx = L::c(i, 0), cy = L::c(i, 1), cz = L::c(i, 2);
        const int xs = cx == 1 ? xm : (cx == -1 ? xp : x);
        const int ys = cy == 1 ? ym : (cy == -1 ? yp : y);
        const int zs = cz == 1 ? zm : (cz == -1 ? zp : z);
        f[i] = src[int64_t(i) * g.N + xs + int64_t(g.nx) * (ys + int64_t(g.ny) * zs)];
    }
}

// n(x) = rho0 + dn in double of the rows row0 .. row0 + rows - 1, as a program
// reads it: formed here, the host only receives it (converting 256^3 values on
// the host took longer than moving them).
// (Out float: dn itself.)
template <class L, typename real, typename Out>
__global__ void __launch_bounds__(256) k_density(Geometry g, const real *__restrict__ src, double rho0,
                                                 int64_t row0, Out *__restrict__ out) {
    const int strips = (g.nx + 255) / 256;
    const int64_t r = int(blockIdx.x) / strips, row = row0 + r;
    const int x = (int(blockIdx.x) % strips) * 256 + threadIdx.x;
    if (x >= g.nx) return;
    real f[L::Q];
    gather_node<L, real>(src, g, x, int(row % g.ny), int(row / g.ny), f);
    real dn = real(0);
#pragma unroll
    for (int i = 0; i < L::Q; ++i) dn += f[i];
    if constexpr (sizeof(Out) == 4) out[r * g.nx + x] = dn;
    else out[r * g.nx + x] = rho0 + double(dn);
}

template <typename Out, typename Kernel, typename real>
static hipError_t density_rows(Kernel kernel, const Geometry &g, const real *buf, double rho0, int64_t row0, int64_t rows,
                               Out *out, hipStream_t s) {
    const int64_t blocks = int64_t((g.nx + 255) / 256) * rows;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kernel, dim3(unsigned(blocks)), dim3(256), 0, s, g, buf, rho0, row0, out);
    return hipGetLastError();
}

hipError_t launch_density(const Geometry &g, int precision, const void *buf, double rho0, int64_t row0,
                          int64_t rows, double *out, hipStream_t s) {
    const float *f = static_cast<const float *>(buf);
    const double *d = static_cast<const double *>(buf);
    if (g.D == 2)
        return precision == 0 ? density_rows(k_density<D2Q9, float, double>, g, f, rho0, row0, rows, out, s)
                              : density_rows(k_density<D2Q9, double, double>, g, d, rho0, row0, rows, out, s);
    return precision == 0 ? density_rows(k_density<D3Q19, float, double>, g, f, rho0, row0, rows, out, s)
                          : density_rows(k_density<D3Q19, double, double>, g, d, rho0, row0, rows, out, s);
}

hipError_t launch_deviation(const Geometry &g, const float *buf, float *out, hipStream_t s) {
    const int64_t rows = int64_t(g.ny) * g.nz;
    return g.D == 2 ? density_rows(k_density<D2Q9, float, float>, g, buf, 0.0, 0, rows, out, s)
                    : density_rows(k_density<D3Q19, float, float>, g, buf, 0.0, 0, rows, out, s);
}

// The streamed populations w_i rho0 + df_i(x) in double, layout [i][z][y][x],
// elements e0 .. e0 + n - 1 (shift[i] = w_i rho0, formed by the caller).
struct PopShift {
    double v[19];
};
template <class L, typename real>
__global__ void __launch_bounds__(256) k_streamed(Geometry g, const real *__restrict__ src, PopShift shift,
                                                  int64_t e0, int64_t n, double *__restrict__ out) {
    const int64_t k = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (k >= n) return;
    const int64_t e = e0 + k;
    const int i = int(e / g.N);
    const int64_t s = e - i * g.N, row = s / g.nx;
    const int x = int(s - row * g.nx), y = int(row % g.ny), z = int(row / g.ny);
    const int xs = wrap_any(x - L::c(i, 0), g.nx), ys = wrap_any(y - L::c(i, 1), g.ny),
              zs = wrap_any(z - L::c(i, 2), g.nz);
    out[k] = shift.v[i] + double(src[int64_t(i) * g.N + xs + int64_t(g.nx) * (ys + int64_t(g.ny) * zs)]);
}

hipError_t launch_streamed(const Geometry &g, int precision, const void *buf, const double *shift, int64_t e0,
                           int64_t n, double *out, hipStream_t s) {
    const int64_t blocks = (n + 255) / 256;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    PopShift sh{};
    for (int i = 0; i < (g.D == 2 ? D2Q9::Q : D3Q19::Q); ++i) sh.v[i] = shift[i];
    auto go = [&](auto kernel, auto p) {
        hipLaunchKernelGGL(kernel, dim3(unsigned(blocks)), dim3(256), 0, s, g, p, sh, e0, n, out);
        return hipGetLastError();
    };
    const float *f = static_cast<const float *>(buf);
    const double *d = static_cast<const double *>(buf);
    if (g.D == 2) return precision == 0 ? go(k_streamed<D2Q9, float>, f) : go(k_streamed<D2Q9, double>, d);
    return precision == 0 ? go(k_streamed<D3Q19, float>, f) : go(k_streamed<D3Q19, double>, d);
}

// ---------------------------------------------------------------------------
// Results that the host waits for.  A kernel writes them to pinned memory and
// then stores a sequence number beside them, which the host polls: 7 us from
// launch to answer, where waiting for the stream takes 11.5 and a copy to pinned
// memory 12 more.  Beyond 8 KB the copy is as fast (19 KB: the same).
// ---------------------------------------------------------------------------
// Both go out as system-scope stores, past the caches, so that the sender waits
// for its stores alone: a release fence writes back the XCD's L2 (by every wave of
// a copy, 10 us).
__device__ inline void mail_put(const Mail &mail, int k, double v) {
    __hip_atomic_store(&mail.out[k], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ inline void mail_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// after every wave's mail_wait; one thread
__device__ inline void mail_send(const Mail &mail) {
    __hip_atomic_store(mail.flag, mail.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ void __launch_bounds__(1024) k_mail(const double *__restrict__ src, int n, Mail mail) {
    for (int k = threadIdx.x; k < n; k += 1024) mail_put(mail, k, src[k]);
    mail_wait();
    __syncthreads();
    if (threadIdx.x == 0) mail_send(mail);
}

hipError_t launch_mail(const double *src, int n, const Mail &mail, hipStream_t s) {
    hipLaunchKernelGGL(k_mail, dim3(1), dim3(1024), 0, s, src, n, mail);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// FP64 reductions: sum dn, sum j, min/max n, bad-node count.  A fixed grid of at
// most STAT_BLOCKS blocks strides over rows, or over nodes where a row does not
// fill a block; the last one to finish reduces the partials in a fixed order, so
// the result is deterministic, and sends it to the host.  A call on 64^2 takes
// 15 us, 7.3 of them this launch (17 and 9.1 with one shuffle chain per value; 23 with
// a wait for the stream).
// ---------------------------------------------------------------------------
constexpr int STAT_BLOCKS = 1024;
constexpr int STAT_W = 8;
size_t stats_partials_len() { return size_t(STAT_BLOCKS) * STAT_W; }

__device__ inline double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Reduces acc[STAT_W] over a 256-thread block; thread k < STAT_W returns value k.
// Lanes first share out the values (half of them to each half of the wave, and so
// on), which takes 10 shuffles where reducing one value after the other takes 48,
// half of the launch on small lattices (2 x 4700 cycles of 18800).
__device__ inline double block_reduce_stats(const double (&acc)[STAT_W]) {
    static_assert(STAT_W == 8, "three halvings");
    __shared__ double sh[4][STAT_W];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    auto op = [](double x, double y, int k) { return k == 4 ? fmin(x, y) : (k == 5 ? fmax(x, y) : x + y); };
    const bool h5 = lane & 32, h4 = lane & 16, h3 = lane & 8;
    double v4[4], v2[2];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        v4[j] = op(h5 ? acc[4 + j] : acc[j], __shfl_xor(h5 ? acc[j] : acc[4 + j], 32, 64), (h5 ? 4 : 0) + j);
#pragma unroll
    for (int j = 0; j < 2; ++j)
        v2[j] = op(h4 ? v4[2 + j] : v4[j], __shfl_xor(h4 ? v4[j] : v4[2 + j], 16, 64), (h5 ? 4 : 0) + (h4 ? 2 : 0) + j);
    const int held = lane >> 3;
    double v = op(h3 ? v2[1] : v2[0], __shfl_xor(h3 ? v2[0] : v2[1], 8, 64), held);
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) v = op(v, __shfl_xor(v, o, 64), held);
    __syncthreads();  // a second call reuses sh
    if ((lane & 7) == 0) sh[wv][held] = v;
    __syncthreads();
    const int k = threadIdx.x & (STAT_W - 1);
    return op(op(sh[0][k], sh[1][k], k), op(sh[2][k], sh[3][k], k), k);
}

template <class L, typename real>
__global__ void __launch_bounds__(256) k_stats(Geometry g, const real *__restrict__ src, double rho0,
                                               double n_rho0, double *__restrict__ partials,
                                               int *__restrict__ done, Mail mail) {
    __shared__ bool last;
    double acc[STAT_W] = {0.0, 0.0, 0.0, 0.0, 1e300, -1e300, 0.0, 0.0};
    auto add_node = [&](int x, int y, int z) {
        real f[L::Q];
        gather_node<L, real>(src, g, x, y, z, f);
        double dn = 0.0, j[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < L::Q; ++i) {
            const double v = double(f[i]);
            dn += v;
#pragma unroll
            for (int q = 0; q < 3; ++q) j[q] += double(L::c(i, q)) * v;
        }
        const double n = rho0 + dn;
        acc[0] += dn;
        acc[1] += j[0];
        acc[2] += j[1];
        acc[3] += j[2];
        acc[4] = fmin(acc[4], n);
        acc[5] = fmax(acc[5], n);
        acc[6] += (isfinite(n) && n > 0.0) ? 0.0 : 1.0;
        acc[7] += 1.0;
    };
    if (g.nx < 256) {
        for (int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x; e < g.N; e += int64_t(gridDim.x) * 256) {
            const int row = int(e / g.nx);
            add_node(int(e - int64_t(row) * g.nx), row % g.ny, row / g.ny);
        }
    } else {
        const int rows = g.ny * g.nz;
        for (int row = blockIdx.x; row < rows; row += gridDim.x)
            for (int x = threadIdx.x; x < g.nx; x += 256) add_node(x, row % g.ny, row / g.ny);
    }
    const double mine = block_reduce_stats(acc);
    // partials go to the last block by atomic stores and loads, which pass by
    // the XCDs' L2s, so no cache is written back for them
    if (threadIdx.x < 64) {
        if (threadIdx.x < STAT_W)
            __hip_atomic_store(&partials[blockIdx.x * STAT_W + threadIdx.x], mine, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        mail_wait();
        if (threadIdx.x == 0)
            last = __hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == int(gridDim.x) - 1;
    }
    __syncthreads();
    if (!last) return;
    double t[STAT_W] = {0.0, 0.0, 0.0, 0.0, 1e300, -1e300, 0.0, 0.0};
    for (int b = threadIdx.x; b < int(gridDim.x); b += 256) {
        double *p = partials + b * STAT_W;
        for (int k = 0; k < STAT_W; ++k) {
            const double v = __hip_atomic_load(&p[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            t[k] = (k == 4) ? fmin(t[k], v) : (k == 5 ? fmax(t[k], v) : t[k] + v);
        }
    }
    const double all = block_reduce_stats(t);
    if (threadIdx.x >= 64) return;
    if (threadIdx.x < STAT_W) mail_put(mail, threadIdx.x, threadIdx.x == 0 ? n_rho0 + all : all);
    mail_wait();
    if (threadIdx.x == 0) {
        __hip_atomic_store(done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        mail_send(mail);
    }
}

hipError_t launch_stats(const Geometry &g, int precision, const void *buf, double rho0,
                        double *partials, int *done, const Mail &mail, hipStream_t s) {
    const int64_t want = g.nx < 256 ? (g.N + 255) / 256 : int64_t(g.ny) * g.nz;
    const unsigned nb = unsigned(std::min<int64_t>(want, STAT_BLOCKS));
    auto go = [&](auto kernel, auto p) {
        hipLaunchKernelGGL(kernel, dim3(nb), dim3(256), 0, s, g, p, rho0, double(g.N) * rho0, partials, done, mail);
        return hipGetLastError();
    };
    const float *f = static_cast<const float *>(buf);
    const double *d = static_cast<const double *>(buf);
    if (g.D == 2) return precision == 0 ? go(k_stats<D2Q9, float>, f) : go(k_stats<D2Q9, double>, d);
    return precision == 0 ? go(k_stats<D3Q19, float>, f) : go(k_stats<D3Q19, double>, d);
}

// ---------------------------------------------------------------------------
// Structure factor.  One sample of a lattice is
//   rows: density gather and transform along x.  The density is real, so two
//     rows share one complex transform and only kx = 0 .. nx/2 is kept; a block
//     takes 2 lc rows and writes the half spectrum with y (the next axis)
//     contiguous, [kx][z][y], in pieces of 2 lc values;
//   mid (3D): transform along y of lc lines (kx, z .. z + lc - 1), written
//     [kx][ky][z];
//   last: transform along the last axis of lc lines and, from LDS, the bins, the
//     moments of L(t) and the recorded modes; the spectrum goes nowhere else.
// The modes with 0 < kx < nx/2 stand for themselves and
// their mirror images -k, which have the same |X|^2.
//
// Traffic of a 2D FP32 sample: 36 B per node read, 4 written, 4 read.  (Complex
// transforms with a rotation pass per axis and a binning pass moved 36 + 88.)
// Measured, before and now, us: 4096^2 FP32 840 and 395 (rows 207: 2.9 TB/s of
// populations; last 190 to 310); 256^3 FP32 2000 and 410; 750 x 487 FP64 480 and
// 52; 16 fields of 128^2 1390 and 20.
// ---------------------------------------------------------------------------
// Lines in LDS: element i of line l at l sk_stride(m) + sk_pad(i).  One pad
// element in eight keeps the strided accesses of the radix-8 passes off each
// other's banks; the odd stride does it for accesses across lines.
__host__ __device__ inline int sk_stride(int m) { return m + (m >> 3) + 1; }
__device__ inline int sk_pad(int i) { return i + (i >> 3); }

constexpr int SK_HELD = 16;  // complex values a thread holds in one pass

template <typename real>
__device__ __forceinline__ cplx<real> c_mul(cplx<real> a, cplx<real> b) {
    return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <typename real>
__device__ __forceinline__ cplx<real> c_add(cplx<real> a, cplx<real> b) {
    return {a.re + b.re, a.im + b.im};
}
template <typename real>
__device__ __forceinline__ cplx<real> c_sub(cplx<real> a, cplx<real> b) {
    return {a.re - b.re, a.im - b.im};
}

// X_k = sum_r v_r exp(-2 pi i r k / R) in place
template <typename real>
__device__ __forceinline__ void dft_r(cplx<real> (&v)[2]) {
    const cplx<real> t = v[0];
    v[0] = c_add(t, v[1]);
    v[1] = c_sub(t, v[1]);
}
template <typename real>
__device__ __forceinline__ void dft_r(cplx<real> (&v)[4]) {
    const cplx<real> s = c_add(v[0], v[2]), d = c_sub(v[0], v[2]);
    const cplx<real> p = c_add(v[1], v[3]), q = c_sub(v[1], v[3]);
    v[0] = c_add(s, p);
    v[2] = c_sub(s, p);
    v[1] = {d.re + q.im, d.im - q.re};
    v[3] = {d.re - q.im, d.im + q.re};
}
template <typename real>
__device__ __forceinline__ void dft_r(cplx<real> (&v)[8]) {
    cplx<real> e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft_r(e);
    dft_r(o);
    constexpr real h = real(0.70710678118654752440);
    const cplx<real> o1 = {(o[1].re + o[1].im) * h, (o[1].im - o[1].re) * h};
    const cplx<real> o2 = {o[2].im, -o[2].re};
    const cplx<real> o3 = {(o[3].im - o[3].re) * h, -(o[3].re + o[3].im) * h};
    v[0] = c_add(e[0], o[0]);
    v[4] = c_sub(e[0], o[0]);
    v[1] = c_add(e[1], o1);
    v[5] = c_sub(e[1], o1);
    v[2] = c_add(e[2], o2);
    v[6] = c_sub(e[2], o2);
    v[3] = c_add(e[3], o3);
    v[7] = c_sub(e[3], o3);
}

// One radix-R Stockham pass over lines of m = 2^logm (2^nsl: product of the
// radices before): every value is in a register between the two barriers, so
// the pass works in place.  Needs lines * m <= SK_HELD * blockDim.x.
template <typename real, int R>
__device__ __forceinline__ void sk_pass(cplx<real> *a, int lines, int m, int logm, int nsl,
                               const cplx<real> *__restrict__ tw) {
    constexpr int LR = R == 8 ? 3 : (R == 4 ? 2 : 1), M = SK_HELD / R;
    const int lper = logm - LR, per = 1 << lper, total = lines << lper, ls = sk_stride(m);
    cplx<real> v[M][R];
#pragma unroll
    for (int q = 0; q < M; ++q) {
        const int id = threadIdx.x + q * blockDim.x;
        if (id < total) {
            const int j = id & (per - 1);
            const cplx<real> *b = a + (id >> lper) * ls;
#pragma unroll
            for (int r = 0; r < R; ++r) v[q][r] = b[sk_pad(j + (r << lper))];
            if (nsl > 0) {
                const int k = (j & ((1 << nsl) - 1)) << (lper - nsl);
#pragma unroll
                for (int r = 1; r < R; ++r) v[q][r] = c_mul(v[q][r], tw[k * r]);
            }
            dft_r(v[q]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < M; ++q) {
        const int id = threadIdx.x + q * blockDim.x;
        if (id < total) {
            const int j = id & (per - 1), k = j & ((1 << nsl) - 1);
            cplx<real> *b = a + (id >> lper) * ls;
            const int o = ((j >> nsl) << (nsl + LR)) + k;
#pragma unroll
            for (int r = 0; r < R; ++r) b[sk_pad(o + (r << nsl))] = v[q][r];
        }
    }
    __syncthreads();
}

template <typename real>
__device__ __forceinline__ void sk_pow2(cplx<real> *a, int lines, int m, int logm, const cplx<real> *__restrict__ tw) {
    int nsl = 0;
    for (; logm - nsl >= 3; nsl += 3) sk_pass<real, 8>(a, lines, m, logm, nsl, tw);
    if (logm - nsl == 2) sk_pass<real, 4>(a, lines, m, logm, nsl, tw);
    else if (logm - nsl == 1) sk_pass<real, 2>(a, lines, m, logm, nsl, tw);
}

// Transforms `lines` lines of n values in LDS, in place, natural order in and
// out.  Starts and ends at a barrier.  Table `tab` (see sk_table):
//   n a power of two (m = n): radix-8 passes;
//   other n: the chirp transform (Bluestein) over m = 2^logm >= 2n - 1, jk =
//     (j^2 + k^2 - (k - j)^2)/2: multiply by the chirp, convolve by a transform,
//     a product with the chirp's spectrum and an inverse transform, multiply by
//     the chirp.  O(m log m) where the direct sum is O(n^2): at 750 x 487 in
//     FP64 a sample's transforms took 458 us as direct sums;
//   logm < 0 (FP64 lines beyond 4096 whose chirp form does not fit the LDS): the
//     direct sum.
template <typename real>
__device__ __forceinline__ void sk_fft(cplx<real> *a, int lines, const SkAxis &x, const cplx<real> *__restrict__ tab) {
    const int n = x.n, m = x.m, ls = sk_stride(m);
    __syncthreads();
    if (n == 1) return;
    if (x.logm < 0) {
        cplx<real> acc[SK_HELD];
#pragma unroll
        for (int q = 0; q < SK_HELD; ++q) {
            const int id = threadIdx.x + q * blockDim.x;
            if (id < lines * n) {
                const int k = id % n;
                const cplx<real> *b = a + (id / n) * ls;
                real sr = real(0), si = real(0);
                int idx = 0;
                for (int j = 0; j < n; ++j) {
                    const cplx<real> w = tab[idx], v = b[sk_pad(j)];
                    sr += v.re * w.re - v.im * w.im;
                    si += v.re * w.im + v.im * w.re;
                    idx += k;
                    if (idx >= n) idx -= n;
                }
                acc[q] = {sr, si};
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < SK_HELD; ++q) {
            const int id = threadIdx.x + q * blockDim.x;
            if (id < lines * n) a[(id / n) * ls + sk_pad(id % n)] = acc[q];
        }
        __syncthreads();
        return;
    }
    const bool chirped = n != m;
    const cplx<real> *chirp = tab + m, *bhat = tab + m + n;
    for (int half = 0; half < (chirped ? 2 : 1); ++half) {
        if (chirped) {
            for (int id = threadIdx.x; id < lines << x.logm; id += blockDim.x) {
                const int j = id & (m - 1);
                cplx<real> *b = a + (id >> x.logm) * ls + sk_pad(j);
                if (half == 0) {
                    *b = j < n ? c_mul(*b, chirp[j]) : cplx<real>{real(0), real(0)};
                } else {  // the inverse transform, as the conjugate of a forward one
                    const cplx<real> v = c_mul(*b, bhat[j]);
                    *b = {v.re, -v.im};
                }
            }
            __syncthreads();
        }
        sk_pow2<real>(a, lines, m, x.logm, tab);
    }
    if (!chirped) return;
    for (int id = threadIdx.x; id < lines << x.logm; id += blockDim.x) {
        const int j = id & (m - 1);
        if (j < n) {
            cplx<real> *b = a + (id >> x.logm) * ls + sk_pad(j);
            *b = c_mul(cplx<real>{b->re, -b->im}, chirp[j]);
        }
    }
    __syncthreads();
}

// Device part of a transform table: tw[k] = exp(-2 pi i k / m), k < m, then for
// the chirp form chirp[j] = exp(-pi i j^2 / n), j < n (both exactly reduced);
// the chirp's spectrum behind them comes from the host.  `zero` words are
// cleared by the same launch.
template <typename real>
__global__ void __launch_bounds__(256) k_sk_table(cplx<real> *__restrict__ tab, SkAxis x,
                                                  uint32_t *__restrict__ zero, int64_t words) {
    const int64_t k = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (k < x.m) {
        double s, c;
        sincospi(-2.0 * double(k) / double(x.m), &s, &c);
        tab[k] = {real(c), real(s)};
    } else if (x.logm >= 0 && x.m != x.n && k < x.m + x.n) {
        const int64_t j = k - x.m;
        double s, c;
        sincospi(-double((j * j) % (2 * x.n)) / double(x.n), &s, &c);
        tab[k] = {real(c), real(s)};
    }
    if (k < words) zero[k] = 0u;
}

// floor(sqrt(v)) of 0 <= v < 2^29
__device__ inline int isqrt(int v) {
    int b = int(sqrtf(float(v)));
    while (b * b > v) --b;
    while ((b + 1) * (b + 1) <= v) ++b;
    return b;
}
// shell round(sqrt(v)): (b - 1/2)^2 <= v < (b + 1/2)^2, that is b^2 - b < v <= b^2 + b
__device__ inline int shell_of(int v) {
    const int b = isqrt(v);
    return v > b * b + b ? b + 1 : b;
}

__device__ inline int signed_mode(int q, int n) { return q <= n / 2 ? q : q - n; }

// Closes one sample: the time series' row gets (step, L) with L = 2 pi sum P /
// sum |k| P, the moments are cleared, the row counter advances.  One thread,
// after every block of the replica has added its share.
__device__ __forceinline__ void sk_close(const MeasRep &m, uint64_t step) {
    if (m.t.mom != nullptr) {
        const double p0 = __hip_atomic_load(&m.t.mom[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const double p1 = __hip_atomic_load(&m.t.mom[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int row = m.series_n[0];
        if (m.t.series != nullptr && row < m.t.series_cap) {
            double *s = m.t.series + size_t(row) * (2 + m.t.n_rad);
            s[0] = double(step);
            s[1] = p1 > 0.0 ? 2.0 * M_PI * p0 / p1 : 0.0;
        }
        __hip_atomic_store(&m.t.mom[0], 0.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&m.t.mom[1], 0.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        m.series_n[0] = row + 1;
    }
}

// Bins of `lines` transformed lines in LDS.  Line l holds the modes (kx, ky, kz)
// of its own last component, element i = signed mode i of the last axis (length
// n); the others are (kx, ky) = (o, i0 + l) in 3D and kx = i0 + l in 2D.
//
// Along a line the shell grows with |k_last|, so every shell is a range of it
// whose ends are integer square roots: the lanes go over (line, shell) pairs
// and sum their few modes in registers, instead of one shell lookup and two
// contended atomics per mode.  `wnd` [2][W] collects the lines' shells in LDS
// (nullptr: one line, added to memory directly).  srow, mrow: this sample's rows of
// the time series and of the mode recorder.
template <typename real>
__device__ __forceinline__ void sk_bin(const MeasRep &m, const cplx<real> *a, int ls, int lines, int o, int i0,
                              double *wnd, int srow, int mrow) {
    const Geometry &g = m.g;
    const BinTargets &t = m.t;
    const bool d3 = g.D == 3;
    const int n = d3 ? g.nz : g.ny, half = n / 2, nt = blockDim.x;
    const double invN = m.invN;
    auto other = [&](int l, int &kx, int &ky) {
        kx = d3 ? o : i0 + l;
        ky = d3 ? signed_mode(i0 + l, g.ny) : 0;
    };
    auto weight = [&](int kx) { return kx == 0 || 2 * kx == g.nx ? 1.0 : 2.0; };
    auto power = [&](int l, int i) {
        const cplx<real> v = a[l * ls + sk_pad(i)];
        return (double(v.re) * double(v.re) + double(v.im) * double(v.im)) * invN;
    };
    double *srow_bins = t.mom && t.series && srow < t.series_cap ? t.series + size_t(srow) * (2 + t.n_rad) + 2 : nullptr;
    auto add_shell = [&](int b, double s, double q) {
        unsafeAtomicAdd(&t.rad_sum[b], s);
        if (t.rad_sq) unsafeAtomicAdd(&t.rad_sq[b], q);
        if (srow_bins) unsafeAtomicAdd(&srow_bins[b], s);
    };
    if (t.n_rad > 0) {
        // the other components' |k|^2 of the lines: kx grows with l, |ky| grows up
        // to ny / 2 and falls from there
        const int i1 = i0 + lines - 1;
        int lo2, hi2;
        if (d3) {
            const int p = abs(signed_mode(i0, g.ny)), q = abs(signed_mode(i1, g.ny)), top = g.ny / 2;
            const int lo = min(p, q), hi = i0 <= top && top <= i1 ? top : max(p, q);
            lo2 = o * o + lo * lo;
            hi2 = o * o + hi * hi;
        } else {
            lo2 = i0 * i0;
            hi2 = i1 * i1;
        }
        const int blo = shell_of(lo2), W = shell_of(hi2 + half * half) - blo + 1;
        if (wnd) {
            for (int k = threadIdx.x; k < 2 * W; k += nt) wnd[k] = 0.0;
            __syncthreads();
        }
        for (int id = threadIdx.x; id < lines * W; id += nt) {
            const int l = id / W, b = blo + id % W;
            int kx, ky;
            other(l, kx, ky);
            const int base = kx * kx + ky * ky;
            const int top = b * b + b - base;  // |k_last|^2 <= top and > top - 2b
            if (b == 0 || top < 0) continue;
            const int hi = min(half, isqrt(top));
            const int lo = top - 2 * b < 0 ? 0 : isqrt(top - 2 * b) + 1;
            double s = 0.0, q = 0.0;
            for (int k = lo; k <= hi; ++k) {
                const double p = power(l, k);
                s += p;
                q += p * p;
                if (k > 0 && 2 * k != n) {
                    const double r = power(l, n - k);
                    s += r;
                    q += r * r;
                }
            }
            if (s == 0.0) continue;
            const double w = weight(kx);
            if (wnd) {
                atomicAdd(&wnd[b - blo], w * s);
                atomicAdd(&wnd[W + b - blo], w * q);
            } else {
                add_shell(b, w * s, w * q);
            }
        }
        if (wnd) {
            __syncthreads();
            for (int k = threadIdx.x; k < W; k += nt)
                if (wnd[k] != 0.0 || wnd[W + k] != 0.0) add_shell(blo + k, wnd[k], wnd[W + k]);
        }
    }
    if (t.axis_sum) {
        auto add_axis = [&](int d, int k, double w, double p) {
            unsafeAtomicAdd(&t.axis_sum[d * t.n_axis + abs(k)], w * p);
            unsafeAtomicAdd(&t.axis_sq[d * t.n_axis + abs(k)], w * p * p);
        };
        // (from the other end of the block: beside the shells' flush, not after it)
        const int back = nt - 1 - int(threadIdx.x);
        for (int l = back; l < lines; l += nt) {  // modes with no last component
            int kx, ky;
            other(l, kx, ky);
            if (ky == 0 && kx != 0) add_axis(0, kx, weight(kx), power(l, 0));
            if (kx == 0 && ky != 0) add_axis(1, ky, 1.0, power(l, 0));
        }
        if ((!d3 || o == 0) && i0 == 0)  // line 0 has no other component
            for (int i = ((back + nt / 2) & (nt - 1)) + 1; i < n; i += nt)
                add_axis(g.D - 1, signed_mode(i, n), 1.0, power(0, i));
    }
    if (t.mom) {
        const double ux = 2.0 * M_PI / g.nx, uy = 2.0 * M_PI / g.ny, uz = 2.0 * M_PI / n;
        double sp = 0.0, sk = 0.0;
        for (int id = threadIdx.x; id < lines * n; id += nt) {
            const int l = id / n, i = id % n;
            int kx, ky;
            other(l, kx, ky);
            const int kl = signed_mode(i, n);
            if (kx == 0 && ky == 0 && kl == 0) continue;
            const double p = weight(kx) * power(l, i);
            const double x = ux * kx, y = uy * ky, z = uz * kl;
            sp += p;
            sk += sqrt(x * x + y * y + z * z) * p;
        }
        sp = wave_sum(sp);
        sk = wave_sum(sk);
        __shared__ double red[2][16];
        if ((threadIdx.x & 63) == 0) {
            red[0][threadIdx.x >> 6] = sp;
            red[1][threadIdx.x >> 6] = sk;
        }
        __syncthreads();
        if (threadIdx.x < 2) {
            double v = 0.0;
            for (int w = 0; w < nt >> 6; ++w) v += red[threadIdx.x][w];
            unsafeAtomicAdd(&t.mom[threadIdx.x], v);
        }
    }
    if (mrow >= 0 && mrow < m.modes_cap) {
        // amplitudes of the modes 1 .. nm along each axis, row [D][nm][2]
        double *row = m.modes + size_t(mrow) * g.D * m.modes_nm * 2;
        auto put = [&](int d, int k, int l, int i) {
            const cplx<real> v = a[l * ls + sk_pad(i)];
            row[(d * m.modes_nm + k - 1) * 2] = double(v.re);
            row[(d * m.modes_nm + k - 1) * 2 + 1] = double(v.im);
        };
        for (int l = threadIdx.x; l < lines; l += nt) {
            int kx, ky;
            other(l, kx, ky);
            if (ky == 0 && kx >= 1 && kx <= m.modes_nm) put(0, kx, l, 0);
            if (d3 && kx == 0 && ky >= 1 && ky <= m.modes_nm) put(1, ky, l, 0);
        }
        if ((!d3 || o == 0) && i0 == 0)
            for (int k = threadIdx.x + 1; k <= m.modes_nm; k += nt) put(g.D - 1, k, 0, k);
    }
}

// Half spectra of two rows from the transform of (row 0) + i (row 1).
template <typename real>
__device__ __forceinline__ void sk_unpack(const cplx<real> *line, int n, int k, cplx<real> &r0, cplx<real> &r1) {
    const cplx<real> p = line[sk_pad(k)], q = line[sk_pad(k == 0 ? 0 : n - k)];
    constexpr real h = real(0.5);
    r0 = {(p.re + q.re) * h, (p.im - q.im) * h};
    r1 = {(p.im + q.im) * h, (q.re - p.re) * h};
}

// the rows y0, y0 + 1, .. of plane z as packed lines; val(x, y, z) is the field
template <typename T, class Val>
__device__ __forceinline__ void sk_load_rows(const Geometry &g, int y0, int z, int lines, int ls, cplx<T> *a, Val val) {
    for (int id = threadIdx.x; id < lines * g.nx; id += blockDim.x) {
        const int l = id / g.nx, x = id % g.nx, y = y0 + 2 * l;
        a[l * ls + sk_pad(x)] = {T(val(x, y, z)), y + 1 < g.ny ? T(val(x, y + 1, z)) : T(0)};
    }
}

// In the three passes real is the type of the spectra in memory, T that of the
// lines in LDS (double where the axis is wide).
template <typename T, typename real, class Val>
__device__ __forceinline__ void sk_rows_block(const MeasRep &m, int blk, unsigned char *smem, Val val) {
    cplx<T> *a = reinterpret_cast<cplx<T> *>(smem);
    const Geometry &g = m.g;
    const int lc = m.lc[0], per = (g.ny + 2 * lc - 1) / (2 * lc);
    const int z = blk / per, y0 = (blk % per) * 2 * lc;
    const int lines = min(lc, (g.ny - y0 + 1) / 2), ls = sk_stride(m.ax[0].m);
    sk_load_rows<T>(g, y0, z, lines, ls, a, val);
    sk_fft<T>(a, lines, m.ax[0], static_cast<const cplx<T> *>(m.tab[0]));
    cplx<real> *out = static_cast<cplx<real> *>(m.cbuf);
    const int hx = g.nx / 2 + 1;
    for (int id = threadIdx.x; id < hx * lines; id += blockDim.x) {
        const int l = id % lines, k = id / lines, y = y0 + 2 * l;
        cplx<T> r0, r1;
        sk_unpack<T>(a + l * ls, g.nx, k, r0, r1);
        cplx<real> *o = out + (int64_t(k) * g.nz + z) * g.ny + y;
        o[0] = {real(r0.re), real(r0.im)};
        if (y + 1 < g.ny) o[1] = {real(r1.re), real(r1.im)};
    }
}

// transform of `lines` contiguous lines of `in` into LDS
template <typename T, typename real>
__device__ __forceinline__ void sk_lines(const cplx<real> *__restrict__ in, int lines, const SkAxis &x, const void *tab,
                                cplx<T> *a) {
    const int ls = sk_stride(x.m);
    for (int id = threadIdx.x; id < lines * x.n; id += blockDim.x)
        a[(id / x.n) * ls + sk_pad(id % x.n)] = {T(in[id].re), T(in[id].im)};
    sk_fft<T>(a, lines, x, static_cast<const cplx<T> *>(tab));
}

// 3D: transform along y of lines (kx, z)
template <typename T, typename real>
__device__ __forceinline__ void sk_mid_block(const MeasRep &m, int blk, unsigned char *smem) {
    cplx<T> *a = reinterpret_cast<cplx<T> *>(smem);
    const Geometry &g = m.g;
    const int lc = m.lc[1], per = (g.nz + lc - 1) / lc;
    const int kx = blk / per, z0 = (blk % per) * lc, lines = min(lc, g.nz - z0), ls = sk_stride(m.ax[1].m);
    sk_lines<T>(static_cast<const cplx<real> *>(m.cbuf) + (int64_t(kx) * g.nz + z0) * g.ny, lines, m.ax[1], m.tab[1], a);
    cplx<real> *out = static_cast<cplx<real> *>(m.ctmp) + int64_t(kx) * g.ny * g.nz + z0;
    for (int id = threadIdx.x; id < lines * g.ny; id += blockDim.x) {
        const int l = id % lines, k = id / lines;
        const cplx<T> v = a[l * ls + sk_pad(k)];
        out[int64_t(k) * g.nz + l] = {real(v.re), real(v.im)};
    }
}

template <typename T, typename real>
__device__ __forceinline__ void sk_last_block(const MeasRep &m, int blk, unsigned char *smem) {
    const Geometry &g = m.g;
    const bool d3 = g.D == 3;
    const SkAxis &x = m.ax[d3 ? 2 : 1];
    const int inner = d3 ? g.ny : g.nx / 2 + 1, lc = m.lc[2];
    const int per = (inner + lc - 1) / lc, o = blk / per, i0 = (blk % per) * lc;
    const int lines = min(lc, inner - i0), ls = sk_stride(x.m);
    cplx<T> *a = reinterpret_cast<cplx<T> *>(smem);
    double *wnd = lc > 1 ? reinterpret_cast<double *>(smem + sk_line_bytes(sizeof(cplx<T>), lc, x.m)) : nullptr;
    const cplx<real> *in = static_cast<const cplx<real> *>(d3 ? m.ctmp : m.cbuf);
    // (asked for here, ahead of the transform)
    const int srow = m.t.mom && m.t.series ? m.t.series_n[0] : 0;
    const int mrow = m.modes_cap > 0 ? m.modes_n[0] - 1 : 0;  // k_sk_rows counted this sample
    sk_lines<T>(in + (int64_t(o) * inner + i0) * x.n, lines, x, m.tab[d3 ? 2 : 1], a);
    sk_bin<T>(m, a, ls, lines, o, i0, wnd, srow, mrow);
}

// ---------------------------------------------------------------------------
// One sample of every replica of an ensemble in two or three launches, whatever
// the number of replicas.  Each launch is a flat grid over the replicas: block b
// belongs to the replica r with pre[r] <= b < pre[r + 1] (a prefix table per
// kind of work).
// ---------------------------------------------------------------------------
template <class L, typename real>
__device__ inline auto sk_density(const MeasRep &m, int par) {
    const real *src = static_cast<const real *>(m.buf[par]);
    return [&m, src](int x, int y, int z) {
        real f[L::Q];
        gather_node<L, real>(src, m.g, x, y, z, f);
        real dn = real(0);
#pragma unroll
        for (int i = 0; i < L::Q; ++i) dn += f[i];
        return dn;
    };
}

// WIDE: some replica's lines are transformed in doubles (real is float); a kernel
// of its own, so that the others keep their registers.
template <class L, typename real, bool WIDE>
__global__ void __launch_bounds__(1024) k_sk_rows(const MeasRep *__restrict__ mr, const int *__restrict__ pre,
                                                  int nrep, int par, uint64_t *__restrict__ step_base,
                                                  uint64_t advance) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    if (blockIdx.x == 0 && threadIdx.x == 0 && advance) step_base[0] += advance;
    const int r = owner_of(pre, nrep, int(blockIdx.x));
    // the recorder's row counter, which nothing else in this launch reads
    if (threadIdx.x == 0 && int(blockIdx.x) == pre[r] && mr[r].modes_cap > 0) mr[r].modes_n[0] += 1;
    const int blk = int(blockIdx.x) - pre[r];
    if (WIDE && mr[r].ax[0].wide) sk_rows_block<double, real>(mr[r], blk, smem_raw, sk_density<L, real>(mr[r], par));
    else sk_rows_block<real, real>(mr[r], blk, smem_raw, sk_density<L, real>(mr[r], par));
}

template <typename real, bool WIDE>
__global__ void __launch_bounds__(1024) k_sk_mid(const MeasRep *__restrict__ mr, const int *__restrict__ pre,
                                                 int nrep) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int r = owner_of(pre, nrep, int(blockIdx.x)), blk = int(blockIdx.x) - pre[r];
    if (WIDE && mr[r].ax[1].wide) sk_mid_block<double, real>(mr[r], blk, smem_raw);
    else sk_mid_block<real, real>(mr[r], blk, smem_raw);
}

// The replica's last block to finish closes the sample (series row, counter).
// What it reads of the others went through atomics and is read back by atomics,
// so every wave only has to see its own ones done before the block counts
// itself; a device-wide fence writes back the L2 of the block's XCD, which cost
// 40 us of a launch of 544 blocks.
__device__ __forceinline__ void sk_finish(const MeasRep &m, int blocks, const uint64_t *step_base,
                                          uint32_t step_off) {
    if (m.t.mom == nullptr) return;
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x != 0) return;
    if (blocks > 1 &&
        __hip_atomic_fetch_add(m.done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != blocks - 1)
        return;
    sk_close(m, step_base[0] + step_off);
    if (blocks > 1) __hip_atomic_store(m.done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename real, bool WIDE>
__global__ void __launch_bounds__(1024) k_sk_last(const MeasRep *__restrict__ mr, const int *__restrict__ pre,
                                                  int nrep, const uint64_t *__restrict__ step_base,
                                                  uint32_t step_off) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int r = owner_of(pre, nrep, int(blockIdx.x));
    const int blk = int(blockIdx.x) - pre[r];
    if (WIDE && mr[r].ax[mr[r].g.D - 1].wide) sk_last_block<double, real>(mr[r], blk, smem_raw);
    else sk_last_block<real, real>(mr[r], blk, smem_raw);
    sk_finish(mr[r], pre[r + 1] - pre[r], step_base, step_off);
}

// ---------------------------------------------------------------------------
// Host side of the plan.
// ---------------------------------------------------------------------------
constexpr size_t SK_LDS = 160 * 1024 - 1024;  // dynamic part

static int sk_cap(size_t csz) { return csz == 8 ? 16384 : 8192; }  // lines x m of one block, in values of csz bytes

// The chirp form takes doubles, of FP32 data too, as far as they fit the LDS (sides
// up to 4096).  In floats its two transforms and three products with rounded tables
// lose a relative 2e-7 of every |X|^2 (white fields of side 48 to 4100; direct FP32
// sums 1e-9 to 7e-8) and leave 4 to 8 times the noise of direct sums where a spectrum
// is steep.  A sample of 100^2 takes 17.9 us so and 17.0 in floats, 1000^2 60 and 66,
// 3000^2 631 and 443, 100^3 83 and 70 (direct sums: 29, 1833, 58100, 440).  Beyond 4096 direct sums are the
// noisier ones (0.2 sqrt(n) of a rounding, the chirp 2.4), and it stays in floats, with
// the loss taken out (root_loss).
SkAxis sk_axis(int n, int precision) {
    SkAxis x{n, 1, 0, 0};
    const bool pow2 = (n & (n - 1)) == 0;
    while (x.m < (pow2 ? n : 2 * n - 1)) x.m <<= 1;
    while ((1 << x.logm) < x.m) ++x.logm;
    x.wide = precision == 0 && !pow2 && x.m <= sk_cap(16);
    if (x.m > sk_cap(sk_value_bytes(precision, x))) x = SkAxis{n, n, -1, 0};
    return x;
}

size_t sk_table_len(const SkAxis &x) { return size_t(x.m) + (x.logm >= 0 && x.m != x.n ? size_t(x.n) + x.m : 0); }

// Spectrum of the convolution kernel of the chirp form, exp(+pi i j^2 / n) at j
// and m - j, over m points and divided by m (the inverse transform's factor).
static void chirp_spectrum(const SkAxis &x, std::vector<double> &re, std::vector<double> &im) {
    const int n = x.n, m = x.m;
    re.assign(size_t(m), 0.0);
    im.assign(size_t(m), 0.0);
    for (int64_t j = 0; j < n; ++j) {
        const double ang = M_PI * double((j * j) % (2 * n)) / double(n);
        re[size_t(j)] = std::cos(ang) / m;
        im[size_t(j)] = std::sin(ang) / m;
        if (j > 0) {
            re[size_t(m - j)] = re[size_t(j)];
            im[size_t(m - j)] = im[size_t(j)];
        }
    }
    // radix-2, decimation in frequency, then bit reversal
    std::vector<double> c(size_t(m / 2) + 1), s(size_t(m / 2) + 1);
    for (int k = 0; k < m / 2; ++k) {
        c[size_t(k)] = std::cos(2.0 * M_PI * k / m);
        s[size_t(k)] = -std::sin(2.0 * M_PI * k / m);
    }
    for (int len = m; len >= 2; len >>= 1)
        for (int b = 0; b < m; b += len)
            for (int k = 0; k < len / 2; ++k) {
                const size_t p = size_t(b + k), q = p + size_t(len / 2), w = size_t(k) * size_t(m / len);
                const double dr = re[p] - re[q], di = im[p] - im[q];
                re[p] += re[q];
                im[p] += im[q];
                re[q] = dr * c[w] - di * s[w];
                im[q] = dr * s[w] + di * c[w];
            }
    for (int i = 0, j = 0; i < m; ++i) {
        if (i < j) {
            std::swap(re[size_t(i)], re[size_t(j)]);
            std::swap(im[size_t(i)], im[size_t(j)]);
        }
        int bit = m >> 1;
        for (; bit && (j & bit); bit >>= 1) j ^= bit;
        j ^= bit;
    }
}

// Power left, on average over the inputs, of a chirp transform with tables rounded to
// floats (1 - 1.2e-7 beyond 4096 points; exact arithmetic on the same tables agrees to
// 4e-9): the mean |root|^2 over each pass, the chirp's twice and its spectrum's.
static double root_loss(const SkAxis &x, const std::vector<double> &re, const std::vector<double> &im) {
    auto sq = [](double a, double b) { return double(float(a)) * float(a) + double(float(b)) * float(b); };
    auto root = [&](int64_t k) { return sq(std::cos(2.0 * M_PI * double(k) / x.m), std::sin(2.0 * M_PI * double(k) / x.m)); };
    double fft = 1.0;
    for (int nsl = 0; nsl < x.logm;) {
        const int lr = std::min(3, x.logm - nsl), R = 1 << lr;
        double sum = 0.0;
        for (int64_t k = 0; nsl > 0 && k < (int64_t(1) << nsl); ++k)
            for (int r = 1; r < R; ++r) sum += root((k << (x.logm - lr - nsl)) * r);
        if (nsl > 0) fft *= (1.0 + sum / double(1 << nsl)) / R;
        if (lr == 3) fft *= 1.0 + (sq(std::sqrt(0.5), std::sqrt(0.5)) - 1.0) / 4.0;  // two of the eight
        nsl += lr;
    }
    double chirp = 0.0, spec = 0.0, exact = 0.0;
    for (int64_t j = 0; j < x.n; ++j) {
        const double a = M_PI * double((j * j) % (2 * x.n)) / x.n;
        chirp += sq(std::cos(a), std::sin(a)) / x.n;
    }
    for (size_t k = 0; k < re.size(); ++k) {
        spec += sq(re[k], im[k]);
        exact += re[k] * re[k] + im[k] * im[k];
    }
    return fft * fft * chirp * chirp * spec / exact;
}

hipError_t sk_table(int precision, const SkAxis &x, void *tab, void *zero, int64_t zero_words, hipStream_t s) {
    const int64_t n = std::max(int64_t(sk_table_len(x)), zero_words);
    const dim3 nb(unsigned((n + 255) / 256));
    const size_t csz = sk_value_bytes(precision, x);
    if (csz == 8)
        hipLaunchKernelGGL(k_sk_table<float>, nb, dim3(256), 0, s, static_cast<cplx<float> *>(tab), x,
                           static_cast<uint32_t *>(zero), zero_words);
    else
        hipLaunchKernelGGL(k_sk_table<double>, nb, dim3(256), 0, s, static_cast<cplx<double> *>(tab), x,
                           static_cast<uint32_t *>(zero), zero_words);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || x.logm < 0 || x.m == x.n) return e;
    std::vector<double> re, im;
    chirp_spectrum(x, re, im);
    const size_t m = size_t(x.m);
    std::vector<double> d(2 * m);
    if (csz == 8) {
        const double up = 1.0 / std::sqrt(root_loss(x, re, im));
        float *f = reinterpret_cast<float *>(d.data());
        for (size_t k = 0; k < m; ++k) f[2 * k] = float(re[k] * up), f[2 * k + 1] = float(im[k] * up);
    } else {
        for (size_t k = 0; k < m; ++k) d[2 * k] = re[k], d[2 * k + 1] = im[k];
    }
    e = hipMemcpyAsync(static_cast<char *>(tab) + csz * (m + size_t(x.n)), d.data(), csz * m,
                       hipMemcpyHostToDevice, s);
    const hipError_t es = hipStreamSynchronize(s);  // the host copy goes with this call
    return e != hipSuccess ? e : es;
}

// Lines per block: enough to write pieces of 64 to 256 bytes (of up to 16384
// values, whose LDS still leaves a block its 160 KB), but not so many that an
// axis with few lines leaves CUs without a block.
static int sk_lines_per_block(int m, size_t csz, int64_t lines) {
    const int cap = sk_cap(csz), base = cap / 2;
    int lc = std::min(16, std::max(std::max(1, base / m), std::min(4, cap / m)));
    while (lc > 2 && lines / lc < 512) lc >>= 1;
    return std::max(1, std::min(lc, cap / m));
}

// Threads of a block: SK_HELD values each, half as many in wide lines, whose LDS admits
// half the blocks (160^3 347 us a sample and 310 so, 192^3 505 and 456, 1000^2 71 and 60)
static int sk_threads(int lines, const SkAxis &x) {
    const int held = x.wide ? SK_HELD / 2 : SK_HELD, t = (lines * x.m + held - 1) / held;
    return t <= 256 ? 256 : (t <= 512 ? 512 : 1024);
}

static size_t sk_window(const Geometry &g, int lc) {
    return sizeof(double) * 2 * size_t((g.D == 3 ? g.nz : g.ny) / 2 + lc + 4);
}

int measure_plan(MeasRep *reps, int nrep, MeasPlan &P) {
    P.nrep = nrep;
    P.pre.assign(size_t(MK_COUNT) * (nrep + 1), 0);
    for (int k = 0; k < MK_COUNT; ++k) P.shm[k] = 0, P.threads[k] = 256, P.wide[k] = false;
    if (nrep < 1) return -1;
    const int D = reps[0].g.D, prec = P.esz == 4 ? 0 : 1;
    P.D = D;
    int64_t nlines[3] = {};
    for (int r = 0; r < nrep; ++r) {
        const Geometry &g = reps[r].g;
        const int64_t hx = g.nx / 2 + 1;
        if (g.D != D) return -1;
        nlines[0] += int64_t((g.ny + 1) / 2) * g.nz;
        nlines[1] += hx * g.nz;
        nlines[2] += D == 3 ? hx * g.ny : hx;
    }
    int64_t tot[MK_COUNT] = {};
    for (int r = 0; r < nrep; ++r) {
        MeasRep &m = reps[r];
        const Geometry &g = m.g;
        const int side[3] = {g.nx, g.ny, g.nz}, hx = g.nx / 2 + 1;
        for (int d = 0; d < D; ++d) {
            if (side[d] > 8192) return -1;
            m.ax[d] = sk_axis(side[d], prec);
        }
        for (int k = 0; k < 3; ++k) {
            const int d = k == 2 ? D - 1 : k;
            if (k == 1 && D == 2) continue;
            m.lc[k] = sk_lines_per_block(m.ax[d].m, sk_value_bytes(prec, m.ax[d]), nlines[k]);
            P.wide[k] = P.wide[k] || m.ax[d].wide;
        }
        const SkAxis &last = m.ax[D - 1];
        auto line_bytes = [&](const SkAxis &x, int lc) { return sk_line_bytes(sk_value_bytes(prec, x), lc, x.m); };
        while (m.lc[2] > 1 && line_bytes(last, m.lc[2]) + sk_window(g, m.lc[2]) > SK_LDS) m.lc[2] >>= 1;
        int64_t n[MK_COUNT] = {};
        auto need = [&](int k, size_t shm, int threads) {
            P.shm[k] = std::max(P.shm[k], shm);
            P.threads[k] = std::max(P.threads[k], threads);
        };
        n[MK_ROWS] = int64_t((g.ny + 2 * m.lc[0] - 1) / (2 * m.lc[0])) * g.nz;
        need(MK_ROWS, line_bytes(m.ax[0], m.lc[0]), sk_threads(m.lc[0], m.ax[0]));
        if (D == 3) {
            n[MK_MID] = int64_t(hx) * ((g.nz + m.lc[1] - 1) / m.lc[1]);
            need(MK_MID, line_bytes(m.ax[1], m.lc[1]), sk_threads(m.lc[1], m.ax[1]));
        }
        const int inner = D == 3 ? g.ny : hx;
        n[MK_LAST] = int64_t((inner + m.lc[2] - 1) / m.lc[2]) * (D == 3 ? hx : 1);
        need(MK_LAST, line_bytes(last, m.lc[2]) + (m.lc[2] > 1 ? sk_window(g, m.lc[2]) : 0), sk_threads(m.lc[2], last));
        for (int k = 0; k < MK_COUNT; ++k) {
            P.pre[size_t(k) * (nrep + 1) + r] = int(tot[k]);
            tot[k] += n[k];
            if (tot[k] > 0x7fffffff) return -1;
        }
    }
    for (int k = 0; k < MK_COUNT; ++k) {
        P.pre[size_t(k) * (nrep + 1) + nrep] = int(tot[k]);
        if (P.shm[k] > SK_LDS) return -1;
    }
    return 0;
}

template <class L, typename real>
static hipError_t measure_impl(const MeasPlan &P, const MeasRep *mr, const int *pre, int par,
                               uint64_t *step_base, uint64_t advance, uint32_t step_off, hipStream_t s) {
    const int nrep = P.nrep;
    auto grid = [&](int k) { return dim3(unsigned(P.pre[size_t(k) * (nrep + 1) + nrep])); };
    auto pk = [&](int k) { return pre + size_t(k) * (nrep + 1); };
    auto block = [&](int k) { return dim3(unsigned(P.threads[k])); };
    constexpr bool F32 = sizeof(real) == 4;  // doubles have no wide axes
    auto launch = [&](int k, auto narrow, auto wide, auto... args) {
        hipLaunchKernelGGL(P.wide[k] ? wide : narrow, grid(k), block(k), P.shm[k], s, mr, pk(k), nrep, args...);
    };
    launch(MK_ROWS, k_sk_rows<L, real, false>, k_sk_rows<L, real, F32>, par, step_base, advance);
    if (L::D == 3) launch(MK_MID, k_sk_mid<real, false>, k_sk_mid<real, F32>);
    launch(MK_LAST, k_sk_last<real, false>, k_sk_last<real, F32>, step_base, step_off);
    return hipGetLastError();
}

hipError_t launch_measure(const MeasPlan &P, const MeasRep *dev_reps, const int *dev_pre, int precision,
                          int parity, uint64_t *step_base, uint64_t advance, uint32_t step_off, hipStream_t s) {
    if (P.nrep < 1 || P.pre.size() != size_t(MK_COUNT) * (P.nrep + 1)) return hipErrorInvalidValue;
    auto go = [&](auto impl) { return impl(P, dev_reps, dev_pre, parity, step_base, advance, step_off, s); };
    if (P.D == 2) return precision == 0 ? go(measure_impl<D2Q9, float>) : go(measure_impl<D2Q9, double>);
    return precision == 0 ? go(measure_impl<D3Q19, float>) : go(measure_impl<D3Q19, double>);
}

// ---------------------------------------------------------------------------
// S(k) of device fields: the same passes over a batch of equal square fields.
// Field f has its half spectrum at spec + f spec_len and its sums at acc +
// f acc_len: the shells, then sum P and sum |k| P.
// ---------------------------------------------------------------------------
struct FieldJob {
    const float *fields;
    cplx<float> *spec;
    double *acc;
    const void *tab;
    SkAxis ax;
    int n, n_rad, lc_rows, lc_last;
};

__device__ inline MeasRep field_rep(const FieldJob &j, int f) {
    MeasRep m{};
    m.g = Geometry{2, j.n, j.n, 1, int64_t(j.n) * j.n};
    m.cbuf = j.spec + size_t(f) * (j.n / 2 + 1) * j.n;
    m.tab[0] = m.tab[1] = j.tab;
    m.ax[0] = m.ax[1] = j.ax;
    m.lc[0] = j.lc_rows;
    m.lc[2] = j.lc_last;
    m.invN = 1.0 / double(m.g.N);
    m.t.n_rad = j.n_rad;
    m.t.rad_sum = j.acc + size_t(f) * field_acc_len(j.n_rad);
    m.t.mom = m.t.rad_sum + j.n_rad;
    return m;
}

template <typename T>
__global__ void __launch_bounds__(1024) k_field_rows(FieldJob j, int per) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int f = int(blockIdx.x) / per;
    const MeasRep m = field_rep(j, f);
    const float *src = j.fields + size_t(f) * j.n * j.n;
    sk_rows_block<T, float>(m, int(blockIdx.x) % per, smem_raw,
                            [&](int x, int y, int) { return src[size_t(y) * j.n + x]; });
}

template <typename T>
__global__ void __launch_bounds__(1024) k_field_last(FieldJob j, int per) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const MeasRep m = field_rep(j, int(blockIdx.x) / per);
    sk_last_block<T, float>(m, int(blockIdx.x) % per, smem_raw);
}

hipError_t launch_field_sk(const float *fields, int batch, int n, int n_rad, void *spec, const void *tab,
                           double *acc, hipStream_t s) {
    FieldJob j{fields, static_cast<cplx<float> *>(spec), acc, tab, sk_axis(n, 0), n, n_rad, 0, 0};
    const Geometry g{2, n, n, 1, int64_t(n) * n};
    const int hx = n / 2 + 1;
    const size_t csz = sk_value_bytes(0, j.ax);
    j.lc_rows = sk_lines_per_block(j.ax.m, csz, int64_t(batch) * ((n + 1) / 2));
    j.lc_last = sk_lines_per_block(j.ax.m, csz, int64_t(batch) * hx);
    while (j.lc_last > 1 && sk_line_bytes(csz, j.lc_last, j.ax.m) + sk_window(g, j.lc_last) > SK_LDS) j.lc_last >>= 1;
    const int pr = (n + 2 * j.lc_rows - 1) / (2 * j.lc_rows), pl = (hx + j.lc_last - 1) / j.lc_last;
    if (int64_t(batch) * std::max(pr, pl) > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(j.ax.wide ? k_field_rows<double> : k_field_rows<float>, dim3(unsigned(batch * pr)), dim3(unsigned(sk_threads(j.lc_rows, j.ax))),
                       sk_line_bytes(csz, j.lc_rows, j.ax.m), s, j, pr);
    hipLaunchKernelGGL(j.ax.wide ? k_field_last<double> : k_field_last<float>, dim3(unsigned(batch * pl)), dim3(unsigned(sk_threads(j.lc_last, j.ax))),
                       sk_line_bytes(csz, j.lc_last, j.ax.m) + (j.lc_last > 1 ? sk_window(g, j.lc_last) : 0), s, j, pl);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Plain device copy (16-byte lanes, grid-stride): the practical HBM
// read+write ceiling and the calibration for the memory-traffic counters.
// ---------------------------------------------------------------------------
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(256) k_copy(const u32x4 *__restrict__ src,
                                              u32x4 *__restrict__ dst, int64_t n16) {
    // One 16-byte element per lane and a grid that covers the buffer once
    // (the loop runs only for buffers beyond 2^38 bytes).  Blocks are
    // dispatched in address order, so the lanes in flight at any moment touch
    // one compact address range; a grid-stride copy with fewer, longer-lived
    // blocks spreads them over the whole buffer and measured 10% slower.
    // Non-temporal loads and stores.
    const int64_t stride = int64_t(gridDim.x) * 256;
    for (int64_t k = int64_t(blockIdx.x) * 256 + threadIdx.x; k < n16; k += stride)
        __builtin_nontemporal_store(__builtin_nontemporal_load(src + k), dst + k);
}

hipError_t launch_copy(const void *src, void *dst, int64_t bytes, hipStream_t s) {
    if (bytes <= 0 || (bytes & 15)) return hipErrorInvalidValue;
    const int64_t n16 = bytes / 16;
    const int64_t want = (n16 + 255) / 256;
    const unsigned blocks = unsigned(want < (int64_t(1) << 30) ? want : (int64_t(1) << 30));
    hipLaunchKernelGGL(k_copy, dim3(blocks), dim3(256), 0, s, static_cast<const u32x4 *>(src),
                       static_cast<u32x4 *>(dst), n16);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Generator checks.
// ---------------------------------------------------------------------------
__global__ void k_philox(const uint32_t *ctr, const uint32_t *key, uint32_t *out, int64_t n) {
    const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const U4 r = philox4x32_10(U4{ctr[4 * k], ctr[4 * k + 1], ctr[4 * k + 2], ctr[4 * k + 3]},
                               key[2 * k], key[2 * k + 1]);
    out[4 * k] = r.x;
    out[4 * k + 1] = r.y;
    out[4 * k + 2] = r.z;
    out[4 * k + 3] = r.w;
}

hipError_t launch_philox(const uint32_t *ctr, const uint32_t *key, uint32_t *out, int64_t n,
                         hipStream_t s) {
    const int64_t nb = (n + 255) / 256;
    if (nb > 0x7fffffff) return hipErrorInvalidValue;
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(k_philox, dim3(unsigned(nb)), dim3(256), 0, s, ctr, key, out, n);
    return hipGetLastError();
}

template <class L, typename real>
__global__ void k_normals(uint64_t seed, uint32_t replica, const int64_t *node,
                          const int64_t *step, int64_t n, double *out) {
    constexpr int NN = L::NNORM;
    const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= n) return;
    real z[NN];
    node_normals<L, real>(uint32_t(node[k]), uint32_t(step[k]), uint32_t(seed >> 32), z,
                          uint32_t(seed), replica);
    for (int q = 0; q < NN; ++q) out[k * NN + q] = double(z[q]);
}

hipError_t launch_normals(int D, int precision, uint64_t seed, uint32_t replica,
                          const int64_t *node, const int64_t *step, int64_t n, double *out,
                          hipStream_t s) {
    const int64_t nb = (n + 255) / 256;
    if (nb > 0x7fffffff) return hipErrorInvalidValue;
    if (nb == 0) return hipSuccess;
    if (D == 2) {
        if (precision == 0)
            hipLaunchKernelGGL((k_normals<D2Q9, float>), dim3(unsigned(nb)), dim3(256), 0,
                               s, seed, replica, node, step, n, out);
        else
            hipLaunchKernelGGL((k_normals<D2Q9, double>), dim3(unsigned(nb)), dim3(256), 0,
                               s, seed, replica, node, step, n, out);
    } else {
        if (precision == 0)
            hipLaunchKernelGGL((k_normals<D3Q19, float>), dim3(unsigned(nb)), dim3(256), 0,
                               s, seed, replica, node, step, n, out);
        else
            hipLaunchKernelGGL((k_normals<D3Q19, double>), dim3(unsigned(nb)), dim3(256),
                               0, s, seed, replica, node, step, n, out);
    }
    return hipGetLastError();
}

}  // namespace fsc
