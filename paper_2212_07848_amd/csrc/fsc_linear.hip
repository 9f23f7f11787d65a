// fsc_linear.hip -- exact structure factor of the linearised fluctuating step
// for any wave vector (the generalisation of Eq. 16 off the lattice axes).
//
// Around the homogeneous state n0 the step of Eq. 12, with the Shan-Chen
// force of Eq. 1 linearised (dF = G psi0 psi0' dn sum_a w_a e_a e^{ik.e_a}),
// acts on the Fourier amplitude of the populations as f_k <- A(k) f_k + noise,
// A = P C: C the moment-space collision with the linearised Guo source, P the
// streaming phases diag(e^{-i c_i.k}).  The noise covariance is
// Qn = P (sum over non-conserved rows a of amp_a^2 m_a m_a^T) P^H with
// m_a = M^{-1} e_a.  The stationary covariance X = sum_j A^j Qn (A^j)^H
// is summed by doubling (X <- X + A X A^H, A <- A A); S(k) = 1^T X 1.
// Doubling stays well posed where A has a unit-modulus eigenvalue the
// noise does not excite (k = pi on an axis at tau = 1).
//
// With every relaxation rate 1 (the paper's case) the collision forgets all but
// the conserved moments, and the same sum is one over (D + 1) x (D + 1) real
// matrices, one wave vector per lane (k_linear_conserved).  Other rates: one
// 64-lane workgroup per wave vector, the three Q x Q complex matrices in LDS
// (17 KB for D3Q19).  FP64 throughout.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

#include "../../include/fsc.h"
#include "fsc_internal.h"

namespace fsc {
namespace {

struct cplx64 {
    double re, im;
};
__device__ __forceinline__ cplx64 cmul(cplx64 a, cplx64 b) {
    return cplx64{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ __forceinline__ cplx64 cmulc(cplx64 a, cplx64 b) {  // a * conj(b)
    return cplx64{a.re * b.re + a.im * b.im, a.im * b.re - a.re * b.im};
}

struct LinArgs {
    double n0, coupling;  // n0 and G psi0 psi0'
    double mu;            // kBT / c_s^2
    double lam[4];        // per class
    int doublings;
};

// c_i is the one of +-c_i whose first non-zero component is positive
template <class L>
__host__ __device__ constexpr bool first_of_pair(int i) {
    return L::c(i, 0) != 0 ? L::c(i, 0) > 0 : (L::c(i, 1) != 0 ? L::c(i, 1) > 0 : L::c(i, 2) > 0);
}
// per moment row: 1/b_a, and whether M_ai takes the same value at c_i and -c_i
template <class L>
struct RowTable {
    double inv_norm[L::Q];
    bool even[L::Q];
    constexpr RowTable() : inv_norm{}, even{} {
        for (int a = 0; a < L::Q; ++a) {
            inv_norm[a] = 1.0 / moment_norm<L>(a);
            even[a] = true;
            for (int i = 0; i < L::Q; ++i)
                for (int j = 0; j < L::Q; ++j)
                    if (L::c(i, 0) == -L::c(j, 0) && L::c(i, 1) == -L::c(j, 1) && L::c(i, 2) == -L::c(j, 2) &&
                        L::M(a, i) != L::M(a, j))
                        even[a] = false;
        }
    }
};

// C = A B (all Q x Q), lanes stride over the entries.
template <int Q>
__device__ void matmul(const cplx64 (&a)[Q][Q], const cplx64 (&b)[Q][Q], cplx64 (&c)[Q][Q]) {
    for (int e = threadIdx.x; e < Q * Q; e += 64) {
        const int i = e / Q, l = e % Q;
        cplx64 s{0.0, 0.0};
#pragma unroll
        for (int m = 0; m < Q; ++m) {
            const cplx64 p = cmul(a[i][m], b[m][l]);
            s.re += p.re;
            s.im += p.im;
        }
        c[i][l] = s;
    }
}

// C += A B^H
template <int Q>
__device__ void matmul_add_h(const cplx64 (&a)[Q][Q], const cplx64 (&b)[Q][Q], cplx64 (&c)[Q][Q]) {
    for (int e = threadIdx.x; e < Q * Q; e += 64) {
        const int i = e / Q, l = e % Q;
        cplx64 s = c[i][l];
#pragma unroll
        for (int m = 0; m < Q; ++m) {
            const cplx64 p = cmulc(a[i][m], b[l][m]);
            s.re += p.re;
            s.im += p.im;
        }
        c[i][l] = s;
    }
}

// A(k) and the noise covariance Qn(k) into A and X (T is scratch); ends
// with a barrier.
template <class L, class ST>
__device__ void build_operator(const LinArgs &la, const double (&k)[3], cplx64 (&A)[L::Q][L::Q],
                               cplx64 (&X)[L::Q][L::Q], cplx64 (&T)[L::Q][L::Q]) {
    constexpr int D = L::D, Q = L::Q;
    constexpr double CS2 = 1.0 / 3.0;
    const int lane = threadIdx.x;
    // dF per unit dn: coupling * sum over the full stencil of w e e^{ik.e}
    // = coupling * sum over the half set of 2 i w e sin(k.e)
    double gim[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < ST::NH; ++a) {
        const double kd = k[0] * ST::e(a, 0) + k[1] * ST::e(a, 1) + (D == 3 ? k[2] * ST::e(a, 2) : 0.0);
        const double s = 2.0 * ST::w(a) * sin(kd);
#pragma unroll
        for (int d = 0; d < D; ++d) gim[d] += s * ST::e(a, d);
    }
    cplx64 dF[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) dF[d] = cplx64{0.0, la.coupling * gim[d]};
    // column j of A: a unit perturbation of population j through the
    // collision; the post-collision moments go through T (LDS)
    if (lane < Q) {
        const int j = lane;
        cplx64 du[3];
#pragma unroll
        for (int d = 0; d < 3; ++d)
            du[d] = cplx64{(double(L::c(j, d)) + 0.5 * dF[d].re) / la.n0, 0.5 * dF[d].im / la.n0};
        // c_i . du and c_i . dF of every population, as the equilibrium and
        // source need them
#pragma unroll 1
        for (int a = 0; a < Q; ++a) {
            const double m = double(L::M(a, j));
            cplx64 meq{0.0, 0.0}, src{0.0, 0.0};
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                const double Mw = double(L::M(a, i)) * L::w(i);
                double cur = 0.0, cui = 0.0, cfr = 0.0, cfi = 0.0;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    const double c = double(L::c(i, d));
                    cur += c * du[d].re;
                    cui += c * du[d].im;
                    cfr += c * dF[d].re;
                    cfi += c * dF[d].im;
                }
                meq.re += Mw * (1.0 + la.n0 * cur / CS2);
                meq.im += Mw * (la.n0 * cui / CS2);
                src.re += Mw * cfr / CS2;
                src.im += Mw * cfi / CS2;
            }
            const int cl = L::cls(a);  // select, not an indexed load (no scratch copy)
            const double lam = cl == 1 ? la.lam[1] : (cl == 2 ? la.lam[2] : (cl == 3 ? la.lam[3] : 1.0));
            T[a][j] = cplx64{m - lam * (m - meq.re) + (1.0 - 0.5 * lam) * src.re,
                             lam * meq.im + (1.0 - 0.5 * lam) * src.im};
        }
        // back-transform f_i = w_i sum_a M_ai ms_a / b_a, then the streaming phase
#pragma unroll 1
        for (int i = 0; i < Q; ++i) {
            cplx64 f{0.0, 0.0};
#pragma unroll
            for (int a = 0; a < Q; ++a) {
                const double cf = L::w(i) * double(L::M(a, i)) / moment_norm<L>(a);
                f.re += cf * T[a][j].re;
                f.im += cf * T[a][j].im;
            }
            double ph = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) ph -= double(L::c(i, d)) * k[d];
            A[i][j] = cmul(cplx64{cos(ph), sin(ph)}, f);
        }
    }
    // noise covariance P (sum_a amp_a^2 m_a m_a^T) P^H
    for (int e = lane; e < Q * Q; e += 64) {
        const int i = e / Q, l = e % Q;
        double s = 0.0;
#pragma unroll
        for (int a = D + 1; a < Q; ++a) {
            const double lam = la.lam[L::cls(a)];
            const double amp2 = la.mu * la.n0 * (1.0 - (1.0 - lam) * (1.0 - lam)) / moment_norm<L>(a);
            s += double(L::M(a, i)) * double(L::M(a, l)) * amp2;
        }
        s *= L::w(i) * L::w(l);
        double ph = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) ph += double(L::c(l, d) - L::c(i, d)) * k[d];
        X[i][l] = cplx64{s * cos(ph), s * sin(ph)};
    }
    __syncthreads();
}

// X <- sum_j A^j X (A^j)^H by doubling; A is overwritten.
template <int Q>
__device__ void doubling_sum(const LinArgs &la, cplx64 (&A)[Q][Q], cplx64 (&X)[Q][Q],
                             cplx64 (&T)[Q][Q], double (&red)[64]) {
    const int lane = threadIdx.x;
    for (int it = 0; it < la.doublings; ++it) {
        matmul<Q>(A, X, T);  // T = A X
        __syncthreads();
        matmul_add_h<Q>(T, A, X);  // X += A X A^H
        __syncthreads();
        matmul<Q>(A, A, T);  // T = A A
        __syncthreads();
        double amax = 0.0;
        for (int e = lane; e < Q * Q; e += 64) {
            const cplx64 v = T[e / Q][e % Q];
            A[e / Q][e % Q] = v;
            amax = fmax(amax, fabs(v.re) + fabs(v.im));
        }
        red[lane] = amax;
        __syncthreads();
        // the remaining terms are below 1e-40 of X once A^(2^it) has decayed
        bool done = true;
        for (int q = 0; q < 64; ++q) done = done && (red[q] < 1e-20);
        __syncthreads();
        if (done) break;
    }
}

// The wave vectors of one call: a caller's list, or (kv null) the fundamental
// domain of an n^D lattice's square / cubic group, 0 <= m_z <= m_y <= m_x <= n/2
// without the origin, in ascending (m_x, m_y, m_z).
struct KSource {
    const double *kv;
    int64_t nk;
    double unit;  // 2 pi / n
};

__host__ __device__ inline int64_t tri(int64_t a) { return a * (a + 1) / 2; }
__host__ __device__ inline int64_t tet(int64_t a) { return a * (a + 1) * (a + 2) / 6; }

__device__ __forceinline__ void wave_vector(const KSource &ks, int D, int64_t id, double (&k)[3]) {
    k[2] = 0.0;
    if (ks.kv) {
        for (int d = 0; d < D; ++d) k[d] = ks.kv[D * id + d];
        return;
    }
    const int64_t r = id + 1;  // rank, the origin included
    int64_t a = 0, rest = r;
    if (D == 3) {
        a = int64_t(cbrt(6.0 * double(r)));
        while (tet(a) > r) --a;
        while (tet(a + 1) <= r) ++a;
        rest = r - tet(a);
    }
    int64_t b = int64_t(sqrt(2.0 * double(rest)));
    while (tri(b) > rest) --b;
    while (tri(b + 1) <= rest) ++b;
    const int64_t c = rest - tri(b);
    k[0] = ks.unit * double(D == 3 ? a : b);
    k[1] = ks.unit * double(D == 3 ? b : c);
    if (D == 3) k[2] = ks.unit * double(c);
}

// All relaxation rates 1.  After a collision the populations depend on the
// conserved moments (n, j) alone, f* = E (n, j) with
//   f*_i = w_i (n + c_i . (j + dF) / c_s^2),
// so with B = (1, c) the moments' covariance is Z = sum_m K^m W (K^m)^H, K = B P E
// and W = B Qn B^H, both (D + 1) x (D + 1), and S = Z_00.  Rows and columns of j
// taken times i make K and W real: with theta_i = c_i . k, dF = i g dn,
//   s_d = sum w_i c_id sin theta_i,  q_de = sum w_i c_id c_ie cos theta_i,
//   K_00 = sum w_i cos theta_i + s . g / c_s^2,  K_0d = s_d / c_s^2,
//   K_d0 = -s_d + sum_e q_de g_e / c_s^2,        K_de = q_de / c_s^2,
// and W = sum_a amp_a^2 u_a u_a^T over the noise rows m_a, with u_a = (sum m_ai
// cos theta_i, -sum c_id m_ai sin theta_i) for rows even in c and (sum m_ai sin
// theta_i, sum c_id m_ai cos theta_i) for odd ones.
//
// Near k = 0, K is 1 + O(k) and the sum has O(1/k^2) terms, so what is held is
// K - 1, from -2 sin^2(theta/2) instead of cos theta - 1 (the ones fall out of
// every sum by the rows' orthogonality): squaring keeps it to a relative
// rounding, (1 + L)^2 - 1 = 2L + L L.
//
// A lane holds its three matrices in registers: 4 to 15 doublings of 170 FMAs where
// the Q x Q complex form takes 82000 each in 3D.  What bounds it is the one wave's
// serial FP64 chain (a 64^3 lattice has 103 waves of wave vectors).  The radial
// S(k) of 64^3, whole call: 1785 us as Q x Q matrices, 31 us so (this kernel 14), with
// half the error (2e-14).
template <class L, class ST>
__global__ void __launch_bounds__(64) k_linear_conserved(LinArgs la, KSource ks, double *__restrict__ out) {
    constexpr int D = L::D, Q = L::Q, N = D + 1;
    constexpr double ICS2 = 3.0;
    constexpr RowTable<L> rows;
    const int64_t id = int64_t(blockIdx.x) * 64 + threadIdx.x;
    double k[3];
    wave_vector(ks, D, id < ks.nk ? id : ks.nk - 1, k);

    double g[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < ST::NH; ++a) {
        double kd = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) kd += k[d] * ST::e(a, d);
        const double s = la.coupling * 2.0 * ST::w(a) * sin(kd);
#pragma unroll
        for (int d = 0; d < D; ++d) g[d] += s * ST::e(a, d);
    }
    // one of each pair +-c: sin theta and cos theta - 1
    double sn[Q], cm[Q];
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        if (!first_of_pair<L>(i)) continue;
        double th = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) th += k[d] * L::c(i, d);
        sn[i] = sin(th);
        const double h = sin(0.5 * th);
        cm[i] = -2.0 * h * h;
    }

    double Lm[N][N], X[N][N];  // K - 1 and the covariance (lower triangle)
#pragma unroll
    for (int a = 0; a < N; ++a)
#pragma unroll
        for (int b = 0; b < N; ++b) Lm[a][b] = X[a][b] = 0.0;
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        if (!first_of_pair<L>(i)) continue;
        Lm[0][0] += 2.0 * L::w(i) * cm[i];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (L::c(i, d) == 0) continue;
            Lm[0][d + 1] += 2.0 * ICS2 * L::w(i) * L::c(i, d) * sn[i];
#pragma unroll
            for (int e = 0; e < D; ++e)
                if (L::c(i, e) != 0) Lm[d + 1][e + 1] += 2.0 * ICS2 * L::w(i) * (L::c(i, d) * L::c(i, e)) * cm[i];
        }
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
        Lm[0][0] = fma(Lm[0][d + 1], g[d], Lm[0][0]);
        double v = g[d] - Lm[0][d + 1] / ICS2;
#pragma unroll
        for (int e = 0; e < D; ++e) v = fma(Lm[d + 1][e + 1], g[e], v);
        Lm[d + 1][0] = v;
    }
#pragma unroll
    for (int a = N; a < Q; ++a) {
        double u[N];
        const bool even = rows.even[a];
#pragma unroll
        for (int r = 0; r < N; ++r) {
            double v = 0.0;
#pragma unroll
            for (int i = 1; i < Q; ++i) {
                if (!first_of_pair<L>(i)) continue;
                const double cf = 2.0 * L::w(i) * L::M(a, i) * (r == 0 ? 1 : L::c(i, r > 0 ? r - 1 : 0));
                if (cf == 0.0) continue;
                const double t = (r == 0) == even ? cm[i] : sn[i];
                v += (r > 0 && even ? -cf : cf) * t;
            }
            u[r] = v;
        }
        const double amp2 = la.mu * la.n0 * rows.inv_norm[a];
#pragma unroll
        for (int r = 0; r < N; ++r)
#pragma unroll
            for (int q = 0; q <= r; ++q) X[r][q] = fma(amp2 * u[r], u[q], X[r][q]);
    }

    for (int it = 0; it < la.doublings; ++it) {
        double T[N][N];  // K X
#pragma unroll
        for (int a = 0; a < N; ++a)
#pragma unroll
            for (int b = 0; b < N; ++b) {
                double v = a >= b ? X[a][b] : X[b][a];
#pragma unroll
                for (int m = 0; m < N; ++m) v = fma(Lm[a][m], m >= b ? X[m][b] : X[b][m], v);
                T[a][b] = v;
            }
#pragma unroll
        for (int a = 0; a < N; ++a)  // X += T K^T
#pragma unroll
            for (int b = 0; b <= a; ++b) {
                double v = T[a][b];
#pragma unroll
                for (int m = 0; m < N; ++m) v = fma(T[a][m], Lm[b][m], v);
                X[a][b] += v;
            }
        double P[N][N];
#pragma unroll
        for (int a = 0; a < N; ++a)
#pragma unroll
            for (int b = 0; b < N; ++b) {
                double v = 2.0 * Lm[a][b];
#pragma unroll
                for (int m = 0; m < N; ++m) v = fma(Lm[a][m], Lm[m][b], v);
                P[a][b] = v;
            }
#pragma unroll
        for (int a = 0; a < N; ++a)
#pragma unroll
            for (int b = 0; b < N; ++b) Lm[a][b] = P[a][b];
        // What Z_00 still lacks goes through the first row of K, below 1e-24 of Z.
        // (The whole of K need not decay: at k = (pi, 0, 0) a transverse mode never
        // does, and one such lane kept its wave for 48 doublings where the others
        // take 4 to 15.)  A lane that is done adds nothing while the others go on.
        bool small = fabs(P[0][0] + 1.0) < 1e-12;
#pragma unroll
        for (int b = 1; b < N; ++b) small = small && fabs(P[0][b]) < 1e-12;
        if (__all(small)) break;
    }
    // no stationary value (an unstable state): NaN, as the general form gives, not infinity
    if (id < ks.nk) out[id] = X[0][0] + (X[0][0] - X[0][0]);
}

template <class L, class ST>
__global__ void __launch_bounds__(64) k_linear_sk(LinArgs la, KSource ks, double *__restrict__ out) {
    constexpr int Q = L::Q;
    __shared__ cplx64 A[Q][Q], X[Q][Q], T[Q][Q];
    __shared__ double red[64];
    const int lane = threadIdx.x;
    for (int64_t kid = blockIdx.x; kid < ks.nk; kid += gridDim.x) {
        double k[3];
        wave_vector(ks, L::D, kid, k);
        build_operator<L, ST>(la, k, A, X, T);
        doubling_sum<Q>(la, A, X, T, red);
        double s = 0.0;
        for (int e = lane; e < Q * Q; e += 64) s += X[e / Q][e % Q].re;
        red[lane] = s;
        __syncthreads();
        if (lane == 0) {
            double t = 0.0;
            for (int q = 0; q < 64; ++q) t += red[q];
            out[kid] = t;
        }
        __syncthreads();
    }
}

// C(k, tau) = 1^T A^tau X 1 at ascending lags: v = X 1, then v <- A v.
template <class L, class ST>
__global__ void __launch_bounds__(64) k_linear_corr(LinArgs la, const double *__restrict__ kv,
                                                    int64_t nk, const int *__restrict__ lags,
                                                    int nlag, double *__restrict__ out) {
    constexpr int D = L::D, Q = L::Q;
    __shared__ cplx64 A[Q][Q], X[Q][Q], T[Q][Q], A0[Q][Q];
    __shared__ cplx64 v[Q], vn[Q];
    __shared__ double red[64];
    const int lane = threadIdx.x;
    for (int64_t kid = blockIdx.x; kid < nk; kid += gridDim.x) {
        const double k[3] = {kv[3 * kid], kv[3 * kid + 1], D == 3 ? kv[3 * kid + 2] : 0.0};
        build_operator<L, ST>(la, k, A, X, T);
        for (int e = lane; e < Q * Q; e += 64) A0[e / Q][e % Q] = A[e / Q][e % Q];
        __syncthreads();
        doubling_sum<Q>(la, A, X, T, red);
        if (lane < Q) {
            cplx64 t{0.0, 0.0};
            for (int m = 0; m < Q; ++m) {
                t.re += X[lane][m].re;
                t.im += X[lane][m].im;
            }
            v[lane] = t;
        }
        __syncthreads();
        int tau = 0;
        for (int q = 0; q < nlag; ++q) {
            while (tau < lags[q]) {
                if (lane < Q) {
                    cplx64 t{0.0, 0.0};
                    for (int m = 0; m < Q; ++m) {
                        const cplx64 p = cmul(A0[lane][m], v[m]);
                        t.re += p.re;
                        t.im += p.im;
                    }
                    vn[lane] = t;
                }
                __syncthreads();
                if (lane < Q) v[lane] = vn[lane];
                __syncthreads();
                ++tau;
            }
            if (lane == 0) {
                double re = 0.0, im = 0.0;
                for (int m = 0; m < Q; ++m) {
                    re += v[m].re;
                    im += v[m].im;
                }
                out[(kid * nlag + q) * 2] = re;
                out[(kid * nlag + q) * 2 + 1] = im;
            }
            __syncthreads();
        }
    }
}

// floor(sqrt(v)), v >= 0
__device__ inline int64_t root(int64_t v) {
    int64_t b = int64_t(sqrt(double(v)));
    while (b * b > v) --b;
    while ((b + 1) * (b + 1) <= v) ++b;
    return b;
}

// Shell sums over the fundamental domain (see KSource): one block per shell
// round(|m|), its lanes over (m_x, m_y) (2D: m_x), whose last components in the
// shell are a range.  out[b]: sum of modes times S, out[nbins + b]: modes, both in a
// fixed order.  On the host the loop over all wave vectors and the copy of their S
// took as long as forming them (64^3: 44 us a call, 31 so).
template <int D>
__global__ void __launch_bounds__(256) k_linear_shells(const double *__restrict__ S, int n, int nbins,
                                                       double *__restrict__ out) {
    __shared__ double sh[2][4];
    const int64_t h = n / 2, b = blockIdx.x;
    const int64_t pairs = D == 3 ? tri(h + 1) : h + 1;
    auto signs = [&](int64_t v) { return v == 0 || 2 * v == n ? 1 : 2; };
    double sum = 0.0, modes = 0.0;
    for (int64_t p = threadIdx.x; p < pairs; p += 256) {
        int64_t x = p, y = 0;
        if (D == 3) {
            x = int64_t(sqrt(2.0 * double(p)));
            while (tri(x) > p) --x;
            while (tri(x + 1) <= p) ++x;
            y = p - tri(x);
        }
        // the last component m: b^2 - b < base + m^2 <= b^2 + b (b = 0: the origin)
        const int64_t base = x * x + y * y, top = b * b + b - base;
        if (b == 0 || top < 0) continue;
        const int64_t last = D == 3 ? y : x;
        const int64_t hi = min(last, root(top));
        const int64_t lo = top - 2 * b < 0 ? 0 : root(top - 2 * b) + 1;
        const int64_t first = (D == 3 ? tet(x) + tri(y) : tri(x)) - 1;
        for (int64_t m = lo; m <= hi; ++m) {
            const int perms = D == 2 ? (x == m ? 1 : 2) : (x == y && y == m ? 1 : (x == y || y == m ? 3 : 6));
            const double w = double(perms * signs(x) * signs(m) * (D == 3 ? signs(y) : 1));
            sum += w * S[first + m];
            modes += w;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        sum += __shfl_xor(sum, o, 64);
        modes += __shfl_xor(modes, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        sh[0][threadIdx.x >> 6] = sum;
        sh[1][threadIdx.x >> 6] = modes;
    }
    __syncthreads();
    if (threadIdx.x < 2)
        out[threadIdx.x * nbins + b] = (sh[threadIdx.x][0] + sh[threadIdx.x][1]) + (sh[threadIdx.x][2] + sh[threadIdx.x][3]);
}

// rates of exactly 1 take the conserved-moment form (any other rate keeps its
// class of moments from step to step)
template <class L, class ST>
hipError_t launch_linear(const LinArgs &la, const KSource &ks, double *out, hipStream_t s) {
    const int64_t waves = (ks.nk + 63) / 64;
    if (la.lam[1] == 1.0 && la.lam[2] == 1.0 && la.lam[3] == 1.0 && waves <= 0x7fffffff) {
        LinArgs unit = la;
        if (la.mu == 0.0) unit.doublings = 0;  // without noise the sum is 0, also where K grows beyond all bounds
        hipLaunchKernelGGL((k_linear_conserved<L, ST>), dim3(unsigned(waves)), dim3(64), 0, s, unit, ks, out);
        return hipGetLastError();
    }
    const unsigned blocks = unsigned(ks.nk < 65536 ? ks.nk : 65536);
    hipLaunchKernelGGL((k_linear_sk<L, ST>), dim3(blocks), dim3(64), 0, s, la, ks, out);
    return hipGetLastError();
}

hipError_t launch_linear(const fsc_params *p, const LinArgs &la, const KSource &ks, double *out, hipStream_t s) {
    if (p->D == 2 && p->stencil == FSC_E4) return launch_linear<D2Q9, StencilE4_2D>(la, ks, out, s);
    if (p->D == 2) return launch_linear<D2Q9, StencilE8_2D>(la, ks, out, s);
    return launch_linear<D3Q19, StencilE4_3D>(la, ks, out, s);
}

template <class L, class ST>
hipError_t launch_corr(const LinArgs &la, const double *kv, int64_t nk, const int *lags, int nlag,
                       double *out, hipStream_t s) {
    const unsigned blocks = unsigned(nk < 65536 ? nk : 65536);
    hipLaunchKernelGGL((k_linear_corr<L, ST>), dim3(blocks), dim3(64), 0, s, la, kv, nk, lags, nlag, out);
    return hipGetLastError();
}

int resolve_linear(const fsc_params *p, LinArgs &la) {
    if (!p || (p->D != 2 && p->D != 3) || (p->stencil != FSC_E4 && p->stencil != FSC_E8) ||
        (p->D == 3 && p->stencil == FSC_E8) || !(p->rho0 > 0.0) || !(p->kBT >= 0.0))
        return FSC_E_INVAL;
    const double lams[3] = {p->lambda_bulk, p->lambda_shear, p->lambda_ghost};
    for (double l : lams)
        if (!(l > 0.0 && l < 2.0)) return FSC_E_INVAL;
    const double CS2 = 1.0 / 3.0;
    double G = p->G;
    if (std::isnan(G)) {
        if (!(p->T_hat > 0.0)) return FSC_E_INVAL;
        G = std::exp(2.0) * CS2 / p->T_hat;
    }
    const double psi0 = std::exp(-1.0 / p->rho0);
    la.n0 = p->rho0;
    la.coupling = G * psi0 * psi0 / (p->rho0 * p->rho0);
    la.mu = p->kBT / CS2;
    la.lam[0] = 1.0;
    la.lam[1] = p->lambda_bulk;
    la.lam[2] = p->lambda_shear;
    la.lam[3] = p->lambda_ghost;
    la.doublings = 48;
    return FSC_OK;
}

}  // namespace
}  // namespace fsc

using namespace fsc;

extern "C" {

int fsc_linear_sk(const fsc_params *p, const double *host_k, int64_t nk, double *host_s,
                  void *stream) {
    LinArgs la;
    if (!host_k || !host_s || nk < 0) return FSC_E_INVAL;
    int rc = resolve_linear(p, la);
    if (rc) return rc;
    if (nk == 0) return FSC_OK;
    const hipStream_t st = static_cast<hipStream_t>(stream);
    double *dk = nullptr, *ds = nullptr;
    const size_t kbytes = sizeof(double) * size_t(p->D) * size_t(nk);
    if (hipMalloc(&dk, kbytes) != hipSuccess || hipMalloc(&ds, sizeof(double) * nk) != hipSuccess) {
        (void)hipGetLastError();
        if (dk) (void)hipFree(dk);
        return FSC_E_OOM;
    }
    hipError_t e = hipMemcpyAsync(dk, host_k, kbytes, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = launch_linear(p, la, KSource{dk, nk, 0.0}, ds, st);
    if (e == hipSuccess) e = hipMemcpyAsync(host_s, ds, sizeof(double) * nk, hipMemcpyDeviceToHost, st);
    const hipError_t es = hipStreamSynchronize(st);
    if (e == hipSuccess) e = es;
    (void)hipFree(dk);
    (void)hipFree(ds);
    return e == hipSuccess ? FSC_OK : FSC_E_HIP;
}

int fsc_linear_corr(const fsc_params *p, const double *host_k, int64_t nk, const int *host_lags,
                    int nlag, double *host_c, void *stream) {
    LinArgs la;
    if (!host_k || !host_lags || !host_c || nk < 0 || nlag < 0) return FSC_E_INVAL;
    int rc = resolve_linear(p, la);
    if (rc) return rc;
    for (int q = 0; q < nlag; ++q)
        if (host_lags[q] < 0 || (q > 0 && host_lags[q] < host_lags[q - 1])) return FSC_E_INVAL;
    if (nk == 0 || nlag == 0) return FSC_OK;
    const hipStream_t st = static_cast<hipStream_t>(stream);
    std::vector<double> k3(size_t(nk) * 3, 0.0);
    for (int64_t i = 0; i < nk; ++i)
        for (int d = 0; d < p->D; ++d) k3[3 * i + d] = host_k[p->D * i + d];
    double *dk = nullptr, *dc = nullptr;
    int *dl = nullptr;
    if (hipMalloc(&dk, sizeof(double) * 3 * nk) != hipSuccess ||
        hipMalloc(&dc, sizeof(double) * 2 * nk * nlag) != hipSuccess ||
        hipMalloc(&dl, sizeof(int) * nlag) != hipSuccess) {
        (void)hipGetLastError();
        if (dk) (void)hipFree(dk);
        if (dc) (void)hipFree(dc);
        return FSC_E_OOM;
    }
    hipError_t e = hipMemcpyAsync(dk, k3.data(), sizeof(double) * 3 * nk, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(dl, host_lags, sizeof(int) * nlag, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) {
        if (p->D == 2 && p->stencil == FSC_E4) e = launch_corr<D2Q9, StencilE4_2D>(la, dk, nk, dl, nlag, dc, st);
        else if (p->D == 2) e = launch_corr<D2Q9, StencilE8_2D>(la, dk, nk, dl, nlag, dc, st);
        else e = launch_corr<D3Q19, StencilE4_3D>(la, dk, nk, dl, nlag, dc, st);
    }
    if (e == hipSuccess)
        e = hipMemcpyAsync(host_c, dc, sizeof(double) * 2 * nk * nlag, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(dk);
    (void)hipFree(dc);
    (void)hipFree(dl);
    return e == hipSuccess ? FSC_OK : FSC_E_HIP;
}

int fsc_linear_sk_radial(const fsc_params *p, double *host_shell_mean, int64_t *host_count,
                         int nbins, void *stream) {
    if (!p || !host_shell_mean || nbins < 1) return FSC_E_INVAL;
    const int D = p->D, n = p->nx;
    if (n < 2 || p->ny != n || (D == 3 && p->nz != n) || (D == 2 && p->nz != 1)) return FSC_E_INVAL;
    LinArgs la;
    int rc = resolve_linear(p, la);
    if (rc) return rc;
    // the wave vectors of the fundamental domain of the square / cubic group,
    // 0 <= m_z <= m_y <= m_x <= n/2, each with the number of lattice modes it stands
    // for (sign choices x distinct permutations), and their shell sums: all on the
    // device
    const int64_t h = n / 2;
    const int64_t nk = (D == 2 ? tri(h + 1) : tet(h + 1)) - 1;
    const int64_t most = (D == 2 ? 2 * h : 3 * h) + 1;  // shells beyond are empty
    const int nb = int(std::min<int64_t>(nbins, most));
    const hipStream_t st = static_cast<hipStream_t>(stream);
    ThreadWork &work = thread_work();
    void *area = nullptr;
    rc = work.take(sizeof(double) * (size_t(nk) + 2 * size_t(nb)), &area);
    if (rc) return rc;
    double *ds = static_cast<double *>(area), *sums = ds + nk;
    std::vector<double> host(2 * size_t(nb));
    Mailbox *box = sizeof(double) * host.size() <= ThreadWork::MAIL ? work.mailbox() : nullptr;
    hipError_t e = launch_linear(p, la, KSource{nullptr, nk, 2.0 * M_PI / n}, ds, st);
    if (e == hipSuccess) {
        hipLaunchKernelGGL((D == 3 ? k_linear_shells<3> : k_linear_shells<2>), dim3(unsigned(nb)), dim3(256), 0, st, ds,
                           n, nb, sums);
        e = hipGetLastError();
    }
    if (e == hipSuccess)
        e = box ? launch_mail(sums, 2 * nb, box->next(), st)
                : hipMemcpyAsync(host.data(), sums, sizeof(double) * host.size(), hipMemcpyDeviceToHost, st);
    const hipError_t es = box && e == hipSuccess ? box->wait(st) : hipStreamSynchronize(st);
    if (e == hipSuccess) e = es;
    work.done(area);
    if (e != hipSuccess) return FSC_E_HIP;
    const double *sum = box ? box->data() : host.data(), *modes = sum + nb;
    for (int b = 0; b < nbins; ++b) {
        const bool any = b < nb && modes[b] > 0.0;
        host_shell_mean[b] = any ? sum[b] / modes[b] : 0.0;
        if (host_count) host_count[b] = any ? int64_t(modes[b]) : 0;
    }
    return FSC_OK;
}

}  // extern "C"
