// fsc_block_kernel.h -- several time steps per launch on 2D lattices small
// enough that a launch per step leaves the GPU waiting: a workgroup holds a tile
// of the lattice with its halo in LDS, advances it T steps there and writes the
// tile back.
//
// A lattice of 64^2 nodes takes 4 us per step as one launch per step, almost all
// of it launch, memory latency and the three-row chain of a one-row march; 88 of
// them take 12 us where their arithmetic alone takes about 4.  Here the chain of
// loads and stores is paid once per T steps and the state in between never
// leaves the CU.  The price is the halo: a step spoils h = R + 1 rows (and
// columns, unless the tile holds whole periodic rows) on each side of the tile,
// so a tile of TY rows is loaded with h T more on either side and the rows
// computed in step s = 0 .. T - 1 shrink from TY + 2h (T - 1) to TY.
//
// Layout: [row][population 0..8, psi][WS columns], so that every access of a
// node's neighbours is one of 3 (E8: 5) column addresses plus a constant.  A
// wave owns 64 columns of a row; rows go round the waves.  Per step:
//   pull f_i(x - c_i) from LDS into registers, n and psi(n) -> LDS; barrier;
//   Shan-Chen force from psi, noise, collision, f* back to LDS in place (every
//   pull of the step lies before the barrier); barrier.
// The per-node arithmetic is the single-step kernel's (same functions, same
// order, noise keyed by node and step), so the results are the same bits.
//
// What bounds it: the two phases' latency for the smallest lattices (about 1.6 us
// per step), vector issue with the halo's share for the largest.  Measured, us
// per step, one launch per step against this: E4 FP32 64^2 4.1 and 2.5, 32 x 64^2
// 7.4 and 3.3, 88 x 64^2 11.7 and 5.9, 48 x 128^2 18.7 and 11.7, 1000^2 21.8 and
// 13.9; E8 FP32 512^2 9.2 and 6.3; E4 FP64 64^2 6.5 and 4.7.  From 2^20 nodes on the
// tuned marching kernels are faster (4096^2: 9.4 us per 10^6 nodes).
#pragma once

#include "fsc_step_kernel.h"

namespace fsc {

template <class ST, typename real, bool NOISE, int WS, int NW>
__global__ void __launch_bounds__(NW * 64)
    k_block(const RepDesc *__restrict__ reps, const BlockTile *__restrict__ tiles, int nrep, int parity,
            const uint64_t *__restrict__ step_base, uint32_t step_off, int T) {
    using L = D2Q9;
    constexpr int Q = 9, R = ST::R, h = R + 1, NN = L::NNORM;
    constexpr int RS = (Q + 1) * WS;                 // values per row
    constexpr int WPR = WS / 64, RP = NW / WPR;      // waves per row, rows at a time
    constexpr int K = BLOCK_ROWS;                    // rows per wave at most
    constexpr uint32_t ES = sizeof(real);
    constexpr bool F32 = sizeof(real) == 4;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    real *cell = reinterpret_cast<real *>(smem_raw);

    const int lb = xcd_remap(blockIdx.x, gridDim.x);
    const int lo = owner_of<sizeof(BlockTile) / sizeof(int)>(&tiles[0].begin, nrep, lb);
    const RepDesc &d = reps[lo];
    const BlockTile bt = tiles[lo];
    const int nx = d.nx, ny = d.ny;
    const int t = lb - bt.begin;
    const int x0 = (t % bt.tiles_x) * bt.tx, y0 = (t / bt.tiles_x) * bt.ty;
    const int TXe = min(bt.tx, nx - x0), TYe = min(bt.ty, ny - y0);
    const bool whole = bt.tiles_x == 1 && bt.tx == nx;  // whole periodic rows: no halo columns
    const int hx = whole ? 0 : h * T, hy = h * T;
    const int W = TXe + 2 * hx, H = TYe + 2 * hy;        // the region held

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q0 = wave / WPR, c0 = (wave % WPR) * 64;
    const bool idle = c0 >= W;  // wave-uniform: only takes part in the barriers
    // lanes past the region repeat its last column and write nothing
    const int cl = c0 + int(threadIdx.x & 63);
    const bool on = cl < W;
    const int c = min(cl, W - 1);
    // columns c - R .. c + R: periodic in whole rows, else kept inside the region
    // (where that changes a column, the node is one of the spoiled ones)
    int col[2 * R + 1];
#pragma unroll
    for (int k = -R; k <= R; ++k) col[k + R] = whole ? wrap_any(c + k, nx) : min(max(c + k, 0), W - 1);
    const int gx = wrap_any(x0 - hx + c, nx);
    const bool out = on && c >= hx && c < hx + TXe;

    const uint64_t buf_bytes = uint64_t(Q) * uint64_t(d.N) * sizeof(real);
    const rsrc_t src = make_rsrc(d.buf[parity], buf_bytes);
    const rsrc_t dst = make_rsrc(d.buf[parity ^ 1], buf_bytes);
    const uint32_t pop_bytes = uint32_t(d.N) * ES, pbytes = uint32_t(nx) * ES;
    const real rho0 = F32 ? real(d.rho0f) : real(d.rho0);
    const real psi0 = F32 ? real(d.psi0f) : real(d.psi0);
    const real G = F32 ? real(d.Gf) : real(d.G);
    const real inv_rho0 = F32 ? real(d.inv_rho0f) : real(1.0 / d.rho0);
    real lc[4], ac[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        lc[k] = F32 ? real(d.lamcf[k]) : real(d.lamc[k]);
        ac[k] = F32 ? real(d.ampcf[k] * BM_SCALE) : real(d.ampc[k]);
    }
    const uint32_t step32 = uint32_t(step_base[0] + step_off);

#ifdef FSC_LDS_POISON
    lds_poison(cell, H * RS);
    __syncthreads();
#endif

    // ---- the tile and its halo into LDS, post-collision values as they lie ----
    real F[K][Q];
    if (!idle) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int r = q0 + k * RP;
            if (r < H) {
                const uint32_t ro = uint32_t(wrap_any(y0 - hy + r, ny)) * pbytes;
#pragma unroll
                for (int i = 0; i < Q; ++i) F[k][i] = bload<real>(src, uint32_t(gx) * ES, uint32_t(i) * pop_bytes + ro);
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int r = q0 + k * RP;
            if (r < H && on) {
#pragma unroll
                for (int i = 0; i < Q; ++i) cell[r * RS + i * WS + c] = F[k][i];
            }
        }
    }
    __syncthreads();

    for (int s = 0; s < T; ++s) {
        const int a0 = h * (s + 1), a1 = H - a0;  // rows that this step leaves valid
        const bool last = s + 1 == T;
        if (!idle) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int r = a0 - R + q0 + k * RP;
                if (r < a1 + R) {
                    const real *p = cell + r * RS;
                    real dn = real(0);
#pragma unroll
                    for (int i = 0; i < Q; ++i) {
                        F[k][i] = p[i * WS - L::c(i, 1) * RS + col[R - L::c(i, 0)]];
                        dn += F[k][i];
                    }
                    const real v = psi0 * fexpm1(dn * inv_rho0 * fast_rcp(rho0 + dn));
                    if (on) cell[r * RS + Q * WS + c] = v;
                }
            }
        }
        __syncthreads();
        if (!idle) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int r = a0 - R + q0 + k * RP;
                if (r >= a0 && r < a1) {
                    const int row = wrap_any(y0 - hy + r, ny);
                    // (drawn here: before the barrier, beside the pulls, it is 2-6% slower)
                    real z[NN];
                    if constexpr (NOISE) {
                        node_normals<L, real, !F32>(uint32_t(gx + nx * row), step32 + uint32_t(s), d.seed_hi, z,
                                                    d.key0, d.key1);
                    } else {
#pragma unroll
                        for (int j = 0; j < NN; ++j) z[j] = real(0);
                    }
                    const real *p = cell + r * RS + Q * WS;
                    real g[3] = {real(0), real(0), real(0)};
#pragma unroll
                    for (int a = 0; a < ST::NH; ++a) {
                        const int ex = ST::e(a, 0), ey = ST::e(a, 1);
                        const real diff = p[ey * RS + col[R + ex]] - p[-ey * RS + col[R - ex]];
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            const int ej = ST::e(a, j);
                            if (ej != 0) g[j] = fmadd(real(ST::w(a) * ej), diff, g[j]);
                        }
                    }
                    const real pre = G * (psi0 + p[c]);
                    const real Fv[3] = {pre * g[0], pre * g[1], pre * g[2]};
                    collide_d2q9<real, NOISE>(F[k], rho0, Fv, lc, ac, z);
                    if (last) {
                        if (out) {
                            const uint32_t so = uint32_t(row) * pbytes + uint32_t(gx) * ES;
#pragma unroll
                            for (int i = 0; i < Q; ++i) bstore<0>(dst, so, uint32_t(i) * pop_bytes, F[k][i]);
                        }
                    } else if (on) {
#pragma unroll
                        for (int i = 0; i < Q; ++i) cell[r * RS + i * WS + c] = F[k][i];
                    }
                }
            }
        }
        if (!last) __syncthreads();
    }
}

template <class ST, typename real, bool NOISE, int WS, int NW>
inline hipError_t launch_block_one(const BlockLaunch &P, hipStream_t s) {
    hipLaunchKernelGGL((k_block<ST, real, NOISE, WS, NW>), dim3(unsigned(P.blocks)), dim3(NW * 64), P.lds, s,
                       P.reps, P.tiles, P.nrep, P.parity, P.step_base, P.step_off, P.T);
    return hipGetLastError();
}

template <class ST, typename real>
inline hipError_t launch_block_kind(const BlockLaunch &P, hipStream_t s) {
    constexpr int NW2 = sizeof(real) == 4 ? 16 : 8;
    if (P.ws == 64)
        return P.noise ? launch_block_one<ST, real, true, 64, 8>(P, s)
                       : launch_block_one<ST, real, false, 64, 8>(P, s);
    if (P.ws == 128)
        return P.noise ? launch_block_one<ST, real, true, 128, NW2>(P, s)
                       : launch_block_one<ST, real, false, 128, NW2>(P, s);
    return hipErrorInvalidValue;
}

}  // namespace fsc
