// Fused, LDS-tiled FAS V-cycle kernels for gfx950.
//
// Each multigrid level above 32x32 cells costs two launches per V-cycle:
//   down: complete the FAS right-hand side, nu1 red-black nonlinear
//         Gauss-Seidel passes (App. B smoother), write u, then the residual
//         and its 2x2-average restriction together with the restriction of u
//         onto the next level (one read of the level, one write);
//   up:   load u with the bilinear coarse-grid correction applied, nu2
//         passes, write u; on the finest level also the residual norm of the
//         stopping test.
// All levels of at most 32x32 cells run in one persistent single-workgroup
// kernel that keeps them in LDS and solves the coarsest grid directly.
//
// Tiles.  A workgroup owns a tx x ty interior tile and loads it with a halo
// of H cells (periodic wrap, or reflection on a Neumann axis) into LDS.  After p half-sweeps the cells at
// distance >= p from the loaded border hold exactly the values of a global
// red-black sweep (a red cell only reads black neighbours and vice versa), so
// H >= number of half-sweeps (+1 when a residual follows) makes the interior
// exact.  Output goes to a second buffer (ping-pong), so neighbouring tiles
// always read the values from before the launch.  H is even, so the loaded
// region starts on an even global index: 2x2 blocks of the loaded region are
// exactly the fine cells under one coarse cell.
//
// Threads own 2x2 blocks of the loaded region: both red cells of a block in
// red passes, both black cells in black passes, all four for the residual,
// restriction and prolongation.  Right-hand side and phi^k of owned cells
// live in registers.  LDS holds the unknowns split by colour: U[f][c][y][x/2]
// with c = (x + y) & 1, so a thread's own cells and all neighbours of one
// colour are contiguous across lanes (no bank conflicts on 8-byte accesses).
#pragma once
#include <type_traits>

#include "kernels.hpp"

namespace mpfc {

// ---------------------------------------------------------------------------
// Cell operators.  ns[f] is the sum of the four neighbours of field f.

// MPFC system N(u) = f (App. B.1 / B.2), optionally in correction (DEFECT) form.
// PIN: the pinning of Sec. 4.6 adds the per-cell weight w to the coefficient
// of phi in N^(2) (the unknown mu is mu~); w = 0 otherwise.
template <typename T, int SCHEME, bool NEWTON, bool DEFECT, bool PIN = false>
struct MpfcOp {
    using real = T;
    static constexpr int NF = 3;
    static constexpr bool XK = SCHEME == 2;
    static constexpr bool PB = DEFECT;
    static constexpr bool PW = PIN;
    LevelOp<T> op;

    // The functions take K cells (which do not neighbour each other where they
    // are updated) and do every operation for all of them in turn: a wave issues
    // in order and a dependent FP64 operation waits 8 clocks against 4 to issue,
    // so one cell's chain after the other left the unit idle half of the time.

    // r = f - N(u).
    template <int K>
    __device__ __forceinline__ void resid(const T (&u)[K][3], const T (&ns)[K][3],
                                          const T (&f)[K][3], const T (&xk)[K], const T (&pb)[K],
                                          const T (&w)[K], T (&r)[K][3]) const {
        T g[K], lap[K][3];
#pragma unroll
        for (int k = 0; k < K; ++k) g[k] = nl_value<T, SCHEME, DEFECT>(u[k][0], pb[k], xk[k]);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            r[k][0] = f[k][0] - u[k][0];
            r[k][1] = (f[k][1] - u[k][1]) + (g[k] + (PIN ? op.al + w[k] : op.al) * u[k][0]);
            r[k][2] = f[k][2] - u[k][2];
        }
        residual_lap(u, ns, lap, r);
    }
    // Collective update of the cells: J_loc delta = f - N(u) (App. B), the
    // 3x3 system J_loc = [[1, a, 0], [-d, 1, b], [ec, 0, 1]], a = 4c/h^2, b = 4/h^2,
    // ec = 4e/h^2, d = al + linearised nonlinear coefficient, by elimination.
    // What does not depend on the neighbours comes first (their LDS reads are
    // in flight meanwhile).
    template <int K>
    __device__ __forceinline__ void relax(T (&u)[K][3], const T (&ns)[K][3], const T (&f)[K][3],
                                          const T (&xk)[K], const T (&pb)[K],
                                          const T (&w)[K]) const {
        T d[K], det[K], rec[K], r[K][3], lap[K][3];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            T g;
            nl_both<T, SCHEME, NEWTON, DEFECT>(u[k][0], pb[k], xk[k], g, d[k]);
            if constexpr (PIN) d[k] += w[k];
            r[k][0] = f[k][0] - u[k][0];
            r[k][1] = (f[k][1] - u[k][1]) + (g + (PIN ? op.al + w[k] : op.al) * u[k][0]);
            r[k][2] = f[k][2] - u[k][2];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) det[k] = op.det0 + op.a * d[k];
        recip_ge1_n(det, rec);
        residual_lap(u, ns, lap, r);
        T dm[K], dx[K];
#pragma unroll
        for (int k = 0; k < K; ++k) dm[k] = r[k][1] + (op.dd0 + d[k]) * r[k][0];
#pragma unroll
        for (int k = 0; k < K; ++k) dm[k] = (dm[k] - op.b * r[k][2]) * rec[k];
#pragma unroll
        for (int k = 0; k < K; ++k) dx[k] = r[k][0] - op.a * dm[k];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            u[k][1] += op.w * dm[k];
            u[k][0] += op.w * dx[k];
            u[k][2] += op.w * (r[k][2] - op.ec * dx[k]);
        }
    }
    // r (f - N without its Laplacians) completed with them.
    template <int K>
    __device__ __forceinline__ void residual_lap(const T (&u)[K][3], const T (&ns)[K][3],
                                                 T (&lap)[K][3], T (&r)[K][3]) const {
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
            for (int k = 0; k < K; ++k) lap[k][f] = ns[k][f] - T(4) * u[k][f];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            r[k][0] += op.k1 * lap[k][1];
            r[k][2] += op.e1 * lap[k][0];
            r[k][1] += op.ih2 * lap[k][2];
        }
    }
};

// Poisson problem -Lap_h w = b (App. A "-1" norm), same interface.
template <typename T>
struct PoissonOp {
    using real = T;
    static constexpr int NF = 1;
    static constexpr bool XK = false;
    static constexpr bool PB = false;
    static constexpr bool PW = false;
    T ih2, h2;
    template <int K>
    __device__ __forceinline__ void resid(const T (&u)[K][1], const T (&ns)[K][1],
                                          const T (&f)[K][1], const T (&)[K], const T (&)[K],
                                          const T (&)[K], T (&r)[K][1]) const {
#pragma unroll
        for (int k = 0; k < K; ++k) r[k][0] = f[k][0] - (T(4) * u[k][0] - ns[k][0]) * ih2;
    }
    template <int K>
    __device__ __forceinline__ void relax(T (&u)[K][1], const T (&ns)[K][1], const T (&f)[K][1],
                                          const T (&)[K], const T (&)[K], const T (&)[K]) const {
#pragma unroll
        for (int k = 0; k < K; ++k) u[k][0] = T(0.25) * (h2 * f[k][0] + ns[k][0]);
    }
};

// ---------------------------------------------------------------------------
template <typename T>
struct TileArgs {
    Grid g;                 // this level
    const T* uin[3];        // u before the launch
    T* uout[3];             // u after the launch (interior cells)
    const T* f[3];          // right-hand side: complete (finest down, every up) or the
                            // restricted residual R r (coarse down, completed in-kernel)
    T* fout[3];             // coarse down: completed right-hand side f = R r + N(u)
    const T* xk;            // phi^k on this level (scheme 2)
    const T* pb;            // base phi (correction form)
    T* uH[3]; T* vH[3]; T* rH[3];          // down: restricted u (twice) and residual
    T* xkH; T* pbH;         // down (nullable): 2x2 averages of phi^k and of the base phi
    const T* pin;           // pinning weight on this level (Op::PW)
    const T* cuH[3]; const T* cvH[3];      // up: coarse u after and before its solve
    int complete_f;         // down on a coarse level
    int zero_in;            // u before the launch is zero (uin is not read); in a batch: in
                            // launches marked `first`
    int nsweep;             // red-black half-sweeps (2 nu)
    int H;                  // halo (even)
    int tx, ty;             // interior tile (even, divides m, n)
    // residual norm (finest up): per-block FP64 sums of r^2 into part[]
    int norm;
    double* part;
    int ntx;                // tiles in x (set by the launch)
};

// Cell index along one axis inside the tile and coarse kernels: plain
// wrap-around in the periodic instantiation (NEU = false), the per-axis ghost
// rule (axis_index) in the instantiation for grids with a Neumann axis.
// GEN: instantiation for grids whose sides need not be powers of two.
template <bool NEU, bool GEN = false>
__device__ __forceinline__ int bidx(int i, int m, int neumann_axis) {
    if constexpr (GEN) return axis_index_any(i, m, NEU && neumann_axis);
    else if constexpr (NEU) return axis_index(i, m, neumann_axis);
    else return i & (m - 1);
}
template <bool GEN>
__device__ __forceinline__ size_t tat(int i, int j, const Grid& g) {
    if constexpr (GEN) return (size_t)j * (size_t)g.m + (size_t)i;
    else return ((size_t)j << g.lm) + (size_t)i;
}

// XCD-aware order of nt work items: workgroups are dealt round-robin to the 8
// XCDs, each with its own L2.  Workgroup b (on XCD b % 8) takes item
// (b % 8) * (nt / 8) + b / 8, so every XCD sweeps one contiguous strip of
// tiles and the halos it re-reads are mostly in its own L2.
__device__ __forceinline__ int xcd_item(int b, int nt) {
    return (nt & 7) == 0 ? (b & 7) * (nt >> 3) + (b >> 3) : b;
}

#ifndef MPFC_TILE_THREADS
#define MPFC_TILE_THREADS 512
#endif
// Threads of a tile workgroup.
constexpr int kTileThreads = MPFC_TILE_THREADS;
static_assert(kTileThreads == kNormThreads, "a tile launch runs a pending stopping test");

// One tile of a tiled level, in phases:
//   load_direct  u (tile + halo) and, for up launches, u_H - v_H over the
//                tile's coarse footprint, from global memory into LDS;
//   fetch_rhs    the right-hand side and coefficients of the owned blocks
//                into registers;
//   compute      prolongation (up), completion of the coarse right-hand side
//                (coarse down), the red-black passes, the store of u, and the
//                residual with its restriction (down) or norm (finest up).
// EXACT: the launch's tile is the shape's (A.tx = TX, A.ty = TY) and its halo
// the shape's allowance (A.H = HMAX), so every extent is a compile-time
// constant.
template <class Op, int TX, int TY, int HMAX, bool UP, bool NEU, bool GEN, bool EXACT>
struct TileWork {
    using T = typename Op::real;
    static constexpr int NF = Op::NF;
    static constexpr int NT = kTileThreads;
    static constexpr int LX2M = (TX + 2 * HMAX) / 2;
    static constexpr int LYM = TY + 2 * HMAX;
    static constexpr int SL = (LX2M * (LYM / 2) + NT - 1) / NT;  // owned blocks per thread
    // LDS row length (doubles per colour and row), padded so that a wave's
    // consecutive blocks continue across a block-row break on the next banks:
    // the block-row stride 2 P equals LX2 modulo the 32 doubles of a bank cycle.
    static constexpr int pad_row(int l) {
        int p = l;
        while (((2 * p - l) % 32 + 32) % 32 != 0) ++p;
        return p;
    }
    static constexpr int LXP = pad_row(LX2M);
    static constexpr int CXM = LX2M + 2, CYM = LYM / 2 + 2;       // coarse footprint

    struct Lds {
        T U[NF][2][LYM][LXP];
        T E[UP ? NF : 1][UP ? CYM : 1][UP ? CXM : 1];  // up: uH - vH
        union {
            double red[NT / 64];
            int saw[NT / 64];  // the waves' looks at a stop flag that may rise
        };
    };
    // Extents of the tile (tbx, tby) of a launch.
    struct Geo {
        int H, tx, ty, LX, LY, LX2, nblk, x0, y0, tbx, tby;
    };
    // Right-hand side and coefficients of the owned blocks' four cells (cell
    // order: (0,0) (1,1) red, (1,0) (0,1) black).
    struct Rhs {
        T f[SL][4][NF];
        T xk[SL][4];
        T pb[SL][4];
        T w[SL][4];
    };
    // OWN (a thread owns at most one block): the block's four cells are also
    // kept in registers, updated together with LDS.  Two of each cell's four
    // neighbours lie in its own block, so half of the neighbour reads come
    // from registers and LDS traffic per relaxation halves.  Only the owner
    // writes a cell (except the Neumann ghost restore, after which the copy
    // is reloaded).
    static constexpr bool OWN = SL == 1;
    struct Own {
        T u[4][NF];
    };
    // cell offsets within a block: 0 = (0,0), 1 = (1,1) red; 2 = (1,0), 3 = (0,1) black
    static constexpr int cdx(int c) { return (c == 1 || c == 2) ? 1 : 0; }
    static constexpr int cdy(int c) { return (c == 1 || c == 3) ? 1 : 0; }
    static constexpr int cid(int dx, int dy) { return dx == dy ? dx : (dx ? 2 : 3); }

    // Neighbour sums of cell C of the owned block (bx, by), every field, in
    // the order (east + west) + (north + south): own-block neighbours from
    // registers, the others from LDS.
    // Indices are clamped to the loaded region: a cell on its border gets a
    // meaningless sum, and its result is discarded by the caller.
    template <int C>
    static __device__ __forceinline__ void nsum_own(const Lds& S, const Own& O, const Geo& G,
                                                    int bx, int by, T (&ns)[NF]) {
        constexpr int dx = cdx(C), dy = cdy(C), oc = ((dx + dy) & 1) ^ 1;
        const int y = 2 * by + dy;
        const int ke = min(bx + 1, G.LX2 - 1), kw = max(bx - 1, 0);
        const int yn = min(y + 1, G.LY - 1), ys = max(y - 1, 0);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const T e = dx == 0 ? O.u[cid(1, dy)][f] : S.U[f][oc][y][ke];
            const T w = dx == 1 ? O.u[cid(0, dy)][f] : S.U[f][oc][y][kw];
            const T n = dy == 0 ? O.u[cid(dx, 1)][f] : S.U[f][oc][yn][bx];
            const T s = dy == 1 ? O.u[cid(dx, 0)][f] : S.U[f][oc][ys][bx];
            ns[f] = (e + w) + (n + s);
        }
    }
    // f - N(u) (ZF: -N(u)) at cells C0 and C1 of the owned block.
    template <int C0, int C1, bool ZF>
    static __device__ __forceinline__ void resid2(const Op& op, const Lds& S, const Own& O,
                                                  const Geo& G, int bx, int by, const Rhs& R,
                                                  T (&r)[2][NF]) {
        T u[2][NF], ns[2][NF], fv[2][NF];
        nsum_own<C0>(S, O, G, bx, by, ns[0]);
        nsum_own<C1>(S, O, G, bx, by, ns[1]);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            u[0][f] = O.u[C0][f];
            u[1][f] = O.u[C1][f];
            fv[0][f] = ZF ? T(0) : R.f[0][C0][f];
            fv[1][f] = ZF ? T(0) : R.f[0][C1][f];
        }
        op.resid(u, ns, fv, {R.xk[0][C0], R.xk[0][C1]}, {R.pb[0][C0], R.pb[0][C1]},
                 {R.w[0][C0], R.w[0][C1]}, r);
    }
    // The owned block's cells from LDS into registers (after a barrier).
    static __device__ __forceinline__ void load_own(const Lds& S, const Geo& G, Own& O) {
        const int b = threadIdx.x;
        if (b >= G.nblk) return;
        const int by = b / G.LX2, bx = b - by * G.LX2;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int y = 2 * by + cdy(c);
#pragma unroll
            for (int f = 0; f < NF; ++f) O.u[c][f] = S.U[f][(cdx(c) + cdy(c)) & 1][y][bx];
        }
    }

    static __device__ __forceinline__ Geo geo(const TileArgs<T>& A, int tbx, int tby) {
        Geo G;
        G.H = EXACT ? HMAX : A.H;
        G.tx = EXACT ? TX : A.tx;
        G.ty = EXACT ? TY : A.ty;
        G.LX = G.tx + 2 * G.H;
        G.LY = G.ty + 2 * G.H;
        G.LX2 = G.LX >> 1;
        G.nblk = G.LX2 * (G.LY >> 1);
        G.x0 = tbx * G.tx - G.H;
        G.y0 = tby * G.ty - G.H;
        G.tbx = tbx;
        G.tby = tby;
        return G;
    }

    static __device__ __forceinline__ size_t cell(const Grid& g, int x, int y) {
        return tat<GEN>(bidx<NEU, GEN>(x, g.m, g.bc & BC_NEUMANN_X),
                        bidx<NEU, GEN>(y, g.n, g.bc & BC_NEUMANN_Y), g);
    }
    static __device__ __forceinline__ size_t coarse_cell(const Grid& g, int cx, int cy) {
        const int mc = g.m >> 1, nc = g.n >> 1;
        return (size_t)bidx<NEU, GEN>(cy, nc, g.bc & BC_NEUMANN_Y) * mc +
               bidx<NEU, GEN>(cx, mc, g.bc & BC_NEUMANN_X);
    }

    static __device__ __forceinline__ void fetch_rhs(const TileArgs<T>& A, const Geo& G, Rhs& R) {
        const Grid g = A.g;
        const int t = threadIdx.x;
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const int b = t + s * NT;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
#pragma unroll
                for (int f = 0; f < NF; ++f) R.f[s][c][f] = T(0);
                R.xk[s][c] = T(0);
                R.pb[s][c] = T(0);
                R.w[s][c] = T(0);
            }
            if (b >= G.nblk) continue;
            const int by = b / G.LX2, bx = b - by * G.LX2;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int dx = (c == 1 || c == 2) ? 1 : 0, dy = (c == 1 || c == 3) ? 1 : 0;
                const int x = 2 * bx + dx, y = 2 * by + dy;
                if (x < 1 || y < 1 || x >= G.LX - 1 || y >= G.LY - 1) continue;  // never updated
                const size_t gq = cell(g, G.x0 + x, G.y0 + y);
                if constexpr (Op::XK) R.xk[s][c] = A.xk[gq];
                if constexpr (Op::PB) R.pb[s][c] = A.pb[gq];
                if constexpr (Op::PW) R.w[s][c] = A.pin[gq];
#pragma unroll
                for (int f = 0; f < NF; ++f) R.f[s][c][f] = A.f[f][gq];
            }
        }
    }

    // u (tile + halo) and, up, uH - vH into LDS, coalesced along rows; a
    // barrier must follow.
    // Loads of LCH consecutive strides are issued together, so a thread waits
    // once per LCH strides rather than once per stride.  Indices past the end
    // are clamped to the last cell, for the load and the store alike (the
    // same value stored twice), so no load sits behind a branch.
    static constexpr int LCH = 4;
    // `mid` runs once the first stride group's loads are issued (before any of
    // them is waited for): the caller requests the right-hand side there.
    template <class Mid>
    static __device__ __forceinline__ void load_direct(const TileArgs<T>& A, const Geo& G, Lds& S,
                                                       bool zero_in, Mid&& mid) {
        const Grid g = A.g;
        const int t = threadIdx.x;
        const int total = G.LX * G.LY;
        constexpr int NLD = (2 * LX2M * LYM + NT - 1) / NT;  // strides of the largest tile
        // up: u_H - v_H over the tile's coarse footprint, requested first so
        // that its loads are in flight together with the tile's
        constexpr int NE = UP ? (CXM * CYM + NT - 1) / NT : 1;
        T ev[NE][NF];
        int exs[NE], eys[NE];
        if constexpr (UP) {
            const int CX = G.LX2 + 2, CY = (G.LY >> 1) + 2, ctot = CX * CY;
            const int cx0 = (G.x0 >> 1) - 1, cy0 = (G.y0 >> 1) - 1;
            (void)CY;
#pragma unroll
            for (int j = 0; j < NE; ++j) {
                const int q = min(t + j * NT, ctot - 1);
                eys[j] = q / CX;
                exs[j] = q - eys[j] * CX;
                const size_t gq = coarse_cell(g, cx0 + exs[j], cy0 + eys[j]);
#pragma unroll
                for (int f = 0; f < NF; ++f) ev[j][f] = A.cuH[f][gq] - A.cvH[f][gq];
            }
        }
        if (zero_in) {
            mid();
            for (int q = t; q < total; q += NT) {
                const int y = q / G.LX, x = q - y * G.LX;
#pragma unroll
                for (int f = 0; f < NF; ++f) S.U[f][(x + y) & 1][y][x >> 1] = T(0);
            }
        } else {
#pragma unroll
            for (int k0 = 0; k0 < NLD; k0 += LCH) {
                T v[LCH][NF];
                int xs[LCH], ys[LCH];
#pragma unroll
                for (int j = 0; j < LCH; ++j) {
                    if (k0 + j >= NLD) break;
                    const int q = min(t + (k0 + j) * NT, total - 1);
                    ys[j] = q / G.LX;
                    xs[j] = q - ys[j] * G.LX;
                    const size_t gq = cell(g, G.x0 + xs[j], G.y0 + ys[j]);
#pragma unroll
                    for (int f = 0; f < NF; ++f) v[j][f] = A.uin[f][gq];
                }
                if (k0 == 0) mid();
#pragma unroll
                for (int j = 0; j < LCH; ++j) {
                    if (k0 + j >= NLD) break;
                    const int x = xs[j], y = ys[j];
#pragma unroll
                    for (int f = 0; f < NF; ++f) S.U[f][(x + y) & 1][y][x >> 1] = v[j][f];
                }
            }
        }
        if constexpr (UP) {
#pragma unroll
            for (int j = 0; j < NE; ++j)
#pragma unroll
                for (int f = 0; f < NF; ++f) S.E[f][eys[j]][exs[j]] = ev[j][f];
        }
    }

    // Everything after the tile is in LDS (entered after a barrier).  `pslot`
    // is where the workgroup's residual sum goes in A.part.
    static __device__ __forceinline__ void compute(const Op& op, const TileArgs<T>& A,
                                                   const Geo& G, Lds& S, Rhs& R, int pslot) {
        const Grid g = A.g;
        const int H = G.H, tx = G.tx, ty = G.ty, LX = G.LX, LY = G.LY, LX2 = G.LX2;
        const int nblk = G.nblk, x0 = G.x0, y0 = G.y0, tbx = G.tbx, tby = G.tby;
        const int t = threadIdx.x;
        auto& U = S.U;
        auto& E = S.E;
        auto& red = S.red;
        auto& fr = R.f;
        const auto& xkr = R.xk;
        const auto& pbr = R.pb;
        const auto& wr = R.w;
        Own O;
        if constexpr (OWN && !UP) load_own(S, G, O);
    // 3. up: add the coarse-grid correction P(uH - vH) to every loaded cell
    //    (uH - vH over the tile's coarse footprint, one coarse cell of margin,
    //    staged in LDS).
    if constexpr (UP && OWN) {
        // the block's 3x3 coarse neighbourhood once per field, then its four cells
        if (t < nblk) {
            const int by = t / LX2, bx = t - by * LX2;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                T e9[3][3];
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int i = 0; i < 3; ++i) e9[j][i] = E[f][by + j][bx + i];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int dx = cdx(c), dy = cdy(c);
                    const int x = 2 * bx + dx, y = 2 * by + dy;
                    const int si = dx ? 2 : 0, sj = dy ? 2 : 0;
                    const T v = U[f][(x + y) & 1][y][x >> 1] +
                                (T(9.0 / 16.0) * e9[1][1] +
                                 T(3.0 / 16.0) * (e9[1][si] + e9[sj][1]) +
                                 T(1.0 / 16.0) * e9[sj][si]);
                    U[f][(x + y) & 1][y][x >> 1] = v;
                    O.u[c][f] = v;
                }
            }
        }
        __syncthreads();
    } else if constexpr (UP) {
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const int b = t + s * NT;
            if (b >= nblk) continue;
            const int by = b / LX2, bx = b - by * LX2;
            const int cx = bx + 1, cy = by + 1;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int dx = (c == 1 || c == 2) ? 1 : 0, dy = (c == 1 || c == 3) ? 1 : 0;
                const int x = 2 * bx + dx, y = 2 * by + dy;
                const int sx = dx ? cx + 1 : cx - 1, sy = dy ? cy + 1 : cy - 1;
#pragma unroll
                for (int f = 0; f < NF; ++f)
                    U[f][(x + y) & 1][y][x >> 1] +=
                        T(9.0 / 16.0) * E[f][cy][cx] +
                        T(3.0 / 16.0) * (E[f][cy][sx] + E[f][sy][cx]) +
                        T(1.0 / 16.0) * E[f][sy][sx];
            }
        }
        __syncthreads();
    }

    // 3'. coarse down: f = R r + N(u) at every cell that can be updated.
    if (!UP && OWN && A.complete_f) {
        if (t < nblk) {
            const int by = t / LX2, bx = t - by * LX2;
            // all four cells computed without branches, kept only where the
            // cell can be updated
            auto cells_f = [&](auto c0_, auto c1_) {
                constexpr int c0 = decltype(c0_)::value, c1 = decltype(c1_)::value;
                T r[2][NF];
                resid2<c0, c1, true>(op, S, O, G, bx, by, R, r);
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int c = k ? c1 : c0;
                    const int x = 2 * bx + cdx(c), y = 2 * by + cdy(c);
                    const bool in = x >= 1 && y >= 1 && x < LX - 1 && y < LY - 1;
#pragma unroll
                    for (int f = 0; f < NF; ++f)
                        fr[0][c][f] = in ? fr[0][c][f] - r[k][f] : fr[0][c][f];
                }
            };
            cells_f(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
            cells_f(std::integral_constant<int, 2>{}, std::integral_constant<int, 3>{});
        }
        __syncthreads();
    } else if (!UP && A.complete_f) {
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const int b = t + s * NT;
            if (b >= nblk) continue;
            const int by = b / LX2, bx = b - by * LX2;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int dx = (c == 1 || c == 2) ? 1 : 0, dy = (c == 1 || c == 3) ? 1 : 0;
                const int x = 2 * bx + dx, y = 2 * by + dy;
                if (x < 1 || y < 1 || x >= LX - 1 || y >= LY - 1) continue;
                const int col = (x + y) & 1, oc = col ^ 1, k = x >> 1;
                const int ke = (x + 1) >> 1, kw = (x - 1) >> 1;
                T u[1][NF], ns[1][NF], r[1][NF];
                const T zero[1][NF] = {};
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    u[0][f] = U[f][col][y][k];
                    ns[0][f] = (U[f][oc][y][ke] + U[f][oc][y][kw]) +
                               (U[f][oc][y + 1][k] + U[f][oc][y - 1][k]);
                }
                op.resid(u, ns, zero, {xkr[s][c]}, {pbr[s][c]}, {wr[s][c]}, r);
#pragma unroll
                for (int f = 0; f < NF; ++f) fr[s][c][f] -= r[0][f];
            }
        }
        // every N(u) above reads u as loaded: no pass may write before all
        // waves are done (waves with a second owned block finish later)
        __syncthreads();
    }

    // 4. red-black passes; pass p is exact on cells at distance >= p.  The
    //    colour is a compile-time constant inside `pass`, so the per-cell
    //    register arrays are indexed statically.
    auto pass = [&](auto colc, int p) {
        constexpr int colour = decltype(colc)::value;
        constexpr int oc = colour ^ 1;
        if constexpr (OWN) {
            if (t >= nblk) return;
            const int by = t / LX2, bx = t - by * LX2;
            // both cells of the colour are relaxed without branches, then stored
            // where the pass updates them
            constexpr int c0 = colour == 0 ? 0 : 2, c1 = colour == 0 ? 1 : 3;
            T u[2][NF], ns[2][NF], f2[2][NF];
            nsum_own<c0>(S, O, G, bx, by, ns[0]);
            nsum_own<c1>(S, O, G, bx, by, ns[1]);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                u[0][f] = O.u[c0][f];
                u[1][f] = O.u[c1][f];
                f2[0][f] = fr[0][c0][f];
                f2[1][f] = fr[0][c1][f];
            }
            op.relax(u, ns, f2, {xkr[0][c0], xkr[0][c1]}, {pbr[0][c0], pbr[0][c1]},
                     {wr[0][c0], wr[0][c1]});
            // (a cell the pass does not update gets its own value back: only
            // its owner writes it, so the store is branch-free)
            auto put = [&](auto cc_, const T (&u)[NF]) {
                constexpr int c = decltype(cc_)::value;
                const int x = 2 * bx + cdx(c), y = 2 * by + cdy(c);
                const bool in = x >= p && y >= p && x < LX - p && y < LY - p;
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    const T v = in ? u[f] : O.u[c][f];
                    U[f][colour][y][bx] = v;
                    O.u[c][f] = v;
                }
            };
            put(std::integral_constant<int, c0>{}, u[0]);
            put(std::integral_constant<int, c1>{}, u[1]);
            return;
        }
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const int b = t + s * NT;
            if (b >= nblk) continue;
            const int by = b / LX2, bx = b - by * LX2;
#pragma unroll
            for (int cc = 0; cc < 2; ++cc) {
                const int c = colour == 0 ? cc : 2 + cc;
                const int dx = (c == 1 || c == 2) ? 1 : 0, dy = (c == 1 || c == 3) ? 1 : 0;
                const int x = 2 * bx + dx, y = 2 * by + dy;
                if (x < p || y < p || x >= LX - p || y >= LY - p) continue;
                const int k = x >> 1, ke = (x + 1) >> 1, kw = (x - 1) >> 1;
                T u[1][NF], ns[1][NF], f1[1][NF];
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    u[0][f] = U[f][colour][y][k];
                    ns[0][f] = (U[f][oc][y][ke] + U[f][oc][y][kw]) +
                               (U[f][oc][y + 1][k] + U[f][oc][y - 1][k]);
                    f1[0][f] = fr[s][c][f];
                }
                op.relax(u, ns, f1, {xkr[s][c]}, {pbr[s][c]}, {wr[s][c]});
#pragma unroll
                for (int f = 0; f < NF; ++f) U[f][colour][y][k] = u[0][f];
            }
        }
    };
    // Neumann boundaries: halo cells outside the grid hold the even reflection
    // of interior cells (App. A ghost rule, extended through the halo).  A pass
    // also relaxes them as if they were cells; afterwards they are restored
    // from their mirror cells, x first, then y (corners get both reflections),
    // so every relaxed grid cell reads ghosts equal to its mirror's value from
    // before the pass, as in a global sweep.
    const bool mir_x = NEU && (g.bc & BC_NEUMANN_X) && (x0 < 0 || x0 + LX > g.m);
    const bool mir_y = NEU && (g.bc & BC_NEUMANN_Y) && (y0 < 0 || y0 + LY > g.n);
    auto restore_ghosts = [&]() {
        if (mir_x) {
            for (int q = t; q < 2 * H * LY; q += NT) {
                const int y = q / (2 * H), k = q - y * (2 * H);
                const int x = k < H ? k : LX - 2 * H + k;
                const int gx = x0 + x;
                if (gx >= 0 && gx < g.m) continue;
                const int xm = (GEN ? axis_index_any(gx, g.m, true) : axis_index(gx, g.m, true)) - x0;
#pragma unroll
                for (int f = 0; f < NF; ++f)
                    U[f][(x + y) & 1][y][x >> 1] = U[f][(xm + y) & 1][y][xm >> 1];
            }
            __syncthreads();
        }
        if (mir_y) {
            for (int q = t; q < 2 * H * LX; q += NT) {
                const int k = q / LX, x = q - k * LX;
                const int y = k < H ? k : LY - 2 * H + k;
                const int gy = y0 + y;
                if (gy >= 0 && gy < g.n) continue;
                const int ym = (GEN ? axis_index_any(gy, g.n, true) : axis_index(gy, g.n, true)) - y0;
#pragma unroll
                for (int f = 0; f < NF; ++f)
                    U[f][(x + y) & 1][y][x >> 1] = U[f][(x + ym) & 1][ym][x >> 1];
            }
            __syncthreads();
        }
    };
    for (int p = 1; p <= A.nsweep; ++p) {
        if (((p - 1) & 1) == 0) pass(std::integral_constant<int, 0>{}, p);
        else pass(std::integral_constant<int, 1>{}, p);
        __syncthreads();
        if constexpr (NEU) {
            restore_ghosts();
            if constexpr (OWN)
                if (mir_x || mir_y) load_own(S, G, O);
        }
    }

    // 5. interior u back to global memory, coalesced along rows.
    const int gx0 = tbx * tx, gy0 = tby * ty;
    for (int q = t; q < tx * ty; q += NT) {
        const int yi = q / tx, xi = q - yi * tx;
        const int x = xi + H, y = yi + H;
        const size_t gq = tat<GEN>(gx0 + xi, gy0 + yi, g);
#pragma unroll
        for (int f = 0; f < NF; ++f) A.uout[f][gq] = U[f][(x + y) & 1][y][x >> 1];
    }

    // 6. interior blocks: residual; down restricts it (and u), finest up sums r^2.
    double acc = 0.0;
    const int mc = g.m >> 1;
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        const int b = t + s * NT;
        if (b >= nblk) continue;
        const int by = b / LX2, bx = b - by * LX2;
        if (2 * bx < H || 2 * bx >= H + tx || 2 * by < H || 2 * by >= H + ty) continue;
        if (UP && !A.norm) continue;
        T su[NF], sr[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) { su[f] = T(0); sr[f] = T(0); }
        auto res_own = [&](auto c0_, auto c1_) {
            constexpr int c0 = decltype(c0_)::value, c1 = decltype(c1_)::value;
            T r[2][NF];
            resid2<c0, c1, false>(op, S, O, G, bx, by, R, r);
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    su[f] += O.u[k ? c1 : c0][f];
                    sr[f] += r[k][f];
                    acc += (double)r[k][f] * (double)r[k][f];
                }
        };
        if constexpr (OWN) {
            res_own(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
            res_own(std::integral_constant<int, 2>{}, std::integral_constant<int, 3>{});
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int dx = (c == 1 || c == 2) ? 1 : 0, dy = (c == 1 || c == 3) ? 1 : 0;
                const int x = 2 * bx + dx, y = 2 * by + dy;
                const int col = (x + y) & 1, oc = col ^ 1, k = x >> 1;
                const int ke = (x + 1) >> 1, kw = (x - 1) >> 1;
                T u[1][NF], ns[1][NF], f1[1][NF], r[1][NF];
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    u[0][f] = U[f][col][y][k];
                    ns[0][f] = (U[f][oc][y][ke] + U[f][oc][y][kw]) +
                               (U[f][oc][y + 1][k] + U[f][oc][y - 1][k]);
                    f1[0][f] = fr[s][c][f];
                }
                op.resid(u, ns, f1, {xkr[s][c]}, {pbr[s][c]}, {wr[s][c]}, r);
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    su[f] += u[0][f];
                    sr[f] += r[0][f];
                    acc += (double)r[0][f] * (double)r[0][f];
                }
            }
        }
        if constexpr (!UP) {
            const int I = (gx0 + 2 * bx - H) >> 1, J = (gy0 + 2 * by - H) >> 1;
            const size_t Q = (size_t)J * mc + I;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const T avg = T(0.25) * su[f];
                A.uH[f][Q] = avg;
                A.vH[f][Q] = avg;
                A.rH[f][Q] = T(0.25) * sr[f];
            }
            // coefficient fields of the coarse level, in the order of additions
            // of a plain 2x2 average: ((f00 + f10) + (f01 + f11)) / 4
            if constexpr (Op::XK)
                if (A.xkH) A.xkH[Q] = T(0.25) * ((xkr[s][0] + xkr[s][2]) + (xkr[s][3] + xkr[s][1]));
            if constexpr (Op::PB)
                if (A.pbH) A.pbH[Q] = T(0.25) * ((pbr[s][0] + pbr[s][2]) + (pbr[s][3] + pbr[s][1]));
        }
    }
    if constexpr (!UP) {
        // completed coarse-level right-hand side for the up launch
        if (A.complete_f) {
#pragma unroll
            for (int s = 0; s < SL; ++s) {
                const int b = t + s * NT;
                if (b >= nblk) continue;
                const int by = b / LX2, bx = b - by * LX2;
                if (2 * bx < H || 2 * bx >= H + tx || 2 * by < H || 2 * by >= H + ty) continue;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int dx = (c == 1 || c == 2) ? 1 : 0, dy = (c == 1 || c == 3) ? 1 : 0;
                    const size_t gq = tat<GEN>(gx0 + 2 * bx - H + dx, gy0 + 2 * by - H + dy, g);
#pragma unroll
                    for (int f = 0; f < NF; ++f) A.fout[f][gq] = fr[s][c][f];
                }
            }
        }
    } else {
        if (A.norm) {
            // per-block sum of r^2; k_norm_finalize adds them and decides
            const double bs = block_sum<NT>(acc, red);
            if (t == 0) A.part[pslot] = bs;
        }
    }
    }
};

// Body of one tile launch: the tile into LDS, its right-hand side into
// registers, then the computation.
// `vote` (VOTE, down): the stop flag may rise beside this launch and `saw` is the
// wave's look at it.  A wave that saw it up loads nothing; behind the barrier the looks
// of all waves decide for the workgroup, which returns if any saw it.
template <class Op, int TX, int TY, int HMAX, bool UP, bool NEU, bool GEN = false,
          bool EXACT = false, bool VOTE = false>
__device__ __forceinline__ void tile_body(const Op& op, const TileArgs<typename Op::real>& A,
                                          int tbx, int tby, int pslot, bool zero_in,
                                          bool vote = false, bool saw = false) {
    using W = TileWork<Op, TX, TY, HMAX, UP, NEU, GEN, EXACT>;
    __shared__ typename W::Lds S;
    const typename W::Geo G = W::geo(A, tbx, tby);
    typename W::Rhs R;
    if constexpr (UP) {
        // the right-hand side is first used after the prolongation, which
        // covers its latency
        W::load_direct(A, G, S, zero_in, [] {});
        __syncthreads();
        if (A.nsweep || A.norm) W::fetch_rhs(A, G, R);  // else only the correction is added
    } else {
        if (!VOTE || !saw) W::load_direct(A, G, S, zero_in, [&] { W::fetch_rhs(A, G, R); });
        if (VOTE && vote && (threadIdx.x & 63) == 0) S.saw[threadIdx.x >> 6] = saw;
        __syncthreads();
        if (VOTE && vote) {
            int any = 0;
#pragma unroll
            for (int w = 0; w < W::NT / 64; ++w) any |= S.saw[w];
            if (any) return;
        }
    }
    W::compute(op, A, G, S, R, pslot);
}

// One level of one grid: (m / tx) (n / ty) workgroups of kTileThreads threads
// (tx, ty divide m, n), and with a pending norm one more, the first, which runs
// its stopping test.  The test used to be a launch of its own between the up
// launch that wrote the sums and the next cycle's finest down launch: 4.4 us and
// a launch gap of every cycle.  Beside the tiles it costs nothing.  The flag may
// rise while the waves of this launch look at it, so a workgroup's waves decide
// together (tile_body): it returns whole or runs whole.  A tile that ran beside the
// test that stops the cycles has written the other copy of u and the next level's
// arrays, all rewritten before they are read again, and not what it read; every
// launch behind this one returns at once.  (2048^2: 122.9 us without the vote, 123.1
// with it, 125.9 with one thread's look and a barrier of its own ahead of the loads.)
// VOTE: the kernel can run a pending norm's test (P.nparts).  Not taken, the vote cost
// a 16 x 16 launch 0.15 to 0.3 of its 5.6 to 11.1 us (behind a possible return the
// arguments are read after the barrier, not ahead of it), so most have a kernel
// without it (tile_launch).
template <class Op, int TX, int TY, int HMAX, bool UP, bool NEU, bool GEN, bool EXACT, bool VOTE>
__global__ void __launch_bounds__(kTileThreads) k_tile(Op op, TileArgs<typename Op::real> A,
                                                       const CycleState* stop, PendingNorm P) {
    int b = blockIdx.x, nt = gridDim.x;
    const bool vote = VOTE && P.nparts;
    bool saw = false;
    if (vote) {
        if (b == 0) {
            norm_finalize_body<kTileThreads>(P.part, P.nparts, P.st, P.hist, P.h2, P.tol,
                                             P.max_norms, P.diverge);
            return;
        }
        --b;
        --nt;
        saw = stopped_now(stop);
    } else if (stopped(stop)) {
        return;
    }
    const int tl = xcd_item(b, nt);
    const int tby = tl / A.ntx, tbx = tl - tby * A.ntx;
    tile_body<Op, TX, TY, HMAX, UP, NEU, GEN, EXACT, VOTE>(op, A, tbx, tby, tl, A.zero_in, vote,
                                                           saw);
}

// Batched launch: one level of many independent grids.  Each (grid, level)
// has its own arguments, operator constants and stop flag; the work list
// holds one entry per tile.
template <class Op>
struct BatchTile {
    Op op;
    TileArgs<typename Op::real> A;
    const CycleState* stop;
    int part_off;         // first slot of this grid's residual sums in A.part
    int ntx;              // tiles in x
};

struct BatchItem {
    int arg;              // index into the BatchTile array
    int tile;             // linear tile index within that grid level
};

// `first` set: the members with zero_in start from u = 0.
template <class Op, int TX, int TY, int HMAX, bool UP, bool NEU, bool EXACT>
__global__ void __launch_bounds__(kTileThreads) k_tile_batched(const BatchTile<Op>* __restrict__ args,
                                                      const BatchItem* __restrict__ items,
                                                      int nitems, int first) {
    const int b = xcd_item(blockIdx.x, nitems);
    const BatchItem it = items[b];
    const BatchTile<Op>& BA = args[it.arg];
    const int tby = it.tile / BA.ntx, tbx = it.tile - tby * BA.ntx;
    if (stopped(BA.stop)) return;  // (behind the record's loads: its pointer is one of them)
    tile_body<Op, TX, TY, HMAX, UP, NEU, false, EXACT>(BA.op, BA.A, tbx, tby,
                                                       BA.part_off + it.tile,
                                                       first && BA.A.zero_in);
}

// ---------------------------------------------------------------------------
// Persistent kernel: every level of at most CP_CELLS cells, in LDS, one
// workgroup.  Same V(nu1, nu2) cycle as the tiled levels; the coarsest grid is
// solved directly.
constexpr int CP_CELLS = 1024;  // largest level handled here (32 x 32)
constexpr int CP_TOTAL = 1368;  // cells of all its levels (1024 + 256 + 64 + 16 + 4, padded)
constexpr int CP_THREADS = CP_CELLS / 2;  // one thread per red-black pair of the largest level

// The top level of the persistent launches (or the coarsest, coarsest launches).
struct CoarseGeom {
    int bc;               // boundary conditions (BC_NEUMANN_X | BC_NEUMANN_Y bits)
    int m, n, lm;         // sides, log2 m
};

template <typename T>
struct CoarseArgs {
    CoarseGeom geo;
    T* u[3];              // top level u (in/out, global)
    const T* rr[3];       // top level restricted residual R r (global)
    const T* xk;          // phi^k on the top level (global)
    const T* pb;          // base phi on the top level (global)
    const T* pin;         // pinning weight on the top level (global; Op::PW)
    int nsw1, nsw2;       // half-sweeps down / up
    int complete_top;     // 1: rr holds R r (add N(u)); 0: rr is already the full f
    const double* G;      // Poisson: Green's matrix of the coarsest grid
    int newton_maxit;
    T newton_tol;
};

// When Newton's method on the coarsest grid may stop: after a step of at most `tol`
// (1 + |phi|) in every cell's phi, and in FP64 also once the error left by the step
// is known to be below that, so that no further step has to show it.  Divided by c
// times -Lap, the equation is the gradient of a convex function whose second
// derivative is at least mu = 1/(8 c/h^2) + min(al + W): 1/(c lam) for the largest
// eigenvalue lam <= 8/h^2 of -Lap, and g' >= 0.  A step s leaves a residual of at
// most |g''| s^2 / 2 per cell, |g''| <= 6 (1 + |phi|), in the second-order scheme 3/2
// (1 + |phi|) + |phi^k| / 2, hence an error of at most sqrt(NC) / 2 |g''| s^2 / mu, and
// NC <= 8.  (A bare test of s^2 against the tolerance left up to 2.3e-14 where c is
// large, al zero and phi small.)
template <class Op, typename T>
struct NewtonStop {
    T tol, w, v;   // the error bound holds where w s^2 <= v
    template <int NC>
    __device__ __forceinline__ NewtonStop(const Op& op, const T (&xk)[NC], const T (&pw)[NC],
                                          T tol_) : tol(tol_) {
        T g = T(9), al = op.op.al;
        if constexpr (Op::XK) {
            T xm = fabs(xk[0]);
#pragma unroll
            for (int a = 1; a < NC; ++a) xm = fmax(xm, fabs(xk[a]));
            g = T(2.25) + T(0.75) * xm;
        }
        if constexpr (Op::PW) {
            T wm = pw[0];
#pragma unroll
            for (int a = 1; a < NC; ++a) wm = fmin(wm, pw[a]);
            al += wm;
        }
        const T q = T(8) * op.op.k1;
        w = g * q;
        v = tol * (T(1) + q * al);
    }
    // (without branches: one thread waits for each)
    __device__ __forceinline__ bool operator()(T step, T xmax) const {
        const T lim = tol + tol * xmax, s2 = step * step;
        return (step <= lim) | ((sizeof(T) == 8) & (s2 <= lim) & (w * s2 <= v));
    }
};

// Coarsest grid, MPFC: eliminate kappa and mu (kappa = f3 + e Lap phi,
// mu = f2 + g(phi) + al phi + Lap kappa) and solve the remaining equation
//   phi - c Lap(g(phi) + al phi + e Lap^2 phi) = f1 + c Lap(f2 + Lap f3)
// by Newton with Gaussian elimination (NC <= 8 unknowns), one thread.  Its
// solution is the unique solution of the three-field system.  Every array is
// indexed with compile-time indices only (row swaps are selects), so that it
// lives in registers.
template <class Op, int NC>
__device__ __forceinline__ void coarse_solve_mpfc(const Op& op, typename Op::real (&u)[3][NC],
                                                  const typename Op::real (&f)[3][NC],
                                                  const typename Op::real (&xk)[NC],
                                                  const typename Op::real (&pb)[NC],
                                                  const typename Op::real (&pw)[NC], int m, int lm,
                                                  int n, int bc, int maxit, typename Op::real tol) {
    using T = typename Op::real;
    const T c = op.op.c, e = op.op.e, al = op.op.al;
    // Laplacian matrix of the m x n grid with its ghost rule (periodic: a
    // 2-cell direction couples each cell twice to its one neighbour; Neumann:
    // the ghost beside a boundary cell is that cell itself).
    const bool nx = bc & BC_NEUMANN_X, ny = bc & BC_NEUMANN_Y;
    T L[NC][NC];
#pragma unroll
    for (int a = 0; a < NC; ++a) {
        const int i = a & (m - 1), j = a >> lm;
        const int e0 = axis_index(i + 1, m, nx) + (j << lm);
        const int e1 = axis_index(i - 1, m, nx) + (j << lm);
        const int e2 = i + (axis_index(j + 1, n, ny) << lm);
        const int e3 = i + (axis_index(j - 1, n, ny) << lm);
#pragma unroll
        for (int b = 0; b < NC; ++b) {
            const int k = (b == a ? -4 : 0) + (b == e0) + (b == e1) + (b == e2) + (b == e3);
            L[a][b] = T(k) * op.op.ih2;
        }
    }
    auto lap = [&](const T (&v)[NC], T (&out)[NC]) {
#pragma unroll
        for (int a = 0; a < NC; ++a) {
            T s = 0;
#pragma unroll
            for (int b = 0; b < NC; ++b) s += L[a][b] * v[b];
            out[a] = s;
        }
    };
    T f1[NC], f2[NC], f3[NC], t1[NC], t2[NC], rhs[NC];
#pragma unroll
    for (int a = 0; a < NC; ++a) { f1[a] = f[0][a]; f2[a] = f[1][a]; f3[a] = f[2][a]; }
    // rhs = f1 + c Lap(f2 + Lap f3)
    lap(f3, t1);
#pragma unroll
    for (int a = 0; a < NC; ++a) t1[a] += f2[a];
    lap(t1, t2);
#pragma unroll
    for (int a = 0; a < NC; ++a) rhs[a] = f1[a] + c * t2[a];
    // L3 = Lap^3 (constant part of the Jacobian)
    T L3[NC][NC];
#pragma unroll
    for (int b = 0; b < NC; ++b) {
        T col[NC], l1[NC];
#pragma unroll
        for (int a = 0; a < NC; ++a) col[a] = L[a][b];
        lap(col, l1);
        lap(l1, col);
#pragma unroll
        for (int a = 0; a < NC; ++a) L3[a][b] = col[a];
    }
    T x[NC], xkv[NC], pbv[NC], alv[NC];
#pragma unroll
    for (int a = 0; a < NC; ++a) {
        x[a] = u[0][a];
        xkv[a] = Op::XK ? xk[a] : T(0);
        pbv[a] = Op::PB ? pb[a] : T(0);
        alv[a] = Op::PW ? al + pw[a] : al;  // pinning: W added to the phi coefficient
    }
    const NewtonStop<Op, T> done(op, xkv, pw, tol);
    for (int it = 0; it < maxit; ++it) {
        // residual R = x - c Lap(g(x) + al x + e Lap^2 x) - rhs
        T w[NC], d[NC], R[NC], J[NC][NC + 1];
        lap(x, t1);
        lap(t1, t2);
#pragma unroll
        for (int a = 0; a < NC; ++a) {
            w[a] = nl_value<T, (Op::XK ? 2 : 1), Op::PB>(x[a], pbv[a], xkv[a]) + alv[a] * x[a] + e * t2[a];
            d[a] = nl_lin<T, (Op::XK ? 2 : 1), true>(pbv[a] + x[a], xkv[a]) + alv[a];
        }
        lap(w, t1);
#pragma unroll
        for (int a = 0; a < NC; ++a) R[a] = x[a] - c * t1[a] - rhs[a];
        // Jacobian J = I - c (Lap diag(d) + e Lap^3), augmented with -R
#pragma unroll
        for (int a = 0; a < NC; ++a) {
#pragma unroll
            for (int b = 0; b < NC; ++b)
                J[a][b] = (a == b ? T(1) : T(0)) - c * (L[a][b] * d[b] + e * L3[a][b]);
            J[a][NC] = -R[a];
        }
        // Gaussian elimination with partial pivoting (one division per pivot)
        T ip[NC];
#pragma unroll
        for (int k = 0; k < NC; ++k) {
#pragma unroll
            for (int r = k + 1; r < NC; ++r) {
                const bool sw = fabs(J[r][k]) > fabs(J[k][k]);
#pragma unroll
                for (int cc = k; cc <= NC; ++cc) {
                    const T hi = J[k][cc], lo = J[r][cc];
                    J[k][cc] = sw ? lo : hi;
                    J[r][cc] = sw ? hi : lo;
                }
            }
            ip[k] = T(1) / J[k][k];
#pragma unroll
            for (int r = k + 1; r < NC; ++r) {
                const T fct = J[r][k] * ip[k];
#pragma unroll
                for (int cc = k; cc <= NC; ++cc) J[r][cc] -= fct * J[k][cc];
            }
        }
#pragma unroll
        for (int k = NC - 1; k >= 0; --k) {
            T s = J[k][NC];
#pragma unroll
            for (int cc = k + 1; cc < NC; ++cc) s -= J[k][cc] * t1[cc];
            t1[k] = s * ip[k];
        }
        T smax = 0, xmax = 0;
#pragma unroll
        for (int a = 0; a < NC; ++a) {
            x[a] += t1[a];
            smax = fmax(smax, fabs(t1[a]));
            xmax = fmax(xmax, fabs(x[a]));
        }
        if (done(smax, xmax)) break;
    }
    // recover kappa and mu
    lap(x, t1);
#pragma unroll
    for (int a = 0; a < NC; ++a) t1[a] = f3[a] + e * t1[a];
    lap(t1, t2);
#pragma unroll
    for (int a = 0; a < NC; ++a) {
        u[2][a] = t1[a];
        u[1][a] = f2[a] + nl_value<T, (Op::XK ? 2 : 1), Op::PB>(x[a], pbv[a], xkv[a]) + alv[a] * x[a] + t2[a];
        u[0][a] = x[a];
    }
}

// The same problem in the Laplacian's eigenvectors, for the grids whose
// eigenvectors are the sign patterns w_k(a) = (-1)^popcount(k & a) (cell a =
// i + j m): every 2 x 2 grid, and 4 x 2 or 2 x 4 with a periodic 4-cell axis.
// With K = -Lap = diag(lam) in that basis, coefficients z of phi, and mode k's
// equation divided by c lam_k, the Newton system is
//   (1/(c lam) + e lam^2) delta + (W^T D W) delta = residual   (k > 0),
// symmetric positive definite (D = g' + al + W >= 0), its matrix's entry (i, j)
// the transform of D at i xor j: L D L^T without pivoting.  The mean (k = 0)
// does not change in the iteration.  One thread: 1.6 us where the elimination
// above takes 3 us (2 x 2); on 4 x 2 the elimination was about 15 us of a 34 us
// coarse launch.
template <int NC, typename T>
__device__ __forceinline__ void walsh(const T (&x)[NC], T (&out)[NC], T scale) {
#pragma unroll
    for (int a = 0; a < NC; ++a) out[a] = scale * x[a];
#pragma unroll
    for (int h = 1; h < NC; h *= 2)
#pragma unroll
        for (int a = 0; a < NC; ++a)
            if (!(a & h)) {
                const T p = out[a], q = out[a + h];
                out[a] = p + q;
                out[a + h] = p - q;
            }
}

template <class Op, int NC>
__device__ __forceinline__ void coarse_solve_walsh(const Op& op, typename Op::real (&u)[3][NC],
                                                   const typename Op::real (&f)[3][NC],
                                                   const typename Op::real (&xk)[NC],
                                                   const typename Op::real (&pb)[NC],
                                                   const typename Op::real (&pw)[NC], int m, int n,
                                                   int bc, int maxit, typename Op::real tol) {
    using T = typename Op::real;
    constexpr int SCH = Op::XK ? 2 : 1;
    constexpr T SC = T(1) / T(NC), TINY = sizeof(T) == 8 ? T(1e-280) : T(1e-30);
    const T c = op.op.c, e = op.op.e, al = op.op.al, ih2 = op.op.ih2;
    T lam[NC], icl[NC], s[NC], rho[NC], z[NC], fh[3][NC], x[NC], G[NC], D[NC], Gh[NC], Dh[NC];
    // eigenvalue of an axis' sign pattern: 2 cells, (1, -1): 4/h^2 periodic, 2/h^2
    // Neumann; 4 cells, patterns alternating in bit 0, bit 1, both: 4, 2, 2 / h^2
    auto axis = [&](int k, int len, bool neu) {
        if (len == 2) return k ? (neu ? T(2) : T(4)) : T(0);
        return k == 0 ? T(0) : (k == 1 ? T(4) : T(2));
    };
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        const int kx = k & (m - 1), ky = m == 2 ? k >> 1 : k >> 2;
        lam[k] = ih2 * (axis(kx, m, bc & BC_NEUMANN_X) + axis(ky, n, bc & BC_NEUMANN_Y));
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) walsh<NC>(f[i], fh[i], SC);
    walsh<NC>(u[0], z, SC);
    {
        T cl[NC];
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const T t = c * lam[k];
            rho[k] = fh[0][k] - t * (fh[1][k] - lam[k] * fh[2][k]);
            cl[k] = k ? fmax(t, TINY) : T(1);
        }
        recip_ge1_n(cl, icl);
#pragma unroll
        for (int k = 0; k < NC; ++k) s[k] = icl[k] + e * lam[k] * lam[k];
    }
    const NewtonStop<Op, T> done(op, xk, pw, tol);
    z[0] = rho[0];
    for (int it = 0; it < maxit; ++it) {
        walsh<NC>(z, x, T(1));
#pragma unroll
        for (int a = 0; a < NC; ++a) {
            const T ala = Op::PW ? al + pw[a] : al;
            nl_both<T, SCH, true, Op::PB>(x[a], pb[a], xk[a], G[a], D[a]);
            G[a] += ala * x[a];
            D[a] += ala;
        }
        walsh<NC>(G, Gh, SC);
        walsh<NC>(D, Dh, SC);
        // L D L^T of the modes 1 ... NC - 1, the right-hand side carried along
        T M[NC][NC], b[NC];
#pragma unroll
        for (int i = 1; i < NC; ++i) {
#pragma unroll
            for (int j = 1; j <= i; ++j) M[i][j] = Dh[i ^ j] + (i == j ? s[i] : T(0));
            b[i] = (rho[i] - z[i]) * icl[i] - e * lam[i] * lam[i] * z[i] - Gh[i];
        }
        T ip[NC];
#pragma unroll
        for (int k = 1; k < NC; ++k) {
            const T pv[1] = {M[k][k]};
            T rc[1];
            recip_ge1_n(pv, rc);
            ip[k] = rc[0];
#pragma unroll
            for (int i = k + 1; i < NC; ++i) {
                const T l = M[i][k] * ip[k];
#pragma unroll
                for (int j = k + 1; j <= i; ++j) M[i][j] -= l * M[j][k];
                b[i] -= l * b[k];
            }
        }
        T smax = 0, xmax = fabs(z[0]);
#pragma unroll
        for (int k = NC - 1; k >= 1; --k) {
            T t = b[k];
#pragma unroll
            for (int i = k + 1; i < NC; ++i) t -= M[i][k] * b[i];
            b[k] = t * ip[k];
            z[k] += b[k];
            smax += fabs(b[k]);
            xmax += fabs(z[k]);
        }
        // (smax and xmax: sums over the modes, no cell's value is larger)
        if (done(smax, xmax)) break;
    }
    // kappa = f3 + e Lap phi, mu = f2 + g(phi) + al phi + Lap kappa
    walsh<NC>(z, u[0], T(1));
#pragma unroll
    for (int a = 0; a < NC; ++a)
        G[a] = nl_value<T, SCH, Op::PB>(u[0][a], pb[a], xk[a]) + (Op::PW ? al + pw[a] : al) * u[0][a];
    walsh<NC>(G, Gh, SC);
    T kh[NC], mh[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        kh[k] = fh[2][k] - e * lam[k] * z[k];
        mh[k] = fh[1][k] + Gh[k] - lam[k] * kh[k];
    }
    walsh<NC>(kh, u[2], T(1));
    walsh<NC>(mh, u[1], T(1));
}

// The persistent workgroup.  A thread owns one row of a 2x2 block of every
// level it works on: a red and a black cell, beside each other, with unknowns,
// right-hand side and coefficients in registers while the level is relaxed.
// Threads 2b and 2b + 1 hold the rows dy = 0, 1 of block b, so that a block's sums
// (the restriction) are one lane exchange.  The unknowns are in LDS as a red and
// a black array with one entry per thread: a cell's inner x neighbour is the
// owner's other cell, its other three neighbours are of the other array.
// Levels of at most 64 threads (8 x 8 cells and below) run in the first wave
// alone: LDS instructions of one wave complete in order, so its half-sweeps
// need no workgroup barrier.
//
// Bound by latency: a chain of dependent phases (about 46 for V(2,2) from
// 32 x 32), each an LDS round trip (64 clocks and up) and the local solve, some
// 40 FP64 operations that a wave issues in order, 8 clocks each when dependent.
// V(2,2) in FP64 from 32 x 32, in the V-cycle graph of a 1024^2 grid: one cell
// per thread and half-sweep, everything re-read from LDS, 24.7 us; a whole block
// per thread (half the waves, twice the instructions in each) 23.1; this one
// 18.4.
template <class Op, int NC, bool NEU>
struct CoarseWork {
    using T = typename Op::real;
    typedef T T2 __attribute__((ext_vector_type(2)));
    static constexpr int NF = Op::NF;
    static constexpr int CPH = CP_TOTAL / 2;   // cells of one colour, all levels
    struct Lds {
        T u[2][NF][CPH], f[2][NF][CPH], v[2][NF][CPH];   // [colour][field][thread of a level]
        T xk[2][Op::XK ? CPH : 1], pb[2][Op::PB ? CPH : 1], pw[2][Op::PW ? CPH : 1];
        T E[NF][CP_CELLS / 4];  // u_H - v_H of the level below, row-major
    };
    struct Lev {
        int m, n, lm, off, l;   // sides, log2 m, first LDS entry, level number
        __device__ __forceinline__ Lev coarser() const {
            return {m >> 1, n >> 1, lm - 1, off + ((m * n) >> 1), l + 1};
        }
        __device__ __forceinline__ Lev finer() const {
            return {m << 1, n << 1, lm + 1, off - 2 * m * n, l - 1};
        }
        __device__ __forceinline__ bool coarsest() const { return m == 2 || n == 2; }
        __device__ __forceinline__ bool one_wave() const { return m * n <= 128; }
    };
    // A thread's cells of a level: LDS entries of the neighbours outside its own
    // row of the block (h: x neighbour of the red and of the black cell, vi and vo:
    // y neighbour inside and outside the block), and the E entries it reads.  At
    // a Neumann edge the neighbour index is the block itself (the ghost of the
    // correction), and gh, gv say that a cell's own value is its ghost.
    struct Pos {
        bool on, gh[2], gv;
        int dy, bx, by, q, h[2], vi, vo;
        int e, ew, ee, eo, eow, eoe;
    };
    struct Own {
        T u[2][NF], f[2][NF], xk[2], pb[2], pw[2];
    };

    static __device__ __forceinline__ Pos pos(const Lev& L, int bc) {
        const int bw = L.m >> 1, bh = L.n >> 1, nt = 2 * bw * bh;
        const bool nx = NEU && (bc & BC_NEUMANN_X), ny = NEU && (bc & BC_NEUMANN_Y);
        Pos P;
        P.on = (int)threadIdx.x < nt;
        const int t = threadIdx.x & (nt - 1), b = t >> 1, dy = t & 1;
        P.dy = dy;
        P.bx = b & (bw - 1);
        P.by = b >> (L.lm - 1);
        const bool ge = nx && P.bx == bw - 1, gw = nx && P.bx == 0;
        const bool go = ny && P.by == (dy ? bh - 1 : 0);
        const int xe = ge ? P.bx : (P.bx + 1) & (bw - 1);
        const int xw = gw ? P.bx : (P.bx - 1) & (bw - 1);
        const int r = P.by * bw;
        const int ro = (go ? P.by : (P.by + (dy ? 1 : -1)) & (bh - 1)) * bw;
        P.gh[0] = dy ? ge : gw;
        P.gh[1] = dy ? gw : ge;
        P.gv = go;
        P.q = L.off + t;
        P.h[0] = L.off + 2 * (r + (dy ? xe : xw)) + dy;
        P.h[1] = L.off + 2 * (r + (dy ? xw : xe)) + dy;
        P.vi = L.off + (t ^ 1);
        P.vo = L.off + 2 * (ro + P.bx) + (dy ^ 1);
        P.e = r + P.bx; P.ew = r + xw; P.ee = r + xe;
        P.eo = ro + P.bx; P.eow = ro + xw; P.eoe = ro + xe;
        return P;
    }
    // LDS writes of the workgroup (WG) or of this wave before, reads after.
    template <bool WG>
    static __device__ __forceinline__ void sync() {
        if constexpr (WG) {
            __syncthreads();
        } else {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }
    // Value of the thread that holds the block's other row.
    static __device__ __forceinline__ int swap1(int x) {
        return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xf, 0xf, true);  // quad_perm 1, 0, 3, 2
    }
    static __device__ __forceinline__ T other_row(T x) {
        if constexpr (sizeof(T) == 8)
            return __hiloint2double(swap1(__double2hiint(x)), swap1(__double2loint(x)));
        else
            return __int_as_float(swap1(__float_as_int(x)));
    }
    // level l has 2^l times the top level's spacing: scale 1/h^2 (and h^2) by exact powers of two
    static __device__ __forceinline__ Op opl(const Op& top, int l) {
        Op o = top;
        if constexpr (NF == 3) { o.op.ih2 = ldexp(top.op.ih2, -2 * l); o.op.derive(); }
        else { o.ih2 = ldexp(top.ih2, -2 * l); o.h2 = ldexp(top.h2, 2 * l); }
        return o;
    }
    static __device__ __forceinline__ void load_own(const Lds& S, const Pos& P, Own& O) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
#pragma unroll
            for (int f = 0; f < NF; ++f) { O.u[c][f] = S.u[c][f][P.q]; O.f[c][f] = S.f[c][f][P.q]; }
            O.xk[c] = Op::XK ? S.xk[c][P.q] : T(0);
            O.pb[c] = Op::PB ? S.pb[c][P.q] : T(0);
            O.pw[c] = Op::PW ? S.pw[c][P.q] : T(0);
        }
    }
    // Neighbour sums of the cell of colour C, every field: x neighbours first.
    template <int C>
    static __device__ __forceinline__ void nsum(const Lds& S, const Pos& P, const Own& O,
                                                T (&ns)[NF]) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            T h = S.u[C ^ 1][f][P.h[C]], vo = S.u[C ^ 1][f][P.vo];
            const T vi = S.u[C ^ 1][f][P.vi];
            if constexpr (NEU) {
                h = P.gh[C] ? O.u[C][f] : h;
                vo = P.gv ? O.u[C][f] : vo;
            }
            ns[f] = (h + O.u[C ^ 1][f]) + (vi + vo);
        }
    }
    // f - N(u) (ZF: -N(u)) at both cells.
    template <bool ZF>
    static __device__ __forceinline__ void resid(const Op& o, const Lds& S, const Pos& P,
                                                 const Own& O, T (&r)[2][NF]) {
        T ns[2][NF];
        const T zero[2][NF] = {};
        nsum<0>(S, P, O, ns[0]);
        nsum<1>(S, P, O, ns[1]);
        o.resid(O.u, ns, ZF ? zero : O.f, O.xk, O.pb, O.pw, r);
    }
    // f = R r + N(u).
    static __device__ __forceinline__ void complete(const Op& o, const Lds& S, const Pos& P, Own& O) {
        T r[2][NF];
        resid<true>(o, S, P, O, r);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int f = 0; f < NF; ++f) O.f[c][f] -= r[c][f];
    }
    // Half-sweep of one colour, into registers and LDS.
    template <int C>
    static __device__ __forceinline__ void pass(const Op& o, Lds& S, const Pos& P, Own& O) {
        T u[1][NF], ns[1][NF], f1[1][NF];
        nsum<C>(S, P, O, ns[0]);
#pragma unroll
        for (int f = 0; f < NF; ++f) { u[0][f] = O.u[C][f]; f1[0][f] = O.f[C][f]; }
        o.relax(u, ns, f1, {O.xk[C]}, {O.pb[C]}, {O.pw[C]});
#pragma unroll
        for (int f = 0; f < NF; ++f) S.u[C][f][P.q] = O.u[C][f] = u[0][f];
    }
    template <bool WG>
    static __device__ __forceinline__ void sweeps(const Op& o, Lds& S, const Pos& P, Own& O,
                                                  int nsw) {
#pragma unroll 1
        for (int p = 0; p < nsw; p += 2) {
            if (P.on) pass<0>(o, S, P, O);
            sync<WG>();
            if (P.on) pass<1>(o, S, P, O);
            sync<WG>();
        }
    }
    // Down part of one level: completed right-hand side, sweeps, residual and
    // its restriction (with u and the coefficients) onto the next level.
    template <bool WG>
    static __device__ __forceinline__ void down(const Op& top, Lds& S, const Lev& L, int bc,
                                                int nsw, bool compl_f) {
        const Op o = opl(top, L.l);
        const Pos P = pos(L, bc);
        Own O;
        if (P.on) {
            load_own(S, P, O);
            if (compl_f) complete(o, S, P, O);
        }
        if (compl_f) sync<WG>();  // every N(u) reads u as loaded
        if (P.on) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    S.v[c][f][P.q] = O.u[c][f];
                    S.f[c][f][P.q] = O.f[c][f];
                }
        }
        sweeps<WG>(o, S, P, O, nsw);
        if (P.on) {
            T r[2][NF];
            resid<false>(o, S, P, O, r);
            // coarse cell (bx, by): the block's averages, the u part stored by the
            // first of its two threads, the residual by the second
            const Lev C = L.coarser();
            const int q = C.off + 2 * ((P.by >> 1) * (C.m >> 1) + (P.bx >> 1)) + (P.by & 1);
            const int col = (P.bx ^ P.by) & 1;
            T* d = P.dy ? &S.f[0][0][0] : &S.u[0][0][0];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const T su = O.u[0][f] + O.u[1][f], sr = r[0][f] + r[1][f];
                const T au = T(0.25) * (su + other_row(su)), ar = T(0.25) * (sr + other_row(sr));
                d[(col * NF + f) * CPH + q] = P.dy ? ar : au;
            }
            auto avg = [&](const T (&x)[2]) {
                const T sx = x[0] + x[1];
                return T(0.25) * (sx + other_row(sx));
            };
            if constexpr (Op::XK) S.xk[col][q] = avg(O.xk);
            if constexpr (Op::PB) S.pb[col][q] = avg(O.pb);
            if constexpr (Op::PW) S.pw[col][q] = avg(O.pw);
        }
        sync<WG>();
    }
    // Up part: the correction E prolonged onto u, sweeps, and this level's own
    // correction u - v for the level above (on the top level S.u is the result).
    template <bool WG>
    static __device__ __forceinline__ void up(const Op& top, Lds& S, const Lev& L, int bc, int nsw) {
        const Op o = opl(top, L.l);
        const Pos P = pos(L, bc);
        Own O;
        if (P.on) {
            load_own(S, P, O);
            const int cw = P.dy;  // colour of the row's west cell
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                // bilinear, one axis after the other: the west and east cell's
                // column in the block's own coarse row and in the outer one
                const T* E = S.E[f];
                const T c0 = T(0.75) * E[P.e], c1 = T(0.75) * E[P.eo];
                const T w = T(0.75) * (c0 + T(0.25) * E[P.ew]) + T(0.25) * (c1 + T(0.25) * E[P.eow]);
                const T e = T(0.75) * (c0 + T(0.25) * E[P.ee]) + T(0.25) * (c1 + T(0.25) * E[P.eoe]);
                O.u[0][f] += cw ? e : w;
                O.u[1][f] += cw ? w : e;
                S.u[0][f][P.q] = O.u[0][f];
                S.u[1][f][P.q] = O.u[1][f];
            }
        }
        sync<WG>();
        sweeps<WG>(o, S, P, O, nsw);
        if (P.on && L.l > 0) {
            const int row = (2 * P.by + P.dy) << L.lm;
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int f = 0; f < NF; ++f)
                    S.E[f][row + 2 * P.bx + (c ^ P.dy)] = O.u[c][f] - S.v[c][f][P.q];
        }
        sync<WG>();
    }
    // Coarsest grid: the direct solve, and E = u - v for the level above.
    static __device__ __forceinline__ void solve(const Op& top, const CoarseArgs<T>& A, Lds& S,
                                                 const Lev& L, int bc, bool compl_f) {
        const Op o = opl(top, L.l);
        const int t = threadIdx.x;
        if (compl_f) {
            const Pos P = pos(L, bc);
            if (P.on) {
                Own O;
                load_own(S, P, O);
                complete(o, S, P, O);
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int f = 0; f < NF; ++f) S.f[c][f][P.q] = O.f[c][f];
            }
            sync<false>();
        }
        // colour and LDS entry of grid cell a = j m + i
        auto at = [&](int a, int& col) {
            const int i = a & (L.m - 1), j = a >> L.lm;
            col = (i ^ j) & 1;
            return L.off + 2 * ((j >> 1) * (L.m >> 1) + (i >> 1)) + (j & 1);
        };
        int col;
        if constexpr (NF == 3) {
            // the host launches the instantiation whose NC equals the coarsest cell count
            if (t == 0 && L.m * L.n == NC) {
                T u[3][NC], f[3][NC], xk[NC], pb[NC], pw[NC];
#pragma unroll
                for (int a = 0; a < NC; ++a) {
                    const int q = at(a, col);
#pragma unroll
                    for (int k = 0; k < 3; ++k) { u[k][a] = S.u[col][k][q]; f[k][a] = S.f[col][k][q]; }
                    xk[a] = Op::XK ? S.xk[col][q] : T(0);
                    pb[a] = Op::PB ? S.pb[col][q] : T(0);
                    pw[a] = Op::PW ? S.pw[col][q] : T(0);
                }
                const bool cosines = NEU && NC == 8 &&
                                     (bc & (L.m == 4 ? BC_NEUMANN_X : BC_NEUMANN_Y));
                if (NEU && NC == 8 && cosines)
                    coarse_solve_mpfc<Op, NC>(o, u, f, xk, pb, pw, L.m, L.lm, L.n, bc,
                                              A.newton_maxit, A.newton_tol);
                else
                    coarse_solve_walsh<Op, NC>(o, u, f, xk, pb, pw, L.m, L.n, NEU ? bc : 0,
                                               A.newton_maxit, A.newton_tol);
#pragma unroll
                for (int a = 0; a < NC; ++a) {
                    const int q = at(a, col);
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        S.E[k][a] = u[k][a] - S.u[col][k][q];
                        S.u[col][k][q] = u[k][a];
                    }
                }
            }
        } else {
            // Poisson: w = G f + mean(v) (the mean of w is free; the correction
            // stays mean-free); u holds v
            const int nc = L.m * L.n;
            if (t < nc) {
                T mv = T(0), w = T(0);
                for (int k = 0; k < nc; ++k) {
                    const int q = at(k, col);
                    mv += S.u[col][0][q];
                    w += (T)A.G[t * nc + k] * S.f[col][0][q];
                }
                w += mv / T(nc);
                const int q = at(t, col);
                S.E[0][t] = w - S.u[col][0][q];
                S.u[col][0][q] = w;
            }
        }
        sync<false>();
    }
    // Every level from L down to the coarsest and back, in one wave.
    static __device__ __forceinline__ void cycle_wave(const Op& top, const CoarseArgs<T>& A, Lds& S,
                                                      Lev L, int bc) {
        const int l0 = L.l;
#pragma unroll 1
        for (; !L.coarsest(); L = L.coarser())
            down<false>(top, S, L, bc, A.nsw1, L.l > 0 || A.complete_top);
        solve(top, A, S, L, bc, L.l > 0 || A.complete_top);
#pragma unroll 1
        while (L.l > l0) {
            L = L.finer();
            up<false>(top, S, L, bc, A.nsw2);
        }
    }

    static __device__ __forceinline__ void run(const Op& top, const CoarseArgs<T>& A, Lds& S,
                                               const CycleState* stop) {
        Lev L = {A.geo.m, A.geo.n, A.geo.lm, 0, 0};
        const int bc = A.geo.bc;
        const Pos P = pos(L, bc);
        const size_t g0 = ((size_t)(2 * P.by + P.dy) << L.lm) + 2 * P.bx;  // the west cell
        const bool done = stopped(stop);  // looked at behind the loads, in flight with them
        if (P.on) {
            constexpr int NV = 2 * NF + (Op::XK ? 1 : 0) + (Op::PB ? 1 : 0) + (Op::PW ? 1 : 0);
            const T* src[NV];
            T *red[NV], *black[NV];
            int k = 0;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                src[k] = A.u[f]; red[k] = S.u[0][f]; black[k++] = S.u[1][f];
                src[k] = A.rr[f]; red[k] = S.f[0][f]; black[k++] = S.f[1][f];
            }
            if constexpr (Op::XK) { src[k] = A.xk; red[k] = S.xk[0]; black[k++] = S.xk[1]; }
            if constexpr (Op::PB) { src[k] = A.pb; red[k] = S.pb[0]; black[k++] = S.pb[1]; }
            if constexpr (Op::PW) { src[k] = A.pin; red[k] = S.pw[0]; black[k++] = S.pw[1]; }
            T2 v[NV];
#pragma unroll
            for (int i = 0; i < NV; ++i) v[i] = *(const T2*)(src[i] + g0);
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                red[i][P.q] = P.dy ? v[i].y : v[i].x;
                black[i][P.q] = P.dy ? v[i].x : v[i].y;
            }
        }
        if (done) return;
        __syncthreads();
#pragma unroll 1
        for (; !L.one_wave(); L = L.coarser())
            down<true>(top, S, L, bc, A.nsw1, L.l > 0 || A.complete_top);
        if (threadIdx.x < 64) cycle_wave(top, A, S, L, bc);
        __syncthreads();
#pragma unroll 1
        while (L.l > 0) {
            L = L.finer();
            up<true>(top, S, L, bc, A.nsw2);
        }
        if (P.on) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const T r = S.u[0][f][P.q], b = S.u[1][f][P.q];
                *(T2*)(A.u[f] + g0) = P.dy ? T2{b, r} : T2{r, b};
            }
        }
    }
};

template <class Op, int NC, bool NEU>
__global__ void __launch_bounds__(CP_THREADS) k_coarse_persistent(
    Op op_top, CoarseArgs<typename Op::real> A, const CycleState* stop) {
    __shared__ typename CoarseWork<Op, NC, NEU>::Lds S;
    CoarseWork<Op, NC, NEU>::run(op_top, A, S, stop);
}

// Batched: workgroup b runs the coarse levels of grid b.
template <class Op>
struct BatchCoarse {
    Op op;
    CoarseArgs<typename Op::real> A;
    const CycleState* stop;
};

template <class Op, int NC, bool NEU>
__global__ void __launch_bounds__(CP_THREADS) k_coarse_persistent_batched(
    const BatchCoarse<Op>* __restrict__ args) {
    __shared__ typename CoarseWork<Op, NC, NEU>::Lds S;
    const BatchCoarse<Op>& B = args[blockIdx.x];
    CoarseWork<Op, NC, NEU>::run(B.op, B.A, S, B.stop);
}

// ---------------------------------------------------------------------------
// Coarsest level of a grid whose sides are not all powers of two.  Such a grid
// is coarsened while both sides of the next level stay even, so its coarsest
// level (m x n, both even, at most CG_CELLS cells; 64 x 50 for 512 x 400) can
// be far larger than the 2 x 2 grid the dense Newton solve is made for.  One
// workgroup of CG_THREADS threads; every index is general (no power-of-two
// masks), and each axis follows its ghost rule.
constexpr int CG_THREADS = 1024;
constexpr int CG_CELLS = 4096;
constexpr int CG_SLOTS = CG_CELLS / 2 / CG_THREADS;  // cells of one colour per thread

// MPFC system: complete the FAS right-hand side f = R r + N(u), then relax the
// level by A.nsw2 half-sweeps of the red-black collective smoother (the
// coarsest "solve" is approximate; the finer levels correct what it leaves).
// u lives in LDS; f and the coefficients of each thread's cells in registers.
template <class Op, bool NEU>
__global__ void __launch_bounds__(CG_THREADS) k_coarsest_sweeps(Op op,
                                                                CoarseArgs<typename Op::real> A,
                                                                const CycleState* stop) {
    using T = typename Op::real;
    constexpr int NF = Op::NF;
    __shared__ T Su[NF][CG_CELLS];
    if (stopped(stop)) return;
    const int t = threadIdx.x;
    const int m = A.geo.m, n = A.geo.n, N = m * n, mh = m >> 1;
    const bool nbx = NEU && (A.geo.bc & BC_NEUMANN_X), nby = NEU && (A.geo.bc & BC_NEUMANN_Y);
    for (int q = t; q < N; q += CG_THREADS) {
#pragma unroll
        for (int f = 0; f < NF; ++f) Su[f][q] = A.u[f][q];
    }
    __syncthreads();
    auto nsum = [&](const T* a, int i, int j) {
        const int ie = i + 1 < m ? i + 1 : (nbx ? m - 1 : 0);
        const int iw = i > 0 ? i - 1 : (nbx ? 0 : m - 1);
        const int jn = j + 1 < n ? j + 1 : (nby ? n - 1 : 0);
        const int js = j > 0 ? j - 1 : (nby ? 0 : n - 1);
        const int r = j * m;
        return (a[ie + r] + a[iw + r]) + (a[i + jn * m] + a[i + js * m]);
    };
    // slot s of colour c of this thread: cell (i, j), or q = -1 for none
    auto cell = [&](int c, int s, int& i, int& j) {
        const int q2 = t + s * CG_THREADS;
        if (q2 >= (N >> 1)) return -1;
        j = q2 / mh;
        i = 2 * (q2 - j * mh) + ((j + c) & 1);
        return j * m + i;
    };
    T fr[2][CG_SLOTS][NF], xkr[2][CG_SLOTS], pbr[2][CG_SLOTS], wr[2][CG_SLOTS];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int s = 0; s < CG_SLOTS; ++s) {
#pragma unroll
            for (int f = 0; f < NF; ++f) fr[c][s][f] = T(0);
            xkr[c][s] = T(0);
            pbr[c][s] = T(0);
            wr[c][s] = T(0);
            int i = 0, j = 0;
            const int q = cell(c, s, i, j);
            if (q < 0) continue;
            if constexpr (Op::XK) xkr[c][s] = A.xk[q];
            if constexpr (Op::PB) pbr[c][s] = A.pb[q];
            if constexpr (Op::PW) wr[c][s] = A.pin[q];
            T u[1][NF], ns[1][NF], r[1][NF];
            const T zero[1][NF] = {};
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                u[0][f] = Su[f][q];
                ns[0][f] = nsum(Su[f], i, j);
                fr[c][s][f] = A.rr[f][q];
            }
            if (A.complete_top) {
                op.resid(u, ns, zero, {xkr[c][s]}, {pbr[c][s]}, {wr[c][s]}, r);
#pragma unroll
                for (int f = 0; f < NF; ++f) fr[c][s][f] -= r[0][f];
            }
        }
    }
    __syncthreads();  // every N(u) above read u as loaded
    auto pass = [&](auto colc) {
        constexpr int c = decltype(colc)::value;
#pragma unroll
        for (int s = 0; s < CG_SLOTS; ++s) {
            int i = 0, j = 0;
            const int q = cell(c, s, i, j);
            if (q < 0) continue;
            T u[1][NF], ns[1][NF], f1[1][NF];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                u[0][f] = Su[f][q];
                ns[0][f] = nsum(Su[f], i, j);
                f1[0][f] = fr[c][s][f];
            }
            op.relax(u, ns, f1, {xkr[c][s]}, {pbr[c][s]}, {wr[c][s]});
#pragma unroll
            for (int f = 0; f < NF; ++f) Su[f][q] = u[0][f];
        }
    };
    for (int p = 0; p < A.nsw2; ++p) {
        if ((p & 1) == 0) pass(std::integral_constant<int, 0>{});
        else pass(std::integral_constant<int, 1>{});
        __syncthreads();
    }
    for (int q = t; q < N; q += CG_THREADS) {
#pragma unroll
        for (int f = 0; f < NF; ++f) A.u[f][q] = Su[f][q];
    }
}

// Poisson problem -Lap_h w = f on the same coarsest level, solved exactly in
// the separable eigenbasis of the operator: with V_x (m x m) and V_y (n x n)
// the orthonormal eigenvectors of the one-dimensional second difference under
// each axis' boundary rule (columns: modes) and lam the eigenvalue sums,
//   w = V_y [ (V_y^T F V_x) / lam ] V_x^T + mean(v),
// the (0, 0) mode dropped (1/lam stored as 0), F the m x n grid function f.
// A.G holds V_x (row i: cell, column k: mode), then V_y, then 1/lam (row l:
// y mode, column k: x mode).  v is u as loaded (the restricted iterate): the
// correction keeps mean zero, as the dense Green's-matrix solve does.
template <typename T>
__global__ void __launch_bounds__(CG_THREADS) k_coarsest_poisson(PoissonOp<T> op, CoarseArgs<T> A,
                                                                 const CycleState* stop) {
    __shared__ T S0[CG_CELLS];
    __shared__ T S1[CG_CELLS];
    __shared__ double red[CG_THREADS / 64];
    __shared__ double mean_v;
    if (stopped(stop)) return;
    const int t = threadIdx.x;
    const int m = A.geo.m, n = A.geo.n, N = m * n;
    const bool nbx = A.geo.bc & BC_NEUMANN_X, nby = A.geo.bc & BC_NEUMANN_Y;
    const double* Vx = A.G;
    const double* Vy = Vx + (size_t)m * m;
    const double* il = Vy + (size_t)n * n;
    double sv = 0.0;
    for (int q = t; q < N; q += CG_THREADS) {
        S0[q] = A.u[0][q];
        sv += (double)S0[q];
    }
    const double tot = block_sum<CG_THREADS>(sv, red);  // contains a barrier
    if (t == 0) mean_v = tot / (double)N;
    for (int q = t; q < N; q += CG_THREADS) {
        const int j = q / m, i = q - j * m;
        const int ie = i + 1 < m ? i + 1 : (nbx ? m - 1 : 0);
        const int iw = i > 0 ? i - 1 : (nbx ? 0 : m - 1);
        const int jn = j + 1 < n ? j + 1 : (nby ? n - 1 : 0);
        const int js = j > 0 ? j - 1 : (nby ? 0 : n - 1);
        T f = A.rr[0][q];
        if (A.complete_top) {
            const T u[1][1] = {{S0[q]}}, zero[1][1] = {};
            const T ns[1][1] = {
                {(S0[ie + j * m] + S0[iw + j * m]) + (S0[i + jn * m] + S0[i + js * m])}};
            T r[1][1];
            op.resid(u, ns, zero, {T(0)}, {T(0)}, {T(0)}, r);
            f -= r[0][0];
        }
        S1[q] = f;
    }
    __syncthreads();
    // S0 = F V_x   (row j, column k)
    for (int q = t; q < N; q += CG_THREADS) {
        const int j = q / m, k = q - j * m;
        double s = 0.0;
        for (int i = 0; i < m; ++i) s += (double)S1[j * m + i] * Vx[(size_t)i * m + k];
        S0[q] = (T)s;
    }
    __syncthreads();
    // S1 = (V_y^T S0) / lam   (row l, column k)
    for (int q = t; q < N; q += CG_THREADS) {
        const int l = q / m, k = q - l * m;
        double s = 0.0;
        for (int j = 0; j < n; ++j) s += Vy[(size_t)j * n + l] * (double)S0[j * m + k];
        S1[q] = (T)(s * il[q]);
    }
    __syncthreads();
    // S0 = V_y S1   (row j, column k)
    for (int q = t; q < N; q += CG_THREADS) {
        const int j = q / m, k = q - j * m;
        double s = 0.0;
        for (int l = 0; l < n; ++l) s += Vy[(size_t)j * n + l] * (double)S1[l * m + k];
        S0[q] = (T)s;
    }
    __syncthreads();
    // w = S0 V_x^T + mean(v)
    const double mv = mean_v;
    for (int q = t; q < N; q += CG_THREADS) {
        const int j = q / m, i = q - j * m;
        double s = 0.0;
        for (int k = 0; k < m; ++k) s += (double)S0[j * m + k] * Vx[(size_t)i * m + k];
        A.u[0][q] = (T)(s + mv);
    }
}

}  // namespace mpfc
