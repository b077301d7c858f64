// Three-dimensional form of the step: the schemes of Sec. 3.1 / 3.2 and the
// multigrid of App. B with the seven-point Laplacian (the paper notes that the
// extension to three dimensions is straightforward).  Periodic m x n x l grids
// with power-of-two sides, cell (i, j, k) at (k n + j) m + i, FP64.
//
// Kernels are global-memory passes: a red-black half-sweep (two cells of a colour
// per thread), the residual with the 2x2x2 restriction of u, r and phi^k, the
// completion of a coarse right-hand side, the trilinear prolongation and
// correction, and the residual norm (a 2x2x2 block per thread).  On the larger
// levels every pass is bound by memory and streams its level once; the levels of at
// most 4096 cells run in one workgroup.
//
// Storage inside the solver is split by colour: a level of N cells holds its
// red cells ((i + j + k) even) in the first N/2 entries and its black cells in
// the last N/2, each half in (k, j, i/2) order (sidx).  A half-sweep then reads
// and writes its own colour contiguously and reads the other colour as
// neighbours, so no cache line is fetched or written back for half of its
// bytes.  The caller's arrays stay in natural order (at3); the per-step
// kernels convert on the way in and out.  Workgroups take their cells in
// XCD-contiguous order (xcd_item), so the neighbouring rows and planes a
// workgroup reads are mostly in its own XCD's L2.
#pragma once
#include "step.hpp"
#include "tiles.hpp"

namespace mpfc {

struct Grid3 {
    int m, n, l;      // cells along x, y, z (powers of two)
    int lm, ln, ll;   // their log2
};

// Natural index (the caller's arrays).
__device__ __forceinline__ size_t at3(int i, int j, int k, const Grid3& g) {
    return ((((size_t)k << g.ln) + (size_t)j) << g.lm) + (size_t)i;
}
__device__ __forceinline__ size_t cells3(const Grid3& g) { return (size_t)g.m * g.n * g.l; }
// Colour-split index (the solver's arrays).
__device__ __forceinline__ size_t sidx(int i, int j, int k, const Grid3& g) {
    const size_t half = cells3(g) >> 1;
    return (((i + j + k) & 1) ? half : 0) + ((((size_t)k << g.ln) + (size_t)j) << (g.lm - 1)) +
           (size_t)(i >> 1);
}
// Cell (i, j, k) of colour-split entry t.
__device__ __forceinline__ void split_cell(size_t t, const Grid3& g, int& i, int& j, int& k) {
    const size_t half = cells3(g) >> 1;
    const int c = t >= half ? 1 : 0;
    const size_t r = t - (c ? half : 0);
    const int ii = (int)(r & (size_t)((g.m >> 1) - 1));
    const size_t row = r >> (g.lm - 1);
    j = (int)(row & (size_t)(g.n - 1));
    k = (int)(row >> g.ln);
    i = 2 * ii + ((j + k + c) & 1);
}
// Entry handled by thread `threadIdx.x` of workgroup blockIdx.x, blocks dealt
// XCD-contiguously.
__device__ __forceinline__ size_t item3() {
    return (size_t)xcd_item(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
}

// Sum of the six face neighbours (periodic wrap-around), colour-split storage.
__device__ __forceinline__ double nsum6(const double* __restrict__ f, int i, int j, int k,
                                        const Grid3& g) {
    const int ip = (i + 1) & (g.m - 1), im = (i - 1) & (g.m - 1);
    const int jp = (j + 1) & (g.n - 1), jm = (j - 1) & (g.n - 1);
    const int kp = (k + 1) & (g.l - 1), km = (k - 1) & (g.l - 1);
    return ((f[sidx(ip, j, k, g)] + f[sidx(im, j, k, g)]) + (f[sidx(i, jp, k, g)] + f[sidx(i, jm, k, g)])) +
           (f[sidx(i, j, kp, g)] + f[sidx(i, j, km, g)]);
}
// The same in natural storage.
__device__ __forceinline__ double nsum6n(const double* __restrict__ f, int i, int j, int k,
                                         const Grid3& g) {
    const int ip = (i + 1) & (g.m - 1), im = (i - 1) & (g.m - 1);
    const int jp = (j + 1) & (g.n - 1), jm = (j - 1) & (g.n - 1);
    const int kp = (k + 1) & (g.l - 1), km = (k - 1) & (g.l - 1);
    return ((f[at3(ip, j, k, g)] + f[at3(im, j, k, g)]) + (f[at3(i, jp, k, g)] + f[at3(i, jm, k, g)])) +
           (f[at3(i, j, kp, g)] + f[at3(i, j, km, g)]);
}

// MPFC system N(u) = f in three dimensions (App. B.1 / B.2 with the seven-point
// Laplacian): the same algebra as in two dimensions with the centre weight 6.
template <int SCHEME, bool NEWTON>
struct MpfcOp3 {
    static constexpr int NF = 3;
    static constexpr bool XK = SCHEME == 2;
    LevelOp<double> op;   // derived with centre weight 6
    __device__ __forceinline__ void apply(const double* u, const double* ns, double xk,
                                          double* N) const {
        N[0] = u[0] - op.k1 * (ns[1] - 6.0 * u[1]);
        N[1] = u[1] - nl_value<double, SCHEME, false>(u[0], 0.0, xk) - op.al * u[0] -
               op.ih2 * (ns[2] - 6.0 * u[2]);
        N[2] = u[2] - op.e1 * (ns[0] - 6.0 * u[0]);
    }
    // J_loc delta = f - N(u), J_loc = [[1, a, 0], [-d, 1, b], [ec, 0, 1]] with
    // a = 6c/h^2, b = 6/h^2, ec = 6e/h^2, d = al + g'(phi) (Newton) or Picard's.
    __device__ __forceinline__ void relax(double* u, const double* ns, const double* f,
                                          double xk) const {
        double g, d;
        nl_both<double, SCHEME, NEWTON, false>(u[0], 0.0, xk, g, d);
        const double r1 = f[0] - (u[0] - op.k1 * (ns[1] - 6.0 * u[1]));
        const double r2 = f[1] - (u[1] - g - op.al * u[0] - op.ih2 * (ns[2] - 6.0 * u[2]));
        const double r3 = f[2] - (u[2] - op.e1 * (ns[0] - 6.0 * u[0]));
        const double dm = (r2 + (op.dd0 + d) * r1 - op.b * r3) * recip_ge1(op.det0 + op.a * d);
        const double dx = r1 - op.a * dm;
        u[0] += dx;
        u[1] += dm;
        u[2] += r3 - op.ec * dx;
    }
};

// Poisson problem -Lap_h w = b of the -1 norm, same interface.
struct PoissonOp3 {
    static constexpr int NF = 1;
    static constexpr bool XK = false;
    double ih2, h2;
    __device__ __forceinline__ void apply(const double* u, const double* ns, double,
                                          double* N) const {
        N[0] = (6.0 * u[0] - ns[0]) * ih2;
    }
    __device__ __forceinline__ void relax(double* u, const double* ns, const double* f,
                                          double) const {
        u[0] = (h2 * f[0] + ns[0]) * (1.0 / 6.0);
    }
};

// Fields of one level.
struct L3 {
    double* u[3];
    const double* f[3];
    const double* xk;   // phi^k on this level (scheme 2)
};

// One half-sweep: every cell of colour `colour` ((i + j + k) even = 0, red).
// Cells of one colour only read the other colour, so the update is in place.
template <class Op>
__global__ void __launch_bounds__(256) k3_relax(Op op, Grid3 g, L3 A, int colour,
                                                const CycleState* st) {
    if (stopped(st)) return;
    const size_t half = cells3(g) >> 1;
    const size_t t = item3();
    if (t >= half) return;
    int i, j, k;
    const size_t q = (colour ? half : 0) + t;
    split_cell(q, g, i, j, k);
    constexpr int NF = Op::NF;
    double u[NF], ns[NF], fv[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        u[f] = A.u[f][q];
        ns[f] = nsum6(A.u[f], i, j, k, g);
        fv[f] = A.f[f][q];
    }
    op.relax(u, ns, fv, Op::XK ? A.xk[q] : 0.0);
#pragma unroll
    for (int f = 0; f < NF; ++f) A.u[f][q] = u[f];
}

// The same with two neighbouring cells of the colour per thread, for m >= 4: every
// load but the one x-neighbour outside is 16 bytes (rows and halves are even and
// the arrays 256-byte aligned), so a wave makes half as many.  Bound by memory: a
// half-sweep moves 52 bytes a cell.  128^3: 19.1 -> 17.0 us (6.4 TB/s), 64^3
// 4.5 -> 3.7, 32^3 3.3 -> 2.9; the Poisson problem's on 128^3 7.6 -> 5.3.
constexpr int RX_THREADS = 64;
template <class Op>
__global__ void __launch_bounds__(RX_THREADS) k3_relax2(Op op, Grid3 g, L3 A, int colour,
                                                        const CycleState* st) {
    if (stopped(st)) return;
    const size_t half = cells3(g) >> 1;
    const size_t t = 2 * item3();
    if (t >= half) return;
    const int mh = g.m >> 1;
    const int x2 = (int)(t & (size_t)(mh - 1));
    const size_t row = t >> (g.lm - 1);
    const int j = (int)(row & (size_t)(g.n - 1)), k = (int)(row >> g.ln);
    const bool odd = (j + k + colour) & 1;  // the cells' other x-neighbours: at x2 + 1, else x2 - 1
    const size_t own = colour ? half : 0, oth = half - own;
    auto ent = [&](int x, int jj, int kk) {
        return oth + ((((size_t)(kk & (g.l - 1)) << g.ln) + (size_t)(jj & (g.n - 1))) << (g.lm - 1)) +
               (size_t)(x & (mh - 1));
    };
    const size_t yp = ent(x2, j + 1, k), ym = ent(x2, j - 1, k), zp = ent(x2, j, k + 1),
                 zm = ent(x2, j, k - 1), xe = ent(odd ? x2 + 2 : x2 - 1, j, k);
    auto two = [](const double* p) { return *reinterpret_cast<const double2*>(p); };
    constexpr int NF = Op::NF;
    double u[2][NF], ns[2][NF], fv[2][NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const double* v = A.u[f];
        const double2 a = two(v + own + t), b = two(v + oth + t), w = two(A.f[f] + own + t);
        const double2 n = two(v + yp), s = two(v + ym), o = two(v + zp), i = two(v + zm);
        const double e = v[xe];
        u[0][f] = a.x; u[1][f] = a.y;
        fv[0][f] = w.x; fv[1][f] = w.y;
        ns[0][f] = (odd ? b.x + b.y : e + b.x) + (n.x + s.x) + (o.x + i.x);
        ns[1][f] = (odd ? b.y + e : b.x + b.y) + (n.y + s.y) + (o.y + i.y);
    }
    double2 xk{0.0, 0.0};
    if constexpr (Op::XK) xk = two(A.xk + own + t);
    op.relax(u[0], ns[0], fv[0], xk.x);
    op.relax(u[1], ns[1], fv[1], xk.y);
#pragma unroll
    for (int f = 0; f < NF; ++f)
        *reinterpret_cast<double2*>(A.u[f] + own + t) = double2{u[0][f], u[1][f]};
}

// Residual r = f - N(u) at the eight cells of the 2x2x2 block (I, J, K) of g, in
// turn to `cell(u, r, xk)`.  Of a cell's six neighbours three are in the block, so
// a thread makes 32 loads of each field instead of 56, of both colours: the cells
// (0, 0, 0) .. (1, 1, 1) have the colours of their parity, and the two cells of a
// row sit at the same offset of the two halves, so consecutive threads read
// consecutive entries.  (Restriction from 128^3: 32.0 -> 29.8 us, from 32^3 8.8 -> 7.2.)
template <class Op, class Cell>
__device__ __forceinline__ void block_residual3(const Op& op, const Grid3& g, const L3& A, int I,
                                                int J, int K, Cell&& cell) {
    constexpr int NF = Op::NF;
    const size_t half = cells3(g) >> 1;
    const int mh = g.m >> 1;
    auto ent = [&](int x2, int j, int k) {
        return ((((size_t)(k & (g.l - 1)) << g.ln) + (size_t)(j & (g.n - 1))) << (g.lm - 1)) +
               (size_t)(x2 & (mh - 1));
    };
    double u[2][2][2][NF];  // [z][y][x]
#pragma unroll
    for (int z = 0; z < 2; ++z)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const size_t e = ent(I, 2 * J + y, 2 * K + z);
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int f = 0; f < NF; ++f)
                    u[z][y][x][f] = A.u[f][(((x + y + z) & 1) ? half : 0) + e];
        }
#pragma unroll
    for (int z = 0; z < 2; ++z)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const int j = 2 * J + y, k = 2 * K + z;
            const size_t e = ent(I, j, k), ey = ent(I, y ? j + 1 : j - 1, k),
                         ez = ent(I, j, z ? k + 1 : k - 1);
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const size_t ex = ent(x ? I + 1 : I - 1, j, k);
                const size_t own = ((x + y + z) & 1) ? half : 0, oth = half - own;
                double ns[NF], N[NF], r[NF];
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    const double* v = A.u[f] + oth;
                    ns[f] = ((u[z][y][x ^ 1][f] + v[ex]) + (u[z][y ^ 1][x][f] + v[ey])) +
                            (u[z ^ 1][y][x][f] + v[ez]);
                }
                const double xk = Op::XK ? A.xk[own + e] : 0.0;
                op.apply(u[z][y][x], ns, xk, N);
#pragma unroll
                for (int f = 0; f < NF; ++f) r[f] = A.f[f][own + e] - N[f];
                cell(u[z][y][x], r, xk);
            }
        }
}

// Residual at the eight fine cells of each coarse cell and the 2x2x2 averages of
// u (into uH and vH), r (rH) and, if xkH is set, phi^k.  One thread per coarse
// cell, in natural coarse order.  g is the fine grid.
template <class Op>
__global__ void __launch_bounds__(256) k3_restrict(Op op, Grid3 g, L3 A, L3 H, double* vH0,
                                                   double* vH1, double* vH2, double* rH0,
                                                   double* rH1, double* rH2, double* xkH,
                                                   const CycleState* st) {
    if (stopped(st)) return;
    const Grid3 c{g.m >> 1, g.n >> 1, g.l >> 1, g.lm - 1, g.ln - 1, g.ll - 1};
    const size_t Qn = item3();
    if (Qn >= cells3(c)) return;
    const int I = (int)(Qn & (size_t)(c.m - 1));
    const int J = (int)((Qn >> c.lm) & (size_t)(c.n - 1));
    const int K = (int)(Qn >> (c.lm + c.ln));
    const size_t Q = sidx(I, J, K, c);
    constexpr int NF = Op::NF;
    double su[NF], sr[NF], sxk = 0.0;
#pragma unroll
    for (int f = 0; f < NF; ++f) { su[f] = 0.0; sr[f] = 0.0; }
    block_residual3(op, g, A, I, J, K, [&](const double* u, const double* r, double xk) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            su[f] += u[f];
            sr[f] += r[f];
        }
        sxk += xk;
    });
    double* vH[3] = {vH0, vH1, vH2};
    double* rH[3] = {rH0, rH1, rH2};
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        H.u[f][Q] = 0.125 * su[f];
        vH[f][Q] = 0.125 * su[f];
        rH[f][Q] = 0.125 * sr[f];
    }
    if (Op::XK && xkH) xkH[Q] = 0.125 * sxk;
}

// Coarse right-hand side of the FAS: fout = R r + N(u) with u the restricted
// iterate (A.f holds R r).
template <class Op>
__global__ void __launch_bounds__(256) k3_complete(Op op, Grid3 g, L3 A, double* f0, double* f1,
                                                   double* f2, const CycleState* st) {
    if (stopped(st)) return;
    const size_t q = item3();
    if (q >= cells3(g)) return;
    int i, j, k;
    split_cell(q, g, i, j, k);
    constexpr int NF = Op::NF;
    double u[NF], ns[NF], N[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        u[f] = A.u[f][q];
        ns[f] = nsum6(A.u[f], i, j, k, g);
    }
    op.apply(u, ns, Op::XK ? A.xk[q] : 0.0, N);
    double* fo[3] = {f0, f1, f2};
#pragma unroll
    for (int f = 0; f < NF; ++f) fo[f][q] = A.f[f][q] + N[f];
}

// u += trilinear interpolation of the coarse correction E = uH - vH: per axis 3/4
// of the parent's coarse index and 1/4 of the coarse neighbour on the fine cell's side.  One
// thread per pair of fine cells (2I, j, k), (2I + 1, j, k): they share the
// coarse parent, sit at the same offset of the two colour halves (so a wave
// reads and writes both halves contiguously) and need 12 coarse values
// between them.  g is the fine grid.
template <int NF>
__global__ void __launch_bounds__(256) k3_prolong(Grid3 g, L3 A, L3 H, const double* v0_,
                                                  const double* v1_, const double* v2_,
                                                  const CycleState* st) {
    if (stopped(st)) return;
    const size_t t = item3();
    if (t >= (cells3(g) >> 1)) return;
    const int I = (int)(t & (size_t)((g.m >> 1) - 1));
    const size_t row = t >> (g.lm - 1);
    const int j = (int)(row & (size_t)(g.n - 1)), k = (int)(row >> g.ln);
    const Grid3 c{g.m >> 1, g.n >> 1, g.l >> 1, g.lm - 1, g.ln - 1, g.ll - 1};
    // x: coarse I - 1, I, I + 1 (fine 2I takes I - 1 as its side, 2I + 1 takes I + 1)
    const int X[3] = {(I - 1) & (c.m - 1), I, (I + 1) & (c.m - 1)};
    const int Y[2] = {j >> 1, ((j >> 1) + ((j & 1) ? 1 : -1)) & (c.n - 1)};
    const int Z[2] = {k >> 1, ((k >> 1) + ((k & 1) ? 1 : -1)) & (c.l - 1)};
    const double w[2] = {0.75, 0.25};
    const double* vH[3] = {v0_, v1_, v2_};
    const size_t q0 = sidx(2 * I, j, k, g), q1 = sidx(2 * I + 1, j, k, g);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        double e[2][2][3];
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int x = 0; x < 3; ++x) {
                    const size_t Q = sidx(X[x], Y[y], Z[z], c);
                    e[z][y][x] = H.u[f][Q] - vH[f][Q];
                }
        // fine 2I: parent X[1], side X[0]; fine 2I + 1: parent X[1], side X[2]
        double v0 = 0.0, v1 = 0.0;
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    v0 += w[x] * w[y] * w[z] * e[z][y][x == 0 ? 1 : 0];
                    v1 += w[x] * w[y] * w[z] * e[z][y][x == 0 ? 1 : 2];
                }
        A.u[f][q0] += v0;
        A.u[f][q1] += v1;
    }
}

// The same prolongation with the coarse correction formed once in LDS (a launch
// that formed it in memory first cost 5 us and a gap per level), for fine
// grids with m >= 32 (n, l >= 4 hold on every fine level): a workgroup takes
// P3X x-pairs x P3Y rows x P3Z planes, whose coarse footprint (one coarse cell
// of margin on each side) is read from global memory once instead of twelve
// times per pair.  Same values, same order of operations as k3_prolong.
constexpr int P3X = 16, P3Y = 4, P3Z = 4;
template <int NF>
__global__ void __launch_bounds__(256) k3_prolong_blk(Grid3 g, L3 A, L3 H, const double* v0_,
                                                      const double* v1_, const double* v2_,
                                                      const CycleState* st) {
    static_assert(P3X * P3Y * P3Z == 256, "one x-pair per thread");
    constexpr int CXN = P3X + 2, CYN = P3Y / 2 + 2, CZN = P3Z / 2 + 2;
    __shared__ double Es[NF][CZN][CYN][CXN];
    if (stopped(st)) return;
    const int nbx = (g.m >> 1) / P3X, nby = g.n / P3Y;
    const int b = xcd_item(blockIdx.x, gridDim.x);
    const int bx = b % nbx, r = b / nbx, by = r % nby, bz = r / nby;
    const int I0 = bx * P3X, j0 = by * P3Y, k0 = bz * P3Z;
    const Grid3 c{g.m >> 1, g.n >> 1, g.l >> 1, g.lm - 1, g.ln - 1, g.ll - 1};
    const int cx0 = I0 - 1, cy0 = (j0 >> 1) - 1, cz0 = (k0 >> 1) - 1;
    const double* vH[3] = {v0_, v1_, v2_};
    for (int q = threadIdx.x; q < CXN * CYN * CZN; q += 256) {
        const int x = q % CXN, yz = q / CXN, y = yz % CYN, z = yz / CYN;
        const size_t Q = sidx((cx0 + x) & (c.m - 1), (cy0 + y) & (c.n - 1), (cz0 + z) & (c.l - 1), c);
#pragma unroll
        for (int f = 0; f < NF; ++f) Es[f][z][y][x] = H.u[f][Q] - vH[f][Q];
    }
    __syncthreads();
    const int tx = threadIdx.x & (P3X - 1), ty = (threadIdx.x / P3X) & (P3Y - 1),
              tz = threadIdx.x / (P3X * P3Y);
    const int I = I0 + tx, j = j0 + ty, k = k0 + tz;
    // local coarse indices: parent x tx + 1 with sides tx, tx + 2; parent y
    // (ty >> 1) + 1 with its side on the fine cell's side; z alike
    const int LY[2] = {(ty >> 1) + 1, (ty >> 1) + 1 + ((j & 1) ? 1 : -1)};
    const int LZ[2] = {(tz >> 1) + 1, (tz >> 1) + 1 + ((k & 1) ? 1 : -1)};
    const double w[2] = {0.75, 0.25};
    const size_t q0 = sidx(2 * I, j, k, g), q1 = sidx(2 * I + 1, j, k, g);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        double e[2][2][3];
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int x = 0; x < 3; ++x) e[z][y][x] = Es[f][LZ[z]][LY[y]][tx + x];
        double v0 = 0.0, v1 = 0.0;
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    v0 += w[x] * w[y] * w[z] * e[z][y][x == 0 ? 1 : 0];
                    v1 += w[x] * w[y] * w[z] * e[z][y][x == 0 ? 1 : 2];
                }
        A.u[f][q0] += v0;
        A.u[f][q1] += v1;
    }
}

// Per-block sums of r^2 = (f - N(u))^2 over all fields (the stopping test;
// k_norm_finalize / k_p_finalize turn them into the norm).  BLOCK: a 2x2x2 block per
// thread, so that u of both colours is read by one XCD.  128^3: 22.8 us (5.2 TB/s of
// the 56 bytes a cell must read), a cell per thread in 256 long ranges 32.4 us;
// blocks in a loop over a range 47 us (the next block's loads wait for the sums).
// Else a cell per thread: on at most RES_CELLS cells blocks leave fewer than 64
// workgroups, each a chain of eight residuals (32^3: 5.7 us against 3.6 with cells,
// 64 x 64 x 32 6.3 against 4.4; the Poisson problem's 3.8 against 3.0 and 3.9 against
// 3.3.  On 64^3 blocks take 7.0 and 4.0, cells in 256 ranges 6.9 and 5.1).
constexpr size_t RES_CELLS = 131072;
template <class Op, int NT, bool BLOCK>
__global__ void __launch_bounds__(NT) k3_resnorm(Op op, Grid3 g, L3 A, double* part,
                                                 const CycleState* st) {
    if (stopped(st)) return;
    __shared__ double red[NT / 64];
    constexpr int NF = Op::NF;
    double acc = 0.0;
    const size_t q = item3();
    if constexpr (BLOCK) {
        if (q < (cells3(g) >> 3)) {
            const int I = (int)(q & (size_t)((g.m >> 1) - 1));
            const int J = (int)((q >> (g.lm - 1)) & (size_t)((g.n >> 1) - 1));
            const int K = (int)(q >> (g.lm + g.ln - 2));
            block_residual3(op, g, A, I, J, K, [&](const double*, const double* r, double) {
#pragma unroll
                for (int f = 0; f < NF; ++f) acc += r[f] * r[f];
            });
        }
    } else if (q < cells3(g)) {
        int i, j, k;
        split_cell(q, g, i, j, k);
        double u[NF], ns[NF], N[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            u[f] = A.u[f][q];
            ns[f] = nsum6(A.u[f], i, j, k, g);
        }
        op.apply(u, ns, Op::XK ? A.xk[q] : 0.0, N);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const double r = A.f[f][q] - N[f];
            acc += r * r;
        }
    }
    const double bs = block_sum<NT>(acc, red);
    if (threadIdx.x == 0) part[blockIdx.x] = bs;
}

// ---- levels of at most CP3_CELLS cells: one persistent workgroup ---------------
// The small levels of a V-cycle are latency bound (a launch each for every
// half-sweep, restriction, completion and prolongation).  This kernel runs
// them all, from the first level of at most CP3_CELLS cells down to the
// coarsest and back, in one workgroup, with the same arithmetic as the
// per-level kernels: complete the top level's right-hand side, nu1 half-sweep
// pairs, restriction with completion, coarsest sweeps, trilinear correction,
// nu2 pairs; the top level's u returns to global memory.
//
// u lives in LDS, split by colour as in global memory, a cell's fields side by
// side (24 bytes: every bank pair once per half wave, and one address for three
// loads).  On the top level (up to 16^3) each thread owns the four cells
// (2 i2, 2 i2 + 1) x (2 K2, 2 K2 + 1) of one row and keeps their u, right-hand side
// and phi^k in registers: of a cell's six neighbours its thread holds two, and the
// eight fine cells of a coarse cell are in two lanes of a wave.  Levels of up to 512
// cells below it have a red-black pair per thread; from 128 cells down one wave
// runs them without workgroup barriers, and a 2 x 2 x 2 coarsest level stays in
// four lanes' registers.  Bound by the latency of the half-sweeps, which follow one
// another (20 of them on the coarsest level), and on the top level by the issue
// rate of one CU.  From 16^3 down it takes 38 us (16^3: some 22 us of it); the
// kernel from 8^3 down took 25 us and the twelve launches of the 16^3 level 56 us
// more, with a gap each.  Three steps on 128^3 (57 cycles): 28.5 -> 25.1 ms.
constexpr int CP3_CELLS = 4096;
constexpr int CP3_LOW = 592;      // all levels below the top one: 512 + 64 + 8 (+ padding)
constexpr int CP3_MAXLEV = 10;
constexpr int CP3_THREADS = CP3_CELLS / 4;

struct CoarseGeom3 {
    int nlev;
    int m[CP3_MAXLEV], n[CP3_MAXLEV], l[CP3_MAXLEV];
    int lm[CP3_MAXLEV], ln[CP3_MAXLEV];
    int off[CP3_MAXLEV];
};

struct CoarseArgs3 {
    CoarseGeom3 geo;
    double* u[3];          // top level u (in/out)
    const double* f[3];    // top level R r (complete_top = 1) or complete right-hand side
    const double* xk;      // top level phi^k (scheme 2)
    int complete_top;
    int nsw1, nsw2, nswc;  // half-sweep pairs down / up / on the coarsest level
};

// Each level's operator, formed on the host (in vector registers and per level,
// its constants cost the half-sweeps more than their loads).
template <class Op>
struct CoarseOps3 {
    Op o[CP3_MAXLEV];
};

// x of another lane of the quad (0xB1: lane ^ 1, 0x4E: lane ^ 2) or, 0x141, of the
// mirrored lane of the group of eight.
template <int CTRL>
__device__ __forceinline__ double lane_of(double x) {
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true));
}
// Sum over the lanes of an aligned group of eight, in each of them.
__device__ __forceinline__ double sum8(double x) {
    x += lane_of<0xB1>(x);
    x += lane_of<0x4E>(x);
    return x + lane_of<0x141>(x);
}

template <class Op>
__global__ void __launch_bounds__(CP3_THREADS) k3_coarse(CoarseOps3<Op> ops,
                                                         CoarseArgs3 A, const CycleState* st) {
    constexpr int NF = Op::NF;
    __shared__ double U0[CP3_CELLS / 2][2 * NF + 1];  // [pair][colour, field]
    __shared__ double U[CP3_LOW][NF], F[CP3_LOW][NF], V[CP3_LOW][NF];
    __shared__ double X[Op::XK ? CP3_LOW : 1];
    if (stopped(st)) return;
    const int t = threadIdx.x;
    const Op& op_top = ops.o[0];
    const CoarseGeom3& G = A.geo;
    const int L = G.nlev;

    // ---- top level: four cells per thread
    const int n0 = G.n[0], l0 = G.l[0], mh0 = G.m[0] >> 1, lh0 = G.lm[0] - 1;
    const int half0 = mh0 * n0 * l0;
    const bool act = t < (half0 >> 1);
    auto ent = [&](int x2, int j, int k) __attribute__((always_inline)) {
        return (((k & (l0 - 1)) * n0 + (j & (n0 - 1))) << lh0) + (x2 & (mh0 - 1));
    };
    // A thread's pairs (i2, j0, 2 K0 + z), z = 0, 1; plane z holds its red cell at
    // 2 i2 + s, s = jp ^ z.  Entries of the pair and of its neighbours (the other
    // x-neighbour of the cell of colour c in ex[z][c]).
    struct Place { int jp, i2, J0, K0, e0[2], ex[2][2], ey[2][2], ez[2]; };
    // (threads in the order of the pairs' entries, so a wave's loads are contiguous,
    // but the row's parity no higher than lane bit 5: the restriction adds the two)
    const int sh0 = lh0 < 5 ? lh0 : 5;
    auto place = [&](int t) __attribute__((always_inline)) {
        Place P;
        const int hi = t >> (sh0 + 1), r = hi >> (lh0 - sh0);
        P.jp = (t >> sh0) & 1;
        P.i2 = ((hi << sh0) & (mh0 - 1)) | (t & ((1 << sh0) - 1));
        P.J0 = r & ((n0 >> 1) - 1);
        P.K0 = r >> (G.ln[0] - 1);
        const int j = 2 * P.J0 + P.jp;
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            const int k = 2 * P.K0 + z, s = P.jp ^ z;
            P.e0[z] = ent(P.i2, j, k);
            P.ex[z][0] = ent(P.i2 + (s ? 1 : -1), j, k);
            P.ex[z][1] = ent(P.i2 + (s ? -1 : 1), j, k);
            P.ey[z][0] = ent(P.i2, j + 1, k);
            P.ey[z][1] = ent(P.i2, j - 1, k);
            P.ez[z] = ent(P.i2, j, z ? k + 1 : k - 1);
        }
        return P;
    };
    Place P = place(t);
    double ur[2][2][NF], fr[2][2][NF], xr[2][2];   // [plane][colour]
    if (act) {
        // u and phi^k first: the right-hand side, which one CU's loads take as long
        // for, arrives behind the N(u) of its completion
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int q = c * half0 + P.e0[z];
#pragma unroll
                for (int f = 0; f < NF; ++f) ur[z][c][f] = A.u[f][q];
                xr[z][c] = Op::XK ? A.xk[q] : 0.0;
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int f = 0; f < NF; ++f) fr[z][c][f] = A.f[f][c * half0 + P.e0[z]];
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int f = 0; f < NF; ++f) U0[P.e0[z]][c * NF + f] = ur[z][c][f];
    }
    __syncthreads();
    // neighbour sum of the thread's cell of colour c in plane z
    auto ns0 = [&](auto zc, auto cc, double (&ns)[NF]) __attribute__((always_inline)) {
        constexpr int z = decltype(zc)::value, c = decltype(cc)::value, oc = c ^ 1;
#pragma unroll
        for (int f = 0; f < NF; ++f)
            ns[f] = ((ur[z][oc][f] + U0[P.ex[z][c]][oc * NF + f]) +
                     (U0[P.ey[z][0]][oc * NF + f] + U0[P.ey[z][1]][oc * NF + f])) +
                    (ur[z ^ 1][oc][f] + U0[P.ez[z]][oc * NF + f]);
    };
    using Z0 = std::integral_constant<int, 0>;
    using Z1 = std::integral_constant<int, 1>;
    auto half_sweep0 = [&](auto cc) __attribute__((always_inline)) {
        constexpr int c = decltype(cc)::value;
        auto cell = [&](auto zc) __attribute__((always_inline)) {
            constexpr int z = decltype(zc)::value;
            double ns[NF];
            ns0(zc, cc, ns);
            op_top.relax(ur[z][c], ns, fr[z][c], xr[z][c]);
#pragma unroll
            for (int f = 0; f < NF; ++f) U0[P.e0[z]][c * NF + f] = ur[z][c][f];
        };
        if (act) {
            cell(Z0{});
            __builtin_amdgcn_sched_barrier(0);
            cell(Z1{});
        }
        __syncthreads();
    };
    auto sweeps0 = [&](int pairs) __attribute__((always_inline)) {
        for (int p = 0; p < pairs; ++p) {
            half_sweep0(Z0{});
            half_sweep0(Z1{});
        }
    };
    // N(u) of the thread's cell of colour c in plane z
    auto apply0 = [&](auto zc, auto cc, double (&N)[NF]) __attribute__((always_inline)) {
        constexpr int z = decltype(zc)::value, c = decltype(cc)::value;
        double ns[NF];
        ns0(zc, cc, ns);
        op_top.apply(ur[z][c], ns, xr[z][c], N);
    };
    // complete the right-hand side (a finest level's is complete)
    if (act) {
        const bool ct = A.complete_top;
        auto add = [&](auto zc, auto cc) __attribute__((always_inline)) {
            double N[NF];
            apply0(zc, cc, N);
#pragma unroll
            for (int f = 0; f < NF; ++f) fr[decltype(zc)::value][decltype(cc)::value][f] += ct ? N[f] : 0.0;
            __builtin_amdgcn_sched_barrier(0);
        };
        add(Z0{}, Z0{}); add(Z0{}, Z1{}); add(Z1{}, Z0{}); add(Z1{}, Z1{});
    }
    __syncthreads();  // every N(u) reads u as loaded

    // ---- levels below: entry of colour c at (i2, j, k): c half + (k n + j) m/2 + i2
    struct Lev { int m, n, l, lh, ln, half, off; };
    auto lev = [&](int l) __attribute__((always_inline)) {
        return Lev{G.m[l], G.n[l], G.l[l], G.lm[l] - 1, G.ln[l], (G.m[l] * G.n[l] * G.l[l]) >> 1,
                   G.off[l]};
    };
    auto lent = [&](const Lev& v, int x2, int j, int k) __attribute__((always_inline)) {
        return (((((k & (v.l - 1)) << v.ln) + (j & (v.n - 1))) << v.lh)) + (x2 & ((v.m >> 1) - 1));
    };
    // neighbour sum of the cell of colour c at (x2, j, k)
    auto nsl = [&](const Lev& v, int x2, int j, int k, int c, double (&ns)[NF]) __attribute__((always_inline)) {
        const int s = (j + k) & 1, o = v.off + (c ^ 1) * v.half;
        const int e = o + lent(v, x2, j, k), x = o + lent(v, x2 + ((s ^ c) ? 1 : -1), j, k);
        const int yp = o + lent(v, x2, j + 1, k), ym = o + lent(v, x2, j - 1, k);
        const int zp = o + lent(v, x2, j, k + 1), zm = o + lent(v, x2, j, k - 1);
#pragma unroll
        for (int f = 0; f < NF; ++f)
            ns[f] = ((U[e][f] + U[x][f]) + (U[yp][f] + U[ym][f])) + (U[zp][f] + U[zm][f]);
    };
    auto sync = [&](bool wave) __attribute__((always_inline)) {
        if (wave) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        } else {
            __syncthreads();
        }
    };
    // Each of these is run by every thread of the workgroup (wave = false, one
    // pass over at most CP3_THREADS items) or by the first wave alone.
    auto complete = [&](int l, bool wave) __attribute__((always_inline)) {
        const Lev v = lev(l);
        const Op& o = ops.o[l];
        for (int q = t; q < 2 * v.half; q += wave ? 64 : CP3_THREADS) {
            const int c = q >= v.half, e = q - c * v.half;
            const int x2 = e & ((v.m >> 1) - 1), j = (e >> v.lh) & (v.n - 1), k = e >> (v.lh + v.ln);
            double ns[NF], N[NF];
            nsl(v, x2, j, k, c, ns);
            o.apply(U[v.off + q], ns, Op::XK ? X[v.off + q] : 0.0, N);
#pragma unroll
            for (int f = 0; f < NF; ++f) F[v.off + q][f] += N[f];
        }
        sync(wave);
    };
    // A pair's u, right-hand side and phi^k stay in registers; its x-neighbour
    // within the pair too.
    auto sweeps = [&](int l, int pairs, bool wave) __attribute__((always_inline)) {
        const Lev v = lev(l);
        const Op& o = ops.o[l];
        const bool on = t < v.half;
        const int tt = on ? t : 0, b = v.off;
        const int x2 = tt & ((v.m >> 1) - 1), j = (tt >> v.lh) & (v.n - 1), k = tt >> (v.lh + v.ln);
        const int s = (j + k) & 1;
        const int xn[2] = {b + lent(v, x2 + (s ? 1 : -1), j, k), b + lent(v, x2 + (s ? -1 : 1), j, k)};
        const int yp = b + lent(v, x2, j + 1, k), ym = b + lent(v, x2, j - 1, k);
        const int zp = b + lent(v, x2, j, k + 1), zm = b + lent(v, x2, j, k - 1);
        double u[2][NF], fv[2][NF], xk[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int q = b + c * v.half + tt;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                u[c][f] = U[q][f];
                fv[c][f] = F[q][f];
            }
            xk[c] = Op::XK ? X[q] : 0.0;
        }
        auto half_sweep = [&](auto cc) __attribute__((always_inline)) {
            constexpr int c = decltype(cc)::value, oc = c ^ 1;
            const int oo = oc * v.half;
            if (on) {
                double ns[NF];
#pragma unroll
                for (int f = 0; f < NF; ++f)
                    ns[f] = ((u[oc][f] + U[oo + xn[c]][f]) + (U[oo + yp][f] + U[oo + ym][f])) +
                            (U[oo + zp][f] + U[oo + zm][f]);
                o.relax(u[c], ns, fv[c], xk[c]);
#pragma unroll
                for (int f = 0; f < NF; ++f) U[b + c * v.half + t][f] = u[c][f];
            }
            sync(wave);
        };
        for (int p = 0; p < pairs; ++p) {
            half_sweep(Z0{});
            half_sweep(Z1{});
        }
    };
    // 2 x 2 x 2 cells: both neighbours along an axis are one cell, and lane
    // j + 2 k holds the pair (j, k), so the other pairs are one lane exchange away.
    auto sweeps_cube2 = [&](int l, int pairs) __attribute__((always_inline)) {
        const Op& o = ops.o[l];
        if (t < 4) {
            const int b = G.off[l] + t;
            double u[2][NF], fv[2][NF], xk[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    u[c][f] = U[b + 4 * c][f];
                    fv[c][f] = F[b + 4 * c][f];
                }
                xk[c] = Op::XK ? X[b + 4 * c] : 0.0;
            }
            for (int p = 0; p < pairs; ++p) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    double ns[NF];
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        const double w = u[c ^ 1][f];
                        ns[f] = 2.0 * ((w + lane_of<0xB1>(w)) + lane_of<0x4E>(w));
                    }
                    o.relax(u[c], ns, fv[c], xk[c]);
                }
            }
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int f = 0; f < NF; ++f) U[b + 4 * c][f] = u[c][f];
        }
        sync(true);
    };
    // the sums over the eight cells of coarse cell (I, J, K)
    auto put_coarse = [&](const Lev& w, int I, int J, int K, const double (&su)[NF],
                          const double (&sr)[NF], double sx) __attribute__((always_inline)) {
        const int Q = w.off + ((I + J + K) & 1) * w.half + lent(w, I >> 1, J, K);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            U[Q][f] = 0.125 * su[f];
            V[Q][f] = 0.125 * su[f];
            F[Q][f] = 0.125 * sr[f];
        }
        if constexpr (Op::XK) X[Q] = 0.125 * sx;
    };
    auto restrict_to = [&](int l, bool wave) __attribute__((always_inline)) {  // from l - 1 >= 1
        const Lev v = lev(l - 1), w = lev(l);
        const Op& o = ops.o[l - 1];
        for (int q = t; q < 2 * v.half; q += wave ? 64 : CP3_THREADS) {
            const int cc = q & 7, Q = q >> 3;
            const int I = Q & (w.m - 1), J = (Q >> (w.lh + 1)) & (w.n - 1), K = Q >> (w.lh + 1 + w.ln);
            const int j = 2 * J + ((cc >> 1) & 1), k = 2 * K + (cc >> 2);
            const int c = ((cc & 1) + j + k) & 1, e = v.off + c * v.half + lent(v, I, j, k);
            double su[NF], sr[NF], ns[NF], N[NF];
            nsl(v, I, j, k, c, ns);
            const double xk = Op::XK ? X[e] : 0.0;
            o.apply(U[e], ns, xk, N);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                su[f] = sum8(U[e][f]);
                sr[f] = sum8(F[e][f] - N[f]);
            }
            const double sx = Op::XK ? sum8(xk) : 0.0;
            if (cc == 0) put_coarse(w, I, J, K, su, sr, sx);
        }
        sync(wave);
    };
    // the correction of level l (>= 1) into its V
    auto correction = [&](int l, bool wave) __attribute__((always_inline)) {
        const Lev v = lev(l);
        for (int q = t; q < 2 * v.half; q += wave ? 64 : CP3_THREADS)
#pragma unroll
            for (int f = 0; f < NF; ++f) V[v.off + q][f] = U[v.off + q][f] - V[v.off + q][f];
        sync(wave);
    };
    // entry of level w's cell (I, J, K), any integers
    auto cell_of_ = [&](const Lev& w, int I, int J, int K) __attribute__((always_inline)) {
        I &= w.m - 1;
        return w.off + ((I + J + K) & 1) * w.half + lent(w, I >> 1, J, K);
    };
    auto prolong = [&](int l, bool wave) __attribute__((always_inline)) {  // from l + 1 into l >= 1
        const Lev v = lev(l), w = lev(l + 1);
        if (t < v.half) {
            const int I = t & ((v.m >> 1) - 1), j = (t >> v.lh) & (v.n - 1), k = t >> (v.lh + v.ln);
            const int J = j >> 1, K = k >> 1, dj = (j & 1) ? 1 : -1, dk = (k & 1) ? 1 : -1;
            const int s = (j + k) & 1;
            double e[3][NF];
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                const int q00 = cell_of_(w, I + x - 1, J, K), q10 = cell_of_(w, I + x - 1, J + dj, K);
                const int q01 = cell_of_(w, I + x - 1, J, K + dk), q11 = cell_of_(w, I + x - 1, J + dj, K + dk);
#pragma unroll
                for (int f = 0; f < NF; ++f)
                    e[x][f] = 0.75 * (0.75 * V[q00][f] + 0.25 * V[q10][f]) +
                              0.25 * (0.75 * V[q01][f] + 0.25 * V[q11][f]);
            }
            // cell 2I has colour s, cell 2I + 1 the other
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                U[v.off + s * v.half + t][f] += 0.75 * e[1][f] + 0.25 * e[0][f];
                U[v.off + (s ^ 1) * v.half + t][f] += 0.75 * e[1][f] + 0.25 * e[2][f];
            }
        }
        sync(wave);
    };

    sweeps0(L == 1 ? A.nswc : A.nsw1);
    if (L > 1) {
        if (act) {
            double su[NF], sr[NF], sx = (xr[0][0] + xr[0][1]) + (xr[1][0] + xr[1][1]);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                su[f] = (ur[0][0][f] + ur[0][1][f]) + (ur[1][0][f] + ur[1][1][f]);
                sr[f] = 0.0;
            }
            auto res = [&](auto zc, auto cc) __attribute__((always_inline)) {
                double N[NF];
                apply0(zc, cc, N);
#pragma unroll
                for (int f = 0; f < NF; ++f) sr[f] += fr[decltype(zc)::value][decltype(cc)::value][f] - N[f];
                __builtin_amdgcn_sched_barrier(0);
            };
            res(Z0{}, Z0{}); res(Z0{}, Z1{}); res(Z1{}, Z0{}); res(Z1{}, Z1{});
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                su[f] += __shfl_xor(su[f], 1 << sh0);
                sr[f] += __shfl_xor(sr[f], 1 << sh0);
            }
            if constexpr (Op::XK) sx += __shfl_xor(sx, 1 << sh0);
            if (P.jp == 0) put_coarse(lev(1), P.i2, P.J0, P.K0, su, sr, sx);
        }
        __syncthreads();
        // levels of at most 64 pairs: from `lw` on, the first wave alone
        int lw = 1;
        while (lw < L && (G.m[lw] * G.n[lw] * G.l[lw]) > 128) ++lw;
        for (int l = 1; l < lw; ++l) {
            if (l > 1) restrict_to(l, false);
            complete(l, false);
            sweeps(l, l < L - 1 ? A.nsw1 : A.nswc, false);
        }
        if (lw < L) {
            if (lw > 1) restrict_to(lw, false);
            if (t < 64) {
                const bool cube2 = G.m[L - 1] == 2 && G.n[L - 1] == 2 && G.l[L - 1] == 2;
                for (int l = lw; l < L; ++l) {
                    if (l > lw) restrict_to(l, true);
                    complete(l, true);
                    if (l == L - 1 && cube2) sweeps_cube2(l, A.nswc);
                    else sweeps(l, l < L - 1 ? A.nsw1 : A.nswc, true);
                }
                for (int l = L - 2; l >= lw; --l) {
                    correction(l + 1, true);
                    prolong(l, true);
                    sweeps(l, A.nsw2, true);
                }
            }
            __syncthreads();
        }
        for (int l = (lw < L ? lw : L - 1) - 1; l >= 1; --l) {
            correction(l + 1, false);
            prolong(l, false);
            sweeps(l, A.nsw2, false);
        }
        correction(1, false);
        // The pairs' u come back from LDS and their places are formed anew (from a
        // copy of t that is opaque to the compiler): held in registers across the
        // levels below they were spilled to memory, every half-sweep paying for it.
        int t2 = t;
        asm volatile("" : "+v"(t2));
        P = place(t2);
        if (act) {
            const Lev w = lev(1);
            const int dj = P.jp ? 1 : -1;
            int q[3][3][2];
#pragma unroll
            for (int z = 0; z < 3; ++z)
#pragma unroll
                for (int x = 0; x < 3; ++x) {
                    q[z][x][0] = cell_of_(w, P.i2 + x - 1, P.J0, P.K0 + z - 1);
                    q[z][x][1] = cell_of_(w, P.i2 + x - 1, P.J0 + dj, P.K0 + z - 1);
                }
#pragma unroll
            for (int f = 0; f < NF; ++f) {  // (one field at a time: registers)
                __builtin_amdgcn_sched_barrier(0);
                double e[3][3];  // [plane][x], interpolated along y
#pragma unroll
                for (int z = 0; z < 3; ++z)
#pragma unroll
                    for (int x = 0; x < 3; ++x)
                        e[z][x] = 0.75 * V[q[z][x][0]][f] + 0.25 * V[q[z][x][1]][f];
#pragma unroll
                for (int z = 0; z < 2; ++z) {
                    double v[3];
#pragma unroll
                    for (int x = 0; x < 3; ++x) v[x] = 0.75 * e[1][x] + 0.25 * e[z ? 2 : 0][x];
                    const double a = 0.75 * v[1] + 0.25 * v[0], b = 0.75 * v[1] + 0.25 * v[2];
                    const bool s = P.jp ^ z;  // cell 2 i2 is red where s = 0
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const double u = U0[P.e0[z]][c * NF + f] + (s == (c == 0) ? b : a);
                        ur[z][c][f] = u;
                        U0[P.e0[z]][c * NF + f] = u;
                    }
                }
            }
        }
        __syncthreads();
        sweeps0(A.nsw2);
    }
    if (act) {
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int f = 0; f < NF; ++f) A.u[f][c * half0 + P.e0[z]] = ur[z][c][f];
    }
}

// ---- per-step passes ----------------------------------------------------------
// Source S (App. B.1 / B.2) with the seven-point Laplacian, from the caller's
// (natural-order) fields into colour-split storage.
template <int SCHEME>
__global__ void __launch_bounds__(256) k3_source(Grid3 g, double ih2, double d, double alpha,
                                                 const double* __restrict__ phik,
                                                 const double* __restrict__ phikm1,
                                                 const double* __restrict__ psik, double* S1,
                                                 double* S2, double* S3) {
    const size_t q = item3();
    if (q >= cells3(g)) return;
    int i, j, k;
    split_cell(q, g, i, j, k);
    const size_t p = at3(i, j, k, g);
    const double x = phik[p];
    const double lk = (nsum6n(phik, i, j, k, g) - 6.0 * x) * ih2;
    S1[q] = x + d * psik[p];
    if constexpr (SCHEME == 1) {
        S2[q] = 2.0 * lk;
        S3[q] = 0.0;
    } else {
        // Lap of phi~ = (3 phi^k - phi^{k-1})/2 from the two Laplacians
        const double lm1 = (nsum6n(phikm1, i, j, k, g) - 6.0 * phikm1[p]) * ih2;
        S2[q] = 0.5 * alpha * x + 2.0 * (0.5 * (3.0 * lk - lm1));
        S3[q] = 0.5 * lk;
    }
}

// kappa = S3 + e Lap phi (completion of the guess, first half).
__global__ void __launch_bounds__(256) k3_complete_kappa(Grid3 g, double ih2, double e,
                                                         const double* __restrict__ phi,
                                                         const double* __restrict__ S3,
                                                         double* ka) {
    const size_t q = item3();
    if (q >= cells3(g)) return;
    int i, j, k;
    split_cell(q, g, i, j, k);
    ka[q] = S3[q] + e * ((nsum6(phi, i, j, k, g) - 6.0 * phi[q]) * ih2);
}

// mu = S2 + g(phi) + al phi + Lap kappa (second half).
template <int SCHEME>
__global__ void __launch_bounds__(256) k3_complete_mu(Grid3 g, double ih2, double al,
                                                      const double* __restrict__ phi,
                                                      const double* __restrict__ phik,
                                                      const double* __restrict__ S2,
                                                      const double* __restrict__ ka, double* mu) {
    const size_t q = item3();
    if (q >= cells3(g)) return;
    int i, j, k;
    split_cell(q, g, i, j, k);
    const double x = phi[q];
    mu[q] = S2[q] + nl_value<double, SCHEME, false>(x, 0.0, SCHEME == 2 ? phik[q] : 0.0) +
            al * x + (nsum6(ka, i, j, k, g) - 6.0 * ka[q]) * ih2;
}

// phi^(0) = phi^k (mode 0) or 2 phi^k - phi^{k-1} (mode 1), into split storage;
// the solver's copy of phi^k (xk, split) too.
__global__ void __launch_bounds__(256) k3_guess(Grid3 g, int mode, const double* __restrict__ phik,
                                                const double* __restrict__ phikm1, double* phi,
                                                double* xk) {
    const size_t q = item3();
    if (q >= cells3(g)) return;
    int i, j, k;
    split_cell(q, g, i, j, k);
    const size_t p = at3(i, j, k, g);
    phi[q] = mode == 1 ? 2.0 * phik[p] - phikm1[p] : phik[p];
    if (xk) xk[q] = phik[p];
}

// dst (natural order) = src (split storage).
__global__ void __launch_bounds__(256) k3_from_split(Grid3 g, const double* __restrict__ src,
                                                     double* dst) {
    const size_t q = item3();
    if (q >= cells3(g)) return;
    int i, j, k;
    split_cell(q, g, i, j, k);
    dst[at3(i, j, k, g)] = src[q];
}

// psi^{k+1} in place (eq. discrete_1_b / discrete_2_b) and phi^{k+1} out, both
// in natural order, from the solver's phi (split storage).
template <int SCHEME>
__global__ void __launch_bounds__(256) k3_psi_update(Grid3 g, double s,
                                                     const double* __restrict__ phi,
                                                     const double* __restrict__ phik, double* psi,
                                                     double* phi_out) {
    const size_t q = item3();
    if (q >= cells3(g)) return;
    int i, j, k;
    split_cell(q, g, i, j, k);
    const size_t p = at3(i, j, k, g);
    const double x = phi[q];
    if constexpr (SCHEME == 1) psi[p] = (x - phik[p]) / s;
    else psi[p] = (2.0 / s) * (x - phik[p]) - psi[p];
    phi_out[p] = x;
}

// b = psi - mean(psi) (mean from psisum[0]); per-block sums of b^2 and, with a
// warm start w, of (b + Lap_h w)^2 into part[2 blk], part[2 blk + 1].
template <int NT>
__global__ void __launch_bounds__(NT) k3_p_rhs(Grid3 g, double ih2, const double* __restrict__ psi,
                                               const double* __restrict__ psisum, double* b,
                                               const double* __restrict__ w, double* part) {
    __shared__ double red[NT / 64];
    const size_t total = (size_t)g.m * g.n * g.l;
    const double mean = psisum[0] / (double)total;
    double sb = 0.0, sr = 0.0;
    for (size_t q = (size_t)blockIdx.x * NT + threadIdx.x; q < total; q += (size_t)gridDim.x * NT) {
        int i, j, k;
        split_cell(q, g, i, j, k);
        const double v = psi[at3(i, j, k, g)] - mean;   // psi: natural; b, w: split
        b[q] = v;
        sb += v * v;
        if (w) {
            const double r = v - (6.0 * w[q] - nsum6(w, i, j, k, g)) * ih2;
            sr += r * r;
        }
    }
    const double tb = block_sum<NT>(sb, red);
    __syncthreads();
    const double tr = block_sum<NT>(sr, red);
    if (threadIdx.x == 0) {
        part[(size_t)blockIdx.x * 2] = tb;
        part[(size_t)blockIdx.x * 2 + 1] = tr;
    }
}

// Energy sums, per block into part[blk * 8 + k]: 0: sum phi^4, 1: sum phi^2,
// 2: sum over east/north/top faces of (phi difference)^2, 3: sum (Lap_h phi)^2,
// 4: sum phi, 5: face sum of (difference of phi - phi_prev)^2, 6: sum b w, 7: 0.
template <int NT>
__global__ void __launch_bounds__(NT) k3_energy_terms(Grid3 g, double ih2,
                                                      const double* __restrict__ phi,
                                                      const double* __restrict__ phiprev,
                                                      const double* __restrict__ b,
                                                      const double* __restrict__ w, double* part) {
    __shared__ double red[NT / 64];
    double a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const size_t total = (size_t)g.m * g.n * g.l;
    for (size_t q = (size_t)blockIdx.x * NT + threadIdx.x; q < total; q += (size_t)gridDim.x * NT) {
        int i, j, k;
        split_cell(q, g, i, j, k);
        const size_t qe = at3((i + 1) & (g.m - 1), j, k, g);
        const size_t qn = at3(i, (j + 1) & (g.n - 1), k, g);
        const size_t qt = at3(i, j, (k + 1) & (g.l - 1), g);
        const size_t p = at3(i, j, k, g);   // phi, phi_prev: natural; b, w: split
        const double x = phi[p];
        const double L = (nsum6n(phi, i, j, k, g) - 6.0 * x) * ih2;
        a[0] += (x * x) * (x * x);
        a[1] += x * x;
        a[2] += (phi[qe] - x) * (phi[qe] - x) + (phi[qn] - x) * (phi[qn] - x) +
                (phi[qt] - x) * (phi[qt] - x);
        a[3] += L * L;
        a[4] += x;
        if (phiprev) {
            const double d = x - phiprev[p];
            const double de = phi[qe] - phiprev[qe] - d;
            const double dn = phi[qn] - phiprev[qn] - d;
            const double dt = phi[qt] - phiprev[qt] - d;
            a[5] += de * de + dn * dn + dt * dt;
        }
        a[6] += b[q] * w[q];
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const double t = block_sum<NT>(a[s], red);
        if (threadIdx.x == 0) part[(size_t)blockIdx.x * 8 + s] = t;
        __syncthreads();
    }
}

}  // namespace mpfc
