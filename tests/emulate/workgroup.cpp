// Kernels of a step, one workgroup on the CPU (hip/hip_runtime.h here):
//   tile <first wave>        a finest down tile whose stop flag rises while its waves start
//   coarse <m> <n> <bc>      the persistent levels with the work-items in two orders
//   newton <h> <c> <al> <size> <pivot> <seed>   the coarsest grid's solve against one
//                            that takes every step
//   readback <norms> <max>   what the step's readback writes after that many norms
// Each prints one line, checked by tests/test_workgroup_cpu.py.
#include "kernels.hpp"
#include "tiles.hpp"
#include "step.hpp"

using namespace mpfc;

static std::vector<unsigned> order_from(unsigned nt, unsigned wave, bool back = false) {
    std::vector<unsigned> o(nt);
    for (unsigned k = 0; k < nt; ++k) o[k] = back ? nt - 1 - k : (k + 64 * wave) % nt;
    return o;
}
static std::vector<double> field(size_t n, unsigned seed, double amp) {
    std::vector<double> f(n);
    uint64_t s = seed * 0x9E3779B97F4A7C15ull + 1;
    for (double& x : f) {
        s = s * 6364136223846793005ull + 1442695040888963407ull;
        x = amp * ((double)(s >> 11) / 9007199254740992.0 - 0.5);
    }
    return f;
}
static LevelOp<double> level(double h, double c, double al) {
    LevelOp<double> op;
    op.ih2 = 1.0 / (h * h);
    op.c = c;
    op.al = al;
    op.e = 0.5;
    op.derive();
    return op;
}
using Op = MpfcOp<double, 2, true, false>;

static int tile(unsigned wave) {
    constexpr int M = 32, T = 16;
    const size_t N = M * M;
    std::vector<std::vector<double>> u, f;
    for (int k = 0; k < 3; ++k) {
        u.push_back(field(N, 1 + k, 1.0));
        f.push_back(field(N, 4 + k, 1.0));
    }
    const std::vector<std::vector<double>> u0 = u;
    std::vector<double> xk = field(N, 7, 1.0);
    CycleState st{};
    auto launch = [&](bool rise, std::vector<std::vector<double>>& w) {
        w.assign(3 + 3 * 3 + 1, std::vector<double>(N, 1e300));
        TileArgs<double> A{};
        A.g = Grid{M, M, 5, 5, 0};
        for (int k = 0; k < 3; ++k) {
            A.uin[k] = u[k].data();
            A.f[k] = f[k].data();
            A.uout[k] = w[k].data();
            A.uH[k] = w[3 + k].data();
            A.vH[k] = w[6 + k].data();
            A.rH[k] = w[9 + k].data();
        }
        A.xk = xk.data();
        A.xkH = w[12].data();
        A.nsweep = 4;
        A.H = 6;
        A.tx = A.ty = T;
        A.ntx = M / T;
        st = CycleState{};
        PendingNorm P{};
        P.nparts = 1;  // workgroup 0 is the stopping test's
        emu::run(kTileThreads, dim3(2), dim3(1 + (M / T) * (M / T)),
                 order_from(kTileThreads, wave), [&] {
                     k_tile<Op, T, T, 6, false, false, false, true, true>(Op{level(0.8, 0.02, 0.4)}, A,
                                                                    &st, P);
                 },
                 [&](unsigned k) { if (rise && k == 64) st.done = 1; });
    };
    std::vector<std::vector<double>> full, got;
    launch(false, full);
    launch(true, got);
    bool none = true, untouched = u == u0;
    for (auto& w : got)
        for (double x : w) none = none && x == 1e300;
    bool wrote = false;
    for (double x : full[0]) wrote = wrote || x != 1e300;
    printf("%s %s\n", !wrote ? "broken" : got == full ? "all" : none ? "none" : "part",
           untouched ? "kept" : "overwritten");
    return 0;
}

template <int NC, bool NEU>
static int coarse(int m, int n, int bc) {
    const size_t N = (size_t)m * n;
    using W = CoarseWork<Op, NC, NEU>;
    static typename W::Lds S;
    std::vector<double> xk = field(N, 7, 1.0);
    std::vector<std::vector<double>> first;
    double diff = 0.0, size = 0.0;
    for (int back = 0; back < 2; ++back) {
        std::vector<std::vector<double>> u, f;
        for (int k = 0; k < 3; ++k) {
            u.push_back(field(N, 1 + k, 1.0));
            f.push_back(field(N, 4 + k, 1.0));
        }
        CoarseArgs<double> A{};
        A.geo = CoarseGeom{bc, m, n, __builtin_ctz(m)};
        for (int k = 0; k < 3; ++k) { A.u[k] = u[k].data(); A.rr[k] = f[k].data(); }
        A.xk = xk.data();
        A.nsw1 = A.nsw2 = 4;
        A.complete_top = 1;
        A.newton_maxit = 30;
        A.newton_tol = 1e-15;
        emu::run(CP_THREADS, dim3(0), dim3(1), order_from(CP_THREADS, 0, back),
                 [&] { W::run(Op{level(0.8, 0.02, 0.4)}, A, S, nullptr); }, [](unsigned) {});
        if (!back) first = u;
        for (int k = 0; k < 3; ++k)
            for (size_t q = 0; q < N; ++q) {
                diff = fmax(diff, fabs(u[k][q] - first[k][q]));
                size = fmax(size, fabs(u[k][q]));
            }
    }
    printf("%.17g %.17g\n", diff, size);
    return 0;
}

// `pivot`: the elimination with pivoting, else the sign patterns.
static int newton(double h, double c, double al, double amp, int pivot, unsigned seed) {
    constexpr int NC = 4;
    double f[3][NC], xk[NC], none[NC] = {};
    std::vector<double> a[3];
    for (int k = 0; k < 3; ++k) {
        a[k] = field(NC, seed + k, amp);
        const std::vector<double> b = field(NC, seed + 4 + k, amp);
        for (int q = 0; q < NC; ++q) f[k][q] = b[q];
    }
    const std::vector<double> x = field(NC, seed + 7, amp);
    for (int q = 0; q < NC; ++q) xk[q] = x[q];
    const Op op{level(h, c, al)};
    auto solve = [&](int maxit, double tol) {
        double u[3][NC];
        for (int k = 0; k < 3; ++k)
            for (int q = 0; q < NC; ++q) u[k][q] = a[k][q];
        if (pivot) coarse_solve_mpfc<Op, NC>(op, u, f, xk, none, none, 2, 1, 2, 0, maxit, tol);
        else coarse_solve_walsh<Op, NC>(op, u, f, xk, none, none, 2, 2, 0, maxit, tol);
        return std::vector<double>(u[0], u[0] + NC);
    };
    auto apart = [](const std::vector<double>& p, const std::vector<double>& q) {
        double d = 0.0;
        for (int k = 0; k < NC; ++k) d = fmax(d, fabs(p[k] - q[k]));
        return d;
    };
    const std::vector<double> got = solve(30, 1e-15), late = solve(100, 0.0);
    double noise = 0.0, size = 1.0;   // what the solve's own rounding moves, step after step
    for (int k = 80; k < 100; ++k) noise = fmax(noise, apart(solve(k, 0.0), late));
    for (double v : late) size = fmax(size, fabs(v));
    printf("%.17g %.17g %.17g\n", apart(got, late), noise, size);
    return 0;
}

static int readback(int norms, int most) {
    const int fixed = 32, count = fixed + most + 1;
    std::vector<double> rb = field(count, 3, 1.0), host(count, 1e300);
    CycleState st{};
    st.count = norms;
    memcpy(rb.data(), &st, sizeof st);
    emu::run(256, dim3(0), dim3(1), order_from(256, 0),
             [&] { k_readback(rb.data(), count, host.data()); }, [](unsigned) {});
    int written = 0, wrong = 0;
    for (int k = 0; k < count; ++k) {
        if (host[k] == 1e300) continue;
        ++written;
        wrong += memcmp(&host[k], &rb[k], sizeof(double)) != 0;
    }
    for (int k = 0; k < fixed + norms; ++k) wrong += host[k] == 1e300;
    printf("%d %d\n", written, wrong);
    return 0;
}

int main(int argc, char** argv) {
    auto num = [&](int k) { return k < argc ? atof(argv[k]) : 0.0; };
    const char* what = argc > 1 ? argv[1] : "";
    if (!strcmp(what, "tile")) return tile((unsigned)num(2));
    if (!strcmp(what, "coarse")) {
        const int m = (int)num(2), n = (int)num(3), bc = (int)num(4);
        if (m == n) return bc ? coarse<4, true>(m, n, bc) : coarse<4, false>(m, n, bc);
        return bc ? coarse<8, true>(m, n, bc) : coarse<8, false>(m, n, bc);
    }
    if (!strcmp(what, "newton"))
        return newton(num(2), num(3), num(4), num(5), (int)num(6), (unsigned)num(7));
    if (!strcmp(what, "readback")) return readback((int)num(2), (int)num(3));
    return 1;
}
