// Definitions and explicit instantiations of the launchers declared in
// launch.hpp.  The build compiles this file once per operator group
// (-DMPFC_GROUP=0..7) in parallel; without MPFC_GROUP every group is built.
#include <hip/hip_runtime.h>

#include "launch.hpp"

namespace mpfc {
namespace {

bool general_index(const Grid& g) { return g.lm < 0 || g.ln < 0; }

#ifndef MPFC_TILE_EXACT
#define MPFC_TILE_EXACT 1
#endif

// The halo of up launches of two passes without a residual (every coarse one of
// V(2,2), every FP32 one), and of down and finest up launches of one pass.  As a
// compile-time halo it leaves no extent to run time, and a tile holds 1.1 to 1.25
// times fewer cells in LDS than with the shape's allowance of 6.  Ten steps of
// V(1,1) on 256 x 128 (Neumann): 8.36 -> 7.97 ms; five of 2048^2 in mixed
// precision: 10.3 -> 10.04 ms.  (Shapes 5 and 6 would repeat 2 and 3.)
constexpr int kHaloSmall = 4;

// One tile launch, with one more workgroup for a pending norm.  Two kernels, with the
// vote and without, where a launch without a norm feels it (k_tile): in FP32, and with
// the FP64 tiles of the small levels (6.84 -> 6.98 us on 64^2 with 16 x 16).  Larger
// FP64 tiles have one: the finest level shares its code with the levels below (two
// cost the 512^2 and 1024^2 steps 1.5 % in instruction cache misses).
template <class Op, int TX, int TY, int HMAX, bool UP, bool NEU, bool GEN, bool EXACT>
void tile_launch(const Op& op, TileArgs<typename Op::real>& A, const CycleState* stop,
                 hipStream_t s, const PendingNorm& P) {
    A.ntx = A.g.m / A.tx;
    const dim3 grid(A.ntx * (A.g.n / A.ty) + (P.nparts ? 1 : 0)), blk(kTileThreads);
    constexpr bool norms = !UP && Op::NF == 3;
    constexpr bool f64 = std::is_same<typename Op::real, double>::value;
    constexpr bool two = norms && (!f64 || (!GEN && TX * TY <= 512 && HMAX <= 6));
    if constexpr (two) {
        if (P.nparts) {
            hipLaunchKernelGGL((k_tile<Op, TX, TY, HMAX, UP, NEU, GEN, EXACT, true>), grid, blk, 0,
                               s, op, A, stop, P);
            return;
        }
    }
    hipLaunchKernelGGL((k_tile<Op, TX, TY, HMAX, UP, NEU, GEN, EXACT, norms && !two>), grid, blk, 0,
                       s, op, A, stop, P);
}

template <class Op, bool UP, bool NEU, int K>
void tile_k(const Op& op, TileArgs<typename Op::real> A, const CycleState* stop, hipStream_t s,
            bool gen, const PendingNorm& P) {
    constexpr TileShape S = kShapes[K];
    if constexpr (std::is_same<typename Op::real, double>::value && gen_shape(K)) {
        if (gen) {
            tile_launch<Op, S.tx, S.ty, S.hmax, UP, NEU, true, false>(op, A, stop, s, P);
            return;
        }
    }
    // the shape's own tile and halo (the larger levels): compile-time extents
    if (MPFC_TILE_EXACT && A.tx == S.tx && A.ty == S.ty && A.H == S.hmax) {
        tile_launch<Op, S.tx, S.ty, S.hmax, UP, NEU, false, true>(op, A, stop, s, P);
        return;
    }
    if constexpr (K <= 4) {
        if (MPFC_TILE_EXACT && A.tx == S.tx && A.ty == S.ty && A.H == kHaloSmall) {
            tile_launch<Op, S.tx, S.ty, kHaloSmall, UP, NEU, false, true>(op, A, stop, s, P);
            return;
        }
    }
    tile_launch<Op, S.tx, S.ty, S.hmax, UP, NEU, false, false>(op, A, stop, s, P);
}

template <class Op, bool UP, bool NEU>
void tile_bc(const Op& op, const TileArgs<typename Op::real>& A, int shape,
             const CycleState* stop, hipStream_t s, const PendingNorm& P) {
    const bool gen = general_index(A.g);
    if (gen && !gen_shape(shape)) shape = 0;  // general-index kernels
    switch (shape) {
        case 0: tile_k<Op, UP, NEU, 0>(op, A, stop, s, gen, P); break;
        case 1: tile_k<Op, UP, NEU, 1>(op, A, stop, s, gen, P); break;
        case 2: tile_k<Op, UP, NEU, 2>(op, A, stop, s, gen, P); break;
        case 3: tile_k<Op, UP, NEU, 3>(op, A, stop, s, gen, P); break;
        case 4: tile_k<Op, UP, NEU, 4>(op, A, stop, s, gen, P); break;
        case 5: tile_k<Op, UP, NEU, 5>(op, A, stop, s, gen, P); break;
        default: tile_k<Op, UP, NEU, 6>(op, A, stop, s, gen, P); break;
    }
}

template <class Op, bool UP, bool NEU, int K>
void tile_batched_k(int exact_h, const BatchTile<Op>* args, const BatchItem* items, int n,
                    bool first, hipStream_t s) {
    constexpr TileShape S = kShapes[K];
    const dim3 grid(n), blk(kTileThreads);
    const int f = first;
    if constexpr (K <= 3) {
        if (exact_h == S.hmax) {
            hipLaunchKernelGGL((k_tile_batched<Op, S.tx, S.ty, S.hmax, UP, NEU, true>), grid, blk,
                               0, s, args, items, n, f);
            return;
        }
        if (exact_h == kHaloSmall) {
            hipLaunchKernelGGL((k_tile_batched<Op, S.tx, S.ty, kHaloSmall, UP, NEU, true>), grid,
                               blk, 0, s, args, items, n, f);
            return;
        }
    }
    hipLaunchKernelGGL((k_tile_batched<Op, S.tx, S.ty, S.hmax, UP, NEU, false>), grid, blk, 0, s,
                       args, items, n, f);
}

template <class Op, bool UP, bool NEU>
void tile_batched_bc(int shape, int h, const BatchTile<Op>* args, const BatchItem* items, int n,
                     bool first, hipStream_t s) {
    switch (shape) {
        case 0: tile_batched_k<Op, UP, NEU, 0>(h, args, items, n, first, s); break;
        case 1: tile_batched_k<Op, UP, NEU, 1>(h, args, items, n, first, s); break;
        case 2: tile_batched_k<Op, UP, NEU, 2>(h, args, items, n, first, s); break;
        case 3: tile_batched_k<Op, UP, NEU, 3>(h, args, items, n, first, s); break;
        case 4: tile_batched_k<Op, UP, NEU, 4>(h, args, items, n, first, s); break;
        case 5: tile_batched_k<Op, UP, NEU, 5>(h, args, items, n, first, s); break;
        default: tile_batched_k<Op, UP, NEU, 6>(h, args, items, n, first, s); break;
    }
}

}  // namespace

// Periodic grids run the instantiation without the Neumann ghost handling.
template <class Op, bool UP>
void launch_tile(const Op& op, const TileArgs<typename Op::real>& A, int shape,
                 const CycleState* stop, hipStream_t s, const PendingNorm& pend) {
    if (A.g.bc) tile_bc<Op, UP, true>(op, A, shape, stop, s, pend);
    else tile_bc<Op, UP, false>(op, A, shape, stop, s, pend);
}

template <class Op>
void launch_coarse(const Op& op, const CoarseArgs<typename Op::real>& A, bool four,
                   const CycleState* stop, hipStream_t s) {
    const dim3 g1(1), blk(CP_THREADS);
    if (A.geo.bc) {
        if (four) hipLaunchKernelGGL((k_coarse_persistent<Op, 4, true>), g1, blk, 0, s, op, A, stop);
        else hipLaunchKernelGGL((k_coarse_persistent<Op, 8, true>), g1, blk, 0, s, op, A, stop);
    } else {
        if (four) hipLaunchKernelGGL((k_coarse_persistent<Op, 4, false>), g1, blk, 0, s, op, A, stop);
        else hipLaunchKernelGGL((k_coarse_persistent<Op, 8, false>), g1, blk, 0, s, op, A, stop);
    }
}

template <class Op>
void launch_coarsest_gen(const Op& op, const CoarseArgs<typename Op::real>& A,
                         const CycleState* stop, hipStream_t s) {
    const dim3 g1(1), blk(CG_THREADS);
    if (A.geo.bc) hipLaunchKernelGGL((k_coarsest_sweeps<Op, true>), g1, blk, 0, s, op, A, stop);
    else hipLaunchKernelGGL((k_coarsest_sweeps<Op, false>), g1, blk, 0, s, op, A, stop);
}

template <class Op, bool UP>
void launch_tile_batched(bool neu, int shape, int exact_h, const BatchTile<Op>* args,
                         const BatchItem* items, int n, bool first, hipStream_t s) {
    if (neu) tile_batched_bc<Op, UP, true>(shape, exact_h, args, items, n, first, s);
    else tile_batched_bc<Op, UP, false>(shape, exact_h, args, items, n, first, s);
}

template <class Op, int NC>
void launch_coarse_batched(bool neu, int nsim, const BatchCoarse<Op>* args, hipStream_t s) {
    if (neu) hipLaunchKernelGGL((k_coarse_persistent_batched<Op, NC, true>), dim3(nsim),
                                dim3(CP_THREADS), 0, s, args);
    else hipLaunchKernelGGL((k_coarse_persistent_batched<Op, NC, false>), dim3(nsim),
                            dim3(CP_THREADS), 0, s, args);
}

#define MPFC_INST_TILE(OP)                                                                   \
    template void launch_tile<OP, false>(const OP&, const TileArgs<OP::real>&, int,          \
                                         const CycleState*, hipStream_t,                     \
                                         const PendingNorm&);                                \
    template void launch_tile<OP, true>(const OP&, const TileArgs<OP::real>&, int,           \
                                        const CycleState*, hipStream_t, const PendingNorm&); \
    template void launch_coarse<OP>(const OP&, const CoarseArgs<OP::real>&, bool,            \
                                    const CycleState*, hipStream_t);
#define MPFC_INST_GEN(OP)                                                                    \
    template void launch_coarsest_gen<OP>(const OP&, const CoarseArgs<OP::real>&,            \
                                          const CycleState*, hipStream_t);
#define MPFC_INST_BATCH(OP)                                                                  \
    template void launch_tile_batched<OP, false>(bool, int, int, const BatchTile<OP>*,       \
                                                 const BatchItem*, int, bool, hipStream_t);  \
    template void launch_tile_batched<OP, true>(bool, int, int, const BatchTile<OP>*,        \
                                                const BatchItem*, int, bool, hipStream_t);   \
    template void launch_coarse_batched<OP, 4>(bool, int, const BatchCoarse<OP>*, hipStream_t); \
    template void launch_coarse_batched<OP, 8>(bool, int, const BatchCoarse<OP>*, hipStream_t);

// Operator groups (one compilation each): the FP64 operators by scheme and
// linearisation (with the general-index coarsest level and the batched
// forms), the pinned operator, the FP32 correction operators of mixed
// precision (with the batched forms), and the Poisson operator of the -1 norm.
using S2N = MpfcOp<double, 2, true, false>;
using S2P = MpfcOp<double, 2, false, false>;
using S1N = MpfcOp<double, 1, true, false>;
using S1P = MpfcOp<double, 1, false, false>;
using S2Pin = MpfcOp<double, 2, true, false, true>;
using F2N = MpfcOp<float, 2, true, true>;
using F2P = MpfcOp<float, 2, false, true>;
using F1N = MpfcOp<float, 1, true, true>;
using F1P = MpfcOp<float, 1, false, true>;
using Poi = PoissonOp<double>;

#if !defined(MPFC_GROUP) || MPFC_GROUP == 0
MPFC_INST_TILE(S2N)
MPFC_INST_GEN(S2N)
MPFC_INST_BATCH(S2N)
#endif
#if !defined(MPFC_GROUP) || MPFC_GROUP == 1
MPFC_INST_TILE(S2P)
MPFC_INST_GEN(S2P)
MPFC_INST_BATCH(S2P)
#endif
#if !defined(MPFC_GROUP) || MPFC_GROUP == 2
MPFC_INST_TILE(S1N)
MPFC_INST_GEN(S1N)
MPFC_INST_BATCH(S1N)
#endif
#if !defined(MPFC_GROUP) || MPFC_GROUP == 3
MPFC_INST_TILE(S1P)
MPFC_INST_GEN(S1P)
MPFC_INST_BATCH(S1P)
#endif
#if !defined(MPFC_GROUP) || MPFC_GROUP == 4
MPFC_INST_TILE(S2Pin)
MPFC_INST_GEN(S2Pin)
#endif
#if !defined(MPFC_GROUP) || MPFC_GROUP == 5
MPFC_INST_TILE(F2N)
MPFC_INST_TILE(F2P)
MPFC_INST_BATCH(F2N)
MPFC_INST_BATCH(F2P)
#endif
#if !defined(MPFC_GROUP) || MPFC_GROUP == 6
MPFC_INST_TILE(F1N)
MPFC_INST_TILE(F1P)
MPFC_INST_BATCH(F1N)
MPFC_INST_BATCH(F1P)
#endif
#if !defined(MPFC_GROUP) || MPFC_GROUP == 7
MPFC_INST_TILE(Poi)
void launch_coarsest_poisson(const PoissonOp<double>& op, const CoarseArgs<double>& A,
                             const CycleState* stop, hipStream_t s) {
    hipLaunchKernelGGL((k_coarsest_poisson<double>), dim3(1), dim3(CG_THREADS), 0, s, op, A, stop);
}
#endif

}  // namespace mpfc
