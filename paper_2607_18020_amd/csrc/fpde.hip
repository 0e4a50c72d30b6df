// fpde.hip -- host side of libfpde: argument validation, launch geometry and
// the exported C entry points declared in include/fpde.h.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <tuple>
#include <type_traits>

#include "fpde.h"
#include "fpde_engine.hpp"

namespace fpde {
namespace {

// Launch geometry.  A workgroup owns a TX x TY column tile (TY = 1 for 2-D
// grids, where a "plane" is one row) and marches a chunk of planes of axis 0.
// 3-D grids: the chunk length is chosen per launch (plan_chunks).  Where the
// forward and the backward get the same one (256^3), the backward, which marches
// each chunk top down, starts on the planes the forward read last (still in the
// memory-side infinity cache).
// backward tile widths: a tile's x-halo columns sit in cache lines of the
// neighbouring tiles, which L2 serves only while the two tiles march in step;
// wider tiles have fewer such lines per node
#ifndef FPDE_NS3_BWD_TX
#define FPDE_NS3_BWD_TX 128
#endif
#ifndef FPDE_HEAT_BWD_TX
#define FPDE_HEAT_BWD_TX 64
#endif
// forward tile widths (a tile's side-edge x-neighbours cost a cache line each)
#ifndef FPDE_NS3_FWD_TX
#define FPDE_NS3_FWD_TX 128
#endif
#ifndef FPDE_HEAT_FWD_TX
#define FPDE_HEAT_FWD_TX 256
#endif
#ifndef FPDE_NS3_FWD_TY
#define FPDE_NS3_FWD_TY 4
#endif
#ifndef FPDE_NS3_BWD_TY
#define FPDE_NS3_BWD_TY 8
#endif
#ifndef FPDE_HEAT_FWD_TY
#define FPDE_HEAT_FWD_TY 4
#endif
#ifndef FPDE_HEAT_BWD_TY
#define FPDE_HEAT_BWD_TY 8
#endif
// rows of the narrow 64-node tiles
#ifndef FPDE_NS3_FWD2_TY
#define FPDE_NS3_FWD2_TY 8
#endif
#ifndef FPDE_NS3_BWD2_TY
#define FPDE_NS3_BWD2_TY 8
#endif
#ifndef FPDE_HEAT_FWD2_TY
#define FPDE_HEAT_FWD2_TY 8
#endif
// 2-D rows of the LDS marches (explicit-sensitivity backward; the checking
// build's backward) and of the register-queue forward (the wide ones)
#ifndef FPDE_TX2
#define FPDE_TX2 256
#endif
#ifndef FPDE_TX2_FWD
#define FPDE_TX2_FWD 1024
#endif
#ifndef FPDE_TX2_FWD2
#define FPDE_TX2_FWD2 256
#endif
// register-queue forward: planes held per lane (the centre plane, its two
// neighbours, and Q - 3 planes in flight)
#ifndef FPDE_FWD2_Q
#define FPDE_FWD2_Q 6
#endif
// 3-D operators with one stencil field (heat, Poisson) can use the
// register-queue forward too (five loads per node and plane fit the registers);
// the LDS march is faster there (heat 256^3: 29 against 32 us), so the product
// keeps it and the checking build takes the queue, as a second algorithm
#ifndef FPDE_HEAT_FWD_QUEUE
#define FPDE_HEAT_FWD_QUEUE 0
#endif
// one stencil field and almost no arithmetic per plane: the LDS march forward
// keeps several planes in flight (an 8-slot ring), where one plane per step
// would wait for each plane's latency in turn
#ifndef FPDE_HEAT_FWD_RING
#define FPDE_HEAT_FWD_RING 8
#endif
// 2-D backward, and one-pass value and gradient: the register-queue march
// (bwdq_kernel: no LDS, no barrier; NW waves of 62 output columns, Q rows in
// registers); the checking build takes the LDS march (bwd_kernel with one-row
// tiles) as a second algorithm whose gradients must match bit for bit
#ifndef FPDE_BWD2_QUEUE
#define FPDE_BWD2_QUEUE 1
#endif
#ifndef FPDE_BWD2_NW
#define FPDE_BWD2_NW 4
#endif
#ifndef FPDE_BWD2_Q
#define FPDE_BWD2_Q 7
#endif
// explicit-sensitivity backward tiles (3-D)
#ifndef FPDE_VJP_TX3
#define FPDE_VJP_TX3 64
#endif
#ifndef FPDE_VJP_TY3
#define FPDE_VJP_TY3 4
#endif
#ifndef FPDE_VJP_HEAT_TX
#define FPDE_VJP_HEAT_TX 128
#endif
#ifndef FPDE_VJP_HEAT_TY
#define FPDE_VJP_HEAT_TY 8
#endif
#ifndef FPDE_VJP_HEAT2_TY
#define FPDE_VJP_HEAT2_TY 8
#endif
// The backward marches each chunk top-down (see above).
#ifndef FPDE_BWD_REVERSE
#define FPDE_BWD_REVERSE 1
#endif
constexpr bool kBwdReverse = FPDE_BWD_REVERSE != 0;

// A TX x TY tile of columns.  RES workgroups of its kernel run on a CU at once, by the
// kernel's LDS, threads and registers (a test compares it with the compiler's own resource
// notes), RESL of the kernel that also sums the loss and RESP of that one on a periodic
// grid, where they need more registers; a step of a full round of them takes STEP
// percent of the wide tile's.
template <int TX_, int TY_, int RES_, int STEP_ = 100, int RESL_ = RES_, int RESP_ = RESL_>
struct Tile {
    static constexpr int TX = TX_, TY = TY_, RES = RES_, STEP = STEP_;
    static constexpr int res(bool loss, bool per) { return !loss ? RES : per ? RESP_ : RESL_; }
};
// One kind of launch: its wide tile W (fewer cache lines shared across tile edges: the
// faster on wide rows) and its narrow one N, which leaves fewer lanes idle where the last
// axis is not a multiple of the wide tile, and whose smaller workgroups have the shorter
// step on a grid that does not fill the chip (with_tile picks); and how the march's time
// goes (share, floor, prologue, atom: plan_chunks).  STEP is the ratio of the two tiles'
// full rounds; the others are fitted per kind.  Both from the times of either tile at some 25
// chunk counts each, on 150 to 330 grids per operator of 2^16 to 2^25 nodes: the launches
// that the rule takes are within 0 to 3% of the fastest one measured in the geometric mean
// and 32% at worst.  One share and
// prologue for every march, and the residency of one kernel for all that share a tile, had
// the forwards 3 to 10% off.
template <class W_, class N_ = W_>
struct Plan {
    using W = W_;
    using N = N_;
    double share, floor, prologue, atom = 0.012;
};
// 2-D grids: row segments (TY = 1).  The wide forward wins where the narrow one's loss
// atomics would be more (NS-2D 2048^2 without a workspace: 15.2 us in 256 workgroups of
// 1024, 17.7 in 512 of 256); the narrow one on short rows and small grids (374 x 447:
// 7.9 and 7.0 us; Burgers 128 x 256: 5.9 and 4.7, 5.5 of each the launches), and with a
// workspace (Helmholtz 1024^2: 8.0 and 7.4).
// VGA: where the value and gradient sums its loss by atomics.  One field's workgroups
// finish together, and half as many of eight waves wait for half the atomics (Helmholtz
// 2048^2 19.4 -> 17.7 us, 901 x 480 9.1 -> 8.4, Burgers 1397 x 1661 13.8 -> 11.7); three
// fields are no faster so (2048^2 26.7 -> 28.0).
template <int RL, int RLA>  // value and gradient: workgroups of four and of eight waves per CU
struct Geo2One {
    static constexpr bool D3 = false;
    static constexpr Plan<Tile<FPDE_TX2_FWD, 1, 2>, Tile<FPDE_TX2_FWD2, 1, 8, 140>> FWD{0.85, 0, 3.5},
        FWDR{0.85, 0, 3.5};
    [[maybe_unused]] static constexpr Plan<Tile<62 * FPDE_BWD2_NW, 1, 8>> BWD{1.0, 0, 5.0};
    [[maybe_unused]] static constexpr Plan<Tile<62 * FPDE_BWD2_NW, 1, 8, 100, RL>> VG{0.9, 0, 4.5};
    [[maybe_unused]] static constexpr Plan<Tile<62 * 8, 1, 4, 100, RLA>> VGA{0.9, 0, 4.5};
    static constexpr Plan<Tile<FPDE_TX2, 1, 8>> VJP{0.2, 0, 5.0};
};
using Geo2Burgers = Geo2One<8, 4>;   // 45 VGPRs with the loss
using Geo2Laplace = Geo2One<6, 3>;   // Helmholtz, Poisson: 76 to 78
struct Geo2NS {
    static constexpr bool D3 = false;
    static constexpr Plan<Tile<FPDE_TX2_FWD, 1, 1>, Tile<FPDE_TX2_FWD2, 1, 4>> FWD{0.9, 0, 4.0};
    static constexpr Plan<Tile<FPDE_TX2_FWD, 1, 1>, Tile<FPDE_TX2_FWD2, 1, 4, 94>> FWDR{0, 1.6, 1.5};
    [[maybe_unused]] static constexpr Plan<Tile<62 * FPDE_BWD2_NW, 1, 3>> BWD{0, 1.2, 1.5};
    [[maybe_unused]] static constexpr Plan<Tile<62 * FPDE_BWD2_NW, 1, 3, 100, 3, 2>>
        VG{0, 1.6, 5.0}, VGA{0, 1.6, 5.0};  // (152 to 174 VGPRs)
    static constexpr Plan<Tile<FPDE_TX2, 1, 5>> VJP{0, 2.2, 2.5};
};
// 3-D grids.  Several fields with nonlinear coupling (NS): the LDS decides, but for the
// wide backward's 1024 threads.  Where the narrow tiles win: NS-3D backward
// 150 x 131 x 257 61 -> 54 us (5 tiles of 64 across a row instead of 3 of 128), 64^3
// 10.8 -> 8.1, 28 x 39 x 47 9.0 -> 7.0; forward 64^3 10.4 -> 8.6 (5.5 of it the loss fill
// and the launches).
struct GeoNS3 {
    static constexpr bool D3 = true, FWD_QUEUE = false;  // (forward: the LDS march)
    static constexpr int FWD_RING = 4;                   // slots of the forward's plane ring
    static constexpr double STORE_EDGE = 1.4;            // (launch_fwd3)
    using TF = Tile<FPDE_NS3_FWD_TX, FPDE_NS3_FWD_TY, 2>;
    using TB = Tile<FPDE_NS3_BWD_TX, FPDE_NS3_BWD_TY, 1>;
    static constexpr Plan<TF, Tile<64, FPDE_NS3_FWD2_TY, 3, 152>> FWD{0, 1.45, 2.5};
    static constexpr Plan<TF, Tile<64, FPDE_NS3_FWD2_TY, 3, 155>> FWDR{0, 1.6, 2.5};
    static constexpr Plan<TB, Tile<64, FPDE_NS3_BWD2_TY, 2, 104>> BWD{0, 1.3, 2.5};
    static constexpr Plan<TB, Tile<64, FPDE_NS3_BWD2_TY, 2, 103>> VG{0, 1.3, 2.5, 0.005};
    static constexpr Plan<Tile<FPDE_VJP_TX3, FPDE_VJP_TY3, 2>> VJP{0, 1.6, 2.5};
};
// 2D+t: one field less, so more workgroups per CU
struct GeoNST {
    static constexpr bool D3 = true, FWD_QUEUE = false;
    static constexpr int FWD_RING = 4;
    static constexpr double STORE_EDGE = 1.4;
    using TF = Tile<FPDE_NS3_FWD_TX, FPDE_NS3_FWD_TY, 3>;
    using TB = Tile<FPDE_NS3_BWD_TX, FPDE_NS3_BWD_TY, 1>;
    static constexpr Plan<TF, Tile<64, FPDE_NS3_FWD2_TY, 4, 140>> FWD{0.1, 1.6, 2.5};
    static constexpr Plan<TF, Tile<64, FPDE_NS3_FWD2_TY, 4, 142>> FWDR{0, 1.6, 5.0};
    static constexpr Plan<TB, Tile<64, FPDE_NS3_BWD2_TY, 2, 101>> BWD{0, 1.3, 2.5};
    static constexpr Plan<TB, Tile<64, FPDE_NS3_BWD2_TY, 2, 101>> VG{0, 1.3, 2.5, 0.005};
    static constexpr Plan<Tile<FPDE_VJP_TX3, FPDE_VJP_TY3, 4>> VJP{0, 1.6, 2.5};
};
// 3D+t NS: the forward and the explicit-sensitivity backward run the 3-D marches
// on one time level per workgroup; the backward marches time (bwdt_kernel) over
// blocks of TZ x TY x TX nodes with NT threads, one workgroup per CU.  STEP: one level's
// time, percent of the first one's (4.75, 6.3, 3.75 us on an idle chip, 6.2, 8.7, 4.65 on a
// full one); launch_bwdt takes the block with the shortest estimated march: the larger
// ones evaluate fewer residuals per node (1.65, 1.56, 1.81), the smaller ones fill more
// CUs.  Backward at 20 x 128^3 710, 656, 705 us; 14 x 56 x 55 x 83 70, 81, 79;
// 22 x 29 x 32 x 28 29, 31, 24 (815, 102, 66 with a level march and a time pass).
template <int TZ_, int TY_, int TX_, int NT_, int STEP_>
struct Block4 {
    static constexpr int TZ = TZ_, TY = TY_, TX = TX_, NT = NT_, STEP = STEP_;
};
#ifdef FPDE_T4_CHECK
using Blocks4 = std::tuple<Block4<4, 4, 64, 1024, 100>>;
#else
using Blocks4 =
    std::tuple<Block4<8, 6, 32, 768, 100>, Block4<8, 8, 32, 512, 140>, Block4<4, 8, 32, 1024, 75>>;
#endif
struct GeoNS4 {
    static constexpr bool D3 = true, FWD_QUEUE = false;
    static constexpr int FWD_RING = 4;
    static constexpr double STORE_EDGE = 1.4;
    using TF = Tile<FPDE_NS3_FWD_TX, FPDE_NS3_FWD_TY, 2>;
    static constexpr Plan<TF, Tile<64, FPDE_NS3_FWD2_TY, 3, 150>> FWD{0.3, 0, 3.0};
    static constexpr Plan<TF, Tile<64, FPDE_NS3_FWD2_TY, 3, 140>> FWDR{0.4, 0, 1.5};
    static constexpr Plan<void> BWDT{0.3, 0, 2.2, 0.0025};  // (its tiles: Blocks4)
    static constexpr Plan<Tile<FPDE_VJP_TX3, FPDE_VJP_TY3, 2>> VJP{0.3, 0, 2.5};
};
// one field, a Laplacian (heat, Poisson): 1024-thread wide forward and
// explicit-sensitivity workgroups, the others 512 threads, bound by the 2048
// threads of a CU.  The narrow forward, full rounds: 28.6 -> 29.6 us at 256^3; but 11.8 ->
// 8.4 at 97 x 90 x 41 and 9.1 -> 6.9 at 44 x 56 x 32; explicit sensitivities 26.1 -> 26.8,
// 6.0 -> 4.8 and 4.6 -> 3.8.  (The backward's wide tile is a 64-node one.)
struct GeoHeat {
    static constexpr bool D3 = true, FWD_QUEUE = FPDE_HEAT_FWD_QUEUE != 0;
    [[maybe_unused]] static constexpr int FWD_RING = FPDE_HEAT_FWD_RING;
    static constexpr double STORE_EDGE = 1.0;
    static constexpr Plan<Tile<FPDE_HEAT_FWD_TX, FPDE_HEAT_FWD_TY, 2>,
                          Tile<64, FPDE_HEAT_FWD2_TY, 4, 104>>
        FWD{0.3, 0, 5.0, 0.016}, FWDR{0.3, 0, 5.0, 0.016};
    static constexpr Plan<Tile<FPDE_HEAT_BWD_TX, FPDE_HEAT_BWD_TY, 4>> BWD{0.14, 0, 3.0},
        VG{0.43, 0, 3.4};
    static constexpr Plan<Tile<FPDE_VJP_HEAT_TX, FPDE_VJP_HEAT_TY, 2>,
                          Tile<64, FPDE_VJP_HEAT2_TY, 4, 102>>
        VJP{0.2, 0, 5.0};
};

template <class OP_, class GEO_>
struct OpTag {
    using OP = OP_;    // point functions (fpde_ops.hpp)
    using GEO = GEO_;  // launch shapes
};

// f(OpTag<...>{}) for the op, FPDE_ERR_ARG for an unknown op: the one table
// that maps an op id to its point functions and launch shapes.
template <class F>
int with_op(int op, F&& f) {
    switch (op) {
    case FPDE_BURGERS_1DT: return f(OpTag<OpBurgers, Geo2Burgers>{});
    case FPDE_HELMHOLTZ_2D: return f(OpTag<OpHelmholtz, Geo2Laplace>{});
    case FPDE_HEAT_3D_BE: return f(OpTag<OpHeat, GeoHeat>{});
    case FPDE_NS_2D_STEADY: return f(OpTag<OpNS2, Geo2NS>{});
    case FPDE_NS_3D_BE: return f(OpTag<OpNS3, GeoNS3>{});
    case FPDE_NS_3D_STEADY: return f(OpTag<OpNS3S, GeoNS3>{});
    case FPDE_POISSON_2D: return f(OpTag<OpPoisson<2>, Geo2Laplace>{});
    case FPDE_POISSON_3D: return f(OpTag<OpPoisson<3>, GeoHeat>{});
    case FPDE_NS_2DT: return f(OpTag<OpNST, GeoNST>{});
    // 3D+t: the 3-D marches run on one time level per workgroup
    case FPDE_NS_3DT: return f(OpTag<OpNS3T, GeoNS4>{});
    }
    return FPDE_ERR_ARG;
}

struct OpDesc {
    int ndim, nf, nc, nr;
    bool time;  // 3D+t: the grid has a time axis 0 before the DIM axes the kernels march
};

bool op_desc(int op, OpDesc* d) {
    return with_op(op, [&](auto tag) {
        using OP = typename decltype(tag)::OP;
        // (a 3D+t operator's consts are its own fields at the neighbouring time
        // levels, which the kernels address themselves: the caller passes none)
        *d = {OP::DIM + (OP::TIME ? 1 : 0), OP::NF, OP::TIME ? 0 : OP::NC, OP::NR, OP::TIME};
        return FPDE_OK;
    }) == FPDE_OK;
}

// ops with a time step dt among their coefficients
bool uses_dt(int op) { return op == FPDE_HEAT_3D_BE || op == FPDE_NS_3D_BE; }

struct Req {
    int op;
    OpDesc d;
    Dims dims;
    KCoef K;
    double inv_M, two_over_M;
    long long N, M;
    Ptrs P;
    hipStream_t stream;
    double* ws;  // loss workspace of the call, or nullptr
};

bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return x < y + nb && y < x + na;
}

bool finite_pos(double v) { return isfinite(v) && v > 0.0; }

// Validates everything except the outputs; fills req.  need_consts: the call
// reads the const arrays (the explicit-sensitivity backward does not).
int validate_common(int op, const fpde_grid4* g, const fpde_coeffs* c, const float* const* fields,
                    const float* const* consts, Req* r, bool need_consts = true) {
    if (!op_desc(op, &r->d)) return FPDE_ERR_ARG;
    if (!g || !c || !fields) return FPDE_ERR_ARG;
    if (!need_consts) consts = nullptr;
    const int nc = need_consts ? r->d.nc : 0;
    if (nc > 0 && !consts) return FPDE_ERR_ARG;
    for (int f = 0; f < r->d.nf; ++f)
        if (!fields[f]) return FPDE_ERR_ARG;
    for (int j = 0; j < nc; ++j)
        if (!consts[j]) return FPDE_ERR_ARG;
    if (g->bc_mode != 0 && g->bc_mode != 1) return FPDE_ERR_ARG;
    if (g->ndim != r->d.ndim) return FPDE_ERR_SHAPE;
    const int D = r->d.ndim;
    const bool per = g->bc_mode == 1;
    long long N = 1, M = 1;
    for (int a = 0; a < D; ++a) {
        if (g->n[a] < 3 || g->n[a] >= (1LL << 31)) return FPDE_ERR_SHAPE;
        if (N > (1LL << 62) / g->n[a]) return FPDE_ERR_SHAPE;
        N *= g->n[a];
        M *= per ? g->n[a] : g->n[a] - 2;  // periodic: a residual at every node
    }
    // plane of the last two axes (one row for 2-D grids) addressed with 32-bit byte
    // offsets; a 3D+t grid's time level (the last three axes) as well
    if ((D >= 3 ? g->n[D - 2] * g->n[D - 1] : g->n[1]) >= (1LL << 29)) return FPDE_ERR_SHAPE;
    if (D == 4 && g->n[1] * g->n[2] * g->n[3] >= (1LL << 29)) return FPDE_ERR_SHAPE;
    for (int a = 0; a < D; ++a)
        if (!finite_pos(g->h[a])) return FPDE_ERR_SPACING;
    if (!isfinite(c->nu) || !isfinite(c->k) || !isfinite(c->dt) || !isfinite(c->alpha))
        return FPDE_ERR_COEFF;
    if (uses_dt(op) && !(c->dt > 0.0)) return FPDE_ERR_COEFF;

    // float32 kernel coefficients, derived in float64; a 3D+t grid's kernel axes
    // are its spatial axes 1..3, and its time axis 0 has a coefficient of its own
    const int A0 = r->d.time ? 1 : 0;  // first array axis the kernels march
    KCoef K;
    memset(&K, 0, sizeof K);
    for (int a = 0; a < D - A0; ++a) {
        const double h = g->h[a + A0];
        K.i2hd[a] = 1.0 / (2.0 * h);
        K.i2h[a] = (float)(1.0 / (2.0 * h));
        K.ih2[a] = (float)(1.0 / (h * h));
        if (!isfinite(K.i2h[a]) || !isfinite(K.ih2[a]) || K.ih2[a] == 0.f) return FPDE_ERR_SPACING;
    }
    if (r->d.time) {
        K.i2ht = (float)(1.0 / (2.0 * g->h[0]));
        if (!isfinite(K.i2ht)) return FPDE_ERR_SPACING;
    }
    K.nu = (float)c->nu;
    K.k2 = (float)(c->k * c->k);
    K.inv_dt = uses_dt(op) ? (float)(1.0 / c->dt) : 0.f;
    K.alpha = (float)c->alpha;
    if (!isfinite(K.nu) || !isfinite(K.k2) || !isfinite(K.inv_dt) || !isfinite(K.alpha))
        return FPDE_ERR_COEFF;

    for (int f = 0; f < r->d.nf; ++f)
        if ((uintptr_t)fields[f] & 3u) return FPDE_ERR_ALIGN;
    for (int j = 0; j < nc; ++j)
        if ((uintptr_t)consts[j] & 3u) return FPDE_ERR_ALIGN;

    r->ws = nullptr;
    r->op = op;
    r->K = K;
    r->N = N;
    r->M = M;
    r->inv_M = 1.0 / (double)M;
    r->two_over_M = 2.0 / (double)M;
    memset(&r->P, 0, sizeof r->P);
    for (int f = 0; f < r->d.nf; ++f) r->P.f[f] = fields[f];
    for (int j = 0; j < nc; ++j) r->P.c[j] = consts[j];

    Dims& dm = r->dims;  // sizes only; tiles and chunks are set per launch
    dm.nz = (int)g->n[A0];
    dm.ny = (D - A0 == 3) ? (int)g->n[A0 + 1] : 1;
    dm.nx = (int)g->n[D - 1];
    dm.tiles_x = dm.tiles_y = dm.zc = dm.nblocks = 0;
    dm.per = per ? 1 : 0;
    dm.zlo = per ? 0 : 1;  // the marched planes: 1 .. n0-2, or all of them
    dm.nt = r->d.time ? (int)g->n[0] : 1;
    dm.nlev = 1;  // (set per launch for 3D+t grids)
    dm.lev0 = 0;
    dm.vol = r->d.time ? (long long)dm.nz * dm.ny * dm.nx : 0;
    // every launch shape used below must have fewer than 2^31 workgroups
    // (in 64 bits: an extent of axis 0 may be up to 2^31 - 1)
    if (((long long)dm.nx / 32 + 1) * ((long long)dm.ny + 1) * ((long long)dm.nz + 1) * dm.nt >=
        (1LL << 31))
        return FPDE_ERR_SHAPE;
    return FPDE_OK;
}

// The time levels a 3D+t launch covers: those with residuals (1 .. nt-2), or
// every level (periodic grids; the explicit-sensitivity backward, which writes
// every node).  No-op for other grids.
Dims levels(const Dims& n, bool all) {
    Dims dm = n;
    if (dm.nt > 1) {
        const bool every = all || dm.per;
        dm.lev0 = every ? 0 : 1;
        dm.nlev = every ? dm.nt : dm.nt - 2;
    }
    return dm;
}

// Tiles of TX x TY columns; chunks of zc planes along axis 0.
Dims tile_dims(const Dims& n, int TX, int TY, int zc) {
    Dims dm = n;
    dm.tiles_x = (dm.nx + TX - 1) / TX;
    dm.tiles_y = (dm.ny + TY - 1) / TY;
    const int nplanes = dm.nz - 2 * dm.zlo;
    dm.zc = zc;
    const long long nch = (nplanes + zc - 1) / zc;
    dm.nblocks = (int)((long long)dm.tiles_x * dm.tiles_y * nch * dm.nlev);
    return dm;
}

// Chunk length of a march with TX x TY tiles of which `res` workgroups fit a
// CU at once.  A launch runs in rounds of CUs * res workgroups, each as long as
// one chunk's march (its planes plus `prologue` planes' worth of the first planes' latency
// and the halo planes' residuals), so a launch a little over a whole
// number of rounds idles most of the chip in its last one: at 150 x 131 x 257 the
// NS-3D backward takes 93 us cut into 306 workgroups and 61 us cut into 255, and
// the 2D+t one at 33 x 201 x 259 28 us in 312 and 20 us in 234.  The rule takes,
// among the chunk counts that just fill 1, 2, ... CUs' worth of workgroups, the
// one with the shortest estimated march.  In a last round with k of res
// workgroups per CU (LDS marches: on the fullest CU) a step takes, of a full round's,
//     max(floor / res, s + (1 - s) k / res),
// s (the march's share, a register-queue march's share / res) the latency that remains
// however few there are, and floor the workgroups that it takes to fill a CU's bandwidth:
// one field's marches go by the first (measured, k = 1 .. res: heat backward 0.38, 0.56,
// 0.77, 1; 2-D backward 0.28 at one, 0.33 at two of eight), several fields' by the second
// (NS-3D narrow forward 0.45, 0.68, 1; 2D+t explicit sensitivities 0.45, 0.55, 0.75, 1;
// NS-2D ones 0.37, 0.47, 0.60, 0.78, 1).
// A loss costs one atomic per workgroup of the last round, serialised at 12 ns, `atom`
// of a step (0.012, and 0.0025 of a level of the time march), or through a workspace a
// second level of slots beyond 64 workgroups, as much as 65 of them.
enum class Sum { none, atomics, workspace };
#ifndef FPDE_CUS
#define FPDE_CUS 256
#endif
constexpr int kCUs = FPDE_CUS;
struct Chunks {
    int zc;       // planes per chunk
    double cost;  // estimated time, in steps of a full round of the wide tile's workgroups
};
template <class P>
Chunks plan_chunks(const Dims& n, int TX, int TY, int res, int step, Sum sum, const P& p,
                   bool queue = false) {
    const long long tiles =
        (long long)((n.nx + TX - 1) / TX) * ((n.ny + TY - 1) / TY) * n.nlev;
    const int nplanes = n.nz - 2 * n.zlo;
    const double s = queue ? p.share / res : p.share;
    auto part = [&](double k) {  // a step with k workgroups per CU, of a full round's
        const double v = s + (1.0 - s) * k / res, least = p.floor / res;
        return v > least ? v : least < 1.0 ? least : 1.0;
    };
    Chunks best = {nplanes, 0.0};
    long long tried = 0;
    // an eighth, a quarter, half of the CUs; CU loads 1 .. res (one round, in
    // part); then whole rounds up to 8
    for (int j = -2; j <= res + 7; ++j) {
        const long long slots = j <= 0      ? kCUs >> (1 - j)
                                : j <= res ? (long long)j * kCUs
                                           : (long long)(j - res + 1) * res * kCUs;
        long long nch = slots / tiles;
        nch = nch < 1 ? 1 : nch > nplanes ? nplanes : nch;
        if (nch == tried) continue;
        tried = nch;
        const int zc = (int)((nplanes + nch - 1) / nch);
        const long long W = tiles * ((nplanes + zc - 1) / zc);
        const long long round = (long long)kCUs * res, full = W / round;
        const long long rest = W - full * round;
        const double k = queue ? (double)rest / kCUs : (double)((rest + kCUs - 1) / kCUs);
        double cost = (zc + p.prologue) * ((double)full + (rest ? part(k) : 0.0)) * step / 100.0;
        // (a launch with more workgroups than the workspace has slots adds atomically)
        if (sum == Sum::atomics || (sum == Sum::workspace && W > kWsMaxBlocks))
            cost += p.atom * (double)(W < round ? W : round);
        else if (sum == Sum::workspace && W > kGroup)
            cost += 65.0 * p.atom;
        if (best.cost == 0.0 || cost < best.cost) best = {zc, cost};
    }
    return best;
}
// ... of a launch of tile T of plan p
template <class T, class P>
Chunks plan_tile(const P& p, const Dims& n, Sum sum, bool queue) {
    return plan_chunks(n, T::TX, T::TY, T::res(sum != Sum::none, n.per != 0), T::STEP, sum, p,
                       queue);
}

int check_outputs(const Req& r, const fpde_grid4*, const float* const* fields,
                  const float* const* consts, float* const* outs, int nout, const void* extra,
                  size_t extra_bytes) {
    const size_t bytes = (size_t)r.N * sizeof(float);
    for (int o = 0; o < nout; ++o) {
        if (!outs[o]) return FPDE_ERR_ARG;
        if ((uintptr_t)outs[o] & 3u) return FPDE_ERR_ALIGN;
        for (int f = 0; f < r.d.nf; ++f)
            if (overlaps(outs[o], bytes, fields[f], bytes)) return FPDE_ERR_ARG;
        for (int j = 0; j < r.d.nc; ++j)
            if (overlaps(outs[o], bytes, consts[j], bytes)) return FPDE_ERR_ARG;
        for (int p = 0; p < o; ++p)
            if (overlaps(outs[o], bytes, outs[p], bytes)) return FPDE_ERR_ARG;
        if (extra && overlaps(outs[o], bytes, extra, extra_bytes)) return FPDE_ERR_ARG;
    }
    return FPDE_OK;
}

template <class T>
struct ident {
    using type = T;
};

// Queues kernel k on stream s and returns the status of that launch alone:
// hipLaunchKernel's own return value.  The thread's last-error state, which the
// caller may have left set by an earlier call, is neither read nor cleared.
// (The arguments take the kernel's parameter types, so each is passed in the
// layout the kernel expects.)
template <class... P>
int launch(void (*k)(P...), dim3 grid, dim3 block, hipStream_t s,
           typename ident<P>::type... args) {
    void* a[] = {(void*)&args...};
    return hipLaunchKernel(reinterpret_cast<const void*>(k), grid, block, a, 0, s) == hipSuccess
               ? FPDE_OK
               : FPDE_ERR_HIP;
}

// Before a launch of nblocks workgroups that sums a loss: the workspace it goes
// through, if the call has one large enough for the launch (a longer launch hides its
// atomics, which are spread over its rounds), else *loss zeroed
int begin_loss(const Req& r, int nblocks, double* loss, double** ws) {
    *ws = r.ws && nblocks <= kWsMaxBlocks ? r.ws : nullptr;
    return *ws ? FPDE_OK : launch(fill_f64_kernel, dim3(1), dim3(1), r.stream, loss, 0.0);
}

// ---- launches, per op type

// f(std::bool_constant<v>{}) for a runtime flag v: kernels take flags that
// decide their per-step control flow (periodic wrap, ...) as template arguments
template <class F>
void with_flag(bool v, F&& f) {
    if (v) f(std::true_type{});
    else f(std::false_type{});
}

template <class OP, int TX, int TY, int RD>
int launch_fwd(const Req& r, bool store, double* loss, int zc) {
    const Dims dm = tile_dims(r.dims, TX, TY, zc);
    double* ws;
    int st = begin_loss(r, dm.nblocks, loss, &ws);
    if (st != FPDE_OK) return st;
    if (OP::TIME && store && !dm.per) {  // the end time levels hold no residual node
        st = launch(zero_levels_kernel<OP::NR>, dim3((unsigned)((2 * dm.vol + 255) / 256)),
                    dim3(256), r.stream, r.P, dm);
        if (st != FPDE_OK) return st;
    }
    with_flag(store, [&](auto sr) {
        with_flag(dm.per, [&](auto per) {
            st = launch(fwd_kernel<OP, TX, TY, decltype(sr)::value, decltype(per)::value, RD>,
                        dim3(dm.nblocks), dim3(TX * TY), r.stream, r.P, dm, r.K, r.inv_M, loss,
                        ws);
        });
    });
    return st;
}

// the register-queue forward (no LDS, no barrier)
template <class OP, int TX, int TY>
int launch_fwdq(const Req& r, bool store, double* loss, int zc) {
    const Dims dm = tile_dims(r.dims, TX, TY, zc);
    double* ws;
    int st = begin_loss(r, dm.nblocks, loss, &ws);
    if (st != FPDE_OK) return st;
    with_flag(store, [&](auto sr) {
        with_flag(dm.per, [&](auto per) {
            st = launch(fwdq_kernel<OP, TX, TY, FPDE_FWD2_Q, decltype(sr)::value,
                                    decltype(per)::value>,
                        dim3(dm.nblocks), dim3(TX * TY), r.stream, r.P, dm, r.K, r.inv_M, loss,
                        ws);
        });
    });
    return st;
}

template <class OP, int TX, int TY>
int launch_bwd(const Req& r, const double* dloss, int zc, double* loss) {
    const Dims dm = tile_dims(r.dims, TX, TY, zc);
    // value and gradient in one pass when loss is given
    double* ws = nullptr;
    int st = loss ? begin_loss(r, dm.nblocks, loss, &ws) : FPDE_OK;
    if (st != FPDE_OK) return st;
    with_flag(loss != nullptr, [&](auto lo) {
        with_flag(dm.per, [&](auto per) {
            st = launch(bwd_kernel<OP, TX, TY, kBwdReverse, decltype(lo)::value,
                                   decltype(per)::value>,
                        dim3(dm.nblocks), dim3(TX * TY), r.stream, r.P, dm, r.K, dloss,
                        r.two_over_M, r.inv_M, loss, ws);
        });
    });
    return st;
}

// 2-D register-queue backward (with the loss when given)
template <class OP, int NW>
int launch_bwdq(const Req& r, const double* dloss, int zc, double* loss) {
    const Dims dm = tile_dims(r.dims, 62 * NW, 1, zc);
    double* ws = nullptr;
    int st = loss ? begin_loss(r, dm.nblocks, loss, &ws) : FPDE_OK;
    if (st != FPDE_OK) return st;
    auto go = [&](auto lo) {
        with_flag(dm.per, [&](auto per) {
            st = launch(bwdq_kernel<OP, NW, FPDE_BWD2_Q, decltype(lo)::value, decltype(per)::value>,
                        dim3(dm.nblocks), dim3(64 * NW), r.stream, r.P, dm, r.K, dloss,
                        r.two_over_M, r.inv_M, loss, ws);
        });
    };
    if constexpr (NW == FPDE_BWD2_NW) with_flag(loss != nullptr, go);
    else go(std::true_type{});  // (the other widths are taken with a loss only)
    return st;
}

Sum loss_sum(const Req& r, const double* loss) {
    return !loss ? Sum::none : r.ws ? Sum::workspace : Sum::atomics;
}

// f(Tile<...>{}, zc) for the wide or the narrow tile of a plan, whichever has the shorter
// estimated march (plan_chunks), the narrow one's times `extra`
template <bool QUEUE = false, class P, class F>
int with_tile(const P& p, const Dims& n, Sum sum, double extra, F&& f) {
    using A = typename P::W;
    using B = typename P::N;
    const Chunks a = plan_tile<A>(p, n, sum, QUEUE);
    if (!std::is_same<A, B>::value) {
        const Chunks b = plan_tile<B>(p, n, sum, QUEUE);
        if (extra * b.cost < a.cost) return f(B{}, b.zc);
    }
    return f(A{}, a.zc);
}

// Residual stores beyond the 32 MB of the L2s: rows of a ragged grid are not aligned to
// cache lines, and each tile edge splits one between two workgroups' non-temporal stores
// (NS-3D 150 x 131 x 257: 47 us with 128-wide tiles, 58 with 64-wide ones), so the narrow
// tile's march costs STORE_EDGE times as much: 1.4 for several fields, nothing for one.  (It
// was ruled out there, which left half the lanes of a wide tile idle on rows of up to 64
// nodes and a few more: 3D+t forwards with residuals up to 1.9, heat ones up to 1.6 times the
// narrow tile's time.)
template <class GEO, class OP>
int launch_fwd3(const Req& r, bool store, double* loss) {
    const double extra = store && r.N * OP::NR * 4 > (32LL << 20) ? GEO::STORE_EDGE : 1.0;
    auto go = [&](auto t, int zc) {
        using T = decltype(t);
        if constexpr (GEO::FWD_QUEUE)
            return launch_fwdq<OP, T::TX, T::TY>(r, store, loss, zc);
        else
            return launch_fwd<OP, T::TX, T::TY, GEO::FWD_RING>(r, store, loss, zc);
    };
    const Sum sum = loss_sum(r, loss);
    return store ? with_tile<GEO::FWD_QUEUE>(GEO::FWDR, r.dims, sum, extra, go)
                 : with_tile<GEO::FWD_QUEUE>(GEO::FWD, r.dims, sum, extra, go);
}
template <class GEO, class OP>
int launch_bwd3(const Req& r, const double* dloss, double* loss) {
    auto go = [&](auto t, int zc) {
        using T = decltype(t);
        return launch_bwd<OP, T::TX, T::TY>(r, dloss, zc, loss);
    };
    return loss ? with_tile(GEO::VG, r.dims, loss_sum(r, loss), 1.0, go)
                : with_tile(GEO::BWD, r.dims, Sum::none, 1.0, go);
}

// 2-D launches
template <class GEO, class OP>
int launch_fwd2(const Req& r, bool store, double* loss) {
    auto go = [&](auto t, int zc) {
        return launch_fwdq<OP, decltype(t)::TX, 1>(r, store, loss, zc);
    };
    const Sum sum = loss_sum(r, loss);
    return store ? with_tile<true>(GEO::FWDR, r.dims, sum, 1.0, go)
                 : with_tile<true>(GEO::FWD, r.dims, sum, 1.0, go);
}
template <class GEO, class OP>
int launch_bwd2(const Req& r, const double* dloss, double* loss) {
    if constexpr (FPDE_BWD2_QUEUE) {
        auto run = [&](auto t, int zc) {
            return launch_bwdq<OP, decltype(t)::TX / 62>(r, dloss, zc, loss);
        };
        if (!loss) return with_tile<true>(GEO::BWD, r.dims, Sum::none, 1.0, run);
        if (r.ws) {
            using T = typename decltype(GEO::VG)::W;
            const int zc = plan_tile<T>(GEO::VG, r.dims, Sum::workspace, true).zc;
            if (tile_dims(r.dims, T::TX, 1, zc).nblocks <= kWsMaxBlocks) return run(T{}, zc);
        }
        // no workspace, or a launch with more workgroups than it holds
        return with_tile<true>(GEO::VGA, r.dims, Sum::atomics, 1.0, run);
    } else {
        const int zc =
            plan_chunks(r.dims, FPDE_TX2, 1, 4, 100, loss_sum(r, loss), GEO::VJP).zc;
        return launch_bwd<OP, FPDE_TX2, 1>(r, dloss, zc, loss);
    }
}

template <class OP>
int launch_bc(const Req& r, const double* dloss) {
    if constexpr (OP::TIME) {
        // 3D+t: the two end time levels, 256 consecutive nodes of a level per
        // workgroup (fewer than 2^31: a level holds fewer than 2^29 nodes)
        const long long nb = 2 * ((r.dims.vol + 255) / 256);
        return launch(bc4_kernel<OP>, dim3((unsigned)nb), dim3(256), r.stream, r.P, r.dims, r.K,
                      dloss, r.two_over_M);
    } else {
        // the two end planes of axis 0: one workgroup per 256-node segment of each row
        // (fewer than 2^31 of them: the node count of a plane is below 2^29)
        const long long nb = 2LL * r.dims.ny * ((r.dims.nx + 255) / 256);
        return launch(bc_kernel<OP>, dim3((unsigned)nb), dim3(256), r.stream, r.P, r.dims, r.K,
                      dloss, r.two_over_M);
    }
}

// 3D+t: the time-marching backward (with the loss when given).  A chunk of levels
// evaluates residuals at up to two levels more than it writes: its prologue.
template <class OP, class T>
int launch_bwdt_as(const Req& r, const double* dloss, double* loss, int zc) {
    constexpr int TZ = T::TZ, TY = T::TY, TX = T::TX, NT = T::NT;
    Dims dm = r.dims;
    dm.tiles_x = (dm.nx + TX - 1) / TX;
    dm.tiles_y = (dm.ny + TY - 1) / TY;
    dm.zc = zc;
    dm.nblocks = dm.tiles_x * dm.tiles_y * ((dm.nz + TZ - 1) / TZ) * ((dm.nlev + zc - 1) / zc);
    double* ws = nullptr;
    int st = loss ? begin_loss(r, dm.nblocks, loss, &ws) : FPDE_OK;
    if (st != FPDE_OK) return st;
    with_flag(loss != nullptr, [&](auto lo) {
        with_flag(dm.per, [&](auto per) {
            st = launch(bwdt_kernel<OP, TZ, TY, TX, NT, decltype(lo)::value, decltype(per)::value>,
                        dim3(dm.nblocks), dim3(NT), r.stream, r.P, dm, r.K, dloss, r.two_over_M,
                        r.inv_M, loss, ws);
        });
    });
    return st;
}
template <class OP, class... T>
int launch_bwdt(const Req& r, const double* dloss, double* loss, std::tuple<T...>) {
    Dims q = {};  // a launch's chunks: those of a march over nlev planes of its blocks
    q.ny = q.nlev = 1;
    q.nz = r.dims.nlev;
    int best = -1, zc = 0, i = 0;
    double cost = 0.0;
    auto consider = [&](auto t) {
        using B = decltype(t);
        q.nx = ((r.dims.nx + B::TX - 1) / B::TX) * ((r.dims.ny + B::TY - 1) / B::TY) *
               ((r.dims.nz + B::TZ - 1) / B::TZ);
        const Chunks c = plan_chunks(q, 1, 1, 1, B::STEP, loss_sum(r, loss), GeoNS4::BWDT);
        // (a launch holds fewer than 2^32 threads: on a level a few nodes thin, where a
        // block is mostly empty, the blocks with more threads per node are out; the
        // 8 x 8 x 32 ones, half a thread each, fit every level)
        if ((long long)q.nx * B::NT < (1LL << 32) && (best < 0 || c.cost < cost)) {
            best = i;
            zc = c.zc;
            cost = c.cost;
        }
        ++i;
    };
    (consider(T{}), ...);
    int st = FPDE_ERR_HIP;  // (the runtime would refuse every one of them)
    i = 0;
    ((i++ == best ? (void)(st = launch_bwdt_as<OP, T>(r, dloss, loss, zc)) : (void)0), ...);
    return st;
}

// Explicit-sensitivity backward: every plane of axis 0 is marched (zlo = 0),
// on a 3D+t grid in every time level.
template <class OP, int TX, int TY>
int launch_vjp(const Req& r, bool acc, const Dims& base, int zc) {
    const Dims dm = tile_dims(base, TX, TY, zc);
    int st = FPDE_OK;
    with_flag(acc, [&](auto ac) {
        with_flag(dm.per, [&](auto per) {
            st = launch(vjp_kernel<OP, TX, TY, decltype(ac)::value, decltype(per)::value>,
                        dim3(dm.nblocks), dim3(TX * TY), r.stream, r.P, dm, r.K);
        });
    });
    return st;
}

int run_vjp(const Req& r, bool acc) {
    Dims base = levels(r.dims, true);
    base.zlo = 0;
    return with_op(r.op, [&](auto tag) {
        using OP = typename decltype(tag)::OP;
        using GEO = typename decltype(tag)::GEO;
        return with_tile(
            GEO::VJP, base, Sum::none, 1.0, [&](auto t, int zc) {
                using T = decltype(t);
                return launch_vjp<OP, T::TX, T::TY>(r, acc, base, zc);
            });
    });
}

int run_fwd(const Req& r0, bool store, double* loss) {
    Req r = r0;
    r.dims = levels(r0.dims, false);
    return with_op(r.op, [&](auto tag) {
        using OP = typename decltype(tag)::OP;
        using GEO = typename decltype(tag)::GEO;
        if constexpr (GEO::D3)
            return launch_fwd3<GEO, OP>(r, store, loss);
        else
            return launch_fwd2<GEO, OP>(r, store, loss);
    });
}

// loss: nullptr for the gradient alone (planes 1 .. n0-2; the boundary kernel
// writes the end planes), else also the loss (fused value and grad), marching
// every plane: at the end planes the gather with the residuals off the residual
// set taken as zero is their exact boundary term, so no boundary kernel follows
//
// 3D+t grids: the time march covers every level with residuals; with the loss the
// end time levels follow (bc_mode 0).
int run_bwd(const Req& r0, const double* dloss, double* loss = nullptr) {
    Req r = r0;
    r.dims = levels(r0.dims, false);
    if (loss) r.dims.zlo = 0;
    return with_op(r.op, [&](auto tag) {
        using OP = typename decltype(tag)::OP;
        using GEO = typename decltype(tag)::GEO;
        if constexpr (OP::TIME) {
            int st = launch_bwdt<OP>(r, dloss, loss, Blocks4{});
            if (st == FPDE_OK && loss && !r.dims.per) st = launch_bc<OP>(r, dloss);
            return st;
        } else if constexpr (GEO::D3)
            return launch_bwd3<GEO, OP>(r, dloss, loss);
        else
            return launch_bwd2<GEO, OP>(r, dloss, loss);
    });
}

int run_bc(const Req& r, const double* dloss) {
    if (r.dims.per) return FPDE_OK;  // a periodic grid has no boundary: the march wrote every node
    return with_op(r.op, [&](auto tag) {
        return launch_bc<typename decltype(tag)::OP>(r, dloss);
    });
}

int prepare_grad_call(int op, const fpde_grid4* grid, const fpde_coeffs* coeffs,
                      const float* const* fields, const float* const* consts, const double* dloss,
                      float* const* grads, void* stream, Req* r) {
    int st = validate_common(op, grid, coeffs, fields, consts, r);
    if (st != FPDE_OK) return st;
    if (!dloss || !grads) return FPDE_ERR_ARG;
    if ((uintptr_t)dloss & 7u) return FPDE_ERR_ALIGN;
    st = check_outputs(*r, grid, fields, consts, grads, r->d.nf, dloss, sizeof(double));
    if (st != FPDE_OK) return st;
    for (int f = 0; f < r->d.nf; ++f) r->P.out[f] = grads[f];
    r->stream = (hipStream_t)stream;
    return FPDE_OK;
}

}  // namespace
}  // namespace fpde

using namespace fpde;

extern "C" int fpde_op_info(int op, int* ndim, int* n_fields, int* n_consts, int* n_residuals) {
    OpDesc d;
    if (!op_desc(op, &d)) return FPDE_ERR_ARG;
    if (ndim) *ndim = d.ndim;
    if (n_fields) *n_fields = d.nf;
    if (n_consts) *n_consts = d.nc;
    if (n_residuals) *n_residuals = d.nr;
    return FPDE_OK;
}

// The workspace of a *_ws4 call: checked against every other argument array, and
// left unused while the stream is being captured (the graph's replays would read
// and write it later, when its owner may have given it back or use it itself).
static int take_workspace(Req* r, double* loss, const double* dloss, float* const* outs, int nout,
                          void* ws) {
    if (!ws) return FPDE_ERR_ARG;
    if ((uintptr_t)ws & 7u) return FPDE_ERR_ALIGN;
    const size_t bytes = (size_t)r->N * sizeof(float);
    constexpr size_t wb = kWsDoubles * sizeof(double);
    static_assert(wb == FPDE_WORKSPACE_BYTES, "the header's size");
    if (overlaps(ws, wb, loss, sizeof(double)) ||
        (dloss && overlaps(ws, wb, dloss, sizeof(double))))
        return FPDE_ERR_ARG;
    for (int f = 0; f < r->d.nf; ++f)
        if (overlaps(ws, wb, r->P.f[f], bytes)) return FPDE_ERR_ARG;
    for (int j = 0; j < r->d.nc; ++j)
        if (overlaps(ws, wb, r->P.c[j], bytes)) return FPDE_ERR_ARG;
    for (int o = 0; o < nout; ++o)
        if (overlaps(ws, wb, outs[o], bytes)) return FPDE_ERR_ARG;
    hipStreamCaptureStatus cap;
    if (hipStreamIsCapturing(r->stream, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone)
        r->ws = (double*)ws;
    return FPDE_OK;
}

// ws: a workspace, or nullptr for a call without one (with_ws false)
static int fwd_impl(int op, const fpde_grid4* grid, const fpde_coeffs* coeffs,
                    const float* const* fields, const float* const* consts,
                    float* const* residual_out, double* loss, void* stream, bool with_ws = false,
                    void* ws = nullptr) {
    Req r;
    int st = validate_common(op, grid, coeffs, fields, consts, &r);
    if (st != FPDE_OK) return st;
    if (!loss) return FPDE_ERR_ARG;
    if ((uintptr_t)loss & 7u) return FPDE_ERR_ALIGN;
    const size_t bytes = (size_t)r.N * sizeof(float);
    for (int f = 0; f < r.d.nf; ++f)
        if (overlaps(loss, sizeof(double), fields[f], bytes)) return FPDE_ERR_ARG;
    for (int j = 0; j < r.d.nc; ++j)
        if (overlaps(loss, sizeof(double), consts[j], bytes)) return FPDE_ERR_ARG;
    if (residual_out) {
        st = check_outputs(r, grid, fields, consts, residual_out, r.d.nr, loss, sizeof(double));
        if (st != FPDE_OK) return st;
        for (int b = 0; b < r.d.nr; ++b) r.P.out[b] = residual_out[b];
    }
    r.stream = (hipStream_t)stream;
    if (with_ws) {
        st = take_workspace(&r, loss, nullptr, residual_out, residual_out ? r.d.nr : 0, ws);
        if (st != FPDE_OK) return st;
    }
    return run_fwd(r, residual_out != nullptr, loss);
}

static int bwd_impl(int op, const fpde_grid4* grid, const fpde_coeffs* coeffs,
                                 const float* const* fields, const float* const* consts,
                                 const double* dloss, float* const* grads, void* stream) {
    Req r;
    const int st = prepare_grad_call(op, grid, coeffs, fields, consts, dloss, grads, stream, &r);
    if (st != FPDE_OK) return st;
    return run_bwd(r, dloss);
}

static int bc_impl(int op, const fpde_grid4* grid, const fpde_coeffs* coeffs,
                               const float* const* fields, const float* const* consts,
                               const double* dloss, float* const* grads, void* stream) {
    Req r;
    const int st = prepare_grad_call(op, grid, coeffs, fields, consts, dloss, grads, stream, &r);
    if (st != FPDE_OK) return st;
    return run_bc(r, dloss);
}

static int value_and_grad_impl(int op, const fpde_grid4* grid, const fpde_coeffs* coeffs,
                               const float* const* fields, const float* const* consts,
                               const double* dloss, double* loss, float* const* grads,
                               void* stream, bool with_ws = false, void* ws = nullptr) {
    Req r;
    int st = prepare_grad_call(op, grid, coeffs, fields, consts, dloss, grads, stream, &r);
    if (st != FPDE_OK) return st;
    if (!loss) return FPDE_ERR_ARG;
    if ((uintptr_t)loss & 7u) return FPDE_ERR_ALIGN;
    const size_t bytes = (size_t)r.N * sizeof(float);
    if (overlaps(loss, sizeof(double), dloss, sizeof(double))) return FPDE_ERR_ARG;
    for (int f = 0; f < r.d.nf; ++f)
        if (overlaps(loss, sizeof(double), fields[f], bytes) ||
            overlaps(loss, sizeof(double), grads[f], bytes))
            return FPDE_ERR_ARG;
    for (int j = 0; j < r.d.nc; ++j)
        if (overlaps(loss, sizeof(double), consts[j], bytes)) return FPDE_ERR_ARG;
    if (with_ws) {
        st = take_workspace(&r, loss, dloss, grads, r.d.nf, ws);
        if (st != FPDE_OK) return st;
    }
    return run_bwd(r, dloss, loss);
}

static int vjp_impl(int op, const fpde_grid4* grid, const fpde_coeffs* coeffs,
                                 const float* const* fields, const float* const* sens,
                                 int accumulate, float* const* grads, void* stream) {
    Req r;
    int st = validate_common(op, grid, coeffs, fields, nullptr, &r, false);
    if (st != FPDE_OK) return st;
    if (!sens || !grads) return FPDE_ERR_ARG;
    if (accumulate != 0 && accumulate != 1) return FPDE_ERR_ARG;
    const size_t bytes = (size_t)r.N * sizeof(float);
    for (int b = 0; b < r.d.nr; ++b) {
        if (!sens[b]) return FPDE_ERR_ARG;
        if ((uintptr_t)sens[b] & 3u) return FPDE_ERR_ALIGN;
    }
    for (int f = 0; f < r.d.nf; ++f) {
        if (!grads[f]) return FPDE_ERR_ARG;
        if ((uintptr_t)grads[f] & 3u) return FPDE_ERR_ALIGN;
        for (int q = 0; q < r.d.nf; ++q)
            if (overlaps(grads[f], bytes, fields[q], bytes)) return FPDE_ERR_ARG;
        for (int b = 0; b < r.d.nr; ++b)
            if (overlaps(grads[f], bytes, sens[b], bytes)) return FPDE_ERR_ARG;
        for (int q = 0; q < f; ++q)
            if (overlaps(grads[f], bytes, grads[q], bytes)) return FPDE_ERR_ARG;
    }
    for (int b = 0; b < r.d.nr; ++b) r.P.s[b] = sens[b];
    for (int f = 0; f < r.d.nf; ++f) r.P.out[f] = grads[f];
    r.stream = (hipStream_t)stream;
    return run_vjp(r, accumulate == 1);
}

// fpde_grid (three axes) as fpde_grid4; ndim is checked against the op's later
static const fpde_grid4* widen(const fpde_grid* g, fpde_grid4* w) {
    if (!g) return nullptr;
    memset(w, 0, sizeof *w);
    w->ndim = g->ndim > 3 ? -1 : g->ndim;  // (four axes do not fit an fpde_grid)
    w->bc_mode = g->bc_mode;
    for (int a = 0; a < 3; ++a) {
        w->n[a] = g->n[a];
        w->h[a] = g->h[a];
    }
    return w;
}

extern "C" int fpde_residual_fwd(int op, const fpde_grid* grid, const fpde_coeffs* coeffs,
                                 const float* const* fields, const float* const* consts,
                                 float* const* residual_out, double* loss, void* stream) {
    fpde_grid4 w;
    return fwd_impl(op, widen(grid, &w), coeffs, fields, consts, residual_out, loss, stream);
}

extern "C" int fpde_residual_bwd(int op, const fpde_grid* grid, const fpde_coeffs* coeffs,
                                 const float* const* fields, const float* const* consts,
                                 const double* dloss, float* const* grads, void* stream) {
    fpde_grid4 w;
    return bwd_impl(op, widen(grid, &w), coeffs, fields, consts, dloss, grads, stream);
}

extern "C" int fpde_bc_correct(int op, const fpde_grid* grid, const fpde_coeffs* coeffs,
                               const float* const* fields, const float* const* consts,
                               const double* dloss, float* const* grads, void* stream) {
    fpde_grid4 w;
    return bc_impl(op, widen(grid, &w), coeffs, fields, consts, dloss, grads, stream);
}

extern "C" int fpde_residual_value_and_grad(int op, const fpde_grid* grid,
                                            const fpde_coeffs* coeffs, const float* const* fields,
                                            const float* const* consts, const double* dloss,
                                            double* loss, float* const* grads, void* stream) {
    fpde_grid4 w;
    return value_and_grad_impl(op, widen(grid, &w), coeffs, fields, consts, dloss, loss, grads,
                               stream);
}

extern "C" int fpde_residual_vjp(int op, const fpde_grid* grid, const fpde_coeffs* coeffs,
                                 const float* const* fields, const float* const* sens,
                                 int accumulate, float* const* grads, void* stream) {
    fpde_grid4 w;
    return vjp_impl(op, widen(grid, &w), coeffs, fields, sens, accumulate, grads, stream);
}

extern "C" int fpde_residual_fwd4(int op, const fpde_grid4* grid, const fpde_coeffs* coeffs,
                                  const float* const* fields, const float* const* consts,
                                  float* const* residual_out, double* loss, void* stream) {
    return fwd_impl(op, grid, coeffs, fields, consts, residual_out, loss, stream);
}

extern "C" int fpde_residual_bwd4(int op, const fpde_grid4* grid, const fpde_coeffs* coeffs,
                                  const float* const* fields, const float* const* consts,
                                  const double* dloss, float* const* grads, void* stream) {
    return bwd_impl(op, grid, coeffs, fields, consts, dloss, grads, stream);
}

extern "C" int fpde_bc_correct4(int op, const fpde_grid4* grid, const fpde_coeffs* coeffs,
                                const float* const* fields, const float* const* consts,
                                const double* dloss, float* const* grads, void* stream) {
    return bc_impl(op, grid, coeffs, fields, consts, dloss, grads, stream);
}

extern "C" int fpde_residual_value_and_grad4(int op, const fpde_grid4* grid,
                                             const fpde_coeffs* coeffs, const float* const* fields,
                                             const float* const* consts, const double* dloss,
                                             double* loss, float* const* grads, void* stream) {
    return value_and_grad_impl(op, grid, coeffs, fields, consts, dloss, loss, grads, stream);
}

extern "C" int fpde_residual_vjp4(int op, const fpde_grid4* grid, const fpde_coeffs* coeffs,
                                  const float* const* fields, const float* const* sens,
                                  int accumulate, float* const* grads, void* stream) {
    return vjp_impl(op, grid, coeffs, fields, sens, accumulate, grads, stream);
}

extern "C" int fpde_residual_fwd_ws4(int op, const fpde_grid4* grid, const fpde_coeffs* coeffs,
                                     const float* const* fields, const float* const* consts,
                                     float* const* residual_out, double* loss, void* workspace,
                                     void* stream) {
    return fwd_impl(op, grid, coeffs, fields, consts, residual_out, loss, stream, true, workspace);
}

extern "C" int fpde_residual_value_and_grad_ws4(int op, const fpde_grid4* grid,
                                                const fpde_coeffs* coeffs,
                                                const float* const* fields,
                                                const float* const* consts, const double* dloss,
                                                double* loss, float* const* grads, void* workspace,
                                                void* stream) {
    return value_and_grad_impl(op, grid, coeffs, fields, consts, dloss, loss, grads, stream, true,
                               workspace);
}

extern "C" const char* fpde_status_string(int status) {
    switch (status) {
    case FPDE_OK: return "FPDE_OK";
    case FPDE_ERR_ARG: return "FPDE_ERR_ARG: null pointer, unknown op or overlapping output";
    case FPDE_ERR_SHAPE: return "FPDE_ERR_SHAPE: wrong rank, n_a < 3 or size too large";
    case FPDE_ERR_SPACING: return "FPDE_ERR_SPACING: grid spacing not positive and finite";
    case FPDE_ERR_COEFF: return "FPDE_ERR_COEFF: non-finite coefficient or dt <= 0";
    case FPDE_ERR_ALIGN: return "FPDE_ERR_ALIGN: misaligned device pointer";
    case FPDE_ERR_HIP: return "FPDE_ERR_HIP: HIP runtime error while queueing work";
    case FPDE_ERR_UNSUPPORTED: return "FPDE_ERR_UNSUPPORTED: request not implemented by this library version";
    default: return "unknown fpde status";
    }
}

extern "C" const char* fpde_version(void) { return "fpde 0.2 gfx950"; }
