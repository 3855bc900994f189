// gfx950 kernels of the quadrature-free DG shallow-water right-hand side.
//
// One thread owns one element.  Per stage it
//   1. rebuilds the element geometry from its three vertices (FP64),
//   2. evaluates the volume term (A, grad phi) of (variational_disc_1) as
//      contractions with the exact basis-product tensors: the flux products
//      are projected onto P^{p-1} with C[m][i][j] and mapped back with the
//      derivative matrix D[k][q][m] (eq. (mass_basis) for the mass row, the
//      same tensor algebra for the momentum rows),
//   3. adds the source (r, phi) of (def_A_h_qf),
//   4. gathers its three edges: traces of both sides in 1D Legendre modes,
//      Lax-Friedrichs flux with the constant-part penalty (eq:lambda), 1D
//      triple products G for the flux products, and the trace matrix R to
//      test against its own basis,
//   5. combines the SSP-RK2 stage and solves u H = q (variational_disc_2) for
//      the new state with the truncated depth expansion K(p,i,j) of
//      Sec. "order separation", by LDL^T in registers.
//
// Coefficients are reference-scaled: c_hat = c / sqrt(|det B_e|), which makes
// every tensor contraction independent of the element size; only the inverse
// Jacobian, the edge normals and |E|/|det B_e| enter.  Terms carrying the
// bathymetry (well-balancing: g xi h_b in the flux, g xi grad h_b in the
// source) are always accumulated in FP64.
//
// Kernel families below: the element-gather stage above (k_stage); the
// shared-flux stage (k_stage_sh, stage_sh_block), where each edge flux
// inside a block of 256 elements is computed once from host-built edge
// items and handed to both sides through LDS; the listed elements of the
// order-separated and order-partitioned schemes (k_corr_all, k_full_all,
// k_epi_all), by teams of four waves per 64 entries or one element per
// thread, with the correction kernel doing the epilogue's join itself when
// it runs after the base pass in one chain; a whole order-partitioned stage
// of a smaller mesh in one launch (k_part_all); the order update
// (k_indicator, k_apply_order); the batch forms of the stage and order
// update; the minimum depth control; the FP64 mass reduction; the caller's
// arrays in and out (k_unpack, k_pack).  A uniform order's whole SSP-RK2 step
// in one launch, built from the same device code, is in swe_step.hip.
#include "swe_device.h"

#include <algorithm>
#include <mutex>
#include <thread>
#include <vector>

namespace swe {
namespace {

template <int P, typename Real, int MODE>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(sh_waves<P, Real>(), 8)))
k_stage_sh(StageArgs<Real> a, const unsigned *items, const int *item_off)
{
    __shared__ ShLds<P, Real> S;
    load_trace_lds<P, Real, false>(S);
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    double xihat = a.xihat, dt = a.dt;
    if (a.inst) {
        // the step's clock stopped (failure): the whole block leaves before its first barrier
        if (step_stopped<P <= 1>(a)) return;
        xihat = MODE == MODE_STAGE2 ? a.inst->xh[1] : a.inst->xh[0];
        dt = a.inst->dt;
    }
    const int i0 = item_off[blk], i1 = item_off[blk + 1];
    stage_sh_block<P, Real, MODE>(S, a, (unsigned)blk * BLOCK, (unsigned)a.m.ne, items + i0, i1 - i0, xihat, dt,
                                  a.flag);
}

// ------------------------------------------------------------ kernels
// Full stage of every element at one order P (unseparated scheme), or, with
// SEP, the base part of the order-separated scheme: every element evaluated
// with its first K(P) modes (P = p_base); elements whose right-hand side also
// has a correction store their partial stage value in Lb for the epilogue.
template <int P, typename Real, int MODE, bool SEP>
__device__ __forceinline__ void stage_element(const StageArgs<Real> &a, unsigned e,
                                              const Real (*sR)[Ord<P>::K][Ord<P>::NT], double xihat,
                                              double dt_stage, int *flag)
{
    constexpr int K = Ord<P>::K;
    if constexpr (SEP) {
        if (a.skip_listed && a.inlist[e]) return;   // a full-order kernel owns this element
    }
    const MeshView &m = a.m;
    const int KS = m.KS, stride = m.stride;
    const unsigned off = e * (unsigned)sizeof(Real);
    const Buf<Real> bC(a.Cin, 3 * KS, stride), bU(a.Uin, 2 * KS, stride);
    const Buf<int> bEv(m.ev, 3, stride), bNb(m.enb, 3, stride);
    Geo G;
    load_geo(m.vtx, bEv, e * 4u, G);
    double hbh[3];
    hb_modes(G, hbh);
    Fields<P, Real> s;
    load_state<P, Real>(bC, bU, KS, off, s);
    const int Ke = (!SEP && a.mixed) ? KOFP[m.ep[e]] : K;

    const double dt = MODE == MODE_RHS ? 1.0 : dt_stage;
    Acc<P, Real> A;
    acc_init<P, Real>(A, s, MODE != MODE_RHS);
    element_rhs<P, P, Real>(a, e, bC, bU, bNb, s, G, hbh, dt, sR, A, xihat);
    if (!SEP && a.mixed) {
        // modes above the element's order stay zero
#pragma unroll
        for (int q = 0; q < K; ++q)
            if (q >= Ke) { A.L[0][q] = 0; A.L[1][q] = 0; A.L[2][q] = 0; }
    }
    if constexpr (MODE == MODE_RHS) {
        const Buf<Real> bL(a.Lout, 3 * KS, stride);
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int q = 0; q < K; ++q) bL.st(j * KS + q, off, A.L[j][q]);
        return;
    } else {
        if constexpr (SEP) {
            if (a.inlist[e]) {
                const Buf<Real> bB(a.Lb, 3 * K, stride);
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int q = 0; q < K; ++q) bB.st(j * K + q, off, A.L[j][q]);
                return;
            }
        }
        finish_stage<P, Real, MODE>(a, e, G, hbh, Ke, A.L, flag);
    }
}

template <int P, typename Real, int MODE, bool SEP>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(waves_target<P, Real>(), 8)))
k_stage(StageArgs<Real> a)
{
    constexpr int K = Ord<P>::K, NT = Ord<P>::NT;
    __shared__ Real sR[3][K][NT];
    load_trace_table<K, NT, Real>(sR);
    __syncthreads();
    const unsigned le = (unsigned)xcd_block(blockIdx.x, gridDim.x) * BLOCK + threadIdx.x;
    if (le >= (unsigned)a.m.ne) return;
    double xihat = a.xihat, dt = a.dt;
    if (a.inst) {
        // the clock of a replayed step lives on the device
        if (step_stopped<SEP && P <= 1>(a)) return;
        xihat = MODE == MODE_STAGE2 ? a.inst->xh[1] : a.inst->xh[0];
        dt = a.inst->dt;
    }
    stage_element<P, Real, MODE, SEP>(a, le + (unsigned)a.e_off, sR, xihat, dt, a.flag);
}

// ------------------------------------------------------------ batched instances
// One launch per order class and stage covers the tiles of every resident
// instance of that order (one tile per block, no loop around the element
// evaluation).  All instances of an order share pooled arrays passed as
// kernel arguments; a tile (TILE consecutive elements of one instance) only
// reads its instance's scalars (step, open-sea elevation, physics, clock).
// Each XCD takes a contiguous eighth of the tile list, so the neighbour
// gathers of an instance's elements stay in one L2.  Instances whose clock
// says they are done are skipped: one step graph serves any resident set.
template <int P, typename Real, int MODE, int TILE>
__global__ void __launch_bounds__(TILE) __attribute__((amdgpu_waves_per_eu(waves_target<P, Real>(), 8)))
k_batch_stage(BatchArgs b)
{
    constexpr int K = Ord<P>::K, NT = Ord<P>::NT;
    __shared__ Real sR[3][K][NT];
    load_trace_table<K, NT, Real>(sR);
    __syncthreads();
    // One tile per block.  XCD x (blocks x, x+8, ...) owns the contiguous
    // eighth [lo, hi) of the tile list; the grid is sized from the tile
    // capacity (at least 8 blocks more than there can be tiles), so every
    // XCD has a block for each of its tiles and the surplus blocks exit.
    const int ntiles = b.ntiles[0];
    const int x = (int)(blockIdx.x & 7u), i = (int)(blockIdx.x >> 3);
    const int lo = (int)(((long long)ntiles * x) >> 3), hi = (int)(((long long)ntiles * (x + 1)) >> 3);
    const int t = lo + i;
    if (t >= hi) return;
    StageArgs<Real> a{};   // every field not set below is zero / null (no lists, no skipping)
    a.m.ne = 0;
    a.m.stride = b.pool.cap;
    a.m.KS = K;
    a.m.vtx = b.vtx;
    a.m.ev = b.pool.ev;
    a.m.enb = b.pool.nb;
    a.m.enbk = b.pool.nbk;
    a.m.ep = nullptr;
    a.Cin = static_cast<const Real *>(MODE == MODE_STAGE1 ? b.pool.C0 : b.pool.C1);
    a.Uin = static_cast<const Real *>(MODE == MODE_STAGE1 ? b.pool.U0 : b.pool.U1);
    a.Cn = static_cast<const Real *>(b.pool.C0);
    a.Cout = static_cast<Real *>(MODE == MODE_STAGE1 ? b.pool.C1 : b.pool.C0);
    a.Uout = static_cast<Real *>(MODE == MODE_STAGE1 ? b.pool.U1 : b.pool.U0);
    a.Lout = nullptr;
    a.src = nullptr;
    const int2 tile = b.tiles[t];
    const InstDesc &I = b.inst[tile.x];
    if (!I.run) return;
    // a member with per-element orders (a static order map or indicator-driven
    // orders) masks each element's modes by its order, as on its own
    a.m.ep = b.pool.ep;
    a.mixed = I.mixed;
    a.ph = I.ph;
    const unsigned e = (unsigned)tile.y + threadIdx.x;
    if (e < (unsigned)(I.first + I.ne))
        stage_element<P, Real, MODE, false>(a, e, sR, MODE == MODE_STAGE1 ? I.xh[0] : I.xh[1], I.dt,
                                            b.flags + tile.x);
}

// Shared-flux stage over the 256-element tiles of every resident instance of
// one order (one tile per block, tile list split by XCD as above).  A tile
// starts on a multiple of 256 within its instance, so the instance's edge
// items of that block (local indices) serve it unchanged.
template <int P, typename Real, int MODE>
__global__ void __launch_bounds__(BLOCK)
__attribute__((amdgpu_waves_per_eu(batch_sh_fp32p3<P, Real>() ? 3 : sh_waves<P, Real>(), 8)))
k_batch_stage_sh(BatchArgs b)
{
    __shared__ ShLds<P, Real> S;
    load_trace_lds<P, Real, false>(S);
    // the returns below are uniform over the block (tile and instance)
    const int ntiles = b.ntiles[0];
    const int x = (int)(blockIdx.x & 7u), i = (int)(blockIdx.x >> 3);
    const int lo = (int)(((long long)ntiles * x) >> 3), hi = (int)(((long long)ntiles * (x + 1)) >> 3);
    const int t = lo + i;
    if (t >= hi) return;
    const int2 tile = b.tiles[t];
    const InstDesc &I = b.inst[tile.x];
    if (!I.run) return;
    StageArgs<Real> a{};   // every field not set below is zero / null (no lists, no skipping)
    a.m.ne = 0;
    a.m.stride = b.pool.cap;
    a.m.KS = Ord<P>::K;
    a.m.vtx = b.vtx;
    a.m.ev = b.pool.ev;
    a.m.enb = b.pool.nb;
    a.m.enbk = b.pool.nbk;
    a.m.ep = nullptr;
    a.Cin = static_cast<const Real *>(MODE == MODE_STAGE1 ? b.pool.C0 : b.pool.C1);
    a.Uin = static_cast<const Real *>(MODE == MODE_STAGE1 ? b.pool.U0 : b.pool.U1);
    a.Cn = static_cast<const Real *>(b.pool.C0);
    a.Cout = static_cast<Real *>(MODE == MODE_STAGE1 ? b.pool.C1 : b.pool.C0);
    a.Uout = static_cast<Real *>(MODE == MODE_STAGE1 ? b.pool.U1 : b.pool.U0);
    a.Lout = nullptr;
    a.src = nullptr;
    a.mixed = 0;
    a.ph = I.ph;
    const unsigned e0 = (unsigned)tile.y;
    // the batch form loads the geometry after the edge pass at every order
    stage_sh_block<P, Real, MODE, false>(S, a, e0, (unsigned)(I.first + I.ne), b.pool.items + 3u * e0,
                                         b.pool.nitems[e0 / BLOCK], MODE == MODE_STAGE1 ? I.xh[0] : I.xh[1], I.dt,
                                         b.flags + tile.x);
}

// Copy an instance's edge items (blocks of 256 elements, item_off[nblk + 1])
// into the pool slots of its element range starting at first (a multiple
// of 256): one block per 256-element block.
__global__ void __launch_bounds__(BLOCK) k_place_items(const unsigned *items, const int *item_off, PoolView pool,
                                                       int first)
{
    const int j = blockIdx.x;
    const int i0 = item_off[j], n = item_off[j + 1] - i0;
    const int f = first + j * BLOCK;
    for (int k = threadIdx.x; k < n; k += BLOCK) pool.items[3 * f + k] = items[i0 + k];
    if (threadIdx.x == 0) pool.nitems[f / BLOCK] = n;
}

__global__ void __launch_bounds__(BLOCK) k_relocate(const int *ev, const int *nb, const unsigned char *nbk,
                                                    const signed char *ep, int ne, int stride, PoolView pool,
                                                    int first, int vbase)
{
    const int e = blockIdx.x * BLOCK + threadIdx.x;
    if (e >= ne) return;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        pool.ev[k * pool.cap + first + e] = ev[k * stride + e] + vbase;
        const int n = nb[k * stride + e];
        pool.nb[k * pool.cap + first + e] = n >= 0 ? n + first : n;
    }
    pool.nbk[first + e] = nbk[e];
    pool.ep[first + e] = ep[e];
}

// Per-step clock of every resident instance: open-sea elevation at the two
// stage times, then advance its time and step budget.
// Open-sea elevation of an instance at time t (its forcing constituents).
__device__ __forceinline__ double clock_xihat(const InstDesc &I, double t)
{
    double x = 0.0;
    for (int c = 0; c < I.ncon; ++c) x += I.amp[c] * sin(I.omega[c] * t + I.phase[c]);
    return x;
}

// The device clock of an instance for the step about to run: a failed
// instance (non-positive depth or a non-finite value) or one whose step
// budget is spent stops; otherwise the open-sea elevation at the step's two
// stage times is set and the time advanced.
__device__ __forceinline__ void clock_advance(const InstDesc &I, int flag, InstDesc &to)
{
    const int run = I.active && I.steps_left > 0 && flag == 0;
    to.ran = I.run;
    to.run = run;
    if (!run) return;
    const int done = I.steps_done + 1, left = I.steps_left - 1;
    const double x0 = clock_xihat(I, I.t), x1 = clock_xihat(I, I.t + I.dt);
    to.xh[0] = x0;
    to.xh[1] = x1;
    to.t = I.t0 + (double)done * I.dt;
    to.steps_done = done;
    to.steps_left = left;
}

// The clock of a step graph's next step, from the current step's: another
// descriptor, so that a kernel which reads the current one may run meanwhile.
// It holds the run's constants already.  Failures of the current step are still
// being found, so those are not looked at (see step_stopped); one that kept the
// current step from running is handed on, after a graph's last step (to null)
// to the run's flag.
__device__ __forceinline__ void next_clock(const InstDesc *from, InstDesc *to, int *flag)
{
    if (threadIdx.x != 0) return;
    if (to) clock_advance(*from, !from->run || from->late, *to);
    if (from->late) *(to ? &to->late : flag) = 1;
}

// Whether the list kernels of orders up to PN hold that code, for one block
// more: order-3 kernels lose scalar registers to it (adaptive tsunami, FP64,
// 18,818 elements, which does not even use it: 45.8 -> 51.8 us a step), and at
// p0-1 (204,800 elements) the step took 47.3 instead of 46.4.
template <int PN>
constexpr bool clock_in_lists()
{
    return PN == 2;
}

__global__ void k_next_clock(InstDesc *from, InstDesc *to, const int *flag)
{
    if (threadIdx.x != 0) return;
    if (to != from) *to = *from;
    clock_advance(*to, flag[0], *to);
    from->late = to->late = 0;
}

__global__ void __launch_bounds__(BLOCK) k_batch_clock(InstDesc *inst, const int *flags, int n, int order)
{
    const int i = blockIdx.x * BLOCK + threadIdx.x;
    if (i >= n || inst[i].order != order) return;
    clock_advance(inst[i], flags[i], inst[i]);
}

// ------------------------------------------------------------ listed elements, every order in one launch
// The kernels of the listed elements take every order in one launch (each
// block runs one order's code; order p's list at a.list + p * lcap, its
// length a.count[p]).  A step graph dispatches its nodes one after another,
// microseconds apart, so one node per stage for all orders ends the stage
// sooner than one node per order.  Block b over the orders lo..PN takes
// order lo + b % (PN - lo + 1) and the (b / (PN - lo + 1))-th run of BLOCK
// list entries (of TEAM entries where a team takes them): the orders are
// interleaved, so the blocks dispatched first hold the heads of every
// order's list.  Lists re-chosen on the device are sized
// for every element and are mostly empty; a block past its list's end leaves
// before it loads anything else (the test is uniform over the block).
template <int PN>
__device__ __forceinline__ int list_order(int lo, int b) { return lo + b % (PN - lo + 1); }
template <int PN>
__device__ __forceinline__ int list_block(int lo, int b) { return b / (PN - lo + 1); }
__device__ __forceinline__ int list_len(const int *count, int p, int lcap)
{
    const int n = count[p];
    return n < lcap ? n : lcap;
}

// Element of entry i of order p's list, or -1 past the list's end.  The
// count is capped at the list's capacity and an entry outside the mesh is
// skipped, so a list is only ever read within its allocation and an entry is
// only ever followed into the element arrays.
template <typename Real>
__device__ __forceinline__ int list_element(const StageArgs<Real> &a, int p, int i, int lcap)
{
    const int n = a.count[p];
    if (i >= (n < lcap ? n : lcap)) return -1;
    const int e = a.list[(size_t)p * (size_t)lcap + (size_t)i];
    return (e >= 0 && e < a.m.ne) ? e : -1;
}

// ---- teams: the listed elements' work shared by the waves of a block
// One thread's evaluation of an order-3 element is thousands of dependent
// instructions, and the few such elements end the stage.  A team block takes
// TEAM list entries, one per lane, and each of its four waves does one part
// of every entry's right-hand side: wave 0 the volume and source terms, wave
// 1 + k the term of local edge k.  Waves 1..3 leave their partial sums in
// LDS; wave 0 adds them in edge order and finishes the element.
// Teams take the short lists (at most TEAM_MAX entries), where the stage
// waits on each element's latency, and every list of a kernel that reaches
// order 3; a long list of a kernel up to order 2 keeps one element per
// thread, which does less work in all.  (One thread per order-3 element needs
// more registers than a lane has, and the one-thread code of the lower orders
// beside the order-3 teams would cost those teams registers.)
constexpr int TEAM = 64;
constexpr int TEAM_ROLES = 4;
constexpr int TEAM_MAX = 16384;

template <int PN>
__device__ __forceinline__ bool list_by_teams(int len) { return PN >= 3 || len <= TEAM_MAX; }

template <int PN, typename Real>
struct TeamLds {
    static constexpr int K = Ord<PN>::K;
    static constexpr bool SPLIT = !std::is_same<Real, double>::value;
    Real L[TEAM_ROLES - 1][3][K][TEAM];
    double W[TEAM_ROLES - 1][SPLIT ? 2 : 1][SPLIT ? K : 1][TEAM];
};

template <int P, int PN, typename Real>
__device__ __forceinline__ void team_put(TeamLds<PN, Real> &X, int role, int lane, const Acc<P, Real> &A)
{
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int q = 0; q < Ord<P>::K; ++q) X.L[role - 1][j][q][lane] = A.L[j][q];
    if constexpr (Acc<P, Real>::SPLIT) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < Ord<P>::K; ++q) X.W[role - 1][j][q][lane] = A.W[j][q];
    }
}

// wave 0's sums plus the edge waves' partial sums, in edge order; the FP64
// bathymetry sums of the FP32 path are added to the momentum rows last
template <int P, int PN, typename Real>
__device__ __forceinline__ void team_sum(const TeamLds<PN, Real> &X, int lane, Acc<P, Real> &A)
{
#pragma unroll
    for (int r = 0; r < TEAM_ROLES - 1; ++r) {
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int q = 0; q < Ord<P>::K; ++q) A.L[j][q] += X.L[r][j][q][lane];
        if constexpr (Acc<P, Real>::SPLIT) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int q = 0; q < Ord<P>::K; ++q) A.W[j][q] += X.W[r][j][q][lane];
        }
    }
    if constexpr (Acc<P, Real>::SPLIT) {
#pragma unroll
        for (int q = 0; q < Ord<P>::K; ++q) {
            A.L[1][q] += Real(A.W[0][q]);
            A.L[2][q] += Real(A.W[1][q]);
        }
    }
}

// acc += dt * (extra right-hand side) (wave 0's part)
template <int P, typename Real>
__device__ __forceinline__ void team_src(const StageArgs<Real> &a, unsigned e, double dt, Acc<P, Real> &A)
{
    if (!a.src) return;
    const Buf<Real> bS(a.src, 3 * a.m.KS, a.m.stride);
    const Real rdt = Real(dt);
    const unsigned off = e * (unsigned)sizeof(Real);
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int q = 0; q < Ord<P>::K; ++q) A.L[j][q] = fma(rdt, bS.ld(j * a.m.KS + q, off), A.L[j][q]);
}

// one wave's part (role) of element e's right-hand side, added to A
template <int P, int PN, typename Real>
__device__ __forceinline__ void team_part(int role, const StageArgs<Real> &a, unsigned e, const Buf<Real> &bC,
                                          const Buf<Real> &bU, const Buf<int> &bNb, const Fields<P, Real> &s,
                                          const Geo &G, const double (&hbh)[3], double dt,
                                          const Real (*sR)[Ord<PN>::K][(P > PN ? P : PN) + 1], double xihat,
                                          Acc<P, Real> &A)
{
    switch (role) {
    case 0:
        volume_term<P, Real>(s, hbh, G, a.ph.g, dt, A);
        source_term<P, Real>(s, G, a.ph, dt, A);
        team_src<P, Real>(a, e, dt, A);
        break;
    case 1: edge_one<P, PN, Real, 0>(a.m, e, bC, bU, bNb, s, G, a.ph.g, xihat, dt, sR, A); break;
    case 2: edge_one<P, PN, Real, 1>(a.m, e, bC, bU, bNb, s, G, a.ph.g, xihat, dt, sR, A); break;
    default: edge_one<P, PN, Real, 2>(a.m, e, bC, bU, bNb, s, G, a.ph.g, xihat, dt, sR, A); break;
    }
}

// full stage of listed element e of order P (order-partitioned scheme), one thread
template <int P, int PN, typename Real, int MODE>
__device__ __forceinline__ void full_element(const StageArgs<Real> &a, unsigned e,
                                             const Real (*sR)[Ord<PN>::K][PN + 1], double xihat, double dt)
{
    const MeshView &m = a.m;
    const int KS = m.KS, stride = m.stride;
    const Buf<Real> bC(a.Cin, 3 * KS, stride), bU(a.Uin, 2 * KS, stride);
    const Buf<int> bEv(m.ev, 3, stride), bNb(m.enb, 3, stride);
    const unsigned off = e * (unsigned)sizeof(Real);
    Geo G;
    load_geo(m.vtx, bEv, e * 4u, G);
    double hbh[3];
    hb_modes(G, hbh);
    Fields<P, Real> s;
    load_state<P, Real>(bC, bU, KS, off, s);
    Acc<P, Real> A;
    acc_init<P, Real>(A, s, true);
    element_rhs<P, PN, Real>(a, e, bC, bU, bNb, s, G, hbh, dt, sR, A, xihat);
    finish_stage<P, Real, MODE>(a, e, G, hbh, Ord<P>::K, A.L, a.flag);
}

// the same by a team; live is false on lanes past the list's end, which only
// meet the barrier
template <int P, int PN, typename Real, int MODE>
__device__ __forceinline__ void full_team(const StageArgs<Real> &a, int le, int role,
                                          const Real (*sR)[Ord<PN>::K][PN + 1], TeamLds<PN, Real> &X,
                                          double xihat, double dt)
{
    const MeshView &m = a.m;
    const int KS = m.KS, stride = m.stride, lane = (int)threadIdx.x % TEAM;
    const bool live = le >= 0;
    const unsigned e = live ? (unsigned)le : 0u;
    const Buf<Real> bC(a.Cin, 3 * KS, stride), bU(a.Uin, 2 * KS, stride);
    const Buf<int> bEv(m.ev, 3, stride), bNb(m.enb, 3, stride);
    Geo G;
    double hbh[3];
    Acc<P, Real> A;
    if (live) {
        load_geo(m.vtx, bEv, e * 4u, G);
        hb_modes(G, hbh);
        Fields<P, Real> s;
        load_state<P, Real>(bC, bU, KS, e * (unsigned)sizeof(Real), s);
        acc_init<P, Real>(A, s, role == 0);
        team_part<P, PN, Real>(role, a, e, bC, bU, bNb, s, G, hbh, dt, sR, xihat, A);
        if (role > 0) team_put<P, PN, Real>(X, role, lane, A);
    }
    __syncthreads();
    if (role == 0 && live) {
        team_sum<P, PN, Real>(X, lane, A);
        finish_stage<P, Real, MODE>(a, e, G, hbh, Ord<P>::K, A.L, a.flag);
    }
}

// block b of the listed elements' full stages (every thread of the block calls it)
template <int PN, typename Real, int MODE>
__device__ __forceinline__ void full_block(const StageArgs<Real> &a, int lo, int lcap, int b,
                                           Real (*sR)[Ord<PN>::K][PN + 1], TeamLds<PN, Real> &X)
{
    constexpr int NX = PN + 1, KN = Ord<PN>::K;
    const int p = list_order<PN>(lo, b), len = list_len(a.count, p, lcap);
    const bool team = list_by_teams<PN>(len);
    int c = list_block<PN>(lo, b);
    if (c * (team ? TEAM : BLOCK) >= len) return;
    double xihat = a.xihat, dt = a.dt;
    if (a.inst) {
        if (step_stopped<clock_in_lists<PN>()>(a)) return;   // the step's clock stopped (failure); uniform over the block
        xihat = MODE == MODE_STAGE2 ? a.inst->xh[1] : a.inst->xh[0];
        dt = a.inst->dt;
    }
    load_trace_table<KN, NX, Real>(sR);
    __syncthreads();
    if (team) {
        // one run per block (the grid covers every run, see list_grid)
        const int role = __builtin_amdgcn_readfirstlane((int)threadIdx.x / TEAM);
        const int le = list_element(a, p, c * TEAM + (int)threadIdx.x % TEAM, lcap);
        switch (p) {
        case 0: full_team<0, PN, Real, MODE>(a, le, role, sR, X, xihat, dt); break;
        case 1: if constexpr (PN >= 1) full_team<1, PN, Real, MODE>(a, le, role, sR, X, xihat, dt); break;
        case 2: if constexpr (PN >= 2) full_team<2, PN, Real, MODE>(a, le, role, sR, X, xihat, dt); break;
        case 3: if constexpr (PN >= 3) full_team<3, PN, Real, MODE>(a, le, role, sR, X, xihat, dt); break;
        }
        return;
    }
    // one element per thread
    if constexpr (PN < 3) {
        const int le = list_element(a, p, c * BLOCK + (int)threadIdx.x, lcap);
        if (le < 0) return;
        const unsigned e = (unsigned)le;
        switch (p) {
        case 0: full_element<0, PN, Real, MODE>(a, e, sR, xihat, dt); break;
        case 1: if constexpr (PN >= 1) full_element<1, PN, Real, MODE>(a, e, sR, xihat, dt); break;
        case 2: if constexpr (PN >= 2) full_element<2, PN, Real, MODE>(a, e, sR, xihat, dt); break;
        }
    }
}

template <int PN, typename Real, int MODE>
__global__ void __launch_bounds__(TEAM * TEAM_ROLES) __attribute__((amdgpu_waves_per_eu(1, 8)))
k_full_all(StageArgs<Real> a, int lo, int lcap)
{
    // beside the base kernel over all elements, these end the stage: their
    // waves issue first on a shared SIMD
    __builtin_amdgcn_s_setprio(2);
    __shared__ Real sR[3][Ord<PN>::K][PN + 1];
    __shared__ TeamLds<PN, Real> X;
    if constexpr (clock_in_lists<PN>() && MODE == MODE_STAGE2) {
        if (a.tick && blockIdx.x == gridDim.x - 1) return next_clock(a.inst, a.next, a.flag);
    }
    full_block<PN, Real, MODE>(a, lo, lcap, (int)blockIdx.x, sR, X);
}

// A whole order-partitioned stage in one launch: the blocks of the lists
// first (the longest), then those of the base pass.  The two share nothing
// within a stage, but two launches of a chain follow each other: on a mesh
// whose base blocks leave most of the chip idle this takes the shorter one
// out of the step (adaptive tsunami, FP64, orders 1-3, 18,818 elements: 63.8
// -> 45.2 us a step; static dam break p1-2, 28,800 elements, FP64 46.5 -> 23.4).
// The base blocks run at the list kernel's registers (one block per CU in
// FP64), so larger meshes keep two launches (131,072 elements: 72.0 against
// 77.5).
template <int B, int PN, typename Real, int MODE>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(1, 8)))
k_part_all(StageArgs<Real> a, int lcap, int nlist, int nsh, int e_end, const unsigned *items, const int *item_off)
{
    union PartLds {
        struct {
            Real sR[3][Ord<PN>::K][PN + 1];
            TeamLds<PN, Real> X;
        } L;
        ShLds<B, Real> S;
    };
    __shared__ PartLds T;
    if ((int)blockIdx.x < nlist) {
        __builtin_amdgcn_s_setprio(2);
        if constexpr (clock_in_lists<PN>() && MODE == MODE_STAGE2) {
            if (a.tick && (int)blockIdx.x == nlist - 1) return next_clock(a.inst, a.next, a.flag);
        }
        full_block<PN, Real, MODE>(a, B, lcap, (int)blockIdx.x, T.L.sR, T.L.X);
        return;
    }
    load_trace_lds<B, Real, false>(T.S);
    const int blk = xcd_block((int)blockIdx.x - nlist, (int)gridDim.x - nlist);
    double xihat = a.xihat, dt = a.dt;
    if (a.inst) {
        if (step_stopped<clock_in_lists<PN>()>(a)) return;   // the step's clock stopped (failure); uniform over the block
        xihat = MODE == MODE_STAGE2 ? a.inst->xh[1] : a.inst->xh[0];
        dt = a.inst->dt;
    }
    if (blk >= nsh) {
        // blocks without edge items (the halo of a grouped numbering)
        __syncthreads();
        const int e = blk * BLOCK + (int)threadIdx.x;
        if (e < e_end) stage_element<B, Real, MODE, true>(a, (unsigned)e, T.S.R, xihat, dt, a.flag);
        return;
    }
    const int i0 = item_off[blk], i1 = item_off[blk + 1];
    stage_sh_block<B, Real, MODE, false>(T.S, a, (unsigned)blk * BLOCK, (unsigned)a.m.ne, items + i0, i1 - i0, xihat, dt,
                                         a.flag);
}

// correction of listed element e of order P (order-separated scheme): dt
// times the full right-hand side, minus dt times the base part (rows below
// K(B), the element's and its neighbours' first K(B) modes) in the rows below
// K(B); the base part is evaluated first and kept, negated, in registers
// dt times the correction of listed element e of order P: its full
// right-hand side minus its base one (rows below K(B); the base part reads
// the element's and its neighbours' first K(B) modes); G and hbh are loaded
template <int P, int B, int PN, typename Real>
SWE_HD void corr_value(const StageArgs<Real> &a, unsigned e, const Real (*sR)[Ord<PN>::K][PN + 1],
                       const Real (*sRb)[Ord<B>::K][Ord<B>::NT], double xihat, double dt, Geo &G,
                       double (&hbh)[3], Real (&C)[3][Ord<P>::K])
{
    constexpr int K = Ord<P>::K, KB = Ord<B>::K;
    const MeshView &m = a.m;
    const int KS = m.KS, stride = m.stride;
    const Buf<Real> bC(a.Cin, 3 * KS, stride), bU(a.Uin, 2 * KS, stride);
    const Buf<int> bEv(m.ev, 3, stride), bNb(m.enb, 3, stride);
    const unsigned off = e * (unsigned)sizeof(Real);
    load_geo(m.vtx, bEv, e * 4u, G);
    hb_modes(G, hbh);
    Real minus_base[3][KB];
    {
        Fields<B, Real> sb;
        load_state<B, Real>(bC, bU, KS, off, sb);
        Acc<B, Real> Ab;
        acc_init<B, Real>(Ab, sb, false);
        element_rhs<B, B, Real>(a, e, bC, bU, bNb, sb, G, hbh, dt, sRb, Ab, xihat);
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int q = 0; q < KB; ++q) minus_base[j][q] = -Ab.L[j][q];
    }
    Fields<P, Real> s;
    load_state<P, Real>(bC, bU, KS, off, s);
    Acc<P, Real> A;
    acc_init<P, Real>(A, s, false);
    element_rhs<P, PN, Real>(a, e, bC, bU, bNb, s, G, hbh, dt, sR, A, xihat);
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int q = 0; q < K; ++q) {
            Real v = A.L[j][q];
            if (q < KB) v += minus_base[j][q];
            C[j][q] = v;
        }
}

// the correction of listed element e stored in Lc (for the epilogue)
template <int P, int B, int PN, typename Real>
SWE_HD void corr_element(const StageArgs<Real> &a, unsigned e,
                                             const Real (*sR)[Ord<PN>::K][PN + 1],
                                             const Real (*sRb)[Ord<B>::K][Ord<B>::NT], double xihat, double dt)
{
    constexpr int K = Ord<P>::K;
    const int KS = a.m.KS, stride = a.m.stride;
    const Buf<Real> bL(a.Lc, 3 * KS, stride);
    const unsigned off = e * (unsigned)sizeof(Real);
    Geo G;
    double hbh[3];
    Real C[3][K];
    corr_value<P, B, PN, Real>(a, e, sR, sRb, xihat, dt, G, hbh, C);
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int q = 0; q < K; ++q) bL.st(j * KS + q, off, C[j][q]);
}

// The epilogue joined into the correction kernel (a.finish set: the base
// pass has run before it, not beside it): stage value = (the base partial
// value in Lb, or c for modes >= K(B)) + the correction C, the same sum the
// epilogue forms, then the listed element's stage finished
template <int P, int B, typename Real>
__device__ __forceinline__ void join_finish(const StageArgs<Real> &a, unsigned e, const Geo &G,
                                            const double (&hbh)[3], Real (&C)[3][Ord<P>::K])
{
    constexpr int K = Ord<P>::K, KB = Ord<B>::K;
    const int KS = a.m.KS, stride = a.m.stride;
    const Buf<Real> bC(a.Cin, 3 * KS, stride), bB(a.Lb, 3 * KB, stride);
    const unsigned off = e * (unsigned)sizeof(Real);
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int q = 0; q < K; ++q) C[j][q] = (q < KB ? bB.ld(j * KB + q, off) : bC.ld(j * KS + q, off)) + C[j][q];
    if (a.finish == MODE_STAGE2)
        finish_stage<P, Real, MODE_STAGE2>(a, e, G, hbh, K, C, a.flag);
    else
        finish_stage<P, Real, MODE_STAGE1>(a, e, G, hbh, K, C, a.flag);
}

// correction of listed element e of order P by a team: each wave's part of
// the full right-hand side minus its part of the base one (rows below K(B);
// the base part reads the element's and its neighbours' first K(B) modes),
// summed by wave 0, which stores dt times the correction
template <int P, int B, int PN, typename Real>
__device__ __forceinline__ void corr_team(const StageArgs<Real> &a, int le, int role,
                                          const Real (*sR)[Ord<PN>::K][PN + 1],
                                          const Real (*sRb)[Ord<B>::K][Ord<B>::NT], TeamLds<PN, Real> &X,
                                          double xihat, double dt)
{
    constexpr int K = Ord<P>::K, KB = Ord<B>::K;
    const MeshView &m = a.m;
    const int KS = m.KS, stride = m.stride, lane = (int)threadIdx.x % TEAM;
    const bool live = le >= 0;
    const unsigned e = live ? (unsigned)le : 0u;
    const unsigned off = e * (unsigned)sizeof(Real);
    const Buf<Real> bC(a.Cin, 3 * KS, stride), bU(a.Uin, 2 * KS, stride);
    const Buf<int> bEv(m.ev, 3, stride), bNb(m.enb, 3, stride);
    Acc<P, Real> A;
    Geo G;
    double hbh[3];
    // wave 0 of a kernel that finishes the stage (a.finish) fetches what the
    // join needs before its volume work, so the loads overlap it: the base
    // part (c itself above K(B)) and, in the second stage, c^n
    const bool join = role == 0 && a.finish;
    Real Jb[3][K], Jn[3][K];
    if (live) {
        load_geo(m.vtx, bEv, e * 4u, G);
        hb_modes(G, hbh);
        Fields<P, Real> s;
        load_state<P, Real>(bC, bU, KS, off, s);
        if (join) {
            const Buf<Real> bB(a.Lb, 3 * KB, stride), bN(a.Cn, 3 * KS, stride);
#pragma unroll
            for (int q = 0; q < K; ++q) {
                Jb[0][q] = q < KB ? bB.ld(0 * KB + q, off) : s.xi[q];
                Jb[1][q] = q < KB ? bB.ld(1 * KB + q, off) : s.U[q];
                Jb[2][q] = q < KB ? bB.ld(2 * KB + q, off) : s.V[q];
            }
            if (a.finish == MODE_STAGE2) {
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int q = 0; q < K; ++q) Jn[j][q] = bN.ld(j * KS + q, off);
            }
        }
        {
            Fields<B, Real> sb;
#pragma unroll
            for (int q = 0; q < KB; ++q) {
                sb.xi[q] = s.xi[q]; sb.U[q] = s.U[q]; sb.V[q] = s.V[q]; sb.u[q] = s.u[q]; sb.v[q] = s.v[q];
            }
            Acc<B, Real> Ab;
            acc_init<B, Real>(Ab, sb, false);
            team_part<B, B, Real>(role, a, e, bC, bU, bNb, sb, G, hbh, dt, sRb, xihat, Ab);
            acc_init<P, Real>(A, s, false);
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int q = 0; q < KB; ++q) A.L[j][q] = -Ab.L[j][q];
            if constexpr (Acc<P, Real>::SPLIT) {
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int q = 0; q < KB; ++q) A.W[j][q] = -Ab.W[j][q];
            }
        }
        team_part<P, PN, Real>(role, a, e, bC, bU, bNb, s, G, hbh, dt, sR, xihat, A);
        if (role > 0) team_put<P, PN, Real>(X, role, lane, A);
    }
    __syncthreads();
    if (role == 0 && live) {
        team_sum<P, PN, Real>(X, lane, A);
        if (join) {
            // the epilogue's sum and, in the second stage, the RK combine, in
            // the expressions of join_finish and finish_stage (bit for bit)
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int q = 0; q < K; ++q) A.L[j][q] = Jb[j][q] + A.L[j][q];
            if (a.finish == MODE_STAGE2) {
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int q = 0; q < K; ++q) A.L[j][q] = Real(0.5) * Jn[j][q] + Real(0.5) * A.L[j][q];
            }
            finish_stage<P, Real, MODE_STAGE1>(a, e, G, hbh, K, A.L, a.flag);
            return;
        }
        const Buf<Real> bL(a.Lc, 3 * KS, stride);
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int q = 0; q < K; ++q) bL.st(j * KS + q, off, A.L[j][q]);
    }
}

// correction of listed element e by one thread: stored for the epilogue, or
// joined with the base part and the stage finished (a.finish)
template <int P, int B, int PN, typename Real>
__device__ __forceinline__ void corr_thread(const StageArgs<Real> &a, unsigned e,
                                            const Real (*sR)[Ord<PN>::K][PN + 1],
                                            const Real (*sRb)[Ord<B>::K][Ord<B>::NT], double xihat, double dt)
{
    if (!a.finish) {
        corr_element<P, B, PN, Real>(a, e, sR, sRb, xihat, dt);
        return;
    }
    Geo G;
    double hbh[3];
    Real C[3][Ord<P>::K];
    corr_value<P, B, PN, Real>(a, e, sR, sRb, xihat, dt, G, hbh, C);
    join_finish<P, B, Real>(a, e, G, hbh, C);
}

template <int B, int PN, typename Real>
__global__ void __launch_bounds__(TEAM * TEAM_ROLES) __attribute__((amdgpu_waves_per_eu(1, 8)))
k_corr_all(StageArgs<Real> a, double dt, int lcap)
{
    __builtin_amdgcn_s_setprio(2);   // as in k_full_all
    constexpr int KB = Ord<B>::K, NTB = Ord<B>::NT;
    constexpr int KN = Ord<PN>::K, NX = PN + 1;
    __shared__ Real sR[3][KN][NX];
    __shared__ Real sRb[3][KB][NTB];
    __shared__ TeamLds<PN, Real> X;
    const int p = list_order<PN>(B, (int)blockIdx.x), len = list_len(a.count, p, lcap);
    const bool team = list_by_teams<PN>(len);
    int c = list_block<PN>(B, (int)blockIdx.x);
    if (c * (team ? TEAM : BLOCK) >= len) return;
    double xihat = a.xihat;
    if (a.inst) {
        // the clock of a replayed step lives on the device
        if (!a.inst->run) return;   // the step's clock stopped (failure); uniform over the block
        xihat = a.inst->xh[a.stage];
        dt = a.inst->dt;
    }
    load_trace_table<KN, NX, Real>(sR);
    load_trace_table<KB, NTB, Real>(sRb);
    __syncthreads();
    if (team) {   // as in k_full_all
        const int role = __builtin_amdgcn_readfirstlane((int)threadIdx.x / TEAM);
        const int le = list_element(a, p, c * TEAM + (int)threadIdx.x % TEAM, lcap);
        switch (p) {
        case 0: if constexpr (B <= 0) corr_team<0, B, PN, Real>(a, le, role, sR, sRb, X, xihat, dt); break;
        case 1: if constexpr (B <= 1 && PN >= 1) corr_team<1, B, PN, Real>(a, le, role, sR, sRb, X, xihat, dt); break;
        case 2: if constexpr (B <= 2 && PN >= 2) corr_team<2, B, PN, Real>(a, le, role, sR, sRb, X, xihat, dt); break;
        case 3: if constexpr (B <= 3 && PN >= 3) corr_team<3, B, PN, Real>(a, le, role, sR, sRb, X, xihat, dt); break;
        }
        return;
    }
    if constexpr (PN < 3) {
        const int le = list_element(a, p, c * BLOCK + (int)threadIdx.x, lcap);
        if (le < 0) return;
        const unsigned e = (unsigned)le;
        switch (p) {
        case 0: if constexpr (B <= 0) corr_thread<0, B, PN, Real>(a, e, sR, sRb, xihat, dt); break;
        case 1: if constexpr (B <= 1 && PN >= 1) corr_thread<1, B, PN, Real>(a, e, sR, sRb, xihat, dt); break;
        case 2: if constexpr (B <= 2 && PN >= 2) corr_thread<2, B, PN, Real>(a, e, sR, sRb, xihat, dt); break;
        }
    }
}

// The same correction on the host (the heterogeneous stage): the listed
// elements [e0, e1) of every order, split over nthreads CPU threads; the
// arguments point at host copies of the mesh and of the stage's input state,
// and the correction goes to a host copy of Lc.
template <int B, int PN, typename Real>
void host_corr_t(const StageArgs<Real> &a, double dt, const signed char *order, int e0, int e1, int nthreads)
{
    constexpr int KN = Ord<PN>::K, NX = PN + 1, KB = Ord<B>::K, NTB = Ord<B>::NT;
    Real sR[3][KN][NX], sRb[3][KB][NTB];
    for (int k = 0; k < 3; ++k) {
        for (int n = 0; n < KN; ++n)
            for (int c = 0; c < NX; ++c) sR[k][n][c] = Real(TR[k][n][c]);
        for (int n = 0; n < KB; ++n)
            for (int c = 0; c < NTB; ++c) sRb[k][n][c] = Real(TR[k][n][c]);
    }
    auto work = [&](int lo, int hi) {
        for (int e = lo; e < hi; ++e) {
            const unsigned ue = (unsigned)e;
            switch (order[e]) {
            case 0: if constexpr (B <= 0) corr_element<0, B, PN, Real>(a, ue, sR, sRb, a.xihat, dt); break;
            case 1: if constexpr (B <= 1 && PN >= 1) corr_element<1, B, PN, Real>(a, ue, sR, sRb, a.xihat, dt); break;
            case 2: if constexpr (B <= 2 && PN >= 2) corr_element<2, B, PN, Real>(a, ue, sR, sRb, a.xihat, dt); break;
            case 3: if constexpr (B <= 3 && PN >= 3) corr_element<3, B, PN, Real>(a, ue, sR, sRb, a.xihat, dt); break;
            }
        }
    };
    const int n = e1 - e0;
    if (n <= 0) return;
    const int nt = std::max(1, std::min(nthreads, (n + 63) / 64));
    std::vector<std::thread> pool;
    for (int t = 1; t < nt; ++t)
        pool.emplace_back(work, e0 + (int)((int64_t)n * t / nt), e0 + (int)((int64_t)n * (t + 1) / nt));
    work(e0, e0 + (int)((int64_t)n / nt));
    for (auto &th : pool) th.join();
}

// epilogue of listed element e of order P (order-separated scheme): stage
// value = (base partial value, or c for modes >= K(B)) + correction
template <int P, typename Real, int MODE>
__device__ __forceinline__ void epi_element(const StageArgs<Real> &a, unsigned e, int KB)
{
    constexpr int K = Ord<P>::K;
    const MeshView &m = a.m;
    const int KS = m.KS, stride = m.stride;
    const Buf<Real> bC(a.Cin, 3 * KS, stride), bL(a.Lc, 3 * KS, stride), bB(a.Lb, 3 * KB, stride);
    const Buf<int> bEv(m.ev, 3, stride);
    const unsigned off = e * (unsigned)sizeof(Real);
    Geo G;
#pragma unroll
    for (int v = 0; v < 3; ++v) G.h[v] = m.vtx[(unsigned)bEv.ld(v, e * 4u)].z;
    double hbh[3];
    hb_modes(G, hbh);
    Real L[3][K];
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int q = 0; q < K; ++q)
            L[j][q] = (q < KB ? bB.ld(j * KB + q, off) : bC.ld(j * KS + q, off)) + bL.ld(j * KS + q, off);
    finish_stage<P, Real, MODE>(a, e, G, hbh, K, L, a.flag);
}

template <int PN, typename Real, int MODE>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(1, 8)))
k_epi_all(StageArgs<Real> a, int KB, int lo, int lcap)
{
    const int p = list_order<PN>(lo, (int)blockIdx.x), first = list_block<PN>(lo, (int)blockIdx.x) * BLOCK;
    if (first >= list_len(a.count, p, lcap)) return;
    const int le = list_element(a, p, first + (int)threadIdx.x, lcap);
    if (le < 0) return;
    const unsigned e = (unsigned)le;
    if (a.inst && !a.inst->run) return;   // the step's clock stopped (failure)
    switch (p) {
    case 0: epi_element<0, Real, MODE>(a, e, KB); break;
    case 1: if constexpr (PN >= 1) epi_element<1, Real, MODE>(a, e, KB); break;
    case 2: if constexpr (PN >= 2) epi_element<2, Real, MODE>(a, e, KB); break;
    case 3: if constexpr (PN >= 3) epi_element<3, Real, MODE>(a, e, KB); break;
    }
}

// ------------------------------------------------------------ p-adaptivity
// Indicator (stand-in for the paper's JRL indicator, which its text only
// cites): the largest jump of the P1 part of xi at the edge midpoints; land
// edges contribute 0, open edges compare with xi_hat(t).  New order: p_hi if
// I >= tau, one less for each further factor 10 below tau, never below p_lo.
template <typename Real>
__device__ __forceinline__ void indicator_element(const MeshView &m, const Buf<Real> &bC, unsigned e, double xihat,
                                                  double tau, int p_lo, int p_hi, double *I_out, signed char *p_new)
{
    const Buf<int> bNb(m.enb, 3, m.stride);
    const unsigned off = e * (unsigned)sizeof(Real);
    const double x0 = bC.ld(0, off), x1 = bC.ld(1, off), x2 = bC.ld(2, off);
    const unsigned nbk_all = m.enbk[e];
    double I = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double own = TPMID[k][0] * x0 + TPMID[k][1] * x1 + TPMID[k][2] * x2;
        const int nb = bNb.ld(k, e * 4u);
        double other = own;
        if (nb >= 0) {
            const int kk = (nbk_all >> (2 * k)) & 3;
            const unsigned on = (unsigned)nb * (unsigned)sizeof(Real);
            const double y0 = bC.ld(0, on), y1 = bC.ld(1, on), y2 = bC.ld(2, on);
            other = TPMID[kk][0] * y0 + TPMID[kk][1] * y1 + TPMID[kk][2] * y2;
        } else if (nb == NB_OPEN) {
            other = xihat;
        }
        const double j = fabs(own - other);
        I = j > I ? j : I;
    }
    if (I_out) I_out[e] = I;
    if (p_new) {
        int pn = p_lo;
        double thr = tau;
        for (int pp = p_hi; pp > p_lo; --pp) {
            if (I >= thr) { pn = pp; break; }
            thr *= 0.1;
        }
        p_new[e] = (signed char)pn;
    }
}

template <typename Real>
__global__ void __launch_bounds__(BLOCK) k_indicator(StageArgs<Real> a, double tau, int p_lo, int p_hi,
                                                     double *I_out, signed char *p_new)
{
    const MeshView &m = a.m;
    if (a.cntw && blockIdx.x == 0 && threadIdx.x < 4) a.cntw[threadIdx.x] = 0;   // list counts of the next pass
    const unsigned e = blockIdx.x * BLOCK + threadIdx.x;
    if (e >= (unsigned)m.ne) return;
    const Buf<Real> bC(a.Cin, 3 * m.KS, m.stride);
    // in a step graph the clock advances in the order update after this
    // kernel, so the step's start time is still the clock's time
    indicator_element<Real>(m, bC, e, a.inst ? clock_xihat(*a.inst, a.inst->t) : a.xihat, tau, p_lo, p_hi, I_out,
                            p_new);
}

// Whether element e's right-hand side has a correction: its new order or a
// neighbour's is above p_base.
__device__ __forceinline__ bool listed_element(const MeshView &m, unsigned e, int pn, const signed char *p_new,
                                               int p_base)
{
    const Buf<int> bNb(m.enb, 3, m.stride);
    bool l = pn > p_base;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int nb = bNb.ld(k, e * 4u);
        if (nb >= 0 && p_new[nb] > p_base) l = true;
    }
    return l;
}

// Apply the new order pn of element e: if it differs from the current one,
// drop modes above K(pn) from every state buffer and re-solve u.
template <int PM, typename Real>
__device__ __forceinline__ void apply_element(const StageArgs<Real> &a, unsigned e, int pn, signed char *p_cur)
{
    constexpr int K = Ord<PM>::K;
    const MeshView &m = a.m;
    const int KS = m.KS, stride = m.stride;
    const unsigned off = e * (unsigned)sizeof(Real);
    if (pn == p_cur[e]) return;
    const int Kn = KOFP[pn];
    Buf<Real> b0(a.Cout, 3 * KS, stride), b1(a.Calt, 3 * KS, stride);
    Buf<Real> u1(a.Ualt, 2 * KS, stride);
    Real xi[K], U[K], V[K];
#pragma unroll
    for (int q = 0; q < K; ++q) {
        const bool keep = q < Kn;
        xi[q] = keep ? b0.ld(0 * KS + q, off) : Real(0);
        U[q] = keep ? b0.ld(1 * KS + q, off) : Real(0);
        V[q] = keep ? b0.ld(2 * KS + q, off) : Real(0);
        if (!keep) {
#pragma unroll
            for (int j = 0; j < 3; ++j) { b0.st(j * KS + q, off, Real(0)); b1.st(j * KS + q, off, Real(0)); }
            u1.st(0 * KS + q, off, Real(0));
            u1.st(1 * KS + q, off, Real(0));
        }
    }
    Geo G;
#pragma unroll
    for (int v = 0; v < 3; ++v) G.h[v] = m.vtx[(unsigned)Buf<int>(m.ev, 3, stride).ld(v, e * 4u)].z;
    double hbh[3];
    hb_modes(G, hbh);
    Real u[K], v[K];
    solve_u<PM, Real>(xi, U, V, hbh, Kn, u, v);
    Buf<Real> bu(a.Uout, 2 * KS, stride);
#pragma unroll
    for (int q = 0; q < K; ++q) {
        bu.st(0 * KS + q, off, u[q]);
        bu.st(1 * KS + q, off, v[q]);
    }
    p_cur[e] = (signed char)pn;
}

// Apply the new orders of a context's elements, flag elements that need a
// correction and append them to the list of their order.  The lists come
// first, so that their atomics are under way while the few elements whose
// order changed are solved again, and a block takes its places in every list
// with one atomic each: with one per wave, some 2,000 to 6,000 atomics on one
// cache line held up a 131,072-element update (a tsunami step of 131,072 elements, FP32, 63.2 -> 61.2 us).
template <int PM, typename Real>
__global__ void __launch_bounds__(BLOCK) k_apply_order(StageArgs<Real> a, const signed char *p_new,
                                                       signed char *p_cur, int p_base, int lcap, InstDesc *clock,
                                                       const int *flag)
{
    __shared__ int cnt[4][BLOCK / 64];   // listed elements of an order in each wave, then where they go
    const unsigned e = blockIdx.x * BLOCK + threadIdx.x;
    // a step graph's clock (no other thread of this kernel reads the instance)
    if (clock && e == 0) clock_advance(*clock, flag[0], *clock);
    const bool live = e < (unsigned)a.m.ne;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int pn = 0;
    bool listed = false;
    if (live) {
        pn = p_new[e];
        listed = listed_element(a.m, e, pn, p_new, p_base);
        a.inlist[e] = listed ? 1 : 0;
    }
    int rank = 0;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const bool mine = listed && pn == p;
        const unsigned long long mask = __ballot(mine);
        if (mine) rank = __popcll(mask & ((1ull << lane) - 1ull));
        if (lane == 0) cnt[p][wave] = __popcll(mask);
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        int n = 0;
        for (int w = 0; w < BLOCK / 64; ++w) n += cnt[threadIdx.x][w];
        int base = n ? atomicAdd(&a.cntw[threadIdx.x], n) : 0;
        for (int w = 0; w < BLOCK / 64; ++w) {
            const int k = cnt[threadIdx.x][w];
            cnt[threadIdx.x][w] = base;
            base += k;
        }
    }
    if (live) apply_element<PM, Real>(a, e, pn, p_cur);
    __syncthreads();
    if (listed) {
        // at < lcap: each element is appended at most once per update
        const int at = cnt[pn][wave] + rank;
        if (at < lcap) a.listw[(size_t)pn * (size_t)lcap + (size_t)at] = (int)e;
    }
}

// The order update of the indicator-driven members of a batch, over 256-element
// tiles of their pool (every such member runs the fused scheme: its elements'
// own orders mask the stage, no lists).  Tile lists and instance scalars as
// for the batch stage kernels; instances whose clock stopped are skipped.
template <typename Real>
__global__ void __launch_bounds__(BLOCK) k_batch_indicator(BatchArgs b)
{
    const int nt = b.natiles[0];
    const int x = (int)(blockIdx.x & 7u), i = (int)(blockIdx.x >> 3);
    const int lo = (int)(((long long)nt * x) >> 3), hi = (int)(((long long)nt * (x + 1)) >> 3);
    const int t = lo + i;
    if (t >= hi) return;
    const int2 tile = b.atiles[t];
    const InstDesc &I = b.inst[tile.x];
    if (!I.run) return;
    const unsigned e = (unsigned)tile.y + threadIdx.x;
    if (e >= (unsigned)(I.first + I.ne)) return;
    MeshView m{};
    m.stride = b.pool.cap;
    m.KS = (I.order + 1) * (I.order + 2) / 2;
    m.vtx = b.vtx;
    m.ev = b.pool.ev;
    m.enb = b.pool.nb;
    m.enbk = b.pool.nbk;
    const Buf<Real> bC(static_cast<const Real *>(b.pool.C0), 3 * m.KS, m.stride);
    indicator_element<Real>(m, bC, e, I.xh[0], I.tau, I.p_lo, I.order, nullptr, b.pool.pnew);
}

template <int PM, typename Real>
__global__ void __launch_bounds__(BLOCK) k_batch_apply(BatchArgs b)
{
    const int nt = b.natiles[0];
    const int x = (int)(blockIdx.x & 7u), i = (int)(blockIdx.x >> 3);
    const int lo = (int)(((long long)nt * x) >> 3), hi = (int)(((long long)nt * (x + 1)) >> 3);
    const int t = lo + i;
    if (t >= hi) return;
    const int2 tile = b.atiles[t];
    const InstDesc &I = b.inst[tile.x];
    if (!I.run) return;
    const unsigned e = (unsigned)tile.y + threadIdx.x;
    if (e >= (unsigned)(I.first + I.ne)) return;
    StageArgs<Real> a{};   // no lists: the fused scheme masks by the elements' own orders
    a.m.stride = b.pool.cap;
    a.m.KS = Ord<PM>::K;
    a.m.vtx = b.vtx;
    a.m.ev = b.pool.ev;
    a.m.enb = b.pool.nb;
    a.m.enbk = b.pool.nbk;
    a.Cout = static_cast<Real *>(b.pool.C0);
    a.Calt = static_cast<Real *>(b.pool.C1);
    a.Uout = static_cast<Real *>(b.pool.U0);
    a.Ualt = static_cast<Real *>(b.pool.U1);
    apply_element<PM, Real>(a, e, b.pool.pnew[e], b.pool.ep);
}

// ------------------------------------------------------------ minimum depth control
// After a stage (the paper's minimum depth control, a kernel of its code that
// it does not define; this is the reading): an element whose total depth
// H = xi + h_b is below h_min at one of its vertices or edge midpoints has the
// deviation of H from its element mean scaled by
//   theta = (mean H - h_min) / (mean H - min H)   (0 when mean H <= h_min),
// keeping the mean (the mass), and the momentum's deviation from its mean is
// scaled by the same theta.  h_b is fixed, so xi takes the scaled deviation
// of H minus that of h_b (its modes 1 and 2).  The element's velocity is then
// solved again.  Order-0 elements have no mode to scale.
template <int PM, typename Real>
__global__ void __launch_bounds__(BLOCK) k_depth_limit(StageArgs<Real> a, double h_min)
{
    constexpr int K = Ord<PM>::K;
    const MeshView &m = a.m;
    const unsigned e = blockIdx.x * BLOCK + threadIdx.x;
    if (e >= (unsigned)m.ne) return;
    if (a.inst && step_stopped<true>(a)) return;   // the step's clock stopped (failure)
    const int p = m.ep ? (int)m.ep[e] : PM;
    if (p < 1) return;
    const int Ke = KOFP[p];
    const int KS = m.KS, stride = m.stride;
    const unsigned off = e * (unsigned)sizeof(Real);
    const Buf<Real> bC(a.Cout, 3 * KS, stride);
    Geo G;
#pragma unroll
    for (int v = 0; v < 3; ++v) G.h[v] = m.vtx[(unsigned)Buf<int>(m.ev, 3, stride).ld(v, e * 4u)].z;
    Real xi[K];
#pragma unroll
    for (int q = 0; q < K; ++q) xi[q] = q < Ke ? bC.ld(q, off) : Real(0);
    const double hbm = (G.h[0] + G.h[1] + G.h[2]) * (1.0 / 3.0);
    const double Hm = SQRT2 * double(xi[0]) + hbm;
    // check points: vertex j < 3, the midpoint of edge j - 3 (it joins
    // vertices j - 2 and j - 1, modulo 3) for j >= 3
    double Hlow = HUGE_VAL;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        double x = 0.0;
#pragma unroll
        for (int q = 0; q < K; ++q) x = fma(TCHK[j][q], double(xi[q]), x);
        const double hb = j < 3 ? G.h[j] : 0.5 * (G.h[(j - 2) % 3] + G.h[(j - 1) % 3]);
        Hlow = fmin(Hlow, x + hb);
    }
    if (!(Hlow < h_min)) return;
    const double theta = Hm > h_min ? (Hm - h_min) / (Hm - Hlow) : 0.0;
    double hbh[3];
    hb_modes(G, hbh);
    const Buf<Real> bU(a.Uout, 2 * KS, stride);
    Real U[K], V[K];
#pragma unroll
    for (int q = 0; q < K; ++q) {
        U[q] = q < Ke ? bC.ld(KS + q, off) : Real(0);
        V[q] = q < Ke ? bC.ld(2 * KS + q, off) : Real(0);
    }
#pragma unroll
    for (int q = 1; q < K; ++q) {
        if (q >= Ke) continue;
        xi[q] = Real(q < 3 ? theta * double(xi[q]) + (theta - 1.0) * hbh[q] : theta * double(xi[q]));
        U[q] = Real(theta * double(U[q]));
        V[q] = Real(theta * double(V[q]));
        bC.st(q, off, xi[q]);
        bC.st(KS + q, off, U[q]);
        bC.st(2 * KS + q, off, V[q]);
    }
    Real u[K], v[K];
    solve_u<PM, Real>(xi, U, V, hbh, Ke, u, v);
#pragma unroll
    for (int q = 0; q < K; ++q) {
        if (q >= Ke) continue;
        bU.st(q, off, u[q]);
        bU.st(KS + q, off, v[q]);
    }
}

template <int P, typename Real>
__global__ void __launch_bounds__(BLOCK) k_usolve(StageArgs<Real> a)
{
    constexpr int K = Ord<P>::K;
    const int e = blockIdx.x * BLOCK + threadIdx.x;
    const MeshView &m = a.m;
    if (e >= m.ne) return;
    const int KS = m.KS, stride = m.stride;
    Geo G;
#pragma unroll
    for (int v = 0; v < 3; ++v) G.h[v] = m.vtx[m.ev[v * stride + e]].z;
    double hbh[3];
    hb_modes(G, hbh);
    const int Ke = a.mixed ? KOFP[m.ep[e]] : K;
    Real xi[K], U[K], V[K], u[K], v[K];
#pragma unroll
    for (int q = 0; q < K; ++q) {
        xi[q] = a.Cin[(0 * KS + q) * stride + e];
        U[q] = a.Cin[(1 * KS + q) * stride + e];
        V[q] = a.Cin[(2 * KS + q) * stride + e];
    }
    solve_u<P, Real>(xi, U, V, hbh, Ke, u, v);
#pragma unroll
    for (int q = 0; q < K; ++q) {
        a.Uout[(0 * KS + q) * stride + e] = u[q];
        a.Uout[(1 * KS + q) * stride + e] = v[q];
    }
}

// ------------------------------------------------------------ state in and out
// The caller's coefficients [element][component][mode] (physical basis, FP64,
// caller's element order) and the device's reference-scaled [slot][stride]
// arrays.  A block takes XFER caller elements: its first threads find each
// one's storage index and scale factor sqrt(|det B_e|), then all threads run
// over the XFER * nslots values, so the caller's side is read and written in
// whole cache lines and the device side in the short runs the element
// ordering gives.  The determinant is formed product by product (no
// contraction), so the factor is the host's bit for bit.  Bound by the
// transfer over the host link that follows or precedes it; doing this on the
// host's one thread instead took 27.5 ms of a 524,288-element FP32 p = 2
// read-back (pass of 500 steps and a read-back: 82.0 ms, now 54.9).
constexpr int XFER = 64;

__device__ __forceinline__ double scale_of(const double4 *vtx, const int *ev, int evs, int i)
{
    const double4 a = vtx[(unsigned)ev[i]], b = vtx[(unsigned)ev[evs + i]], d = vtx[(unsigned)ev[2 * evs + i]];
    const double p0 = (b.x - a.x) * (d.y - a.y);
    const double p1 = (d.x - a.x) * (b.y - a.y);
    const double det = p0 - p1;
    return sqrt(det);
}

template <typename Real>
__global__ void __launch_bounds__(BLOCK) k_pack(const Real *src, int stride, int first, int nslots, const int *iperm,
                                                const double4 *vtx, const int *ev, int evs, int u0, int u1,
                                                double *out)
{
    __shared__ double sf[XFER];
    __shared__ int at[XFER];
    const int ub = u0 + (int)blockIdx.x * XFER;
    const int n = u1 - ub < XFER ? u1 - ub : XFER;
    if ((int)threadIdx.x < n) {
        const int i = iperm[ub + (int)threadIdx.x];
        at[threadIdx.x] = first + i;
        sf[threadIdx.x] = scale_of(vtx, ev, evs, i);
    }
    __syncthreads();
    double *o = out + (size_t)(ub - u0) * (size_t)nslots;
    for (int k = threadIdx.x; k < n * nslots; k += BLOCK) {
        const int el = k / nslots, s = k - el * nslots;
        o[k] = double(src[(size_t)s * (size_t)stride + (size_t)at[el]]) * sf[el];
    }
}

// bad[0] is set on a non-finite value of a kept mode (modes at or above
// K(p_e) are stored as zero and not looked at)
template <typename Real>
__global__ void __launch_bounds__(BLOCK) k_unpack(const double *in, int K, const int *iperm, const double4 *vtx,
                                                  const int *ev, int evs, const signed char *ep, int u0, int u1,
                                                  Real *dst, int stride, int *bad)
{
    __shared__ double inv[XFER];
    __shared__ int at[XFER], keep[XFER];
    const int ub = u0 + (int)blockIdx.x * XFER;
    const int n = u1 - ub < XFER ? u1 - ub : XFER;
    if ((int)threadIdx.x < n) {
        const int i = iperm[ub + (int)threadIdx.x];
        at[threadIdx.x] = i;
        inv[threadIdx.x] = 1.0 / scale_of(vtx, ev, evs, i);
        keep[threadIdx.x] = KOFP[ep[i] & 3];
    }
    __syncthreads();
    const double *v = in + (size_t)(ub - u0) * (size_t)(3 * K);
    bool wrong = false;
    for (int k = threadIdx.x; k < n * 3 * K; k += BLOCK) {
        const int el = k / (3 * K), s = k - el * 3 * K;
        const double x = s % K < keep[el] ? v[k] : 0.0;
        wrong = wrong || !isfinite(x);
        dst[(size_t)s * (size_t)stride + (size_t)at[el]] = Real(x * inv[el]);
    }
    if (wrong) bad[0] = 1;
}

// Mass: sum_e int xi = sum_e xi_hat_0 |det B_e| / sqrt(2), fixed-order tree.
template <typename Real>
__global__ void __launch_bounds__(BLOCK) k_mass_partial(MeshView m, const Real *C, double *partial)
{
    __shared__ double red[BLOCK];
    const int e = blockIdx.x * BLOCK + threadIdx.x;
    double v = 0.0;
    if (e < m.ne) {
        Geo G;
        load_geo(m.vtx, Buf<int>(m.ev, 3, m.stride), (unsigned)e * 4u, G);
        v = double(C[e]) * G.det * (1.0 / SQRT2);
    }
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = BLOCK / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(BLOCK) k_mass_final(const double *partial, int n, double *out)
{
    __shared__ double red[BLOCK];
    double v = 0.0;
    for (int i = threadIdx.x; i < n; i += BLOCK) v += partial[i];
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = BLOCK / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = red[0];
}

template <int P, typename Real, bool SEP>
hipError_t stage_p(int mode, const void *args, Sink &s)
{
    StageArgs<Real> a = *static_cast<const StageArgs<Real> *>(args);
    if (a.m.ne <= 0) return hipSuccess;
    const int nb = (a.m.ne + BLOCK - 1) / BLOCK;
    const dim3 grid(a.blocks > 0 && a.blocks < nb ? a.blocks : nb), block(BLOCK);
    void *kargs[] = {&a};
    const void *fn = mode == MODE_RHS      ? reinterpret_cast<const void *>(&k_stage<P, Real, MODE_RHS, false>)
                     : mode == MODE_STAGE1 ? reinterpret_cast<const void *>(&k_stage<P, Real, MODE_STAGE1, SEP>)
                                           : reinterpret_cast<const void *>(&k_stage<P, Real, MODE_STAGE2, SEP>);
    return emit(s, fn, grid, block, kargs);
}

template <typename Real>
hipError_t stage_r(int p, int mode, bool sep, const void *args, Sink &s)
{
    if (sep) {
        switch (p) {
        case 0: return stage_p<0, Real, true>(mode, args, s);
        case 1: return stage_p<1, Real, true>(mode, args, s);
        case 2: return stage_p<2, Real, true>(mode, args, s);
        }
        return hipErrorInvalidValue;
    }
    switch (p) {
    case 0: return stage_p<0, Real, false>(mode, args, s);
    case 1: return stage_p<1, Real, false>(mode, args, s);
    case 2: return stage_p<2, Real, false>(mode, args, s);
    case 3: return stage_p<3, Real, false>(mode, args, s);
    }
    return hipErrorInvalidValue;
}

template <int P, typename Real>
hipError_t usolve_p(const void *args, hipStream_t s)
{
    const StageArgs<Real> &a = *static_cast<const StageArgs<Real> *>(args);
    if (a.m.ne <= 0) return hipSuccess;
    hipLaunchKernelGGL((k_usolve<P, Real>), dim3((a.m.ne + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, s, a);
    return hipGetLastError();
}

template <typename Real>
hipError_t usolve_r(int p, const void *args, hipStream_t s)
{
    switch (p) {
    case 0: return usolve_p<0, Real>(args, s);
    case 1: return usolve_p<1, Real>(args, s);
    case 2: return usolve_p<2, Real>(args, s);
    case 3: return usolve_p<3, Real>(args, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t emit(Sink &k, const void *fn, dim3 grid, dim3 block, void **args)
{
    if (!k.g) return hipLaunchKernel(fn, grid, block, args, 0, k.s);
    hipKernelNodeParams prm{};
    prm.func = const_cast<void *>(fn);
    prm.gridDim = grid;
    prm.blockDim = block;
    prm.sharedMemBytes = 0;
    prm.kernelParams = args;      // copied into the node
    prm.extra = nullptr;
    hipGraphNode_t node = nullptr;
    const hipError_t e = hipGraphAddKernelNode(&node, k.g, k.ndep ? k.dep : nullptr, (size_t)k.ndep, &prm);
    if (e == hipSuccess) {
        k.dep[0] = node;
        k.ndep = 1;
    }
    return e;
}

hipError_t launch_stage(int p, bool fp32, int mode, bool sep, const void *args, Sink &k)
{
    return fp32 ? stage_r<float>(p, mode, sep, args, k) : stage_r<double>(p, mode, sep, args, k);
}

template <int P, typename Real>
hipError_t stage_sh_p(int mode, const void *args, const unsigned *items, const int *item_off, Sink &k)
{
    StageArgs<Real> a = *static_cast<const StageArgs<Real> *>(args);
    if (a.m.ne <= 0) return hipSuccess;
    void *kargs[] = {&a, &items, &item_off};
    const void *fn = mode == MODE_RHS      ? reinterpret_cast<const void *>(&k_stage_sh<P, Real, MODE_RHS>)
                     : mode == MODE_STAGE1 ? reinterpret_cast<const void *>(&k_stage_sh<P, Real, MODE_STAGE1>)
                                           : reinterpret_cast<const void *>(&k_stage_sh<P, Real, MODE_STAGE2>);
    const int nb = (a.m.ne + BLOCK - 1) / BLOCK;
    return emit(k, fn, dim3(a.blocks > 0 && a.blocks < nb ? a.blocks : nb), dim3(BLOCK), kargs);
}

// Order 0 has too little work per edge for the sharing to pay for the LDS
// staging and the barriers.
bool stage_sh_supported(int p, bool fp32)
{
    (void)fp32;
    return p >= 1 && p <= 3;
}

hipError_t launch_stage_sh(int p, bool fp32, int mode, const void *args, const unsigned *items, const int *item_off,
                           Sink &k)
{
    if (fp32) {
        switch (p) {
        case 0: return stage_sh_p<0, float>(mode, args, items, item_off, k);
        case 1: return stage_sh_p<1, float>(mode, args, items, item_off, k);
        case 2: return stage_sh_p<2, float>(mode, args, items, item_off, k);
        case 3: return stage_sh_p<3, float>(mode, args, items, item_off, k);
        }
    } else {
        switch (p) {
        case 0: return stage_sh_p<0, double>(mode, args, items, item_off, k);
        case 1: return stage_sh_p<1, double>(mode, args, items, item_off, k);
        case 2: return stage_sh_p<2, double>(mode, args, items, item_off, k);
        case 3: return stage_sh_p<3, double>(mode, args, items, item_off, k);
        }
    }
    return hipErrorInvalidValue;
}

hipError_t launch_stage(int p, bool fp32, int mode, bool sep, const void *args, hipStream_t s)
{
    Sink k;
    k.s = s;
    return launch_stage(p, fp32, mode, sep, args, k);
}

// Blocks per order of a list kernel whose longest possible list fills nblk
// runs of BLOCK entries: a kernel that reaches order 3 takes every list in
// TEAM-entry runs (4 nblk blocks); below order 3 a block takes a run of BLOCK
// entries (nblk blocks) or, for a list of at most TEAM_MAX entries, a run of
// TEAM entries (at most TEAM_MAX / TEAM blocks).  Lists re-chosen on the
// device are mostly empty, and each block costs a dispatch even when it
// finds nothing to do: no more blocks than these.
int list_grid(int nblk, int pn)
{
    const int runs = nblk * (BLOCK / TEAM);
    if (pn >= 3) return runs;
    const int teams = runs < TEAM_MAX / TEAM ? runs : TEAM_MAX / TEAM;
    return nblk > teams ? nblk : teams;
}

template <int PN, typename Real>
hipError_t full_all_r(int mode, const void *args, int lo, int nblk, int lcap, Sink &s)
{
    StageArgs<Real> a = *static_cast<const StageArgs<Real> *>(args);
    void *kargs[] = {&a, &lo, &lcap};
    // (one block more for the clock)
    const dim3 g((PN - lo + 1) * list_grid(nblk, PN) + (a.tick ? 1 : 0)), b(TEAM * TEAM_ROLES);
    return emit(s,
                mode == MODE_STAGE1 ? reinterpret_cast<const void *>(&k_full_all<PN, Real, MODE_STAGE1>)
                                    : reinterpret_cast<const void *>(&k_full_all<PN, Real, MODE_STAGE2>),
                g, b, kargs);
}

template <int B, int PN, typename Real>
hipError_t part_all_r(int mode, const void *args, int nblk, int lcap, int nsh, int e_end, const unsigned *items,
                      const int *item_off, Sink &s)
{
    StageArgs<Real> a = *static_cast<const StageArgs<Real> *>(args);
    // (a multiple of 8, so that the base blocks keep their XCDs; the last is past
    // every list's end where there is a clock to advance)
    int nlist = ((PN - B + 1) * list_grid(nblk, PN) + (a.tick ? 8 : 7)) / 8 * 8;
    void *kargs[] = {&a, &lcap, &nlist, &nsh, &e_end, &items, &item_off};
    return emit(s,
                mode == MODE_STAGE1 ? reinterpret_cast<const void *>(&k_part_all<B, PN, Real, MODE_STAGE1>)
                                    : reinterpret_cast<const void *>(&k_part_all<B, PN, Real, MODE_STAGE2>),
                dim3(nlist + (e_end + BLOCK - 1) / BLOCK), dim3(BLOCK), kargs);
}

hipError_t launch_part_all(int b, int pn, bool fp32, int mode, const void *args, int nblk, int lcap, int nsh, int e_end,
                           const unsigned *items, const int *item_off, Sink &k)
{
    if (mode != MODE_STAGE1 && mode != MODE_STAGE2) return hipErrorInvalidValue;
    if (b == 1 && pn == 2)
        return fp32 ? part_all_r<1, 2, float>(mode, args, nblk, lcap, nsh, e_end, items, item_off, k)
                    : part_all_r<1, 2, double>(mode, args, nblk, lcap, nsh, e_end, items, item_off, k);
    if (b == 1 && pn == 3 && !fp32)
        return part_all_r<1, 3, double>(mode, args, nblk, lcap, nsh, e_end, items, item_off, k);
    if (b == 2 && pn == 3 && !fp32)
        return part_all_r<2, 3, double>(mode, args, nblk, lcap, nsh, e_end, items, item_off, k);
    return hipErrorInvalidValue;
}

hipError_t launch_full_all(int lo, int pn, bool fp32, int mode, const void *args, int nblk, int lcap, Sink &k)
{
    if (nblk <= 0) return hipSuccess;
    if (lo < 0 || lo > pn || pn < 1 || pn > 3 || (mode != MODE_STAGE1 && mode != MODE_STAGE2))
        return hipErrorInvalidValue;
    switch (pn) {
    case 1: return fp32 ? full_all_r<1, float>(mode, args, lo, nblk, lcap, k) : full_all_r<1, double>(mode, args, lo, nblk, lcap, k);
    case 2: return fp32 ? full_all_r<2, float>(mode, args, lo, nblk, lcap, k) : full_all_r<2, double>(mode, args, lo, nblk, lcap, k);
    case 3: return fp32 ? full_all_r<3, float>(mode, args, lo, nblk, lcap, k) : full_all_r<3, double>(mode, args, lo, nblk, lcap, k);
    }
    return hipErrorInvalidValue;
}

template <int B, int PN, typename Real>
hipError_t corr_all_r(const void *args, double dt, int nblk, int lcap, Sink &s)
{
    StageArgs<Real> a = *static_cast<const StageArgs<Real> *>(args);
    void *kargs[] = {&a, &dt, &lcap};
    return emit(s, reinterpret_cast<const void *>(&k_corr_all<B, PN, Real>), dim3((PN - B + 1) * list_grid(nblk, PN)),
                dim3(TEAM * TEAM_ROLES), kargs);
}

template <typename Real>
hipError_t corr_all_t(int b, int pn, const void *args, double dt, int nblk, int lcap, Sink &k)
{
    if (b == 0 && pn == 1) return corr_all_r<0, 1, Real>(args, dt, nblk, lcap, k);
    if (b == 0 && pn == 2) return corr_all_r<0, 2, Real>(args, dt, nblk, lcap, k);
    if (b == 0 && pn == 3) return corr_all_r<0, 3, Real>(args, dt, nblk, lcap, k);
    if (b == 1 && pn == 2) return corr_all_r<1, 2, Real>(args, dt, nblk, lcap, k);
    if (b == 1 && pn == 3) return corr_all_r<1, 3, Real>(args, dt, nblk, lcap, k);
    if (b == 2 && pn == 3) return corr_all_r<2, 3, Real>(args, dt, nblk, lcap, k);
    return hipErrorInvalidValue;
}

template <typename Real>
int host_corr_r(int b, int pn, const void *args, double dt, const signed char *order, int e0, int e1, int nthreads)
{
    const StageArgs<Real> &a = *static_cast<const StageArgs<Real> *>(args);
    if (b == 0 && pn == 1) host_corr_t<0, 1, Real>(a, dt, order, e0, e1, nthreads);
    else if (b == 0 && pn == 2) host_corr_t<0, 2, Real>(a, dt, order, e0, e1, nthreads);
    else if (b == 0 && pn == 3) host_corr_t<0, 3, Real>(a, dt, order, e0, e1, nthreads);
    else if (b == 1 && pn == 2) host_corr_t<1, 2, Real>(a, dt, order, e0, e1, nthreads);
    else if (b == 1 && pn == 3) host_corr_t<1, 3, Real>(a, dt, order, e0, e1, nthreads);
    else if (b == 2 && pn == 3) host_corr_t<2, 3, Real>(a, dt, order, e0, e1, nthreads);
    else return -1;
    return 0;
}

int host_corr(int b, int pn, bool fp32, const void *args, double dt, const signed char *order, int e0, int e1,
              int nthreads)
{
    return fp32 ? host_corr_r<float>(b, pn, args, dt, order, e0, e1, nthreads)
                : host_corr_r<double>(b, pn, args, dt, order, e0, e1, nthreads);
}

hipError_t launch_corr_all(int b, int pn, bool fp32, const void *args, double dt, int nblk, int lcap, Sink &k)
{
    if (nblk <= 0) return hipSuccess;
    return fp32 ? corr_all_t<float>(b, pn, args, dt, nblk, lcap, k) : corr_all_t<double>(b, pn, args, dt, nblk, lcap, k);
}

template <int PN, typename Real>
hipError_t epi_all_r(int mode, int KB, const void *args, int lo, int nblk, int lcap, Sink &s)
{
    StageArgs<Real> a = *static_cast<const StageArgs<Real> *>(args);
    void *kargs[] = {&a, &KB, &lo, &lcap};
    const dim3 g((PN - lo + 1) * nblk), b(BLOCK);
    return emit(s,
                mode == MODE_STAGE1 ? reinterpret_cast<const void *>(&k_epi_all<PN, Real, MODE_STAGE1>)
                                    : reinterpret_cast<const void *>(&k_epi_all<PN, Real, MODE_STAGE2>),
                g, b, kargs);
}

hipError_t launch_epi_all(int b, int pn, bool fp32, int mode, const void *args, int nblk, int lcap, Sink &k)
{
    if (nblk <= 0) return hipSuccess;
    if (b < 0 || b > pn || pn < 1 || pn > 3 || (mode != MODE_STAGE1 && mode != MODE_STAGE2))
        return hipErrorInvalidValue;
    const int KB = (b + 1) * (b + 2) / 2;
    switch (pn) {
    case 1: return fp32 ? epi_all_r<1, float>(mode, KB, args, b, nblk, lcap, k) : epi_all_r<1, double>(mode, KB, args, b, nblk, lcap, k);
    case 2: return fp32 ? epi_all_r<2, float>(mode, KB, args, b, nblk, lcap, k) : epi_all_r<2, double>(mode, KB, args, b, nblk, lcap, k);
    case 3: return fp32 ? epi_all_r<3, float>(mode, KB, args, b, nblk, lcap, k) : epi_all_r<3, double>(mode, KB, args, b, nblk, lcap, k);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_usolve(int p, bool fp32, const void *args, hipStream_t s)
{
    return fp32 ? usolve_r<float>(p, args, s) : usolve_r<double>(p, args, s);
}

template <typename Real>
hipError_t depth_limit_r(int pm, const void *args, double h_min, Sink &s)
{
    StageArgs<Real> a = *static_cast<const StageArgs<Real> *>(args);
    void *kargs[] = {&a, &h_min};
    const dim3 g((a.m.ne + BLOCK - 1) / BLOCK), b(BLOCK);
    switch (pm) {
    case 1: return emit(s, reinterpret_cast<const void *>(&k_depth_limit<1, Real>), g, b, kargs);
    case 2: return emit(s, reinterpret_cast<const void *>(&k_depth_limit<2, Real>), g, b, kargs);
    case 3: return emit(s, reinterpret_cast<const void *>(&k_depth_limit<3, Real>), g, b, kargs);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_depth_limit(int pm, bool fp32, const void *args, double h_min, Sink &k)
{
    if (pm < 1) return hipSuccess;   // order 0 has nothing to scale
    return fp32 ? depth_limit_r<float>(pm, args, h_min, k) : depth_limit_r<double>(pm, args, h_min, k);
}

hipError_t launch_pack(bool fp32, const void *src, int stride, int first, int nslots, const int *iperm,
                       const double4 *vtx, const int *ev, int evs, int u0, int u1, double *out, hipStream_t s)
{
    if (u1 <= u0) return hipSuccess;
    const dim3 g((u1 - u0 + XFER - 1) / XFER), b(BLOCK);
    if (fp32)
        hipLaunchKernelGGL(k_pack<float>, g, b, 0, s, static_cast<const float *>(src), stride, first, nslots, iperm,
                           vtx, ev, evs, u0, u1, out);
    else
        hipLaunchKernelGGL(k_pack<double>, g, b, 0, s, static_cast<const double *>(src), stride, first, nslots, iperm,
                           vtx, ev, evs, u0, u1, out);
    return hipGetLastError();
}

hipError_t launch_unpack(bool fp32, const double *in, int K, const int *iperm, const MeshView &m, int u0, int u1,
                         void *dst, int *bad, hipStream_t s)
{
    if (u1 <= u0) return hipSuccess;
    const dim3 g((u1 - u0 + XFER - 1) / XFER), b(BLOCK);
    if (fp32)
        hipLaunchKernelGGL(k_unpack<float>, g, b, 0, s, in, K, iperm, m.vtx, m.ev, m.stride, m.ep, u0, u1,
                           static_cast<float *>(dst), m.stride, bad);
    else
        hipLaunchKernelGGL(k_unpack<double>, g, b, 0, s, in, K, iperm, m.vtx, m.ev, m.stride, m.ep, u0, u1,
                           static_cast<double *>(dst), m.stride, bad);
    return hipGetLastError();
}

int mass_partials(int ne) { return (ne + BLOCK - 1) / BLOCK; }

namespace {
template <int P, typename Real, int TILE>
hipError_t batch_pt(int mode, const BatchArgs &b, int grid, Sink &s)
{
    BatchArgs a = b;
    void *kargs[] = {&a};
    const void *fn = mode == MODE_STAGE1 ? reinterpret_cast<const void *>(&k_batch_stage<P, Real, MODE_STAGE1, TILE>)
                                         : reinterpret_cast<const void *>(&k_batch_stage<P, Real, MODE_STAGE2, TILE>);
    return emit(s, fn, dim3(grid), dim3(TILE), kargs);
}

template <typename Real, int TILE>
hipError_t batch_t(int p, int mode, const BatchArgs &b, int grid, Sink &s)
{
    switch (p) {
    case 0: return batch_pt<0, Real, TILE>(mode, b, grid, s);
    case 1: return batch_pt<1, Real, TILE>(mode, b, grid, s);
    case 2: return batch_pt<2, Real, TILE>(mode, b, grid, s);
    case 3: return batch_pt<3, Real, TILE>(mode, b, grid, s);
    }
    return hipErrorInvalidValue;
}

template <typename Real>
hipError_t batch_r(int p, int mode, int tile, const BatchArgs &b, int grid, Sink &s)
{
    switch (tile) {
    case 64: return batch_t<Real, 64>(p, mode, b, grid, s);
    case 128: return batch_t<Real, 128>(p, mode, b, grid, s);
    case 256: return batch_t<Real, 256>(p, mode, b, grid, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_batch_stage(int p, bool fp32, int mode, int tile, const BatchArgs &b, int grid, Sink &k)
{
    if (grid <= 0) return hipSuccess;
    return fp32 ? batch_r<float>(p, mode, tile, b, grid, k) : batch_r<double>(p, mode, tile, b, grid, k);
}

template <int P, typename Real>
hipError_t batch_sh_p(int mode, const BatchArgs &b, int grid, Sink &k)
{
    BatchArgs a = b;
    void *kargs[] = {&a};
    const void *fn = mode == MODE_STAGE1 ? reinterpret_cast<const void *>(&k_batch_stage_sh<P, Real, MODE_STAGE1>)
                                         : reinterpret_cast<const void *>(&k_batch_stage_sh<P, Real, MODE_STAGE2>);
    return emit(k, fn, dim3(grid), dim3(BLOCK), kargs);
}

hipError_t launch_batch_stage_sh(int p, bool fp32, int mode, const BatchArgs &b, int grid, Sink &k)
{
    if (grid <= 0) return hipSuccess;
    if (mode != MODE_STAGE1 && mode != MODE_STAGE2) return hipErrorInvalidValue;
    if (fp32 && p == 1) return batch_sh_p<1, float>(mode, b, grid, k);
    if (fp32 && p == 2) return batch_sh_p<2, float>(mode, b, grid, k);
    if (fp32 && p == 3) return batch_sh_p<3, float>(mode, b, grid, k);
    if (!fp32 && p == 1) return batch_sh_p<1, double>(mode, b, grid, k);
    if (!fp32 && p == 2) return batch_sh_p<2, double>(mode, b, grid, k);
    if (!fp32 && p == 3) return batch_sh_p<3, double>(mode, b, grid, k);
    return hipErrorInvalidValue;
}

hipError_t launch_place_items(const unsigned *items, const int *item_off, int nblk, const PoolView &pool, int first,
                              hipStream_t s)
{
    if (nblk <= 0) return hipSuccess;
    if (first % BLOCK != 0 || !pool.items || !pool.nitems) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_place_items, dim3(nblk), dim3(BLOCK), 0, s, items, item_off, pool, first);
    return hipGetLastError();
}

hipError_t launch_next_clock(InstDesc *from, InstDesc *to, const int *flag, Sink &k)
{
    void *kargs[] = {&from, &to, &flag};
    return emit(k, reinterpret_cast<const void *>(&k_next_clock), dim3(1), dim3(64), kargs);
}

hipError_t launch_batch_clock(InstDesc *inst, const int *flags, int n, int order, Sink &k)
{
    if (n <= 0) return hipSuccess;
    void *kargs[] = {&inst, &flags, &n, &order};
    return emit(k, reinterpret_cast<const void *>(&k_batch_clock), dim3((n + BLOCK - 1) / BLOCK), dim3(BLOCK), kargs);
}

hipError_t launch_relocate(const int *ev, const int *nb, const unsigned char *nbk, const signed char *ep, int ne,
                           int stride, const PoolView &pool, int first, int vbase, hipStream_t s)
{
    if (ne <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_relocate, dim3((ne + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, s, ev, nb, nbk, ep, ne, stride,
                       pool, first, vbase);
    return hipGetLastError();
}

hipError_t launch_batch_indicator(bool fp32, const BatchArgs &b, int grid, Sink &k)
{
    if (grid <= 0) return hipSuccess;
    BatchArgs a = b;
    void *kargs[] = {&a};
    return emit(k, fp32 ? reinterpret_cast<const void *>(&k_batch_indicator<float>)
                        : reinterpret_cast<const void *>(&k_batch_indicator<double>),
                dim3(grid), dim3(BLOCK), kargs);
}

hipError_t launch_batch_apply(int pm, bool fp32, const BatchArgs &b, int grid, Sink &k)
{
    if (grid <= 0) return hipSuccess;
    BatchArgs a = b;
    void *kargs[] = {&a};
    const void *fn = nullptr;
    switch (pm) {
    case 1: fn = fp32 ? reinterpret_cast<const void *>(&k_batch_apply<1, float>)
                      : reinterpret_cast<const void *>(&k_batch_apply<1, double>); break;
    case 2: fn = fp32 ? reinterpret_cast<const void *>(&k_batch_apply<2, float>)
                      : reinterpret_cast<const void *>(&k_batch_apply<2, double>); break;
    case 3: fn = fp32 ? reinterpret_cast<const void *>(&k_batch_apply<3, float>)
                      : reinterpret_cast<const void *>(&k_batch_apply<3, double>); break;
    default: return hipErrorInvalidValue;
    }
    return emit(k, fn, dim3(grid), dim3(BLOCK), kargs);
}

template <typename Real>
hipError_t indicator_r(const void *args, double tau, int p_lo, int p_hi, double *I_out, signed char *p_new,
                       Sink &s)
{
    StageArgs<Real> a = *static_cast<const StageArgs<Real> *>(args);
    void *kargs[] = {&a, &tau, &p_lo, &p_hi, &I_out, &p_new};
    return emit(s, reinterpret_cast<const void *>(&k_indicator<Real>), dim3((a.m.ne + BLOCK - 1) / BLOCK),
                dim3(BLOCK), kargs);
}

hipError_t launch_indicator(bool fp32, const void *args, double tau, int p_lo, int p_hi, double *I_out,
                            signed char *p_new, Sink &k)
{
    return fp32 ? indicator_r<float>(args, tau, p_lo, p_hi, I_out, p_new, k)
                : indicator_r<double>(args, tau, p_lo, p_hi, I_out, p_new, k);
}

hipError_t launch_indicator(bool fp32, const void *args, double tau, int p_lo, int p_hi, double *I_out,
                            signed char *p_new, hipStream_t s)
{
    Sink k;
    k.s = s;
    return launch_indicator(fp32, args, tau, p_lo, p_hi, I_out, p_new, k);
}

template <typename Real>
hipError_t apply_r(int pm, const void *args, const signed char *p_new, signed char *p_cur, int p_base, int lcap,
                   InstDesc *clock, const int *flag, Sink &s)
{
    StageArgs<Real> a = *static_cast<const StageArgs<Real> *>(args);
    void *kargs[] = {&a, &p_new, &p_cur, &p_base, &lcap, &clock, &flag};
    const dim3 g((a.m.ne + BLOCK - 1) / BLOCK), b(BLOCK);
    switch (pm) {
    case 0: return emit(s, reinterpret_cast<const void *>(&k_apply_order<0, Real>), g, b, kargs);
    case 1: return emit(s, reinterpret_cast<const void *>(&k_apply_order<1, Real>), g, b, kargs);
    case 2: return emit(s, reinterpret_cast<const void *>(&k_apply_order<2, Real>), g, b, kargs);
    case 3: return emit(s, reinterpret_cast<const void *>(&k_apply_order<3, Real>), g, b, kargs);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_apply_order(int pm, bool fp32, const void *args, const signed char *p_new, signed char *p_cur,
                              int p_base, int lcap, InstDesc *clock, const int *flag, Sink &k)
{
    return fp32 ? apply_r<float>(pm, args, p_new, p_cur, p_base, lcap, clock, flag, k)
                : apply_r<double>(pm, args, p_new, p_cur, p_base, lcap, clock, flag, k);
}

__global__ void k_inst_set(InstDesc *inst, InstDesc v)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *inst = v;
}

hipError_t launch_inst_set(InstDesc *inst, const InstDesc &v, hipStream_t s)
{
    hipLaunchKernelGGL(k_inst_set, dim3(1), dim3(64), 0, s, inst, v);
    return hipGetLastError();
}

// Partial sums of the mass reduction for callers that cannot allocate: a
// fixed array on each device (the library holds it until the process ends),
// enough for MASS_SCRATCH_PARTIALS blocks of 256 elements.  Host code never
// passes the array's name to a kernel (on the host it only stands in for the
// symbol): it takes the device address once per device with that device
// current and uses that.
static __device__ __align__(256) double scratch[MASS_SCRATCH_PARTIALS];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex scratch_mutex;
double *scratch_ptr[MAX_DEVICES] = {};
}  // namespace

hipError_t mass_scratch(double **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        scratch_ptr[dev] = static_cast<double *>(ptr);
    }
    if (out) *out = scratch_ptr[dev];
    return hipSuccess;
}

hipError_t launch_mass_noalloc(const MeshView &m, bool fp32, const void *C, double *out, hipStream_t s)
{
    const int nb = mass_partials(m.ne);
    if (nb <= 0 || nb > MASS_SCRATCH_PARTIALS) return hipErrorInvalidValue;
    double *part = nullptr;
    hipError_t e = mass_scratch(&part);
    if (e != hipSuccess) return e;
    // every partial the final pass reads is written by the first pass: nothing to clear
    if (fp32)
        hipLaunchKernelGGL(k_mass_partial<float>, dim3(nb), dim3(BLOCK), 0, s, m, static_cast<const float *>(C), part);
    else
        hipLaunchKernelGGL(k_mass_partial<double>, dim3(nb), dim3(BLOCK), 0, s, m, static_cast<const double *>(C),
                           part);
    hipLaunchKernelGGL(k_mass_final, dim3(1), dim3(BLOCK), 0, s, part, nb, out);
    return hipGetLastError();
}

hipError_t launch_mass(const MeshView &m, bool fp32, const void *C, double *partial, double *out,
                       hipStream_t s)
{
    const int nb = mass_partials(m.ne);
    if (nb <= 0) return hipErrorInvalidValue;
    if (fp32)
        hipLaunchKernelGGL(k_mass_partial<float>, dim3(nb), dim3(BLOCK), 0, s, m,
                           static_cast<const float *>(C), partial);
    else
        hipLaunchKernelGGL(k_mass_partial<double>, dim3(nb), dim3(BLOCK), 0, s, m,
                           static_cast<const double *>(C), partial);
    hipLaunchKernelGGL(k_mass_final, dim3(1), dim3(BLOCK), 0, s, partial, nb, out);
    return hipGetLastError();
}

}  // namespace swe
