// gfx950 kernels that advance a uniform-order context by a whole SSP-RK2 step
// in one launch, and the kernel that builds their tile data.
#include "swe_device.h"

namespace swe {
namespace {

// ------------------------------------------------------------ a whole step in one launch
// Both SSP-RK2 stages of a tile of elements in one kernel.  A tile owns
// tv.len consecutive elements and also evaluates the first stage of their
// neighbours outside it (its ring), so the second stage finds every
// neighbour's first-stage value in LDS: the intermediate state is neither
// written nor read back, and a step is one dependent launch instead of two.
// Each owned element is stored by one tile only; a ring element's first stage
// is computed again by its own tile, from the same numbers in the same order
// (a flux is the same bits from either side), so the result equals two stage
// launches bit for bit.
//
// A tile is one block of 256 lanes, one local element each: the owned ones,
// then the ring.  Of a Morton-ordered structured triangulation a tile of 176 to
// 192 elements has a ring of 52 to 55 on average and of 64 to 74 at most (sides
// 160 to 512), so the mesh's longest ring sets its tiles' length: 192 at side
// 512, 184 or 176 at most others.  The ring fits the fourth wave but for a few
// lanes, and that wave sits out the second stage's element work: 1.14 to 1.15
// times the element work of two separate stages (1.17 to 1.2 with the lanes
// past the ring) for about half their traffic.
// Bound by VALU issue at FP32 p = 2 (74 % of the SIMDs' cycles), by latency at
// two blocks and one per CU in FP64 p = 2 and 3.  Two launches / one, us a
// step: FP32 p = 1 50.3 / 39.8 and p = 2 84.3 / 73.5 (524,288 elements), FP64
// p = 1 86 / 64 and p = 2 158 / 142 (524,288), 84 / 81 (260,642), p = 3 FP32
// 33.1 / 26.0 and FP64 49.7 / 38.5 (39,200).  The two stages are unrolled: as
// a loop the invariants of both live across it (FP64 p = 2 spilled, 110 us
// at 260,642 elements).  Tile data is built on the device (k_build_tiles) by the
// first call that steps this way: edge items, ring and outside neighbours, and
// the tile's vertices, which are staged in LDS so that neither the edge pass nor
// the element pass reads vertex ids or vertices from memory.
template <int P, typename Real, bool BOTH>
struct StepLds {
    ShLds<P, Real, BOTH> S;
    double vx[TILE_NV], vy[TILE_NV], vh[TILE_NV];
    unsigned tri[BLOCK];   // an element's three vertices among the tile's, 8 bits each
};

template <int P, typename Real, bool BOTH>
struct TileSrc {
    const StepLds<P, Real, BOTH> &T;
    int ext;               // the item's neighbour outside the tile
    __device__ __forceinline__ void edge(int la, int va, int vb, double3 &pa, double3 &pb) const
    {
        const unsigned t = T.tri[la];
        const int a = (int)((t >> (8 * va)) & 255u), b = (int)((t >> (8 * vb)) & 255u);
        pa = make_double3(T.vx[a], T.vy[a], T.vh[a]);
        pb = make_double3(T.vx[b], T.vy[b], T.vh[b]);
    }
    __device__ __forceinline__ unsigned outside(unsigned w, int &kk) const
    {
        kk = (int)((w >> 18) & 3u);
        return (unsigned)ext;
    }
};

template <int P, typename Real, bool BOTH>
__device__ __forceinline__ void sh_copy_state(ShLds<P, Real, BOTH> &S, int l, const Fields<P, Real> &s)
{
    constexpr int K = Ord<P>::K;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        S.U.C[0 * K + q][l] = s.xi[q];
        S.U.C[1 * K + q][l] = s.U[q];
        S.U.C[2 * K + q][l] = s.V[q];
        S.U.C[3 * K + q][l] = s.u[q];
        S.U.C[4 * K + q][l] = s.v[q];
    }
}

// geometry of local element l from the tile's vertices
template <int P, typename Real, bool BOTH>
__device__ __forceinline__ void tile_geo(const StepLds<P, Real, BOTH> &T, int l, Geo &G)
{
    unsigned t = T.tri[l];
    asm volatile("" : "+v"(t));   // formed anew at each use, not kept in registers between the stages
#pragma unroll
    for (int v = 0; v < 3; ++v) {
        const int i = (int)((t >> (8 * v)) & 255u);
        G.X[v] = T.vx[i];
        G.Y[v] = T.vy[i];
        G.h[v] = T.vh[i];
    }
    geo_finish(G);
}

// One tile, elements [e0, e0 + nown) owned; every thread of the block calls it.
template <int P, typename Real>
__device__ __forceinline__ void step_tile(StepLds<P, Real, false> &T, const StageArgs<Real> &a, const TileView &tv, int tile,
                                          unsigned e0, int nown, double xh0, double xh1, double dt0, int *flag)
{
    constexpr int K = Ord<P>::K;
    const MeshView &m = a.m;
    const int l = (int)threadIdx.x;
    const int KS0 = m.KS, stride0 = m.stride;
    const int *meta = tv.meta + (size_t)tile * BLOCK;
    const unsigned w0 = tv.items[(size_t)tile * (2 * BLOCK) + l], w1 = tv.items[(size_t)tile * (2 * BLOCK) + BLOCK + l];
    // a lane past the ring repeats the tile's first element (its results are
    // not used): no lane's state has to survive a branch it does not take,
    // which cost 30 registers
    const int id = l < nown ? (int)e0 + l : meta[l];
    const int lx = id >= 0 ? l : 0;
    const unsigned off = (id >= 0 ? (unsigned)id : e0) * (unsigned)sizeof(Real);
    T.tri[l] = tv.tri[(size_t)tile * BLOCK + l];
    if (l < TILE_NV) {
        const int v = tv.verts[(size_t)tile * TILE_NV + l];
        if (v >= 0) {
            const double4 p = m.vtx[(unsigned)v];
            T.vx[l] = p.x;
            T.vy[l] = p.y;
            T.vh[l] = p.z;
        }
    }
    int x0 = 0, x1 = 0;
    if (w0 != ITEM_PAD && ((w0 >> 20) & 3u) == EK_EXT) x0 = meta[(w0 >> 10) & 255u];
    if (w1 != ITEM_PAD && ((w1 >> 20) & 3u) == EK_EXT) x1 = meta[(w1 >> 10) & 255u];
    Fields<P, Real> s;
    {
        const Buf<Real> bC(a.Cin, 3 * KS0, stride0), bU(a.Uin, 2 * KS0, stride0);
        load_state<P, Real>(bC, bU, KS0, off, s);
        sh_copy_state<P, Real, false>(T.S, l, s);
    }
    __syncthreads();
#pragma unroll
    for (int st = 0; st < 2; ++st) {
        // opaque copies: what follows from them is formed anew in each pass
        // instead of being kept (and spilled) across the loop
        int stride = stride0;
        unsigned v0 = w0, v1 = w1;
        asm volatile("" : "+s"(stride));
        asm volatile("" : "+v"(v0));
        asm volatile("" : "+v"(v1));
        const int KS = KS0;
        const Buf<Real> bC(a.Cin, 3 * KS, stride), bU(a.Uin, 2 * KS, stride);
        const double xihat = st ? xh1 : xh0;
        Physics ph = a.ph;
        double dt = dt0;
        asm volatile("" : "+s"(ph.g), "+s"(ph.fc), "+s"(ph.fric), "+s"(dt));
        const double g = ph.g;
        // the edges that touch no owned element are not needed a second time
        const bool use0 = v0 != ITEM_PAD && !(st && (v0 & ITEM_RING));
        const bool use1 = v1 != ITEM_PAD && !(st && (v1 & ITEM_RING));
        {
            ShItem<P, Real> r0, r1;
            if (use0) sh_flux<P, Real, false>(T.S, KS, bC, bU, TileSrc<P, Real, false>{T, x0}, v0, xihat, g, r0);
            if (use1) sh_flux<P, Real, false>(T.S, KS, bC, bU, TileSrc<P, Real, false>{T, x1}, v1, xihat, g, r1);
            __syncthreads();
            if (use0) sh_store<P, Real, false>(T.S, l, v0, r0);
            if (use1) sh_store<P, Real, false>(T.S, l + BLOCK, v1, r1);
        }
        __syncthreads();
        if (st && l >= nown) return;   // (no barrier follows)
        Geo G;
        tile_geo<P, Real, false>(T, lx, G);
        double hbh[3];
        hb_modes(G, hbh);
        Acc<P, Real> A;
        acc_init<P, Real>(A, s, true);
        volume_term<P, Real>(s, hbh, G, g, dt, A);
        source_term<P, Real>(s, G, ph, dt, A);
        // c^n again from memory (held in registers across both stages it would
        // cost a wave per SIMD), on its way while the edges are lifted
        Real cn[3][K];
        if (st) {
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int q = 0; q < K; ++q) cn[j][q] = bC.ld(j * KS + q, off);
        }
        sh_lift<P, Real, false>(T.S, G, lx, dt, A);
        if constexpr (Acc<P, Real>::SPLIT) {
#pragma unroll
            for (int q = 0; q < K; ++q) {
                A.L[1][q] += Real(A.W[0][q]);
                A.L[2][q] += Real(A.W[1][q]);
            }
        }
        if (a.src) {
            const Buf<Real> bS(a.src, 3 * KS, stride);
            const Real rdt = Real(dt);
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int q = 0; q < K; ++q) A.L[j][q] = fma(rdt, bS.ld(j * KS + q, off), A.L[j][q]);
        }
        if (st) {
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int q = 0; q < K; ++q) A.L[j][q] = Real(0.5) * cn[j][q] + Real(0.5) * A.L[j][q];
        }
        solve_u<P, Real>(A.L[0], A.L[1], A.L[2], hbh, K, s.u, s.v);
        Real chk = 0;
#pragma unroll
        for (int q = 0; q < K; ++q) {
            s.xi[q] = A.L[0][q];
            s.U[q] = A.L[1][q];
            s.V[q] = A.L[2][q];
            chk += s.xi[q] + s.U[q] + s.V[q] + s.u[q] + s.v[q];
        }
        const double Hmean = SQRT2 * double(s.xi[0]) + (G.h[0] + G.h[1] + G.h[2]) * (1.0 / 3.0);
        if (!(Hmean > 0.0) || !isfinite(chk)) flag[0] = 1;
        if (st == 0) {
            __syncthreads();   // every lane is done with the first stage's fluxes
            sh_copy_state<P, Real, false>(T.S, l, s);
            __syncthreads();
        }
    }
    // written through: the next step reads it from other XCDs' caches, and what
    // is dirty at the end of a kernel is written back then, by every block at
    // once (1-3 % shorter steps than the default or non-temporal policy)
    (void)store_state<P, Real, CPOL_THROUGH>(a, off, s.xi, s.U, s.V, s.u, s.v);
}

// A stopped step (failure in an earlier one).  The state rests in buffer 0:
// where the step before was the last to run and left its result in buffer 1
// (it was the first of a pair), the second of the pair carries it over.
// Thread l of the block takes the tile's owned element l.
template <int P, typename Real>
__device__ __forceinline__ void stopped_step(const StageArgs<Real> &a, int len)
{
    constexpr int K = Ord<P>::K;
    const int l = (int)threadIdx.x, e = xcd_block(blockIdx.x, gridDim.x) * len + l;
    if (!a.stage || !a.inst->ran || l >= len || e >= a.m.ne) return;
    const unsigned off = (unsigned)e * (unsigned)sizeof(Real);
    const int KS = a.m.KS, stride = a.m.stride;
    const Buf<Real> bC(a.Cin, 3 * KS, stride), bU(a.Uin, 2 * KS, stride);
    const Buf<Real> oC(a.Cout, 3 * KS, stride), oU(a.Uout, 2 * KS, stride);
#pragma unroll 1
    for (int q = 0; q < 3 * K; ++q) oC.st(q, off, bC.ld(q, off));
#pragma unroll 1
    for (int q = 0; q < 2 * K; ++q) oU.st(q, off, bU.ld(q, off));
}

template <int P, typename Real>
constexpr int step_waves()
{
    constexpr bool dbl = std::is_same<Real, double>::value;
    return dbl ? (P == 1 ? 3 : P == 3 ? 1 : 2) : (P == 2 ? 3 : P == 3 ? 2 : 4);
}

template <int P, typename Real>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(step_waves<P, Real>(), 8)))
k_step_sh(StageArgs<Real> a, TileView tv, double xihat2)
{
    __shared__ StepLds<P, Real, false> T;
    load_trace_lds<P, Real, false>(T.S);
    double xh0 = a.xihat, xh1 = xihat2, dt = a.dt;
    if (a.inst) {
        // the step's clock stopped (failure): the whole block leaves before its first barrier
        if (!a.inst->run) return stopped_step<P, Real>(a, tv.len);
        xh0 = a.inst->xh[0];
        xh1 = a.inst->xh[1];
        dt = a.inst->dt;
    }
    const int tile = xcd_block(blockIdx.x, gridDim.x);
    const int e0 = tile * tv.len, left = a.m.ne - e0;
    step_tile<P, Real>(T, a, tv, tile, (unsigned)e0, left < tv.len ? left : tv.len, xh0, xh1, dt, a.flag);
}

// The same tile by groups of four waves with roles: NG groups compute the edge
// fluxes (two items per lane, or one with NG = 2) while the first group does
// the volume and source terms of the same stage; then the first lifts the
// fluxes and finishes the elements.  For meshes of at most one tile per CU,
// where each SIMD would hold one wave and a stage is one chain of dependent
// instructions (FP32 p = 3: 18 thousand cycles of fluxes, then 17 of element
// work): the shorter of two parallel parts leaves the chain.  The roles are
// separate code from the first load to the last store, so that neither holds
// the other's registers (joined between the barriers, FP32 p = 2 took 205
// instead of 130).  Measured at 20,000 elements in tiles of 192, us a step with one
// group of waves / with roles: FP32 p = 1 10.3 / 7.7, p = 2 15.9 / 11.7, p = 3 25.8 /
// 20.1, FP64 p = 1 12.1 / 9.5, p = 2 20.3 / 17.4 (with two flux groups 18.3);
// FP64 p = 3 spills with one flux group already (36.7 / 53).  With more tiles
// than CUs the extra waves cost residency (51,200 elements, FP32 p = 2: 19.5 /
// 21.3); order 1 fits two blocks of two groups on a CU (65,522 elements, FP32
// 12.1 / 11.0, FP64 16.4 / 14.8; 96,800: FP32 14.5 / 16.9).
// Looped over the two stages instead of unrolled, half the code ran 1-5 % slower
// (p = 3: 25 %, with spills).
// A block barrier that waves with different roles reach at different places
// of the code: every wave of the block meets the same number of them, in the
// same order (the role is uniform over a wave, and the hardware counts waves).
__device__ __forceinline__ void role_barrier() { __syncthreads(); }

// The edge waves of a tile: group 1..NG of the block's groups of four.
template <int P, typename Real, int NG>
__device__ __forceinline__ void tile_edges(StepLds<P, Real, true> &T, const StageArgs<Real> &a,
                                           const TileView &tv, int tile, int group, double xh0, double xh1)
{
    const MeshView &m = a.m;
    const int KS = m.KS, l = (int)threadIdx.x & (BLOCK - 1), it0 = l + (group > 1 ? BLOCK : 0);
    const Buf<Real> bC(a.Cin, 3 * KS, m.stride), bU(a.Uin, 2 * KS, m.stride);
    const double g = a.ph.g;
    const int *meta = tv.meta + (size_t)tile * BLOCK;
    const unsigned w0 = tv.items[(size_t)tile * (2 * BLOCK) + it0];
    const unsigned w1 = NG == 1 ? tv.items[(size_t)tile * (2 * BLOCK) + it0 + BLOCK] : ITEM_PAD;
    if (group == NG) T.tri[l] = tv.tri[(size_t)tile * BLOCK + l];
    if (group == 1 && l < TILE_NV) {
        const int v = tv.verts[(size_t)tile * TILE_NV + l];
        if (v >= 0) {
            const double4 p = m.vtx[(unsigned)v];
            T.vx[l] = p.x;
            T.vy[l] = p.y;
            T.vh[l] = p.z;
        }
    }
    int x0 = 0, x1 = 0;
    if (w0 != ITEM_PAD && ((w0 >> 20) & 3u) == EK_EXT) x0 = meta[(w0 >> 10) & 255u];
    if (w1 != ITEM_PAD && ((w1 >> 20) & 3u) == EK_EXT) x1 = meta[(w1 >> 10) & 255u];
    role_barrier();
#pragma unroll
    for (int st = 0; st < 2; ++st) {
        const double xihat = st ? xh1 : xh0;
        const bool use0 = w0 != ITEM_PAD && !(st && (w0 & ITEM_RING));
        const bool use1 = w1 != ITEM_PAD && !(st && (w1 & ITEM_RING));
        ShItem<P, Real> r;
        if (use0) {
            sh_flux<P, Real, true>(T.S, KS, bC, bU, TileSrc<P, Real, true>{T, x0}, w0, xihat, g, r);
            sh_store<P, Real, true>(T.S, it0, w0, r);
        }
        if (use1) {
            sh_flux<P, Real, true>(T.S, KS, bC, bU, TileSrc<P, Real, true>{T, x1}, w1, xihat, g, r);
            sh_store<P, Real, true>(T.S, it0 + BLOCK, w1, r);
        }
        role_barrier();                     // the fluxes are in place, the state copies read
        if (st == 0) role_barrier();        // the first stage's state is in place
    }
}

// The element waves of a tile.
template <int P, typename Real>
__device__ __forceinline__ void tile_elements(StepLds<P, Real, true> &T, const StageArgs<Real> &a,
                                              const TileView &tv, int tile, unsigned e0, int nown, double dt, int *flag)
{
    constexpr int K = Ord<P>::K;
    const MeshView &m = a.m;
    const int KS = m.KS, stride = m.stride, l = (int)threadIdx.x & (BLOCK - 1);
    const Buf<Real> bC(a.Cin, 3 * KS, stride), bU(a.Uin, 2 * KS, stride);
    const double g = a.ph.g;
    // a lane past the ring repeats the tile's first element, as in step_tile
    const int id = l < nown ? (int)e0 + l : tv.meta[(size_t)tile * BLOCK + l];
    const int lx = id >= 0 ? l : 0;
    const unsigned off = (id >= 0 ? (unsigned)id : e0) * (unsigned)sizeof(Real);
    Fields<P, Real> s;
    load_state<P, Real>(bC, bU, KS, off, s);
    sh_copy_state<P, Real, true>(T.S, l, s);
    role_barrier();
#pragma unroll
    for (int st = 0; st < 2; ++st) {
        Geo G;
        tile_geo<P, Real, true>(T, lx, G);
        double hbh[3];
        hb_modes(G, hbh);
        Acc<P, Real> A;
        Real cn[3][K];   // c^n for the second stage, under way while the edges are lifted
        acc_init<P, Real>(A, s, true);
        volume_term<P, Real>(s, hbh, G, g, dt, A);
        source_term<P, Real>(s, G, a.ph, dt, A);
        if (st) {
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int q = 0; q < K; ++q) cn[j][q] = bC.ld(j * KS + q, off);
        }
        role_barrier();                     // the fluxes are in place
        if (st && l >= nown) return;         // (no barrier follows)
        sh_lift<P, Real, true>(T.S, G, lx, dt, A);
        if constexpr (Acc<P, Real>::SPLIT) {
#pragma unroll
            for (int q = 0; q < K; ++q) {
                A.L[1][q] += Real(A.W[0][q]);
                A.L[2][q] += Real(A.W[1][q]);
            }
        }
        if (a.src) {
            const Buf<Real> bS(a.src, 3 * KS, stride);
            const Real rdt = Real(dt);
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int q = 0; q < K; ++q) A.L[j][q] = fma(rdt, bS.ld(j * KS + q, off), A.L[j][q]);
        }
        if (st) {
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int q = 0; q < K; ++q) A.L[j][q] = Real(0.5) * cn[j][q] + Real(0.5) * A.L[j][q];
        }
        solve_u<P, Real>(A.L[0], A.L[1], A.L[2], hbh, K, s.u, s.v);
        Real chk = 0;
#pragma unroll
        for (int q = 0; q < K; ++q) {
            s.xi[q] = A.L[0][q];
            s.U[q] = A.L[1][q];
            s.V[q] = A.L[2][q];
            chk += s.xi[q] + s.U[q] + s.V[q] + s.u[q] + s.v[q];
        }
        const double Hmean = SQRT2 * double(s.xi[0]) + (G.h[0] + G.h[1] + G.h[2]) * (1.0 / 3.0);
        if (!(Hmean > 0.0) || !isfinite(chk)) flag[0] = 1;
        if (st == 0) {
            sh_copy_state<P, Real, true>(T.S, l, s);
            role_barrier();
        }
    }
    (void)store_state<P, Real, CPOL_THROUGH>(a, off, s.xi, s.U, s.V, s.u, s.v);
}

// flux groups of the kernel with roles for at most one tile per CU; 0: not built
template <int P, typename Real>
constexpr int flux_groups()
{
    return sizeof(Real) == 4 || P == 1 ? 2 : P == 2 ? 1 : 0;
}

template <int P, typename Real, int NG>
__global__ void __launch_bounds__((1 + NG) * BLOCK) __attribute__((amdgpu_waves_per_eu(1 + NG, 8)))
k_step_roles(StageArgs<Real> a, TileView tv, double xihat2)
{
    __shared__ StepLds<P, Real, true> T;
    load_trace_lds<P, Real, true>(T.S);
    double xh0 = a.xihat, xh1 = xihat2, dt = a.dt;
    if (a.inst) {
        // the step's clock stopped (failure); uniform over the block
        if (!a.inst->run) return stopped_step<P, Real>(a, tv.len);
        xh0 = a.inst->xh[0];
        xh1 = a.inst->xh[1];
        dt = a.inst->dt;
    }
    const int tile = xcd_block(blockIdx.x, gridDim.x);
    const int e0 = tile * tv.len, left = a.m.ne - e0;
    const int group = __builtin_amdgcn_readfirstlane((int)threadIdx.x / BLOCK);
    if (group)
        tile_edges<P, Real, NG>(T, a, tv, tile, group, xh0, xh1);
    else
        tile_elements<P, Real>(T, a, tv, tile, (unsigned)e0, left < tv.len ? left : tv.len, dt, a.flag);
}

// ---- tile data, one block per tile
// ascending sort of N keys (a power of two) in LDS by the whole block
template <int N>
__device__ __forceinline__ void block_sort(int *key)
{
    for (int w = 2; w <= N; w <<= 1)
        for (int d = w >> 1; d > 0; d >>= 1) {
            __syncthreads();
            for (int i = threadIdx.x; i < N; i += BLOCK) {
                const int j = i ^ d;
                if (j > i) {
                    const int x = key[i], y = key[j];
                    if ((x > y) == ((i & w) == 0)) {
                        key[i] = y;
                        key[j] = x;
                    }
                }
            }
        }
    __syncthreads();
}

// exclusive prefix sum over the block's threads; *total the sum
__device__ __forceinline__ int block_scan(int v, int *buf, int *total)
{
    const int t = (int)threadIdx.x;
    buf[t] = v;
    __syncthreads();
    for (int d = 1; d < BLOCK; d <<= 1) {
        const int x = t >= d ? buf[t - d] : 0;
        __syncthreads();
        buf[t] += x;
        __syncthreads();
    }
    const int r = buf[t] - v;
    *total = buf[BLOCK - 1];
    __syncthreads();
    return r;
}

// the distinct keys below INT_MAX of a sorted array of N, in order: at most
// max of them to out; returns how many there are
template <int N>
__device__ __forceinline__ int block_unique(const int *key, int *out, int max, int *buf)
{
    constexpr int PER = N / BLOCK;
    const int b = (int)threadIdx.x * PER;
    int n = 0, total;
    for (int i = b; i < b + PER; ++i) n += key[i] != INT_MAX && (i == 0 || key[i] != key[i - 1]);
    int at = block_scan(n, buf, &total);
    for (int i = b; i < b + PER; ++i)
        if (key[i] != INT_MAX && (i == 0 || key[i] != key[i - 1])) {
            if (at < max) out[at] = key[i];
            ++at;
        }
    __syncthreads();
    return total;
}

__device__ __forceinline__ int find_sorted(const int *a, int n, int v)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < v) lo = mid + 1;
        else hi = mid;
    }
    return lo < n && a[lo] == v ? lo : -1;
}

// Tile data of the mesh arrays' ne elements in tiles of tv.len, one block per
// tile.  over[0] gets the most lanes by which a tile is beyond a block
// (elements, or half its excess edge items), over[1] is set when it does not
// fit for another reason (vertices, outside neighbours).
__global__ void __launch_bounds__(BLOCK) k_build_tiles(MeshView m, int ne, TileView tv, int *over)
{
    __shared__ int key[4 * BLOCK], ring[BLOCK], vert[TILE_NV], buf[BLOCK], ncand;
    __shared__ unsigned items[2 * BLOCK];
    __shared__ int meta[BLOCK];
    const int t = (int)threadIdx.x, e0 = (int)blockIdx.x * tv.len, e1 = e0 + tv.len < ne ? e0 + tv.len : ne;
    const int nown = e1 - e0;
    const size_t tile = blockIdx.x;
    // the ring: neighbours of owned elements outside the tile
    if (t == 0) ncand = 0;
    key[t] = INT_MAX;
    __syncthreads();
    if (t < nown)
        for (int k = 0; k < 3; ++k) {
            const int n = m.enb[k * m.stride + e0 + t];
            if (n >= 0 && (n < e0 || n >= e1)) {
                const int i = atomicAdd(&ncand, 1);
                if (i < BLOCK) key[i] = n;
            }
        }
    __syncthreads();
    bool fits = ncand <= BLOCK;
    int excess = 0;
    block_sort<BLOCK>(key);
    int nr = block_unique<BLOCK>(key, ring, BLOCK, buf);
    if (nown + nr > BLOCK) {
        excess = nown + nr - BLOCK;
        nr = BLOCK - nown;
    }
    const int nloc = nown + nr;
    const int e = t < nown ? e0 + t : t < nloc ? ring[t - nown] : -1;
    // the tile's vertices
    for (int i = t; i < 4 * BLOCK; i += BLOCK) key[i] = INT_MAX;
    __syncthreads();
    int ids[3] = {0, 0, 0};
    if (e >= 0)
        for (int v = 0; v < 3; ++v) {
            ids[v] = m.ev[v * m.stride + e];
            key[3 * t + v] = ids[v];
        }
    block_sort<4 * BLOCK>(key);
    int nv = block_unique<4 * BLOCK>(key, vert, TILE_NV, buf);
    if (nv > TILE_NV) {
        fits = false;
        nv = TILE_NV;
    }
    unsigned tri = 0;
    if (e >= 0)
        for (int v = 0; v < 3; ++v) tri |= (unsigned)(find_sorted(vert, nv, ids[v]) & 255) << (8 * v);
    // edge items by class: those that touch an owned element (pairs, land,
    // open), then the ring's own (pairs, outside neighbours, land, open);
    // within a class local edge by local edge, so that consecutive lanes read
    // consecutive elements and the same trace matrix
    int cls[3], pos[3], other[3];
    unsigned word[3];
    const unsigned nbk = e >= 0 ? m.enbk[e] : 0u;
    for (int k = 0; k < 3; ++k) {
        cls[k] = -1;
        pos[k] = other[k] = 0;
        word[k] = 0;
        if (e < 0) continue;
        const int n = m.enb[k * m.stride + e];
        const int kb = (int)(nbk >> (2 * k)) & 3;
        const bool own = t < nown;
        unsigned kind, lb = 0;
        if (n >= 0) {
            int q = n >= e0 && n < e1 ? n - e0 : find_sorted(ring, nr, n);
            if (q >= 0 && (n < e0 || n >= e1)) q += nown;
            if (q >= 0) {
                if (q < t) continue;           // the pair is taken from the lower local index
                kind = EK_PAIR;
                lb = (unsigned)q;
                cls[k] = own ? 0 : 3;
            } else {
                kind = EK_EXT;
                other[k] = n;
                cls[k] = 4;
            }
        } else {
            kind = n == NB_LAND ? EK_LAND : EK_OPEN;
            cls[k] = (own ? 1 : 5) + (kind == EK_OPEN ? 1 : 0);
        }
        word[k] = (unsigned)t | ((unsigned)k << 8) | (lb << 10) | ((unsigned)kb << 18) | (kind << 20) |
                  (cls[k] >= 3 ? ITEM_RING : 0u);
    }
    int tot[7];
    for (int c = 0; c < 7; ++c) {
        int run = 0;
        for (int k = 0; k < 3; ++k) {
            int n;
            const int r = block_scan(cls[k] == c ? 1 : 0, buf, &n);
            if (cls[k] == c) pos[k] = run + r;
            run += n;
        }
        tot[c] = run;
    }
    // each class starts on a wave boundary while the tile then still fits
    int padded = 0, plain = 0;
    for (int c = 0; c < 7; ++c)
        if (tot[c]) {
            padded = (padded + 63) / 64 * 64 + tot[c];
            plain += tot[c];
        }
    const bool align = padded <= 2 * BLOCK;
    if (plain > 2 * BLOCK && (plain - 2 * BLOCK + 1) / 2 > excess) excess = (plain - 2 * BLOCK + 1) / 2;
    if (tot[4] > nown) fits = false;
    for (int i = t; i < 2 * BLOCK; i += BLOCK) items[i] = ITEM_PAD;
    meta[t] = t >= nown ? e : -1;
    __syncthreads();
    int base = 0;
    for (int c = 0; c < 7; ++c) {
        if (!tot[c]) continue;
        if (align) base = (base + 63) / 64 * 64;
        for (int k = 0; k < 3; ++k)
            if (cls[k] == c && base + pos[k] < 2 * BLOCK) {
                unsigned w = word[k];
                if (c == 4 && pos[k] < nown) {   // outside neighbours' ids sit in the owned elements' slots
                    meta[pos[k]] = other[k];
                    w |= (unsigned)pos[k] << 10;
                }
                items[base + pos[k]] = w;
            }
        base += tot[c];
    }
    __syncthreads();
    for (int i = t; i < 2 * BLOCK; i += BLOCK) tv.items[tile * (2 * BLOCK) + i] = items[i];
    tv.meta[tile * BLOCK + t] = meta[t];
    tv.tri[tile * BLOCK + t] = tri;
    if (t < TILE_NV) tv.verts[tile * TILE_NV + t] = t < nv ? vert[t] : -1;
    if (t == 0 && excess > 0) atomicMax(&over[0], excess);
    if (t == 0 && !fits) over[1] = 1;
}

}  // namespace

// flux groups of the kernel that `tiles` tiles take on ncu compute units; 0: one
// group of waves for everything
template <int P, typename Real>
int step_groups(int tiles, int ncu)
{
    if (tiles <= ncu && flux_groups<P, Real>() > 0) return flux_groups<P, Real>();
    // order 1: two blocks of one flux group each share a CU
    return P == 1 && tiles <= 2 * ncu ? 1 : 0;
}

template <int P, typename Real>
hipError_t step_sh_p(const void *args, const TileView &tv, double xihat2, int ncu, Sink &k)
{
    StageArgs<Real> a = *static_cast<const StageArgs<Real> *>(args);
    TileView t = tv;
    void *kargs[] = {&a, &t, &xihat2};
    const dim3 grid((a.m.ne + t.len - 1) / t.len);
    constexpr int ng = flux_groups<P, Real>();
    const int groups = step_groups<P, Real>((int)grid.x, ncu);
    if constexpr (ng > 0) {
        if (groups == ng)
            return emit(k, reinterpret_cast<const void *>(&k_step_roles<P, Real, ng>), grid, dim3((1 + ng) * BLOCK),
                        kargs);
    }
    if constexpr (P == 1) {
        if (groups == 1)
            return emit(k, reinterpret_cast<const void *>(&k_step_roles<P, Real, 1>), grid, dim3(2 * BLOCK), kargs);
    }
    return emit(k, reinterpret_cast<const void *>(&k_step_sh<P, Real>), grid, dim3(BLOCK), kargs);
}

hipError_t launch_step_sh(int p, bool fp32, const void *args, const TileView &tv, double xihat2, int ncu, Sink &k)
{
    if (tv.len <= 0) return hipErrorInvalidValue;
    switch (p) {
    case 1: return fp32 ? step_sh_p<1, float>(args, tv, xihat2, ncu, k) : step_sh_p<1, double>(args, tv, xihat2, ncu, k);
    case 2: return fp32 ? step_sh_p<2, float>(args, tv, xihat2, ncu, k) : step_sh_p<2, double>(args, tv, xihat2, ncu, k);
    case 3: return fp32 ? step_sh_p<3, float>(args, tv, xihat2, ncu, k) : step_sh_p<3, double>(args, tv, xihat2, ncu, k);
    }
    return hipErrorInvalidValue;
}

int step_flux_groups(int p, bool fp32, int tiles, int ncu)
{
    switch (p) {
    case 1: return fp32 ? step_groups<1, float>(tiles, ncu) : step_groups<1, double>(tiles, ncu);
    case 2: return fp32 ? step_groups<2, float>(tiles, ncu) : step_groups<2, double>(tiles, ncu);
    case 3: return fp32 ? step_groups<3, float>(tiles, ncu) : step_groups<3, double>(tiles, ncu);
    }
    return 0;
}

hipError_t launch_build_tiles(const MeshView &m, int ne, const TileView &tv, int *over, hipStream_t s)
{
    if (ne <= 0) return hipSuccess;
    if (tv.len <= 0 || tv.len > BLOCK) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_build_tiles, dim3((ne + tv.len - 1) / tv.len), dim3(BLOCK), 0, s, m, ne, tv, over);
    return hipGetLastError();
}

}  // namespace swe
