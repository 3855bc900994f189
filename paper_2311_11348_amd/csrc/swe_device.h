// Device code shared by the gfx950 kernel files: the element code of the
// quadrature-free DG right-hand side (see swe_kernels.hip for the method) and
// the passes of the shared-flux kernels.  Everything has internal linkage.
#pragma once

#include "swe_internal.h"
#include "swe_tables.h"

#include <climits>
#include <type_traits>

namespace swe {
namespace {

constexpr double TC[10][10][10] = SWET_C;
constexpr double TD[2][10][10] = SWET_D;
constexpr double TR[3][10][4] = SWET_R;
constexpr double TG[4][4][4] = SWET_G;
constexpr double TW[3][3] = SWET_W;
constexpr double TPMID[3][3] = SWET_PMID;
constexpr double TCHK[6][10] = SWET_PCHK;
constexpr int TDEG[10] = SWET_DEG;
constexpr int KOFP[4] = SWET_K_OF_P;
constexpr double SQRT2 = 1.41421356237309504880;
constexpr double INV_2SQRT3 = 0.28867513459481288225;  // 1 / (2 sqrt 3)

// Minimum resident waves per SIMD the register allocator must allow for the
// stage kernel (more waves hide memory latency; fewer avoid spills).
#ifndef SWE_WAVES_FP64
#define SWE_WAVES_FP64 1
#endif
#ifndef SWE_WAVES_FP32
#define SWE_WAVES_FP32 2
#endif
#ifndef SWE_WAVES_FP32_P3
#define SWE_WAVES_FP32_P3 1
#endif
template <int P, typename Real>
constexpr int waves_target()
{
    // Order 3 needs more than 256 registers per lane: one wave (the
    // accumulation registers then serve as spill space; no kernel loops
    // around such an evaluation, which gave run-to-run differences).
    return P >= 3 ? (std::is_same<Real, double>::value ? 1 : SWE_WAVES_FP32_P3)
                  : P <= 1 ? 2 : (std::is_same<Real, double>::value ? SWE_WAVES_FP64 : SWE_WAVES_FP32);
}

template <int P>
struct Ord {
    static constexpr int K = (P + 1) * (P + 2) / 2;   // modes of P^p
    static constexpr int KM = P * (P + 1) / 2;        // modes of P^{p-1}
    static constexpr int NT = P + 1;                  // Legendre modes of a trace
};

__device__ __forceinline__ int xcd_block(int b, int nb)
{
    // Workgroups are dispatched round-robin over the 8 XCDs.  Give each XCD a
    // contiguous range of element tiles so that neighbour gathers hit its L2.
    const int q = nb >> 3, r = nb & 7;
    const int x = b & 7, i = b >> 3;
    return x * q + (x < r ? x : r) + i;
}

// The element code below is compiled for the host as well: the order-separated
// scheme's correction can run on the CPU beside the GPU's base pass (the
// heterogeneous stage).  Only the element-indexed loads and stores differ.
#define SWE_HD __host__ __device__ __forceinline__

template <typename T>
SWE_HD T tmax(T a, T b) { return a > b ? a : b; }

// FP32 reciprocal and square root by the hardware's single-instruction
// approximations (about 1 ulp) instead of the correctly rounded sequences
// (ten and more instructions each).  Used on FP32 data only, where the
// argument is a positive, well-scaled quantity: the pivots of the depth
// matrix H, the squared wave speed of the penalty, the squared velocity of
// the quadratic friction.  The host build (the heterogeneous stage) rounds
// correctly.
SWE_HD float rcp_approx(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_rcpf(x);
#else
    return 1.0f / x;
#endif
}

SWE_HD float sqrt_approx(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_sqrtf(x);
#else
    return std::sqrt(x);
#endif
}

// Element-indexed arrays are read and written through buffer resources: a
// uniform descriptor (base, byte size) in scalar registers, a uniform byte
// offset per (component, mode) slot and one 32-bit lane offset, so no load
// needs per-lane 64-bit address arithmetic, and an access beyond the array
// (which the host never issues) reads 0 instead of faulting.
constexpr int RSRC_WORD3 = 0x00020000;   // raw 32-bit access, gfx9 family
typedef unsigned int u32x2 __attribute__((__vector_size__(8)));
// cache-policy operands of a buffer access (gfx94x/gfx950): the non-temporal
// bit; the system-scope bit, with which a store is written through the caches
constexpr int CPOL_NT = 2, CPOL_THROUGH = 16;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes, RSRC_WORD3);
}

template <typename T>
struct Buf {
#if defined(__HIP_DEVICE_COMPILE__)
    __amdgpu_buffer_rsrc_t r;
#else
    // on the host: the array and its size, with the same out-of-range
    // behaviour (loads read 0, stores are dropped)
    char *base;
    unsigned size;
#endif
    int slot_bytes;
    SWE_HD Buf(const T *p, int nslots, int stride)
#if defined(__HIP_DEVICE_COMPILE__)
        : r(make_rsrc(p, (unsigned)nslots * (unsigned)stride * (unsigned)sizeof(T))),
#else
        : base(reinterpret_cast<char *>(const_cast<T *>(p))),
          size((unsigned)nslots * (unsigned)stride * (unsigned)sizeof(T)),
#endif
          slot_bytes(stride * (int)sizeof(T)) {}
    // off = element index * sizeof(T)
    SWE_HD T ld(int slot, unsigned off) const
    {
#if defined(__HIP_DEVICE_COMPILE__)
        if constexpr (sizeof(T) == 8)
            return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, slot * slot_bytes, 0));
        else
            return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, slot * slot_bytes, 0));
#else
        const unsigned at = off + (unsigned)(slot * slot_bytes);
        if (!base || at + sizeof(T) > size) return T(0);
        T v;
        __builtin_memcpy(&v, base + at, sizeof(T));
        return v;
#endif
    }
    // a store with a cache policy of its own, for results no block of the same
    // launch reads back
    template <int CPOL>
    SWE_HD void st_policy(int slot, unsigned off, T v) const
    {
#if defined(__HIP_DEVICE_COMPILE__)
        if constexpr (sizeof(T) == 8)
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)off,
                                                  slot * slot_bytes, CPOL);
        else
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)off,
                                                  slot * slot_bytes, CPOL);
#else
        st(slot, off, v);
#endif
    }
    SWE_HD void st(int slot, unsigned off, T v) const
    {
#if defined(__HIP_DEVICE_COMPILE__)
        if constexpr (sizeof(T) == 8)
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)off,
                                                  slot * slot_bytes, 0);
        else
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)off,
                                                  slot * slot_bytes, 0);
#else
        const unsigned at = off + (unsigned)(slot * slot_bytes);
        if (base && at + sizeof(T) <= size) __builtin_memcpy(base + at, &v, sizeof(T));
#endif
    }
};

struct Geo {
    double b00, b01, b10, b11;   // inverse Jacobian: d(xh)/dx, d(xh)/dy, d(yh)/dx, d(yh)/dy
    double det;                  // |det B_e| = 2 area
    double idet;                 // 1 / |det B_e|
    double X[3], Y[3], h[3];     // vertices and depths
};

// The inverse Jacobian and determinant from the vertices in G.
SWE_HD void geo_finish(Geo &G)
{
    const double a00 = G.X[1] - G.X[0], a01 = G.X[2] - G.X[0];
    const double a10 = G.Y[1] - G.Y[0], a11 = G.Y[2] - G.Y[0];
    G.det = a00 * a11 - a01 * a10;
    const double id = 1.0 / G.det;
    G.idet = id;
    G.b00 = a11 * id;
    G.b01 = -a01 * id;
    G.b10 = -a10 * id;
    G.b11 = a00 * id;
}

// Geometry from the element's vertex ids (already loaded).
SWE_HD void geo_from_ids(const double4 *vtx, const int (&id3)[3], Geo &G)
{
#pragma unroll
    for (int v = 0; v < 3; ++v) {
        const double4 p = vtx[(unsigned)id3[v]];
        G.X[v] = p.x;
        G.Y[v] = p.y;
        G.h[v] = p.z;
    }
    geo_finish(G);
}

SWE_HD void load_geo(const double4 *vtx, const Buf<int> &ev, unsigned offi, Geo &G)
{
    const int id3[3] = {ev.ld(0, offi), ev.ld(1, offi), ev.ld(2, offi)};
    geo_from_ids(vtx, id3, G);
}

template <int P, typename Real>
struct Fields {
    static constexpr int K = Ord<P>::K;
    Real xi[K], U[K], V[K], u[K], v[K];
};

template <int P, typename Real>
SWE_HD void load_state(const Buf<Real> &C, const Buf<Real> &Uv, int KS, unsigned off,
                                           Fields<P, Real> &s)
{
    constexpr int K = Ord<P>::K;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        s.xi[i] = C.ld(0 * KS + i, off);
        s.U[i] = C.ld(1 * KS + i, off);
        s.V[i] = C.ld(2 * KS + i, off);
        s.u[i] = Uv.ld(0 * KS + i, off);
        s.v[i] = Uv.ld(1 * KS + i, off);
    }
}

// t_i = sum_j C[m][i][j] g_j with the zero pattern folded at compile time
template <int K, typename T, typename S>
SWE_HD T crow(int m, int i, const S (&g)[K])
{
    T t = T(0);
#pragma unroll
    for (int j = 0; j < K; ++j)
        if (TC[m][i][j] != 0.0) t = fma(T(TC[m][i][j]), T(g[j]), t);
    return t;
}

template <int K>
SWE_HD constexpr bool crow_nonzero(int m, int i)
{
    bool any = false;
    for (int j = 0; j < K; ++j) any = any || (TC[m][i][j] != 0.0);
    return any;
}

// ------------------------------------------------------------ accumulator
// acc = c + dt * L(c), built term by term (every geometric factor carries dt).
// Bathymetry terms go to W: FP64 always; for Real = double W is the momentum
// rows of L itself, for Real = float a separate FP64 array added at the end.
template <int P, typename Real>
struct Acc {
    static constexpr int K = Ord<P>::K;
    static constexpr bool SPLIT = !std::is_same<Real, double>::value;
    Real L[3][K];
    double W[SPLIT ? 2 : 1][SPLIT ? K : 1];
    SWE_HD double &w(int j, int q)
    {
        if constexpr (SPLIT) return W[j][q];
        else return L[1 + j][q];
    }
};

// ------------------------------------------------------------ volume term
// acc[j][q] += dt sum_k sum_m D[k][q][m] (Bi_kx F^j_x,m + Bi_ky F^j_y,m), over the
// projected modes M0 <= m < M1 (all of them by default)
template <int P, typename Real, int M0 = 0, int M1 = Ord<P>::KM>
SWE_HD void volume_term(const Fields<P, Real> &s, const double (&hbh)[3],
                                            const Geo &G, double g, double dt, Acc<P, Real> &A)
{
    constexpr int K = Ord<P>::K, KM = Ord<P>::KM;
    if constexpr (KM > 0 && M0 < M1) {
        Real Fx[3][KM], Fy[3][KM];
        double FW[KM];
        const Real hg = Real(0.5 * g);
#pragma unroll
        for (int m = M0; m < M1; ++m) {
            Real pUu = 0, pUv = 0, pVu = 0, pVv = 0, pxx = 0;
            double pxh = 0.0;
#pragma unroll
            for (int i = 0; i < K; ++i) {
                if (!crow_nonzero<K>(m, i)) continue;
                const Real tu = crow<K, Real>(m, i, s.u);
                const Real tv = crow<K, Real>(m, i, s.v);
                const Real tx = crow<K, Real>(m, i, s.xi);
                pUu = fma(s.U[i], tu, pUu);
                pUv = fma(s.U[i], tv, pUv);
                pVu = fma(s.V[i], tu, pVu);
                pVv = fma(s.V[i], tv, pVv);
                pxx = fma(s.xi[i], tx, pxx);
                double th = 0.0;
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    if (TC[m][i][j] != 0.0) th = fma(TC[m][i][j], hbh[j], th);
                pxh = fma(double(s.xi[i]), th, pxh);
            }
            Fx[0][m] = s.U[m];
            Fy[0][m] = s.V[m];
            Fx[1][m] = fma(hg, pxx, pUu);
            Fy[1][m] = pUv;
            Fx[2][m] = pVu;
            Fy[2][m] = fma(hg, pxx, pVv);
            FW[m] = g * dt * pxh;
        }
        const Real b00 = Real(G.b00 * dt), b01 = Real(G.b01 * dt);
        const Real b10 = Real(G.b10 * dt), b11 = Real(G.b11 * dt);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            Real G0[KM], G1[KM];
#pragma unroll
            for (int m = M0; m < M1; ++m) {
                G0[m] = fma(b00, Fx[j][m], b01 * Fy[j][m]);
                G1[m] = fma(b10, Fx[j][m], b11 * Fy[j][m]);
            }
#pragma unroll
            for (int q = 0; q < K; ++q) {
                Real acc = A.L[j][q];
#pragma unroll
                for (int m = M0; m < M1; ++m) {
                    if (TD[0][q][m] != 0.0) acc = fma(Real(TD[0][q][m]), G0[m], acc);
                    if (TD[1][q][m] != 0.0) acc = fma(Real(TD[1][q][m]), G1[m], acc);
                }
                A.L[j][q] = acc;
            }
        }
        // bathymetry part of the pressure: x-momentum uses Bi_kx, y-momentum Bi_ky
        double Wx[KM], Wy[KM], Zx[KM], Zy[KM];
#pragma unroll
        for (int m = M0; m < M1; ++m) {
            Wx[m] = G.b00 * FW[m];
            Wy[m] = G.b01 * FW[m];
            Zx[m] = G.b10 * FW[m];
            Zy[m] = G.b11 * FW[m];
        }
#pragma unroll
        for (int q = 0; q < K; ++q) {
            double ax = A.w(0, q), ay = A.w(1, q);
#pragma unroll
            for (int m = M0; m < M1; ++m) {
                if (TD[0][q][m] != 0.0) {
                    ax = fma(TD[0][q][m], Wx[m], ax);
                    ay = fma(TD[0][q][m], Wy[m], ay);
                }
                if (TD[1][q][m] != 0.0) {
                    ax = fma(TD[1][q][m], Zx[m], ax);
                    ay = fma(TD[1][q][m], Zy[m], ay);
                }
            }
            A.w(0, q) = ax;
            A.w(1, q) = ay;
        }
    }
}

// ------------------------------------------------------------ source term
template <int P, typename Real>
SWE_HD void source_term(const Fields<P, Real> &s, const Geo &G, const Physics &ph,
                                            double dt, Acc<P, Real> &A)
{
    constexpr int K = Ord<P>::K;
    const double dh1 = G.h[1] - G.h[0], dh2 = G.h[2] - G.h[0];
    const double gx = ph.g * dt * (G.b00 * dh1 + G.b10 * dh2);   // dt g dh_b/dx
    const double gy = ph.g * dt * (G.b01 * dh1 + G.b11 * dh2);   // dt g dh_b/dy
    const Real fc = Real(ph.fc * dt);
    Real tau = 0;
    if (ph.friction == 2) {
        // |constant part of u| = sqrt(2) |(u_0, v_0)| in reference-scaled modes
        const Real um = s.u[0], vm = s.v[0];
        if constexpr (std::is_same<Real, double>::value)
            tau = Real(ph.fric * dt * SQRT2) * sqrt(um * um + vm * vm);
        else
            tau = Real(ph.fric * dt * SQRT2) * sqrt_approx(um * um + vm * vm);
    } else if (ph.friction == 1) {
        tau = Real(ph.fric * dt);
    }
#pragma unroll
    for (int q = 0; q < K; ++q) {
        Real a1 = fma(fc, s.V[q], A.L[1][q]);
        Real a2 = fma(-fc, s.U[q], A.L[2][q]);
        if (ph.friction == 2) {
            a1 = fma(-tau, s.u[q], a1);
            a2 = fma(-tau, s.v[q], a2);
        } else if (ph.friction == 1) {
            a1 = fma(-tau, s.U[q], a1);
            a2 = fma(-tau, s.V[q], a2);
        }
        A.L[1][q] = a1;
        A.L[2][q] = a2;
        A.w(0, q) = fma(gx, double(s.xi[q]), A.w(0, q));
        A.w(1, q) = fma(gy, double(s.xi[q]), A.w(1, q));
    }
}

// ------------------------------------------------------------ edge terms
// trace on a local edge in Legendre modes: t_a = sum_n f_n R[k][n][a]
template <int P, typename Real>
SWE_HD void trace_own(int k, const Real (&f)[Ord<P>::K], Real (&t)[Ord<P>::NT])
{
    constexpr int K = Ord<P>::K, NT = Ord<P>::NT;
#pragma unroll
    for (int a = 0; a < NT; ++a) {
        Real acc = 0;
#pragma unroll
        for (int n = 0; n < K; ++n)
            if (TR[k][n][a] != 0.0) acc = fma(f[n], Real(TR[k][n][a]), acc);
        t[a] = acc;
    }
}

// 1D product projected onto Legendre modes c <= P: out_c = sum_ab G[c][a][b] f_a g_b
template <int NT, typename T>
SWE_HD T prod1(int c, const T (&f)[NT], const T (&g)[NT])
{
    T acc = 0;
#pragma unroll
    for (int a = 0; a < NT; ++a) {
        T t = 0;
        bool any = false;
#pragma unroll
        for (int b = 0; b < NT; ++b)
            if (TG[c][a][b] != 0.0) {
                t = fma(T(TG[c][a][b]), g[b], t);
                any = true;
            }
        if (any) acc = fma(f[a], t, acc);
    }
    return acc;
}

// Edge terms of one element of order P whose neighbours have order <= PN
// (their stored modes above their own order are zero).  Both traces are
// expanded to NX = max(P, PN) + 1 Legendre modes; the flux is projected onto
// the own test space (modes <= P).
// The edge term of local edge k (its flux lifted onto the element's modes).
template <int P, int PN, typename Real, int k>
SWE_HD void edge_one(const MeshView &m, unsigned e, const Buf<Real> &bC, const Buf<Real> &bU,
                     const Buf<int> &bNb, const Fields<P, Real> &s, const Geo &G, double g, double xihat,
                     double dt, const Real (*sR)[Ord<PN>::K][(P > PN ? P : PN) + 1], Acc<P, Real> &A)
{
    constexpr int K = Ord<P>::K, NT = Ord<P>::NT, KN = Ord<PN>::K;
    constexpr int NX = (P > PN ? P : PN) + 1;
    const int KS = m.KS;
    const unsigned nbk_all = m.enbk[e];
    const Real xbm = Real(SQRT2) * s.xi[0];
    const Real ubm = Real(SQRT2) * s.u[0], vbm = Real(SQRT2) * s.v[0];
    // With the edge vector's normal nu = |E| n (no square root), every flux
    // term carries |E| n or |E| lambda, and |E| / |det B| folds into dt / |det B|.
    const double dt_det = dt * G.idet;
    {
        constexpr int ka = (k + 1) % 3, kb = (k + 2) % 3;
        const double dx = G.X[kb] - G.X[ka], dy = G.Y[kb] - G.Y[ka];
        const double len2 = dx * dx + dy * dy;
        const Real nx = Real(dy), ny = Real(-dx);          // |E| n
        const double hmid = 0.5 * (G.h[ka] + G.h[kb]);
        const double hbt[2] = {hmid, (G.h[kb] - G.h[ka]) * INV_2SQRT3};

        Real txm[NX], tUm[NX], tVm[NX], unm[NX], qnm[NX];
        {
            Real tx[NT], tU[NT], tV[NT], tu[NT], tv[NT];
            trace_own<P, Real>(k, s.xi, tx);
            trace_own<P, Real>(k, s.U, tU);
            trace_own<P, Real>(k, s.V, tV);
            trace_own<P, Real>(k, s.u, tu);
            trace_own<P, Real>(k, s.v, tv);
#pragma unroll
            for (int a = 0; a < NT; ++a) {
                txm[a] = tx[a];
                tUm[a] = tU[a];
                tVm[a] = tV[a];
                unm[a] = fma(tu[a], nx, tv[a] * ny);
                qnm[a] = fma(tU[a], nx, tV[a] * ny);
            }
#pragma unroll
            for (int a = NT; a < NX; ++a) {
                txm[a] = 0; tUm[a] = 0; tVm[a] = 0; unm[a] = 0; qnm[a] = 0;
            }
        }

        const int nb = bNb.ld(k, e * 4u);
        Real txp[NX], tUp[NX], tVp[NX], unp[NX], qnp[NX];
        Real xbp, unbp;
        const Real unbm = fabs(fma(ubm, nx, vbm * ny));
        if (nb >= 0) {
            const int kk = (nbk_all >> (2 * k)) & 3;
            Real tup[NX], tvp[NX];
#pragma unroll
            for (int a = 0; a < NX; ++a) {
                txp[a] = 0; tUp[a] = 0; tVp[a] = 0; tup[a] = 0; tvp[a] = 0;
            }
            const unsigned un_ = (unsigned)nb * (unsigned)sizeof(Real);
            Real x0 = 0, u0 = 0, v0 = 0;
#pragma unroll
            for (int n = 0; n < KN; ++n) {
                const Real fx = bC.ld(0 * KS + n, un_);
                const Real fU = bC.ld(1 * KS + n, un_);
                const Real fV = bC.ld(2 * KS + n, un_);
                const Real fu = bU.ld(0 * KS + n, un_);
                const Real fv = bU.ld(1 * KS + n, un_);
                if (n == 0) { x0 = fx; u0 = fu; v0 = fv; }
                // the trace of a degree-d basis function has no Legendre mode above d
#pragma unroll
                for (int a = 0; a < NX && a <= TDEG[n]; ++a) {
                    const Real r = sR[kk][n][a];
                    txp[a] = fma(fx, r, txp[a]);
                    tUp[a] = fma(fU, r, tUp[a]);
                    tVp[a] = fma(fV, r, tVp[a]);
                    tup[a] = fma(fu, r, tup[a]);
                    tvp[a] = fma(fv, r, tvp[a]);
                }
            }
            // the neighbour runs along the edge in the opposite direction
#pragma unroll
            for (int a = 1; a < NX; a += 2) {
                txp[a] = -txp[a]; tUp[a] = -tUp[a]; tVp[a] = -tVp[a]; tup[a] = -tup[a]; tvp[a] = -tvp[a];
            }
#pragma unroll
            for (int a = 0; a < NX; ++a) {
                unp[a] = fma(tup[a], nx, tvp[a] * ny);
                qnp[a] = fma(tUp[a], nx, tVp[a] * ny);
            }
            xbp = Real(SQRT2) * x0;
            unbp = fabs(fma(Real(SQRT2) * u0, nx, Real(SQRT2) * v0 * ny));
        } else if (nb == NB_LAND) {
            // mirror: xi+ = xi-, normal parts of q and u change sign
            Real m2;
        if constexpr (std::is_same<Real, double>::value)
            m2 = -2.0 / len2;
        else
            m2 = -2.0f * rcp_approx(float(len2));
#pragma unroll
            for (int a = 0; a < NX; ++a) {
                txp[a] = txm[a];
                unp[a] = -unm[a];
                qnp[a] = -qnm[a];
                tUp[a] = fma(m2 * qnm[a], nx, tUm[a]);
                tVp[a] = fma(m2 * qnm[a], ny, tVm[a]);
            }
            xbp = xbm;
            unbp = unbm;
        } else {
            // open sea: xi+ = xi_hat(t), q and u copied
#pragma unroll
            for (int a = 0; a < NX; ++a) {
                txp[a] = a == 0 ? Real(xihat) : Real(0);
                tUp[a] = tUm[a];
                tVp[a] = tVm[a];
                unp[a] = unm[a];
                qnp[a] = qnm[a];
            }
            xbp = Real(xihat);
            unbp = unbm;
        }
        // penalty from constant parts at the edge midpoint (eq:lambda), times |E|
        Real lam;
        if constexpr (std::is_same<Real, double>::value)
            lam = tmax(unbm, unbp) + sqrt(g * (tmax(xbm, xbp) + hmid) * len2);
        else
            lam = tmax(unbm, unbp) + sqrt_approx(float(g * (double(tmax(xbm, xbp)) + hmid) * len2));
        // the flux's factor 1/2 rides on the scale (exact: a power of two)
        const Real sc = Real(0.5 * dt_det);
        const Real hg = Real(0.5 * g);
        Real FX[NT], FU[NT], FV[NT];
        double FW[NT];
        double xs[NX];
#pragma unroll
        for (int a = 0; a < NX; ++a) xs[a] = double(txm[a]) + double(txp[a]);
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            const Real pb = hg * (prod1<NX, Real>(c, txm, txm) + prod1<NX, Real>(c, txp, txp));
            const Real mU = prod1<NX, Real>(c, tUm, unm) + prod1<NX, Real>(c, tUp, unp);
            const Real mV = prod1<NX, Real>(c, tVm, unm) + prod1<NX, Real>(c, tVp, unp);
            Real fx = qnm[c] + qnp[c] + lam * (txm[c] - txp[c]);
            if (nb == NB_LAND) fx = 0;   // q.n = 0: no mass flux through land
            FX[c] = sc * fx;
            FU[c] = sc * (mU + pb * nx + lam * (tUm[c] - tUp[c]));
            FV[c] = sc * (mV + pb * ny + lam * (tVm[c] - tVp[c]));
            // bathymetry part of the pressure, (P- + P+)/2 = g (xi- + xi+) h_b / 2
            double w = 0.0;
#pragma unroll
            for (int a = 0; a < NX; ++a)
#pragma unroll
                for (int b = 0; b < 2 && b < NX; ++b)
                    if (TG[c][a][b] != 0.0) w = fma(TG[c][a][b] * hbt[b], xs[a], w);
            FW[c] = 0.5 * g * w * dt_det;
        }
        double FWx[NT], FWy[NT];
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            FWx[c] = FW[c] * dy;
            FWy[c] = FW[c] * -dx;
        }
#pragma unroll
        for (int q = 0; q < K; ++q) {
            Real a0 = A.L[0][q], a1 = A.L[1][q], a2 = A.L[2][q];
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                if (TR[k][q][c] == 0.0) continue;
                const Real r = Real(TR[k][q][c]);
                a0 = fma(-r, FX[c], a0);
                a1 = fma(-r, FU[c], a1);
                a2 = fma(-r, FV[c], a2);
            }
            A.L[0][q] = a0; A.L[1][q] = a1; A.L[2][q] = a2;
            double w0 = A.w(0, q), w1 = A.w(1, q);
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                if (TR[k][q][c] == 0.0) continue;
                w0 = fma(-TR[k][q][c], FWx[c], w0);
                w1 = fma(-TR[k][q][c], FWy[c], w1);
            }
            A.w(0, q) = w0; A.w(1, q) = w1;
        }
    }
}

template <int P, int PN, typename Real>
SWE_HD void edge_terms(const MeshView &m, unsigned e, const Buf<Real> &bC, const Buf<Real> &bU,
                                           const Buf<int> &bNb,
                                           const Fields<P, Real> &s, const Geo &G, double g,
                                           double xihat, double dt,
                                           const Real (*sR)[Ord<PN>::K][(P > PN ? P : PN) + 1],
                                           Acc<P, Real> &A)
{
    edge_one<P, PN, Real, 0>(m, e, bC, bU, bNb, s, G, g, xihat, dt, sR, A);
    edge_one<P, PN, Real, 1>(m, e, bC, bU, bNb, s, G, g, xihat, dt, sR, A);
    edge_one<P, PN, Real, 2>(m, e, bC, bU, bNb, s, G, g, xihat, dt, sR, A);
}

// ------------------------------------------------------------ u H = q
// H_ij = sum_{n < K(max(deg i, deg j))} xi_n C[n][i][j] + sum_{n<3} hb_n C[n][i][j];
// modes at or above Ke are masked to the identity (element order below P).
template <int P, typename Real>
SWE_HD void solve_u(const Real (&xi)[Ord<P>::K], const Real (&U)[Ord<P>::K],
                                        const Real (&V)[Ord<P>::K], const double (&hbh)[3], int Ke,
                                        Real (&u)[Ord<P>::K], Real (&v)[Ord<P>::K])
{
    constexpr int K = Ord<P>::K;
    constexpr bool dbl = std::is_same<Real, double>::value;
    // FP32: the total depth's modes H_n = xi_n + hb_n formed once (hb is
    // linear: modes 0-2), H is needed to FP32's relative accuracy only;
    // FP64: the bathymetry part summed on its own
    Real Hm[K];
#pragma unroll
    for (int n = 0; n < K; ++n) Hm[n] = (!dbl && n < 3) ? xi[n] + Real(hbh[n < 3 ? n : 0]) : xi[n];
    Real M[K][K];
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            const int dmax = TDEG[i] > TDEG[j] ? TDEG[i] : TDEG[j];
            const int kt = KOFP[dmax];
            Real acc = 0;
#pragma unroll
            for (int n = 0; n < kt; ++n)
                if (TC[n][i][j] != 0.0) acc = fma(Real(TC[n][i][j]), Hm[n], acc);
            if constexpr (dbl) {
                double hbp = 0.0;
#pragma unroll
                for (int n = 0; n < 3; ++n)
                    if (TC[n][i][j] != 0.0) hbp = fma(TC[n][i][j], hbh[n], hbp);
                acc += Real(hbp);
            }
            if (i >= Ke || j >= Ke) acc = (i == j) ? Real(1) : Real(0);
            M[i][j] = acc;
        }
    // LDL^T without pivoting: H is symmetric positive definite for positive depth
    Real d[K], id[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
        Real djj = M[j][j];
#pragma unroll
        for (int k = 0; k < j; ++k) djj = fma(-M[j][k] * d[k], M[j][k], djj);
        d[j] = djj;
        if constexpr (std::is_same<Real, double>::value)
            id[j] = 1.0 / djj;
        else
            id[j] = rcp_approx(djj);
#pragma unroll
        for (int i = j + 1; i < K; ++i) {
            Real sij = M[i][j];
#pragma unroll
            for (int k = 0; k < j; ++k) sij = fma(-M[i][k] * d[k], M[j][k], sij);
            M[i][j] = sij * id[j];
        }
    }
    Real y[K], z[K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
        Real a = i < Ke ? U[i] : Real(0), b = i < Ke ? V[i] : Real(0);
#pragma unroll
        for (int k = 0; k < i; ++k) {
            a = fma(-M[i][k], y[k], a);
            b = fma(-M[i][k], z[k], b);
        }
        y[i] = a;
        z[i] = b;
    }
#pragma unroll
    for (int i = 0; i < K; ++i) { y[i] *= id[i]; z[i] *= id[i]; }
#pragma unroll
    for (int i = K - 1; i >= 0; --i) {
        Real a = y[i], b = z[i];
#pragma unroll
        for (int k = i + 1; k < K; ++k) {
            a = fma(-M[k][i], u[k], a);
            b = fma(-M[k][i], v[k], b);
        }
        u[i] = a;
        v[i] = b;
    }
}

SWE_HD void hb_modes(const Geo &G, double (&hbh)[3])
{
#pragma unroll
    for (int n = 0; n < 3; ++n) hbh[n] = TW[n][0] * G.h[0] + TW[n][1] * G.h[1] + TW[n][2] * G.h[2];
}

// ------------------------------------------------------------ kernel pieces
template <int KN, int NX, typename Real>
__device__ __forceinline__ void load_trace_table(Real (*sR)[KN][NX])
{
    for (int i = threadIdx.x; i < 3 * KN * NX; i += blockDim.x) {
        const int k = i / (KN * NX), r = i % (KN * NX);
        sR[k][r / NX][r % NX] = (r % NX) < 4 ? Real(TR[k][r / NX][r % NX]) : Real(0);
    }
}

template <int P, typename Real>
SWE_HD void acc_init(Acc<P, Real> &A, const Fields<P, Real> &s, bool with_state)
{
#pragma unroll
    for (int q = 0; q < Ord<P>::K; ++q) {
        A.L[0][q] = with_state ? s.xi[q] : Real(0);
        A.L[1][q] = with_state ? s.U[q] : Real(0);
        A.L[2][q] = with_state ? s.V[q] : Real(0);
        if constexpr (Acc<P, Real>::SPLIT) { A.W[0][q] = 0.0; A.W[1][q] = 0.0; }
    }
}

// acc += dt L(c) for one element of order P with neighbours of order <= PN
template <int P, int PN, typename Real>
SWE_HD void element_rhs(const StageArgs<Real> &a, unsigned e, const Buf<Real> &bC,
                                            const Buf<Real> &bU, const Buf<int> &bNb,
                                            const Fields<P, Real> &s, const Geo &G, const double (&hbh)[3],
                                            double dt, const Real (*sR)[Ord<PN>::K][(P > PN ? P : PN) + 1],
                                            Acc<P, Real> &A, double xihat)
{
    constexpr int K = Ord<P>::K;
    volume_term<P, Real>(s, hbh, G, a.ph.g, dt, A);
    source_term<P, Real>(s, G, a.ph, dt, A);
    edge_terms<P, PN, Real>(a.m, e, bC, bU, bNb, s, G, a.ph.g, xihat, dt, sR, A);
    if constexpr (Acc<P, Real>::SPLIT) {
#pragma unroll
        for (int q = 0; q < K; ++q) {
            A.L[1][q] += Real(A.W[0][q]);
            A.L[2][q] += Real(A.W[1][q]);
        }
    }
    if (a.src) {
        const Buf<Real> bS(a.src, 3 * a.m.KS, a.m.stride);
        const Real rdt = Real(dt);
        const unsigned off = e * (unsigned)sizeof(Real);
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int q = 0; q < K; ++q) A.L[j][q] = fma(rdt, bS.ld(j * a.m.KS + q, off), A.L[j][q]);
    }
}

// Store an element's new state (CPOL: cache policy, 0 the default); returns a
// value that is finite only if all of it is.
template <int P, typename Real, int CPOL>
__device__ __forceinline__ Real store_state(const StageArgs<Real> &a, unsigned off, const Real (&x)[Ord<P>::K],
                                            const Real (&U)[Ord<P>::K], const Real (&V)[Ord<P>::K],
                                            const Real (&u)[Ord<P>::K], const Real (&v)[Ord<P>::K])
{
    constexpr int K = Ord<P>::K;
    const int KS = a.m.KS, stride = a.m.stride;
    const Buf<Real> bO(a.Cout, 3 * KS, stride), bV(a.Uout, 2 * KS, stride);
    Real chk = 0;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        bO.template st_policy<CPOL>(0 * KS + q, off, x[q]);
        bO.template st_policy<CPOL>(1 * KS + q, off, U[q]);
        bO.template st_policy<CPOL>(2 * KS + q, off, V[q]);
        bV.template st_policy<CPOL>(0 * KS + q, off, u[q]);
        bV.template st_policy<CPOL>(1 * KS + q, off, v[q]);
        chk += x[q] + U[q] + V[q] + u[q] + v[q];
    }
    return chk;
}

// Whether the step of a step graph does not run: its clock stopped, or the step
// before failed when this step's clock was already set (the list kernel that
// sets it runs beside kernels which may still find a failure; they write it to
// the next clock's `late`, which is final when the next step starts).  Uniform
// over the grid.  LATE: the kernel has a place in such graphs (base orders 0 and
// 1, lists up to order 2).  The failure is handed on by the clock's block, not
// here: a store before them would turn the block's scalar loads into vector
// ones (2,097,152 elements, FP64, 496 -> 508 us a step).
template <bool LATE, typename Real>
__device__ __forceinline__ bool step_stopped(const StageArgs<Real> &a)
{
    if constexpr (!LATE) return !a.inst->run;
    const int run = a.inst->run, late = a.inst->late;   // neighbours: one load
    return (run == 0) | (late != 0);
}

// SSP-RK2 combine of acc = c + dt L, u-solve of the new state, store, depth check
template <int P, typename Real, int MODE>
__device__ __forceinline__ void finish_stage(const StageArgs<Real> &a, unsigned e, const Geo &G,
                                             const double (&hbh)[3], int Ke, const Real (&L)[3][Ord<P>::K],
                                             int *flag)
{
    constexpr int K = Ord<P>::K;
    const int KS = a.m.KS, stride = a.m.stride;
    const unsigned off = e * (unsigned)sizeof(Real);
    Real xn[K], Un[K], Vn[K];
    const Buf<Real> bN(a.Cn, 3 * KS, stride);
#pragma unroll
    for (int q = 0; q < K; ++q) {
        Real c0 = L[0][q], c1 = L[1][q], c2 = L[2][q];
        if constexpr (MODE == MODE_STAGE2) {
            c0 = Real(0.5) * bN.ld(0 * KS + q, off) + Real(0.5) * c0;
            c1 = Real(0.5) * bN.ld(1 * KS + q, off) + Real(0.5) * c1;
            c2 = Real(0.5) * bN.ld(2 * KS + q, off) + Real(0.5) * c2;
        }
        xn[q] = c0; Un[q] = c1; Vn[q] = c2;
    }
    Real un[K], vn[K];
    solve_u<P, Real>(xn, Un, Vn, hbh, Ke, un, vn);
    // FP64 results are streamed past the caches (measured: 4 % shorter FP64
    // stages at p = 2, while the same policy lengthens FP32 stages by 4 %)
    const Real chk = store_state<P, Real, sizeof(Real) == 8 ? CPOL_NT : 0>(a, off, xn, Un, Vn, un, vn);
    const double Hmean = SQRT2 * double(xn[0]) + (G.h[0] + G.h[1] + G.h[2]) * (1.0 / 3.0);
    if (!(Hmean > 0.0) || !isfinite(chk)) flag[0] = 1;
}

// ------------------------------------------------------------ shared edge fluxes
// Stage kernel in which each edge flux inside a block of BLOCK consecutive
// elements is computed once and handed to both sides through LDS (the passes
// are described at stage_sh_block).  The block's edge items are host-built:
// a pair of elements of the block (taken once, from the lower index), an
// element and a neighbour outside the block, a land or an open edge.  An
// item packs a (bits 0-7), its local edge (8-9), b (10-17), b's local edge
// (18-19) and the kind (20-21).
constexpr unsigned EK_PAIR = 0, EK_EXT = 1, EK_LAND = 2, EK_OPEN = 3;

// Waves per SIMD the shared-flux kernels are built for at least: what their
// LDS allows and their registers reach without spilling (FP32 p = 2: 32 KB
// per 256-element block, four blocks per CU, 128 registers; FP32 p = 1:
// 22 KB, five waves at 85 registers; FP32 p = 3 and FP64 p = 2: 53 and 63 KB,
// two waves (three would spill); FP64 p = 1: 34 KB, three waves (four would
// spill); FP64 p = 3: 105 KB, one block, whose registers then spill into
// accumulation registers rather than scratch).
template <int P, typename Real>
constexpr int sh_waves()
{
    constexpr bool dbl = std::is_same<Real, double>::value;
    return dbl ? (P == 1 ? 3 : P == 3 ? 1 : 2) : (P == 2 ? 4 : P == 3 ? 2 : 3);
}

// The batch form at FP32 order 3 loads the geometry after the edge pass and
// runs three waves per SIMD (168 registers, no spill; its LDS, 53 KB per
// block, allows three blocks per CU); the single-instance form, which also
// carries the separated scheme's base-pass paths, would spill there.
template <int P, typename Real>
constexpr bool batch_sh_fp32p3()
{
    return !std::is_same<Real, double>::value && P == 3;
}

// Per-block LDS.  The state copy C is read by the edge pass only; the
// per-item results F, W are written after it (every lane holds its items'
// results in registers across a barrier), so the two share the storage.
// Results are stored per edge item (lane i writes column i: consecutive
// words, no bank conflicts), and slot[k][l] tells element l which item
// holds its local edge k (bit 15: l is the item's second side, which sees
// the flux negated and reversed along the edge).
// With BOTH the two have storage of their own: fluxes are then written as
// they are computed, and the next state copy while they are still needed, with
// half the barriers.
template <int P, typename Real, bool BOTH = false>
struct ShLds {
    static constexpr int K = Ord<P>::K, NT = Ord<P>::NT;
    Real R[3][K][NT];              // trace matrices
    unsigned short slot[3][BLOCK]; // item of each (local edge, element)
    struct Fluxes {
        Real F[3 * NT][2 * BLOCK];  // flux modes (component, mode) per item
        double W[NT][2 * BLOCK];    // bathymetry part of the pressure flux, FP64, per item
    };
    union Shared {
        Real C[5 * K][BLOCK];      // xi, U, V, u, v modes of the block's elements
        Fluxes E;
    };
    struct Apart {
        Real C[5 * K][BLOCK];
        Fluxes E;
    };
    std::conditional_t<BOTH, Apart, Shared> U;
};

// An edge item's results, kept in registers until the state copy is no
// longer read.
template <int P, typename Real>
struct ShItem {
    static constexpr int NT = Ord<P>::NT;
    Real F[3][NT];
    double W[NT];
};

template <int P, typename Real, bool BOTH>
__device__ __forceinline__ void traces_of(const ShLds<P, Real, BOTH> &S, int l, int k, Real (&t)[5][Ord<P>::NT])
{
    constexpr int K = Ord<P>::K, NT = Ord<P>::NT;
#pragma unroll
    for (int f = 0; f < 5; ++f)
#pragma unroll
        for (int c = 0; c < NT; ++c) t[f][c] = Real(0);
#pragma unroll
    for (int n = 0; n < K; ++n)
#pragma unroll
        for (int c = 0; c < NT && c <= TDEG[n]; ++c) {
            const Real r = S.R[k][n][c];
#pragma unroll
            for (int f = 0; f < 5; ++f) t[f][c] = fma(S.U.C[f * K + n][l], r, t[f][c]);
        }
}

template <int P, typename Real, bool BOTH>
__device__ __forceinline__ void load_trace_lds(ShLds<P, Real, BOTH> &S)
{
    constexpr int K = Ord<P>::K, NT = Ord<P>::NT;
    for (int i = threadIdx.x; i < 3 * K * NT; i += (int)blockDim.x) {
        const int k = i / (K * NT), r = i % (K * NT);
        S.R[k][r / NT][r % NT] = Real(TR[k][r / NT][r % NT]);
    }
}

// What an edge item reads outside the block's state copies: the two vertices
// of side a's local edge, and the neighbour outside the block with its local
// edge.  BlockSrc: block of consecutive elements from e0, through the mesh
// arrays.
struct BlockSrc {
    const MeshView &m;
    const Buf<int> &bEv, &bNb;
    unsigned e0;
    __device__ __forceinline__ void edge(int la, int va, int vb, double3 &pa, double3 &pb) const
    {
        const unsigned off = (e0 + (unsigned)la) * 4u;
        const double4 a = m.vtx[(unsigned)bEv.ld(va, off)], b = m.vtx[(unsigned)bEv.ld(vb, off)];
        pa = make_double3(a.x, a.y, a.z);
        pb = make_double3(b.x, b.y, b.z);
    }
    __device__ __forceinline__ unsigned outside(unsigned w, int &kk) const
    {
        const int ka = (int)((w >> 8) & 3u);
        const unsigned ea = e0 + (w & 255u);
        const int nb = bNb.ld(ka, ea * 4u);
        kk = (m.enbk[ea] >> (2 * ka)) & 3;
        return (unsigned)nb;
    }
};

// The Lax-Friedrichs flux of one edge item, in the first side's orientation,
// times two (its factor 1/2 is applied with dt / |det B| at the lift) and
// unscaled by dt / |det B| (the edge pass of the shared-flux kernels); the
// FP64 bathymetry part W is complete.
template <int P, typename Real, bool BOTH, typename Src>
__device__ __forceinline__ void sh_flux(const ShLds<P, Real, BOTH> &S, int KS, const Buf<Real> &bC, const Buf<Real> &bU,
                                        const Src &src, unsigned w, double xihat, double g, ShItem<P, Real> &out)
{
    constexpr int K = Ord<P>::K, NT = Ord<P>::NT;
    const int la = (int)(w & 255u), ka = (int)((w >> 8) & 3u), lb = (int)((w >> 10) & 255u);
    const int kb = (int)((w >> 18) & 3u);
    const unsigned kind = (w >> 20) & 3u;
    double3 pa, pb;
    src.edge(la, (ka + 1) % 3, (ka + 2) % 3, pa, pb);
    const double dx = pb.x - pa.x, dy = pb.y - pa.y;
    const double len2 = dx * dx + dy * dy;
    const Real nx = Real(dy), ny = Real(-dx);          // |E| n of side a
    const double hmid = 0.5 * (pa.z + pb.z);
    const double hbt[2] = {hmid, (pb.z - pa.z) * INV_2SQRT3};
    Real tm[5][NT], tp[5][NT];
    traces_of<P, Real, BOTH>(S, la, ka, tm);
    const Real xbm = Real(SQRT2) * S.U.C[0][la];
    const Real unbm = fabs(fma(Real(SQRT2) * S.U.C[3 * K][la], nx, Real(SQRT2) * S.U.C[4 * K][la] * ny));
    Real unm[NT], qnm[NT], unp[NT], qnp[NT];
#pragma unroll
    for (int c = 0; c < NT; ++c) {
        unm[c] = fma(tm[3][c], nx, tm[4][c] * ny);
        qnm[c] = fma(tm[1][c], nx, tm[2][c] * ny);
    }
    Real xbp, unbp;
    if (kind == EK_PAIR || kind == EK_EXT) {
        Real x0, u0, v0;
        if (kind == EK_PAIR) {
            traces_of<P, Real, BOTH>(S, lb, kb, tp);
            x0 = S.U.C[0][lb];
            u0 = S.U.C[3 * K][lb];
            v0 = S.U.C[4 * K][lb];
        } else {
            int kk;
            const unsigned un_ = src.outside(w, kk) * (unsigned)sizeof(Real);
#pragma unroll
            for (int f = 0; f < 5; ++f)
#pragma unroll
                for (int c = 0; c < NT; ++c) tp[f][c] = Real(0);
            x0 = Real(0); u0 = Real(0); v0 = Real(0);
#pragma unroll
            for (int n = 0; n < K; ++n) {
                const Real fv[5] = {bC.ld(0 * KS + n, un_), bC.ld(1 * KS + n, un_), bC.ld(2 * KS + n, un_),
                                    bU.ld(0 * KS + n, un_), bU.ld(1 * KS + n, un_)};
                if (n == 0) { x0 = fv[0]; u0 = fv[3]; v0 = fv[4]; }
#pragma unroll
                for (int c = 0; c < NT && c <= TDEG[n]; ++c) {
                    const Real r = S.R[kk][n][c];
#pragma unroll
                    for (int f = 0; f < 5; ++f) tp[f][c] = fma(fv[f], r, tp[f][c]);
                }
            }
        }
        // the other side runs along the edge in the opposite direction
#pragma unroll
        for (int c = 1; c < NT; c += 2)
#pragma unroll
            for (int f = 0; f < 5; ++f) tp[f][c] = -tp[f][c];
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            unp[c] = fma(tp[3][c], nx, tp[4][c] * ny);
            qnp[c] = fma(tp[1][c], nx, tp[2][c] * ny);
        }
        xbp = Real(SQRT2) * x0;
        unbp = fabs(fma(Real(SQRT2) * u0, nx, Real(SQRT2) * v0 * ny));
    } else if (kind == EK_LAND) {
        // mirror: xi+ = xi-, normal parts of q and u change sign
        Real m2;
        if constexpr (std::is_same<Real, double>::value)
            m2 = -2.0 / len2;
        else
            m2 = -2.0f * rcp_approx(float(len2));
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            tp[0][c] = tm[0][c];
            unp[c] = -unm[c];
            qnp[c] = -qnm[c];
            tp[1][c] = fma(m2 * qnm[c], nx, tm[1][c]);
            tp[2][c] = fma(m2 * qnm[c], ny, tm[2][c]);
        }
        xbp = xbm;
        unbp = unbm;
    } else {
        // open sea: xi+ = xi_hat(t), q and u copied
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            tp[0][c] = c == 0 ? Real(xihat) : Real(0);
            tp[1][c] = tm[1][c];
            tp[2][c] = tm[2][c];
            unp[c] = unm[c];
            qnp[c] = qnm[c];
        }
        xbp = Real(xihat);
        unbp = unbm;
    }
    // penalty from constant parts at the edge midpoint (eq:lambda), times |E|
    Real lam;
    if constexpr (std::is_same<Real, double>::value)
        lam = tmax(unbm, unbp) + sqrt(g * (tmax(xbm, xbp) + hmid) * len2);
    else
        lam = tmax(unbm, unbp) + sqrt_approx(float(g * (double(tmax(xbm, xbp)) + hmid) * len2));
    const Real hg = Real(0.5 * g);
    Real (&F)[3][NT] = out.F;
    double (&Wf)[NT] = out.W;
#pragma unroll
    for (int c = 0; c < NT; ++c) {
        const Real pb = hg * (prod1<NT, Real>(c, tm[0], tm[0]) + prod1<NT, Real>(c, tp[0], tp[0]));
        const Real mU = prod1<NT, Real>(c, tm[1], unm) + prod1<NT, Real>(c, tp[1], unp);
        const Real mV = prod1<NT, Real>(c, tm[2], unm) + prod1<NT, Real>(c, tp[2], unp);
        Real fx = qnm[c] + qnp[c] + lam * (tm[0][c] - tp[0][c]);
        if (kind == EK_LAND) fx = 0;   // q.n = 0: no mass flux through land
        F[0][c] = fx;
        F[1][c] = mU + pb * nx + lam * (tm[1][c] - tp[1][c]);
        F[2][c] = mV + pb * ny + lam * (tm[2][c] - tp[2][c]);
        // bathymetry part of the pressure, (P- + P+)/2 = g (xi- + xi+) h_b / 2
        double wv = 0.0;
#pragma unroll
        for (int aa = 0; aa < NT; ++aa) {
            const double xs = double(tm[0][aa]) + double(tp[0][aa]);
#pragma unroll
            for (int bb = 0; bb < 2 && bb < NT; ++bb)
                if (TG[c][aa][bb] != 0.0) wv = fma(TG[c][aa][bb] * hbt[bb], xs, wv);
        }
        Wf[c] = 0.5 * g * wv;
    }
}

// Store item i's flux in its column and point its sides' slots at it (the
// second side of a pair inside the block marked by bit 15).
template <int P, typename Real, bool BOTH>
__device__ __forceinline__ void sh_store(ShLds<P, Real, BOTH> &S, int i, unsigned w, const ShItem<P, Real> &r)
{
    constexpr int NT = Ord<P>::NT;
    const int la = (int)(w & 255u), ka = (int)((w >> 8) & 3u), lb = (int)((w >> 10) & 255u);
    const int kb = (int)((w >> 18) & 3u);
#pragma unroll
    for (int c = 0; c < NT; ++c) {
#pragma unroll
        for (int j = 0; j < 3; ++j) S.U.E.F[j * NT + c][i] = r.F[j][c];
        S.U.E.W[c][i] = r.W[c];
    }
    S.slot[ka][la] = (unsigned short)i;
    if (((w >> 20) & 3u) == EK_PAIR) S.slot[kb][lb] = (unsigned short)(i | 0x8000);
}

// Lift element l's three edge fluxes from the block's item columns onto its
// modes, with its own geometry.
template <int P, typename Real, bool BOTH>
__device__ __forceinline__ void sh_lift(const ShLds<P, Real, BOTH> &S, const Geo &G, int l, double dt, Acc<P, Real> &A)
{
    constexpr int K = Ord<P>::K, NT = Ord<P>::NT;
    const double dt_det = dt * G.idet;
    // the stored fluxes lack their factor 1/2: the scale carries it (exact)
    const Real sc = Real(0.5 * dt_det);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int ka = (k + 1) % 3, kb = (k + 2) % 3;
        const double dx = G.X[kb] - G.X[ka], dy = G.Y[kb] - G.Y[ka];
        // the item of this edge; as its second side the flux comes negated and
        // reversed along the edge (even Legendre modes change sign, odd ones not)
        const unsigned sl = S.slot[k][l];
        const int it = (int)(sl & 0x7fffu);
        const bool second = (sl & 0x8000u) != 0u;
        Real FX[NT], FU[NT], FV[NT];
        double FWx[NT], FWy[NT];
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            const bool flip = second && !(c & 1);
            const Real f0 = S.U.E.F[0 * NT + c][it], f1 = S.U.E.F[1 * NT + c][it], f2 = S.U.E.F[2 * NT + c][it];
            FX[c] = sc * (flip ? -f0 : f0);
            FU[c] = sc * (flip ? -f1 : f1);
            FV[c] = sc * (flip ? -f2 : f2);
            const double w = S.U.E.W[c][it];
            const double FW = (second && (c & 1) ? -w : w) * dt_det;
            FWx[c] = FW * dy;
            FWy[c] = FW * -dx;
        }
#pragma unroll
        for (int q = 0; q < K; ++q) {
            Real a0 = A.L[0][q], a1 = A.L[1][q], a2 = A.L[2][q];
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                if (TR[k][q][c] == 0.0) continue;
                const Real r = Real(TR[k][q][c]);
                a0 = fma(-r, FX[c], a0);
                a1 = fma(-r, FU[c], a1);
                a2 = fma(-r, FV[c], a2);
            }
            A.L[0][q] = a0; A.L[1][q] = a1; A.L[2][q] = a2;
            double w0 = A.w(0, q), w1 = A.w(1, q);
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                if (TR[k][q][c] == 0.0) continue;
                w0 = fma(-TR[k][q][c], FWx[c], w0);
                w1 = fma(-TR[k][q][c], FWy[c], w1);
            }
            A.w(0, q) = w0; A.w(1, q) = w1;
        }
    }
}

// The passes over the block of elements [e0, e0 + BLOCK) (live below e_end),
// whose edge items are items[0, nitems), nitems <= 2 BLOCK (ITEM_PAD slots
// among them are empty).  Every thread of
// the block calls it (it holds three block barriers); the trace tables in S
// are loaded before (the first barrier orders them before their first use).
//   1. each lane (one element) loads its state into registers and copies it
//      to LDS;
//   2. each lane computes the flux of at most two edge items (a pair of
//      elements of the block, an element and a neighbour outside it, a land
//      or an open edge) from the state copies and keeps it in registers;
//      once every lane is done reading the copies, the fluxes overwrite them,
//      each stored for its first side and, for a pair, for the second;
//   3. each lane adds its volume and source terms, lifts its three edge
//      fluxes with its own geometry and finishes the stage.
template <int P, typename Real, int MODE, bool EARLY_GEO = !std::is_same<Real, double>::value && P == 3>
__device__ __forceinline__ void stage_sh_block(ShLds<P, Real> &S, const StageArgs<Real> &a, unsigned e0,
                                               unsigned e_end, const unsigned *items, int nitems, double xihat,
                                               double dt, int *flag)
{
    constexpr int K = Ord<P>::K;
    const MeshView &m = a.m;
    const int KS = m.KS, stride = m.stride;
    const unsigned l = threadIdx.x, e = e0 + l;
    const bool live = e < e_end;
    if (MODE == MODE_RHS) dt = 1.0;
    const Buf<Real> bC(a.Cin, 3 * KS, stride), bU(a.Uin, 2 * KS, stride);
    const Buf<int> bEv(m.ev, 3, stride), bNb(m.enb, 3, stride);
    const double g = a.ph.g;

    // 1. state to registers and LDS; at FP32 order 3 (two waves per SIMD) also
    //    the geometry, whose latency then hides behind the edge pass (elsewhere
    //    the registers it would hold across that pass cost a wave per SIMD:
    //    only the vertex ids are loaded here, the vertices after the edge pass)
    constexpr bool early_geo = EARLY_GEO;
    Fields<P, Real> s;
    Geo G;
    double hbh[3];
    int id3[3] = {0, 0, 0};
    const unsigned off = e * (unsigned)sizeof(Real);
    if (live) {
        if constexpr (early_geo) {
            load_geo(m.vtx, bEv, e * 4u, G);
        } else {
#pragma unroll
            for (int v = 0; v < 3; ++v) id3[v] = bEv.ld(v, e * 4u);
        }
        load_state<P, Real>(bC, bU, KS, off, s);
#pragma unroll
        for (int q = 0; q < K; ++q) {
            S.U.C[0 * K + q][l] = s.xi[q];
            S.U.C[1 * K + q][l] = s.U[q];
            S.U.C[2 * K + q][l] = s.V[q];
            S.U.C[3 * K + q][l] = s.u[q];
            S.U.C[4 * K + q][l] = s.v[q];
        }
    }
    __syncthreads();

    // 2. the fluxes of this lane's (at most two) edge items
    const int n = nitems < 2 * BLOCK ? nitems : 2 * BLOCK;
    const int it0 = (int)l, it1 = (int)l + BLOCK;
    const unsigned w0 = it0 < n ? items[it0] : ITEM_PAD, w1 = it1 < n ? items[it1] : ITEM_PAD;
    ShItem<P, Real> r0, r1;
    const BlockSrc bsrc{m, bEv, bNb, e0};
    if (w0 != ITEM_PAD) sh_flux<P, Real, false>(S, KS, bC, bU, bsrc, w0, xihat, g, r0);
    if (w1 != ITEM_PAD) sh_flux<P, Real, false>(S, KS, bC, bU, bsrc, w1, xihat, g, r1);
    __syncthreads();
    if (w0 != ITEM_PAD) sh_store<P, Real, false>(S, it0, w0, r0);
    if (w1 != ITEM_PAD) sh_store<P, Real, false>(S, it1, w1, r1);
    __syncthreads();
    if (!live) return;
    // base pass of the order-partitioned scheme: a listed element belongs to
    // the full-order kernel of its order (the fluxes of its edges above were
    // taken at the base order, which is exact only for unlisted elements,
    // whose neighbours all have the base order)
    const bool listed = a.inlist && a.inlist[e];
    if (a.skip_listed && listed) return;

    // 3. volume and source terms, the three edge fluxes lifted, the stage finished
    if constexpr (!early_geo) geo_from_ids(m.vtx, id3, G);
    hb_modes(G, hbh);
    Acc<P, Real> A;
    acc_init<P, Real>(A, s, MODE != MODE_RHS);
    volume_term<P, Real>(s, hbh, G, g, dt, A);
    source_term<P, Real>(s, G, a.ph, dt, A);
    sh_lift<P, Real, false>(S, G, (int)l, dt, A);
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
    if constexpr (MODE == MODE_RHS) {
        const Buf<Real> bL(a.Lout, 3 * KS, stride);
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int q = 0; q < K; ++q) bL.st(j * KS + q, off, A.L[j][q]);
    } else {
        if (a.Lb && listed) {
            // base pass of the order-separated scheme: the listed element's
            // base part waits in Lb for the epilogue
            const Buf<Real> bB(a.Lb, 3 * K, stride);
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int q = 0; q < K; ++q) bB.st(j * K + q, off, A.L[j][q]);
            return;
        }
        finish_stage<P, Real, MODE>(a, e, G, hbh, K, A.L, flag);
    }
}


}  // namespace
}  // namespace swe
