// row3.hpp -- the FP64 3-D step (D3Q19, D3Q27) in one launch: a workgroup owns a
// tile of 16 x BY columns (halo included) and marches along z with the planes
// in registers.
//
// Each column is served by two lanes of a wavefront, l and l ^ 32: half 0 owns
// the velocities k = 0 .. K - 1 (K = index of the rest velocity) and half 1
// their opposites; both hold the rest velocity.  Per-velocity work uses the
// half-0 table with the sign sg = +-1 folded into u, G and the coefficients;
// moments are lane-pair sums.  A 16-lane row of the wave is a tile row, so
// neighbours along x are neighbouring lanes (DPP row shifts); along y they
// exchange through LDS; along z they are the lane's own registers.
//
// With X, Y, Z the terms h xi_t d_t f-bar-plus of a cell, formed once each,
// the interface of axis a between cells L and R takes (Eq. gradient)
//   (1 - w) psi_L + w psi_R - h xi_a (phi_R - phi_L) / (x_R - x_L),
//   psi = phi minus the two terms along the interface.
// When plane N arrives (C the plane before it): phi(N); psi_y(C) and phi(N) to
// LDS; x interfaces of C; barrier; Y(N), X(N), the z interface between C and
// N, the y interfaces of C; their fluxes to LDS; barrier; update of C.
//
// Walls: ghost columns along x are lanes of the tile and extrapolate from the
// two lanes beside them; ghost rows and planes are extrapolated by the row or
// plane at the wall (psi too: the extrapolation commutes with the differences
// along the wall).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "ctx.hpp"
#include "kernels_general.hpp"
#include "march.hpp"
#include "wave.hpp"

namespace dugks {

#pragma clang fp contract(off)

constexpr int ROW_X = 16;  // columns of a tile row: the DPP row of a wave

// a value that every lane holds, in scalar registers: four vector registers that
// the bodies with an acceleration spilled in their loops (128^3 periodic 326 ->
// 298 us a step)
__device__ __forceinline__ double uniform(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b), hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
template <typename T>
__device__ __forceinline__ T row_next(T v) { return row_shift<1>(v); }
template <typename T>
__device__ __forceinline__ T row_prev(T v) { return row_shift<-1>(v); }

// velocities of half 0 with e_A != 0, and the place of k among them
template <class LAT>
__host__ __device__ constexpr int half_slot(int A, int k)
{
    int s = 0;
    for (int r = 0; r < k; ++r)
        if (LAT::e(r, A) != 0) ++s;
    return s;
}
// the velocities of half 0 that are along y alone: psi_y = phi
template <class LAT>
__host__ __device__ constexpr bool only_y(int k) { return LAT::e(k, 0) == 0 && LAT::e(k, 2) == 0; }
template <class LAT>
__host__ __device__ constexpr int psi_slot(int k)
{
    int s = 0;
    for (int r = 0; r < k; ++r)
        if (!only_y<LAT>(r)) ++s;
    return s;
}

// LDS slots of a column: phi of the velocities with e_y != 0 of two planes and
// both halves, psi_y, the rest velocity, the upper y interface's values, the
// force field
template <class LAT>
struct RowSlots {
    static constexpr int K = LAT::REST;
    static constexpr int NY = half_slot<LAT>(1, K);
    static constexpr int NP = psi_slot<LAT>(K);
    static constexpr int PHI = 0, PSI = 4 * NY, RESTV = PSI + 2 * NP, FLUX = RESTV + 1, FORCE = FLUX + 2 * NY;
    static constexpr int count(bool field) { return FORCE + (field ? 3 : 0); }
};

// moments of a column's values and the equilibrium factors in the lane's frame
// (us = sg u, Gs = sg sG G): fe_k = W_k (a + eu (B + C eu)), source (eG - g) fe
template <typename T>
struct EqR {
    T rho, a, B, C, g, us[3], Gs[3];
};

template <class LAT, typename T>
__device__ __forceinline__ T r3_dot(int k, const T (&u)[3])
{
    T s = T(0);
    bool first = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int e = LAT::e(k, a);
        if (e == 0) continue;
        if (first) s = e > 0 ? u[a] : -u[a];
        else s = e > 0 ? s + u[a] : s - u[a];
        first = false;
    }
    return s;
}

template <class LAT, typename T, bool ORIG>
__device__ __forceinline__ void r3_eq(const Inst<T>& P, T rho, const T (&us)[3], EqR<T>& E)
{
    E.rho = rho;
    const T uu = fma_(us[2], us[2], fma_(us[1], us[1], us[0] * us[0]));
    if constexpr (ORIG) {
        E.a = fma_(-(rho * P.hRT), uu, rho);
        E.B = rho * P.cRT;
        E.C = rho * P.c2RT2;
    } else {
        E.a = fma_(-P.eqH, uu, rho);
        E.B = P.eqB;
        E.C = P.eqC;
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) E.us[a] = us[a];
}

// G: acceleration (true frame), hw its time weight
template <class LAT, typename T, bool ORIG, bool ACC>
__device__ __forceinline__ EqR<T> r3_point(const Inst<T>& P, const T (&v)[LAT::REST], T r, T sg, const T (&G)[3], T hw)
{
    constexpr int K = LAT::REST;
    // half 0: first the velocities with e_x = -1, then those with e_x = 0 and
    // e_y = -1, last (0, 0, -1)
    T sa = T(0), sb = T(0), jy = T(0), jz = T(0);
#pragma unroll
    for (int k = 0; k < K - 1; ++k) {
        if (LAT::e(k, 0) != 0) sa += v[k];
        else sb += v[k];
        if (LAT::e(k, 0) != 0 && LAT::e(k, 1) == 1) jy += v[k];
        if (LAT::e(k, 0) != 0 && LAT::e(k, 1) == -1) jy -= v[k];
        if (LAT::e(k, 2) == 1) jz += v[k];
        if (LAT::e(k, 2) == -1) jz -= v[k];
    }
    const T sj[3] = {-sa, jy - sb, jz - v[K - 1]};
    T rs, j[3];
    moment_sums<3>((sa + sb) + v[K - 1], sj, sg, rs, j);
    const T rho = rs + r;
    const T cu = ORIG ? P.c / rho : P.crho;
    T us[3];
    EqR<T> E;
    if constexpr (ACC) {
        T gu = T(0);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const T u = fma_(hw, G[a], cu * j[a]);
            us[a] = sg * u;
            gu = fma_(G[a], u, gu);
            E.Gs[a] = (sg * P.sG) * G[a];
        }
        E.g = gu * P.invRT;
    } else {
        const T cs = sg * cu;
#pragma unroll
        for (int a = 0; a < 3; ++a) us[a] = cs * j[a];
    }
    r3_eq<LAT, T, ORIG>(P, rho, us, E);
    return E;
}

template <class LAT, typename T>
__device__ __forceinline__ T r3_feq(const EqR<T>& E, int k)
{
    const T eu = r3_dot<LAT, T>(k, E.us);
    return T(LAT::w(k)) * fma_(eu, fma_(E.C, eu, E.B), E.a);
}

// v + b (feq - v) + c S
template <class LAT, typename T, bool ACC>
__device__ __forceinline__ T r3_relax(const EqR<T>& E, int k, T b, T c, T v)
{
    const T fe = r3_feq<LAT, T>(E, k);
    v = fma_(b, fe - v, v);
    if constexpr (ACC) v = fma_(c * (r3_dot<LAT, T>(k, E.Gs) - E.g), fe, v);
    return v;
}

// The NEQ rule (Eq. NEQ) of a wall of side s of axis A, from the values v and
// the point E at the opposite interface of the wall cell: the equilibrium of
// the wall plus the non-equilibrium part there, for the crossing velocities
// (those that enter the domain are used).
template <class LAT, typename T, int A, bool ORIG>
__device__ __forceinline__ void r3_enter(const Inst<T>& P, int s, const EqR<T>& E, const T (&v)[LAT::REST], T sg, T gth,
                                         T (&W)[LAT::REST])
{
    EqR<T> B;
    const bool vel = P.bc[s] == BC_NEQ_VELOCITY;
    T ub[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) ub[a] = vel ? sg * P.uw[s][a] : E.us[a];
    r3_eq<LAT, T, ORIG>(P, vel ? E.rho : wall_density(P, s, gth), ub, B);
#pragma unroll
    for (int k = 0; k < LAT::REST; ++k)
        if (LAT::e(k, A) != 0) W[k] = r3_feq<LAT, T>(B, k) + (v[k] - r3_feq<LAT, T>(E, k));
}

// the wall rules of Eqs. (BB), (NEQ; entering values W) on a wall face of side s
// of axis A, for the velocities entering the domain (component `into` along A).
// Both lanes of a column take the same branches.
template <class LAT, typename T, int A>
__device__ __forceinline__ void r3_wall(const Inst<T>& P, int s, int into, T (&v)[LAT::REST], const T (&W)[LAT::REST],
                                        T sg)
{
    const bool plus = (sg > T(0)) == (into > 0);  // the lane's entering velocities have e(k, A) = +1
    const bool bb = P.bc[s] == BC_BOUNCE_BACK;
    const T uw[3] = {sg * P.uw[s][0], sg * P.uw[s][1], sg * P.uw[s][2]};
#pragma unroll
    for (int k = 0; k < LAT::REST; ++k) {
        if (LAT::e(k, A) == 0) continue;
        T nv = W[k];
        // the partner's value leaves where this one enters
        if (bb) nv = fma_(T(2) * P.eqB * T(LAT::w(k)), r3_dot<LAT, T>(k, uw), partner(v[k]));
        if (plus == (LAT::e(k, A) > 0)) v[k] = nv;
    }
}

// coefficients of a cell along one axis in the lane's frame: weight of its
// upper interface, sg h c / (x_R - x_L), sg h c times the derivative
// coefficients, sg c dt / Delta
template <typename T>
struct RowCoef {
    T w, k, kp, km, fd;
};
template <typename T, bool UNI>
__device__ __forceinline__ RowCoef<T> row_coef(const Inst<T>& P, int a, int j, int f, T sg)
{
    const T hc = sg * (P.h * P.c);
    if constexpr (UNI) return RowCoef<T>{T(0.5), hc * P.ugn[a], T(2) * (hc * P.uct[a]), T(0), sg * (P.ufdx[a] * P.c)};
    const AxisMetric<T>& m = P.m[a];
    return RowCoef<T>{m.w[f], hc * m.gn[f], hc * m.cp[j], hc * m.cm[j], sg * (m.fdx[j] * P.c)};
}

// h xi_t d_t phi for a velocity with component e = +1 along t
template <typename T, bool UNI>
__device__ __forceinline__ T r3_deriv(const RowCoef<T>& c, T dn, T ph, T up)
{
    if constexpr (UNI) return c.kp * (up - dn);
    else return fma_(c.kp, up - ph, c.km * (dn - ph));
}
template <typename T>
__device__ __forceinline__ T r3_minus(T a, int e, T d) { return e > 0 ? a - d : e < 0 ? a + d : a; }

template <typename T, bool UNI>
__device__ __forceinline__ T r3_recon(int e, T w, T k, T psL, T psR, T phL, T phR)
{
    T v;
    if constexpr (UNI) v = T(0.5) * (psL + psR);
    else v = fma_(w, psR - psL, psL);
    if (e > 0) v = fma_(-k, phR - phL, v);
    if (e < 0) v = fma_(k, phR - phL, v);
    return v;
}

// One workgroup's work: tile `tile` (of tiles0 along x) and march chunk `ck`
// of instance P.  ACC: there is an acceleration; FIELD: part of it is a force
// field (force may be null: a batch where only some instances have one); NW:
// the tile and chunk touch no wall; LOW: the chunk may begin at a low z wall.
template <class LAT, typename T, int BY, bool UNI, bool ACC, bool FIELD, bool ORIG, bool NW, bool LOW>
__device__ __forceinline__ void row_body(const Inst<T>& P, const T* __restrict__ fin, const T* __restrict__ force,
                                         T* __restrict__ fout, T gt, T gth, int chunk, int tiles0, int tile, int ck,
                                         T* lds)
{
    constexpr int K = LAT::REST, Q = LAT::Q, SQ = ROW_X * BY;
    using S = RowSlots<LAT>;
    // OWN: a plane's state stays in registers until its update instead of being
    // loaded a second time
    constexpr bool OWN = NW && LAT::Q == 19;
    const int tid = (int)threadIdx.x;
    const int h = (tid >> 5) & 1;
    const int col = (tid >> 6) * 32 + (tid & 31);
    const int tx = col & (ROW_X - 1), ty = col / ROW_X;
    const T sg = h ? T(-1) : T(1);
    const int nx = P.n[0], ny = P.n[1], nz = P.n[2];
    const long long nc = P.nc;
    const bool perx = P.per[0] != 0, pery = P.per[1] != 0, perz = P.per[2] != 0;
    const int b0 = tile % tiles0, b1 = tile / tiles0;
    const int gx = b0 * (ROW_X - 2) - 1 + tx, gy = b1 * (BY - 2) - 1 + ty;
    const int sx = gx < 0 ? (perx ? nx - 1 : 0) : (gx >= nx ? (perx && gx == nx ? 0 : nx - 1) : gx);
    const int sy = gy < 0 ? (pery ? ny - 1 : 0) : (gy >= ny ? (pery && gy == ny ? 0 : ny - 1) : gy);
    const bool own = tx >= 1 && tx <= ROW_X - 2 && gx < nx && ty >= 1 && ty <= BY - 2 && gy < ny;
    const bool glo = !NW && !perx && gx == -1, ghi = !NW && !perx && gx == nx;
    const bool xlo = !NW && !perx && b0 == 0, xhi = !NW && !perx && b0 * (ROW_X - 2) - 1 + ROW_X > nx;
    const bool bot = !NW && !pery && gy == 0, top = !NW && !pery && gy == ny - 1;
    const T rxl = P.rlo[0], rxh = P.rhi[0], ryl = P.rlo[1], ryh = P.rhi[1];
    const int gxc = min(max(gx, 0), nx - 1), gyc = min(max(gy, 0), ny - 1);
    const RowCoef<T> cx = row_coef<T, UNI>(P, 0, perx ? sx : gxc, perx ? sx + 1 : min(max(gx + 1, 0), nx), sg);
    const RowCoef<T> cy = row_coef<T, UNI>(P, 1, pery ? sy : gyc, (pery ? sy : gyc) + 1, sg);
    T wyl = T(0.5), kyl = cy.k;
    if constexpr (!UNI && !NW) {
        wyl = P.m[1].w[gyc];
        kyl = sg * (P.h * P.c) * P.m[1].gn[gyc];
    }
    const int p0 = ck * chunk, p1 = min(p0 + chunk, nz);
    const int cbase = ty * ROW_X + tx;
    const int up = min(ty + 1, BY - 1) * ROW_X + tx, dn = max(ty - 1, 0) * ROW_X + tx;
    auto at = [&](int slot, int c) -> T& { return lds[slot * SQ + c]; };
    const int hY = h * S::NY, hP = h * S::NP;
    auto phi_at = [&](int buf, int k, int c) -> T& { return at(S::PHI + 2 * S::NY * buf + half_slot<LAT>(1, k) + hY, c); };

    // global element of the lane's first velocity in its column, per plane
    const long long qstep = h ? -nc : nc, plane = (long long)nx * ny;
    const long long q0 = (h ? (long long)(Q - 1) * nc : 0) + (long long)sy * nx + sx;
    const long long rcol = (long long)LAT::REST * nc + (long long)sy * nx + sx;
    const long long gcol = (long long)sy * nx + sx;
    auto plane_of = [&](int p) -> int { return perz ? (p < 0 ? nz - 1 : (p >= nz ? p - nz : p)) : min(max(p, 0), nz - 1); };
    auto load_plane = [&](int p, T (&f)[K], T& r, T (&g)[3]) {
        const long long o = (long long)plane_of(p) * plane;
        const T* fp = fin + (q0 + o);
#pragma unroll
        for (int k = 0; k < K; ++k) f[k] = fp[k * qstep];
        r = fin[rcol + o];
        if constexpr (FIELD) {
#pragma unroll
            for (int d = 0; d < 3; ++d) g[d] = force ? force[d * nc + gcol + o] : T(0);
        }
    };
    auto load_own = [&](int p, T (&f)[K], T& r) {
        const long long o = (long long)p * plane;
        const T* fp = fin + (q0 + o);
#pragma unroll
        for (int k = 0; k < K; ++k) f[k] = fp[k * qstep];
        r = fin[rcol + o];
    };
    // f-bar-plus (Eq. f_bar_+) of a loaded plane, ghost columns included
    auto make_phi = [&](const T (&f)[K], T r, T (&g)[3], T (&phi)[K], T& pr) {
        T G[3] = {T(0), T(0), T(0)};
        if constexpr (ACC) {
#pragma unroll
            for (int d = 0; d < 3; ++d) G[d] = gt * (FIELD ? P.G0[d] + g[d] : P.G0[d]);
        }
        const EqR<T> E = r3_point<LAT, T, ORIG, ACC>(P, f, r, sg, G, P.h);
#pragma unroll
        for (int k = 0; k < K; ++k) phi[k] = r3_relax<LAT, T, ACC>(E, k, P.B1, P.C1, f[k]);
        const T fe = T(LAT::w(LAT::REST)) * E.a;
        pr = fma_(P.B1, fe - r, r);
        if constexpr (ACC) pr = fma_(P.C1 * (T(0) - E.g), fe, pr);
        if (xlo) {
            auto ghost = [&](T& a) {
                const T s1 = row_next(a), s2 = row_next(s1), v = fma_(rxl, s2 - s1, s1);
                a = glo ? v : a;
            };
#pragma unroll
            for (int k = 0; k < K; ++k) ghost(phi[k]);
            ghost(pr);
            if constexpr (FIELD) {
#pragma unroll
                for (int d = 0; d < 3; ++d) ghost(g[d]);
            }
        }
        if (xhi) {
            auto ghost = [&](T& a) {
                const T s1 = row_prev(a), s2 = row_prev(s1), v = fma_(rxh, s2 - s1, s1);
                a = ghi ? v : a;
            };
#pragma unroll
            for (int k = 0; k < K; ++k) ghost(phi[k]);
            ghost(pr);
            if constexpr (FIELD) {
#pragma unroll
                for (int d = 0; d < 3; ++d) ghost(g[d]);
            }
        }
    };
    // X and Y of a plane whose phi is in LDS buffer `buf`
    auto make_xy = [&](int buf, const T (&phi)[K], T (&X)[K], T (&Y)[K]) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (LAT::e(k, 0) != 0) X[k] = r3_deriv<T, UNI>(cx, row_prev(phi[k]), phi[k], row_next(phi[k]));
            if (LAT::e(k, 1) != 0) {
                T u = phi_at(buf, k, up), d = phi_at(buf, k, dn);
                if constexpr (!NW) {
                    const T gu = fma_(ryh, d - phi[k], phi[k]), gd = fma_(ryl, u - phi[k], phi[k]);
                    u = top ? gu : u;
                    d = bot ? gd : d;
                }
                Y[k] = r3_deriv<T, UNI>(cy, d, phi[k], u);
            }
        }
    };
    auto psi_z = [&](int k, const T (&phi)[K], const T (&X)[K], const T (&Y)[K]) -> T {
        return r3_minus(r3_minus(phi[k], LAT::e(k, 0), X[k]), LAT::e(k, 1), Y[k]);
    };
    const T hh = T(0.5) * P.h;
    auto face_acc = [&](const T (&l)[3], const T (&r)[3], T w, T (&G)[3]) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if constexpr (!ACC) G[d] = T(0);
            else if constexpr (!FIELD) G[d] = gth * P.G0[d];
            else G[d] = gth * (P.G0[d] + fma_(w, r[d] - l[d], l[d]));
        }
    };
    auto to_lds = [&](int b, const T (&phi)[K]) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (LAT::e(k, 1) != 0) phi_at(b, k, cbase) = phi[k];
    };
    // Planes arrive one after the other: p0 - 1, p0, .., p1.  Beyond the high wall
    // lies a ghost plane, extrapolated from the two planes that arrived last.  At
    // the low wall the march starts with plane 1: what plane 0 needs from below is
    // formed before it, from planes 0 and 1.
    const bool low = LOW && !perz && p0 == 0;
    const int prime = 2;  // arrivals before the first update
    auto plane_at = [&](int i) { return p0 - 1 + i; };
    // phi of the plane before the one that arrives is C, of the one before that
    // M (the e_z != 0 part; all of it at walls); X and Y of C; the z interface
    // below C; the entering values of the NEQ rule of a z wall.  The e_y != 0 part
    // of phi is read back from LDS where it is needed.
    T phM[K], prM = T(0), zlo[K], zW[K];
    T gM[3] = {T(0), T(0), T(0)}, gC[3] = {T(0), T(0), T(0)}, gN[3] = {T(0), T(0), T(0)};
    int buf = 0;

    // Arrival i.  The register sets C and N (phi, X, Y and the state f of the
    // plane) change places from one arrival to the next in the wall-free body.
    auto arrive = [&](int i, T (&phC)[K], T& prC, T (&XC)[K], T (&YC)[K], T (&fC)[K], T& rC, T (&phN)[K], T& prN,
                      T (&XN)[K], T (&YN)[K], T (&fN)[K], T& rN) {
        const int p = plane_at(i);
        const bool full = i >= prime;  // plane p - 1 is updated
        const bool ghost = !NW && !perz && p == nz;
        RowCoef<T> m = row_coef<T, UNI>(P, 2, plane_of(p - 1), p < 0 ? 0 : p, sg);
        T acc[K], fp[K], fpr = T(0), gP[3] = {T(0), T(0), T(0)};  // fluxes; f~+ of Eq. (f_tilde_+)
        // a: f-bar-plus of plane p
        if (ghost) {
            // beyond C with M inside
            const T q = P.rhi[2];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (LAT::e(k, 1) != 0) phC[k] = phi_at(buf ^ 1, k, cbase);
                phN[k] = fma_(q, phM[k] - phC[k], phC[k]);
            }
            prN = fma_(q, prM - prC, prC);
            if constexpr (FIELD) {
#pragma unroll
                for (int d = 0; d < 3; ++d) gN[d] = fma_(q, gM[d] - gC[d], gC[d]);
            }
        } else {
            make_phi(fN, rN, gN, phN, prN);
        }
        if (full) {
            // b: Z of plane p - 1 and its psi_y (to LDS)
            T Z[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (LAT::e(k, 1) != 0) phC[k] = phi_at(buf ^ 1, k, cbase);
                if (LAT::e(k, 2) != 0) Z[k] = r3_deriv<T, UNI>(m, phM[k], phC[k], phN[k]);
                if (!only_y<LAT>(k))
                    at(S::PSI + psi_slot<LAT>(k) + hP, cbase) =
                        r3_minus(r3_minus(phC[k], LAT::e(k, 0), XC[k]), LAT::e(k, 2), Z[k]);
            }
            if (h == 0) at(S::RESTV, cbase) = prC;
            if constexpr (FIELD) {
                if (h == 0) {
#pragma unroll
                    for (int d = 0; d < 3; ++d) at(S::FORCE + d, cbase) = gC[d];
                }
            }
            to_lds(buf, phN);
            // c: x interfaces of plane p - 1: the lane's upper one, the lower
            // one is that of the lane before
            T v[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const T ps = r3_minus(r3_minus(phC[k], LAT::e(k, 1), YC[k]), LAT::e(k, 2), Z[k]);
                const T psR = row_next(ps);
                const T phR = LAT::e(k, 0) != 0 ? row_next(phC[k]) : psR;
                v[k] = r3_recon<T, UNI>(LAT::e(k, 0), cx.w, cx.k, ps, psR, phC[k], phR);
            }
            const T r = r3_recon<T, UNI>(0, cx.w, cx.k, prC, row_next(prC), prC, prC);
            T G[3], gR[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) gR[d] = FIELD ? row_next(gC[d]) : T(0);
            face_acc(gC, gR, cx.w, G);
            EqR<T> E = r3_point<LAT, T, ORIG, ACC>(P, v, r, sg, G, hh);
            if (xlo || xhi) {
                // wall faces: the opposite interface is the upper one of the
                // next lane (low wall, ghost lane) or of the previous one
#pragma unroll 1
                for (int side = 0; side < 2; ++side) {
                    if (!(side ? xhi : xlo)) continue;
                    T W[K];
                    r3_enter<LAT, T, 0, ORIG>(P, side, E, v, sg, gth, W);
#pragma unroll
                    for (int k = 0; k < K; ++k)
                        if (LAT::e(k, 0) != 0) W[k] = side ? row_prev(W[k]) : row_next(W[k]);
                    if (side ? gx == nx - 1 : glo) r3_wall<LAT, T, 0>(P, side, side ? -1 : 1, v, W, sg);
                }
                E = r3_point<LAT, T, ORIG, ACC>(P, v, r, sg, G, hh);
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if constexpr (OWN) fp[k] = fma_(phC[k] - fC[k], T(1.0 / 3.0), phC[k]);
                acc[k] = LAT::e(k, 2) != 0 ? T(LAT::e(k, 2)) * m.fd * zlo[k] : T(0);
                if (LAT::e(k, 0) == 0) continue;
                const T u = r3_relax<LAT, T, ACC>(E, k, P.B7, P.C7, v[k]);
                acc[k] = fma_(T(-LAT::e(k, 0)) * cx.fd, u - row_prev(u), acc[k]);
            }
            if constexpr (OWN) fpr = fma_(prC - rC, T(1.0 / 3.0), prC);
        } else {
            to_lds(buf, phN);
        }
        __syncthreads();
        // d: X, Y of plane p; the z interface below it
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (LAT::e(k, 1) != 0) phN[k] = phi_at(buf, k, cbase);
        make_xy(buf, phN, XN, YN);
        if (i >= 1) {
            T v[K], r, G[3];
#pragma unroll
            for (int k = 0; k < K; ++k)
                v[k] = r3_recon<T, UNI>(LAT::e(k, 2), m.w, m.k, psi_z(k, phC, XC, YC), psi_z(k, phN, XN, YN), phC[k],
                                        phN[k]);
            r = r3_recon<T, UNI>(0, m.w, m.k, prC, prN, prC, prN);
            face_acc(gC, gN, m.w, G);
            if (ghost) r3_wall<LAT, T, 2>(P, 5, -1, v, zW, sg);
            const EqR<T> E = r3_point<LAT, T, ORIG, ACC>(P, v, r, sg, G, hh);
            if (!NW && !perz && p == nz - 1) r3_enter<LAT, T, 2, ORIG>(P, 5, E, v, sg, gth, zW);
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (LAT::e(k, 2) != 0) zlo[k] = r3_relax<LAT, T, ACC>(E, k, P.B7, P.C7, v[k]);
        }
        if (full) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (LAT::e(k, 2) != 0) acc[k] = fma_(T(-LAT::e(k, 2)) * m.fd, zlo[k], acc[k]);
            asm volatile("" ::: "memory");
            // e: y interfaces of plane p - 1
            T v[K], r, G[3], u[K];
            // between this row and the one below (lower) or above; ghost: the
            // row beyond is extrapolated with the row inside
            auto row_face = [&](bool lower, bool ghost_row) {
                const int c = lower != ghost_row ? dn : up;
                const T re = lower ? ryl : ryh;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const T ho = LAT::e(k, 1) != 0 ? phi_at(buf ^ 1, k, cbase) : T(0);
                    const T po = only_y<LAT>(k) ? ho : at(S::PSI + psi_slot<LAT>(k) + hP, cbase);
                    T hn = LAT::e(k, 1) != 0 ? phi_at(buf ^ 1, k, c) : T(0);
                    T pn = only_y<LAT>(k) ? hn : at(S::PSI + psi_slot<LAT>(k) + hP, c);
                    if (ghost_row) {
                        pn = fma_(re, pn - po, po);
                        if (LAT::e(k, 1) != 0) hn = fma_(re, hn - ho, ho);
                    }
                    v[k] = r3_recon<T, UNI>(LAT::e(k, 1), lower ? wyl : cy.w, lower ? kyl : cy.k, lower ? pn : po,
                                            lower ? po : pn, lower ? hn : ho, lower ? ho : hn);
                }
                T rn = at(S::RESTV, c);
                if (ghost_row) rn = fma_(re, rn - prC, prC);
                r = r3_recon<T, UNI>(0, lower ? wyl : cy.w, T(0), lower ? rn : prC, lower ? prC : rn, T(0), T(0));
                T gl[3], gr[3];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    T gn = FIELD ? at(S::FORCE + d, c) : T(0);
                    if (FIELD && ghost_row) gn = fma_(re, gn - gC[d], gC[d]);
                    gl[d] = lower ? gn : gC[d];
                    gr[d] = lower ? gC[d] : gn;
                }
                face_acc(gl, gr, lower ? wyl : cy.w, G);
            };
            row_face(false, false);
            {
                const EqR<T> E = r3_point<LAT, T, ORIG, ACC>(P, v, r, sg, G, hh);
#pragma unroll
                for (int k = 0; k < K; ++k)
                    if (LAT::e(k, 1) != 0) u[k] = r3_relax<LAT, T, ACC>(E, k, P.B7, P.C7, v[k]);
            }
            if constexpr (!NW) {
                // wall rows: the opposite interface, then the wall face
#pragma unroll 1
                for (int side = 0; side < 2; ++side) {
                    if (!__any(side ? top : bot)) continue;
                    if (side ? top : bot) {
                        T W[K];
#pragma unroll 1
                        for (int pass = 0; pass < 2; ++pass) {
                            row_face((side != 0) != (pass != 0), pass != 0);
                            if (pass) r3_wall<LAT, T, 1>(P, 2 + side, side ? -1 : 1, v, W, sg);
                            const EqR<T> E = r3_point<LAT, T, ORIG, ACC>(P, v, r, sg, G, hh);
                            if (!pass) {
                                r3_enter<LAT, T, 1, ORIG>(P, 2 + side, E, v, sg, gth, W);
                                continue;
                            }
#pragma unroll
                            for (int k = 0; k < K; ++k) {
                                if (LAT::e(k, 1) == 0) continue;
                                const T w = r3_relax<LAT, T, ACC>(E, k, P.B7, P.C7, v[k]);
                                if (side) u[k] = w;
                                else if (ty > 0) at(S::FLUX + half_slot<LAT>(1, k) + hY, dn) = w;
                            }
                        }
                    }
                }
            }
            // the row below a wall stores nothing: its slot holds the wall face
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (LAT::e(k, 1) == 0) continue;
                if (NW || pery || gy != -1) at(S::FLUX + half_slot<LAT>(1, k) + hY, cbase) = u[k];
                acc[k] = fma_(T(-LAT::e(k, 1)) * cy.fd, u[k], acc[k]);
            }
        }
        // the next plane (and without OWN f~ of plane p - 1 again) is on its way
        // during the barrier
        T fo[K], ro = T(0);
        if (!OWN && full) load_own(p - 1, fo, ro);
        if (i < prime + p1 - p0 - 1) load_plane(plane_at(i + 1), fC, rC, gP);
        __syncthreads();
        if (full) {
            // f: the lower y interface's fluxes; store
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (LAT::e(k, 1) != 0) {
                    acc[k] = fma_(T(LAT::e(k, 1)) * cy.fd, at(S::FLUX + half_slot<LAT>(1, k) + hY, dn), acc[k]);
                    if (!OWN) phC[k] = phi_at(buf ^ 1, k, cbase);
                }
                if constexpr (!OWN) fp[k] = fma_(phC[k] - fo[k], T(1.0 / 3.0), phC[k]);
            }
            if constexpr (!OWN) fpr = fma_(prC - ro, T(1.0 / 3.0), prC);
            if (own) {
                T* o = fout + (q0 + (long long)(p - 1) * plane);
#pragma unroll
                for (int k = 0; k < K; ++k) o[k * qstep] = fp[k] + acc[k];
                if (h == 0) fout[rcol + (long long)(p - 1) * plane] = fpr;
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (!NW || LAT::e(k, 2) != 0) phM[k] = LAT::e(k, 1) != 0 ? phi_at(buf ^ 1, k, cbase) : phC[k];
        if constexpr (!NW) prM = prC;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            gM[d] = gC[d];
            gC[d] = gN[d];
            gN[d] = gP[d];
        }
        buf ^= 1;
    };
    const int count = prime + p1 - p0;
    T phA[K], prA = T(0), XA[K], YA[K], fA[K], rA, phB[K], prB, XB[K], YB[K], fB[K], rB;
#pragma unroll
    for (int k = 0; k < K; ++k) phA[k] = XA[k] = YA[k] = fA[k] = T(0);
    const int i0 = low ? 2 : 0;
    load_plane(plane_at(i0), fB, rB, gN);
    if constexpr (LOW) {
        if (low) {
            // planes 0 and 1, the interface between them and from it the wall's
            // face, whose ghost plane is extrapolated (psi too, as beside the rows
            // at y walls): as many planes as a march inside the mesh primes.  With
            // planes 0 and 1, the ghost plane, 0 and 1 as arrivals of the march, a
            // 24 x 22 x 29 stretched cavity took 21.2 us a step, now 15.6 (19.4 on
            // the LDS march before), 822 x 215 x 6 308, now 225 (274).
            T ph1[K], pr1, X1[K], Y1[K], v[K], W[K], G[3], gl[3];
            load_plane(0, fA, rA, gC);
            make_phi(fA, rA, gC, phA, prA);
            make_phi(fB, rB, gN, ph1, pr1);
            to_lds(1, phA);
            to_lds(0, ph1);
            __syncthreads();
            make_xy(1, phA, XA, YA);
            make_xy(0, ph1, X1, Y1);
            const RowCoef<T> m = row_coef<T, UNI>(P, 2, 0, 1, sg), m0 = row_coef<T, UNI>(P, 2, 0, 0, sg);
            const T q = P.rlo[2];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                X1[k] = psi_z(k, ph1, X1, Y1);  // psi of the planes
                Y1[k] = psi_z(k, phA, XA, YA);
                v[k] = r3_recon<T, UNI>(LAT::e(k, 2), m.w, m.k, Y1[k], X1[k], phA[k], ph1[k]);
            }
            face_acc(gC, gN, m.w, G);
            const EqR<T> E = r3_point<LAT, T, ORIG, ACC>(P, v, r3_recon<T, UNI>(0, m.w, m.k, prA, pr1, T(0), T(0)), sg, G, hh);
            r3_enter<LAT, T, 2, ORIG>(P, 4, E, v, sg, gth, W);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                phM[k] = fma_(q, ph1[k] - phA[k], phA[k]);
                v[k] = r3_recon<T, UNI>(LAT::e(k, 2), m0.w, m0.k, fma_(q, X1[k] - Y1[k], Y1[k]), Y1[k], phM[k], phA[k]);
            }
#pragma unroll
            for (int d = 0; d < 3; ++d) gl[d] = fma_(q, gN[d] - gC[d], gC[d]);
            face_acc(gl, gC, m0.w, G);
            r3_wall<LAT, T, 2>(P, 4, 1, v, W, sg);
            const EqR<T> B = r3_point<LAT, T, ORIG, ACC>(
                P, v, r3_recon<T, UNI>(0, m0.w, m0.k, fma_(q, pr1 - prA, prA), prA, T(0), T(0)), sg, G, hh);
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (LAT::e(k, 2) != 0) zlo[k] = r3_relax<LAT, T, ACC>(B, k, P.B7, P.C7, v[k]);
            __syncthreads();
        }
    }
    // two arrivals per trip, so that no register is copied from set to set; the
    // wall body of D3Q19 has no registers left for it (spills: 375 -> 386 us a
    // step of the 128^3 cavity; D3Q27 at 96^3 363 -> 344 with it)
    if constexpr (NW || LAT::Q != 19) {
        for (int i = i0;; i += 2) {
            arrive(i, phA, prA, XA, YA, fA, rA, phB, prB, XB, YB, fB, rB);
            if (i + 1 == count) break;
            arrive(i + 1, phB, prB, XB, YB, fB, rB, phA, prA, XA, YA, fA, rA);
            if (i + 2 == count) break;
        }
    } else {
#pragma unroll 1
        for (int i = i0; i < count; ++i) {
            arrive(i, phA, prA, XA, YA, fA, rA, phB, prB, XB, YB, fB, rB);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                phA[k] = phB[k];
                if (LAT::e(k, 0) != 0) XA[k] = XB[k];
                if (LAT::e(k, 1) != 0) YA[k] = YB[k];
                const T x = fA[k];
                fA[k] = fB[k];
                fB[k] = x;
            }
            prA = prB;
            const T x = rA;
            rA = rB;
            rB = x;
        }
    }
}

#pragma clang fp contract(fast)

// does the tile and march chunk stay clear of every wall?
template <typename T>
__device__ __forceinline__ bool row_no_wall(const Inst<T>& P, int BY, int tiles0, int tile, int ck, int chunk)
{
    const int b0 = tile % tiles0, b1 = tile / tiles0;
    const int x0 = b0 * (ROW_X - 2) - 1, y0 = b1 * (BY - 2) - 1;
    if (!P.per[0] && (x0 < 0 || x0 + ROW_X > P.n[0])) return false;
    if (!P.per[1] && (y0 <= 0 || y0 + BY >= P.n[1])) return false;
    const int p0 = ck * chunk, p1 = min(p0 + chunk, P.n[2]);
    if (!P.per[2] && (p0 < 1 || p1 > P.n[2] - 1)) return false;
    return true;
}

// Tile rows, and waves per SIMD the kernel is compiled for: the most that its
// registers allow.  D3Q19 at two takes 248 to 256 and spills none on uniform
// meshes without a field, 2 to 21 on stretched ones, 24 to 52 with a field, 17 and
// 71 in the batch's kernels (four bodies each); one more wave spills throughout
// and runs 1.5 times as long.  Eight rows give workgroups of
// four waves, two of which share a CU, so that one computes while
// another waits at a barrier; 16 rows (one workgroup per CU) were slower in
// spite of their smaller halo (128^3 periodic: 308 against 272 us).
template <class LAT, typename T>
struct RowShape {
    static constexpr int BY = 8;
    static constexpr int WPE = LAT::Q == 19 ? 2 : 1;
    static constexpr int NT = 2 * ROW_X * BY;
};

#define ROW_BOUNDS(LAT, T)                                                            \
    __attribute__((amdgpu_flat_work_group_size(RowShape<LAT, T>::NT, RowShape<LAT, T>::NT), \
                   amdgpu_waves_per_eu(RowShape<LAT, T>::WPE)))

// Planes marched per workgroup.  x = tiles x ceil(n / c) / S rounds of
// workgroups on S resident ones; the last round is full or not, so their
// number is taken as the mean of x + 0.8 and of ceil(x), each of c + 0.9
// arrivals (the two that prime a march are worth about one).  The chunk of 1, 2,
// 3, 4, 6, 8, .. 32 planes that minimises the product, the larger one on
// ties.  Measured (us a step for c = 2, 3, 4, 6, 8): 128^3 cavity 415, 378, 355,
// 353, 337 (16: 355); 120 x 101 x 90 cavity 240, 222, 216, 208, 225; 96 x 64 x 75
// with a field 112, 103, 105, 107, 118; 40 x 90 x 30 49, 42, 52, 62, 76; 48 x 40 x
// 36 41, 51, 52, 69, 87; D3Q27 75 x 66 x 50 127, 121, 126, 131, 144.  Over
// sixteen such meshes its choice is within 2 % of the best but for two (7, 10 %).
inline int row_chunk(long long tiles, int nz, long long slots)
{
    slots = slots > 1 ? slots : 1;
    int best = 1;
    double best_cost = 1e300;
    for (int c : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32}) {
        const int cc = c < nz ? c : nz;
        const long long wgs = tiles * ((nz + cc - 1) / cc);
        const double rounds = 0.5 * ((double)wgs / (double)slots + 0.8) + 0.5 * (double)((wgs + slots - 1) / slots);
        const double cost = rounds * (cc + 0.9);
        if (cost <= best_cost) {
            best_cost = cost;
            best = cc;
        }
        if (cc >= nz) break;
    }
    return best;
}

template <class LAT, typename T, bool UNI, bool ACC, bool FIELD, bool ORIG>
__global__ ROW_BOUNDS(LAT, T) void k_row(const Inst<T>* __restrict__ Pp, const T* __restrict__ fin,
                                         const T* __restrict__ force, T* __restrict__ fout, double t, int chunk,
                                         int tiles0, int tiles)
{
    constexpr int BY = RowShape<LAT, T>::BY;
    __shared__ T lds[RowSlots<LAT>::count(FIELD) * ROW_X * BY];
    const Inst<T>& P = *Pp;
    T gt = T(1), gth = T(1);
    if (ACC || P.osc) {
        gt = tfac_dev(P, t);
        gth = tfac_dev(P, t + 0.5 * P.dtd);
    }
    gt = uniform(gt);
    gth = uniform(gth);
    // the chunks at the z walls first, then the others, each part in XCD order:
    // every tile of theirs is on the wall body, and with all chunks in one order
    // the first and the last XCD have nothing else (128^3 cavity 357 -> 336 us a
    // step, 120 x 101 x 90 181 -> 176; bands of tiles with all their chunks per
    // XCD gain as much there, but then the y walls sit on two XCDs, D3Q27 136 -> 150)
    const int nck = (P.n[2] + chunk - 1) / chunk, nb = (int)gridDim.x, wz = P.per[2] || nck < 3 ? 0 : 2 * tiles;
    const bool zw = (int)blockIdx.x < wz;
    const int b = zw ? xcd_order((int)blockIdx.x, wz) : xcd_order((int)blockIdx.x - wz, nb - wz);
    const int tile = b % tiles, ck = zw ? (b < tiles ? 0 : nck - 1) : b / tiles + (wz ? 1 : 0);
    // D3Q19's wall body begins at a low wall by itself; D3Q27's has no registers
    // left for that (75 x 66 x 50: 124 us a step, 120 with a body of its own)
#define DUGKS_ROW(NW, LOW) \
    row_body<LAT, T, BY, UNI, ACC, FIELD, ORIG, NW, LOW>(P, fin, force, fout, gt, gth, chunk, tiles0, tile, ck, lds)
    if (row_no_wall(P, BY, tiles0, tile, ck, chunk)) DUGKS_ROW(true, false);
    else if (LAT::Q == 19 || (!P.per[2] && ck == 0)) DUGKS_ROW(false, true);
    else if constexpr (LAT::Q != 19) DUGKS_ROW(false, false);
#undef DUGKS_ROW
}

template <class LAT, typename T, bool UNI, bool ACC, bool FIELD, bool ORIG>
static int launch_row(dugks_ctx* ctx, const Inst<T>& P, const void* fin, void* fout, const void* force, double t,
                      hipStream_t st, int chunk)
{
    constexpr int BY = RowShape<LAT, T>::BY, NT = RowShape<LAT, T>::NT;
    auto kern = k_row<LAT, T, UNI, ACC, FIELD, ORIG>;
    static const long long slots = resident_slots(kern, NT, 0, ctx->n_cu);
    const int tiles0 = (P.n[0] + ROW_X - 3) / (ROW_X - 2), tiles1 = (P.n[1] + BY - 3) / (BY - 2);
    const long long tiles = (long long)tiles0 * tiles1;
    chunk = chunk > 0 ? std::min(chunk, P.n[2]) : row_chunk(tiles, P.n[2], slots);
    const long long nb = tiles * ((P.n[2] + chunk - 1) / chunk);
    if (nb > 0x7fffffffLL) return fail(ctx, DUGKS_EUNSUPPORTED, "mesh too large for one launch");
    hipLaunchKernelGGL(kern, dim3((unsigned)nb), dim3(NT), 0, st, (const Inst<T>*)ctx->inst_dev, (const T*)fin,
                       (const T*)force, (T*)fout, t, chunk, tiles0, (int)tiles);
    return hip_check(ctx, hipGetLastError(), "step launch");
}

template <class LAT, typename T, bool UNI, bool ORIG>
static int launch_row_acc(dugks_ctx* ctx, const Inst<T>& P, const void* fin, void* fout, const void* force, double t,
                          hipStream_t st, int chunk)
{
    if (force) return launch_row<LAT, T, UNI, true, true, ORIG>(ctx, P, fin, fout, force, t, st, chunk);
    if (P.G0[0] != T(0) || P.G0[1] != T(0) || P.G0[2] != T(0))
        return launch_row<LAT, T, UNI, true, false, ORIG>(ctx, P, fin, fout, force, t, st, chunk);
    return launch_row<LAT, T, UNI, false, false, ORIG>(ctx, P, fin, fout, force, t, st, chunk);
}

// many instances in one launch: workgroup b in XCD order belongs to the
// instance i with bstart[i] <= b < bstart[i + 1], whose tile counts and chunk are
// geom[i]; instance i is at time (*step0 + step) dt_i (a device counter, so a
// captured graph replays with advancing time).
// Four bodies in one kernel spill more than a single mesh's (RowShape).  us a step,
// LDS march with its own kernel -> this one: eight 40^3 boxes with walls 177 -> 127,
// with a field 314 -> 149; it stays a little behind for few boxes of uneven sides,
// where most tiles hold walls (two of 23 x 18 x 73: 53.3 -> 55.6)
template <class LAT, typename T, bool FIELD>
__global__ ROW_BOUNDS(LAT, T) void k_row_batch(const Inst<T>* __restrict__ insts, const long long* __restrict__ bstart,
                                               const BatchGeom* __restrict__ geom, int ninst,
                                               const T* __restrict__ fin, const T* __restrict__ forces,
                                               T* __restrict__ fout, const long long* __restrict__ step0, int step)
{
    constexpr int BY = RowShape<LAT, T>::BY;
    __shared__ T lds[RowSlots<LAT>::count(FIELD) * ROW_X * BY];
    const long long b = xcd_order((int)blockIdx.x, (int)gridDim.x);
    int lo = 0, hi = ninst - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (bstart[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    const Inst<T>& P = insts[lo];
    const BatchGeom g = geom[lo];
    const int local = (int)(b - bstart[lo]), ntile = g.tiles0 * g.tiles1;
    const int tile = local % ntile, ck = local / ntile;
    const double t = (double)(*step0 + step) * P.dtd;
    const T gt = uniform(tfac_dev(P, t)), gth = uniform(tfac_dev(P, t + 0.5 * P.dtd));
    const T* force = (FIELD && forces && P.foff >= 0) ? forces + P.foff : nullptr;
    const bool nw = row_no_wall(P, BY, g.tiles0, tile, ck, g.chunk);
    fin += P.off;
    fout += P.off;
    if (P.uni) {
        if (nw) row_body<LAT, T, BY, true, true, FIELD, false, true, false>(P, fin, force, fout, gt, gth, g.chunk, g.tiles0, tile, ck, lds);
        else row_body<LAT, T, BY, true, true, FIELD, false, false, true>(P, fin, force, fout, gt, gth, g.chunk, g.tiles0, tile, ck, lds);
    } else {
        if (nw) row_body<LAT, T, BY, false, true, FIELD, false, true, false>(P, fin, force, fout, gt, gth, g.chunk, g.tiles0, tile, ck, lds);
        else row_body<LAT, T, BY, false, true, FIELD, false, false, true>(P, fin, force, fout, gt, gth, g.chunk, g.tiles0, tile, ck, lds);
    }
}

// tile of the batched form (halo included), and the workgroups of it resident
// on the device at once
template <class LAT, typename T>
long long row_batch_slots(int n_cu)
{
    return resident_slots(k_row_batch<LAT, T, false>, RowShape<LAT, T>::NT, 0, n_cu);
}

template <class LAT, typename T>
void row_batch_launch(const void* insts, const long long* bstart, const BatchGeom* geom, int n, long long nblocks,
                      const void* fin, const void* forces, void* fout, const long long* step0, int step, hipStream_t st)
{
    auto kern = forces ? k_row_batch<LAT, T, true> : k_row_batch<LAT, T, false>;
    hipLaunchKernelGGL(kern, dim3((unsigned)nblocks), dim3(RowShape<LAT, T>::NT), 0, st, (const Inst<T>*)insts, bstart,
                       geom, n, (const T*)fin, (const T*)forces, (T*)fout, step0, step);
}

// one step on the row kernel
template <class LAT, typename T>
int row_step(dugks_ctx* ctx, const Inst<T>& P, const void* fin, void* fout, const void* force, double t, hipStream_t st,
             int chunk)
{
    if (P.orig)
        return P.uni ? launch_row_acc<LAT, T, true, true>(ctx, P, fin, fout, force, t, st, chunk)
                     : launch_row_acc<LAT, T, false, true>(ctx, P, fin, fout, force, t, st, chunk);
    return P.uni ? launch_row_acc<LAT, T, true, false>(ctx, P, fin, fout, force, t, st, chunk)
                 : launch_row_acc<LAT, T, false, false>(ctx, P, fin, fout, force, t, st, chunk);
}

}  // namespace dugks
