// wave.hpp -- register exchange between the lanes of a wavefront, and the
// per-cell stages of the D2Q9 step with every rounding written out.
//
// The stages are used by several kernels that must give the same bits for
// the same cell whatever tile, chunk or batch it is computed in, and with or
// without the acceleration terms where the acceleration is zero.  So no
// contraction is left to the compiler here (fp contract off): every fused
// multiply-add is spelled out, and an acceleration term is one more fused
// multiply-add whose multiplier is zero without acceleration.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels_general.hpp"

namespace dugks {

// DPP control words: the value of lane l + 1 (wave_shl:1) or l - 1
// (wave_shr:1) of the 64-lane wave; a lane without a source gets 0
constexpr int DPP_NEXT = 0x130, DPP_PREV = 0x138;

template <int CTRL>
__device__ __forceinline__ float lane_dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double lane_dpp(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <typename T>
__device__ __forceinline__ T lane_next(T v) { return lane_dpp<DPP_NEXT>(v); }
template <typename T>
__device__ __forceinline__ T lane_prev(T v) { return lane_dpp<DPP_PREV>(v); }

__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// ---------------------------------------------------------------------------
// D2Q9, one lane per cell.  q = 3 (ex + 1) + (ey + 1), opposite 8 - q; the
// velocities with e_x != 0 are 0, 1, 2 (-1) and 6, 7, 8 (+1), those with
// e_y != 0 are 0, 3, 6 (-1) and 2, 5, 8 (+1).
// ---------------------------------------------------------------------------
#pragma clang fp contract(off)

// rho and e-weighted sums of nine values
template <typename T>
__device__ __forceinline__ void d2_sums(const T (&f)[9], T& rho, T& jx, T& jy)
{
    const T l = f[0] + f[2], r = f[6] + f[8];
    const T sl = l + f[1], sr = r + f[7];
    const T d = f[0] + f[6], u = f[2] + f[8];
    rho = (sl + sr) + ((f[3] + f[5]) + f[4]);
    jx = sr - sl;
    jy = (u - d) + (f[5] - f[3]);
}

// Eqs. (icfeq) and (S) at a point: fe_q = W_q (s_q + e.u B), s_q = a + C
// (e.u)^2; the source is (sG e.G - g) fe_q
template <typename T>
struct EqD2 {
    T a, ux, uy, g, Gx, Gy, B, C;
};

template <typename T, bool ORIG>
__device__ __forceinline__ EqD2<T> d2_eq(const Inst<T>& P, T rho, T ux, T uy, T Gx, T Gy)
{
    EqD2<T> E;
    const T uu = fma_(uy, uy, ux * ux);
    if constexpr (ORIG) {
        E.a = fma_(-(rho * P.hRT), uu, rho);
        E.B = rho * P.cRT;
        E.C = rho * P.c2RT2;
    } else {
        E.a = fma_(-P.eqH, uu, rho);
        E.B = P.eqB;
        E.C = P.eqC;
    }
    E.ux = ux;
    E.uy = uy;
    E.Gx = Gx * P.sG;
    E.Gy = Gy * P.sG;
    E.g = fma_(Gy, uy, Gx * ux) * P.invRT;
    return E;
}

// velocity from the momentum sum (Eq. macro_values), hw the time weight of
// the acceleration
template <typename T, bool ORIG>
__device__ __forceinline__ T d2_vel(const Inst<T>& P, T cir, T j, T G, T hw)
{
    return fma_(hw, G, (ORIG ? cir : P.crho) * j);
}

// moments of nine values and their equilibrium
template <typename T, bool ORIG, bool ACC>
__device__ __forceinline__ EqD2<T> d2_point(const Inst<T>& P, const T (&f)[9], T Gx, T Gy, T hw, T& rho)
{
    T jx, jy;
    d2_sums(f, rho, jx, jy);
    const T cir = ORIG ? P.c / rho : T(0);
    const T ux = ACC ? d2_vel<T, ORIG>(P, cir, jx, Gx, hw) : (ORIG ? cir : P.crho) * jx;
    const T uy = ACC ? d2_vel<T, ORIG>(P, cir, jy, Gy, hw) : (ORIG ? cir : P.crho) * jy;
    return d2_eq<T, ORIG>(P, rho, ux, uy, ACC ? Gx : T(0), ACC ? Gy : T(0));
}

template <typename T>
__device__ __forceinline__ constexpr T d2_w(int q)
{
    return T(D2Q9::w(q));
}

// equilibria of the opposite pair (q, 8 - q), q > 4
template <typename T>
__device__ __forceinline__ void d2_feq_pair(const EqD2<T>& E, int q, T& fp, T& fm)
{
    const T eu = q == 5 ? E.uy : (q == 6 ? E.ux - E.uy : (q == 7 ? E.ux : E.ux + E.uy));
    const T s = fma_(E.C * eu, eu, E.a);
    fp = d2_w<T>(q) * fma_(E.B, eu, s);
    fm = d2_w<T>(q) * fma_(-E.B, eu, s);
}

// v + b (feq - v) + c S for the pair (q, 8 - q), in place
template <typename T, bool ACC>
__device__ __forceinline__ void d2_relax_pair(const EqD2<T>& E, int q, T b, T c, T& vp, T& vm)
{
    T fp, fm;
    d2_feq_pair(E, q, fp, fm);
    vp = fma_(b, fp - vp, vp);
    vm = fma_(b, fm - vm, vm);
    if constexpr (ACC) {
        const T eG = q == 5 ? E.Gy : (q == 6 ? E.Gx - E.Gy : (q == 7 ? E.Gx : E.Gx + E.Gy));
        vp = fma_(c * (eG - E.g), fp, vp);
        vm = fma_(c * (-eG - E.g), fm, vm);
    }
}

// f-bar-plus of one cell (Eq. f_bar_+)
template <typename T, bool ORIG, bool ACC>
__device__ __forceinline__ void d2_phi(const Inst<T>& P, const T (&f)[9], T Gx, T Gy, T (&phi)[9])
{
    T rho;
    const EqD2<T> E = d2_point<T, ORIG, ACC>(P, f, Gx, Gy, P.h, rho);
#pragma unroll
    for (int q = 0; q < 9; ++q) phi[q] = f[q];
#pragma unroll
    for (int q = 5; q < 9; ++q) d2_relax_pair<T, ACC>(E, q, P.B1, P.C1, phi[q], phi[8 - q]);
    const T fe = d2_w<T>(4) * E.a;
    phi[4] = fma_(P.B1, fe - f[4], f[4]);
    if constexpr (ACC) phi[4] = fma_(P.C1 * (T(0) - E.g), fe, phi[4]);
}

// what the NEQ rule takes from the opposite interface of a wall cell: its
// moments and the non-equilibrium part of the three entering velocities
template <typename T>
struct NeqD2 {
    T rho, ux, uy, ne[3];
};

// index of the k-th velocity with component e along axis A
__host__ __device__ constexpr int d2_q(int A, int e, int k) { return A == 0 ? 3 * (e + 1) + k : 3 * k + (e + 1); }

// Capture on an interface of axis A for the wall the velocities of sign
// `into` (+1: low wall) enter through
template <typename T, int A>
__device__ __forceinline__ void d2_capture(const EqD2<T>& E, T rho, const T (&v)[9], int into, NeqD2<T>& I)
{
    T fp[3], fm[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int q = d2_q(A, 1, k);
        if (q > 4) d2_feq_pair(E, q, fp[k], fm[k]);
        else d2_feq_pair(E, 8 - q, fm[k], fp[k]);
    }
    I.rho = rho;
    I.ux = E.ux;
    I.uy = E.uy;
    // the opposite of (+1, k) is (-1, 2 - k)
#pragma unroll
    for (int k = 0; k < 3; ++k)
        I.ne[k] = into > 0 ? v[d2_q(A, 1, k)] - fp[k] : v[d2_q(A, -1, k)] - fm[2 - k];
}

// the wall rules of Eqs. (BB), (NEQ) on a wall face of side s of axis A, in
// place on the entering velocities (component `into` along A)
template <typename T, int A, bool ORIG>
__device__ __forceinline__ void d2_wall(const Inst<T>& P, int s, int into, T (&v)[9], const NeqD2<T>& I, T gth)
{
    const int kind = P.bc[s];
    if (kind == BC_BOUNCE_BACK) {
        T nv[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int t = k - 1;  // component across A
            const T eu = A == 0 ? fma_(T(t), P.uw[s][1], T(into) * P.uw[s][0])
                                : fma_(T(t), P.uw[s][0], T(into) * P.uw[s][1]);
            const T w = t == 0 ? d2_w<T>(1) : d2_w<T>(0);
            const T src = into > 0 ? v[d2_q(A, -1, 2 - k)] : v[d2_q(A, 1, 2 - k)];
            nv[k] = fma_(T(2) * P.eqB * w, eu, src);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (into > 0) v[d2_q(A, 1, k)] = nv[k];
            else v[d2_q(A, -1, k)] = nv[k];
        }
        return;
    }
    const bool vel = kind == BC_NEQ_VELOCITY;
    const T r = vel ? I.rho : wall_density(P, s, gth);
    const T ux = vel ? P.uw[s][0] : I.ux, uy = vel ? P.uw[s][1] : I.uy;
    const EqD2<T> E = d2_eq<T, ORIG>(P, r, ux, uy, T(0), T(0));
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int q = d2_q(A, 1, k);
        T fp, fm;  // of (+1, k) and of its opposite (-1, 2 - k)
        if (q > 4) d2_feq_pair(E, q, fp, fm);
        else d2_feq_pair(E, 8 - q, fm, fp);
        if (into > 0) v[q] = fp + I.ne[k];
        else v[8 - q] = fm + I.ne[2 - k];
    }
}

// interface value of one velocity with component e along the face normal
// (Eq. gradient) from psi = phi - h xi_t d_t phi and phi of its two cells:
// (1 - w) psi_L + w psi_R - e k (phi_R - phi_L), k = h c / (x_R - x_L)
template <typename T, bool UNI>
__device__ __forceinline__ T d2_recon(int e, T w, T k, T psL, T psR, T phL, T phR)
{
    T v;
    if constexpr (UNI) v = T(0.5) * (psL + psR);
    else v = fma_(w, psR - psL, psL);
    if (e > 0) v = fma_(-k, phR - phL, v);
    if (e < 0) v = fma_(k, phR - phL, v);
    return v;
}

// psi of a velocity with tangential component e: phi - e h c d, d the
// cell-centred derivative, from the two neighbours along the tangent.
// Uniform mesh: kp = h c / (2 Delta); stretched: kp = h c cp, km = h c cm
// (the coefficients of the three cells sum to zero).
template <typename T, bool UNI>
__device__ __forceinline__ T d2_psi(int e, T kp, T km, T dn, T ph, T up)
{
    T d;
    if constexpr (UNI) d = kp * (up - dn);
    else d = fma_(kp, up - ph, km * (dn - ph));
    return e > 0 ? ph - d : ph + d;
}

#pragma clang fp contract(fast)

}  // namespace dugks
