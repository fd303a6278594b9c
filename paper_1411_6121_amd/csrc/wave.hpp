// wave.hpp -- register exchange between the lanes of a wavefront, and the
// per-cell stages of the steps with every rounding written out.
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

// value of the partner lane (same column, other half): v_permlane32_swap
// exchanges lanes 32..63 of its first operand with lanes 0..31 of its second;
// with both operands = v the partner's value is the second result in the
// lower half-wave and the first in the upper one.  Both lanes of a pair are
// always active together.
__device__ __forceinline__ unsigned partner_u32(unsigned v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return __lane_id() < 32 ? r[1] : r[0];
}
__device__ __forceinline__ float partner(float v)
{
    return __builtin_bit_cast(float, partner_u32(__builtin_bit_cast(unsigned, v)));
}
__device__ __forceinline__ double partner(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = partner_u32((unsigned)b), hi = partner_u32((unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Lane-pair sums of two values at once: v_permlane32_swap(a, b) leaves
// (a(l), b(l-32)) in its first result and (a(l+32), b(l)) in its second, so
// one add gives the pair sum of a in the lower half-wave and that of b in
// the upper one; a second swap of that sum with a copy of itself hands both
// halves to every lane.  Each sum is the lower lane's value plus the upper
// one's, bitwise what both lanes get from v + partner(v).  The copy is made
// opaque to the compiler so that the swap never sees two equal operands.
__device__ __forceinline__ void pair_sum2_u32(unsigned a, unsigned b, unsigned& r0, unsigned& r1)
{
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    r0 = r[0];
    r1 = r[1];
}
// M: how the pair is combined: 0 both sums plain; 1 a plain, b signed (the
// lane's sign sg, +1 in the lower and -1 in the upper half-wave); 2 both
// signed.  A signed sum is that of sg * x: the lower lane's value minus the
// upper one's, bitwise what sg * x + partner(sg * x) gives, since
// multiplying by -1 is exact.
template <int M>
__device__ __forceinline__ float pair_combine(float x0, float x1, float sg)
{
    if constexpr (M == 0) return x0 + x1;
    else if constexpr (M == 1) return __builtin_fmaf(sg, x1, x0);
    else return x0 - x1;
}
template <int M>
__device__ __forceinline__ double pair_combine(double x0, double x1, double sg)
{
    if constexpr (M == 0) return x0 + x1;
    else if constexpr (M == 1) return __builtin_fma(sg, x1, x0);
    else return x0 - x1;
}
template <int M = 0>
__device__ __forceinline__ void pair_sum2(float a, float b, float& sa, float& sb, float sg = 1.0f)
{
    unsigned x0, x1;
    pair_sum2_u32(__float_as_uint(a), __float_as_uint(b), x0, x1);
    const float sum = pair_combine<M>(__uint_as_float(x0), __uint_as_float(x1), sg);
    unsigned c = __float_as_uint(sum);
    asm volatile("" : "+v"(c));
    unsigned y0, y1;
    pair_sum2_u32(__float_as_uint(sum), c, y0, y1);
    sa = __uint_as_float(y0);
    sb = __uint_as_float(y1);
}
template <int M = 0>
__device__ __forceinline__ void pair_sum2(double a, double b, double& sa, double& sb, double sg = 1.0)
{
    const unsigned long long ua = (unsigned long long)__double_as_longlong(a);
    const unsigned long long ub = (unsigned long long)__double_as_longlong(b);
    unsigned l0, l1, h0, h1;
    pair_sum2_u32((unsigned)ua, (unsigned)ub, l0, l1);
    pair_sum2_u32((unsigned)(ua >> 32), (unsigned)(ub >> 32), h0, h1);
    const double sum = pair_combine<M>(__longlong_as_double((long long)(((unsigned long long)h0 << 32) | l0)),
                                       __longlong_as_double((long long)(((unsigned long long)h1 << 32) | l1)), sg);
    const unsigned long long us = (unsigned long long)__double_as_longlong(sum);
    unsigned clo = (unsigned)us, chi = (unsigned)(us >> 32);
    asm volatile("" : "+v"(clo), "+v"(chi));
    pair_sum2_u32((unsigned)us, clo, l0, l1);
    pair_sum2_u32((unsigned)(us >> 32), chi, h0, h1);
    sa = __longlong_as_double((long long)(((unsigned long long)h0 << 32) | l0));
    sb = __longlong_as_double((long long)(((unsigned long long)h1 << 32) | l1));
}
// the moments of a column from the two lanes' partial sums: rho = rh + rh
// of the partner lane, j[a] = the pair sum of sg * sj[a]
template <int D, typename T>
__device__ __forceinline__ void moment_sums(T rh, const T (&sj)[3], T sg, T& rho, T (&j)[3])
{
    pair_sum2<1>(rh, sj[0], rho, j[0], sg);
    if constexpr (D == 3) {
        pair_sum2<2>(sj[1], sj[2], j[1], j[2], sg);
    } else {
        const T x = sg * sj[1];
        j[1] = x + partner(x);
    }
}

// value of lane l + N (N > 0) or l - N (N < 0) of the lane's 16-lane row
// (DPP row shift; 0 where the source is outside the row)
template <int N>
__device__ __forceinline__ unsigned row_shift_u32(unsigned v)
{
    constexpr int ctrl = N > 0 ? 0x100 + N : 0x110 - N;  // row_shl:N / row_shr:-N
    return (unsigned)__builtin_amdgcn_mov_dpp((int)v, ctrl, 0xf, 0xf, true);
}
template <int N>
__device__ __forceinline__ float row_shift(float v)
{
    return __uint_as_float(row_shift_u32<N>(__float_as_uint(v)));
}
template <int N>
__device__ __forceinline__ double row_shift(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = row_shift_u32<N>((unsigned)b), hi = row_shift_u32<N>((unsigned)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

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
            const T vm = v[d2_q(A, -1, 2 - k)], vp = v[d2_q(A, 1, 2 - k)], src = into > 0 ? vm : vp;
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
