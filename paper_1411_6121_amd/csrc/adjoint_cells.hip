// adjoint_cells.hip -- reverse mode of one D3Q19 step in FP64, any boundary
// set, in three launches: f-bar-plus; the faces; the cells.
//
// The ghost rule is linear, so it is folded into the two cells next to a wall:
// a tangential derivative at a wall cell takes cp' = cp + r cm and cm' = 0 (low
// side), and a wall face is a face of the pair of cells next to it with its own
// weight and difference,
//   low:  w' = (1 - w) r,  g' = -g r;   high: w' = 1 - w r,  g' = -g r,
// r the extrapolation ratio.  The opposite interface of the NEQ rule lies
// between the same pair.  No ghost points are stored or visited.
//
// With fbar(b) = (1-w) psi_L + w psi_R - e k (phi_R - phi_L) and psi = phi -
// sum_t e_t d_t, d_t = kp (phi_+ - phi) + km (phi_- - phi):
//   faces  one thread per interface of an axis between two cells (and per pair
//          next to a wall, which does the wall face too): the adjoints of the
//          interface's values and of its acceleration;
//   cells  one lane per cell and one wave per group of velocities: psi-hat of
//          the cell and of its neighbours from their faces, the transposed
//          derivatives, then (over the four waves) Eq. (f_bar_+) and the
//          moments -> lam_n and the force gradient.
// Faces of axis a are stored with n_a + 1 slots along a: slot c is the
// interface below cell c, slot 0 and n_a of a wall axis are its wall faces.
//
// Bound by the latency of loads from the caches up to some ten thousand cells,
// then by L1 (a load of 64 doubles takes 17 tag lookups) and, beyond the 256 MB
// cache, by memory (two of the three passes read or write 57 values a cell).
// 48 x 40 x 36, us a step: in NEQ walls 147 (five passes over the
// ghost-extended grid) -> 78 (7.5 + 37 + 34), periodic 61.  Taking x
// neighbours by lane shifts drops 40 % of the loads but waits for those at the
// row ends in a branch: 5 and 14 us more.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "ctx.hpp"
#include "march.hpp"
#include "wave.hpp"

namespace dugks {

namespace {

using LA = D3Q19;
constexpr int AQ = 19;

// per axis: face arrays (values, acceleration), faces in all
struct A3Faces {
    double* v[3];
    double* g[3];
    unsigned nb[3];  // bytes of one value's faces
};

// Arrays are read through buffer descriptors: an element is the lane's 32-bit
// byte offset (the same for all velocities) plus a uniform one (the velocity's),
// so a load takes no address arithmetic of its own.  With 64-bit addresses the
// faces spilled 300 registers.
using Buf = __amdgpu_buffer_rsrc_t;
typedef unsigned a3_u2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ Buf a3_buf(const double* p)
{
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, -1, 0x00020000);
}
__device__ __forceinline__ double a3_ld(Buf b, unsigned off, unsigned base)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(b, (int)off, (int)base, 0));
}
__device__ __forceinline__ void a3_st(Buf b, unsigned off, unsigned base, double x)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(a3_u2, x), b, (int)off, (int)base, 0);
}

// moments and equilibrium factors at a point: fe_q = W_q (a + eu (B + C eu)),
// source (sG e.G - g) fe
struct A3Eq {
    double rho, a, g, u[3], G[3];
};

__device__ __forceinline__ double a3_dot(int q, const double (&u)[3]) { return e_dot<LA, double>(q, u); }

template <class P_>
__device__ __forceinline__ A3Eq a3_point(const P_& P, const double (&v)[AQ], const double (&G)[3], double hw)
{
    A3Eq E;
    double j[3] = {0, 0, 0}, uu = 0, gu = 0;
    E.rho = 0;
#pragma unroll
    for (int q = 0; q < AQ; ++q) {
        E.rho += v[q];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if (LA::e(q, d) > 0) j[d] += v[q];
            if (LA::e(q, d) < 0) j[d] -= v[q];
        }
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        E.G[d] = G[d];
        E.u[d] = P.crho * j[d] + hw * G[d];
        uu += E.u[d] * E.u[d];
        gu += E.u[d] * G[d];
    }
    E.a = E.rho - P.eqH * uu;
    E.g = gu * P.invRT;
    return E;
}
template <class P_>
__device__ __forceinline__ double a3_feq(const P_& P, const A3Eq& E, int q)
{
    const double eu = a3_dot(q, E.u);
    return LA::w(q) * (E.a + eu * (P.eqB + P.eqC * eu));
}

// reverse of v + b (feq - v) + c S: the sums over the velocities, and from
// them the adjoints
struct A3Sums {
    double rb, s0, p[3], s[3];
};
__device__ __forceinline__ void a3_sum(const Inst<double>& P, const A3Eq& E, int q, double h, double b, double c, A3Sums& S)
{
    const double eu = a3_dot(q, E.u), a = LA::w(q) * h;
    const double m = a * (b + c * (P.sG * a3_dot(q, E.G) - E.g));
    const double s = a * (E.a + eu * (P.eqB + P.eqC * eu)), d = m * (P.eqB + 2.0 * P.eqC * eu);
    S.rb += m;
    S.s0 += s;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        if (LA::e(q, i) > 0) { S.p[i] += d; S.s[i] += s; }
        if (LA::e(q, i) < 0) { S.p[i] -= d; S.s[i] -= s; }
    }
}
// adjoints of c / rho0 sums (j), of the density (rb) and of the acceleration (g)
struct A3Adj {
    double rb, j[3], g[3];
};
__device__ __forceinline__ A3Adj a3_adj(const Inst<double>& P, const A3Eq& E, const A3Sums& S, double c, double hw)
{
    A3Adj R;
    R.rb = S.rb;
    const double k = 2.0 * P.eqH * S.rb, ci = c * P.invRT * S.s0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const double u = S.p[i] - k * E.u[i] - ci * E.G[i];
        R.j[i] = P.crho * u;
        R.g[i] = c * P.sG * S.s[i] - ci * E.u[i] + hw * u;
    }
    return R;
}

// coefficients of the derivative at cell i of axis a, times h c, the ghost rule
// folded in
__device__ __forceinline__ void a3_coef(const Inst<double>& P, int a, int i, double& kp, double& km)
{
    const double hc = P.h * P.c;
    kp = hc * P.m[a].cp[i];
    km = hc * P.m[a].cm[i];
    if (!P.per[a]) {
        const double p0 = kp, m0 = km;
        if (i == 0) { kp += P.rlo[a] * m0; km = 0; }
        if (i == P.n[a] - 1) { km += P.rhi[a] * p0; kp = 0; }
    }
}
// a wall face as a face of the pair next to it: weight of the upper cell and
// h c times the difference's coefficient
__device__ __forceinline__ void a3_wall_coef(const Inst<double>& P, int a, int side, double& w, double& k)
{
    const int f = side ? P.n[a] : 0;
    const double r = side ? P.rhi[a] : P.rlo[a], wf = P.m[a].w[f];
    w = side ? 1.0 - wf * r : (1.0 - wf) * r;
    k = -P.h * P.c * P.m[a].gn[f] * r;
}

// group of a velocity in the cells' launch: the diagonals of the planes xy, xz
// and yz (four each), then the others
__host__ __device__ constexpr int a3_group(int q)
{
    const int x = LA::e(q, 0) != 0, y = LA::e(q, 1) != 0, z = LA::e(q, 2) != 0;
    return x + y + z != 2 ? 3 : (x && y ? 0 : (x && z ? 1 : 2));
}
__host__ __device__ constexpr int a3_place(int q)
{
    int s = 0;
    for (int r = 0; r < q; ++r)
        if (a3_group(r) == a3_group(q)) ++s;
    return s;
}
constexpr int A3_MAX = 7;  // velocities of the largest group

}  // namespace

// f-bar-plus of every cell; a wave per group of velocities, all of which read
// the cell's state
__global__ __launch_bounds__(256) void k_adj3_phi(const Inst<double>* __restrict__ Pp, const double* __restrict__ f,
                                                  const double* __restrict__ force, double gt, double* __restrict__ phi)
{
    const Inst<double>& P = *Pp;
    const int grp = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const long long c = (long long)blockIdx.x * 64 + (threadIdx.x & 63);
    if (c >= P.nc) return;
    const unsigned o = (unsigned)c * 8u, nb = (unsigned)P.nc * 8u;
    const Buf bf = a3_buf(f), bg = a3_buf(force), bp = a3_buf(phi);
    double v[AQ], G[3];
#pragma unroll
    for (int q = 0; q < AQ; ++q) v[q] = a3_ld(bf, o, q * nb);
#pragma unroll
    for (int d = 0; d < 3; ++d) G[d] = gt * (P.G0[d] + (force ? a3_ld(bg, o, d * nb) : 0.0));
    const A3Eq E = a3_point(P, v, G, P.h);
#pragma unroll
    for (int q = 0; q < AQ; ++q) {
        if (a3_group(q) != grp) continue;
        const double fe = a3_feq(P, E, q);
        a3_st(bp, o, q * nb, v[q] + P.B1 * (fe - v[q]) + P.C1 * (P.sG * a3_dot(q, G) - E.g) * fe);
    }
}

// velocities whose loads are in flight together (2 to 6 and 1 to 4 measured
// within 2 %)
constexpr int A3_STEP = 3, A3_PAIR = 2;

// the faces of the pair of cells (R - 1, R) along A, at coordinates x of its
// upper cell: the interface between them and, side >= 0, the face of the wall next
// to them
template <int A, bool WALL>
__device__ __forceinline__ void a3_faces(const Inst<double>& P, const int (&x)[3], int side, const double* phi,
                                         const double* force, const double* lam, double gth, const A3Faces& F)
{
    constexpr int T1 = A == 0 ? 1 : 0, T2 = A == 2 ? 1 : 2;
    const int st[3] = {1, P.n[0], P.n[0] * P.n[1]};
    const int cR = x[0] + x[1] * st[1] + x[2] * st[2];
    const int cL = cR + (x[A] > 0 ? -st[A] : (P.n[A] - 1) * st[A]);
    const unsigned oR = (unsigned)cR * 8u, oL = (unsigned)cL * 8u, nb = (unsigned)P.nc * 8u;
    const Buf bp = a3_buf(phi), bl = a3_buf(lam), bv = a3_buf(F.v[A]), bg = a3_buf(F.g[A]);
    // neighbours along the two tangents, as offsets from either cell
    unsigned up[2], dn[2];
    double kp[2], km[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int t = i ? T2 : T1, n = P.n[t];
        const bool per = P.per[t] != 0;
        const int u = x[t] < n - 1 ? 1 : (per ? 1 - n : 0), d = x[t] > 0 ? -1 : (per ? n - 1 : 0);
        up[i] = (unsigned)(u * st[t]) * 8u;
        dn[i] = (unsigned)(d * st[t]) * 8u;
        a3_coef(P, t, x[t], kp[i], km[i]);
    }
    double fL[3] = {0, 0, 0}, fR[3] = {0, 0, 0};
    if (force) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            fL[d] = a3_ld(a3_buf(force), oL, d * nb);
            fR[d] = a3_ld(a3_buf(force), oR, d * nb);
        }
    }
    const double hh = 0.5 * P.h;
    // values of the interface (v), and with a wall of the wall's face (v2), from
    // the same loads
    double w2 = 0, k2 = 0;
    if constexpr (WALL) a3_wall_coef(P, A, side, w2, k2);
    const double w = P.m[A].w[x[A]], k = P.h * P.c * P.m[A].gn[x[A]];
    double v[AQ], v2[AQ];
#pragma unroll
    for (int q = 0; q < AQ; ++q) {
        const unsigned qb = q * nb;
        const double hR = a3_ld(bp, oR, qb), hL = a3_ld(bp, oL, qb);
        double sR = hR, sL = hL;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int e = LA::e(q, i ? T2 : T1);
            if (e == 0) continue;
            const double dR = kp[i] * (a3_ld(bp, oR + up[i], qb) - hR) + km[i] * (a3_ld(bp, oR + dn[i], qb) - hR);
            const double dL = kp[i] * (a3_ld(bp, oL + up[i], qb) - hL) + km[i] * (a3_ld(bp, oL + dn[i], qb) - hL);
            sR = e > 0 ? sR - dR : sR + dR;
            sL = e > 0 ? sL - dL : sL + dL;
        }
        const double d = LA::e(q, A) > 0 ? hR - hL : (LA::e(q, A) < 0 ? hL - hR : 0.0);
        v[q] = sL + w * (sR - sL);
        if (LA::e(q, A) != 0) v[q] -= k * d;
        if constexpr (WALL) {
            v2[q] = sL + w2 * (sR - sL);
            if (LA::e(q, A) != 0) v2[q] -= k2 * d;
        }
        // values formed here, not where they are used: else all loads come
        // first and are held
        if (q % A3_STEP == A3_STEP - 1) {
#pragma unroll
            for (int r = q - A3_STEP + 1; r <= q; ++r) {
                if constexpr (WALL) asm volatile("" : "+v"(v[r]), "+v"(v2[r])::"memory");
                else asm volatile("" : "+v"(v[r])::"memory");
            }
        }
    }
    auto face_acc = [&](double w, double (&G)[3]) {
#pragma unroll
        for (int d = 0; d < 3; ++d) G[d] = gth * (P.G0[d] + (fL[d] + w * (fR[d] - fL[d])));
    };
    const int F0 = P.n[0] + (A == 0 ? 1 : 0), F1 = P.n[1] + (A == 1 ? 1 : 0);
    auto slot = [&](int c) -> unsigned {
        const int y[3] = {A == 0 ? c : x[0], A == 1 ? c : x[1], A == 2 ? c : x[2]};
        return (unsigned)((y[2] * F1 + y[1]) * F0 + y[0]) * 8u;
    };
    const unsigned nf = F.nb[A];
    const double sR = P.c * P.m[A].fdx[x[A]], sL = P.c * P.m[A].fdx[x[A] > 0 ? x[A] - 1 : P.n[A] - 1];
    auto lam_at = [&](int q, unsigned o) { return a3_ld(bl, o, q * nb); };

    double G[3];
    face_acc(w, G);
    const A3Eq E = a3_point(P, v, G, hh);
    A3Sums S{};
    double h[AQ];
    auto inner_h = [&](int q) {  // adjoint of the flux of the interface
        const double l = sR * lam_at(q, oR) - sL * lam_at(q, oL);
        return LA::e(q, A) > 0 ? l : -l;
    };
#pragma unroll
    for (int q = 0; q < AQ; ++q) {
        h[q] = LA::e(q, A) != 0 ? inner_h(q) : 0.0;
        if (LA::e(q, A) != 0) a3_sum(P, E, q, h[q], P.B7, P.C7, S);
    }
    A3Adj R = a3_adj(P, E, S, P.C7, hh);
    // adjoint of value q from the sums (and its own)
    auto value = [&](const A3Adj& X, int q) { return X.rb + a3_dot(q, X.j); };
    double ne[AQ], rep[AQ];  // of the velocities across the face
    if constexpr (WALL) {
        const bool neq = P.bc[2 * A + side] != BC_BOUNCE_BACK;
#pragma unroll
        for (int q = 0; q < AQ; ++q)
            if (LA::e(q, A) != 0) ne[q] = neq ? v[q] - a3_feq(P, E, q) : 0.0;
    }
    const unsigned os = slot(x[A]);
    if constexpr (!WALL) {
#pragma unroll
        for (int q = 0; q < AQ; ++q) a3_st(bv, os, q * nf, value(R, q) + (1.0 - P.B7) * h[q]);
#pragma unroll
        for (int d = 0; d < 3; ++d) a3_st(bg, os, d * nf, R.g[d]);
    } else {
        const int s = 2 * A + side, kind = P.bc[s];
        const bool pos = side == 0;  // the entering velocities have component +1
        face_acc(w2, G);
        // the rule (Eqs. BB, NEQ)
        const bool vel = kind == BC_NEQ_VELOCITY;
        A3Eq B;
        {
            double uu = 0;
            B.rho = vel ? E.rho : wall_density(P, s, gth);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const double wu = P.uw[s][d];
                B.u[d] = vel ? wu : E.u[d];
                uu += B.u[d] * B.u[d];
                B.G[d] = 0;
            }
            B.a = B.rho - P.eqH * uu;
            B.g = 0;
        }
        const double uw[3] = {P.uw[s][0], P.uw[s][1], P.uw[s][2]};
        // (pairs of opposites: one enters)
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            if (LA::e(q, A) <= 0) continue;
            const int p = LA::opp(q);
            const double vq = v2[q], vp = v2[p];
            const double bbq = vp + 2.0 * P.eqB * LA::w(q) * a3_dot(q, uw), bbp = vq - 2.0 * P.eqB * LA::w(q) * a3_dot(q, uw);
            const bool bb = kind == BC_BOUNCE_BACK;
            const double nq = bb ? bbq : a3_feq(P, B, q) + ne[q], np = bb ? bbp : a3_feq(P, B, p) + ne[p];
            v2[q] = pos ? nq : vq;
            v2[p] = pos ? vp : np;
        }
        const A3Eq E2 = a3_point(P, v2, G, hh);
        A3Sums S2{};
        const double sc = pos ? sL : -sR;
        const unsigned ol = pos ? oL : oR;
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const int e = LA::e(q, A);
            h[q] = 0;
            if (e == 0) continue;
            const double l = sc * lam_at(q, ol);
            h[q] = e > 0 ? l : -l;
            a3_sum(P, E2, q, h[q], P.B7, P.C7, S2);
        }
        const A3Adj R2 = a3_adj(P, E2, S2, P.C7, hh);
        const unsigned ow = slot(pos ? 0 : P.n[A]);
        // the adjoints of the replaced values leave the face: to the opposite
        // velocity, or to the opposite interface
        const bool bb = kind == BC_BOUNCE_BACK;
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const int e = LA::e(q, A);
            if (e == 0) {
                a3_st(bv, ow, q * nf, value(R2, q));
                continue;
            }
            if (e < 0) continue;
            const int p = LA::opp(q);
            const double bq = value(R2, q) + (1.0 - P.B7) * h[q], bp = value(R2, p) + (1.0 - P.B7) * h[p];
            const double in = pos ? bq : bp;
            rep[q] = pos ? bq : 0.0;
            rep[p] = pos ? 0.0 : bp;
            const double out = (pos ? bp : bq) + (bb ? in : 0.0);
            a3_st(bv, ow, q * nf, pos ? 0.0 : out);
            a3_st(bv, ow, p * nf, pos ? out : 0.0);
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) a3_st(bg, ow, d * nf, R2.g[d]);
        if (!bb) {
            // replaced value = feq(r_a, u_a) + v - feq(rho, u) of the opposite
            // interface; velocity wall: r_a = rho, so rho drops out; pressure
            // wall: u_a = u, so u drops out
            double p[3] = {0, 0, 0}, rb = 0;
#pragma unroll
            for (int q = 0; q < AQ; ++q) {
                if (LA::e(q, A) == 0) continue;
                const double a = LA::w(q) * rep[q], d = a * (P.eqB + 2.0 * P.eqC * a3_dot(q, E.u));
                rb -= a;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    if (LA::e(q, i) > 0) p[i] -= d;
                    if (LA::e(q, i) < 0) p[i] += d;
                }
            }
            R.rb += vel ? 0.0 : rb;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const double u = vel ? p[i] - 2.0 * P.eqH * rb * E.u[i] : 0.0;
                R.j[i] += P.crho * u;
                R.g[i] += hh * u;
            }
        }
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            double b = value(R, q);
            if (LA::e(q, A) != 0) b += (1.0 - P.B7) * inner_h(q) + (bb ? 0.0 : rep[q]);
            a3_st(bv, os, q * nf, b);
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) a3_st(bg, os, d * nf, R.g[d]);
    }
}

// where the blocks of an axis' walls begin and all end (walls first: they take
// longer), and from `inner` on, a multiple of the XCDs, those of the interfaces
// between cells
struct A3Blocks {
    int wall[4], inner;
};
// wall lines of a block: along x no two lanes share a cache line, and eight
// of them a wave, on eight times the waves, take a quarter of the time
__host__ __device__ constexpr int a3_wall_lanes(int a) { return a == 0 ? 8 : 64; }

template <int A>
__device__ __forceinline__ void a3_face_thread(const Inst<double>& P, bool wall, int i, const double* phi,
                                               const double* force, const double* lam, double gth, const A3Faces& F)
{
    int x[3];
    if (wall) {
        constexpr int B = A == 0 ? 1 : 0, C = A == 2 ? 1 : 2;
        const int lines = P.n[B] * P.n[C];
        if (i >= 2 * lines) return;
        const int side = i >= lines ? 1 : 0, l = i - side * lines;
        x[A] = side ? P.n[A] - 1 : 1;
        x[B] = l % P.n[B];
        x[C] = l / P.n[B];
        a3_faces<A, true>(P, x, side, phi, force, lam, gth, F);
        return;
    }
    if (i >= (int)P.nc) return;
    x[0] = i % P.n[0];
    const int r = i / P.n[0];
    x[1] = r % P.n[1];
    x[2] = r / P.n[1];
    // (next to a wall: with the wall's face)
    if (!P.per[A] && (x[A] <= 1 || x[A] == P.n[A] - 1)) return;
    a3_faces<A, false>(P, x, 0, phi, force, lam, gth, F);
}

// (three waves per SIMD: with four the wall path spills 270 registers, 78 -> 87 us)
__global__ __attribute__((amdgpu_flat_work_group_size(1, 256), amdgpu_waves_per_eu(3))) void k_adj3_faces(
    const Inst<double>* __restrict__ Pp, const double* __restrict__ phi, const double* __restrict__ force,
    const double* __restrict__ lam, double gth, A3Blocks nb, A3Faces F)
{
    const Inst<double>& P = *Pp;
    const int b = (int)blockIdx.x, tid = (int)threadIdx.x;
    const bool wall = b < nb.inner;
    int a, i;
    if (wall) {
        if (b >= nb.wall[3]) return;
        a = b < nb.wall[1] ? 0 : (b < nb.wall[2] ? 1 : 2);
        const int first = a == 0 ? 0 : (a == 1 ? nb.wall[1] : nb.wall[2]), lanes = a3_wall_lanes(a);
        if ((tid & 63) >= lanes) return;
        i = ((b - first) * 4 + (tid >> 6)) * lanes + (tid & 63);
    } else {
        // in XCD order, the three axes of 256 cells one after the other: they
        // read the same cells through one L2
        const int j = xcd_order(b - nb.inner, (int)gridDim.x - nb.inner);
        a = j % 3;
        i = j / 3 * 256 + tid;
    }
    if (a == 0) a3_face_thread<0>(P, wall, i, phi, force, lam, gth, F);
    else if (a == 1) a3_face_thread<1>(P, wall, i, phi, force, lam, gth, F);
    else a3_face_thread<2>(P, wall, i, phi, force, lam, gth, F);
}

namespace {

// how a cell takes from the faces of one axis: its lower and upper one with
// weights (psi) and difference coefficients (phi), and next to the wall cell
// (more) the wall face again; and the derivative along the axis: the cell's own
// coefficients and those of the neighbours that read the cell.  One wave of a
// workgroup forms those of an axis, all read them from LDS.
enum { C_WL, C_WU, C_WE, C_KL, C_KU, C_KE, C_OWN, C_DN, C_UP, C_COUNT };

__device__ __forceinline__ void a3_weights(const Inst<double>& P, int a, int c, double (*cf)[64], int lane)
{
    const int n = P.n[a];
    const bool per = P.per[a] != 0;
    const double hc = P.h * P.c;
    double wl = P.m[a].w[c], kl = -hc * P.m[a].gn[c];
    double wu = 1.0 - P.m[a].w[c + 1], ku = hc * P.m[a].gn[c + 1], we = 0, ke = 0;
    if (!per) {
        double w0, k0, w1, k1;
        a3_wall_coef(P, a, 0, w0, k0);
        a3_wall_coef(P, a, 1, w1, k1);
        if (c == 0) { wl = 1.0 - w0; kl = k0; }
        if (c == 1) { we = w0; ke = -k0; }
        if (c == n - 1) { wu = w1; ku = -k1; }
        if (c == n - 2) { we = 1.0 - w1; ke = k1; }
    }
    double p, m, p2, m2, un;
    a3_coef(P, a, c, p, m);
    a3_coef(P, a, c > 0 ? c - 1 : (per ? n - 1 : 0), p2, un);
    a3_coef(P, a, c < n - 1 ? c + 1 : (per ? 0 : n - 1), un, m2);
    cf[C_WL][lane] = wl;
    cf[C_WU][lane] = wu;
    cf[C_WE][lane] = we;
    cf[C_KL][lane] = kl;
    cf[C_KU][lane] = ku;
    cf[C_KE][lane] = ke;
    cf[C_OWN][lane] = p + m;
    cf[C_DN][lane] = (per || c > 0) ? p2 : 0.0;
    cf[C_UP][lane] = (per || c < n - 1) ? m2 : 0.0;
}

struct A3Axis {
    unsigned lo, up, ex;
    double wl, wu, we;
    bool more;
};

// psi-hat of an axis for one velocity at the cell shifted by `d` bytes
__device__ __forceinline__ double a3_psi(const A3Axis& r, Buf v, unsigned base, unsigned d)
{
    double s = r.wl * a3_ld(v, r.lo + d, base) + r.wu * a3_ld(v, r.up + d, base);
    if (r.more) s += r.we * a3_ld(v, r.ex + d, base);
    return s;
}

}  // namespace

// what the cell takes from the faces of axis A, for the velocities of a group
// (ph) and one component of the force (g); one axis after the other, so that
// only one's offsets and weights are held
template <int A, int GRP>
__device__ __forceinline__ void a3_gather(const Inst<double>& P, const A3Faces& F, const int (&x)[3],
                                          const double (*cf)[C_COUNT][64], int lane, double (&ph)[A3_MAX], double gth,
                                          double& g)
{
    const Buf v = a3_buf(F.v[A]);
    const int F0 = P.n[0] + (A == 0 ? 1 : 0), F1 = P.n[1] + (A == 1 ? 1 : 0);
    const int sa = A == 0 ? 1 : (A == 1 ? F0 : F0 * F1), i = (x[2] * F1 + x[1]) * F0 + x[0];
    const bool pa = P.per[A] != 0;
    A3Axis ax;
    ax.lo = (unsigned)i * 8u;
    ax.up = (unsigned)(i + (pa && x[A] == P.n[A] - 1 ? -x[A] * sa : sa)) * 8u;
    ax.ex = (unsigned)(i + (x[A] == 1 ? -sa : 2 * sa)) * 8u;
    ax.more = !pa && (x[A] == 1 || x[A] == P.n[A] - 2);
    ax.wl = cf[A][C_WL][lane];
    ax.wu = cf[A][C_WU][lane];
    ax.we = cf[A][C_WE][lane];
    const double kl = cf[A][C_KL][lane], kup = cf[A][C_KU][lane], ke = cf[A][C_KE][lane];
    unsigned sp[3], sm[3];  // the neighbours' slots along a tangent
    double k0[3], kd[3], ku[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        if (t == A || (GRP < 3 && t == 2 - GRP)) continue;  // the group has no velocity along the latter
        const int n = P.n[t], st = t == 0 ? 1 : (t == 1 ? F0 : F0 * F1);
        const bool per = P.per[t] != 0;
        sm[t] = (unsigned)((x[t] > 0 ? -1 : (per ? n - 1 : 0)) * st) * 8u;
        sp[t] = (unsigned)((x[t] < n - 1 ? 1 : (per ? 1 - n : 0)) * st) * 8u;
        k0[t] = cf[t][C_OWN][lane];
        kd[t] = cf[t][C_DN][lane];
        ku[t] = cf[t][C_UP][lane];
    }
#pragma unroll
    for (int q = 0; q < AQ; ++q) {
        if (a3_group(q) != GRP) continue;
        const unsigned qb = q * F.nb[A];
        const double l = a3_ld(v, ax.lo, qb), u = a3_ld(v, ax.up, qb);
        double psi = ax.wl * l + ax.wu * u, k = kl * l + kup * u;
        if (ax.more) {
            const double e = a3_ld(v, ax.ex, qb);
            psi += ax.we * e;
            k += ke * e;
        }
        double r = psi;
        if (LA::e(q, A) > 0) r += k;
        if (LA::e(q, A) < 0) r -= k;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            if (t == A || LA::e(q, t) == 0) continue;
            const double s = k0[t] * psi - kd[t] * a3_psi(ax, v, qb, sm[t]) - ku[t] * a3_psi(ax, v, qb, sp[t]);
            r += LA::e(q, t) > 0 ? s : -s;
        }
        ph[a3_place(q)] += r;
        // formed here: else all loads come first and are held
        if (a3_place(q) % A3_PAIR == A3_PAIR - 1) {
#pragma unroll
            for (int i = a3_place(q) - A3_PAIR + 1; i <= a3_place(q); ++i) asm volatile("" : "+v"(ph[i])::"memory");
        }
    }
    if constexpr (GRP < 3) g += gth * a3_psi(ax, a3_buf(F.g[A]), GRP * F.nb[A], 0u);
    asm volatile("" ::: "memory");
}

template <int GRP>
__device__ __forceinline__ void a3_cell(const Inst<double>& P, const A3Faces& F, const int (&x)[3],
                                        const double (*cf)[C_COUNT][64], int lane, const double* f,
                                        const double* force, const double* lam, double gt, double gth, unsigned o,
                                        A3Eq& E, double (&ph)[A3_MAX], double& g, A3Sums& S)
{
    const unsigned nb = (unsigned)P.nc * 8u;
    const Buf bf = a3_buf(f), bg = a3_buf(force), bl = a3_buf(lam);
#pragma unroll
    for (int q = 0; q < AQ; ++q)
        if (a3_group(q) == GRP) ph[a3_place(q)] = (4.0 / 3.0) * a3_ld(bl, o, q * nb);
    a3_gather<0, GRP>(P, F, x, cf, lane, ph, gth, g);
    a3_gather<1, GRP>(P, F, x, cf, lane, ph, gth, g);
    a3_gather<2, GRP>(P, F, x, cf, lane, ph, gth, g);
    double v[AQ], G[3];
#pragma unroll
    for (int q = 0; q < AQ; ++q) v[q] = a3_ld(bf, o, q * nb);
#pragma unroll
    for (int d = 0; d < 3; ++d) G[d] = gt * (P.G0[d] + (force ? a3_ld(bg, o, d * nb) : 0.0));
    E = a3_point(P, v, G, P.h);
#pragma unroll
    for (int q = 0; q < AQ; ++q)
        if (a3_group(q) == GRP) a3_sum(P, E, q, ph[a3_place(q)], P.B1, P.C1, S);
}

template <int GRP>
__device__ __forceinline__ void a3_store(const Inst<double>& P, const A3Adj& R, const double (&ph)[A3_MAX],
                                         const double* lam, double* lam_out, unsigned o)
{
    const unsigned nb = (unsigned)P.nc * 8u;
#pragma unroll
    for (int q = 0; q < AQ; ++q) {
        if (a3_group(q) != GRP) continue;
        const int pl = a3_place(q);
        a3_st(a3_buf(lam_out), o, q * nb,
              (1.0 - P.B1) * ph[pl] + R.rb + a3_dot(q, R.j) - (1.0 / 3.0) * a3_ld(a3_buf(lam), o, q * nb));
    }
}

// (five waves per SIMD, three registers spilled: four, at 102 registers, take 92
// us a step in walls and 74 periodic at 48 x 40 x 36, whose 4320 waves then need a
// second round, and 5 % more at 96 x 80 x 64)
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(5))) void k_adj3_cells(
    const Inst<double>* __restrict__ Pp, const double* __restrict__ f, const double* __restrict__ force,
    const double* __restrict__ lam, double gt, double gth, A3Faces F, double* __restrict__ lam_out,
    double* __restrict__ grad)
{
    __shared__ double part[4][8][64];
    __shared__ double cf[3][C_COUNT][64];
    const Inst<double>& P = *Pp;
    const int grp = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    const int b = xcd_order((int)blockIdx.x, (int)gridDim.x);
    const long long cell = (long long)b * 64 + lane;
    const bool own = cell < P.nc;
    const int c = (int)(own ? cell : P.nc - 1);
    int x[3];
    x[0] = c % P.n[0];
    const int yz = c / P.n[0];
    x[1] = yz % P.n[1];
    x[2] = yz / P.n[1];
    const unsigned o = (unsigned)c * 8u;
    if (grp < 3) a3_weights(P, grp, grp == 0 ? x[0] : (grp == 1 ? x[1] : x[2]), cf[grp], lane);
    __syncthreads();
    A3Eq E;
    double ph[A3_MAX], g = 0;
    A3Sums S{};
    if (grp == 0) a3_cell<0>(P, F, x, cf, lane, f, force, lam, gt, gth, o, E, ph, g, S);
    else if (grp == 1) a3_cell<1>(P, F, x, cf, lane, f, force, lam, gt, gth, o, E, ph, g, S);
    else if (grp == 2) a3_cell<2>(P, F, x, cf, lane, f, force, lam, gt, gth, o, E, ph, g, S);
    else a3_cell<3>(P, F, x, cf, lane, f, force, lam, gt, gth, o, E, ph, g, S);
    part[grp][0][lane] = S.rb;
    part[grp][1][lane] = S.s0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        part[grp][2 + d][lane] = S.p[d];
        part[grp][5 + d][lane] = S.s[d];
    }
    __syncthreads();
    auto total = [&](int i) { return (part[0][i][lane] + part[1][i][lane]) + (part[2][i][lane] + part[3][i][lane]); };
    S.rb = total(0);
    S.s0 = total(1);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        S.p[d] = total(2 + d);
        S.s[d] = total(5 + d);
    }
    if (!own) return;
    const A3Adj R = a3_adj(P, E, S, P.C1, P.h);
    if (grp == 0) a3_store<0>(P, R, ph, lam, lam_out, o);
    else if (grp == 1) a3_store<1>(P, R, ph, lam, lam_out, o);
    else if (grp == 2) a3_store<2>(P, R, ph, lam, lam_out, o);
    else a3_store<3>(P, R, ph, lam, lam_out, o);
    if (grad && grp < 3) {
        // component grp of the force gradient
        const double gc = grp == 0 ? R.g[0] : (grp == 1 ? R.g[1] : R.g[2]);
        grad[grp * P.nc + c] += gt * gc + g;
    }
}

static long long a3_slots(const Inst<double>& P, int a)
{
    long long n = 1;
    for (int b = 0; b < 3; ++b) n *= (long long)P.n[b] + (b == a ? 1 : 0);
    return n;
}

// wall axes of four cells or more (no cell next to both walls' faces but its
// own), offsets within 32 bits
bool adjoint_cells_fit(const Inst<double>& P)
{
    for (int a = 0; a < 3; ++a) {
        if (!P.per[a] && P.n[a] < 4) return false;
        if (a3_slots(P, a) * AQ * (long long)sizeof(double) > 0xffffffffLL) return false;
    }
    return true;
}

size_t adjoint_cells_bytes(const Inst<double>& P)
{
    size_t n = (size_t)AQ * P.nc;
    for (int a = 0; a < 3; ++a) n += (size_t)(AQ + 3) * a3_slots(P, a);
    return n * sizeof(double);
}

void adjoint_cells_launch(const Inst<double>* Pd, const Inst<double>& P, void* work, const void* f_, const void* force_,
                          double gt, double gth, const void* lam_, void* lam_out, void* grad, hipStream_t st)
{
    const double *f = (const double*)f_, *force = (const double*)force_, *lam = (const double*)lam_;
    double* phi = (double*)work;
    double* p = phi + (size_t)AQ * P.nc;
    A3Faces F;
    A3Blocks nb;
    nb.wall[0] = 0;
    for (int a = 0; a < 3; ++a) {
        const size_t slots = (size_t)a3_slots(P, a);
        F.nb[a] = (unsigned)(slots * sizeof(double));
        F.v[a] = p;
        p += AQ * slots;
        F.g[a] = p;
        p += 3 * slots;
        const int lines = 4 * a3_wall_lanes(a);
        nb.wall[a + 1] = nb.wall[a] + (P.per[a] ? 0 : (int)((2 * (P.nc / P.n[a]) + lines - 1) / lines));
    }
    nb.inner = (nb.wall[3] + 7) / 8 * 8;
    const unsigned inner = 3 * (unsigned)((P.nc + 255) / 256);
    const unsigned n64 = (unsigned)((P.nc + 63) / 64);
    hipLaunchKernelGGL(k_adj3_phi, dim3(n64), dim3(256), 0, st, Pd, f, force, gt, phi);
    hipLaunchKernelGGL(k_adj3_faces, dim3((unsigned)nb.inner + inner), dim3(256), 0, st, Pd, (const double*)phi, force, lam,
                       gth, nb, F);
    hipLaunchKernelGGL(k_adj3_cells, dim3(n64), dim3(256), 0, st, Pd, f, force, lam, gt, gth, F, (double*)lam_out,
                       (double*)grad);
}

}  // namespace dugks
