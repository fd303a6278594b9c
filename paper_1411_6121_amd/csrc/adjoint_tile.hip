// adjoint_tile.hip -- reverse mode of one D2Q9 step in FP64, any boundary
// set, in one launch: one lane per cell on tiles with a two-cell halo, nothing
// but f_n, lam_{n+1} and the force read and lam_n and the force gradient
// written.
//
// The ghost rule is linear, so it is folded into coefficients of the two
// cells next to a wall: a tangential derivative at a wall cell takes
// cp' = cp + r cm and cm' = 0 (low side), and a wall face is a face of the
// pair of cells next to it with its own weight and difference,
//   low:  w' = (1 - w) r,  g' = -g r;   high: w' = 1 - w r,  g' = -g r,
// r the extrapolation ratio.  The opposite interface of the NEQ rule lies
// between the same two cells.  So every lane reverses the faces of one pair
// (its cell and the one below along the axis): the interface between them
// and, next to a wall, the wall face, whose share in the opposite interface
// stays in the lane.  What a pair gives to its lower cell is handed over by a
// lane shift (x) or through LDS (y).
//
// With fbar(b) = (1-w) psi_L + w psi_R - e k (phi_R - phi_L) and psi = phi -
// e_t d, d = kp (phi_+ - phi) + km (phi_- - phi), the reverse of a step is
//   lam_{n+1} -> fluxes -> Eq. (original_f), moments -> wall rule -> psi, phi
//   of the pair -> transposed derivative -> phi -> Eq. (f_bar_+) -> lam_n.
//
// Bound by FP64 issue and latency, not by memory (33 values a cell, all in
// the cache): about 1500 instructions a lane.  Two waves per SIMD have the 256
// registers that a pair of cells takes without spills: one workgroup of 32 x 16
// lanes (28 x 12 cells) per CU, or two of 32 x 8 (28 x 4 cells), which waste
// more lanes on the halo but spread a small mesh over more CUs.  256^2 periodic:
// 21.0 us (two launches: faces, then cells) -> 11.0; 200 x 150 in a box of NEQ
// walls, stretched: 39 us (five launches) -> 13.2.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ctx.hpp"
#include "march.hpp"
#include "wave.hpp"

namespace dugks {

namespace {

constexpr int A2_X = 32, A2_HALO = 2, A2_OX = A2_X - 2 * A2_HALO;
// tile rows: on many cells, and on few (see adjoint_rows)
constexpr int A2_ROWS = 16, A2_FEW = 8;

// LDS planes of one value per lane: phi (e_y != 0, and the rest velocity), lam
// (e_y != 0) and the force, the first eleven of them overwritten by the
// adjoints of the y faces (values, acceleration); psi across y (e_x != 0);
// psi-hat of x faces (e_y != 0).
constexpr int A2_PHI = 0, A2_LAM = 7, A2_FRC = 13, A2_PSI = 15, A2_DH = 21, A2_SLOTS = 27;

__host__ __device__ constexpr int a2_e(int A, int q) { return A == 0 ? D2Q9::ex(q) : D2Q9::ey(q); }
// index among the six velocities with a component along axis A
__host__ __device__ constexpr int a2_six(int A, int q)
{
    int s = 0;
    for (int r = 0; r < q; ++r)
        if (a2_e(A, r) != 0) ++s;
    return s;
}
// reverse of v + b (feq - v) + c S at a point with moments (E; G the plain
// acceleration, weight hw in the velocity): from the adjoints h of the
// velocities with a component along axis A (A < 0: of all) to those of all v
// and of G
template <typename T, int A>
__device__ __forceinline__ void a2_relax(const Inst<T>& P, const EqD2<T>& E, T Gx, T Gy, T hw, T b, T c,
                                         const T (&h)[9], T (&v)[9], T& gx, T& gy)
{
    T rb = T(0), px = T(0), py = T(0), s0 = T(0), s1 = T(0), s2 = T(0);
    const T C2 = E.C + E.C;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        if (A >= 0 && a2_e(A, q) == 0) continue;
        const int ex = D2Q9::ex(q), ey = D2Q9::ey(q);
        T eu = T(0), eG = T(0);
        if (ex > 0) { eu += E.ux; eG += E.Gx; }
        if (ex < 0) { eu -= E.ux; eG -= E.Gx; }
        if (ey > 0) { eu += E.uy; eG += E.Gy; }
        if (ey < 0) { eu -= E.uy; eG -= E.Gy; }
        const T a = d2_w<T>(q) * h[q];
        const T m = a * (b + c * (eG - E.g));
        const T s = a * (E.a + eu * (E.B + E.C * eu));
        const T d = m * (E.B + C2 * eu);
        rb += m;
        s0 += s;
        if (ex > 0) { px += d; s1 += s; }
        if (ex < 0) { px -= d; s1 -= s; }
        if (ey > 0) { py += d; s2 += s; }
        if (ey < 0) { py -= d; s2 -= s; }
    }
    const T k = T(2) * P.eqH * rb, ci = c * P.invRT * s0;
    const T ux = px - k * E.ux - ci * Gx, uy = py - k * E.uy - ci * Gy;
    gx = c * P.sG * s1 - ci * E.ux + hw * ux;
    gy = c * P.sG * s2 - ci * E.uy + hw * uy;
    const T jx = P.crho * ux, jy = P.crho * uy;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const int ex = D2Q9::ex(q), ey = D2Q9::ey(q);
        T r = rb;
        if (A < 0 || a2_e(A, q) != 0) r += (T(1) - b) * h[q];
        if (ex > 0) r += jx;
        if (ex < 0) r -= jx;
        if (ey > 0) r += jy;
        if (ey < 0) r -= jy;
        v[q] = r;
    }
}

// the two cells of a pair along one axis: psi, phi and lam of the lower (L)
// and upper (R) one (phi only where e != 0 or e_t = 0, lam where e != 0) and
// their force field
template <typename T>
struct A2Pair {
    T psL[9], psR[9], phL[9], phR[9], lamL[9], lamR[9], fL[2], fR[2];
};

// values of a face of the pair and its acceleration
template <typename T, int A>
__device__ __forceinline__ void a2_recon(const Inst<T>& P, const A2Pair<T>& p, T w, T k, T gth, T (&v)[9], T& Gx,
                                         T& Gy)
{
#pragma unroll
    for (int q = 0; q < 9; ++q) v[q] = d2_recon<T, false>(a2_e(A, q), w, k, p.psL[q], p.psR[q], p.phL[q], p.phR[q]);
    Gx = gth * (P.G0[0] + (p.fL[0] + w * (p.fR[0] - p.fL[0])));
    Gy = gth * (P.G0[1] + (p.fL[1] + w * (p.fR[1] - p.fL[1])));
}

// the interface between the cells of a pair reversed (sL, sR: flux scales of
// the cells, zero where the pair does not exist): adjoints of its values and
// of its acceleration
template <typename T, int A>
__device__ __forceinline__ void a2_face(const Inst<T>& P, const A2Pair<T>& p, T w, T k, T sL, T sR, T gth, T (&b)[9],
                                        T& gx, T& gy)
{
    T v[9], h[9], rho, Gx, Gy;
    a2_recon<T, A>(P, p, w, k, gth, v, Gx, Gy);
    const EqD2<T> E = d2_point<T, false, true>(P, v, Gx, Gy, T(0.5) * P.h, rho);
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const int e = a2_e(A, q);
        if (e > 0) h[q] = sR * p.lamR[q] - sL * p.lamL[q];
        else if (e < 0) h[q] = sL * p.lamL[q] - sR * p.lamR[q];
        else h[q] = T(0);
    }
    a2_relax<T, A>(P, E, Gx, Gy, T(0.5) * P.h, P.B7, P.C7, h, b, gx, gy);
}

// what face adjoints b give to one cell of the face's pair (up: the upper
// one): to phi, psi included, to psi of the velocities with e_t != 0, and to
// the force
template <typename T, int A>
__device__ __forceinline__ void a2_take(bool up, T w, T k, const T (&b)[9], T gx, T gy, T (&phat)[9], T (&psi)[9],
                                        T& g0, T& g1)
{
    const T c = up ? w : T(1) - w, kk = up ? -k : k;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const int e = a2_e(A, q);
        const T s = c * b[q];
        phat[q] += e == 0 ? s : (e > 0 ? s + kk * b[q] : s - kk * b[q]);
        if (a2_e(1 - A, q) != 0) psi[q] += s;
    }
    g0 += c * gx;
    g1 += c * gy;
}

// the face of a wall (side of axis A) reversed, for one cell (up: the upper
// one) of the pair next to it; w, k: of the interface inside the pair, the
// opposite one of the NEQ rule.  Both cells' lanes evaluate it, so nothing
// has to be handed over.
template <typename T, int A>
__device__ __forceinline__ void a2_wall(const Inst<T>& P, int side, bool up, const A2Pair<T>& p, T w, T k, T gth,
                                        T (&phat)[9], T (&psi)[9], T& g0, T& g1)
{
    const T hh = T(0.5) * P.h;
    const int s = 2 * A + side, fc = side ? P.n[A] : 0;
    const bool pos = side == 0;  // the entering velocities have component +1
    const int kind = P.bc[s];
    EqD2<T> E;
    NeqD2<T> I;
    {
        T v[9], rho, Gx, Gy;
        a2_recon<T, A>(P, p, w, k, gth, v, Gx, Gy);
        E = d2_point<T, false, true>(P, v, Gx, Gy, hh, rho);
        d2_capture<T, A>(E, rho, v, pos ? 1 : -1, I);
    }
    const T r = side ? P.rhi[A] : P.rlo[A], wf = P.m[A].w[fc];
    const T w2 = side ? T(1) - wf * r : (T(1) - wf) * r, k2 = -P.h * P.c * P.m[A].gn[fc] * r;
    T b[9], hx, hy;
    {
        T v[9], h[9], rho, Gx, Gy;
        a2_recon<T, A>(P, p, w2, k2, gth, v, Gx, Gy);
        d2_wall<T, A, false>(P, s, pos ? 1 : -1, v, I, gth);
        const EqD2<T> E2 = d2_point<T, false, true>(P, v, Gx, Gy, hh, rho);
        const T sc = P.c * (side ? -P.m[A].fdx[P.n[A] - 1] : P.m[A].fdx[0]);  // into the one cell next to it
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            const int e = a2_e(A, q);
            const T ll = p.lamL[q], lr = p.lamR[q], l = e == 0 ? T(0) : sc * (side ? lr : ll);
            h[q] = e == 0 ? T(0) : (e > 0 ? l : -l);
        }
        a2_relax<T, A>(P, E2, Gx, Gy, hh, P.B7, P.C7, h, b, hx, hy);
    }
    // the rule: the adjoints of the replaced values leave the face
    T rep[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const T in = b[d2_q(A, 1, i)], out = b[d2_q(A, -1, i)];
        rep[i] = pos ? in : out;
        b[d2_q(A, 1, i)] = pos ? T(0) : in;
        b[d2_q(A, -1, i)] = pos ? out : T(0);
    }
    if (kind == BC_BOUNCE_BACK) {
        // the opposite of (e, i) is (-e, 2 - i)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            b[d2_q(A, -1, 2 - i)] += pos ? rep[i] : T(0);
            b[d2_q(A, 1, 2 - i)] += pos ? T(0) : rep[i];
        }
    } else {
        // replaced value = feq(r_a, u_a) + v - feq(rho, u) of the opposite
        // interface; velocity wall: r_a = rho, so rho drops out; pressure
        // wall: u_a = u, so u drops out
        T rb = T(0), qx = T(0), qy = T(0), x[9];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const T t = T(i - 1), n = pos ? T(1) : T(-1);
            const T eu = A == 0 ? n * E.ux + t * E.uy : t * E.ux + n * E.uy;
            const T a = d2_w<T>(i == 1 ? 1 : 0) * rep[i], d = a * (E.B + T(2) * E.C * eu);
            rb -= a;
            qx -= (A == 0 ? n : t) * d;
            qy -= (A == 0 ? t : n) * d;
        }
        const bool vel = kind == BC_NEQ_VELOCITY;
        const T ux = vel ? qx - T(2) * P.eqH * rb * E.ux : T(0), uy = vel ? qy - T(2) * P.eqH * rb * E.uy : T(0);
        const T rr = vel ? T(0) : rb, jx = P.crho * ux, jy = P.crho * uy;
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            const int ex = D2Q9::ex(q), ey = D2Q9::ey(q), e = a2_e(A, q), i = (A == 0 ? ey : ex) + 1;
            x[q] = rr;
            if (ex > 0) x[q] += jx;
            if (ex < 0) x[q] -= jx;
            if (ey > 0) x[q] += jy;
            if (ey < 0) x[q] -= jy;
            if (e > 0) x[q] += pos ? rep[i] : T(0);
            if (e < 0) x[q] += pos ? T(0) : rep[i];
        }
        a2_take<T, A>(up, w, k, x, hh * ux, hh * uy, phat, psi, g0, g1);
    }
    a2_take<T, A>(up, w2, k2, b, hx, hy, phat, psi, g0, g1);
}

// coefficients of the tangential derivative at cell i of axis a, times h c,
// with the ghost rule folded in
template <typename T>
__device__ __forceinline__ void a2_coef(const Inst<T>& P, int a, int i, T& kp, T& km)
{
    const T hc = P.h * P.c;
    kp = hc * P.m[a].cp[i];
    km = hc * P.m[a].cm[i];
    if (!P.per[a]) {
        const T p0 = kp, m0 = km;
        if (i == 0) { kp += P.rlo[a] * m0; km = T(0); }
        if (i == P.n[a] - 1) { km += P.rhi[a] * p0; kp = T(0); }
    }
}

__device__ __forceinline__ int a2_wrap(int i, int n)
{
    // halos pass the mesh's edge by at most a tile
    if ((unsigned)i < (unsigned)n) return i;
    const int m = i % n;
    return m < 0 ? m + n : m;
}

}  // namespace

template <typename T, int A2_Y>
__global__ __attribute__((amdgpu_flat_work_group_size(A2_X * A2_Y, A2_X * A2_Y), amdgpu_waves_per_eu(2))) void k_adj2(
    const Inst<T>* __restrict__ Pp, const T* __restrict__ fin, const T* __restrict__ force,
    const T* __restrict__ lam_in, T gt, T gth, int tiles_x, T* __restrict__ lam_out, T* __restrict__ grad)
{
    constexpr int A2_NT = A2_X * A2_Y, A2_OY = A2_Y - 2 * A2_HALO;
    __shared__ T lds[A2_SLOTS * A2_NT];
    const Inst<T>& P = *Pp;
    const int blk = xcd_order((int)blockIdx.x, (int)gridDim.x);
    const int tid = (int)threadIdx.x, cx = tid & (A2_X - 1), r = tid / A2_X;
    const int nx = P.n[0], ny = P.n[1];
    const bool perx = P.per[0] != 0, pery = P.per[1] != 0;
    const long long nc = P.nc;
    const int gx = (blk % tiles_x) * A2_OX - A2_HALO + cx, gy = (blk / tiles_x) * A2_OY - A2_HALO + r;
    // source cell: wrapped on a periodic axis; beyond a wall the nearest cell,
    // whose pairs do not exist (their flux scales are zero)
    const int sx = perx ? a2_wrap(gx, nx) : min(max(gx, 0), nx - 1);
    const int sy = pery ? a2_wrap(gy, ny) : min(max(gy, 0), ny - 1);
    const bool inx = perx || (gx >= 0 && gx < nx), iny = pery || (gy >= 0 && gy < ny);
    const bool own = cx >= A2_HALO && cx < A2_X - A2_HALO && r >= A2_HALO && r < A2_Y - A2_HALO && gx < nx && gy < ny;
    const long long ci = (long long)sy * nx + sx;
    const int rd = max(r - 1, 0), ru = min(r + 1, A2_Y - 1);
    auto at = [&](int slot, int row) -> T& { return lds[slot * A2_NT + row * A2_X + cx]; };

    // the tile holds cells next to a wall of the axis (workgroup-uniform)
    const int tx0 = gx - cx, ty0 = gy - r;
    const bool wx[2] = {!perx && tx0 <= 1, !perx && tx0 + A2_X > nx - 2};
    const bool wy[2] = {!pery && ty0 <= 1, !pery && ty0 + A2_Y > ny - 2};

    T phi[9], lam[9], fc[2] = {T(0), T(0)};
    {
        T f[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) f[q] = fin[q * nc + ci];
#pragma unroll
        for (int q = 0; q < 9; ++q) lam[q] = lam_in[q * nc + ci];
        if (force) {
            fc[0] = force[ci];
            fc[1] = force[nc + ci];
        }
        d2_phi<T, false, true>(P, f, gt * (P.G0[0] + fc[0]), gt * (P.G0[1] + fc[1]), phi);
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        if (D2Q9::ey(q) != 0) {
            at(A2_PHI + a2_six(1, q), r) = phi[q];
            at(A2_LAM + a2_six(1, q), r) = lam[q];
        }
    }
    at(A2_PHI + 6, r) = phi[4];
    at(A2_FRC, r) = fc[0];
    at(A2_FRC + 1, r) = fc[1];
    T kxp, kxm, kyp, kym;
    a2_coef(P, 0, sx, kxp, kxm);
    a2_coef(P, 1, sy, kyp, kym);
    // psi across y faces, from the x derivative
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const int e = D2Q9::ex(q);
        if (e != 0) {
            const T d = kxp * (lane_next(phi[q]) - phi[q]) + kxm * (lane_prev(phi[q]) - phi[q]);
            at(A2_PSI + a2_six(0, q), r) = e > 0 ? phi[q] - d : phi[q] + d;
        }
    }
    __syncthreads();

    const T hc = P.h * P.c;
    T phat[9], g0 = T(0), g1 = T(0);
#pragma unroll
    for (int q = 0; q < 9; ++q) phat[q] = T(4.0 / 3.0) * lam[q];
    {
        // x faces: psi across them, from the y derivative
        T ps[9], psi[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            const int e = D2Q9::ey(q);
            ps[q] = phi[q];
            psi[q] = T(0);
            if (e != 0) {
                const int s = A2_PHI + a2_six(1, q);
                const T d = kyp * (at(s, ru) - phi[q]) + kym * (at(s, rd) - phi[q]);
                ps[q] = e > 0 ? phi[q] - d : phi[q] + d;
            }
        }
        const T w = P.m[0].w[sx], k = hc * P.m[0].gn[sx];
        {
            A2Pair<T> p;
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                p.psR[q] = ps[q];
                p.phR[q] = phi[q];
                p.lamR[q] = lam[q];
                p.psL[q] = lane_prev(ps[q]);
                p.phL[q] = D2Q9::ex(q) == 0 ? T(0) : (D2Q9::ey(q) == 0 ? p.psL[q] : lane_prev(phi[q]));
                p.lamL[q] = D2Q9::ex(q) == 0 ? T(0) : lane_prev(lam[q]);
            }
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                p.fR[d] = fc[d];
                p.fL[d] = lane_prev(fc[d]);
            }
            const bool pair = iny && (perx || (gx >= 1 && gx < nx));
            const T sR = pair ? P.c * P.m[0].fdx[sx] : T(0);
            const T sL = pair ? P.c * P.m[0].fdx[sx > 0 ? sx - 1 : nx - 1] : T(0);
            T b[9], bx, by;
            a2_face<T, 0>(P, p, w, k, sL, sR, gth, b, bx, by);
            a2_take<T, 0>(true, w, k, b, bx, by, phat, psi, g0, g1);
#pragma unroll
            for (int q = 0; q < 9; ++q) b[q] = lane_next(b[q]);
            a2_take<T, 0>(false, lane_next(w), lane_next(k), b, lane_next(bx), lane_next(by), phat, psi, g0, g1);
        }
#pragma unroll 1
        for (int side = 0; side < 2; ++side) {
            if (!(side ? wx[1] : wx[0])) continue;
            const int at_low = side ? nx - 2 : 0;  // the pair's lower cell
            const bool up = gx != at_low;
            A2Pair<T> p;
            auto pick = [&](T v, T& L, T& R) {
                const T a = lane_prev(v), b = lane_next(v);
                L = up ? a : v;
                R = up ? v : b;
            };
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                pick(ps[q], p.psL[q], p.psR[q]);
                p.phL[q] = p.phR[q] = p.lamL[q] = p.lamR[q] = T(0);
                if (D2Q9::ey(q) == 0) {
                    p.phL[q] = p.psL[q];
                    p.phR[q] = p.psR[q];
                } else if (D2Q9::ex(q) != 0) {
                    pick(phi[q], p.phL[q], p.phR[q]);
                }
                if (D2Q9::ex(q) != 0) pick(lam[q], p.lamL[q], p.lamR[q]);
            }
#pragma unroll
            for (int d = 0; d < 2; ++d) pick(fc[d], p.fL[d], p.fR[d]);
            if (iny && (gx == at_low || gx == at_low + 1))
                a2_wall<T, 0>(P, side, up, p, P.m[0].w[at_low + 1], hc * P.m[0].gn[at_low + 1], gth, phat, psi, g0, g1);
        }
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            if (D2Q9::ey(q) == 0) continue;
            at(A2_DH + a2_six(1, q), r) = psi[q];
            // the derivative's own-cell part: psi = phi - e (kp (phi_+ - phi) + km (phi_- - phi))
            phat[q] += D2Q9::ey(q) > 0 ? (kyp + kym) * psi[q] : -(kyp + kym) * psi[q];
        }
    }
    asm volatile("" ::: "memory");  // the y faces' reads are not hoisted into the x faces
    T psi[9];                       // psi-hat of the y faces
    {
        // a pair of cells at LDS rows rl and rl + 1
        auto pair_at = [&](int rl, A2Pair<T>& p) {
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                const int e = D2Q9::ey(q), t = D2Q9::ex(q);
                const int sp = e != 0 ? A2_PHI + a2_six(1, q) : A2_PHI + 6, ss = A2_PSI + a2_six(0, q);
                const bool need = e != 0 || t == 0;
                p.phL[q] = need ? at(sp, rl) : T(0);
                p.phR[q] = need ? at(sp, rl + 1) : T(0);
                p.psL[q] = t != 0 ? at(ss, rl) : p.phL[q];
                p.psR[q] = t != 0 ? at(ss, rl + 1) : p.phR[q];
                p.lamL[q] = e != 0 ? at(A2_LAM + a2_six(1, q), rl) : T(0);
                p.lamR[q] = e != 0 ? at(A2_LAM + a2_six(1, q), rl + 1) : T(0);
            }
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                p.fL[d] = at(A2_FRC + d, rl);
                p.fR[d] = at(A2_FRC + d, rl + 1);
            }
        };
#pragma unroll
        for (int q = 0; q < 9; ++q) psi[q] = T(0);
#pragma unroll 1
        for (int side = 0; side < 2; ++side) {
            if (!(side ? wy[1] : wy[0])) continue;
            const int at_low = side ? ny - 2 : 0;
            const bool up = gy != at_low;
            if (inx && (gy == at_low || gy == at_low + 1)) {
                A2Pair<T> p;
                pair_at(min(max(up ? r - 1 : r, 0), A2_Y - 2), p);
                a2_wall<T, 1>(P, side, up, p, P.m[1].w[at_low + 1], hc * P.m[1].gn[at_low + 1], gth, phat, psi, g0, g1);
            }
        }
        T b[9], bx, by;
        const T w = P.m[1].w[sy], k = hc * P.m[1].gn[sy];
        {
            const bool pair = inx && (pery || (gy >= 1 && gy < ny));
            const T sR = pair ? P.c * P.m[1].fdx[sy] : T(0);
            const T sL = pair ? P.c * P.m[1].fdx[sy > 0 ? sy - 1 : ny - 1] : T(0);
            A2Pair<T> p;
            pair_at(rd, p);
            a2_face<T, 1>(P, p, w, k, sL, sR, gth, b, bx, by);
            a2_take<T, 1>(true, w, k, b, bx, by, phat, psi, g0, g1);
        }
        __syncthreads();  // phi and lam planes are read
#pragma unroll
        for (int q = 0; q < 9; ++q) at(q, r) = b[q];
        at(9, r) = bx;
        at(10, r) = by;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 9; ++q) b[q] = at(q, ru);
        a2_take<T, 1>(false, P.m[1].w[sy + 1], hc * P.m[1].gn[sy + 1], b, at(9, ru), at(10, ru), phat, psi, g0, g1);
    }
    // transposed derivatives: a cell takes kp of the cell below and km of the
    // cell above times their psi-hat (times -e), and its own with kp + km
    const T xp = lane_prev(kxp), xm = lane_next(kxm);
    T yp, ym, unused;
    a2_coef(P, 1, pery ? (sy > 0 ? sy - 1 : ny - 1) : max(sy - 1, 0), yp, unused);
    a2_coef(P, 1, pery ? (sy < ny - 1 ? sy + 1 : 0) : min(sy + 1, ny - 1), unused, ym);
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const int ex = D2Q9::ex(q), ey = D2Q9::ey(q);
        if (ex != 0) {
            const T s = (kxp + kxm) * psi[q] - xp * lane_prev(psi[q]) - xm * lane_next(psi[q]);
            phat[q] += ex > 0 ? s : -s;
        }
        if (ey != 0) {
            const T s = yp * at(A2_DH + a2_six(1, q), rd) + ym * at(A2_DH + a2_six(1, q), ru);
            phat[q] -= ey > 0 ? s : -s;
        }
    }
    if (!own) return;
    // the cell's moments again: cheaper than held over the faces
    asm volatile("" ::: "memory");
    T f[9], v[9], cgx, cgy, rho;
#pragma unroll
    for (int q = 0; q < 9; ++q) f[q] = fin[q * nc + ci];
    const T Gx = gt * (P.G0[0] + fc[0]), Gy = gt * (P.G0[1] + fc[1]);
    const EqD2<T> E = d2_point<T, false, true>(P, f, Gx, Gy, P.h, rho);
    a2_relax<T, -1>(P, E, Gx, Gy, P.h, P.B1, P.C1, phat, v, cgx, cgy);
#pragma unroll
    for (int q = 0; q < 9; ++q) lam_out[q * nc + ci] = v[q] - T(1.0 / 3.0) * lam[q];
    if (grad) {
        grad[ci] += gt * cgx + gth * g0;
        grad[nc + ci] += gt * cgy + gth * g1;
    }
}

static long long adjoint_tiles(const Inst<double>& P, int rows)
{
    const int oy = rows - 2 * A2_HALO;
    return (long long)((P.n[0] + A2_OX - 1) / A2_OX) * ((P.n[1] + oy - 1) / oy);
}

// Time of a launch in microseconds by tile rows: 16 rows, one workgroup per CU: 10.1 a
// round, 14.1 with walls; 8 rows, two per CU: 7.6 (11.6) while no CU has two,
// else 1.2 + 8.6 (12.6) a round.  Measured on periodic meshes, 8 against 16 rows:
// 128^2 7.6, 10.1; 200 x 150 9.8, 10.4; 256^2 15.0, 11.0; 300^2 18.0, 19.2; 512^2
// 42.9, 40.3.  (walls: the share of the tiles that holds one where an XCD has most
// of them)
static double adjoint_rows_us(const Inst<double>& P, int rows, bool walls, int n_cu)
{
    const long long cu = n_cu > 0 ? n_cu : 1, tiles = adjoint_tiles(P, rows);
    const double tx = (P.n[0] + A2_OX - 1) / A2_OX, ty = (double)tiles / tx;
    const double fx = P.per[0] ? 1.0 : std::max(0.0, 1.0 - 2.0 / tx), fy = P.per[1] ? 1.0 : std::max(0.0, 1.0 - 8.0 / ty);
    const double w = walls ? 4.0 * (1.0 - fx * fy) : 0.0;
    if (rows == A2_ROWS) return (10.1 + w) * (double)((tiles + cu - 1) / cu);
    return tiles <= cu ? 7.6 + w : 1.2 + (8.6 + w) * (double)((tiles + 2 * cu - 1) / (2 * cu));
}

// The rows of a launch, compared without walls, as the time of both kinds of tiles
// grows alike: with each kind's own share 5035 x 54 inside walls takes 8 rows, 55
// us against 46.
static int adjoint_rows(const Inst<double>& P, int n_cu)
{
    return adjoint_rows_us(P, A2_FEW, false, n_cu) < adjoint_rows_us(P, A2_ROWS, false, n_cu) ? A2_FEW : A2_ROWS;
}

double adjoint_tile_us(const Inst<double>& P, int n_cu)
{
    return adjoint_rows_us(P, adjoint_rows(P, n_cu), true, n_cu);
}

void adjoint_tile_launch(const Inst<double>* Pd, const Inst<double>& P, const void* f, const void* force, double gt,
                         double gth, const void* lam, void* lam_out, void* grad, int n_cu, hipStream_t st)
{
    const int tiles_x = (P.n[0] + A2_OX - 1) / A2_OX;
    auto launch = [&](auto kern, int rows) {
        hipLaunchKernelGGL(kern, dim3((unsigned)adjoint_tiles(P, rows)), dim3(A2_X * rows), 0, st, Pd, (const double*)f,
                           (const double*)force, (const double*)lam, gt, gth, tiles_x, (double*)lam_out, (double*)grad);
    };
    if (adjoint_rows(P, n_cu) == A2_FEW)
        launch(k_adj2<double, A2_FEW>, A2_FEW);
    else
        launch(k_adj2<double, A2_ROWS>, A2_ROWS);
}

}  // namespace dugks
