// kernels_tile.hip -- the FP64 D2Q9 step on tiles of 32 x 16 cells, one lane per
// cell, several time steps per launch; on flatter tiles, one step per launch,
// where most of those would be halo or hold a wall.
//
// A workgroup loads a tile of the state into registers and advances it S
// steps; cells within S of the tile's edge lose their neighbours one layer
// per step, so neighbouring tiles overlap by 2 S and the 32 - 2 S by 16 - 2 S
// cells inside are written.  Along x a lane's neighbours are the lanes beside
// it (DPP wave shifts; a wave holds two rows of 32); along y they are
// exchanged through LDS.  With
//   psi_y(c) = f-bar-plus(c) - h xi_x d_x f-bar-plus(c)   (psi_x likewise)
// formed once per cell, an interface value is (1 - w) psi_L + w psi_R - h
// xi_n (f-bar-plus_R - f-bar-plus_L) / (x_R - x_L) (Eq. gradient), and every
// interface of a tile is evaluated once: a lane takes its cell's upper x and
// upper y interface.  The LDS holds 13 values per cell for the row above and
// below and the 6 fluxes of the upper y interface: 76 KB in FP64, two
// workgroups per CU.
//
// What bounds it: FP64 issue (about 570 instructions per wave and step, 8
// waves a tile) on meshes that fill the chip, the latency of one tile's chain
// on small ones; the state crosses memory once per launch.  us a step, against
// the kernel that marches rows of 128 columns with two lanes per column, one
// step per launch: 1024^2 cavity FP64 28.7 against 52.7, 128^2 stretched cavity FP64 3.5 against 8.95, 40 x 20 channel FP64 3.8
// against 8.9, 64 uneven instances FP64 126 against 175.  A march along y with
// the rows in registers and no LDS (one lane per column, one step per launch)
// took 41, 8.5 and 8.3 for the first three.  Long meshes of few rows: see
// tile_pick.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <utility>

#include "ctx.hpp"
#include "kernels_general.hpp"
#include "march.hpp"
#include "wave.hpp"

namespace dugks {

// cells of a tile, halo included: along x 32 or 64 (a wave holds whole rows), a
// multiple of 64 in all
constexpr int TILES[TILE_SHAPES][2] = {{32, 16}, {32, 8}, {32, 6}, {64, 4}};
constexpr int TILE_SLOTS = 19;
static_assert(2 * TILE_MAX_STEPS < TILES[0][1], "a tile needs rows of its own");

// LDS slots of a cell: f-bar-plus of the velocities with e_y != 0 in 0..5,
// psi_y of those with e_x != 0 in 6..11, the rest velocity in 12, the upper y
// interface's original values in 13..18
__host__ __device__ constexpr int slot_phi(int q) { return q == 0 ? 0 : q == 2 ? 1 : q == 3 ? 2 : q == 5 ? 3 : q == 6 ? 4 : 5; }
__host__ __device__ constexpr int slot_psi(int q)
{
    return q == 4 ? 12 : (q == 3 || q == 5) ? slot_phi(q) : 6 + (q < 3 ? q : q - 3);
}

// coefficients of one cell along one axis: its upper interface's weight and
// h c / (x_R - x_L), h c times its derivative coefficients, c dt / Delta
template <typename T>
struct AxisCoef {
    T w, k, kp, km, fd;
};

template <typename T, bool UNI>
__device__ __forceinline__ AxisCoef<T> axis_coef(const Inst<T>& P, int a, int j, int f)
{
    const T hc = P.h * P.c;
    if constexpr (UNI) return AxisCoef<T>{T(0.5), hc * P.ugn[a], T(2) * (hc * P.uct[a]), T(0), P.ufdx[a] * P.c};
    const AxisMetric<T>& m = P.m[a];
    return AxisCoef<T>{m.w[f], hc * m.gn[f], hc * m.cp[j], hc * m.cm[j], m.fdx[j] * P.c};
}

// cell of coordinate i on a periodic axis of n cells (-64 < i < n + 64)
__device__ __forceinline__ int tile_wrap(int i, int n)
{
    if (n >= 64) return i < 0 ? i + n : (i >= n ? i - n : i);
    return ((i % n) + n) % n;
}

// One workgroup's work: tile (tx, ty) of instance P, `steps` steps from time
// index k0 (time t0 + k dt).  ACC: there is an acceleration; FIELD: part of it
// is a force field (force may still be null: a batch where only some
// instances have one).
// NW: no cell of the tile lies at or beyond a wall.  REREAD: the y stage reads
// the cell's own values back from LDS instead of holding them in registers
// over the x stage (the wall body at four waves per SIMD).
template <typename T, int TX, int TY, bool UNI, bool ACC, bool FIELD, bool ORIG, bool NW, bool REREAD>
__device__ __forceinline__ void tile_body(const Inst<T>& P, const T* __restrict__ fin, const T* __restrict__ force,
                                          T* __restrict__ fout, double t0, long long k0, int steps, int btx, int bty,
                                          T* lds)
{
#pragma clang fp contract(off)
    const int tid = (int)threadIdx.x;
    const int cx = tid & (TX - 1), r = tid / TX;
    const int nx = P.n[0], ny = P.n[1];
    const long long nc = P.nc;
    const bool perx = P.per[0] != 0, pery = P.per[1] != 0;
    const int gx = btx * (TX - 2 * steps) - steps + cx, gy = bty * (TY - 2 * steps) - steps + r;
    // source cell: wrapped on a periodic axis; beyond a wall the nearest cell
    // (ghost columns are overwritten, what lies further is never used)
    const int sx = perx ? tile_wrap(gx, nx) : min(max(gx, 0), nx - 1);
    const int sy = pery ? tile_wrap(gy, ny) : min(max(gy, 0), ny - 1);
    const bool own = cx >= steps && cx < TX - steps && r >= steps && r < TY - steps && gx < nx && gy < ny;
    const bool glo = !NW && !perx && gx == -1, ghi = !NW && !perx && gx == nx;
    const bool bot = !NW && !pery && gy == 0, top = !NW && !pery && gy == ny - 1;
    // the tile holds a ghost column of the low / high x wall (workgroup-uniform)
    const bool xlo = !NW && !perx && btx * (TX - 2 * steps) - steps < 0;
    const bool xhi = !NW && !perx && btx * (TX - 2 * steps) - steps + TX > nx;
    const long long ci = (long long)sy * nx + sx;
    T f[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) f[q] = fin[q * nc + ci];
    const int fx_i = min(max(gx + 1, 0), nx);
    const AxisCoef<T> mx = axis_coef<T, UNI>(P, 0, sx, perx ? sx + 1 : fx_i);
    const AxisCoef<T> my = axis_coef<T, UNI>(P, 1, sy, sy + 1);
    const T rxl = P.rlo[0], rxh = P.rhi[0], ryl = P.rlo[1], ryh = P.rhi[1];
    // the force field of the cell and, interpolated, of its upper interfaces
    // (and of a wall row's lower one): constant over the steps
    T g0 = T(0), g1 = T(0), gyu[2] = {T(0), T(0)}, gyl[2] = {T(0), T(0)}, gxu[2] = {T(0), T(0)};
    T wyl = T(0.5), kyl = my.k;  // lower y interface of a wall row
    if constexpr (!UNI) {
        wyl = P.m[1].w[sy];
        kyl = P.h * P.c * P.m[1].gn[sy];
    }
    if constexpr (FIELD) {
        if (force) {
            const int up = top ? max(sy - 1, 0) : (pery && sy == ny - 1 ? 0 : min(sy + 1, ny - 1));
            const int dn = pery && sy == 0 ? ny - 1 : max(sy - 1, 0);
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                const T* fd = force + d * nc;
                T own_v = fd[ci], up_v = fd[(long long)up * nx + sx], dn_v = fd[(long long)dn * nx + sx];
                if (xlo) {
                    const T a1 = lane_next(own_v), b1 = lane_next(up_v), c1 = lane_next(dn_v);
                    const T a2 = lane_next(a1), b2 = lane_next(b1), c2 = lane_next(c1);
                    if (glo) {
                        own_v = fma_(rxl, a2 - a1, a1);
                        up_v = fma_(rxl, b2 - b1, b1);
                        dn_v = fma_(rxl, c2 - c1, c1);
                    }
                }
                if (xhi) {
                    const T a1 = lane_prev(own_v), b1 = lane_prev(up_v), c1 = lane_prev(dn_v);
                    const T a2 = lane_prev(a1), b2 = lane_prev(b1), c2 = lane_prev(c1);
                    if (ghi) {
                        own_v = fma_(rxh, a2 - a1, a1);
                        up_v = fma_(rxh, b2 - b1, b1);
                        dn_v = fma_(rxh, c2 - c1, c1);
                    }
                }
                if (d == 0) g0 = own_v;
                else g1 = own_v;
                const T ab = top ? fma_(ryh, up_v - own_v, own_v) : up_v;
                const T be = bot ? fma_(ryl, up_v - own_v, own_v) : dn_v;
                gyu[d] = fma_(my.w, ab - own_v, own_v);
                gyl[d] = fma_(wyl, own_v - be, be);
                const T rt = lane_next(own_v);
                gxu[d] = fma_(mx.w, rt - own_v, own_v);
            }
        }
    }
    // the time factors of the steps: lane 2 s takes step s's, lane 2 s + 1
    // that of its interface time
    T tf = (T)P.gphase;
    if (P.omega != 0.0) {
        const int l = tid & 63, s = l >> 1;
        const double t = t0 + (double)(k0 + s) * P.dtd;
        tf = tfac(P, (l & 1) ? t + 0.5 * P.dtd : t);
    }
    auto ghost1 = [&](T& a) {
        if (xlo) {
            const T s1 = lane_next(a), s2 = lane_next(s1);
            if (glo) a = fma_(rxl, s2 - s1, s1);
        }
        if (xhi) {
            const T s1 = lane_prev(a), s2 = lane_prev(s1);
            if (ghi) a = fma_(rxh, s2 - s1, s1);
        }
    };
    auto at = [&](int slot, int row) -> T& { return lds[(slot * TY + row) * TX + cx]; };
    const int ru = min(r + 1, TY - 1), rd = max(r - 1, 0);
    const T hh = T(0.5) * P.h;

    for (int s = 0; s < steps; ++s) {
        const T gt = P.omega != 0.0 ? __shfl(tf, 2 * s) : tf, gth = P.omega != 0.0 ? __shfl(tf, 2 * s + 1) : tf;
        T phi[9], ps[9];
        {
            T Gx = T(0), Gy = T(0);
            if constexpr (ACC) {
                Gx = gt * (P.G0[0] + g0);
                Gy = gt * (P.G0[1] + g1);
            }
            d2_phi<T, ORIG, ACC>(P, f, Gx, Gy, phi);
        }
        if (xlo || xhi) {
#pragma unroll
            for (int q = 0; q < 9; ++q) ghost1(phi[q]);
        }
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            const int e = D2Q9::ex(q);
            ps[q] = e == 0 ? phi[q] : d2_psi<T, UNI>(e, mx.kp, mx.km, lane_prev(phi[q]), phi[q], lane_next(phi[q]));
            if (D2Q9::ey(q) != 0) at(slot_phi(q), r) = phi[q];
            if (e != 0 || q == 4) at(slot_psi(q), r) = ps[q];
        }
        // f~+ of Eq. (f_tilde_+); the fluxes are added as they come
#pragma unroll
        for (int q = 0; q < 9; ++q) f[q] = fma_(phi[q] - f[q], T(1.0 / 3.0), phi[q]);
        __syncthreads();
        // the upper x interface; the lower one is that of the lane before
        {
            T v[9];
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                const int e = D2Q9::ey(q);
                T p = phi[q];
                if (e != 0) {
                    // the ghost row beyond a wall by extrapolation
                    T u = at(slot_phi(q), ru), d = at(slot_phi(q), rd);
                    if constexpr (!NW) {
                        const T gu = fma_(ryh, d - p, p), gd = fma_(ryl, u - p, p);
                        u = top ? gu : u;
                        d = bot ? gd : d;
                    }
                    p = d2_psi<T, UNI>(e, my.kp, my.km, d, p, u);
                }
                const T pR = lane_next(p);
                const T hR = (e != 0 && D2Q9::ex(q) != 0) ? lane_next(phi[q]) : pR;
                v[q] = d2_recon<T, UNI>(D2Q9::ex(q), mx.w, mx.k, p, pR, phi[q], hR);
            }
            const T Gx = ACC ? gth * (P.G0[0] + gxu[0]) : T(0), Gy = ACC ? gth * (P.G0[1] + gxu[1]) : T(0);
            T rho;
            EqD2<T> E = d2_point<T, ORIG, ACC>(P, v, Gx, Gy, hh, rho);
            if (xlo || xhi) {
                // wall faces: the opposite interface is the upper face of the
                // next lane (low wall, ghost lane) or of the previous one
                if (xlo) {
                    NeqD2<T> I;
                    d2_capture<T, 0>(E, rho, v, 1, I);
                    I.rho = lane_next(I.rho);
                    I.ux = lane_next(I.ux);
                    I.uy = lane_next(I.uy);
#pragma unroll
                    for (int k = 0; k < 3; ++k) I.ne[k] = lane_next(I.ne[k]);
                    if (glo) d2_wall<T, 0, ORIG>(P, 0, 1, v, I, gth);
                }
                if (xhi) {
                    NeqD2<T> I;
                    d2_capture<T, 0>(E, rho, v, -1, I);
                    I.rho = lane_prev(I.rho);
                    I.ux = lane_prev(I.ux);
                    I.uy = lane_prev(I.uy);
#pragma unroll
                    for (int k = 0; k < 3; ++k) I.ne[k] = lane_prev(I.ne[k]);
                    if (gx == nx - 1) d2_wall<T, 0, ORIG>(P, 1, -1, v, I, gth);
                }
                E = d2_point<T, ORIG, ACC>(P, v, Gx, Gy, hh, rho);
            }
            d2_relax_pair<T, ACC>(E, 6, P.B7, P.C7, v[6], v[2]);
            d2_relax_pair<T, ACC>(E, 7, P.B7, P.C7, v[7], v[1]);
            d2_relax_pair<T, ACC>(E, 8, P.B7, P.C7, v[8], v[0]);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                f[k] = fma_(mx.fd, v[k] - lane_prev(v[k]), f[k]);
                f[6 + k] = fma_(-mx.fd, v[6 + k] - lane_prev(v[6 + k]), f[6 + k]);
            }
        }
        asm volatile("" ::: "memory");  // the y stage's LDS reads are not hoisted into the x stage
        T vy[6];                        // the upper y interface
        {
            if constexpr (REREAD) {
#pragma unroll
                for (int q = 0; q < 9; ++q) {
                    ps[q] = at(slot_psi(q), r);
                    if (D2Q9::ey(q) != 0) phi[q] = at(slot_phi(q), r);
                }
            }
            // the interface between this row and the row at LDS index rr
            // (above: the upper interface; below: its mirror, the lower one)
            auto face_values = [&](bool lower, T (&v)[9]) {
#pragma unroll
                for (int q = 0; q < 9; ++q) {
                    const int rr = lower ? rd : ru;
                    const T pn = at(slot_psi(q), rr);
                    const T hn = D2Q9::ey(q) == 0 ? T(0) : D2Q9::ex(q) == 0 ? pn : at(slot_phi(q), rr);
                    if (lower) v[q] = d2_recon<T, UNI>(D2Q9::ey(q), wyl, kyl, pn, ps[q], hn, phi[q]);
                    else v[q] = d2_recon<T, UNI>(D2Q9::ey(q), my.w, my.k, ps[q], pn, phi[q], hn);
                }
            };
            // a wall face: the row beyond it by extrapolation through this
            // row and the one inside
            auto wall_values = [&](bool lower, T (&v)[9]) {
                const T re = lower ? ryl : ryh;
                const int rr = lower ? ru : rd;
#pragma unroll
                for (int q = 0; q < 9; ++q) {
                    T pn = at(slot_psi(q), rr);
                    T hn = D2Q9::ey(q) == 0 ? T(0) : D2Q9::ex(q) == 0 ? pn : at(slot_phi(q), rr);
                    pn = fma_(re, pn - ps[q], ps[q]);
                    if (D2Q9::ey(q) != 0) hn = fma_(re, hn - phi[q], phi[q]);
                    if (lower) v[q] = d2_recon<T, UNI>(D2Q9::ey(q), wyl, kyl, pn, ps[q], hn, phi[q]);
                    else v[q] = d2_recon<T, UNI>(D2Q9::ey(q), my.w, my.k, ps[q], pn, phi[q], hn);
                }
            };
            const T Gu0 = ACC ? gth * (P.G0[0] + gyu[0]) : T(0), Gu1 = ACC ? gth * (P.G0[1] + gyu[1]) : T(0);
            const T Gl0 = ACC ? gth * (P.G0[0] + gyl[0]) : T(0), Gl1 = ACC ? gth * (P.G0[1] + gyl[1]) : T(0);
            T v[9], rho;
            if (!top) {
                face_values(false, v);
            } else {
                // high wall: its opposite interface is this row's lower one
                NeqD2<T> info;
                face_values(true, v);
                const EqD2<T> O = d2_point<T, ORIG, ACC>(P, v, Gl0, Gl1, hh, rho);
                d2_capture<T, 1>(O, rho, v, -1, info);
                wall_values(false, v);
                d2_wall<T, 1, ORIG>(P, 3, -1, v, info, gth);
            }
            const EqD2<T> E = d2_point<T, ORIG, ACC>(P, v, Gu0, Gu1, hh, rho);
            NeqD2<T> info;
            if (bot) d2_capture<T, 1>(E, rho, v, 1, info);
            d2_relax_pair<T, ACC>(E, 5, P.B7, P.C7, v[5], v[3]);
            d2_relax_pair<T, ACC>(E, 6, P.B7, P.C7, v[6], v[2]);
            d2_relax_pair<T, ACC>(E, 8, P.B7, P.C7, v[8], v[0]);
            // the row below a wall stores nothing: its slot holds the wall
            // face
            if (NW || pery || gy != -1) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    at(13 + k, r) = v[3 * k];
                    at(16 + k, r) = v[3 * k + 2];
                }
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                vy[k] = v[3 * k];
                vy[3 + k] = v[3 * k + 2];
            }
            if (bot) {
                // low wall: the opposite interface was the upper one
                wall_values(true, v);
                d2_wall<T, 1, ORIG>(P, 2, 1, v, info, gth);
                const EqD2<T> B = d2_point<T, ORIG, ACC>(P, v, Gl0, Gl1, hh, rho);
                d2_relax_pair<T, ACC>(B, 5, P.B7, P.C7, v[5], v[3]);
                d2_relax_pair<T, ACC>(B, 6, P.B7, P.C7, v[6], v[2]);
                d2_relax_pair<T, ACC>(B, 8, P.B7, P.C7, v[8], v[0]);
                if (r > 0) {
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        at(13 + k, r - 1) = v[3 * k];
                        at(16 + k, r - 1) = v[3 * k + 2];
                    }
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            f[3 * k] = fma_(my.fd, vy[k] - at(13 + k, rd), f[3 * k]);
            f[3 * k + 2] = fma_(-my.fd, vy[3 + k] - at(16 + k, rd), f[3 * k + 2]);
        }
    }
    if (own) {
        T* o = fout + ((long long)gy * nx + gx);
#pragma unroll
        for (int q = 0; q < 9; ++q) o[q * nc] = f[q];
    }
}

// does the tile, halo included, stay clear of every wall and its ghosts?
template <int TX, int TY, typename T>
__device__ __forceinline__ bool tile_no_wall(const Inst<T>& P, int steps, int btx, int bty)
{
    const int x0 = btx * (TX - 2 * steps) - steps, y0 = bty * (TY - 2 * steps) - steps;
    if (!P.per[0] && (x0 < 0 || x0 + TX > P.n[0])) return false;
    if (!P.per[1] && (y0 <= 0 || y0 + TY >= P.n[1])) return false;
    return true;
}

// Waves per SIMD the kernel is compiled for.  Four (32 x 16: two tiles per CU) with
// both bodies: the body without wall code fits 128 registers, the wall body
// spills 26 (uniform mesh, no acceleration) to 73 (stretched, field, original
// model).  ALONE, the wall body for every tile: two or three, without spills.
// That pays where no more waves come (at most one 32 x 16 tile per CU: 128^2
// cavity FP64 3.7 against 4.6 us a step, and less code is fetched on a first
// pass) and where most tiles hold a wall: a wall tile's chain is three times that of
// the others when it spills.
#define TILE_BOUNDS(N, W) __attribute__((amdgpu_flat_work_group_size(N, N), amdgpu_waves_per_eu(W)))

template <typename T, int TX, int TY, bool UNI, bool ACC, bool FIELD, bool ORIG, bool ALONE>
__global__ TILE_BOUNDS(TX* TY, (ALONE ? 2 : 4)) void k_tile(const Inst<T>* __restrict__ Pp, const T* __restrict__ fin,
                                                           const T* __restrict__ force, T* __restrict__ fout, double t0,
                                                           long long k0, int steps, int tiles_x)
{
    __shared__ T lds[TILE_SLOTS * TX * TY];
    const int b = xcd_order((int)blockIdx.x, (int)gridDim.x);
    const Inst<T>& P = *Pp;
    const int bx = b % tiles_x, by = b / tiles_x;
    if (!ALONE && tile_no_wall<TX, TY>(P, steps, bx, by))
        tile_body<T, TX, TY, UNI, ACC, FIELD, ORIG, true, false>(P, fin, force, fout, t0, k0, steps, bx, by, lds);
    else
        tile_body<T, TX, TY, UNI, ACC, FIELD, ORIG, false, false>(P, fin, force, fout, t0, k0, steps, bx, by, lds);
}

// many instances in one launch: blocks[b] is the instance and the tile of
// workgroup b in XCD order; instance i is at time index *step0 + step (a device
// counter, so a captured graph replays with advancing time)
template <typename T, bool FIELD>
__global__ TILE_BOUNDS(TILES[0][0] * TILES[0][1], 4) void k_tile_batch(const Inst<T>* __restrict__ insts,
                                                                      const TileBlock* __restrict__ blocks,
                                                                      const T* __restrict__ fin, const T* __restrict__ forces,
                                                                      T* __restrict__ fout, const long long* __restrict__ step0,
                                                                      long long step, int steps)
{
    constexpr int TX = TILES[0][0], TY = TILES[0][1];
    __shared__ T lds[TILE_SLOTS * TX * TY];
    const TileBlock k = blocks[xcd_order((int)blockIdx.x, (int)gridDim.x)];
    const Inst<T>& P = insts[k.inst];
    const int bx = k.bx, by = k.by;
    const long long k0 = *step0 + step;
    const T* force = (FIELD && forces && P.foff >= 0) ? forces + P.foff : nullptr;
    const bool nw = tile_no_wall<TX, TY>(P, steps, bx, by);
    fin += P.off;
    fout += P.off;
    if (P.uni) {
        if (nw) tile_body<T, TX, TY, true, true, FIELD, false, true, false>(P, fin, force, fout, 0.0, k0, steps, bx, by, lds);
        else tile_body<T, TX, TY, true, true, FIELD, false, false, true>(P, fin, force, fout, 0.0, k0, steps, bx, by, lds);
    } else {
        if (nw) tile_body<T, TX, TY, false, true, FIELD, false, true, false>(P, fin, force, fout, 0.0, k0, steps, bx, by, lds);
        else tile_body<T, TX, TY, false, true, FIELD, false, false, true>(P, fin, force, fout, 0.0, k0, steps, bx, by, lds);
    }
}

// the same on flat tiles, every tile on the wall body (two waves per SIMD)
template <typename T, int TX, int TY, bool FIELD>
__global__ TILE_BOUNDS(TX* TY, 2) void k_flat_batch(const Inst<T>* __restrict__ insts, const TileBlock* __restrict__ blocks,
                                                    const T* __restrict__ fin, const T* __restrict__ forces,
                                                    T* __restrict__ fout, const long long* __restrict__ step0, long long step)
{
    __shared__ T lds[TILE_SLOTS * TX * TY];
    const TileBlock k = blocks[xcd_order((int)blockIdx.x, (int)gridDim.x)];
    const Inst<T>& P = insts[k.inst];
    const long long k0 = *step0 + step;
    const T* force = (FIELD && forces && P.foff >= 0) ? forces + P.foff : nullptr;
    fin += P.off;
    fout += P.off;
    if (P.uni) tile_body<T, TX, TY, true, true, FIELD, false, false, false>(P, fin, force, fout, 0.0, k0, 1, k.bx, k.by, lds);
    else tile_body<T, TX, TY, false, true, FIELD, false, false, false>(P, fin, force, fout, 0.0, k0, 1, k.bx, k.by, lds);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// tiles of a launch of `steps` steps on an nx x ny mesh along each axis
void tile_grid(int nx, int ny, int shape, int steps, int* tiles_x, int* tiles_y)
{
    const int ox = TILES[shape][0] - 2 * steps, oy = TILES[shape][1] - 2 * steps;
    *tiles_x = (nx + ox - 1) / ox;
    *tiles_y = (ny + oy - 1) / oy;
}

// Time of a launch of `steps` steps on `tiles` tiles in microseconds, `walls` the
// share of them that holds a wall where the CUs have most of those.  A launch costs
// 4.5, a tile with its CU to itself 2.9 per step (latency; a spilling wall body 6.5,
// but 5.5 where no tile has `corners`, the wall code of both axes, and all run at
// once, two per CU), and a CU with several tiles what follows for each.  Fitted
// on MI355X to meshes of 40 x 20 to 2048^2, 10^6 x 1 to 65536 x 64 and 16 x 65536
// cells and 1 to 6 steps a launch (1024^2: 32.6, 27.1 and 29.8 us a step for 1, 2
// and 3 steps; 128^2 cavity: 7.4, 4.8, 4.1, 3.8, 3.7 and 3.7 us for 1 to 6).
static double tile_us(int shape, int steps, bool alone, double tiles, double walls, bool corners, int n_cu)
{
    const double cu = n_cu > 0 ? n_cu : 1, per_cu = std::ceil(tiles / cu), s = steps;
    // per tile of a CU that has several: without a wall, with one, all on the wall body
    static const double each[TILE_SHAPES][3] = {{0, 0, 0}, {0, 0, 1.40}, {0, 0, 1.15}, {1.15, 3.0, 1.5}};
    if (alone) return 4.5 + std::max(2.9 * s, shape == 0 ? 0.0 : per_cu * each[shape][2]);
    const double free_ = shape == 0 ? 1.5 + 1.25 * s : each[shape][0], wall = shape == 0 ? 3.5 + 2.9 * s : each[shape][1];
    return 4.5 + std::max((walls <= 0 ? 2.9 : corners || per_cu > 2 ? 6.5 : 5.5) * s, per_cu * (free_ + walls * (wall - free_)));
}

// How to take a mesh: the shape and steps per launch (at most `most`) of the
// shortest time per step.  More steps save launches and passes over memory, but
// overlap the tiles more.  Flat tiles waste fewer lanes on few rows, and alone
// (the wall body without spills) they are the better ones while the rows of tiles at
// the y walls are a large share: an XCD takes a range of rows, so with up to
// eight rows of tiles one has walls only.  us a step, 32 x 16 tiles and their
// best steps against the choice (marched rows of 128 columns before both): 10^6 x
// 1 periodic 260 -> 72 (79), 10^6 x 2 cavity 642 -> 100 (121), 65536 x 16 cavity
// 82 -> 40 (55), 65536 x 64 254 -> 164 (177), 16384 x 128 109 -> 92 (101).  Between
// near equals (3 % in steps, the fit's errors) the fewer steps stay, several steps
// have to be worth 7 % against 32 x 16 alone, and a flatter shape 10 % (at 7 %
// 1024^2 cavities took 32 x 8 for single steps: plain 38 -> 38 us, but stretched 45 ->
// 48, with a field 47 -> 50).  Walls across one axis (one step alone against the
// choice): 3654 x 16 8.9 -> 6.6, 450 x 200 7.3 -> 6.7.  The results do not depend
// on the choice.
// (32 x 16 alone: up to one tile per CU, where no more waves come.  32 x 8 and 32 x 6
// have no other form: a wall-free one would take 10 to 15 % less on periodic
// meshes of three rows and more.)
static TilePick tile_pick(int nx, int ny, bool wall_x, bool wall_y, int most, int n_cu)
{
    TilePick best;
    double best_us = 1e300;
    for (int shape = 0; shape < TILE_SHAPES; ++shape)
        for (int s = 1; s <= (shape == 0 ? most : 1); ++s) {
            int tx, ty;
            tile_grid(nx, ny, shape, s, &tx, &ty);
            const double fx = wall_x ? std::max(0.0, 1.0 - 2.0 / tx) : 1.0, fy = wall_y ? std::max(0.0, 1.0 - 8.0 / ty) : 1.0;
            const double tiles = (double)tx * ty, walls = 1.0 - fx * fy;
            for (const bool alone : {false, true}) {
                if (shape == 0 && alone && (tiles > n_cu || !(wall_x || wall_y))) continue;
                if ((shape == 1 || shape == 2) && !alone) continue;
                const double us = tile_us(shape, s, alone, tiles, walls, wall_x && wall_y, n_cu) / s;
                const bool easy = shape == 0 ? alone || !best.alone : best.shape != 0;
                if (us < (easy ? (shape == 0 ? 0.97 : 1.0) : shape == 0 ? 0.93 : 0.90) * best_us) {
                    best_us = us;
                    best.shape = shape, best.steps = s, best.alone = alone;
                }
            }
        }
    return best;
}

template <typename T, bool UNI, bool ACC, bool FIELD, bool ORIG, int SHAPE, bool ALONE>
static int launch_tile(dugks_ctx* ctx, const Inst<T>& P, const void* fin, void* fout, const void* force, double t0,
                       long long k0, int steps, hipStream_t st)
{
    constexpr int TX = TILES[SHAPE][0], TY = TILES[SHAPE][1];
    int tx, ty;
    tile_grid(P.n[0], P.n[1], SHAPE, steps, &tx, &ty);
    if ((long long)tx * ty * (TX * TY) > 0xffffffffLL) return fail(ctx, DUGKS_EUNSUPPORTED, "mesh too large for one launch");
    hipLaunchKernelGGL((k_tile<T, TX, TY, UNI, ACC, FIELD, ORIG, ALONE>), dim3((unsigned)(tx * ty)), dim3(TX * TY), 0, st,
                       (const Inst<T>*)ctx->inst_dev, (const T*)fin, (const T*)force, (T*)fout, t0, k0, steps, tx);
    return hip_check(ctx, hipGetLastError(), "step launch");
}

template <typename T, bool UNI, bool ACC, bool FIELD, bool ORIG>
static int launch_tile_as(dugks_ctx* ctx, const Inst<T>& P, const void* fin, void* fout, const void* force, double t0,
                          long long k0, TilePick pick, hipStream_t st)
{
#define DUGKS_TILE(SHAPE, ALONE) \
    launch_tile<T, UNI, ACC, FIELD, ORIG, SHAPE, ALONE>(ctx, P, fin, fout, force, t0, k0, pick.steps, st)
    if (pick.shape == 1) return DUGKS_TILE(1, true);
    if (pick.shape == 2) return DUGKS_TILE(2, true);
    if (pick.shape == 3) return pick.alone ? DUGKS_TILE(3, true) : DUGKS_TILE(3, false);
    return pick.alone ? DUGKS_TILE(0, true) : DUGKS_TILE(0, false);
#undef DUGKS_TILE
}

template <typename T, bool UNI, bool ORIG>
static int launch_tile_acc(dugks_ctx* ctx, const Inst<T>& P, const void* fin, void* fout, const void* force, double t0,
                           long long k0, TilePick pick, hipStream_t st)
{
    if (force) return launch_tile_as<T, UNI, true, true, ORIG>(ctx, P, fin, fout, force, t0, k0, pick, st);
    if (P.G0[0] != T(0) || P.G0[1] != T(0))
        return launch_tile_as<T, UNI, true, false, ORIG>(ctx, P, fin, fout, force, t0, k0, pick, st);
    return launch_tile_as<T, UNI, false, false, ORIG>(ctx, P, fin, fout, force, t0, k0, pick, st);
}

// pick.steps steps from time index k0 (time t0 + k0 dt), fin -> fout
static int tile_launch(dugks_ctx* ctx, const void* fin, void* fout, const void* force, double t0, long long k0, TilePick pick,
                       hipStream_t st)
{
    const Inst<double>& P = ctx->pd;
    if (P.orig)
        return P.uni ? launch_tile_acc<double, true, true>(ctx, P, fin, fout, force, t0, k0, pick, st)
                     : launch_tile_acc<double, false, true>(ctx, P, fin, fout, force, t0, k0, pick, st);
    return P.uni ? launch_tile_acc<double, true, false>(ctx, P, fin, fout, force, t0, k0, pick, st)
                 : launch_tile_acc<double, false, false>(ctx, P, fin, fout, force, t0, k0, pick, st);
}

// the context's picks (the calls only read them)
void tile_setup(dugks_ctx* ctx)
{
    const Inst<double>& P = ctx->pd;
    ctx->tile_one = tile_pick(P.n[0], P.n[1], !P.per[0], !P.per[1], 1, ctx->n_cu);
    ctx->tile_many = tile_pick(P.n[0], P.n[1], !P.per[0], !P.per[1], TILE_MAX_STEPS, ctx->n_cu);
}

// one step at time t
int tile_step(dugks_ctx* ctx, const void* fin, void* fout, const void* force, double t, hipStream_t st)
{
    return tile_launch(ctx, fin, fout, force, t, 0, ctx->tile_one, st);
}

// nsteps steps from f_a, as dugks_run; *which_out as there
int tile_run(dugks_ctx* ctx, void* f_a, void* f_b, const void* force, double t0, int nsteps, hipStream_t st,
             int* which_out)
{
    void* cur = f_a;
    void* nxt = f_b;
    long long k = 0;
    const TilePlan plan(nsteps, ctx->tile_many.steps);
    for (long long i = 0; i < plan.launches(); ++i) {
        TilePick pick = plan.steps(i) == 1 ? ctx->tile_one : ctx->tile_many;
        pick.steps = plan.steps(i);
        const int rc = tile_launch(ctx, cur, nxt, force, t0, k, pick, st);
        if (rc != DUGKS_OK) return rc;
        std::swap(cur, nxt);
        k += pick.steps;
    }
    if (which_out) *which_out = nsteps & 1;
    return DUGKS_OK;
}

// Shape and steps per launch of a batch of n instances of nx[i] x ny[i] cells, with
// walls across x (walls[i] & 1) and y (& 2), as tile_pick; wall tiles lie
// between others here, so their mean share counts.  us a step, 32 x 16 tiles against
// the choice (marched rows before both): 64 of 4096 x 2 cells, cavities 145 -> 32
// (43), periodic 77 -> 29 (40); 64 of 4096 x 4, cavities with a field 211 -> 58
// (98); 16 of 4096 x 16, cavities 73 -> 44 (61); 56 cavities of 28 to 460 cells a
// side 83 -> 65 (211).
TilePick tile_batch_pick(int n, const int* nx, const int* ny, const unsigned char* walls, int n_cu)
{
    TilePick best;
    double best_us = 1e300;
    for (int shape = 0; shape < TILE_SHAPES; ++shape)
        for (int s = 1; s <= (shape == 0 ? TILE_MAX_STEPS : 1); ++s) {
            double tiles = 0, at_walls = 0;
            for (int i = 0; i < n; ++i) {
                int tx, ty;
                tile_grid(nx[i], ny[i], shape, s, &tx, &ty);
                const int fx = (walls[i] & 1) ? std::max(0, tx - 2) : tx, fy = (walls[i] & 2) ? std::max(0, ty - 2) : ty;
                tiles += (double)tx * ty;
                at_walls += (double)tx * ty - (double)fx * fy;
            }
            const double us = tile_us(shape, s, shape != 0, tiles, at_walls / tiles, at_walls > 0, n_cu) / s;
            if (us < (shape == 0 ? 0.97 : best.shape == 0 ? 0.93 : 1.0) * best_us) {
                best_us = us;
                best.shape = shape, best.steps = s;
            }
        }
    return best;
}

// `steps` steps of every instance; blocks: the nblocks workgroups of a launch of
// `steps` steps on tiles of shape `shape`.  (In parts where they are many: a launch
// holds less than 2^32 threads.)
template <typename K, typename... Args>
static hipError_t batch_parts(K kern, int threads, const void* insts, const TileBlock* blocks, long long nblocks,
                              const void* fin, const void* forces, void* fout, const long long* step0, hipStream_t st,
                              Args... args)
{
    constexpr long long PART = 1LL << 22;  // of at most 512 threads
    for (long long b = 0; b < nblocks; b += PART) {
        hipLaunchKernelGGL(kern, dim3((unsigned)std::min(PART, nblocks - b)), dim3(threads), 0, st,
                           (const Inst<double>*)insts, blocks + b, (const double*)fin, (const double*)forces,
                           (double*)fout, step0, args...);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int SHAPE>
static hipError_t flat_launch(const void* insts, const TileBlock* blocks, long long nblocks, const void* fin,
                              const void* forces, void* fout, const long long* step0, long long step, hipStream_t st)
{
    constexpr int TX = TILES[SHAPE][0], TY = TILES[SHAPE][1];
    auto kern = forces ? k_flat_batch<double, TX, TY, true> : k_flat_batch<double, TX, TY, false>;
    return batch_parts(kern, TX * TY, insts, blocks, nblocks, fin, forces, fout, step0, st, step);
}

hipError_t tile_batch_launch(int shape, const void* insts, const TileBlock* blocks, long long nblocks, const void* fin,
                             const void* forces, void* fout, const long long* step0, long long step, int steps,
                             hipStream_t st)
{
    if (shape == 1) return flat_launch<1>(insts, blocks, nblocks, fin, forces, fout, step0, step, st);
    if (shape == 2) return flat_launch<2>(insts, blocks, nblocks, fin, forces, fout, step0, step, st);
    if (shape == 3) return flat_launch<3>(insts, blocks, nblocks, fin, forces, fout, step0, step, st);
    auto kern = forces ? k_tile_batch<double, true> : k_tile_batch<double, false>;
    return batch_parts(kern, TILES[0][0] * TILES[0][1], insts, blocks, nblocks, fin, forces, fout, step0, st, step, steps);
}

}  // namespace dugks
