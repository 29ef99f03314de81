// Device helpers shared by the forward kernels and their reverse (adjoint)
// kernels: the D2Q9 lattice, the BGK + forcing relaxation, the pull with the
// Zou-He walls, and the staging of a capsule's fluid patch.
#pragma once

#include "lbib_internal.h"

#include <math.h>

namespace lbib {

// ------------------------------------------------------------------ lattice
// Eq. 3 velocities in the order rest, E, N, W, S, NE, NW, SW, SE.
__device__ constexpr int kEx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
__device__ constexpr int kEy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};

template <typename T>
__device__ __forceinline__ T lat_w(int i)
{
    return i == 0 ? T(4.0 / 9.0) : (i < 5 ? T(1.0 / 9.0) : T(1.0 / 36.0));
}

template <typename T>
__device__ __forceinline__ T fix_to_real(long long v)
{
    return (T)v * (T)kFixInv;
}

// First-order weights 3 w_i of the equilibrium and forcing terms.  3 w_axis is
// the rounded 1/3 and 3 w_diag is chosen as (1 - 2 * 3 w_axis) / 4, so that
// 2 (3 w_axis) + 4 (3 w_diag) = 1 exactly in binary: the first moment of the
// equilibrium then returns the momentum exactly instead of (1 + 7e-9) times it,
// a bias that would otherwise add up coherently over a channel flow in FP32.
template <typename T>
struct FirstOrderW {
    static constexpr T axis = T(1.0 / 3.0);
    static constexpr T diag = (T(1) - T(2) * axis) / T(4);
};

// Stored populations: slot i at a node of row y holds
//   f_i - w_i - (3 w_i) e_ix u_ref(y),
// the deviation from the rest weights and from the first-order term of the
// equilibrium of a reference flow along x, u_ref(y) = uref_c y (H - y)
// (H = ny - 1): the Poiseuille profile a periodic channel starts from, 0 for
// every other lattice.  In a channel the stored values are then the
// non-equilibrium and second-order parts (about 1e-4) instead of the whole
// first-order term (about 1e-2), so the FP32 rounding of every store is about
// a hundred times finer; in a steady flow each store rounds the same way at
// every step, and at the coarser scale those roundings add up to a drift of
// 1e-5 of the velocity over 2e4 steps.  (3 w_i) are the first-order weights
// above, whose moments give u_ref back exactly.
// u_ref as its two factors: it is added with one rounding (FMA).  Rounded by
// itself it would put a fixed error of 1e-9 on the velocity of every row, 2e-6 of
// the shear between rows, and twice the error on dJ/dk_s (2.6e-6 instead of 1.4e-6).
template <typename T>
struct Uref {
    T c, yy;
    __device__ __forceinline__ T plus(T x) const { return fma(c, yy, x); }
};

template <typename T>
__device__ __forceinline__ Uref<T> uref_at(const GridArgs& g, int y)
{
    return {(T)g.uref_c, (T)(y * (g.ny - 1 - y))};
}

// A population pulled from row y - e_iy to row y changes reference:
// d_i = stored_i + (3 w_i) e_ix (u_ref(y - e_iy) - u_ref(y)), nonzero for the
// four diagonals only: dm = (3 w_d)(u_ref(y - 1) - u_ref(y)) =
// (3 w_d) uref_c (2y - H - 1) and dp = (3 w_d)(u_ref(y + 1) - u_ref(y)) =
// (3 w_d) uref_c (H - 2y - 1), in the population type (the integer factors
// are exact there; the offsets are about 1e-6 and carry a rounding of 1e-13).
// Without a reference they are +0, which leaves every value unchanged; adding
// them unconditionally measured no slower than a branch around them.
template <typename T>
__device__ __forceinline__ void add_pull_offsets(const GridArgs& g, int y, T s[9])
{
    const T c3 = (T)((double)FirstOrderW<T>::diag * g.uref_c);
    const T dm = c3 * (T)(2 * y - g.ny);
    const T dp = c3 * (T)(g.ny - 2 - 2 * y);
    s[5] += dm;
    s[6] -= dm;
    s[7] -= dp;
    s[8] += dp;
}

// 1 / x by Newton steps on the hardware's estimate (one in FP32, two in FP64).
__device__ __forceinline__ float recip(float x)
{
    const float r = __builtin_amdgcn_rcpf(x);
    return fma(fma(-x, r, 1.0f), r, r);
}

__device__ __forceinline__ double recip(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

// BGK collision with the forcing term at one node (Eqs. 2, 4-7), deviation
// form.  s: the pulled populations less r = w + 3 w e.u_ref, the reference of
// the stored values (ur = u_ref at the node); om = 1 / tau.  With
//   m = sum s e + F / 2 = rho u - u_ref  (Eq. 7; taken as is in the first-order
//       term, so that rho * (m / rho) rounding does not leak into the momentum)
//   M = u_ref + m = rho u,  u = M / rho,  p F = (1 - om/2) F,
//   G = om/2 M + p F,  C = om (rho - 1) - 3 u.G,
// the populations after the collision are
//   s + [w (C + 9 (e.u)(e.G)) - om s_even] + [om (3 w e.m - s_odd) + 3 w e.pF]:
// the even bracket (s_even = half the sum with the opposite direction's) and the
// odd one (s_odd = half the difference) are shared by opposite directions, and
// (e.u)(e.G) by t_x = u_x G_x, t_y = u_y G_y and X = u_x G_y + u_y G_x.  Both
// brackets are small near equilibrium and are added to s last, so that a value
// as large as the flow's first-order term (where there is no reference flow) is
// rounded once.  About 90 operations instead of 180 with every direction on its
// own: one step is bound by memory either way, two steps in one pass
// (k_grid_two) would not be.  The rest population takes C less the other eight
// shares, so that mass is conserved whatever 1/9 rounds to.
// put(i, v) takes population i: EACH, as soon as it is known (collide_pulled), or
// else all of them last.
template <bool EACH, typename T, typename Put>
__device__ __forceinline__ void collide(const T (&s)[9], Uref<T> ur, T om, T Fx, T Fy, Put put)
{
    const T d13 = s[1] - s[3], d24 = s[2] - s[4], d57 = s[5] - s[7], d68 = s[6] - s[8];
    const T p13 = s[1] + s[3], p24 = s[2] + s[4], p57 = s[5] + s[7], p68 = s[6] + s[8];
    const T drho = ((s[0] + p13) + p24) + (p57 + p68);
    const T jx = d13 + (d57 - d68), jy = d24 + (d57 + d68);
    const T mx = fma(T(0.5), Fx, jx), my = fma(T(0.5), Fy, jy);
    const T Mx = ur.plus(mx);
    const T irho = recip(T(1) + drho);
    const T ux = Mx * irho, uy = my * irho;
    const T hom = T(0.5) * om, pre = T(1) - hom;
    const T pFx = pre * Fx, pFy = pre * Fy;
    const T Gx = fma(hom, Mx, pFx), Gy = fma(hom, my, pFy);
    const T tx = ux * Gx, ty = uy * Gy, S = tx + ty;
    const T X = fma(ux, Gy, uy * Gx);
    const T C = fma(T(-3), S, om * drho);
    const T c9 = C * T(1.0 / 9.0);
    const T q = c9 + S;
    const T w3a = FirstOrderW<T>::axis, w3d = FirstOrderW<T>::diag;
    const auto Ex = [&] { return fma(-hom, p13, tx + c9); };
    const auto Ey = [&] { return fma(-hom, p24, ty + c9); };
    const auto Ep = [&] { return fma(-hom, p57, T(0.25) * (q + X)); };
    const auto Em = [&] { return fma(-hom, p68, T(0.25) * (q - X)); };
    const auto Ox = [&] { return fma(om, fma(w3a, mx, T(-0.5) * d13), w3a * pFx); };
    const auto Oy = [&] { return fma(om, fma(w3a, my, T(-0.5) * d24), w3a * pFy); };
    const auto Op = [&] { return fma(om, fma(w3d, mx + my, T(-0.5) * d57), w3d * (pFx + pFy)); };
    const auto Om = [&] { return fma(om, fma(w3d, my - mx, T(-0.5) * d68), w3d * (pFy - pFx)); };
    const auto rest = [&] { put(0, s[0] + fma(-om, s[0], fma(T(-5), c9, C))); };
    const auto pair = [&](int i, T E, T O) {
        put(i, s[i] + (E + O));
        put(i + 2, s[i + 2] + (E - O));
    };
    if (EACH) {
        rest();
        pair(1, Ex(), Ox());
        pair(2, Ey(), Oy());
        pair(5, Ep(), Op());
        pair(6, Em(), Om());
    } else {
        const T ex = Ex(), ey = Ey(), ep = Ep(), em = Em();
        const T ox = Ox(), oy = Oy(), op = Op(), on = Om();
        rest();
        put(1, s[1] + (ex + ox));
        put(2, s[2] + (ey + oy));
        put(3, s[3] + (ex - ox));
        put(4, s[4] + (ey - oy));
        put(5, s[5] + (ep + op));
        put(6, s[6] + (em + on));
        put(7, s[7] + (ep - op));
        put(8, s[8] + (em - on));
    }
}

template <typename T>
__device__ __forceinline__ void collide(const T (&s)[9], Uref<T> ur, T om, T Fx, T Fy, T (&o)[9])
{
    collide<false>(s, ur, om, Fx, Fy, [&o](int i, T v) { o[i] = v; });
}

// Population loads of the pull.  The lines of the three directions with
// e_x = 0 (rest, north, south) are read by one wave only, so they are loaded
// as streaming (non-temporal) reads and leave the L2 to the lines of the
// x-shifted directions, which the neighbouring segment's wave reads too.
// Measured on a 4096 x 4096 pass: streaming the three e_x = 0 loads 2 % faster
// than plain loads, streaming all nine 0.5 % slower.
// Without STREAM they are plain loads: a small lattice's lines still lie in the
// L2 from the step that wrote them, and the buffer is written again in the step
// after this one (single pass, us per step, streaming -> plain: FP64 4039 x 51
// 7.55 -> 6.50, 900^2 20.1 -> 19.1, 1200^2 31.7 -> 31.5, but 4000 x 500 43.7 ->
// 51.2, 1448^2 49.4 -> 53.3; FP32 3041 x 134 6.24 -> 5.71, 1448^2 24.8 -> 23.6,
// 2048^2 50.5 -> 51.0: kPlainLoadMaxBytes lies between them).
template <typename T>
__device__ __forceinline__ T ld_stream(const T* p)
{
    return __builtin_nontemporal_load(p);
}

template <bool STREAM, typename T>
__device__ __forceinline__ T ld_pop(const T* p)
{
    return STREAM ? __builtin_nontemporal_load(p) : *p;
}

// Raw pull of the nine populations arriving at an interior node.
template <typename T>
__device__ __forceinline__ void pull_interior(const T* __restrict__ src, int x, int y,
                                              const GridArgs& g, T s[9])
{
    const size_t plane = (size_t)g.ny * g.nxp;
    const size_t r0 = (size_t)y * g.nxp, rm = (size_t)(y - 1) * g.nxp, rp = (size_t)(y + 1) * g.nxp;
    s[0] = ld_stream(&src[r0 + x]);
    s[1] = src[plane + r0 + x - 1];
    s[2] = ld_stream(&src[2 * plane + rm + x]);
    s[3] = src[3 * plane + r0 + x + 1];
    s[4] = ld_stream(&src[4 * plane + rp + x]);
    s[5] = src[5 * plane + rm + x - 1];
    s[6] = src[6 * plane + rm + x + 1];
    s[7] = src[7 * plane + rp + x + 1];
    s[8] = src[8 * plane + rp + x - 1];
}

// Open channel (Sec. 3.2): Zou-He velocity inlet at x = 0 with the parabolic
// profile u_x = 4 u_max y (H - y) / H^2, u_y = 0 (f1, f5, f8 unknown), and
// Zou-He pressure outlet at x = nx - 1 with rho = rho_out, u_y = 0 (f3, f6, f7
// unknown); no force acts on these columns.  Corners (u = 0): each unknown
// opposite a known population takes it, the two buried diagonal populations
// share the mass deficit, with the density of the inner diagonal neighbour at
// this time level.  Deviation form: the known weights sum to 1, so the
// textbook formulas keep their shape with 1 + sum(s) for sum(f).
template <typename T>
__device__ __forceinline__ void open_boundary(const T* __restrict__ src, int x, int y,
                                              const GridArgs& g, T s[9])
{
    // Every case below sets all of n1..n8 (the untouched ones to themselves),
    // so that the branches store to the same slots of s and s stays in
    // registers (stores to different slots get merged into one with a computed
    // index, which puts s in scratch memory).
    T n1 = s[1], n2 = s[2], n3 = s[3], n4 = s[4], n5 = s[5], n6 = s[6], n7 = s[7], n8 = s[8];
    const bool bot = y == 0, top = y == g.ny - 1;
    if (bot || top) {
        T h[9];
        pull_interior(src, x == 0 ? 1 : g.nx - 2, bot ? 1 : g.ny - 2, g, h);
        const T drho = ((h[0] + h[1]) + (h[2] + h[3])) + ((h[4] + h[5]) + (h[6] + h[7])) + h[8];
        if (x == 0 && bot) {
            n1 = n3;
            n2 = n4;
            n5 = n7;
            n6 = n8 = T(0.5) * (drho - (s[0] + n1 + n2 + n3 + n4 + n5 + n7));
        } else if (x == 0) {
            n1 = n3;
            n4 = n2;
            n8 = n6;
            n5 = n7 = T(0.5) * (drho - (s[0] + n1 + n2 + n3 + n4 + n6 + n8));
        } else if (bot) {
            n3 = n1;
            n2 = n4;
            n6 = n8;
            n5 = n7 = T(0.5) * (drho - (s[0] + n1 + n2 + n3 + n4 + n6 + n8));
        } else {
            n3 = n1;
            n4 = n2;
            n7 = n5;
            n6 = n8 = T(0.5) * (drho - (s[0] + n1 + n2 + n3 + n4 + n5 + n7));
        }
    } else {
        const T H = (T)(g.ny - 1);
        if (x == 0) {
            const T ux = T(4) * (T)g.u_in * (T)y * (H - (T)y) / (H * H);
            const T rho = (T(1) + s[0] + n2 + n4 + T(2) * (n3 + n6 + n7)) / (T(1) - ux);
            const T m = rho * ux;
            n1 = n3 + T(2.0 / 3.0) * m;
            n5 = n7 - T(0.5) * (n2 - n4) + m * T(1.0 / 6.0);
            n8 = n6 + T(0.5) * (n2 - n4) + m * T(1.0 / 6.0);
        } else {
            const T ro = (T)g.rho_out;
            const T uo = (T(1) + s[0] + n2 + n4 + T(2) * (n1 + n5 + n8)) / ro - T(1);
            const T m = ro * uo;
            n3 = n1 - T(2.0 / 3.0) * m;
            n7 = n5 + T(0.5) * (n2 - n4) - m * T(1.0 / 6.0);
            n6 = n8 - T(0.5) * (n2 - n4) - m * T(1.0 / 6.0);
        }
    }
    s[1] = n1;
    s[2] = n2;
    s[3] = n3;
    s[4] = n4;
    s[5] = n5;
    s[6] = n6;
    s[7] = n7;
    s[8] = n8;
}

// Pulls the nine populations arriving at (x, y) from the post-collision field
// (pull_loads: the loads and the storage reference's row change) and completes
// the wall rows with Zou-He (unknowns from the knowns, tangential momentum
// target rho_w u_w - F_x / 2) and, in an open channel, the inlet and outlet
// columns (pull_complete).  OPEN = false compiles the periodic-x lattice only
// (the hot path, and callers that never reach the end columns of an open
// channel).  The split lets the grid pass issue the nine loads before it reads
// the segment's flags, whose value the completion (F_x) depends on.
template <typename T, bool OPEN = true, bool STREAM = true>
__device__ __forceinline__ void pull_loads(const T* __restrict__ src, int x, int y,
                                           const GridArgs& g, T s[9])
{
    const size_t plane = (size_t)g.ny * g.nxp;
    int xm = x == 0 ? g.nx - 1 : x - 1;
    int xp = x == g.nx - 1 ? 0 : x + 1;
    if (OPEN && !g.periodic_x) {  // clamped: the unknown slots are replaced below
        xm = x == 0 ? 0 : xm;
        xp = x == g.nx - 1 ? x : xp;
    }
    int ym, yp;
    if (g.periodic_y) {
        ym = y == 0 ? g.ny - 1 : y - 1;
        yp = y == g.ny - 1 ? 0 : y + 1;
    } else {  // clamped: the out-of-domain slots are replaced by Zou-He below
        ym = y == 0 ? 0 : y - 1;
        yp = y == g.ny - 1 ? y : y + 1;
    }
    const size_t r0 = (size_t)y * g.nxp, rm = (size_t)ym * g.nxp, rp = (size_t)yp * g.nxp;
    s[0] = ld_pop<STREAM>(&src[r0 + x]);
    s[1] = src[plane + r0 + xm];
    s[2] = ld_pop<STREAM>(&src[2 * plane + rm + x]);
    s[3] = src[3 * plane + r0 + xp];
    s[4] = ld_pop<STREAM>(&src[4 * plane + rp + x]);
    s[5] = src[5 * plane + rm + xm];
    s[6] = src[6 * plane + rm + xp];
    s[7] = src[7 * plane + rp + xp];
    s[8] = src[8 * plane + rp + xm];
    add_pull_offsets(g, y, s);
}

template <typename T, bool OPEN = true>
__device__ __forceinline__ void pull_complete(const T* __restrict__ src, int x, int y,
                                              const GridArgs& g, T Fx, T s[9])
{
    if (OPEN && !g.periodic_x && (x == 0 || x == g.nx - 1)) {
        open_boundary(src, x, y, g, s);
        return;
    }
    if (!g.periodic_y && (y == 0 || y == g.ny - 1)) {
        // bottom row: s2, s5, s6 unknown from s4, s7, s8; top row: s4, s7, s8
        // from s2, s5, s6 (the same formulas with e_y and the sign of the
        // tangential terms mirrored).  Written with selects, so that every slot
        // of s stays a register.
        const bool top = y == g.ny - 1;
        const T a2 = top ? s[2] : s[4], a5 = top ? s[5] : s[7], a6 = top ? s[6] : s[8];
        const T rw = T(1) + s[0] + s[1] + s[3] + T(2) * (a2 + a5 + a6);
        const T mx = rw * (top ? (T)g.u_top : (T)g.u_bot) - T(0.5) * Fx;
        const T d13 = s[1] - s[3];
        const T h = top ? T(-0.5) : T(0.5);
        const T u5 = a5 - h * d13 + h * mx;  // bottom s5, top s7
        const T u6 = a6 + h * d13 - h * mx;  // bottom s6, top s8
        s[2] = top ? s[2] : a2;
        s[4] = top ? a2 : s[4];
        s[5] = top ? s[5] : u5;
        s[7] = top ? u5 : s[7];
        s[6] = top ? s[6] : u6;
        s[8] = top ? u6 : s[8];
    }
}

template <typename T, bool OPEN = true>
__device__ __forceinline__ void pull(const T* __restrict__ src, int x, int y, const GridArgs& g,
                                     T Fx, T s[9])
{
    pull_loads<T, OPEN>(src, x, y, g, s);
    pull_complete<T, OPEN>(src, x, y, g, Fx, s);
}

// One axis of an MLS fit (Eq. 9) at p on the nodes c - 1, c, c + 1: with the
// weights w_i = exp(-(X_i / 0.78)^2), X_i = c + i - 1 - p (0.78 = r_w alpha)
// and their moments S_q = sum w X^q, D = S_0 S_2 - S_1^2,
//   a = w / S_0                  the weighted mean,
//   b = w (S_2 - S_1 X) / D      the value at p of the weighted straight line,
//   s = w (S_0 X - S_1) / D      its slope.
// Offsets and weights in the population type, the fit in FP64.
struct AxisFit {
    double a[3], b[3], s[3];
};

// exp(-x), 0 <= x <= 8: FP32 by the hardware's 2^t (1 ulp) with the rounding of
// t = -x log2(e) put back to first order.
__device__ __forceinline__ float gauss(float x)
{
    const float c = -1.44269504088896341f;                          // -log2(e), rounded
    const float cl = (float)(-1.44269504088896341 - (double)c);     // and the rest
    const float t = x * c;
    const float r = fma(x, c, -t) + x * cl;
    const float e = __builtin_amdgcn_exp2f(t);
    return fma(e, r * 0.693147180559945309f, e);
}

__device__ __forceinline__ double gauss(double x) { return exp(-x); }

template <typename T>
__device__ __forceinline__ AxisFit axis_fit(T p, int c)
{
    const T inv2 = T(1.0 / (2.6 * 0.3 * 2.6 * 0.3));
    double W[3], X[3];
#pragma unroll
    for (int i = 0; i < 3; i++) {
        const T x = (T)(c + i - 1) - p;
        X[i] = (double)x;
        W[i] = (double)gauss(x * x * inv2);
    }
    const double S0 = W[0] + W[1] + W[2];
    const double V0 = W[0] * X[0], V1 = W[1] * X[1], V2 = W[2] * X[2];
    const double S1 = V0 + V1 + V2;
    const double S2 = V0 * X[0] + V1 * X[1] + V2 * X[2];
    const double D = S0 * S2 - S1 * S1;
    const double r = recip(S0 * D), i0 = r * D, iD = r * S0;
    AxisFit f;
#pragma unroll
    for (int i = 0; i < 3; i++) {
        const double w = W[i] * iD;
        f.a[i] = W[i] * i0;
        f.b[i] = w * (S2 - S1 * X[i]);
        f.s[i] = w * (S0 * X[i] - S1);
    }
    return f;
}

// Moments of the capsule's fluid patch, staged in LDS: density deviation
// rho - 1 and the force-corrected velocity.  Cells on a wall row hold NaN
// and raise ST_WALL if a support touches them.
template <typename T>
struct Patch {
    T* drho;
    T* ux;
    T* uy;
    int ox, oy, W, H;  // origin relative to the capsule reference point, size
};

template <typename T>
__device__ __forceinline__ bool patch_index(const Patch<T>& P, int cx, int cy, int k, int& idx)
{
    const int lx = cx + k % 3 - 1 - P.ox, ly = cy + k / 3 - 1 - P.oy;
    idx = ly * P.W + lx;
    return lx >= 0 && lx < P.W && ly >= 0 && ly < P.H;
}

// Moments of one patch cell from its pulled populations s (f^n) and the force
// F^{n-1} of the last collision (Eqs. 6-7, fixed-point force, g added):
// rho - 1 and the force-corrected velocity.
template <typename T>
__device__ __forceinline__ void stage_moments(const Patch<T>& P, int i, const T (&s)[9], T Fx,
                                              T Fy, Uref<T> ur)
{
    const T drho = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7])) + s[8];
    const T jx = (s[1] - s[3]) + (s[5] - s[6]) + (s[8] - s[7]);
    const T jy = (s[2] - s[4]) + (s[5] + s[6]) - (s[7] + s[8]);
    const T irho = T(1) / (T(1) + drho);
    P.drho[i] = drho;
    P.ux[i] = ur.plus(jx + T(0.5) * Fx) * irho;
    P.uy[i] = (jy + T(0.5) * Fy) * irho;
}

// Lattice coordinate ref + off on a periodic axis of n nodes.  The reference
// point (64-bit, unwrapped) is reduced once per call site with wrap_ref; each
// coordinate then takes an add and at most one correction while |off| < n.  Beyond
// that the correction is the largest n 2^k that cannot overshoot, so that any int (a
// diverged capsule's offset) is reduced in under 80 rounds, n at a time would be
// 2^31 / n.  (A remainder there took 30 registers of k_step.)
__host__ __device__ __forceinline__ int wrap_ref(long long ref, int n)
{
    // the quotient in FP64 (off by one at most for |ref| < 2^50), the remainder exact
    const long long r = ref - (long long)floor((double)ref * (1.0 / n)) * n;
    return (int)(r < 0 ? r + n : (r >= n ? r - n : r));
}

__host__ __device__ __forceinline__ int wrap_add(int base, int off, int n)
{
    int v = (int)((unsigned)base + (unsigned)off);
#pragma unroll 1
    while ((unsigned)v >= (unsigned)n) {
        const unsigned a = v < 0 ? 0u - (unsigned)v : (unsigned)v;
        const int k = __builtin_clz((unsigned)n) - __builtin_clz(a) - 1;
        const int d = n << (k > 0 ? k : 0);
        v += v < 0 ? d : -d;
    }
    return v;
}

// ---- near regions (NearRect; any ints: a diverged capsule's box can hold whatever
// the conversion of its coordinates gives)
// Rows and 64-cell segments of a capsule's near region (rect in world cells,
// x unwrapped).  The IB kernel stamps exactly these (row, segment) units into
// the near map and the near kernel computes exactly these, so near and far
// cover the lattice once.
struct RectUnits {
    int ry0, nrows;  // first row (wrapped) and row count
    int sa, nA, nsegs;  // segments: sa .. sa + nA - 1, then 0 .. (nsegs - nA) - 1
};

// The cells of the rect grown by `more` on every side: rows y0 .. y0 + rows - 1 and
// columns x0 .. x0 + w - 1, those past the lattice's end from 0 on again.
struct NearCells {
    int x0, y0, w, rows;
};

__host__ __device__ __forceinline__ int wrapped(int x, int n)
{
    const int r = x % n;
    return r < 0 ? r + n : r;
}

// Numbers a .. b, at most `most` of them.
__host__ __device__ __forceinline__ int count_of(long long a, long long b, int most)
{
    const long long n = b - a + 1;
    return n < 0 ? 0 : (n > most ? most : (int)n);
}

__host__ __device__ __forceinline__ NearCells near_cells(const NearRect& r, const GridArgs& g,
                                                         int more)
{
    NearCells c;
    c.w = count_of((long long)r.x0 - more, (long long)r.x1 + more, g.nx);
    c.x0 = wrap_add(wrapped(r.x0, g.nx), -more, g.nx);
    if (g.periodic_y) {
        c.rows = count_of((long long)r.y0 - more, (long long)r.y1 + more, g.ny);
        c.y0 = wrap_add(wrapped(r.y0, g.ny), -more, g.ny);
    } else {
        const long long a = (long long)r.y0 - more, b = (long long)r.y1 + more;
        c.y0 = a < 0 ? 0 : (a > g.ny ? g.ny : (int)a);
        c.rows = count_of(c.y0, b < g.ny ? b : g.ny - 1, g.ny);
    }
    return c;
}

__host__ __device__ __forceinline__ RectUnits rect_units(const NearRect& r, const GridArgs& g)
{
    const NearCells c = near_cells(r, g, 0);
    RectUnits u;
    u.ry0 = c.y0;
    u.nrows = c.rows;
    if (c.w >= g.nx) {
        u.sa = 0;
        u.nA = g.nseg;
        u.nsegs = g.nseg;
    } else {
        const int b = c.x0 + c.w - 1;
        u.sa = c.x0 / kSegW;
        if (b < g.nx) {
            u.nA = b / kSegW - u.sa + 1;
            u.nsegs = u.nA;
        } else {
            u.nA = g.nseg - u.sa;
            u.nsegs = u.nA + (b - g.nx) / kSegW + 1;
        }
        if (c.w == 0) u.nA = u.nsegs = 0;
    }
    return u;
}

// Raw buffer access: a scalar base and offset per row and plane, one 32-bit
// offset per lane; an offset past the end reads 0 and stores nothing, so a lane
// without a cell needs no branch (kNoCell).  Streaming loads and stores as
// ld_stream, st_stream (aux 2: non-temporal).
constexpr unsigned kNoCell = 0xffffffffu;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00027000);
}

template <int AUX, typename T>
__device__ __forceinline__ void buf_load(__amdgpu_buffer_rsrc_t r, unsigned v, unsigned s, T& out)
{
    if constexpr (sizeof(T) == 4) {
        out = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)v, (int)s, AUX));
    } else {
        out = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)v, (int)s, AUX));
    }
}

template <int AUX, typename T>
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, unsigned v, unsigned s, T x)
{
    if constexpr (sizeof(T) == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), r, (int)v, (int)s, AUX);
    } else {
        typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), r, (int)v, (int)s, AUX);
    }
}

// ---- staging of a capsule's patch
// Where a patch lies and what its cells are read from.  Staging is the
// instruction stream of one or two waves per SIMD (each issues at most one
// instruction in four cycles), so it is written for few instructions: one 32-bit
// offset addresses the nine loads of a cell (raw buffers, the neighbour and
// plane offsets in scalars), no integer division, and the force is converted only
// where it is not zero.  Cells that need another rule than "load the nine
// neighbours" (beside a periodic wrap, on a wall or an end column) are left to a
// second loop that most patches skip.
template <typename T>
struct PatchGeo {
    const T* src;          // populations of the lattice
    const long long* fib;  // its force level
    T* post;               // k_step: post-collision values, [9][cells of a band with its ring]
    int W, H, RW;          // patch size, ring width
    int by0, rows;         // k_step: first patch row and rows of the band
    int bx, by;            // lattice coordinates of the patch origin, wrapped on periodic axes
    float inv_rw, inv_w;
    T gx, om, uc, c3;      // body force, 1 / tau, storage reference (uref_at, add_pull_offsets)
    bool plain;            // every cell of the patch and its ring takes the nine plain loads
    bool far_offsets;      // the lattice is past the 32-bit offsets: no plain loads
};

// (wx, wy): lattice coordinates of the reference point (CapsuleDev).
template <typename T>
__device__ __forceinline__ void set_geo(PatchGeo<T>& Q, const Patch<T>& P, const GridArgs& g,
                                        const T* src, const long long* fib, int wx, int wy)
{
    Q.src = src;
    Q.fib = fib;
    Q.W = P.W;
    Q.H = P.H;
    Q.RW = P.W + 2;
    Q.inv_w = 1.0f / (float)P.W;
    Q.inv_rw = 1.0f / (float)Q.RW;
    Q.by0 = 0;
    Q.rows = P.H;
    Q.bx = g.periodic_x ? wrap_add(wx, P.ox, g.nx) : wx + P.ox;
    Q.by = g.periodic_y ? wrap_add(wy, P.oy, g.ny) : wy + P.oy;
    Q.gx = (T)g.gx;
    Q.om = (T)g.omega;
    Q.uc = (T)g.uref_c;
    Q.c3 = (T)((double)FirstOrderW<T>::diag * g.uref_c);
    Q.far_offsets = (unsigned long long)g.ny * (unsigned)g.nxp >= 0xfffff000u / (9 * sizeof(T)) ||
                    (unsigned long long)g.ny * (unsigned)g.nxp >= 0xfffff000u / 16;
    Q.plain = !Q.far_offsets && Q.bx >= 2 && Q.bx <= g.nx - 2 - P.W && Q.by >= 2 &&
              Q.by <= g.ny - 2 - P.H;
}

// Row i / width of item i (width = 1 / inv): exact, as (i + 1/2) / width is at
// least 1 / (2 width) from the next integer and a patch has under 2^14 cells.
__host__ __device__ __forceinline__ int row_of(int i, float inv)
{
    return (int)(((float)i + 0.5f) * inv);
}

// Lattice coordinates of patch column lx (-1 .. W) and row ly (-1 .. H); false
// if off the lattice.
template <typename T>
__device__ __forceinline__ bool patch_cell(const PatchGeo<T>& Q, const GridArgs& g, int lx, int ly,
                                           int& x, int& y)
{
    bool on = true;
    if (g.periodic_y) {
        y = wrap_add(Q.by, ly, g.ny);
    } else {
        y = Q.by + ly;
        on = y >= 0 && y < g.ny;
    }
    if (g.periodic_x) {
        x = wrap_add(Q.bx, lx, g.nx);
    } else {
        x = Q.bx + lx;
        on = on && x >= 0 && x < g.nx;
    }
    return on;
}

template <typename T>
__device__ __forceinline__ Uref<T> ref_at(const PatchGeo<T>& Q, const GridArgs& g, int y)
{
    return {Q.uc, (T)(y * (g.ny - 1 - y))};
}

template <typename T>
__device__ __forceinline__ void ref_offsets(const PatchGeo<T>& Q, const GridArgs& g, int y,
                                            T (&s)[9])
{
    const T dm = Q.c3 * (T)(2 * y - g.ny);
    const T dp = Q.c3 * (T)(g.ny - 2 - 2 * y);
    s[5] += dm;
    s[6] -= dm;
    s[7] -= dp;
    s[8] += dp;
}

// Collides ring cell i (ring column lx, band row ly) at lattice row y from its
// pulled populations and keeps the result; a patch cell's force is left in its
// (ux, uy) slots for the moments.
template <typename T>
__device__ __forceinline__ void collide_ring_cell(const PatchGeo<T>& Q, const GridArgs& g,
                                                  const Patch<T>& P, int i, int lx, int ly, int y,
                                                  const T (&s)[9], T Fx, T Fy)
{
    T o[9];
    collide(s, ref_at(Q, g, y), Q.om, Fx, Fy, o);
    const int nring = Q.RW * (Q.rows + 2);
    T* p = Q.post + i;
#pragma unroll
    for (int q = 0; q < 9; q++) p[q * nring] = o[q];
    if (lx >= 1 && lx <= Q.W && ly >= 1 && ly <= Q.rows) {
        const int pi = (Q.by0 + ly - 1) * Q.W + lx - 1;
        P.ux[pi] = Fx;
        P.uy[pi] = Fy;
    }
}

// Positions 0 .. count - 1 of an axis from lattice coordinate o on whose coordinate is
// on an end of it (0, size - 1) or off the lattice: s0 .. s0 + n0 - 1 and s1 .. s1 + n1 - 1.
// A periodic axis wraps, with 0 <= o < size and count <= size.
struct AxisEnds {
    int n0, s1, n1;  // s0 = 0
    __host__ __device__ __forceinline__ int count() const { return n0 + n1; }
};

__host__ __device__ __forceinline__ AxisEnds axis_ends(int o, int count, int size, int periodic)
{
    AxisEnds e;
    const int a = 1 - o, b = size - 1 - o, c = size + 1 - o;
    e.n0 = periodic ? (o == 0 ? 1 : 0) : (a < 0 ? 0 : (a > count ? count : a));
    e.s1 = b < e.n0 ? e.n0 : (b > count ? count : b);
    e.n1 = (periodic && c < count ? c : count) - e.s1;
    return e;
}

// The cells of a box (w columns from lattice coordinate x on, h rows from y on) that
// need another rule than the nine plain loads, one after the other (those at a corner
// twice): its rows and then its columns at the lattice's ends, so that a block takes
// them in one round (the whole box, a row of it at a time, took a memory latency in
// every round).  A box that wraps onto itself, or one without plain loads: all cells.
struct OtherCells {
    AxisEnds cols, rows;
    int w, h, n, in_rows;
    float inv_w, inv_h;
    __host__ __device__ __forceinline__ OtherCells(const GridArgs& g, bool all, int x, int y, int w_, int h_)
    {
        w = w_;
        h = h_;
        inv_w = 1.0f / (float)w;
        inv_h = 1.0f / (float)h;
        all = all || (g.periodic_x && w > g.nx) || (g.periodic_y && h > g.ny);
        cols = axis_ends(g.periodic_x ? wrap_add(x, 0, g.nx) : x, w, g.nx, g.periodic_x);
        rows = axis_ends(g.periodic_y ? wrap_add(y, 0, g.ny) : y, h, g.ny, g.periodic_y);
        if (all) {
            rows.n0 = h;
            rows.n1 = cols.n0 = cols.n1 = 0;
        }
        in_rows = rows.count() * w;
        n = in_rows + cols.count() * h;
    }
    __host__ __device__ __forceinline__ void cell(int i, int& lx, int& ly) const
    {
        const bool r = i < in_rows;  // (selects: both halves stay in registers)
        const int q = r ? i : i - in_rows, k = row_of(q, r ? inv_w : inv_h);
        const int n0 = r ? rows.n0 : cols.n0, s1 = r ? rows.s1 : cols.s1;
        const int line = k < n0 ? k : s1 + k - n0, along = q - k * (r ? w : h);
        lx = r ? along : line;
        ly = r ? line : along;
    }
};

// Whether the nine sources of a cell are its plain neighbours.
__host__ __device__ __forceinline__ bool plain_cell(const GridArgs& g, int x, int y)
{
    return (unsigned)(x - 1) < (unsigned)(g.nx - 2) && (unsigned)(y - 1) < (unsigned)(g.ny - 2);
}

// The nine plain loads of lattice cell `cell` (kNoCell: none) and its force.
template <typename T>
struct PlainLoads {
    __amdgpu_buffer_rsrc_t in, ff;
    unsigned row, plane;
    __device__ __forceinline__ PlainLoads(const PatchGeo<T>& Q, const GridArgs& g)
    {
        row = (unsigned)g.nxp * sizeof(T);
        plane = (unsigned)g.ny * row;
        in = buffer_of(Q.src, 9 * plane);
        ff = buffer_of(Q.fib, 16u * (unsigned)g.ny * (unsigned)g.nxp);
    }
    __device__ __forceinline__ void operator()(unsigned cell, bool on, T (&s)[9], long long& fx,
                                               long long& fy) const
    {
        const unsigned v = on ? cell * (unsigned)sizeof(T) : kNoCell;
        buf_load<0>(in, v, 0, s[0]);
        buf_load<0>(in, v, plane - sizeof(T), s[1]);
        buf_load<0>(in, v, 2 * plane - row, s[2]);
        buf_load<0>(in, v, 3 * plane + sizeof(T), s[3]);
        buf_load<0>(in, v, 4 * plane + row, s[4]);
        buf_load<0>(in, v, 5 * plane - row - sizeof(T), s[5]);
        buf_load<0>(in, v, 6 * plane - row + sizeof(T), s[6]);
        buf_load<0>(in, v, 7 * plane + row + sizeof(T), s[7]);
        buf_load<0>(in, v, 8 * plane + row - sizeof(T), s[8]);
        const unsigned vf = on ? cell * 16u : kNoCell;
        buf_load<0>(ff, vf, 0, fx);
        buf_load<0>(ff, vf, 8, fy);
    }
};

// Whether the patch cell (x, y) carries moments (not on a wall or an end column).
__device__ __forceinline__ bool has_moments(const GridArgs& g, int x, int y)
{
    return (g.periodic_y || (unsigned)(y - 1) < (unsigned)(g.ny - 2)) &&
           (g.periodic_x || (unsigned)(x - 1) < (unsigned)(g.nx - 2));
}

// Total force of a cell from its level's values.
template <typename T>
__device__ __forceinline__ void cell_force(T gx, long long fx, long long fy, T& Fx, T& Fy)
{
    Fx = gx;
    Fy = T(0);
    if ((fx | fy) != 0) {
        Fx += fix_to_real<T>(fx);
        Fy += fix_to_real<T>(fy);
    }
}

// The plain patch cells among first, first + stride, ... (K of them, below
// `end`): loads of all in flight together, then their moments.
template <typename T, int K>
__device__ __forceinline__ void stage_cells(const PatchGeo<T>& Q, const GridArgs& g,
                                            const Patch<T>& P, int first, int stride, int end)
{
    const PlainLoads<T> load(Q, g);
    T s[K][9];
    long long fx[K], fy[K];
    int ys[K];
    bool on[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        const int i = first + k * stride;
        const int ly = row_of(i, Q.inv_w), lx = i - ly * Q.W;
        int x, y;
        on[k] = patch_cell(Q, g, lx, ly, x, y) && i < end && plain_cell(g, x, y) && !Q.far_offsets;
        ys[k] = y;
        load((unsigned)y * (unsigned)g.nxp + (unsigned)x, on[k], s[k], fx[k], fy[k]);
    }
#pragma unroll
    for (int k = 0; k < K; k++) {
        if (!on[k]) continue;
        T Fx, Fy;
        cell_force(Q.gx, fx[k], fy[k], Fx, Fy);
        ref_offsets(Q, g, ys[k], s[k]);
        stage_moments(P, first + k * stride, s[k], Fx, Fy, ref_at(Q, g, ys[k]));
    }
}

// The other patch cells: NaN on a wall row or an end column, else pulled with
// the wrap.
template <typename T>
__device__ void stage_other_cells(const PatchGeo<T>& Q, const GridArgs& g, const Patch<T>& P)
{
    if (Q.plain) return;
    const OtherCells others(g, Q.far_offsets, Q.bx, Q.by, Q.W, Q.H);
    for (int j = threadIdx.x; j < others.n; j += blockDim.x) {
        int lx, ly, x, y;
        others.cell(j, lx, ly);
        const int i = ly * Q.W + lx;
        if (!patch_cell(Q, g, lx, ly, x, y) || !has_moments(g, x, y)) {
            P.drho[i] = P.ux[i] = P.uy[i] = T(NAN);
            continue;
        }
        if (plain_cell(g, x, y) && !Q.far_offsets) continue;
        T s[9], Fx, Fy;
        pull_loads<T, true, false>(Q.src, x, y, g, s);
        const longlong2 f = *reinterpret_cast<const longlong2*>(Q.fib + 2 * ((size_t)y * g.nxp + x));
        cell_force(Q.gx, f.x, f.y, Fx, Fy);
        stage_moments(P, i, s, Fx, Fy, ref_at(Q, g, y));
    }
}

// ---- the patch's own grid step (k_step)
// The patch moments of time n + 1 from the populations P^n and the force F^n of
// the collision in between: the post-collision values of the patch and a ring
// of one cell, computed here as the grid pass of the same launch computes them
// (the same functions, so the same bits), go to LDS, and the patch cells pull
// from there.  Patch rows are taken in bands that fit the LDS left.

// The plain ring cells among first, first + stride, ... (K of them, below `end`)
// of the band: loads of all in flight together, then collide.
template <typename T, int K>
__device__ __forceinline__ void step_cells(const PatchGeo<T>& Q, const GridArgs& g,
                                           const Patch<T>& P, int first, int stride, int end)
{
    const PlainLoads<T> load(Q, g);
    T s[K][9];
    long long fx[K], fy[K];
    int lxs[K], lys[K], ys[K];
    bool on[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        const int i = first + k * stride;
        lys[k] = row_of(i, Q.inv_rw);
        lxs[k] = i - lys[k] * Q.RW;
        int x, y;
        on[k] = patch_cell(Q, g, lxs[k] - 1, Q.by0 + lys[k] - 1, x, y) && i < end &&
                plain_cell(g, x, y);
        ys[k] = y;
        load((unsigned)y * (unsigned)g.nxp + (unsigned)x, on[k], s[k], fx[k], fy[k]);
    }
#pragma unroll
    for (int k = 0; k < K; k++) {
        if (!on[k]) continue;
        T Fx, Fy;
        cell_force(Q.gx, fx[k], fy[k], Fx, Fy);
        ref_offsets(Q, g, ys[k], s[k]);
        collide_ring_cell(Q, g, P, first + k * stride, lxs[k], lys[k], ys[k], s[k], Fx, Fy);
    }
}

// The band's other ring cells.
template <typename T>
__device__ void step_other_cells(const PatchGeo<T>& Q, const GridArgs& g, const Patch<T>& P)
{
    // (likely: otherwise the compiler spills scalars of the plain path for this one, 5 %
    // of an FP64 Kinematic step)
    if (__builtin_expect(Q.plain, 1)) return;
    const OtherCells others(g, false, Q.bx - 1, Q.by + Q.by0 - 1, Q.RW, Q.rows + 2);
    for (int j = threadIdx.x; j < others.n; j += blockDim.x) {
        int lx, ly, x, y;
        others.cell(j, lx, ly);
        const int i = ly * Q.RW + lx;
        if (!patch_cell(Q, g, lx - 1, Q.by0 + ly - 1, x, y) || plain_cell(g, x, y)) continue;
        const longlong2 f = *reinterpret_cast<const longlong2*>(Q.fib + 2 * ((size_t)y * g.nxp + x));
        T s[9], Fx, Fy;
        cell_force(Q.gx, f.x, f.y, Fx, Fy);
        pull<T, true>(Q.src, x, y, g, Fx, s);
        collide_ring_cell(Q, g, P, i, lx, ly, y, s, Fx, Fy);
    }
}

// Moments of the band's patch cells from their neighbours' post-collision
// values in LDS.
template <typename T>
__device__ __forceinline__ void step_moments(const PatchGeo<T>& Q, const GridArgs& g,
                                             const Patch<T>& P)
{
    constexpr int K = 2;
    const int nring = Q.RW * (Q.rows + 2), n = Q.W * Q.rows, nt = blockDim.x;
    for (int i0 = threadIdx.x; i0 < n; i0 += K * nt) {
        T s[K][9], Fx[K], Fy[K];
        int ys[K], state[K];  // 0: past the band, 1: no moments, 2: moments
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int i = i0 + k * nt < n ? i0 + k * nt : i0;
            const int ly = row_of(i, Q.inv_w), lx = i - ly * Q.W;
            int x, y;
            const bool on = patch_cell(Q, g, lx, Q.by0 + ly, x, y) && has_moments(g, x, y);
            state[k] = i0 + k * nt < n ? (on ? 2 : 1) : 0;
            ys[k] = y;
            const T* c = Q.post + (ly + 1) * Q.RW + lx + 1;
#pragma unroll
            for (int q = 0; q < 9; q++) s[k][q] = c[q * nring - kEy[q] * Q.RW - kEx[q]];
            Fx[k] = P.ux[Q.by0 * Q.W + i];
            Fy[k] = P.uy[Q.by0 * Q.W + i];
        }
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int pi = Q.by0 * Q.W + i0 + k * nt;
            if (state[k] == 2) {
                ref_offsets(Q, g, ys[k], s[k]);
                stage_moments(P, pi, s[k], Fx[k], Fy[k], ref_at(Q, g, ys[k]));
            } else if (state[k] == 1) {
                P.drho[pi] = P.ux[pi] = P.uy[pi] = T(NAN);
            }
        }
    }
}

// A patch so wide that no row of it fits beside its moments (or a lattice past
// the 32-bit offsets): every cell computes its nine neighbours' collisions.
template <typename T>
__device__ void step_cells_direct(const PatchGeo<T>& Q, const GridArgs& g, const Patch<T>& P)
{
    for (int pi = threadIdx.x; pi < Q.W * Q.H; pi += blockDim.x) {
        const int py = row_of(pi, Q.inv_w), px = pi - py * Q.W;
        int x, y;
        if (!patch_cell(Q, g, px, py, x, y) || !has_moments(g, x, y)) {
            P.drho[pi] = P.ux[pi] = P.uy[pi] = T(NAN);
            continue;
        }
        T s[9] = {}, Fx0 = 0, Fy0 = 0;
#pragma unroll 1
        for (int q = 0; q < 9; q++) {
            const int ex = q == 0 ? 0 : (q < 5 ? (q & 1 ? 2 - q : 0) : (q == 5 || q == 8 ? 1 : -1));
            const int ey = q == 0 ? 0 : (q < 5 ? (q & 1 ? 0 : 3 - q) : (q < 7 ? 1 : -1));
            int xn, yn;
            patch_cell(Q, g, px - ex, py - ey, xn, yn);
            const longlong2 f =
                *reinterpret_cast<const longlong2*>(Q.fib + 2 * ((size_t)yn * g.nxp + xn));
            T t[9], o[9], Fx, Fy;
            cell_force(Q.gx, f.x, f.y, Fx, Fy);
            pull<T, true>(Q.src, xn, yn, g, Fx, t);
            collide(t, ref_at(Q, g, yn), Q.om, Fx, Fy, o);
            Fx0 = q == 0 ? Fx : Fx0;
            Fy0 = q == 0 ? Fy : Fy0;
#pragma unroll
            for (int i = 0; i < 9; i++) s[i] = i == q ? o[i] : s[i];
        }
        ref_offsets(Q, g, y, s);
        stage_moments(P, pi, s, Fx0, Fy0, ref_at(Q, g, y));
    }
}

// Wave-wide reductions with DPP lane moves (register to register, no LDS
// round trip): exchange within lane pairs and quads (quad_perm), mirror within
// half-rows and rows of 16, then the row broadcasts of lanes 15 and 31 carry
// the row results into the last row.  Lane 63 ends with the result, which is
// broadcast from there; the combination order is fixed by the lane pattern.
// Call with the whole wave active.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_move(int old, int v)
{
    return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xf, false);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move_f64(double v)  // rows outside ROWS read 0
{
    const long long b = __double_as_longlong(v);
    const int lo = dpp_move<CTRL, ROWS>(0, (int)(unsigned int)(b & 0xffffffffLL));
    const int hi = dpp_move<CTRL, ROWS>(0, (int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned int)lo);
}

__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_move_f64<0xB1, 0xF>(v);   // quad_perm [1, 0, 3, 2]
    v += dpp_move_f64<0x4E, 0xF>(v);   // quad_perm [2, 3, 0, 1]
    v += dpp_move_f64<0x141, 0xF>(v);  // row_half_mirror
    v += dpp_move_f64<0x140, 0xF>(v);  // row_mirror
    v += dpp_move_f64<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_move_f64<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(unsigned int)(b & 0xffffffffLL), 63);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned int)lo);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_move_f32(float v)  // rows outside ROWS keep v
{
    return __int_as_float(dpp_move<CTRL, ROWS>(__float_as_int(v), __float_as_int(v)));
}

template <bool MAX>
__device__ __forceinline__ float wave_extreme(float v)
{
#define LBIB_STEP(C, R)                         \
    {                                           \
        const float o = dpp_move_f32<C, R>(v);  \
        v = MAX ? fmaxf(v, o) : fminf(v, o);    \
    }
    LBIB_STEP(0xB1, 0xF)
    LBIB_STEP(0x4E, 0xF)
    LBIB_STEP(0x141, 0xF)
    LBIB_STEP(0x140, 0xF)
    LBIB_STEP(0x142, 0xA)
    LBIB_STEP(0x143, 0xC)
#undef LBIB_STEP
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Deterministic block reductions over the wavefronts of a block (at most
// kIBThreads / 64): a DPP reduction within each wave, then the wave partials in
// order.

// Lane l of every wave holds partial l % 8 of group l / 8 (value k of wave w at
// l = 8 k + w): the combination within groups of eight lanes.
template <typename F>
__device__ __forceinline__ double combine8(double v, F&& op)
{
    v = op(v, dpp_move_f64<0xB1, 0xF>(v));   // quad_perm [1, 0, 3, 2]
    v = op(v, dpp_move_f64<0x4E, 0xF>(v));   // quad_perm [2, 3, 0, 1]
    return op(v, dpp_move_f64<0x141, 0xF>(v));  // row_half_mirror
}

__device__ __forceinline__ double lane_value(double v, int lane)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(unsigned int)(b & 0xffffffffLL), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned int)lo);
}

template <int N>
__device__ __forceinline__ void block_sum(double (&v)[N], double (*red)[8])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < N; k++) v[k] = wave_sum(v[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < N; k++) red[wave][k] = v[k];
    __syncthreads();
    const bool has = (lane & 7) < (int)(blockDim.x >> 6);
    const double t = combine8(has ? red[lane & 7][lane >> 3] : 0.0,
                              [](double a, double b) { return a + b; });
#pragma unroll
    for (int k = 0; k < N; k++) v[k] = lane_value(t, 8 * k);
    __syncthreads();
}

// Minima and maxima of two coordinates: the maxima go through as minima of the
// negated values.
__device__ __forceinline__ void block_minmax(float (&mn)[2], float (&mx)[2], double (*red)[8],
                                             bool closing_barrier = true)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float* r = reinterpret_cast<float*>(red);  // [wave][16], four used
    float m[4] = {mn[0], mn[1], -mx[0], -mx[1]};
#pragma unroll
    for (int k = 0; k < 4; k++) m[k] = wave_extreme<false>(m[k]);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < 4; k++) r[16 * wave + k] = m[k];
    }
    __syncthreads();
    const bool has = (lane & 7) < (int)(blockDim.x >> 6);
    float t = has ? r[16 * (lane & 7) + ((lane >> 3) & 3)] : 3e38f;
    t = fminf(t, dpp_move_f32<0xB1, 0xF>(t));
    t = fminf(t, dpp_move_f32<0x4E, 0xF>(t));
    t = fminf(t, dpp_move_f32<0x141, 0xF>(t));
    auto at = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), l)); };
    mn[0] = at(0);
    mn[1] = at(8);
    mx[0] = -at(16);
    mx[1] = -at(24);
    if (closing_barrier) __syncthreads();
}

}  // namespace lbib
