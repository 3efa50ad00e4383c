// Device code shared by the HIP kernels (gfx950) of the batched D2Q9 BGK ensemble and its
// statistics: OpenLB-UQ (arXiv 2508.13867), Sec. "Lattice Boltzmann
// methods" (Eqs. deterministicLBE, bgkCollision, equilibrium, the D2Q9 set
// and weights, the collide/stream split) and Sec. "Uncertainty
// quantification methods" (Eqs. meanMCS, varMCS, coef_discrete, gpc_mean,
// gpc_std).
//
// Storage: shifted populations f~_i = f_i - w_i in slabs [S][9][ny][pitch]
// (x fastest, pitch a multiple of 64 elements). Two layouts:
//
// AA (one slab, in place; Bailey et al. 2009):
//   even step t: node x reads its own slots i, collides, and writes f*_i to
//                its own slot opp(i);
//   odd step t:  node x reads f_i(x,t) = f*_i(x - c_i, t-1) from slot opp(i)
//                of node x - c_i, collides, and writes f*_i to slot i of
//                node x + c_i, leaving the natural layout for step t+1.
//   Each node reads and writes exactly the same nine locations in either
//   parity, so one launch per step needs no second lattice and no barrier.
//
// AB (two slabs, pull): slab t&1 holds g_i(x) = f*_i(x, t-1), the
//   post-collision populations of the previous step; step t reads
//   f_i(x,t) = g_i(x - c_i) (bounce-back: g_opp(i)(x)), collides and writes
//   f*_i(x,t) to slot i of node x in the other slab: every store is aligned
//   and can bypass the caches. Twice the memory of AA; on MI355X a
//   two-buffer stream reaches a higher HBM rate than an in-place one.
//
// Direction order i = 0..8: (0,0), (1,0), (0,1), (-1,0), (0,-1), (1,1),
// (-1,1), (-1,-1), (1,-1); opposite pairs (1,3), (2,4), (5,7), (6,8).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "uq_internal.h"

// Every fused multiply-add in these kernels is written out (fma_c). Implicit
// contraction is off so that the compiler cannot fuse the last fma of the
// collision with the conversion to a 16-bit storage format (one rounding
// where the storage model has two), which it would do in some kernels and
// not in others: with it off, every kernel rounds the same operations the
// same way and their results agree bit for bit in every format.
#pragma clang fp contract(off)

namespace uqi {

// ------------------------------------------------------------------ storage types
template <int P>
struct Prec;

template <>
struct Prec<UQ_FP64> {
    using T = double;
    using C = double;
    __device__ static inline C ld(const T *p, float) { return *p; }
    __device__ static inline void st(T *p, C v, float) { *p = v; }
    __device__ static inline void st_nt(T *p, C v, float) { __builtin_nontemporal_store(v, p); }
    // the value a store and a reload would give back
    __device__ static inline C rt(C v, float, float) { return v; }
};
template <>
struct Prec<UQ_FP32> {
    using T = float;
    using C = float;
    __device__ static inline C ld(const T *p, float) { return *p; }
    __device__ static inline void st(T *p, C v, float) { *p = v; }
    __device__ static inline void st_nt(T *p, C v, float) { __builtin_nontemporal_store(v, p); }
    __device__ static inline C rt(C v, float, float) { return v; }
};
template <>
struct Prec<UQ_FP16S> {
    using T = _Float16;
    using C = float;
    // stored value = f~ * 2^s (power-of-two scale, exact); rounding to half is
    // round-to-nearest-even (v_cvt_f16_f32 in the default mode). Back to
    // float as h * 2^-s + 0: one mixed-precision fma (v_fma_mix_f32) where a
    // product would take a conversion and a multiply; the same value, except
    // that -0 comes back as +0.
    __device__ static inline C up(_Float16 h, float inv) { return __builtin_fmaf((float)h, inv, 0.0f); }
    __device__ static inline C ld(const T *p, float inv) { return up(*p, inv); }
    __device__ static inline void st(T *p, C v, float sc) { *p = (_Float16)(v * sc); }
    __device__ static inline void st_nt(T *p, C v, float sc) { __builtin_nontemporal_store((_Float16)(v * sc), p); }
    __device__ static inline C rt(C v, float sc, float inv) { return up((_Float16)(v * sc), inv); }
};
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
template <>
struct Prec<UQ_BF16S> {
    // bfloat16 has float's exponent range: stored unscaled (the job's scale
    // exponent is 0 and sc, inv are not used)
    using T = uint16_t;
    using C = float;
    __device__ static inline C ld(const T *p, float) { return __uint_as_float((uint32_t)(*p) << 16); }
    // round to nearest, ties to even (the conversion instruction of gfx950)
    __device__ static inline uint16_t rne(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }
    __device__ static inline void st(T *p, C v, float) { *p = rne(v); }
    __device__ static inline void st_nt(T *p, C v, float) { __builtin_nontemporal_store(rne(v), p); }
    // the rounded value in the upper half of a word whose lower half is +0:
    // that word is the float itself, from one conversion instruction
    __device__ static inline C rt(C v, float, float) {
        return __builtin_bit_cast(float, __builtin_convertvector((f32x2_t){0.0f, v}, bf16x2_t));
    }
};

// ------------------------------------------------------------------ lattice
__device__ constexpr int CXd[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
__device__ constexpr int CYd[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
__device__ constexpr int OPPd[9] = {0, 3, 4, 1, 2, 7, 8, 5, 6};
// index of a direction among the three that share its c_y
__device__ constexpr int GJd[9] = {0, 1, 0, 2, 0, 1, 2, 1, 2};

template <typename C>
__device__ inline C wgt(int i) {
    return i == 0 ? C(4) / C(9) : (i < 5 ? C(1) / C(9) : C(1) / C(36));
}

// BGK relaxation of shifted populations toward the second-order equilibrium
// (Eqs. bgkCollision, equilibrium with c_s^2 = 1/3). With j = rho u, the
// equilibrium minus the weight is
//   f_eq,i - w_i = w_i (drho - 3/2 j.u + 9/2 (c_i.j)(c_i.u)) + 3 w_i (c_i.j),
// which equals the textbook form in exact arithmetic. It is evaluated this way
// so that single-precision rounding does not bias the flow:
//  - the first-order term uses j itself, not rho * (j / rho);
//  - the first-order term omega 3 w_i (c_i.j) is one rounded product per
//    direction pair, a1 (c_i.j) on the axes and a2 (c_i.j) on the diagonals,
//    with coefficients whose momentum sum 2 a1 + 4 a2 is omega exactly, so
//    that the collision conserves momentum to rounding. In double precision
//    a1 = omega/3 is carried as a two-term split (hi + lo, one fused
//    multiply-add per term) and a2 = a1/4. In single precision a1 =
//    fl(omega fl(1/3)) and a2 = (omega - 2 a1)/4, whose subtraction is exact
//    (Sterbenz: omega and 2 a1 are within a factor of two), one multiply per
//    term; a2 then differs from omega/12 by O(1e-7), which touches only a
//    third moment of the equilibrium (Q_xyy), not mass, momentum or stress.
//    Multiplying both by a rounded omega/3 instead scales these terms by a
//    fixed 1 + O(1e-8) every step: the collision then does not conserve
//    momentum, and in single precision the decay of the kinetic energy
//    drifts by ~1e-5..1e-4 over a few thousand steps (measured), against
//    ~1e-7 in this form.
// Returns rho - 1 and u.
template <typename C>
struct Third;
template <>
struct Third<float> {
    static constexpr float hi = 0x1.555556p-2f, lo = -0x1.555556p-27f;  // hi + lo = 1/3 to ~2^-48
};
template <>
struct Third<double> {
    static constexpr double hi = 0x1.5555555555555p-2, lo = 0x1.5555555555555p-56;
};
__device__ inline float fma_c(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fma_c(double a, double b, double c) { return __builtin_fma(a, b, c); }
// 1/x from the hardware reciprocal estimate refined by Newton steps (one in
// single, two in double precision): within an ulp of the quotient, a third of
// the instructions of the IEEE division sequence
__device__ inline float recip(float x) {
    const float r = __builtin_amdgcn_rcpf(x);
    return __builtin_fmaf(r, __builtin_fmaf(-x, r, 1.0f), r);
}
__device__ inline double recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
    return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

// 1/(1 + drho) inside the collision. The velocity it gives enters only the
// second-order terms of the equilibrium (the first-order term uses j), so
// in single precision the hardware estimate (within an ulp) is used as it
// is; double precision refines it to full accuracy.
__device__ inline float coll_recip(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline double coll_recip(double x) { return recip(x); }

template <typename C>
__device__ inline void bgk(C f[9], C omega, C &drho_o, C &ux_o, C &uy_o) {
    // moments from the sums of the c_y = +1 and c_y = -1 populations (j_y is
    // their difference), with the c_y = -1 terms last: the fused kernels
    // read the others a row ahead, so most of this runs while those loads
    // are in flight
    const C cs = f[2] + (f[5] + f[6]), as = f[4] + (f[7] + f[8]);
    const C drho = ((f[0] + (f[1] + f[3])) + cs) + as;
    const C jx = ((f[1] - f[3]) + (f[5] - f[6])) + (f[8] - f[7]);
    const C jy = cs - as;
    const C ir = coll_recip(C(1) + drho);
    const C ux = jx * ir, uy = jy * ir;
    // second-order terms from the products j_x u_x, j_y u_y and j_x u_y
    // (= j_y u_x): (c.j)(c.u) is j_x u_x or j_y u_y on the axes and
    // j_x u_x + j_y u_y +- 2 j_x u_y on the diagonals
    const C px = jx * ux, py = jy * uy, pp = px + py;
    const C db = fma_c(C(-1.5), pp, drho);
    // omega folded into the constants (per sample: the compiler hoists them
    // out of the node loops): omega w_i, and omega / 3 as an unevaluated sum
    // hi + lo (exact product of omega with the split of 1/3, rounded once to
    // the pair; unused in single precision), so that the first-order term is
    // still formed with a single rounding. Every multiply-add is an explicit
    // fma.
    const C ow0 = omega * (C(4) / C(9)), ow1 = omega * (C(1) / C(9)), ow2 = omega * (C(1) / C(36));
    const C o3h = omega * Third<C>::hi;
    const C o3l = fma_c(omega, Third<C>::lo, fma_c(omega, Third<C>::hi, -o3h));
    // diagonal coefficient: in single precision the exact remainder of omega
    // after the two axis terms, so that 2 o3h + 4 o12h = omega
    const C o12h = std::is_same<C, float>::value ? (omega - C(2) * o3h) * C(0.25) : o3h * C(0.25);
    const C o12l = o3l * C(0.25);
    // the first-order term, rounded once (single precision: one multiply)
    auto first = [&](C cj, C h, C l) -> C {
        if constexpr (std::is_same<C, float>::value) return cj * h;
        else return fma_c(cj, h, cj * l);
    };
    const C om1 = C(1) - omega;
    f[0] = fma_c(om1, f[0], ow0 * db);
    {
        const C q = fma_c(C(4.5), px, db), l = first(jx, o3h, o3l);
        f[1] = fma_c(om1, f[1], fma_c(q, ow1, l));
        f[3] = fma_c(om1, f[3], fma_c(q, ow1, -l));
    }
    {
        const C q = fma_c(C(4.5), py, db), l = first(jy, o3h, o3l);
        f[2] = fma_c(om1, f[2], fma_c(q, ow1, l));
        f[4] = fma_c(om1, f[4], fma_c(q, ow1, -l));
    }
    const C t = fma_c(C(4.5), pp, db), jx9 = C(9) * jx;
    {
        const C cj = jx + jy;
        const C q = fma_c(jx9, uy, t), l = first(cj, o12h, o12l);
        f[5] = fma_c(om1, f[5], fma_c(q, ow2, l));
        f[7] = fma_c(om1, f[7], fma_c(q, ow2, -l));
    }
    {
        const C cj = jy - jx;
        const C q = fma_c(-jx9, uy, t), l = first(cj, o12h, o12l);
        f[6] = fma_c(om1, f[6], fma_c(q, ow2, l));
        f[8] = fma_c(om1, f[8], fma_c(q, ow2, -l));
    }
    drho_o = drho;
    ux_o = ux;
    uy_o = uy;
}

// moments only
template <typename C>
__device__ inline void moments(const C f[9], C &drho, C &ux, C &uy) {
    drho = ((f[0] + (f[1] + f[3])) + (f[2] + f[4])) + ((f[5] + f[7]) + (f[6] + f[8]));
    const C jx = ((f[1] - f[3]) + (f[5] - f[7])) + (f[8] - f[6]);
    const C jy = ((f[2] - f[4]) + (f[5] - f[7])) + (f[6] - f[8]);
    const C ir = recip(C(1) + drho);
    ux = jx * ir;
    uy = jy * ir;
}

// inflow ramp s(t) = sin^2(pi t / (2 T_r)) for t < T_r, else 1
__device__ inline double ramp_factor(int64_t t, double T) {
    if (T <= 0.0 || (double)t >= T) return 1.0;
    double s = sin(M_PI * (double)t / (2.0 * T));
    return s * s;
}

// inflow profile u_x at row y, time t: s(t) 4 u_peak (y+1/2)(H-y-1/2)/H^2,
// from a = s(t) 4 u_peak
__device__ inline double inflow_u_a(double a, int ny, int y) {
    // 1/H^2 depends on the lattice only: the compiler hoists its division
    // out of the row loops, leaving three multiplies per row
    const double H = (double)ny, yy = (double)y + 0.5, inv_h2 = 1.0 / (H * H);
    return a * yy * (H - yy) * inv_h2;
}
__device__ inline double inflow_u(int ny, double ramp, int y, int64_t t, double u_peak) {
    return inflow_u_a(ramp_factor(t, ramp) * 4.0 * u_peak, ny, y);
}

// Zou-He (1997) completion of the unknown populations on the open columns,
// written for shifted populations (the weights cancel in every relation):
// the inlet with the imposed velocity u, the outlet at rho = 1.
// (explicit fmas, as in the collision: the same result in every kernel)
// The outlet's relations are the inlet's mirrored, with -v = -(1 - rho u) for
// rho u, so one side's arithmetic serves both and only its arguments are
// selected: two branches that store to different populations made the compiler
// keep a fused kernel's populations in LDS (2 us per row step).
template <typename C>
__device__ inline void zou_he_u(C f[9], bool inlet, C u) {
    const C h = C(0.5) * (f[2] - f[4]), hs = inlet ? -h : h;
    const C a = inlet ? f[3] : f[1], b = inlet ? f[6] : f[5], c = inlet ? f[7] : f[8];
    const C S = fma_c(C(2), (a + b) + c, (f[0] + f[2]) + f[4]);
    const C drho = (S + u) / (C(1) - u);
    const C r = inlet ? (C(1) + drho) * u : -S;
    const C n1 = fma_c(C(2) / C(3), r, a);
    const C n2 = fma_c(C(1) / C(6), r, (inlet ? c : b) + hs);
    const C n3 = fma_c(C(1) / C(6), r, (inlet ? b : c) - hs);
    f[1] = inlet ? n1 : f[1];
    f[3] = inlet ? f[3] : n1;
    f[5] = inlet ? n2 : f[5];
    f[7] = inlet ? f[7] : n2;
    f[8] = inlet ? n3 : f[8];
    f[6] = inlet ? f[6] : n3;
}

template <typename C>
__device__ inline void zou_he(C f[9], const JobDev &j, int x, int y, int64_t t, double u_peak) {
    zou_he_u(f, x == 0, x == 0 ? (C)inflow_u(j.ny, j.ramp, y, t, u_peak) : C(0));
}

// Addressing inside one sample's slab.
struct Site {
    int x, y, xm, xp, ym, yp;
};

__device__ inline Site site(const JobDev &j, int x, int y) {
    Site s;
    s.x = x;
    s.y = y;
    s.xm = x == 0 ? j.nx - 1 : x - 1;
    s.xp = x == j.nx - 1 ? 0 : x + 1;
    s.ym = y == 0 ? j.ny - 1 : y - 1;
    s.yp = y == j.ny - 1 ? 0 : y + 1;
    return s;
}

__device__ inline int sx_of(const Site &s, int dx) { return dx == 0 ? s.x : (dx > 0 ? s.xp : s.xm); }
__device__ inline int sy_of(const Site &s, int dy) { return dy == 0 ? s.y : (dy > 0 ? s.yp : s.ym); }

// Access modes of a step / QoI read.
enum : int { AA_EVEN = 0, AA_ODD = 1, AB_PULL = 2 };

template <int LAYOUT, int PARITY>
struct ModeOf {
    static constexpr int value = LAYOUT == UQ_LAYOUT_AB ? AB_PULL : (PARITY ? AA_ODD : AA_EVEN);
};

// Interpolated bounce-back (Bouzidi, Firdaouss & Lallemand 2001) for pull
// direction i of a node whose link x -> x - c_i meets the cylinder at
// fraction q; AB layout, where the source slab holds every node's f* of the
// previous step. With k = opp(i):
//   q <  1/2: f_i(x) = 2q f*_k(x) + (1 - 2q) f*_k(x + c_i)
//   q >= 1/2: f_i(x) = f*_k(x)/(2q) + (1 - 1/(2q)) f*_i(x)
// (x + c_i is fluid: the circle keeps clear of the walls, and by convexity
// the node behind a fluid node on a link into the circle is outside it). The
// weights of the shifted populations cancel (the coefficients sum to 1).
template <int P>
__device__ inline typename Prec<P>::C wall_return(const JobDev &j, const typename Prec<P>::T *base, const Site &s,
                                                  int64_t own, int i) {
    using PR = Prec<P>;
    using C = typename PR::C;
    const int k = OPPd[i];
    const C fk = PR::ld(base + k * j.plane + own, j.inv_scale);
    const double q = j.q[(int64_t)i * j.ny * j.pitch + own];
    if (!(q > 0.0)) return fk;  // a half-way link (channel wall)
    if (q >= 0.5) {
        const C fi = PR::ld(base + i * j.plane + own, j.inv_scale);
        const double a = 1.0 / (2.0 * q);
        return (C)a * fk + (C)(1.0 - a) * fi;
    }
    const int xb = sx_of(s, CXd[i]), yb = sy_of(s, CYd[i]);
    const C fb = PR::ld(base + k * j.plane + (int64_t)yb * j.pitch + xb, j.inv_scale);
    return (C)(2.0 * q) * fk + (C)(1.0 - 2.0 * q) * fb;
}

template <int P, bool CHANNEL, int MODE, bool FD = true, bool QL = true>
__device__ inline void gather(const JobDev &j, const typename Prec<P>::T *base, const Site &s, uint32_t m,
                              int64_t t, double u_peak, double omega, typename Prec<P>::C f[9]);

__device__ inline double inlet_ux(const JobDev &j, int y, int64_t t, double u_peak) {
    return inflow_u(j.ny, j.ramp, y, t, u_peak);
}

// velocity of an outlet-column node from its known populations (rho = 1)
template <int P>
__device__ inline double outlet_ux(const JobDev &j, const typename Prec<P>::T *base, int x, int y, int64_t t,
                                   double u_peak, double omega) {
    typename Prec<P>::C g[9];
    gather<P, true, AB_PULL, false>(j, base, site(j, x, y), j.mask[(int64_t)y * j.pitch + x], t, u_peak, omega, g);
    return (double)((g[0] + g[2] + g[4]) + (g[1] + g[5] + g[8]) + (g[1] + g[5] + g[8]));
}

// velocity of an interior node from its streamed populations
template <int P>
__device__ inline void node_u(const JobDev &j, const typename Prec<P>::T *base, int x, int y, int64_t t,
                              double u_peak, double omega, double &ux, double &uy) {
    using C = typename Prec<P>::C;
    C g[9], drho, gx, gy;
    gather<P, true, AB_PULL, false>(j, base, site(j, x, y), j.mask[(int64_t)y * j.pitch + x], t, u_peak, omega, g);
    moments(g, drho, gx, gy);
    ux = (double)gx;
    uy = (double)gy;
}

// Finite-difference reconstruction of an open-column node (the paper's
// interpolated inlet / outlet after Latt et al. 2008): f_i = f_i^eq(rho, u)
// + f_i^neq, f_i^neq = -3 w_i rho tau Q_i : grad u, Q_i = c_i c_i - I/3.
// grad u: across the column the one-sided second-order difference
// (-3 u_0 + 4 u_1 - u_2)/2 into the fluid; along it the central difference,
// one-sided at the two end rows. Inlet: u prescribed, rho from the known
// populations; outlet: rho = 1, u_y = 0, u_x from the known populations.

// imposed state of an open-column node from its streamed populations
// (unknown ones unset)
template <typename C>
__device__ inline void fd_state_u(const C f[9], bool inlet, double u_in, double &rho, double &ux) {
    if (inlet) {
        ux = u_in;
        const double S = (double)((f[0] + f[2] + f[4]) + (f[3] + f[6] + f[7]) + (f[3] + f[6] + f[7]));
        rho = 1.0 + (S + ux) / (1.0 - ux);
    } else {
        rho = 1.0;
        ux = (double)((f[0] + f[2] + f[4]) + (f[1] + f[5] + f[8]) + (f[1] + f[5] + f[8]));
    }
}
template <typename C>
__device__ inline void fd_state(const JobDev &j, const C f[9], bool inlet, int y, int64_t t, double u_peak,
                                double &rho, double &ux) {
    fd_state_u(f, inlet, inlet ? inlet_ux(j, y, t, u_peak) : 0.0, rho, ux);
}

// d(u_x)/dy along the column from the column values at y-2 .. y+2
// (um2, um1, u0, up1, up2; only those inside the column are read)
__device__ inline double fd_dy(int y, int ny, double um2, double um1, double u0, double up1, double up2) {
    if (y == 0) return (-3.0 * u0 + 4.0 * up1 - up2) * 0.5;
    if (y == ny - 1) return (3.0 * u0 - 4.0 * um1 + um2) * 0.5;
    return (up1 - um1) * 0.5;
}

// f = f^eq + f^neq from the imposed state and the gradient (u_y = 0)
template <typename C>
__device__ inline void fd_rebuild(C f[9], double rho, double ux, double dxux, double dxuy, double dyux, double omega) {
    const double uy = 0.0, dyuy = 0.0;
    const double tau = 1.0 / omega, drho = rho - 1.0, uu = ux * ux + uy * uy;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const double cx = CXd[i], cy = CYd[i], w = wgt<double>(i);
        const double cu = cx * ux + cy * uy;
        const double QS = (cx * cx - 1.0 / 3.0) * dxux + (cy * cy - 1.0 / 3.0) * dyuy + cx * cy * (dxuy + dyux);
        f[i] = (C)(w * (drho + rho * (3.0 * cu + 4.5 * cu * cu - 1.5 * uu)) - 3.0 * w * rho * tau * QS);
    }
}

// the whole reconstruction for one node, neighbours gathered here (QoI and
// export kernels; the step shares them in LDS, fd_column_chunk)
template <int P>
__device__ inline void fd_column(const JobDev &j, const typename Prec<P>::T *base, const Site &s, int64_t t,
                                 double u_peak, double omega, typename Prec<P>::C f[9]) {
    const int x = s.x, y = s.y, ny = j.ny;
    const bool inlet = x == 0;
    const int sd = inlet ? 1 : -1;
    double rho, ux;
    fd_state(j, f, inlet, y, t, u_peak, rho, ux);
    double u1x, u1y, u2x, u2y;
    node_u<P>(j, base, x + sd, y, t, u_peak, omega, u1x, u1y);
    node_u<P>(j, base, x + 2 * sd, y, t, u_peak, omega, u2x, u2y);
    const double dxux = sd * (-3.0 * ux + 4.0 * u1x - u2x) * 0.5;
    const double dxuy = sd * (-3.0 * 0.0 + 4.0 * u1y - u2y) * 0.5;
    auto col_ux = [&](int yy) {
        return inlet ? inlet_ux(j, yy, t, u_peak) : outlet_ux<P>(j, base, x, yy, t, u_peak, omega);
    };
    double dyux;
    if (y == 0)
        dyux = fd_dy(y, ny, 0.0, 0.0, ux, col_ux(1), col_ux(2));
    else if (y == ny - 1)
        dyux = fd_dy(y, ny, col_ux(ny - 3), col_ux(ny - 2), ux, 0.0, 0.0);
    else
        dyux = fd_dy(y, ny, 0.0, col_ux(y - 1), ux, col_ux(y + 1), 0.0);
    fd_rebuild(f, rho, ux, dxux, dxuy, dyux, omega);
}

// Gather f~(x, t) of one node, with the wall rules and the open columns
// (FD = false leaves the open-column populations of a finite-difference job
// unset: the reconstruction reads its neighbours that way; QL = false omits
// the interpolated links: the bulk step kernel never meets those nodes).
template <int P, bool CHANNEL, int MODE, bool FD, bool QL>
__device__ inline void gather(const JobDev &j, const typename Prec<P>::T *base, const Site &s, uint32_t m,
                              int64_t t, double u_peak, double omega, typename Prec<P>::C f[9]) {
    using PR = Prec<P>;
    using C = typename PR::C;
    const float inv = j.inv_scale;
    const int64_t pitch = j.pitch, plane = j.plane;
    const int64_t own = (int64_t)s.y * pitch + s.x;
    // Every direction issues its one load unconditionally, the wall rule only
    // selecting the address: with no branches between them all nine loads
    // are in flight together (per-direction branches made the compiler wait
    // for each load at the block boundaries).
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        if (MODE == AA_EVEN) {
            f[i] = PR::ld(base + i * plane + own, inv);
            continue;
        }
        // pull: f_i(x,t) = f*_i(x - c_i, t-1) (AA odd: slot opp(i) there;
        // AB: slot i); bounce-back: f*_opp(i)(x, t-1) at this node (AA odd:
        // slot i; AB: slot opp(i))
        const int xs = sx_of(s, -CXd[i]), ys = sy_of(s, -CYd[i]);
        int64_t off = (int64_t)(MODE == AA_ODD ? OPPd[i] : i) * plane + (int64_t)ys * pitch + xs;
        bool bb = false;
        if (CHANNEL) {
            bb = (m >> (M_BB + i)) & 1u;
            const int64_t off_bb = (int64_t)(MODE == AA_ODD ? i : OPPd[i]) * plane + own;
            off = bb ? off_bb : off;
        }
        C v = PR::ld(base + off, inv);
        if (CHANNEL) {
            // interpolated links (AB only) combine it with a second value
            if (MODE == AB_PULL && QL && bb && (m & M_QLINK)) v = wall_return<P>(j, base, s, own, i);
            // beyond an open column: rest state at t = 0, else filled below
            // (the wrapped pull address is in bounds; its value is unused)
            v = ((m >> (M_OPEN + i)) & 1u) ? C(0) : v;
        }
        f[i] = v;
    }
    if (CHANNEL && (m & (0x1FFu << M_OPEN)) && t > 0) {
        if (j.xbc != UQ_XBC_INTERP)
            zou_he(f, j, s.x, s.y, t, u_peak);
        else if (MODE == AB_PULL && FD)
            fd_column<P>(j, base, s, t, u_peak, omega, f);
    }
}

// Scatter post-collision f*(x, t) to where step t+1 reads it.
template <int P, bool CHANNEL, int MODE, bool NT>
__device__ inline void scatter(const JobDev &j, typename Prec<P>::T *base, const Site &s, uint32_t m,
                               const typename Prec<P>::C f[9]) {
    using PR = Prec<P>;
    const float sc = j.scale;
    const int64_t pitch = j.pitch, plane = j.plane;
    const int64_t own = (int64_t)s.y * pitch + s.x;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        if (MODE == AB_PULL) {
            if (NT)
                PR::st_nt(base + i * plane + own, f[i], sc);
            else
                PR::st(base + i * plane + own, f[i], sc);
        } else if (MODE == AA_EVEN) {
            PR::st(base + OPPd[i] * plane + own, f[i], sc);
        } else {
            // AA odd: f*_i goes to slot i of x + c_i; if that is a wall it
            // returns to this node as f_opp(i) (slot opp(i) here). A value
            // leaving through an open column is parked in that same own slot,
            // which nothing else writes and the next gather overrides (no
            // branch: the stores stay back to back).
            const int o = OPPd[i];
            const int xd = sx_of(s, CXd[i]), yd = sy_of(s, CYd[i]);
            int64_t off = (int64_t)i * plane + (int64_t)yd * pitch + xd;
            if (CHANNEL) {
                const bool back = ((m >> (M_BB + o)) | (m >> (M_OPEN + o))) & 1u;
                off = back ? (int64_t)o * plane + own : off;
            }
            PR::st(base + off, f[i], sc);
        }
    }
}

// Slab holding the state at step t (AA: the only one; AB: slab t & 1).
template <int LAYOUT>
__device__ inline void *state_slab(const JobDev &j, int64_t t) {
    return (LAYOUT == UQ_LAYOUT_AB && (t & 1)) ? j.f2 : j.f;
}

// ------------------------------------------------------------------ tile walk
// Blocks are dealt round-robin to the 8 XCDs; renumber them so that each XCD
// gets a contiguous run of tiles (neighbouring rows share its L2).
__device__ inline int64_t xcd_logical(int64_t b, int64_t G) {
    const int64_t xcd = b & 7, k = b >> 3;
    const int64_t q = G >> 3, r = G & 7;
    return xcd * q + (xcd < r ? xcd : r) + k;
}

constexpr int BX = 64;  // default workgroup shape: 64 nodes along x (one
constexpr int BY = 4;   // wavefront) by 4 rows; the step kernel takes any
                        // 256-thread shape bx x (256/bx) from its launch
// ------------------------------------------------------------------ buffer access
// Buffer loads for the fused kernel: base address and size in a (uniform)
// resource descriptor, a 32-bit byte offset per lane and a uniform offset per
// population plane; no 64-bit address arithmetic per load. 0x00020000 is the
// descriptor's fourth word for raw 32-bit data on this GPU family.
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void *p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, bytes, 0x00020000);
}
template <int P>
struct BufLd;
// raw(): the stored value as loaded; cvt(): its compute value (kept apart so
// that a load's register is not consumed before it is needed)
template <>
struct BufLd<UQ_FP64> {
    using R = double;
    __device__ static inline R raw(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    }
    __device__ static inline double cvt(R v, float) { return v; }
    __device__ static inline double ld(__amdgpu_buffer_rsrc_t r, int voff, int soff, float inv) {
        return cvt(raw(r, voff, soff), inv);
    }
};
template <>
struct BufLd<UQ_FP32> {
    using R = float;
    __device__ static inline R raw(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
    }
    __device__ static inline float cvt(R v, float) { return v; }
    __device__ static inline float ld(__amdgpu_buffer_rsrc_t r, int voff, int soff, float inv) {
        return cvt(raw(r, voff, soff), inv);
    }
};
template <>
struct BufLd<UQ_FP16S> {
    using R = unsigned short;
    __device__ static inline R raw(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
        return __builtin_bit_cast(unsigned short, __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0));
    }
    __device__ static inline float cvt(R v, float inv) { return Prec<UQ_FP16S>::up(__builtin_bit_cast(_Float16, v), inv); }
    __device__ static inline float ld(__amdgpu_buffer_rsrc_t r, int voff, int soff, float inv) {
        return cvt(raw(r, voff, soff), inv);
    }
};
template <>
struct BufLd<UQ_BF16S> {
    using R = unsigned short;
    __device__ static inline R raw(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
        return __builtin_bit_cast(unsigned short, __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0));
    }
    __device__ static inline float cvt(R v, float) { return __uint_as_float((uint32_t)v << 16); }
    __device__ static inline float ld(__amdgpu_buffer_rsrc_t r, int voff, int soff, float inv) {
        return cvt(raw(r, voff, soff), inv);
    }
};

// buffer stores: per-lane byte offset + wave-uniform byte offset (cached)
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
template <int P>
struct BufSt;
template <>
struct BufSt<UQ_FP64> {
    __device__ static inline void st(__amdgpu_buffer_rsrc_t r, double v, int voff, int soff, float) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, v), r, voff, soff, 0);
    }
};
template <>
struct BufSt<UQ_FP32> {
    __device__ static inline void st(__amdgpu_buffer_rsrc_t r, float v, int voff, int soff, float) {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, voff, soff, 0);
    }
};
template <>
struct BufSt<UQ_FP16S> {
    __device__ static inline void st(__amdgpu_buffer_rsrc_t r, float v, int voff, int soff, float sc) {
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, (_Float16)(v * sc)), r, voff, soff, 0);
    }
};
template <>
struct BufSt<UQ_BF16S> {
    __device__ static inline void st(__amdgpu_buffer_rsrc_t r, float v, int voff, int soff, float) {
        __builtin_amdgcn_raw_buffer_store_b16(Prec<UQ_BF16S>::rne(v), r, voff, soff, 0);
    }
};

// wrap a coordinate into [0, n) (it is at most a ring away from it, but the
// ring may exceed a tiny lattice)
__device__ inline int wrap_coord(int v, int n) {
    while (v < 0) v += n;
    while (v >= n) v -= n;
    return v;
}
// Job of work item wk in a batched table (work0 ascending, job 0 at 0).
__device__ inline int fused_job_of(const FusedJob *jobs, int njobs, int64_t wk) {
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].work0 <= wk) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The table entry of a work item, in scalar registers. Every lane of the
// workgroup reads the same entry, but the compiler cannot tell, and a job's
// pointers built from vector registers would put every buffer access of the
// pipeline in a loop over the distinct descriptors (v_readfirstlane per
// access); each dword goes through readfirstlane once per item instead.
__device__ inline FusedJob fused_entry(const FusedJob *jobs, int njobs, int64_t wk) {
    static_assert(sizeof(FusedJob) % 4 == 0, "FusedJob is a whole number of dwords");
    constexpr int NW = (int)(sizeof(FusedJob) / 4);
    uint32_t w[NW];
    __builtin_memcpy(w, &jobs[fused_job_of(jobs, njobs, wk)], sizeof(FusedJob));
#pragma unroll
    for (int i = 0; i < NW; ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
    FusedJob q;
    __builtin_memcpy(&q, w, sizeof(FusedJob));
    return q;
}

}  // namespace uqi
