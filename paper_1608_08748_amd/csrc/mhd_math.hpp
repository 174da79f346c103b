// Device-side arithmetic of the step: grid indexing, the local parabola
// (Sec. 2.1), the NONADV face Riemann solve (Sec. 2.4 and the eigenvector
// appendix), FP64 chemistry (Sec. 2.7, rate appendix), the CFL speed sum
// (Sec. 2.3) and wavefront reductions.  Included by mhd.hip only.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace mhd {

constexpr int NTH = 256;           // threads per block for cell-parallel kernels
constexpr int NF = 11;             // conserved fields (the last, H+, used by the ionisation network)
constexpr int NFACE = 7;           // per-face outputs
enum { RHO = 0, MX, MY, MZ, EN, EI, BX, BY, BZ, H2, HP };

// ---------------------------------------------------------------- geometry

// Division of 0 <= n < 2^31 by a fixed d >= 1 as one product and a shift: with
// l = ceil(log2 d) and m = ceil(2^(31 + l) / d), n m / 2^(31 + l) exceeds n / d
// by less than 1 / d, so its whole part is the quotient.  (The compiler's
// division by a run-time value takes about 20 instructions.)
struct FastDiv {
    uint32_t m, sh;
    __host__ __device__ __forceinline__ int div(int n) const { return (int)(((uint64_t)(uint32_t)n * m) >> sh); }
};

inline FastDiv fast_div(int d)
{
    uint32_t l = 0;
    while (((uint64_t)1 << l) < (uint64_t)d) l++;
    FastDiv f;
    f.sh = 31 + l;
    f.m = (uint32_t)((((uint64_t)1 << f.sh) + (uint64_t)d - 1) / (uint64_t)d);
    return f;
}

struct Geo {
    int nx, ny, nz;
    int nxy;
    int n;          // nx * ny * nz
    FastDiv dx, dy, dz;
};

inline Geo make_geo(int nx, int ny, int nz)
{
    Geo g;
    g.nx = nx;
    g.ny = ny;
    g.nz = nz;
    g.nxy = nx * ny;
    g.n = nx * ny * nz;
    g.dx = fast_div(nx);
    g.dy = fast_div(ny);
    g.dz = fast_div(nz);
    return g;
}

__device__ __forceinline__ int wrapc(int x, int n)
{
    if (x < 0) x += n;
    if (x >= n) x -= n;
    if ((unsigned)x >= (unsigned)n) {   // only for boxes thinner than the stencil
        x %= n;
        if (x < 0) x += n;
    }
    return x;
}

// cell index of the neighbour at offset s along direction D
template <int D>
__device__ __forceinline__ int nbr(const Geo& g, int c, int i, int j, int k, int s)
{
    if (D == 0) return c - i + wrapc(i + s, g.nx);
    if (D == 1) return c + (wrapc(j + s, g.ny) - j) * g.nx;
    return c + (wrapc(k + s, g.nz) - k) * g.nxy;
}

__device__ __forceinline__ void decompose(const Geo& g, int c, int& i, int& j, int& k)
{
    const int row = g.dx.div(c);
    i = c - row * g.nx;
    k = g.dy.div(row);
    j = row - k * g.ny;
}

// How the kernels of a launch reach the fields.  Near: a field is at most 4 GiB,
// so a value's byte offset is 32 bits wide; the load takes the base from scalar
// registers and one offset serves every field of a cell (with 64-bit offsets
// each access costs a 64-bit vector addition of its own, 49 of 1190
// instructions of the FP32 x-row kernel).  Streamed: the same, and the outputs
// go past the caches: a box whose arrays exceed the 256 MB Infinity Cache
// several times over finds nothing of them there in the next kernel, and the
// stores only evict what neighbouring blocks still read (steps of 256^3 1.2%
// shorter in FP64 and 2.4% in FP32; of 96^3 FP64 6% longer).  Far: longer
// fields, streamed.
struct Near { using Off = uint32_t; static constexpr bool stream = false; };
struct Streamed { using Off = uint32_t; static constexpr bool stream = true; };
struct Far { using Off = uint64_t; static constexpr bool stream = true; };

// Value i of an array that starts at the same address in every lane.  The
// global address space is stated because the pointers of a multi-box launch
// come from its table in memory, where the compiler would take them for
// generic ones (flat loads, which also wait for the LDS).
template <typename T> using Global = __attribute__((address_space(1))) T;
template <class O, typename T>
__device__ __forceinline__ Global<T>& at(T* p, int i)
{
    using C = std::conditional_t<std::is_const<T>::value, const char, char>;
    using B = typename O::Off;
    return *(Global<T>*)((Global<C>*)p + (B)((B)(unsigned)i * (B)sizeof(T)));
}
template <class O, typename T>
__device__ __forceinline__ void put(T* p, int i, T v)
{
    if constexpr (O::stream) __builtin_nontemporal_store(v, &at<O>(p, i));
    else at<O>(p, i) = v;
}

template <typename T> struct Fields { T* f[NF]; };
template <typename T> struct CFields { const T* f[NF]; };

// ---------------------------------------------------------------- roots and reciprocals

// Square root, reciprocal square root and reciprocal used by the face solvers.
// FP64: the hardware estimate refined by Newton-Raphson steps, which converge
// quadratically, so the result lands within about one ulp of the correctly
// rounded value at a third of the instruction count of the library forms.
// Arguments are positive and normal (densities, pressures, squared speeds);
// root_nr(0) = 0.  FP32: the single hardware instruction (about one ulp).
__device__ __forceinline__ double rsqrt_nr(double x)
{
    double h = 0.5 * x;
    double y = __builtin_amdgcn_rsq(x);
    double t = h * y;
    double e = fma(-t, y, 0.5);
    y = fma(y, e, y);
    t = h * y;
    e = fma(-t, y, 0.5);
    return fma(y, e, y);
}
// coupled iteration on sqrt(x) and 1/(2 sqrt(x)), then one correction of the
// root from its exact residual x - g^2
__device__ __forceinline__ double root_nr(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    double r = fma(-g, h, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    double d = fma(-g, g, x);
    g = fma(d, h, g);
    return x > 0.0 ? g : 0.0;
}
__device__ __forceinline__ double rcp_nr(double b)
{
    double r = __builtin_amdgcn_rcp(b);
    double e = fma(-b, r, 1.0);
    r = fma(r, e, r);
    e = fma(-b, r, 1.0);
    return fma(r, e, r);
}
__device__ __forceinline__ float rsqrt_nr(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ float root_nr(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ float rcp_nr(float b) { return __builtin_amdgcn_rcpf(b); }

// ---------------------------------------------------------------- local parabola (Sec. 2.1)

template <typename T> struct Par { T qL, qR, dq, q6; };

// Step 1: limited central difference (min of the three candidates, sign of
// the central difference; zero at extrema)
__device__ __forceinline__ double limited_slope(double qm, double q0, double qp)
{
    double dq = 0.5 * (qp - qm);
    double m = fmin(fabs(dq), 2.0 * fmin(fabs(qp - q0), fabs(q0 - qm)));
    return ((qp - q0) * (q0 - qm) > 0.0) ? copysign(m, dq) : 0.0;
}
// FP32: the median of zero and two numbers is the smaller one of the same sign,
// or zero, so two median instructions give the same value in 7 instructions
// instead of 11.  (Where the product above would underflow, differences below
// 1e-22, this is the slope and not zero.)
__device__ __forceinline__ float limited_slope(float qm, float q0, float qp)
{
    const float lim = 2.0f * __builtin_amdgcn_fmed3f(0.0f, qp - q0, q0 - qm);
    return __builtin_amdgcn_fmed3f(0.0f, 0.5f * (qp - qm), lim);
}

// Step 1: fourth-order interface value q_{j+1/2} = 1/2 (q_j + q_{j+1}) - 1/6 (dm_{j+1} - dm_j)
template <typename T>
__device__ __forceinline__ T interface_value(T q0, T q1, T dm0, T dm1)
{
    return T(0.5) * (q0 + q1) - T(1.0 / 6.0) * (dm1 - dm0);
}

// margins that decide a saturated Step-4 weight without the division
template <typename T> struct EtaMargin;
template <> struct EtaMargin<double> { static constexpr double lo = 0.05 * (1.0 - 1e-9), hi = 0.1 * (1.0 + 1e-9); };
template <> struct EtaMargin<float> { static constexpr float lo = 0.05f * (1.0f - 1e-5f), hi = 0.1f * (1.0f + 1e-5f); };

// t where d is positive, -t where it is negative
__device__ __forceinline__ float along(float t, float d)
{
    return __uint_as_float(__float_as_uint(t) ^ (__float_as_uint(d) & 0x80000000u));
}
__device__ __forceinline__ double along(double t, double d)
{
    return __hiloint2double(__double2hiint(t) ^ (__double2hiint(d) & (int)0x80000000u), __double2loint(t));
}

// Steps 2-5 for cell j with line values qmm..qpp, Step-1 edge values qL, qR
// and limited slope dm of the cell
template <typename T>
__device__ __forceinline__ Par<T> parabola_finish(T qmm, T qm, T q0, T qp, T qpp, T qL, T qR, T dm)
{
    // Step 2: monotone edge values
    T dq = qR - qL;
    T q6 = T(6) * (q0 - T(0.5) * (qL + qR));
    bool flat = (qL - q0) * (q0 - qR) <= T(0);
    bool overL = dq * q6 > dq * dq;
    bool overR = dq * q6 < -(dq * dq);
    T fL = flat ? q0 : (overL ? T(3) * q0 - T(2) * qR : qL);
    T fR = flat ? q0 : ((!overL && overR) ? T(3) * q0 - T(2) * qL : qR);
    // Step 4: discontinuity detector on second differences (h^2 cancels):
    // eta = t / d with the weight w = clamp(20 (eta - 0.05), 0, 1), zero for
    // eta at most 0.05 or second differences of one sign.  Those two tests
    // alone, without the quotient and with a relative margin far above
    // rounding, leave only the cells around jumps to the rest, so most waves
    // skip it (18 of 84 instructions; a step of 256^3 6-7% shorter in FP64 and
    // FP32.  With the first test alone the extrema come in too: 2% more at 64^3
    // where nearly every wave then holds one; with every test here, 1% less at
    // 256^3).  The first compares magnitudes, in range wherever t and d are:
    // t d against d^2, level in time, lost the jumps whose square overflows.
    const T Dm = q0 - T(2) * qm + qmm;
    const T Dp = qpp - T(2) * qp + q0;
    const T t = -(Dp - Dm);
    const T d = T(6) * (qp - qm);
    if ((along(t, d) > EtaMargin<T>::lo * fabs(d)) & !(Dp * Dm > T(0))) {
        // the smallest of |q_{i+1}|, |q_{i-1}| and their sum is one of the two
        const T mn = fmin(fabs(qp), fabs(qm));
        const bool zero_eta = fabs(qp - qm) - T(0.01) * mn <= T(0);
        // exactly one above eta = 0.1, whatever the quotient rounds to
        const T eta = t * rcp_nr(d);
        T w = fmin(fmax(T(20) * (eta - T(0.05)), T(0)), T(1));
        w = fabs(t) >= EtaMargin<T>::hi * fabs(d) ? T(1) : w;
        w = zero_eta ? T(0) : w;
        // q0 -/+ dm / 4 with one rounding each: dm / 2 is exact, and the fused
        // product (dm / 2) / 2 is the exact dm / 4 (inline constants only)
        const T hdm = T(0.5) * dm;
        const T qLp = fma(T(-0.5), hdm, q0);
        const T qRp = fma(T(0.5), hdm, q0);
        fL = (T(1) - w) * fL + w * qLp;
        fR = (T(1) - w) * fR + w * qRp;
    }
    // Step 5
    Par<T> p;
    p.qL = fL;
    p.qR = fR;
    p.dq = fR - fL;
    p.q6 = T(6) * (q0 - T(0.5) * (fL + fR));
    return p;
}

// Sec. 2.4: average over the right part of relative width y (the q(-nu t) formula)
template <typename T>
__device__ __forceinline__ T avg_right(const Par<T>& p, T y)
{
    return p.qR - T(0.5) * y * (p.dq - p.q6 * (T(1) - T(2.0 / 3.0) * y));
}

// Sec. 2.4: average over the left part of relative width y (the q(+nu t) formula)
template <typename T>
__device__ __forceinline__ T avg_left(const Par<T>& p, T y)
{
    return p.qL + T(0.5) * y * (p.dq + p.q6 * (T(1) - T(2.0 / 3.0) * y));
}

template <typename T> struct Eps;
template <> struct Eps<double> { static constexpr double v = 1e-12; };
template <> struct Eps<float> { static constexpr float v = 1e-6f; };

// ---------------------------------------------------------------- kernels

// What one side of a face needs from a cell's parabolas (6 variables): the
// edge value facing the face (qR of the left cell, qL of the right cell), dq
// and q6.
template <typename T> struct Side { T e[6], dq[6], q6[6]; };

template <typename T>
__device__ __forceinline__ void side_left(const Par<T>& P, Side<T>& S, int v)
{
    S.e[v] = P.qR;
    S.dq[v] = P.dq;
    S.q6[v] = P.q6;
}

template <typename T>
__device__ __forceinline__ void side_right(const Par<T>& P, Side<T>& S, int v)
{
    S.e[v] = P.qL;
    S.dq[v] = P.dq;
    S.q6[v] = P.q6;
}

// NONADV face state (Sec. 2.4) of one face and the fluxes and edge-field
// contributions it produces.  Inputs: cell-centre rho, p, Bt1, Bt2 of the left
// and right cells, the face normal field bn, the two sides' parabolas of
// (vn, vt1, vt2, Bt1, Bt2, p), the adiabatic index gm, or with ion the two
// cells' gamma_eff.  Outputs (7): momentum flux (normal, t1, t2),
// energy flux, face normal velocity, E along t1 (B_t2 U_n - B_n U_t2), E along
// t2 (B_n U_t1 - B_t1 U_n).
template <typename T>
__device__ __forceinline__ void face_solve(T rl, T pl, T b1l, T b2l, T rr, T pr, T b1r, T b2r, T bn,
                                           const Side<T>& L, const Side<T>& R, T gm, T gml, T gmr, bool ion, T ydx,
                                           T sl, T sr, T out[7])
{
    const T eps = Eps<T>::v;
    // face averages (sqrt(rho) weights, sl = root_nr(rl) and sr = root_nr(rr)
    // formed once per cell by the caller; cross weights for Bt); with the
    // ionisation network the adiabatic index is the cells' gamma_eff averaged
    // with the weights of p
    T iw = rcp_nr(sl + sr);
    T rho = (sl * rl + sr * rr) * iw;
    T p = (sl * pl + sr * pr) * iw;
    if (ion) gm = (sl * gml + sr * gmr) * iw;
    T bt1 = (sl * b1r + sr * b1l) * iw;
    T bt2 = (sl * b2r + sr * b2l) * iw;

    // eigen-structure (Sec. 2.3, 2.4, eigenvector appendix); every root and
    // reciprocal of rho and gamma p derives from their two reciprocal roots
    T rs = rsqrt_nr(rho);                // 1 / sqrt(rho)
    T irho = rs * rs;
    T srho = rho * rs;
    T gp = gm * p;
    T rg = rsqrt_nr(gp);                 // 1 / sqrt(gamma p) = 1 / (sqrt(rho) c)
    T c2 = gp * irho;
    T ca2 = bn * bn * irho;
    T b2 = (bn * bn + bt1 * bt1 + bt2 * bt2) * irho;
    T s = c2 + b2;
    T disc = fmax(s * s - T(4) * c2 * ca2, T(0));
    T sd = root_nr(disc);
    T cf2 = T(0.5) * (s + sd);
    T cs2 = fmax(T(0.5) * (s - sd), T(0));
    T cc = (gp * rg) * rs, ca = fabs(bn) * rs, cf = root_nr(cf2), cs = root_nr(cs2);
    const T r2i = T(0.70710678118654752440);
    T den = cf2 - cs2;
    T af = r2i, as = r2i;
    if (den > eps * s) {
        T iden = rcp_nr(den);
        af = root_nr(fmax(c2 - cs2, T(0)) * iden);
        as = root_nr(fmax(cf2 - c2, T(0)) * iden);
    }
    T by = r2i, bz = r2i;
    T btsq = bt1 * bt1 + bt2 * bt2;
    if (btsq > eps * (bn * bn + btsq + gm * p)) {
        T ibt = rsqrt_nr(btsq);
        by = bt1 * ibt;
        bz = bt2 * ibt;
    }
    T sg = bn >= T(0) ? T(1) : T(-1);

    // parabola averages on the upwind side of each wave: waves +cf, +cs, +ca
    // read the left cell (right part, q(-nu t)), waves -cf, -cs, -ca the right
    // cell (left part, q(+nu t))
    T qf[6], qfm[6], qs[6], qsm[6], qa[6], qam[6];
    T y3[3] = { ydx * cf, ydx * cs, ydx * ca };
    T hy[3], ky[3];
#pragma unroll
    for (int w = 0; w < 3; w++) {
        hy[w] = T(0.5) * y3[w];
        ky[w] = T(1) - T(2.0 / 3.0) * y3[w];
    }
#pragma unroll
    for (int v = 0; v < 6; v++) {
        qf[v] = L.e[v] - hy[0] * (L.dq[v] - L.q6[v] * ky[0]);
        qs[v] = L.e[v] - hy[1] * (L.dq[v] - L.q6[v] * ky[1]);
        qa[v] = L.e[v] - hy[2] * (L.dq[v] - L.q6[v] * ky[2]);
        qfm[v] = R.e[v] + hy[0] * (R.dq[v] + R.q6[v] * ky[0]);
        qsm[v] = R.e[v] + hy[1] * (R.dq[v] + R.q6[v] * ky[1]);
        qam[v] = R.e[v] + hy[2] * (R.dq[v] + R.q6[v] * ky[2]);
    }

    // characteristic amplitudes s_k = l_k . q_up(k)
    T A = T(0.5) * (rho * (rg * rg));    // 1 / (2 c^2)
    T Bc = T(0.5) * rg;                  // 1 / (2 sqrt(rho) c)
    T Cc = T(0.5) * (rg * rg);           // 1 / (2 rho c^2)
    T Dc = r2i * rs;                     // 1 / sqrt(2 rho)
    T afcf = af * cf, ascs = as * cs;
    auto vtb = [&](const T* q) { return by * q[1] + bz * q[2]; };
    auto btb = [&](const T* q) { return by * q[3] + bz * q[4]; };
    auto vtp = [&](const T* q) { return -bz * q[1] + by * q[2]; };
    auto btp = [&](const T* q) { return -bz * q[3] + by * q[4]; };
    T s0 = (afcf * qf[0] - ascs * sg * vtb(qf)) * A + as * btb(qf) * Bc + af * qf[5] * Cc;
    T s1 = (-afcf * qfm[0] + ascs * sg * vtb(qfm)) * A + as * btb(qfm) * Bc + af * qfm[5] * Cc;
    T s2 = (ascs * qs[0] + afcf * sg * vtb(qs)) * A - af * btb(qs) * Bc + as * qs[5] * Cc;
    T s3 = (-ascs * qsm[0] - afcf * sg * vtb(qsm)) * A - af * btb(qsm) * Bc + as * qsm[5] * Cc;
    T s4 = sg * r2i * vtp(qa) - btp(qa) * Dc;
    T s5 = sg * r2i * vtp(qam) + btp(qam) * Dc;

    // face state q = sum_k r_k s_k
    T fdm = s0 - s1, fsm = s0 + s1, sdm = s2 - s3, ssm = s2 + s3, adm = s4 - s5, asm_ = s4 + s5;
    T src = gp * rg;                     // sqrt(rho) c = sqrt(gamma p)
    T sr2 = r2i * srho;
    T Vn = afcf * fdm + ascs * sdm;
    T Vt1 = sg * by * (-ascs * fdm + afcf * sdm) - bz * sg * r2i * asm_;
    T Vt2 = sg * bz * (-ascs * fdm + afcf * sdm) + by * sg * r2i * asm_;
    T Bt1 = by * src * (as * fsm - af * ssm) + sr2 * bz * adm;
    T Bt2 = bz * src * (as * fsm - af * ssm) - sr2 * by * adm;
    T P = gp * (af * fsm + as * ssm);

    // fluxes of the non-advective equations and edge-field contributions
    T Pst = P + T(0.5) * (bn * bn + Bt1 * Bt1 + Bt2 * Bt2);
    T BV = bn * Vn + Bt1 * Vt1 + Bt2 * Vt2;
    out[0] = Pst - bn * bn;
    out[1] = -(bn * Bt1);
    out[2] = -(bn * Bt2);
    out[3] = Pst * Vn - bn * BV;
    out[4] = Vn;
    out[5] = Bt2 * Vn - bn * Vt2;
    out[6] = bn * Vt1 - Bt1 * Vn;
}

// ---------------------------------------------------------------- FP64 per-cell physics

// The per-cell physics of the tail is FP64 arithmetic on both precision paths
// and bound the tail pass (470 us of a 6.1 ms FP32 step at 256^3 against 170 us
// for its memory), so quotients share their reciprocals and a rate with two
// exponentials selects its exponent and factor before one.  Quotients carry one
// residual correction, as close to the exact value as a division rounds.  Powers
// of ten are exp10 and the 0.77 powers pow: as exp of a multiple of ln 10, whose
// rounding at exponents near 30 is the error, the limits of reaction 2 were 2.5
// times as far off (rms 9e-15 against 3.6e-15), and a rate applied to num / den
// instead of the quotient left the H2 update a fifth further off.  That costs
// 7 of 56 us of the tail at 96^3 with everything on, 16 of 241 us at 256^3 FP32.

struct ChemArgs {
    int on;     // chemistry stage
    int cool;   // heating/cooling stage
    int ion;    // ionisation network (reactions 5-8, H+ field, gamma_eff)
    double n_unit, T_unit, t_unit;
    double n_inv;   // 1 / n_unit
    double e_rate;  // t_unit / (n_unit k_B T_unit): erg cm^-3 s^-1 to code energy density per code time
};

// a / b from r = rcp_nr(b); the last instruction gives the quotients with zeros
// and infinities, which have no residual
__device__ __forceinline__ double quot(double a, double b, double r)
{
    const double q = a * r;
    return __builtin_amdgcn_div_fixup(fma(fma(-b, q, a), r, q), b, a);
}
__device__ __forceinline__ double quot(double a, double b) { return quot(a, b, rcp_nr(b)); }

// Sec. 4.3: effective adiabatic index (5 n_H + 5 n_e + 7 n_H2) / (3 n_H +
// 3 n_e + 5 n_H2) of a cell with the ionisation network (n_e = n_H+), the
// constant gamma without it
__device__ __forceinline__ double gamma_cell(int ion, double gamma, double rho, double h2, double hp)
{
    if (!ion) return gamma;
    double nH = rho - h2 - hp, nH2 = 0.5 * h2, ne = hp;
    return quot(5.0 * nH + 5.0 * ne + 7.0 * nH2, 3.0 * nH + 3.0 * ne + 5.0 * nH2);
}

constexpr double LN10 = 2.302585092994045684;
constexpr double INV_LN10 = 0.43429448190325182765;

// number densities (cm^-3) and temperature of a cell: n_H = n_u (rho - h2 -
// hp), T = T_u mu p / rho with the mean mass mu = 1 / (1 - x_H2/2 + x_H+).  In a
// cell whose hydrogen is all molecular or ionised the chemistry's quotients by
// n_u can leave h2 + hp a unit in the last place above rho; the cooling takes a
// power of n_H, so a negative remainder counts as none.
struct Gas {
    double nH, nH2, ne, n, T, iT;
};

__device__ __forceinline__ Gas gas_state(const ChemArgs& ch, double gamma, double rho, double e, double h2, double hp)
{
    Gas g;
    const double atomic = rho - h2 - hp;
    g.nH = ch.n_unit * (atomic < 0.0 ? 0.0 : atomic);
    g.nH2 = ch.n_unit * h2 / 2.0;
    g.ne = ch.n_unit * hp;
    g.n = g.nH + g.nH2 + g.ne;
    g.T = quot(ch.T_unit * ((gamma - 1.0) * e), rho - 0.5 * h2 + hp);
    g.iT = rcp_nr(g.T);
    return g;
}

// formation rate C = k1' n n_H of reaction 1 as num / den
__device__ __forceinline__ void formation(const Gas& g, double& num, double& den)
{
    const double t2 = 0.01 * g.T, st2 = root_nr(t2);
    num = 3e-17 * st2 * g.n * g.nH;
    den = 1.0 + 0.4 * st2 + 0.2 * t2 + 0.08 * t2 * t2;
}

// D = k2 n_H + k3 n_H2 + k4 of H2 (reactions 2-4, optically thin k4)
__device__ __forceinline__ double h2_loss(const Gas& g)
{
    const double a = 6750.0 * g.iT, b = 7500.0 * g.iT;
    const bool hot2 = g.T > 7390.0, hot3 = g.T > 7291.0;
    const double k2 = (hot2 ? 6.11e-14 : 2.67e-15) * exp(hot2 ? -2.93e4 * g.iT : -(a * a));
    const double k3 = (hot3 ? 5.22e-14 : 3.17e-15) * exp(hot3 ? -3.22e4 * g.iT : -(4060.0 * g.iT) - b * b);
    return k2 * g.nH + k3 * g.nH2 + 3.3 * 1.7e-11;
}

// semi-implicit update (Sec. 2.7) of n with the creation rate C and the loss
// rate D over ts: n + ts (C - D n) / (1 + ts D)
__device__ __forceinline__ double semi_implicit(double n, double C, double D, double ts)
{
    return n + quot(ts * (C - D * n), 1.0 + ts * D);
}

// rates of reactions 5-8 (appendix): cosmic-ray ionisation per H atom (s^-1),
// collisional ionisation (a polynomial in ln of T in eV), radiative and grain
// recombination (cm^3 s^-1, log = log10)
__device__ __forceinline__ double rate_k6(double T)
{
    const double l = log(T * 8.617333262e-5);
    const double c[9] = { -32.7, 13.5, -5.7, 1.5, -0.3, 3.4e-2, -2.6e-3, 1.1e-4, -2.1e-6 };
    double s = c[8];
#pragma unroll
    for (int i = 7; i >= 0; i--) s = s * l + c[i];
    return exp(s);
}

__device__ __forceinline__ double rate_k7(double lnT)
{
    const double x = lnT * INV_LN10;
    const double num = -10.78 + x * (4.68 + x * (-0.87 + x * (0.08 + x * -3.87e-3)));
    const double den = 1.0 + x * (-0.38 + x * (0.06 + x * (-5.1e-3 + x * 2.4e-4)));
    return exp10(quot(num, den));
}

__device__ __forceinline__ double rate_k8(double lnT)
{
    // T^0.01586 10^(-1.8892 - 4.4e-5 log10 T) as one exponential; the last
    // factor is 10^2.756
    const double inner = 1.0 + 5.087e2 * exp((1.586e-2 - 4.4e-5) * lnT - 1.8892 * LN10);
    return quot(12.25e-14, 1.0 + 8.074e-6 * 570.1642722807472 * inner);
}

// Sec. 2.7 with the appendix rates of reactions 1-4 (optically thin k4)
__device__ __forceinline__ double chem_h2(const ChemArgs& ch, double gamma, double rho, double e, double h2, double dt)
{
    const Gas g = gas_state(ch, gamma, rho, e, h2, 0.0);
    double num, den;
    formation(g, num, den);
    double nn = semi_implicit(g.nH2, quot(num, den), h2_loss(g), dt * ch.t_unit);
    const double nmax = ch.n_unit * rho / 2.0;
    nn = nn > nmax ? nmax : nn;
    nn = nn < 0.0 ? 0.0 : nn;
    return 2.0 * quot(nn, ch.n_unit, ch.n_inv);
}

// Sec. 2 stage 5 and Sec. 2.8 with the appendix heating and cooling of
// reactions 1-4 (erg cm^-3 s^-1, x = log10(T / 1e4)): H2 formation heating
// 7.2e-12 erg per formed molecule (formation rate of reaction 1) thermalised
// by the fraction 1 / (1 + n_cr / n), n_cr = 10^(4 - 0.416 x - 0.327 x^2);
// photodissociation heating 6.4e-13 erg per event; the two cooling terms
// n_H2 L_H / (1 + L_H / L_L) of reactions 2 and 3.  In reaction 3's low-density
// limit k_H = k_H2 = 6.29e-15 * 1.38 f(T) / f(4500), f = sqrt(T) a exp(-a),
// a = 1 + 1 / (k_B T) with k_B T in eV, evaluated in logarithms.  Returns
// Gamma - Lambda; with the ionisation network n = n_H + n_H2 + n_H+, plus
// cosmic-ray heating 1.92e-28 n and collisional-ionisation cooling 2.18e-11
// erg k6 n_H n_e.
__device__ __forceinline__ double heat_cool(int ion, const Gas& g)
{
    const double ikb_ev = 1.0 / 8.617333262e-5;
    const double lnT = log(g.T);
    const double x = log10(1e-4 * g.T);
    double num, den;
    formation(g, num, den);
    const double ncr = exp10(4.0 - 0.416 * x - 0.327 * x * x);
    // num / den / (1 + n_cr / n)
    const double g1 = 7.2e-12 * quot(num * g.n, den * (g.n + ncr));
    const double g4 = 6.4e-13 * (3.3 * 1.7e-11) * g.nH2;
    const bool hoth = g.T > 1087.0, hotl = g.T > 4031.0;
    const double lh2 = hoth ? 3.9e-19 * exp(-6118.0 * g.iT) : exp10(-19.24 + 0.474 * x - 1.247 * x * x);
    const double fl2 = hotl ? 1.38e-22 * exp(-9243.0 * g.iT) : exp10(-22.9 - 0.553 * x - 1.148 * x * x);
    const double ll2 = (pow(g.nH2, 0.77) + 1.2 * pow(g.nH, 0.77)) * fl2;
    // n_H2 L_H / (1 + L_H / L_L); both limits underflow in the coldest gas, and
    // the reciprocal of a sum below the normal range is infinite
    const double l2 = quot(g.nH2 * (lh2 * ll2), lh2 + ll2 + 1e-300);
    const double a = 1.0 + ikb_ev * g.iT;
    const double a45 = 1.0 + 1.0 / (8.617333262e-5 * 4500.0);
    const double lnf = 0.5 * lnT + log(a * g.n) - a;   // with the log(n) of the limit
    const double lnf45 = 0.5 * log(4500.0) + log(a45) - a45;
    const double ln_ll3 = log(8.18e-13) + log(6.29e-15 * 1.38) + lnf - lnf45;
    const double ln_lh3 = log(1.1e-13) - 6744.0 * g.iT;
    // the second exponential is far from overflow where the first is not zero
    const double l3 = g.nH2 * quot(exp(ln_lh3), 1.0 + exp(fmin(ln_lh3 - ln_ll3, 600.0)));
    double gain = g1 + g4, loss = l2 + l3;
    if (ion) {
        gain += 1.92e-28 * g.n;
        loss += 2.18e-11 * rate_k6(g.T) * g.nH * g.ne;
    }
    return gain - loss;
}

// explicit Euler step of the internal energy over dt with Gamma - Lambda
// frozen; energy unit n_unit k_B T_unit; cooling stops at the internal energy
// of 10 K, or at e where the cell is already colder
__device__ __forceinline__ double cooled_e(const ChemArgs& ch, double gamma, double rho, double e, double h2, double hp,
                                           double dt)
{
    const Gas g = gas_state(ch, gamma, rho, e, h2, hp);
    const double de = dt * ch.e_rate * heat_cool(ch.ion, g);
    const double efloor = quot(10.0 * (rho - 0.5 * h2 + hp), ch.T_unit * (gamma - 1.0));
    const double lo = e < efloor ? e : efloor;
    const double en = e + de;
    return en < lo ? lo : en;
}

// Sec. 2.7 with reactions 1-8 (ionisation network): semi-implicit updates of
// n_H2 and n_H+ = n_e from the state at the start of the step, n_H = n_u (rho
// - h2 - hp); H2 clamped to [0, n_u (rho - hp) / 2], then H+ to [0, n_u (rho -
// h2')]; temperature from gamma_eff and the mean mass 1 / (1 - x_H2/2 + x_H+)
__device__ __forceinline__ void chem_ion(const ChemArgs& ch, double rho, double e, double h2, double hp, double dt,
                                         double& h2_out, double& hp_out)
{
    const Gas g = gas_state(ch, gamma_cell(1, 0.0, rho, h2, hp), rho, e, h2, hp);
    const double ts = dt * ch.t_unit;
    double num, den;
    formation(g, num, den);
    double m2 = semi_implicit(g.nH2, quot(num, den), h2_loss(g), ts);
    const double m2max = ch.n_unit * (rho - hp) / 2.0;
    m2 = m2 > m2max ? m2max : m2;
    m2 = m2 < 0.0 ? 0.0 : m2;
    const double lnT = log(g.T);
    const double Ci = 6e-18 * g.nH + rate_k6(g.T) * g.nH * g.ne;
    const double Di = (rate_k7(lnT) + rate_k8(lnT)) * g.ne;
    double mi = semi_implicit(g.ne, Ci, Di, ts);
    const double h2n = 2.0 * quot(m2, ch.n_unit, ch.n_inv);
    const double mimax = ch.n_unit * (rho - h2n);
    mi = mi > mimax ? mimax : mi;
    mi = mi < 0.0 ? 0.0 : mi;
    h2_out = h2n;
    hp_out = quot(mi, ch.n_unit, ch.n_inv);
}

// Sec. 2.3: the speed sum of the CFL rule for one cell (FP64), v + b + c + c_a
// + c_s + c_f; c_f^2 + c_s^2 = c^2 + b^2 and c_f c_s = c c_a, so c_f + c_s =
// sqrt(c^2 + b^2 + 2 c c_a), without the differences of the two speeds
__device__ __forceinline__ double cell_speed(double gamma, double rho, double mx, double my, double mz, double e,
                                             double bx, double by, double bz)
{
    const double rs = rsqrt_nr(rho);   // 1 / sqrt(rho)
    // the velocities are squared, not the momenta, whose squares leave the range
    // in units of very large or very small density
    const double ir = rs * rs, vx = mx * ir, vy = my * ir, vz = mz * ir;
    const double v = root_nr(vx * vx + vy * vy + vz * vz);
    const double c = root_nr(gamma * ((gamma - 1.0) * e)) * rs;
    const double ca = fabs(bx) * rs;
    const double b = root_nr(bx * bx + by * by + bz * bz) * rs;
    const double s = v + b + c + ca + root_nr(c * c + b * b + 2.0 * c * ca);
    // squares beyond the range of the refined roots: no step is short enough
    return s <= 1e300 ? s : INFINITY;
}

__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        double o = __shfl_xor(v, off, 64);
        v = o > v ? o : v;
    }
    return v;
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

template <int NT = NTH>
__device__ __forceinline__ void block_max_store(double v, double* out, int blk)
{
    __shared__ double red[NT / 64];
    v = wave_max(v);
    int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) red[wv] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = red[0];
        for (int w = 1; w < NT / 64; w++) m = red[w] > m ? red[w] : m;
        out[blk] = m;
    }
}


}  // namespace mhd
