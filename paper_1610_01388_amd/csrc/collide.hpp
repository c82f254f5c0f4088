// collide.hpp -- node-local physics of the GPU library: moments, the
// Papanastasiou-regularised (PR) and implicitly-regularised (IR) collision of
// Regulski, Leonardi & Szumbarski (arXiv:1610.01388).
//
// All functions work on deviations h_i = f_i - w_i rho0 of the transformed
// populations (Sec. 2, Eq. 11), which keeps the small non-equilibrium
// moments accurate in reduced precision.  With Pi' = sum c c h the moments
// are rho = rho0 + sum h, j = sum c h, Pi = Pi' + rho0 cs^2 I.
#pragma once

#include <hip/hip_runtime.h>

#include "lattice.hpp"

namespace lbm {

// PR: Papanastasiou-regularised with the explicit relaxation-time update
// (the strain rate uses the previous step's tau, kept per node); IR:
// implicitly regularised; PRI: PR with the implicit update of Sec. 3 (the
// tau consistent with its own strain rate, found per node; no state);
// IRHB: the IR construction for a Herschel-Bulkley fluid (K = nu_p, flow
// index n), its collision moment found per node (Sec. 3.2).
// OP_MRT is a flag on PR and PRI: MRT base collision (Sec. 2.1) instead of
// TRT, a separate kernel instantiation so that the TRT kernels do not carry
// its registers.  OP_FB, for FP32 / FP16 storage only, compiles in the FP64
// redo of near-yield nodes (without it the reduced-precision kernels carry
// no FP64 registers).
enum { OP_PR = 0, OP_IR = 1, OP_PRI = 2, OP_IRHB = 3, OP_MRT = 4, OP_FB = 8 };
__host__ __device__ constexpr int op_base(int op) { return op & 3; }
// TRT (or MRT) + EDM with a Papanastasiou viscosity
__host__ __device__ constexpr bool pr_family(int op) { return op_base(op) == OP_PR || op_base(op) == OP_PRI; }
// carries a relaxation-time field from step to step
__host__ __device__ constexpr bool has_tau(int op) { return op_base(op) == OP_PR; }
__host__ __device__ constexpr bool is_mrt(int op) { return (op & OP_MRT) != 0; }

__device__ __forceinline__ double d_sqrt(double v) { return sqrt(v); }
__device__ __forceinline__ float d_sqrt(float v) { return sqrtf(v); }
__device__ __forceinline__ double d_expm1(double v) { return expm1(v); }
__device__ __forceinline__ float d_expm1(float v) { return expm1f(v); }

// Per-launch constants in compute precision C.
template <class C> struct Coll {
    C rho0, nu_p, sigma_y, m, gamma_c, lambda, g[3];
    C sqrt2_sy;   // sqrt(2) sigma_y: IR yield threshold on |dev T|
    C ir_a, ir_b; // IR yielded: lambda = ir_a + ir_b / T, ir_a = (6nu_p-1)/(1+6nu_p),
                  // ir_b = 2 sqrt2 sigma_y/(1+6nu_p)  (Eqs. 39-40 combined)
    C pr_ec;      // PR: -expm1(-m gamma_c) / gamma_c  (nu_app at the cut-off is nu_p + sigma_y pr_ec / rho)
    C band;       // FP64 fallback band
    int axis;     // 0, or 1..3: known flow axis whose normal component the collision drops (Sec. 4.2.2)
    C mrt_b, mrt_e;  // MRT rates of the bulk moment and of the even moments of order >= 4 (<= 0: shear rate)
    C hb_n, hb_c;    // IRHB: flow index n and 3 K (3/sqrt 2)^(n-1)
};

template <class C> struct Moments {
    C drho, j[3];
    C p[6];  // Pi' = sum c c h: xx, yy, zz, xy, xz, yz
};

// Node state after the rheology solve, before relaxation.
template <class C> struct Pre {
    C rho, u[3];  // u: velocity inside the equilibrium (PR: j/rho; IR: j/rho + g/2)
    C a[6];       // IR: post-collision stress tensor A = lambda dev(T)
    C tau_p, tau_m, om_m, nu_app, gamma, Tn;
    bool unyielded, near_yield;
};

template <int LAT, class C>
__device__ __forceinline__ void add_c(C& acc, C v, int c)
{
    if (c == 1) acc += v;
    else if (c == -1) acc -= v;
}

// Eq. 9: zeroth, first and second moments (of the deviations).
// Accumulated in C from populations stored as H (the FP64 redo of a
// reduced-precision node sums its float values in double, no double copy).
// The velocities come in opposite pairs (i, i + 1 for odd i): the pair's sum
// carries the even moments (rho, Pi) and its difference the odd one (j), so
// each pair is combined once.
template <int LAT, class C, class H>
__device__ __forceinline__ Moments<C> moments_as(const H (&h)[Lattice<LAT>::Q])
{
    using L = Lattice<LAT>;
    Moments<C> mo;
    mo.drho = (C)h[0];
#pragma unroll
    for (int a = 0; a < 3; ++a) mo.j[a] = 0;
#pragma unroll
    for (int a = 0; a < 6; ++a) mo.p[a] = 0;
#pragma unroll
    for (int i = 1; i < L::Q; i += 2) {
        const C hp = (C)h[i], hm = (C)h[i + 1];
        const C sum = hp + hm, dif = hp - hm;
        mo.drho += sum;
        add_c<LAT>(mo.j[0], dif, L::cx[i]);
        add_c<LAT>(mo.j[1], dif, L::cy[i]);
        add_c<LAT>(mo.j[2], dif, L::cz[i]);
        add_c<LAT>(mo.p[0], sum, L::cx[i] * L::cx[i]);
        add_c<LAT>(mo.p[1], sum, L::cy[i] * L::cy[i]);
        add_c<LAT>(mo.p[2], sum, L::cz[i] * L::cz[i]);
        add_c<LAT>(mo.p[3], sum, L::cx[i] * L::cy[i]);
        add_c<LAT>(mo.p[4], sum, L::cx[i] * L::cz[i]);
        add_c<LAT>(mo.p[5], sum, L::cy[i] * L::cz[i]);
    }
    return mo;
}

// Classes of velocities: face pairs 1 + 2 a along axis a; in each plane (a, b)
// of axes (x y, then x z and y z in 3-D) the edge pairs +a+b and +a-b; in
// D3Q27 the corner pairs +++, ++-, +-+, -++.  FP64 forms moments and
// post-collision values class by class: the sums that a plane's or the
// corners' pairs share are taken once, and the weight is the class's (D3Q27:
// 81 operations for the moments and 110 for IR's post-collision values, where
// the direction-wise form takes 137 and 190; TRT 160 for 364).  Rounding
// differs from the direction-wise form at 1e-15; FP32 and FP16 keep that one
// and with it their states bit for bit (there the class form gained 1 to 3%,
// their kernels being bound by memory).
template <int LAT> constexpr int kPlanes = Lattice<LAT>::D == 3 ? 3 : 1;
template <int LAT> constexpr int edge0(int plane) { return (Lattice<LAT>::D == 3 ? 7 : 5) + 4 * plane; }
constexpr int plane_a(int p) { return p == 2 ? 1 : 0; }
constexpr int plane_b(int p) { return p == 0 ? 1 : 2; }
constexpr int kCorner0 = 19;

template <int LAT, class C>
__device__ __forceinline__ Moments<C> moments_by_class(const C (&h)[Lattice<LAT>::Q])
{
    using L = Lattice<LAT>;
    constexpr int D = L::D;
    Moments<C> mo;
#pragma unroll
    for (int a = 0; a < 3; ++a) mo.j[a] = 0;
#pragma unroll
    for (int a = 0; a < 6; ++a) mo.p[a] = 0;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        mo.p[a] = h[1 + 2 * a] + h[2 + 2 * a];
        mo.j[a] = h[1 + 2 * a] - h[2 + 2 * a];
    }
    C all = mo.p[0] + mo.p[1];  // sum over the moving velocities
    if (D == 3) all += mo.p[2];
#pragma unroll
    for (int e = 0; e < kPlanes<LAT>; ++e) {
        const int i = edge0<LAT>(e), a = plane_a(e), b = plane_b(e);
        const C sp = h[i] + h[i + 1], dp = h[i] - h[i + 1];
        const C sm = h[i + 2] + h[i + 3], dm = h[i + 2] - h[i + 3];
        const C both = sp + sm;
        mo.p[a] += both;
        mo.p[b] += both;
        all += both;
        mo.p[3 + e] = sp - sm;
        mo.j[a] += dp + dm;
        mo.j[b] += dp - dm;
    }
    if constexpr (L::Q == 27) {
        constexpr int i = kCorner0;
        const C s1 = h[i] + h[i + 1], d1 = h[i] - h[i + 1];          // + + +
        const C s2 = h[i + 2] + h[i + 3], d2 = h[i + 2] - h[i + 3];  // + + -
        const C s3 = h[i + 4] + h[i + 5], d3 = h[i + 4] - h[i + 5];  // + - +
        const C s4 = h[i + 6] + h[i + 7], d4 = h[i + 6] - h[i + 7];  // - + +
        const C s12 = s1 + s2, t12 = s1 - s2, s34 = s3 + s4, t34 = s3 - s4;
        const C four = s12 + s34;
        mo.p[0] += four;
        mo.p[1] += four;
        mo.p[2] += four;
        all += four;
        mo.p[3] += s12 - s34;
        mo.p[4] += t12 + t34;
        mo.p[5] += t12 - t34;
        const C d12 = d1 + d2, d34 = d3 - d4;
        mo.j[0] += d12 + d34;
        mo.j[1] += d12 - d34;
        mo.j[2] += (d1 - d2) + (d3 + d4);
    }
    mo.drho = all + h[0];
    return mo;
}

template <int LAT, class C>
__device__ __forceinline__ Moments<C> moments(const C (&h)[Lattice<LAT>::Q])
{
    if constexpr (sizeof(C) == 8) return moments_by_class<LAT, C>(h);
    else return moments_as<LAT, C, C>(h);
}

// Non-equilibrium second moment Pi - rho cs^2 I - rho v v, from the
// deviation moments: Pi' - drho cs^2 I_d - rho v v.
template <int LAT, class C>
__device__ __forceinline__ void noneq_second(const Moments<C>& mo, C rho, const C (&v)[3], C (&t)[6])
{
    constexpr int D = Lattice<LAT>::D;
    const C third = C(1) / C(3);
    t[0] = mo.p[0] - mo.drho * third - rho * v[0] * v[0];
    t[1] = mo.p[1] - mo.drho * third - rho * v[1] * v[1];
    t[2] = (D == 3) ? mo.p[2] - mo.drho * third - rho * v[2] * v[2] : C(0);
    t[3] = mo.p[3] - rho * v[0] * v[1];
    t[4] = (D == 3) ? mo.p[4] - rho * v[0] * v[2] : C(0);
    t[5] = (D == 3) ? mo.p[5] - rho * v[1] * v[2] : C(0);
}

template <class C>
__device__ __forceinline__ C frob2(const C (&t)[6])
{
    return t[0] * t[0] + t[1] * t[1] + t[2] * t[2] + C(2) * (t[3] * t[3] + t[4] * t[4] + t[5] * t[5]);
}

// PRI: the relaxation time tau with tau = 1/2 + 3 nu_app(G / tau), G being
// the strain rate Eq. 24 gives at tau = 1.  F(tau) = tau - 1/2 - 3 nu_app(G /
// tau) is convex in tau and changes sign once on [1/2 + 3 nu_p, 1/2 + 3
// nu_0]; Newton's method, kept inside the shrinking bracket (bisection
// whenever a step would leave it), stops when a step is below the
// precision's resolution.  It starts at the root of the yielded asymptote
// when that lies in the bracket, else at the upper end.
template <class C>
__device__ __forceinline__ C implicit_tau(C G, const Coll<C>& p, C irho)
{
    const C s = p.sigma_y * irho;
    const C nu0 = p.nu_p + p.m * s;
    const C nuc = p.nu_p + s * p.pr_ec;
    C lo = C(0.5) + C(3) * p.nu_p;
    C hi = C(0.5) + C(3) * nu0;
    // Start: where the root lies once m gamma is large (yielded node,
    // nu_app ~ nu_p + s tau / G, linear in tau), else the upper end.
    const C r = C(3) * s;
    C x = hi;
    if (r < G) x = fmin(fmax(lo * G / (G - r), lo), hi);
    const C tol = sizeof(C) == 8 ? C(1e-14) : C(2e-7);
    for (int it = 0; it < 64; ++it) {
        const C gam = G / x;
        C nu, dnu;  // nu_app(gam) and d nu_app / d gam
        if (gam >= p.gamma_c) {
            const C em = -d_expm1(-p.m * gam);  // 1 - exp(-m gam)
            nu = p.nu_p + s * em / gam;
            dnu = s / gam * (p.m * (C(1) - em) - em / gam);
        } else {
            nu = nu0 + (gam / p.gamma_c) * (nuc - nu0);
            dnu = (nuc - nu0) / p.gamma_c;
        }
        const C F = x - C(0.5) - C(3) * nu;
        if (F > C(0)) hi = x;
        else lo = x;
        const C dF = C(1) + C(3) * dnu * G / (x * x);
        const C step = F / dF;
        C xn = x - step;
        // A step within tolerance ends the search before the bracket test:
        // at an exact root (F = 0) x has just become a bracket end, and the
        // strict test would send the next iterate off to the midpoint.
        const bool conv = fabs(step) <= tol * x;
        if (!conv && !(xn > lo && xn < hi)) xn = C(0.5) * (lo + hi);
        const bool done = conv || hi - lo <= tol * hi;
        x = xn;
        if (done) break;
    }
    return x;
}

__device__ __forceinline__ double d_pow(double b, double e) { return pow(b, e); }
__device__ __forceinline__ float d_pow(float b, float e) { return powf(b, e); }

// IRHB: magnitude s of the collision's second moment for a yielded node
// (Tn > sqrt(2) sigma_y).  The Herschel-Bulkley law written in s with the
// strain rate 3 s / sqrt(2) turns the contraction of Eq. 31 into
// F(s) = s/2 + c s^n + sqrt(2) sigma_y - Tn = 0, c = 3 K (3/sqrt 2)^(n-1):
// increasing in s and negative at 0; with e = Tn - sqrt(2) sigma_y the root
// lies below both 2 e (from s/2 <= e) and (e / c)^(1/n) (from c s^n <= e),
// the second bound close to it when the power term dominates (small n).
// Newton's method kept inside the shrinking bracket (bisection whenever a
// step would leave it) from the n = 1 closed form (exact for Bingham), until
// a step falls below the precision's resolution.  A bound that underflows
// to zero returns zero (s is then negligible against Tn).
//
// In FP64 the search starts from a root found in single precision by the same
// rule (fast base-2 powers), good to about 1e-6, and ends with the first step
// below 1e-9 x: Newton's error after a step d is about (n - 1)/2 (d/x)^2 x, so
// that step lands within 1e-17 of the root.  Two evaluations of the FP64 power
// instead of six or seven (one of them for the bound).
__device__ __forceinline__ float fast_powf(float b, float e) { return __builtin_amdgcn_exp2f(e * __builtin_amdgcn_logf(b)); }

__device__ __forceinline__ float hb_start(float e, float c, float n)
{
    float lo = 0.0f, hi = fminf(2.0f * e, fast_powf(e / c, 1.0f / n) * 1.0001f);
    float x = fminf(e / (0.5f + c), hi);
    for (int it = 0; it < 12; ++it) {
        const float xn1 = fast_powf(x, n - 1.0f);
        const float F = 0.5f * x + c * xn1 * x - e;
        if (F > 0.0f) hi = x;
        else lo = x;
        const float step = F / (0.5f + c * n * xn1);
        float xn = x - step;
        const bool conv = fabsf(step) <= 3e-6f * x;
        if (!conv && !(xn > lo && xn < hi)) xn = 0.5f * (lo + hi);
        x = xn;
        if (conv) break;
    }
    return x;
}

template <class C>
__device__ __forceinline__ C hb_moment(C Tn, const Coll<C>& p)
{
    const C e = Tn - p.sqrt2_sy;
    C lo = C(0), hi, x;
    const C tol = sizeof(C) == 8 ? C(1e-14) : C(2e-7);
    const C last = sizeof(C) == 8 ? C(1e-9) : tol;  // a step this small ends the search
    if constexpr (sizeof(C) == 8) {
        hi = C(2) * e;
        if (!(hi > C(0))) return C(0);
        x = (C)hb_start((float)e, (float)p.hb_c, (float)p.hb_n);
        if (!(x > C(1e-30))) {  // below the float range: the bound and start of FP32, in double
            hi = fmin(hi, d_pow(e / p.hb_c, C(1) / p.hb_n));
            if (!(hi > C(0))) return C(0);
            x = fmin(e / (C(0.5) + p.hb_c), hi);
        } else if (!(x < hi)) {
            x = C(0.5) * hi;
        }
    } else {
        hi = fmin(C(2) * e, d_pow(e / p.hb_c, C(1) / p.hb_n));
        if (!(hi > C(0))) return C(0);
        x = fmin(e / (C(0.5) + p.hb_c), hi);
    }
    for (int it = 0; it < 64; ++it) {
        const C xn1 = d_pow(x, p.hb_n - C(1));  // s^(n-1); x > 0 here
        const C F = C(0.5) * x + p.hb_c * xn1 * x - e;
        if (F > C(0)) hi = x;
        else lo = x;
        const C step = F / (C(0.5) + p.hb_c * p.hb_n * xn1);
        C xn = x - step;
        const bool conv = fabs(step) <= last * x;
        if (!conv && !(xn > lo && xn < hi)) xn = C(0.5) * (lo + hi);
        const bool done = conv || hi - lo <= tol * hi;
        x = xn;
        if (done) break;
    }
    return x;
}

// Rheology: everything up to, but not including, the relaxation.
//  PR (Sec. 2.2 Eq. 24, Sec. 3.1 Eqs. 36-37, Sec. 2.1): D from the
//   non-equilibrium second moment at the bare velocity with the previous
//   step's tau (density kept, as in Eq. 33), gamma = sqrt(2 D:D) on the full
//   tensor, nu_app with the linear interpolation below gamma_c (denominator
//   gamma_c), tau_even = 1/2 + 3 nu_app, tau_odd from Lambda.
//  PRI: as PR with tau_prev replaced by implicit_tau.
//  IR (Sec. 2.3, 3.2): T = sum c c (f - f_eq + Phi/2) at u = (j + F/2)/rho,
//   deviatoric part (trace / d), yielded iff |dev T| > sqrt(2) sigma_y,
//   A = -sigma + s/2 = lambda dev T with the closed forms of Eqs. 39-40.
template <int LAT, int OP, class C>
__device__ __forceinline__ Pre<C> rheology(const Moments<C>& mo, const Coll<C>& p, C tau_prev)
{
    constexpr int D = Lattice<LAT>::D;
    Pre<C> r;
    r.rho = p.rho0 + mo.drho;
    const C irho = C(1) / r.rho;
    if (pr_family(OP)) {
#pragma unroll
        for (int a = 0; a < 3; ++a) r.u[a] = mo.j[a] * irho;
        C t[6];
        noneq_second<LAT>(mo, r.rho, r.u, t);
        C tau_s = tau_prev;
        if (op_base(OP) == OP_PRI) {  // strain rate at tau = 1, then the self-consistent tau
            const C c1 = C(-1.5) * irho;
            C d1[6];
#pragma unroll
            for (int a = 0; a < 6; ++a) d1[a] = c1 * t[a];
            if (p.axis == 1) d1[0] = C(0);
            if (p.axis == 2) d1[1] = C(0);
            if (p.axis == 3) d1[2] = C(0);
            tau_s = implicit_tau(d_sqrt(C(2) * frob2(d1)), p, irho);
        }
        const C coef = C(-1.5) / (r.rho * tau_s);  // -1 / (2 rho cs^2 tau)
        C dd[6];
#pragma unroll
        for (int a = 0; a < 6; ++a) dd[a] = coef * t[a];
        if (is_mrt(OP) && p.mrt_b > C(0)) {
            // Eq. 23 with MRT: the trace part relaxes at the bulk rate
            const C trd = ((D == 3) ? t[0] + t[1] + t[2] : t[0] + t[1]) / C(D);
            const C corr = C(-1.5) * irho * (p.mrt_b - C(1) / tau_s) * trd;
            dd[0] += corr;
            dd[1] += corr;
            if (D == 3) dd[2] += corr;
        }
        if (is_mrt(OP)) {
#pragma unroll
            for (int a = 0; a < 6; ++a) r.a[a] = t[a];  // non-equilibrium second moment
        }
        // known flow axis: its normal strain rate is a Burnett-order artefact
        if (p.axis == 1) dd[0] = C(0);
        if (p.axis == 2) dd[1] = C(0);
        if (p.axis == 3) dd[2] = C(0);
        const C gamma = d_sqrt(C(2) * frob2(dd));
        C nu;
        if (gamma >= p.gamma_c) {
            nu = p.nu_p + p.sigma_y * irho * (-d_expm1(-p.m * gamma)) / gamma;
        } else {
            const C nu0 = p.nu_p + p.m * p.sigma_y * irho;
            const C nuc = p.nu_p + p.sigma_y * irho * p.pr_ec;
            nu = nu0 + (gamma / p.gamma_c) * (nuc - nu0);
        }
        r.nu_app = nu;
        r.gamma = gamma;
        r.tau_p = C(0.5) + C(3) * nu;
        r.tau_m = C(0.5) + p.lambda / (r.tau_p - C(0.5));
        // 1 / tau_m, with tau_p - 1/2 = 3 nu
        r.om_m = sizeof(C) == 8 ? (C(3) * nu) / (C(1.5) * nu + p.lambda) : C(1) / r.tau_m;
        // the regularised stress magnitude sqrt(sigma:sigma / 2) = rho nu gamma
        // against the yield stress: unyielded below it, redone in FP64 (when
        // enabled) within the band around it
        const C stress = r.rho * nu * gamma;
        r.unyielded = stress < p.sigma_y;
        r.near_yield = p.sigma_y > C(0) && fabs(stress - p.sigma_y) < p.band * p.sigma_y;
        r.Tn = 0;
    } else {
#pragma unroll
        for (int a = 0; a < 3; ++a) r.u[a] = mo.j[a] * irho + C(0.5) * p.g[a];
        C t[6];
        noneq_second<LAT>(mo, r.rho, r.u, t);
        // known flow axis: drop its normal component before the deviator
        if (p.axis == 1) t[0] = C(0);
        if (p.axis == 2) t[1] = C(0);
        if (p.axis == 3) t[2] = C(0);
        const C tr = (D == 3) ? t[0] + t[1] + t[2] : t[0] + t[1];
        const C trd = sizeof(C) == 8 ? tr * (C(1) / C(D)) : tr / C(D);
        t[0] -= trd;
        t[1] -= trd;
        if (D == 3) t[2] -= trd;
        const C Tn = d_sqrt(frob2(t));
        const bool yielded = Tn > p.sqrt2_sy;
        C lam = C(1);
        if (yielded) {
            if constexpr (op_base(OP) == OP_IRHB) lam = C(1) - hb_moment(Tn, p) / Tn;
            else lam = p.ir_a + p.ir_b / Tn;
        }
#pragma unroll
        for (int a = 0; a < 6; ++a) r.a[a] = lam * t[a];
        r.Tn = Tn;
        r.unyielded = !yielded;
        r.near_yield = p.sigma_y > C(0) && fabs(Tn - p.sqrt2_sy) < p.band * p.sqrt2_sy;
        r.tau_p = tau_prev;
        r.tau_m = r.om_m = tau_prev;
        r.nu_app = p.nu_p;
        r.gamma = 0;
    }
    return r;
}

// Values of an even quadratic form and an odd linear form on the velocities:
// visit(i, E, O) is called for each opposite pair (i, i + 1) with E = e0 + M :
// c c and O = B . c, c the velocity i; m holds xx, yy, zz and twice xy, xz, yz.
template <int LAT, class C, class F>
__device__ __forceinline__ void pair_forms(C e0, const C (&m)[6], const C (&v)[3], F&& visit)
{
    using L = Lattice<LAT>;
#pragma unroll
    for (int a = 0; a < L::D; ++a) visit(1 + 2 * a, e0 + m[a], v[a]);
#pragma unroll
    for (int p = 0; p < kPlanes<LAT>; ++p) {
        const int i = edge0<LAT>(p), a = plane_a(p), b = plane_b(p);
        const C base = e0 + (m[a] + m[b]);
        visit(i, base + m[3 + p], v[a] + v[b]);
        visit(i + 2, base - m[3 + p], v[a] - v[b]);
    }
    if constexpr (L::Q == 27) {
        const C base = e0 + (m[0] + m[1] + m[2]);
        const C up = base + m[3], dn = base - m[3];
        const C zp = m[4] + m[5], zm = m[4] - m[5];
        const C vp = v[0] + v[1], vm = v[0] - v[1];
        visit(kCorner0, up + zp, vp + v[2]);      // + + +
        visit(kCorner0 + 2, up - zp, vp - v[2]);  // + + -
        visit(kCorner0 + 4, dn + zm, vm + v[2]);  // + - +
        visit(kCorner0 + 6, dn - zm, v[2] - vm);  // - + +
    }
}

// Relaxation class by class (TRT and IR; see relax).
//  TRT: the EDM difference is absorbed in the state relaxed to: with E and O the
//   even and odd parts of h_eq + tau (f_eq(u + g) - f_eq(u)) (tau_p for the
//   even, tau_m for the odd part), h_i += om_p (E - even) + om_m (O - odd), the
//   changes small against h_i.
template <int LAT, int OP, class C>
__device__ __forceinline__ void relax_by_class(C (&h)[Lattice<LAT>::Q], const Moments<C>& mo, const Pre<C>& r,
                                               const Coll<C>& p)
{
    using L = Lattice<LAT>;
    const C* u = r.u;
    const C rho15 = C(1.5) * r.rho, rho45 = C(4.5) * r.rho, rho3 = C(3) * r.rho;
    if constexpr (pr_family(OP)) {
        const C om_p = C(1) / r.tau_p;
        C tg[3], s[3], B[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            tg[a] = r.tau_p * p.g[a];
            s[a] = u[a] + p.g[a];
            B[a] = rho3 * (u[a] + r.tau_m * p.g[a]);
        }
        // u u + tau_p (u g + g u + g g)
        const C q0 = u[0] * (u[0] + tg[0]) + tg[0] * s[0];
        const C q1 = u[1] * (u[1] + tg[1]) + tg[1] * s[1];
        const C q2 = u[2] * (u[2] + tg[2]) + tg[2] * s[2];
        const C rho9 = C(9) * r.rho;
        const C M[6] = {rho45 * q0, rho45 * q1, rho45 * q2,
                        rho9 * (u[0] * (u[1] + tg[1]) + tg[0] * s[1]),
                        rho9 * (u[0] * (u[2] + tg[2]) + tg[0] * s[2]),
                        rho9 * (u[1] * (u[2] + tg[2]) + tg[1] * s[2])};
        const C e0 = mo.drho - rho15 * (q0 + q1 + q2);
        h[0] += om_p * (C(L::w[0]) * e0 - h[0]);
        const C hp = C(0.5) * om_p, hm = C(0.5) * r.om_m;
        pair_forms<LAT>(e0, M, B, [&](int i, C E, C O) {
            const C w2 = C(2 * L::w[i]);
            C hi = h[i], hk = h[i + 1];
            // form the pair's sum and difference again instead of holding those
            // of the moments (two registers each per pair); no instruction
            asm("" : "+v"(hi), "+v"(hk));
            const C x = hp * (w2 * E - (hi + hk)), y = w2 * O - (hi - hk);
            h[i] = hi + (x + hm * y);
            h[i + 1] = hk + (x - hm * y);
        });
    } else {
        const C* A = r.a;
        const C uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
        const C ru[3] = {rho45 * u[0], rho45 * u[1], rho45 * u[2]};
        const C M[6] = {ru[0] * u[0] + C(4.5) * A[0], ru[1] * u[1] + C(4.5) * A[1], ru[2] * u[2] + C(4.5) * A[2],
                        C(2) * (ru[0] * u[1] + C(4.5) * A[3]), C(2) * (ru[0] * u[2] + C(4.5) * A[4]),
                        C(2) * (ru[1] * u[2] + C(4.5) * A[5])};
        const C B[3] = {rho3 * u[0] + rho15 * p.g[0], rho3 * u[1] + rho15 * p.g[1], rho3 * u[2] + rho15 * p.g[2]};
        const C e0 = mo.drho - rho15 * uu - C(1.5) * (A[0] + A[1] + A[2]);
        h[0] = C(L::w[0]) * e0;
        pair_forms<LAT>(e0, M, B, [&](int i, C E, C O) {
            const C w = C(L::w[i]), wo = w * O;
            h[i] = w * E + wo;
            h[i + 1] = w * E - wo;
        });
    }
}

// Relaxation: overwrite h with the post-collision deviations.
//  PR: TRT on the even/odd parts of h - h_eq, plus the EDM difference
//   f_eq(u + g) - f_eq(u) written out (Sec. 2.4, Eq. 34).
//  IR: f_eq(u) + f_sigma + Phi/2 with f_sigma = w/(2 cs^4)(c c - cs^2 I):A
//   and Phi = 3 w c.F, F = rho g (Sec. 2.3 Eqs. 28-29, Sec. 2.4 Eq. 35).
// Computed in C, read from and written to populations stored as H (H = C
// except in the FP64 redo of a reduced-precision node).
template <int LAT, int OP, class C, class H>
__device__ __forceinline__ void relax(H (&h)[Lattice<LAT>::Q], const Moments<C>& mo, const Pre<C>& r,
                                      const Coll<C>& p)
{
    if constexpr (sizeof(H) == 8 && !is_mrt(OP)) {
        relax_by_class<LAT, OP>(h, mo, r, p);
        return;
    }
    using L = Lattice<LAT>;
    const C* u = r.u;
    const C uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    if (pr_family(OP)) {
        const C om_p = C(1) / r.tau_p;
        const C om_m = r.om_m;
        // MRT (Sec. 2.1): with the weights' inner product the second-order
        // Hermite projection of h - h_eq splits into shear (cc : Pi_dev) and
        // bulk ((tr/d)(|c|^2 - d cs^2)) parts; the remaining even moments take
        // om_e, the odd ones om_m:  even change = om_e n_s + (om_p - om_e) f2d
        // + (om_b - om_e) f2b.  Without MRT, om_e = om_b = om_p (TRT).
        constexpr bool mrt = is_mrt(OP);
        const C om_e = (mrt && p.mrt_e > C(0)) ? p.mrt_e : om_p;
        const C om_b = (mrt && p.mrt_b > C(0)) ? p.mrt_b : om_p;
        constexpr int D = L::D;
        const C* pn = r.a;
        const C trd = ((D == 3) ? pn[0] + pn[1] + pn[2] : pn[0] + pn[1]) / C(D);
        const C dsh = om_p - om_e, dbu = om_b - om_e;
        const C ug = p.g[0] * (C(2) * u[0] + p.g[0]) + p.g[1] * (C(2) * u[1] + p.g[1]) +
                     p.g[2] * (C(2) * u[2] + p.g[2]);
        {  // rest velocity: symmetric only (f2d = 0, f2b = -cs^2 d trd * 9/2 w = -1.5 w d trd)
            const C w = C(L::w[0]);
            const C es = w * (mo.drho - C(1.5) * r.rho * uu);
            const C h0 = (C)h[0];
            C ns0 = om_e * (h0 - es);
            if (mrt) ns0 += dbu * (C(-1.5) * w * C(D) * trd);
            h[0] = (H)(h0 - ns0 - C(1.5) * r.rho * w * ug);
        }
#pragma unroll
        for (int i = 1; i < L::Q; i += 2) {
            const int k = i + 1;
            const C w = C(L::w[i]);
            C cu = 0, cg = 0;
            add_c<LAT>(cu, u[0], L::cx[i]);
            add_c<LAT>(cu, u[1], L::cy[i]);
            add_c<LAT>(cu, u[2], L::cz[i]);
            add_c<LAT>(cg, p.g[0], L::cx[i]);
            add_c<LAT>(cg, p.g[1], L::cy[i]);
            add_c<LAT>(cg, p.g[2], L::cz[i]);
            const C es = w * (mo.drho + r.rho * (C(4.5) * cu * cu - C(1.5) * uu));
            const C ea = C(3) * w * r.rho * cu;
            const C hi = (C)h[i], hk = (C)h[k];
            const C hs = C(0.5) * (hi + hk);
            const C ha = C(0.5) * (hi - hk);
            C ns = om_e * (hs - es);
            if (mrt) {
                C cpc = 0;  // c c : Pi_neq
                add_c<LAT>(cpc, pn[0], L::cx[i] * L::cx[i]);
                add_c<LAT>(cpc, pn[1], L::cy[i] * L::cy[i]);
                add_c<LAT>(cpc, pn[2], L::cz[i] * L::cz[i]);
                add_c<LAT>(cpc, C(2) * pn[3], L::cx[i] * L::cy[i]);
                add_c<LAT>(cpc, C(2) * pn[4], L::cx[i] * L::cz[i]);
                add_c<LAT>(cpc, C(2) * pn[5], L::cy[i] * L::cz[i]);
                const int c2 = L::cx[i] * L::cx[i] + L::cy[i] * L::cy[i] + L::cz[i] * L::cz[i];
                const C f2d = C(4.5) * w * (cpc - trd * C(c2));
                const C f2b = C(4.5) * w * trd * (C(c2) - C(D) / C(3));
                ns += dsh * f2d + dbu * f2b;
            }
            const C na = om_m * (ha - ea);
            // f_eq(u+g) - f_eq(u) for +c and -c
            const C fs = r.rho * w * (C(4.5) * cg * (C(2) * cu + cg) - C(1.5) * ug);
            const C fa = r.rho * w * C(3) * cg;
            // the pair's post-collision symmetric and antisymmetric parts
            const C ps = hs - ns + fs, pa = ha - na + fa;
            h[i] = (H)(ps + pa);
            h[k] = (H)(ps - pa);
        }
    } else {
        // Per opposite pair (i, i + 1): the equilibrium's even part and the
        // stress term are shared, the odd part (velocity and force) changes
        // sign, so h_i = E + O and h_{i+1} = E - O.
        const C* A = r.a;
        const C trA = A[0] + A[1] + A[2];
        const C third = C(1) / C(3);
        const C trd = trA * third;
        const C even0 = mo.drho - C(1.5) * r.rho * uu;
        {
            const C w = C(L::w[0]);
            h[0] = (H)(w * even0 + C(4.5) * w * (C(0) - trd));
        }
        const C rho3 = C(3) * r.rho, rho15 = C(1.5) * r.rho, rho45 = C(4.5) * r.rho;
#pragma unroll
        for (int i = 1; i < L::Q; i += 2) {
            const C w = C(L::w[i]);
            C cu = 0, cg = 0;
            add_c<LAT>(cu, u[0], L::cx[i]);
            add_c<LAT>(cu, u[1], L::cy[i]);
            add_c<LAT>(cu, u[2], L::cz[i]);
            add_c<LAT>(cg, p.g[0], L::cx[i]);
            add_c<LAT>(cg, p.g[1], L::cy[i]);
            add_c<LAT>(cg, p.g[2], L::cz[i]);
            C cac = 0;
            add_c<LAT>(cac, A[0], L::cx[i] * L::cx[i]);
            add_c<LAT>(cac, A[1], L::cy[i] * L::cy[i]);
            add_c<LAT>(cac, A[2], L::cz[i] * L::cz[i]);
            add_c<LAT>(cac, C(2) * A[3], L::cx[i] * L::cy[i]);
            add_c<LAT>(cac, C(2) * A[4], L::cx[i] * L::cz[i]);
            add_c<LAT>(cac, C(2) * A[5], L::cy[i] * L::cz[i]);
            const C E = w * (even0 + rho45 * cu * cu) + C(4.5) * w * (cac - trd);
            const C O = w * (rho3 * cu + rho15 * cg);
            h[i] = (H)(E + O);
            h[i + 1] = (H)(E - O);
        }
    }
}

// Reported velocity j/rho + g/2 (both operators).
template <class C>
__device__ __forceinline__ void out_velocity(const Moments<C>& mo, const Pre<C>& r, const Coll<C>& p, C (&uo)[3])
{
    const C irho = C(1) / r.rho;
#pragma unroll
    for (int a = 0; a < 3; ++a) uo[a] = mo.j[a] * irho + C(0.5) * p.g[a];
}

}  // namespace lbm
