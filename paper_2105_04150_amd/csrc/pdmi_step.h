// pdmi_step.h -- the step kernels of the bond-based PMB peridynamics library (templates;
// each launcher file instantiates its share of them).
//
// One fused kernel per time step (paper Sec. 3: the bond force, the critical-stretch
// check and the per-node reduction are fused, Algorithm 2; here the time integration
// is fused too).  It reads displacement level k from one node-record buffer and writes
// level k+1 into the other, so no wavefront can observe a half-updated field (the race
// that forces the paper to keep integration in a separate kernel, Sec. 3.3).
//
// Mapping (sliced kernels): a wavefront serves one slice of W = 64/G nodes; each node's bonds
// are split over G lanes, each lane sums its bonds sequentially, and the G partial sums
// meet in a butterfly of cross-lane shuffles.  No atomics and no LDS: a node's force is
// owned by its slice and the result is deterministic.  The staged kernel is described at
// step_staged.
//
// Bond arithmetic (per slot b = (i, j), Eqs. microelastic and simpleBond):
//   xi = x_j - x_i,  eta = u_j - u_i,  y = xi + eta
//   q  = |y|^2/|xi|^2 - 1, the numerator as |y|^2 - |xi|^2, both sums in the same order
//   break when s >= s0, i.e. q >= (1 + s0)^2 - 1
//   f  = c s V_j y/|y| = c V_j (1/|xi|) (1 - (1+q)^(-1/2)) y
// The FP64 numerator cancels: q carries an absolute error of a few units of 2^-53 (plus
// 1e-14 relative from 1/|xi|), the same order as the rounding of the oracle's own
// (|y| - |xi|)/|xi|, and is exactly zero for an unstretched bond (y = xi).
// The sliced kernel sums 1 - (1+q)^(-1/2) as its binomial series for |q| < 4e-3, so the force
// adds no second cancellation; the staged kernel takes the same force from an even series
// about the mean square length (slot_mid).  Both carry about 1e-14 a slot beside the
// numerator's rounding.  The FP32 kernels keep the cancellation-free numerator
// eta.(xi + y): in single precision the difference of squares would lose most digits of
// a small stretch.
// The break decision is made on q except within a narrow margin around the threshold,
// where a rare branch recomputes s = (|y| - |xi|)/|xi| in the oracle's exact order of
// operations (stretch_exact): in the FP64 build, the same x and u break the same bonds
// whatever the rounding of the fast form.
//
// Every kernel also has a force-evaluation mode (kModeForce): the same gather at the
// current level, no breaking, the bond force density written out (the reaction-force
// readout of the quasi-static examples, Sec. 6).
//
// EXT variants carry the bond-model branch: no-failure zones and n-linear damage laws
// per bond class.  A slot over the instance's threshold (or already softened) takes a rare
// branch that asks its damage state for a weight w (breaking: w = 0): the sliced kernel's common
// path adds every live bond's elastic contribution and the branch moves it from 1 to w, the
// staged one leaves such slots out and adds w times theirs.  Problems without zones or laws
// run the plain kernels.
#pragma once

#include "pdmi_tile.h"

#include <type_traits>

namespace pdmi {
namespace {

// What the bond-model branch needs of a slot: its q and its elastic contribution
// coef * y to the force density.
struct SlotTerm {
    double q, coef, y0, y1, y2;
};
// Contribution of one slot.  live: the slot holds an intact bond; breakable: the bond may
// break in this pass (intact, outside the no-failure zones, not a force evaluation).
// (X, U) are the owner's position and displacement, p0..p2 the neighbour's node record,
// kv = stiffness times neighbour volume, q0 the lower edge of the break decision.  Adds
// the force density to F, except for a breakable slot at or above q0: for such a
// candidate the function returns true and leaves the decision (and, if the bond holds,
// its contribution) to the caller's rare branch.
__device__ __forceinline__ bool slot_force(bool live, bool breakable, const double2 p0, const double2 p1, const double2 p2,
                                           double X0, double X1, double X2, double U0, double U1, double U2,
                                           double kv, double q0, double& F0, double& F1, double& F2, SlotTerm& st,
                                           const SeriesCoef& sk = SeriesCoef())
{
    const double xi0 = p0.x - X0, xi1 = p0.y - X1, xi2 = p1.x - X2;
    const double e0 = p1.y - U0, e1 = p2.x - U1, e2 = p2.y - U2;
    const double y0 = xi0 + e0, y1 = xi1 + e1, y2 = xi2 + e2;
    const double L2 = __builtin_fma(xi2, xi2, __builtin_fma(xi1, xi1, xi0 * xi0));
    // |y|^2 - |xi|^2 with both squares summed in the same order: two fewer operations than
    // eta.(xi + y), an absolute error in q below 7e-16 (six orders of magnitude inside the
    // decision margin), and exactly zero when y = xi (a body at rest or rigidly translated
    // feels no bond force)
    const double Y2 = __builtin_fma(y2, y2, __builtin_fma(y1, y1, y0 * y0));
    const double tq = Y2 - L2;
    const double iL = rsq64<1>(L2);
    const double q = tq * (iL * iL);
    // one comparison decides both ways (a NaN q, from a non-finite state, is a candidate:
    // the rare branch adds it)
    const bool below = q < q0;
    const bool cand = breakable && !below;
    const bool alive = live && !cand;
    // broken and padding slots (and candidates) evaluate g(0) = 0 and add nothing
    const double coef = (kv * iL) * one_minus_rsqrt1p(alive ? q : 0.0, sk);
    st = SlotTerm{q, coef, y0, y1, y2};
    F0 = __builtin_fma(coef, y0, F0);
    F1 = __builtin_fma(coef, y1, F1);
    F2 = __builtin_fma(coef, y2, F2);
    return cand;
}

// The same contribution without a branch, for the kernels whose rows run interleaved.
// With S = |y|^2 + |xi|^2 and d = (|y|^2 - |xi|^2) / S,
//   (1/|xi|) (1 - |xi|/|y|) = sqrt(2) S^(-1/2) d H(d),
//   H = 1 + 5/8 d^2 + 63/128 d^4 + 429/1024 d^6 + 12155/32768 d^8 + ...,
// an even series about the mean square length: two terms reach as far as six of the series in
// q, one reciprocal square root serves length and stretch, and an unstretched bond gives
// exactly zero.  The estimate r of S^(-1/2) takes one Newton step, as rsq64<1> does, in the
// form r (3 - S r^2) = 2 S^(-1/2), so that the term carries 4 d and 16 d^2 and coef lacks the
// factor kMidScale = sqrt(2) / 8.  Error: 9/8 e^2, e = 1 - S r^2 of the estimate (below 2^-22
// by its specification: 6.4e-14; 1.6e-14 for 2^-23), the same as slot_force's; without the step
// two operations fewer a slot (4 % of a step) and up to 2e-12.
// LEVEL 1: two more terms, left out where |d| < kMidRange.  LEVEL 2: the closed form too, from
// kWideRange on (NaN: squares beyond the type's range).  A slot's form follows from its own d
// alone, so that the two slots of a bond, whose d are the same number, carry the same
// coefficient whatever blocks they lie in.
// d rises with q (d = q / (2 + q)), so its high word orders slots against the decision
// edge and the series' range.
constexpr double kMidScale = 0.17677669529663688110;
template <typename Real>
struct MidTerm {
    Real coef, y0, y1, y2;
    Real L2, d;  // |xi|^2, d (FP64: 4 d)
    Real q;      // level 2 only
    int32_t hi;  // high word of d (FP32: its bits)
};
struct MidCoef {
    double c2 = 5.0 / 128.0, c4 = 63.0 / 32768.0;
};
__device__ __forceinline__ MidCoef mid_coef_regs()
{
    MidCoef k;
    asm volatile("" : "+s"(k.c2));
    asm volatile("" : "+v"(k.c4));
    return k;
}
template <int LEVEL>
__device__ __forceinline__ MidTerm<double> slot_mid(const NodeRec& n, double X0, double X1, double X2, double U0, double U1,
                                                    double U2, const MidCoef& k)
{
    const double xi0 = n.p0.x - X0, xi1 = n.p0.y - X1, xi2 = n.p1.x - X2;
    const double e0 = n.p1.y - U0, e1 = n.p2.x - U1, e2 = n.p2.y - U2;
    MidTerm<double> m;
    m.q = 0.0;
    m.y0 = xi0 + e0;
    m.y1 = xi1 + e1;
    m.y2 = xi2 + e2;
    const double L2 = __builtin_fma(xi2, xi2, __builtin_fma(xi1, xi1, xi0 * xi0));
    const double Y2 = __builtin_fma(m.y2, m.y2, __builtin_fma(m.y1, m.y1, m.y0 * m.y0));
    const double tq = Y2 - L2, S = Y2 + L2;  // the numerator as in slot_force
    const double r = __builtin_amdgcn_rsq(S);
    const double r2 = r * __builtin_fma(-S, r * r, 3.0);
    const double d = tq * (r2 * r2);
    const double z = d * d;
    double h = k.c4;
    if constexpr (LEVEL > 0) {
        double t = __builtin_fma(scalar_const(12155.0 / 2147483648.0), z, scalar_const(429.0 / 4194304.0));
        t = fabs(d) < 4.0 * kMidRange ? 0.0 : t;
        h = __builtin_fma(t, z, h);
    }
    m.coef = (d * r2) * __builtin_fma(__builtin_fma(h, z, k.c2), z, 1.0);
    if constexpr (LEVEL > 1) {
        const double iL = rsq64<1>(L2);
        m.q = tq * (iL * iL);
        const double c = scalar_const(1.0 / kMidScale) * (iL * (1.0 - rsq64<2>(1.0 + m.q)));
        m.coef = fabs(d) < 4.0 * kWideRange ? m.coef : c;
    }
    m.L2 = L2;
    m.d = d;
    m.hi = static_cast<int32_t>(__double_as_longlong(d) >> 32);
    return m;
}

// High word of 4 range (FP32: the bits of range32), for comparison with MidTerm::hi.
template <bool FP32>
constexpr uint32_t range_bits(double range, double range32)
{
    if constexpr (FP32)
        return __builtin_bit_cast(uint32_t, static_cast<float>(range32));
    else
        return static_cast<uint32_t>(__builtin_bit_cast(uint64_t, 4.0 * range) >> 32);
}

// The FP32 build's: the bond vector formed in f64 and rounded once, tq without cancellation
// as eta.(xi + y), S = 2 |xi|^2 + tq; the hardware's reciprocal square root is good to single
// precision, and H needs one term (63/128 d^4 is below 5e-9 for |d| < kMidRange32; from there three).  coef lacks
// the factor kMidScale32 = sqrt(2).
constexpr double kMidScale32 = 1.4142135623730950488;
template <int LEVEL>
__device__ __forceinline__ MidTerm<float> slot_mid32(const NodeRec& n, double X0, double X1, double X2, float U0, float U1,
                                                     float U2)
{
    const float xi0 = static_cast<float>(n.p0.x - X0), xi1 = static_cast<float>(n.p0.y - X1),
                xi2 = static_cast<float>(n.p1.x - X2);
    const uint64_t b1 = __double_as_longlong(n.p1.y), b2 = __double_as_longlong(n.p2.x);
    const float e0 = __uint_as_float(static_cast<uint32_t>(b1)) - U0, e1 = __uint_as_float(static_cast<uint32_t>(b1 >> 32)) - U1,
                e2 = __uint_as_float(static_cast<uint32_t>(b2)) - U2;
    MidTerm<float> m;
    m.y0 = xi0 + e0;
    m.y1 = xi1 + e1;
    m.y2 = xi2 + e2;
    const float z0 = xi0 + m.y0, z1 = xi1 + m.y1, z2 = xi2 + m.y2;
    const float tq = __builtin_fmaf(e2, z2, __builtin_fmaf(e1, z1, e0 * z0));
    m.L2 = __builtin_fmaf(xi2, xi2, __builtin_fmaf(xi1, xi1, xi0 * xi0));
    const float S = __builtin_fmaf(2.0f, m.L2, tq);
    const float r = __builtin_amdgcn_rsqf(S);
    const float d = tq * (r * r);
    const float z = d * d;
    float h = 0.625f;
    if constexpr (LEVEL > 0) {
        float t = __builtin_fmaf(429.0f / 1024.0f, z, 63.0f / 128.0f);
        t = fabsf(d) < static_cast<float>(kMidRange32) ? 0.0f : t;
        h = __builtin_fmaf(t, z, h);
    }
    m.coef = (d * r) * __builtin_fmaf(h, z, 1.0f);
    if constexpr (LEVEL > 1) {
        const float iL = __builtin_amdgcn_rsqf(m.L2);
        m.q = tq * (iL * iL);
        const float c = (1.0f / static_cast<float>(kMidScale32)) * (iL * (1.0f - __builtin_amdgcn_rsqf(1.0f + m.q)));
        m.coef = fabsf(d) < static_cast<float>(kWideRange32) ? m.coef : c;
    }
    m.d = d;
    m.hi = static_cast<int32_t>(__float_as_uint(d));
    return m;
}

// Stretch from q without cancellation: s = q / (1 + sqrt(1 + q)).
__device__ __forceinline__ double stretch_of(double q)
{
    const double r = rsq64<2>(1.0 + q);
    return q * rcp64(__builtin_fma(1.0 + q, r, 1.0));
}

// Weight of a slot in the bond-model branch (EXT kernels): the slot is live and either at
// or over the instance's lower decision edge q0, or softened.  q and s are its q and
// stretch of this pass, nofail / soft its word's flags, sold its stored largest stretch (prefetched by the
// caller when soft), exact_s() the slot's exact stretch (stretch_exact; the FP64 build
// decides on it near every threshold and stores it as a new maximum, the FP32 build
// decides on q).  The bond adds `share` times its elastic force; it breaks now, softens for
// the first time, or reaches a new maximum smax, which the caller stores.  A zone bond, and every
// bond in a force evaluation, keeps its damage state as it stands.
struct BondWeight {
    double share = 1.0, smax = 0.0;
    bool broke = false, newly_soft = false, grew = false;
};
template <int MODE, bool FP32, typename ExactS>
__device__ __forceinline__ BondWeight bond_weight(const StepArgs& A, const InstParams& P, int64_t ds, double q, double s, bool nofail,
                                                  bool soft, double sold, ExactS exact_s)
{
    // a single law per instance is the same for the whole wavefront (scalar loads, which the
    // constant address space asks for: the kernel's own stores rule them out otherwise)
    const auto& one = *(const __attribute__((address_space(4))) LawRec*)(A.laws + P.law_off);
    const LawRec* const own = A.laws + P.law_off + (P.nlaw > 1 ? A.cls[ds] : 0);
    auto secant = [&](double sm) { return P.nlaw == 1 ? law_secant(one, sm) : law_secant(*own, sm); };
    BondWeight w;
    if (!soft) sold = 0.0;
    if (nofail || MODE == kModeForce) {
        if (soft) w.share = secant(sold);
        return w;
    }
    double s_first = P.s0, s_last = P.s0;  // the brittle law with the instance's s0
    if (P.nlaw == 1) {
        s_first = one.s[0];
        s_last = one.s[one.nb - 1];
    } else if (P.nlaw > 1) {
        s_first = own->s[0];
        s_last = own->s[own->nb - 1];
    } else if (FP32) {  // which the FP32 build decides on q
        s = static_cast<float>(q) >= static_cast<float>(P.q0) ? s_last : 0.0;
    }
    // the exact stretch wherever rounding could decide: at or near the stored maximum (a
    // new maximum is stored exact) or near the law's elastic limit or last breakpoint
    if (!FP32 && (s >= sold - decision_margin(sold) || fabs(s - s_first) <= decision_margin(s_first) ||
                  fabs(s - s_last) <= decision_margin(s_last)))
        s = exact_s();
    w.smax = s > sold ? s : sold;
    if (w.smax >= s_last) {
        w.broke = true;
        w.share = 0.0;
    } else if (w.smax > s_first) {
        w.grew = w.smax > sold;
        w.newly_soft = !soft;
        w.share = secant(w.smax);
    }
    return w;
}

// Stiffness corrections that a staged kernel forms per slot: the profile and the surface factor,
// or the partial volume too (its four operations in a slot's 55 are worth a variant).
constexpr int kCorrNone = 0, kCorrPlain = 1, kCorrPartial = 2;

// The correction factor of a slot of squared reference length L2, without the instance's
// 2 V0 of the surface factor (FP64: and four times it); V the sum of the two ends' family
// volumes.  The parameters of a factor that the instance does not have make it 1.  One
// reciprocal square root t = 1 / (L V) gives both 1 / L = V t and 1 / V = L t; its Newton step
// as in slot_mid, t (3 - x t^2) = 2 t.
struct CorrCoef {
    double hidelta, hidx, pvhi;  // 1 / (2 delta), 1 / (2 dx), (delta + dx/2) / dx
};
template <int CORR>
__device__ __forceinline__ double corr_factor(const CorrCoef& P, double L2, double V)
{
    const double x = L2 * (V * V), t = __builtin_amdgcn_rsq(x), t2 = t * __builtin_fma(-x, t * t, 3.0);
    const double L = L2 * (V * t2);  // twice |xi|
    double f = fmax(__builtin_fma(-L, P.hidelta, 1.0), 0.0);
    if constexpr (CORR == kCorrPartial) f *= fmin(fmax(__builtin_fma(-L, P.hidx, P.pvhi), 0.0), 1.0);
    return f * (L * t2);
}

template <int CORR>
__device__ __forceinline__ float corr_factor(const CorrCoef& P, float L2, float V)
{
    const float L = 2.0f * (L2 * __builtin_amdgcn_rsqf(L2));
    float f = fmaxf(__builtin_fmaf(-L, static_cast<float>(P.hidelta), 1.0f), 0.0f);
    if constexpr (CORR == kCorrPartial)
        f *= fminf(fmaxf(__builtin_fmaf(-L, static_cast<float>(P.hidx), static_cast<float>(P.pvhi)), 0.0f), 1.0f);
    return f * __builtin_amdgcn_rcpf(V);
}

// Integration and boundary conditions of one node given its force density F (the tail
// of every step kernel).  U is the node's displacement at the level the forces used.
template <int MODE, bool FP32 = false>
__device__ __forceinline__ void node_update(const StepArgs& A, const InstParams& P, int64_t node,
                                            double U0, double U1, double U2, double F0, double F1, double F2)
{
    const int32_t bcid = A.bc_id[node];
    if (bcid == kNodePad) return;

    const int64_t nn = A.nn;
    if (MODE == kModeForce) {  // bond force density of the current level, nothing else
        A.force[node] = F0;
        A.force[nn + node] = F1;
        A.force[2 * nn + node] = F2;
        return;
    }
    const double dt = A.dt;
    const int64_t k = *A.step_base + A.step_local;
    double F[3] = {F0, F1, F2};
    if (P.has_body)
        for (int d = 0; d < 3; ++d) F[d] += P.bmag * A.bhat[d * nn + node];
    double u[3] = {U0, U1, U2};
    if (FP32)  // the integrator advances the f64 master displacement
        for (int d = 0; d < 3; ++d) u[d] = A.um_in[d * nn + node];
    double vv[3], un[3], vn[3], an[3];
    for (int d = 0; d < 3; ++d) vv[d] = A.v[d * nn + node];
    BCRec bc;
    bc.code = 0;
    if (bcid >= 0) bc = A.bc[bcid];

    if (MODE == kModeEC || MODE == kModeFE) {
        const double t1 = static_cast<double>(k + 1) * dt;
        for (int d = 0; d < 3; ++d) {
            const double acc = (F[d] - P.eta * vv[d]) / P.rho;
            if (MODE == kModeEC) {
                vn[d] = vv[d] + dt * acc;
                un[d] = u[d] + dt * vn[d];
            } else {
                un[d] = u[d] + dt * vv[d];
                vn[d] = vv[d] + dt * acc;
            }
            if (constrained(bc, d)) {
                vn[d] = bc_vel(bc, d, t1);
                un[d] = bc_disp(bc, d, t1, u[d], dt);
            }
        }
    } else if (MODE == kModeVV) {
        // u holds level k+1; v, a hold level k.  Finish step k -> k+1, then move the
        // displacement on to level k+2 (Eq. Velocity_Verlet1) for the next launch.
        const double t1 = static_cast<double>(k + 1) * dt, t2 = static_cast<double>(k + 2) * dt;
        const double hdt = 0.5 * dt, hdt2 = 0.5 * dt * dt;
        for (int d = 0; d < 3; ++d) {
            const double aa = A.a[d * nn + node];
            const double vh = vv[d] + hdt * aa;
            an[d] = (F[d] - P.eta * vh) / P.rho;
            vn[d] = vv[d] + hdt * (aa + an[d]);
            if (constrained(bc, d)) {
                vn[d] = bc_vel(bc, d, t1);
                an[d] = 0.0;
            }
            un[d] = (u[d] + dt * vn[d]) + hdt2 * an[d];
            if (constrained(bc, d)) un[d] = bc_disp(bc, d, t2, u[d], dt);
        }
    } else {  // kModeVVInit: u holds level k; acceleration of level k, then u of level k+1
        const double t1 = static_cast<double>(k + 1) * dt;
        const double hdt2 = 0.5 * dt * dt;
        for (int d = 0; d < 3; ++d) {
            an[d] = constrained(bc, d) ? 0.0 : (F[d] - P.eta * vv[d]) / P.rho;
            un[d] = (u[d] + dt * vv[d]) + hdt2 * an[d];
            if (constrained(bc, d)) un[d] = bc_disp(bc, d, t1, u[d], dt);
            vn[d] = vv[d];
        }
    }

    bool finite = true;
    for (int d = 0; d < 3; ++d) finite = finite && __builtin_isfinite(un[d]) && __builtin_isfinite(vn[d]);
    if (!finite) atomicOr(A.status, 1);
    double* ro = A.rec_out + 6 * node;
    if (FP32) {
        float* rf = reinterpret_cast<float*>(ro + 3);
        for (int d = 0; d < 3; ++d) {
            rf[d] = static_cast<float>(un[d]);
            A.um_out[d * nn + node] = un[d];
        }
    } else {
        ro[3] = un[0];
        ro[4] = un[1];
        ro[5] = un[2];
    }
    if (MODE != kModeVVInit)
        for (int d = 0; d < 3; ++d) A.v[d * nn + node] = vn[d];
    if (MODE == kModeVV || MODE == kModeVVInit)
        for (int d = 0; d < 3; ++d) A.a[d * nn + node] = an[d];
}

template <int G, int MODE, bool STIFF, bool VOLN, bool KNODE, bool EXT>
__global__ __launch_bounds__(kBlock) void step_f64(StepArgs A)
{
    constexpr int W = kWave / G;
    constexpr int U = kRowUnroll;  // slot rows in flight per iteration
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t slice =
        wave_uniform(xcd_remap(blockIdx.x, gridDim.x) * (kBlock / kWave) + (threadIdx.x >> 6));
    if (slice >= A.nslices) return;
    const int32_t* __restrict__ slice_inst = A.slice_inst;
    const InstParams* __restrict__ params = A.params;
    const int64_t* __restrict__ slice_ptr = A.slice_ptr;
    const int32_t* __restrict__ slice_T = A.slice_T;
    const InstParams P = params[slice_inst[slice]];
    const int w = lane / G, g = lane % G;
    const int64_t node = slice * W + w;

    const double2* __restrict__ rin = reinterpret_cast<const double2*>(A.rec_in);
    const double2 o0 = rin[3 * node], o1 = rin[3 * node + 1], o2 = rin[3 * node + 2];
    const double X0 = o0.x, X1 = o0.y, X2 = o1.x;
    const double U0 = o1.y, U1 = o2.x, U2 = o2.y;
    // 32-bit byte offsets from wave-uniform bases (the host keeps every offset below 2^32)
    const char* __restrict__ recb = reinterpret_cast<const char*>(A.rec_in);
    const int64_t base = slice_ptr[slice];
    const int T = slice_T[slice];
    const char* __restrict__ colb = reinterpret_cast<const char*>(A.col + base);
    const char* __restrict__ kb = STIFF ? reinterpret_cast<const char*>(A.kslot + base) : nullptr;
    const double* __restrict__ volp = A.vol;
    const double* __restrict__ nwp = A.nw;
    const double ai = KNODE ? A.na[node] : 0.0;  // own stiffness factor
    const uint32_t lane4 = static_cast<uint32_t>(lane) * 4u;
    const double cv = P.c * P.volume;

    // Rows are fetched one iteration ahead.  T is a multiple of kRowUnroll and the slot
    // arrays end with kRowUnroll spare rows, so every prefetch is in bounds and no load
    // sits behind a branch (rows prefetched past T belong to the next slice; unused).
    double F0 = 0.0, F1 = 0.0, F2 = 0.0;
    const SeriesCoef sk = series_coef_regs();
    if (T > 0) {
        auto col_at = [&](int t) -> int32_t {
            const uint32_t off = static_cast<uint32_t>(t) * (kWave * 4u) + lane4;
            return __builtin_nontemporal_load(reinterpret_cast<const int32_t*>(colb + off));
        };
        // stiffness times neighbour volume of row t's slot with neighbour j
        auto kv_of = [&](int t, uint32_t j) -> double {
            if (KNODE) return ai * nwp[j];  // sqrt(k_i) sqrt(k_j) V_j
            if (STIFF || VOLN) {
                double k = P.c;
                if (STIFF) {
                    const uint32_t off = static_cast<uint32_t>(t) * (kWave * 8u) + 2u * lane4;
                    k = __builtin_nontemporal_load(reinterpret_cast<const double*>(kb + off));
                }
                return k * (VOLN ? volp[j] : P.volume);
            }
            return cv;
        };
        // stored stretch of softened slots, fetched with their words (EXT with damage laws)
        auto smax_at = [&](int t, int32_t cw) -> double {
            if (!EXT || P.nlaw == 0 || cw < 0 || !(cw & kColSoft)) return 0.0;
            return A.smax[base + static_cast<int64_t>(t) * kWave + lane];
        };
        // Rare branch of a flagged slot in row t (plain: a break candidate, decided on the
        // exact stretch; EXT: the bond-model branch).  It runs after a block of 32 rows, from
        // the slot's word and neighbour record read again, so the common path keeps its
        // registers.
        auto flagged = [&](int t) {
            const int64_t ds = base + static_cast<int64_t>(t) * kWave + lane;
            const int32_t step = static_cast<int32_t>(*A.step_base + A.step_local);
            const int32_t cw = col_at(t);
            const uint32_t j = col_node(cw);
            const char* rj = recb + __umul24(j, 48u);
            const double2 r0 = *reinterpret_cast<const double2*>(rj), r1 = *reinterpret_cast<const double2*>(rj + 16),
                          r2 = *reinterpret_cast<const double2*>(rj + 32);
            auto exact = [&]() { return stretch_exact_rec(r0, r1, r2, X0, X1, X2, U0, U1, U2); };
            if constexpr (EXT) {
                // the slot's terms as the common path formed them (into scratch accumulators),
                // then move its elastic contribution from weight 1 to w
                SlotTerm st;
                double d0 = 0.0, d1 = 0.0, d2 = 0.0;
                slot_force(true, false, r0, r1, r2, X0, X1, X2, U0, U1, U2, kv_of(t, j), P.q0, d0, d1, d2, st, sk);
                const BondWeight bw = bond_weight<MODE, false>(A, P, ds, st.q, stretch_of(st.q), (cw & kColNoFail) != 0,
                                                               (cw & kColSoft) != 0, smax_at(t, cw), exact);
                const double wt = bw.share;
                if (bw.grew) A.smax[ds] = bw.smax;
                if (bw.broke) {
                    A.col[ds] = ~cw;
                    A.bstep[ds] = step;
                } else if (bw.newly_soft) {
                    A.col[ds] = cw | kColSoft;
                }
                if (wt != 1.0) {
                    const double m = (wt - 1.0) * st.coef;
                    F0 = __builtin_fma(m, st.y0, F0);
                    F1 = __builtin_fma(m, st.y1, F1);
                    F2 = __builtin_fma(m, st.y2, F2);
                }
            } else if (exact() >= P.s0) {
                A.col[ds] = ~cw;  // irreversible
                A.bstep[ds] = step;
            } else {  // it holds: the contribution the common path left out
                SlotTerm sh;
                slot_force(true, false, r0, r1, r2, X0, X1, X2, U0, U1, U2, kv_of(t, j), P.q0, F0, F1, F2, sh, sk);
            }
        };
        int32_t cn[U];
#pragma unroll
        for (int u = 0; u < U; ++u) cn[u] = col_at(u);
        uint32_t flags = 0;  // flagged rows of the current block of 32 (from row tb)
        int tb = 0;
        for (int t = 0; t < T; t += U) {
            int32_t c[U];
            double2 p[U][3];
            double kv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                c[u] = cn[u];
                const uint32_t j = static_cast<uint32_t>(c[u] ^ (c[u] >> 31)) &
                                   (EXT ? static_cast<uint32_t>(kColNode) : 0xffffffffu);
                const char* rj = recb + __umul24(j, 48u);  // full-rate 24-bit multiply: j < 2^24
                p[u][0] = *reinterpret_cast<const double2*>(rj);
                p[u][1] = *reinterpret_cast<const double2*>(rj + 16);
                p[u][2] = *reinterpret_cast<const double2*>(rj + 32);
                kv[u] = kv_of(t + u, j);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) cn[u] = col_at(t + U + u);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                SlotTerm st;
                bool flag;  // plain: a break candidate; EXT: takes the bond-model branch
                if constexpr (EXT) {
                    slot_force(c[u] >= 0, false, p[u][0], p[u][1], p[u][2], X0, X1, X2, U0, U1, U2, kv[u], P.q0, F0,
                               F1, F2, st, sk);
                    const bool soft = (c[u] & kColSoft) != 0;
                    flag = c[u] >= 0 && (MODE == kModeForce ? soft : (st.q >= P.q0 || soft));
                } else {
                    flag = slot_force(c[u] >= 0, MODE != kModeForce && c[u] >= 0, p[u][0], p[u][1], p[u][2], X0, X1,
                                      X2, U0, U1, U2, kv[u], P.q0, F0, F1, F2, st, sk);
                }
                flags |= flag ? 1u << (t + u - tb) : 0u;
            }
            if (t + U - tb == 32 || t + U >= T) {  // end of a block: its rare branches
                if (__builtin_amdgcn_ballot_w64(flags != 0) != 0)
#pragma unroll 1
                    for (int k = 0; k < 32; ++k)
                        if (flags & (1u << k)) flagged(tb + k);
                flags = 0;
                tb = t + U;
            }
        }
    }
#pragma unroll
    for (int m = 1; m < G; m <<= 1) {
        F0 += __shfl_xor(F0, m);
        F1 += __shfl_xor(F1, m);
        F2 += __shfl_xor(F2, m);
    }
    if (g != 0) return;
    node_update<MODE>(A, P, node, U0, U1, U2, F0, F1, F2);
}

// Staged step kernel (see pdmi_tile.h for the tile and its staging): one lane a node, 2 to 8
// wavefronts a slice.  A lane reads its slots' neighbours from LDS, a row ahead of their use;
// entries (and the per-slot stiffness) stream from global memory a block of row pairs ahead.
// The common path adds every live bond's term without a branch: broken, padding and softened
// slots read the sentinel record, whose term is exactly zero.  What a level of the series
// does not cover is seen on the slots' d once a block, which is then taken again at
// the level it asks for.  The last level covers every d and leaves out the slots at the
// decision edge.  Those and the softened ones are kept as bits of each lane's window of
// 32 row pairs and settled after it (the tiles at a crack are the launch's tail).
// The partial forces of a slice's wavefronts meet in LDS in a fixed order.
// Bound: FP64 vector issue at the clock the chip holds under it (248 of the 277 vector
// instructions of four row pairs).  us a step, and where each wavefront staged runs of
// consecutive records itself and took a reciprocal root and a six-term series per slot: 1M
// nodes at horizon 3.015 191 and 233, 216000 at 5.015 161 and 327, 1000 at 3.015 8.0 and 14.1.
// STIFF per-slot stiffness, VOLN per-node volumes, KNODE per-node stiffness factors, CORR
// stiffness corrections formed per slot (uniform stiffness and volume), EXT no-failure zones
// and damage laws.
template <bool FP32, int MODE, bool STIFF, bool VOLN, bool KNODE, bool EXT, int CORR>
__global__ __launch_bounds__(kTileWaves * kWave, 4) void step_staged(StepArgs A, const TileRec* __restrict__ tiles,
                                                                  const int2* __restrict__ phases,
                                                                  const int2* __restrict__ segs,
                                                                  const int32_t* __restrict__ list)
{
    using Real = std::conditional_t<FP32, float, double>;
    extern __shared__ double2 lds[];
    constexpr bool NODEW = VOLN || KNODE || CORR != kCorrNone;  // a double per neighbour node staged beside the records
    constexpr bool WEIGHT = STIFF || NODEW;
    constexpr int B = STIFF ? 2 : kPairsAhead;     // row pairs of a block
    constexpr bool BREAKS = MODE != kModeForce;
    static_assert(CORR == kCorrNone || (!STIFF && !VOLN && !KNODE), "per-slot corrections: uniform stiffness and volume");
    __builtin_amdgcn_s_setprio(3);
    const TileRec T = tiles[wave_uniform(xcd_remap(blockIdx.x, gridDim.x))];
    const TileLane tl(T);
    const int lane = tl.lane;
    double2* const lrec = lds;
    double* const lw = reinterpret_cast<double*>(lrec + 3 * (A.stage_max + 1));
    uint16_t* const litem = reinterpret_cast<uint16_t*>(lw + (NODEW ? A.stage_max + 1 : 0)) + tl.wv * kWave;  // see settle
    const double* __restrict__ wsrc = KNODE ? A.nw : CORR ? A.cfv : A.vol;
    const uint32_t* __restrict__ ent = reinterpret_cast<const uint32_t*>(A.ent) + lane;
    const double2* __restrict__ kslot = reinterpret_cast<const double2*>(A.kslot) + lane;
    const InstParams* __restrict__ params = A.params;
    const MidCoef mc = mid_coef_regs();
    const bool laws = EXT && A.laws != nullptr;

    if (threadIdx.x < 3) lrec[threadIdx.x] = sentinel_part<FP32>(threadIdx.x);
    if (NODEW && threadIdx.x == 0) lw[0] = CORR ? 1.0 : 0.0;

    if (T.nphases > 0) stage_records(A.rec_in, list + T.list, T.n, tl.wv, lane, lrec);
    const InstParams& P = params[T.inst];
    const int64_t node = tl.node(T);
    const double2* __restrict__ rin = reinterpret_cast<const double2*>(A.rec_in);
    const double2 o0 = rin[3 * node], o1 = rin[3 * node + 1], o2 = rin[3 * node + 2];
    const double X0 = o0.x, X1 = o0.y, X2 = o1.x;
    const double U0 = o1.y, U1 = o2.x, U2 = o2.y;  // FP64 build
    const uint64_t ub1 = __double_as_longlong(o1.y), ub2 = __double_as_longlong(o2.x);
    const float Uf0 = __uint_as_float(static_cast<uint32_t>(ub1)),
                Uf1 = __uint_as_float(static_cast<uint32_t>(ub1 >> 32)),
                Uf2 = __uint_as_float(static_cast<uint32_t>(ub2));  // FP32 build
    const double fvi = CORR ? A.cfv[node] : 0.0;
    // scalar loads, once: the kernel's own stores make the compiler load a parameter again for
    // every slot otherwise (corrections 2 % of a step)
    CorrCoef cc{0.0, 0.0, 1.0};
    if (CORR) {
        const auto& Q = *(const __attribute__((address_space(4))) InstParams*)(params + T.inst);
        cc = CorrCoef{Q.cr_hidelta, CORR == kCorrPartial ? Q.cr_hidx : 0.0, CORR == kCorrPartial ? Q.cr_pvhi : 1.0};
        asm volatile("" : "+s"(cc.hidelta));
        if (CORR == kCorrPartial) asm volatile("" : "+s"(cc.hidx), "+s"(cc.pvhi));
    }
    const float q0f = static_cast<float>(P.q0);
    // where the levels end, as high words of a slot's d: their ranges, above zero the decision edge too
    const int32_t edge = !BREAKS ? std::numeric_limits<int32_t>::max() : FP32 ? P.hi_edge32 : P.hi_edge;
    constexpr uint32_t range = range_bits<FP32>(kMidRange, kMidRange32), wrange = range_bits<FP32>(kWideRange, kWideRange32);
    constexpr uint32_t neg = 0x80000000u | range, wneg = 0x80000000u | wrange;
    constexpr uint32_t nan_neg = FP32 ? 0xff800000u : 0xfff00000u;
    Real F0 = 0, F1 = 0, F2 = 0;   // sums without kMidScale and (FP64; FP32: uniform ones) the factors shared by the node's bonds

    auto term = [&](const NodeRec& r, auto level) {
        if constexpr (FP32)
            return slot_mid32<decltype(level)::value>(r, X0, X1, X2, Uf0, Uf1, Uf2);
        else
            return slot_mid<decltype(level)::value>(r, X0, X1, X2, U0, U1, U2, mc);
    };
    // the factor of a slot that its node's bonds do not share (FP32: the whole of it, formed in
    // double precision, whose parts may leave the single one's range while their product, a force
    // density, does not; of the corrections the ratio to 2 V0)
    auto weight = [&](uint32_t idx, double k, Real L2, double fv, double own) -> Real {
        if constexpr (CORR != kCorrNone) {
            return corr_factor<CORR>(cc, L2, static_cast<Real>(FP32 ? (fv + lw[idx]) * own : fv + lw[idx]));
        } else if constexpr (NODEW) {
            const double v = lw[idx];
            return static_cast<Real>(STIFF ? k * v : FP32 ? own * v : v);
        } else {
            return static_cast<Real>(!STIFF ? 1.0 : FP32 ? k * own : k);
        }
    };
    const double own = !FP32 ? 1.0 : CORR ? 1.0 / P.cr_2v0 : KNODE ? A.na[node] : STIFF ? P.volume : P.c;
    auto add = [&](Real coef, const MidTerm<Real>& m) {
        F0 = __builtin_elementwise_fma(coef, m.y0, F0);
        F1 = __builtin_elementwise_fma(coef, m.y1, F1);
        F2 = __builtin_elementwise_fma(coef, m.y2, F2);
    };
    uint32_t en[B];  // the next block's entries and stiffness
    double2 kn[B];
    auto fetch = [&](int t) {  // (one address a stream, the pairs of the block by immediate offset)
        const int64_t at = static_cast<int64_t>(t) * kWave;
#pragma unroll
        for (int u = 0; u < B; ++u) {
            en[u] = (ent + at)[u * kWave];
            if (STIFF) kn[u] = (kslot + at)[u * kWave];
        }
    };
    uint64_t todo = 0;  // slots of the window from pair `base` on that are settled after it
    int base = 0;
    // FP32: their sum in double precision, beside the others' single one (a softening law
    // amplifies a force's rounding by up to 60)
    double E0 = 0, E1 = 0, E2 = 0;
    auto& S0 = [&]() -> auto& { if constexpr (FP32) return E0; else return F0; }();
    auto& S1 = [&]() -> auto& { if constexpr (FP32) return E1; else return F1; }();
    auto& S2 = [&]() -> auto& { if constexpr (FP32) return E2; else return F2; }();
    // Marks the softened and not broken slots of a block; true if nothing is left for its rows.
    auto mark_soft = [&](const uint32_t (&e)[B], int t, int end) {
        if (!laws) return false;
        uint32_t s[B], any = 0;
#pragma unroll
        for (int u = 0; u < B; ++u) {
            s[u] = t + u < end ? e[u] & ~(e[u] >> 2) & 0x20002000u : 0u;
            any |= s[u];
        }
        if (__builtin_amdgcn_ballot_w64(any != 0) == 0) return false;
        uint32_t bits = 0, left = 0;
#pragma unroll
        for (int u = 0; u < B; ++u) {
            bits |= ((s[u] >> 13 & 1u) | (s[u] >> 28 & 2u)) << (2 * u);
            left |= t + u < end ? live_indices<EXT>(e[u]) : 0u;
        }
        todo |= static_cast<uint64_t>(bits) << (2 * (t - base));
        return __builtin_amdgcn_ballot_w64(left != 0) == 0;
    };
    // The pairs [t, end), after fetch(t), block by block at level 0 or 1, up to the first block with
    // a slot that the level does not cover; that block is taken back, and `need` is the level
    // that covers it.  kMark: level 1 with the slots at the decision edge left out and marked
    // (eight more operations a slot), also the level of zone bonds over the edge, which stay
    // in: once a share needs it, it keeps it.
    int need = 0;
    constexpr int kMark = 3;
    auto rows = [&](int t, int end, auto level) {
        constexpr bool wide = decltype(level)::value > 0, MARK = decltype(level)::value == kMark;
        using Level = std::integral_constant<int, wide ? 1 : 0>;
        const int32_t pos = MARK ? static_cast<int32_t>(wrange) : min(static_cast<int32_t>(wide ? wrange : range), edge);
#pragma unroll 1
        for (; t < end; t += B) {
            uint32_t e[B];
            double2 k[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                e[u] = en[u];
                if (STIFF) k[u] = kn[u];
            }
            fetch(t + B);
            if constexpr (EXT)
                if (mark_soft(e, t, end)) continue;
            const Real B0 = F0, B1 = F1, B2 = F2;
            int32_t himax = std::numeric_limits<int32_t>::min();  // of the block's d: the largest high word
            uint32_t himin = 0;  // and the one furthest below zero (sign bit set: large)
            uint32_t bits = 0;
            auto one = [&](const NodeRec& r, uint32_t idx, double kslot, uint32_t word, int bit) {
                const MidTerm<Real> m = term(r, Level{});
                Real coef = WEIGHT ? m.coef * weight(idx, kslot, m.L2, fvi, own) : m.coef;
                if constexpr (MARK) {
                    const bool over = m.hi >= edge && (word & (EXT ? kEntBroken | kEntSoft | kEntNoFail : kEntBroken)) == 0;
                    coef = over ? Real(0) : coef;
                    bits |= over ? 1u << bit : 0u;
                }
                add(coef, m);
                himax = max(himax, m.hi);
                himin = max(himin, static_cast<uint32_t>(m.hi));
            };
            uint32_t v = live_indices<EXT>(e[0]);
            NodeRec ra = staged_record(lrec, v & 0xffffu);
#pragma unroll
            for (int u = 0; u < B; ++u) {
                if (t + u >= end) break;
                const uint32_t ia = v & 0xffffu, ib = v >> 16;
                const NodeRec rb = staged_record(lrec, ib);
                // (past the share's end: another share's entry, read but not added)
                if (u + 1 < B) v = live_indices<EXT>(e[u + 1]);
                __builtin_amdgcn_sched_barrier(0);
                one(ra, ia, STIFF ? k[u].x : 0.0, e[u], 2 * u);
                if (u + 1 < B) ra = staged_record(lrec, v & 0xffffu);
                __builtin_amdgcn_sched_barrier(0);
                one(rb, ib, STIFF ? k[u].y : 0.0, e[u] >> 16, 2 * u + 1);
            }
            if (__builtin_amdgcn_ballot_w64(himax >= pos || himin >= (wide ? wneg : neg)) != 0) {
                F0 = B0;
                F1 = B1;
                F2 = B2;
                need = __builtin_amdgcn_ballot_w64(himax >= static_cast<int32_t>(wrange) || himin >= wneg) != 0 ? 2
                       : __builtin_amdgcn_ballot_w64(himax >= edge) != 0                                        ? kMark
                                                                                                                : 1;
                return t;
            }
            if constexpr (MARK) todo |= static_cast<uint64_t>(bits) << (2 * (t - base));
        }
        return t;
    };
    // One block or more from pair t on at level 2, one slot at a time (two interleaved do not fit
    // the registers), as long as blocks have slots beyond the long series.
    auto rows_general = [&](int t, int end) {
#pragma unroll 1
        for (bool on = true; on && t < end; t += B) {
            uint32_t e[B];
            double2 k[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                e[u] = en[u];
                if (STIFF) k[u] = kn[u];
            }
            fetch(t + B);
            if constexpr (EXT)
                if (mark_soft(e, t, end)) continue;
            int32_t himax = std::numeric_limits<int32_t>::min();
            uint32_t himin = 0, bits = 0;
#pragma unroll 1
            for (int u = 0; u < 2 * B; ++u) {
                const bool in = t + (u >> 1) < end;
                const uint32_t h = in ? e[0] & 0xffffu : kEntBroken;
                const double kh = STIFF ? k[0].x : 0.0;
                // the next slot's entry and stiffness
                if (u & 1) {
#pragma unroll
                    for (int w = 0; w + 1 < B; ++w) {
                        e[w] = e[w + 1];
                        if (STIFF) k[w] = k[w + 1];
                    }
                } else {
                    e[0] >>= 16;
                    if (STIFF) k[0].x = k[0].y;
                }
                const bool live = !(h & (EXT ? kEntBroken | kEntSoft : kEntBroken));
                const uint32_t idx = live ? h & kEntIdx : 0u;
                const MidTerm<Real> m = term(staged_record(lrec, idx), std::integral_constant<int, 2>{});
                const bool over = BREAKS && live && !(EXT && (h & kEntNoFail)) &&
                                  (m.hi >= edge || static_cast<uint32_t>(m.hi) >= nan_neg);
                bits |= over ? 1u << u : 0u;
                // a slot that is not live adds nothing, whatever its numbers
                if (live && !over) add(WEIGHT ? m.coef * weight(idx, kh, m.L2, fvi, own) : m.coef, m);
                const int32_t hi = live ? m.hi : 0;
                himax = max(himax, hi);
                himin = max(himin, static_cast<uint32_t>(hi));
            }
            todo |= static_cast<uint64_t>(bits) << (2 * (t - base));
            on = __builtin_amdgcn_ballot_w64(himax >= static_cast<int32_t>(wrange) || himin >= wneg) != 0;
        }
        return t;
    };
    // The marked slots of the window: a break candidate is decided on its exact stretch, a
    // softened one takes the weight of its damage state.  Where few lanes have some (at a crack 9
    // of a wavefront's 2000 slots, up to 7 in one lane) a round takes several of each, so that all
    // lanes work, each on one slot whoever owns it; the owners then collect their sums in slot order.
    // A slot of each lane in turn takes a pass of 400 instructions for every slot of the
    // fullest lane: 117 x 33 x 33 nodes with a grown crack 61.8 us a step, shared out 43.4.  None,
    // 1 % and all of the slots softened: 37.8, 59.6 and 153 us, and 41.9, 116 and 146 where a
    // slice's flagged rows were taken one by one.
    // The next round's words are loaded during a round's arithmetic and waited for before its
    // stores, so that the wave waits for no store.
    auto settle = [&] {
        if (__builtin_amdgcn_ballot_w64(todo != 0) == 0) return false;
        struct Round {
            int m;          // slots of a lane that has some, 0: nothing left
            int at, n;      // this lane's: first place in the round, number
            bool on;        // this lane works on a slot: its owner, place and words
            int owner;
            int64_t ds;
            uint32_t word;
            double sold, k;
        };
        auto next = [&] {
            Round w;
            const uint64_t some = __builtin_amdgcn_ballot_w64(todo != 0);
            w.m = some ? kWave / __builtin_popcountll(some) : 0;
            w.at = lane;
            w.n = 0;
            w.owner = lane;
            w.on = todo != 0;
            int bit = w.on ? __builtin_ctzll(todo) : 0;
            if (w.m == 1) {
                w.n = w.on;
                todo &= todo - 1;
            } else if (w.m > 1) {
                w.at = w.m * static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(some >> 32),
                                                                        __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(some), 0u)));
                litem[lane] = 0xffff;
                __builtin_amdgcn_wave_barrier();
#pragma unroll 1
                for (; w.n < w.m && todo != 0; ++w.n) {
                    litem[w.at + w.n] = static_cast<uint16_t>(lane | __builtin_ctzll(todo) << 8);
                    todo &= todo - 1;
                }
                __builtin_amdgcn_wave_barrier();
                const uint32_t item = litem[lane];
                w.on = item != 0xffffu;
                w.owner = w.on ? static_cast<int>(item & 63u) : lane;
                bit = w.on ? static_cast<int>(item >> 8) : 0;
            }
            w.ds = static_cast<int64_t>(base + (bit >> 1)) * (2 * kWave) + 2 * w.owner + (bit & 1);
            w.word = A.ent[w.ds];
            w.sold = laws ? A.smax[w.ds] : 0.0;
            w.k = STIFF ? A.kslot[w.ds] : 0.0;
            return w;
        };
        Round w = next();
#pragma unroll 1
        while (w.m != 0) {
            Round wn = next();
            double x0 = X0, x1 = X1, x2 = X2, u0 = U0, u1 = U1, u2 = U2, fv = fvi, ow = own;
            float v0 = Uf0, v1 = Uf1, v2 = Uf2;
            if (w.m > 1) {
                x0 = __shfl(X0, w.owner), x1 = __shfl(X1, w.owner), x2 = __shfl(X2, w.owner);
                if constexpr (FP32)
                    v0 = __shfl(Uf0, w.owner), v1 = __shfl(Uf1, w.owner), v2 = __shfl(Uf2, w.owner);
                else
                    u0 = __shfl(U0, w.owner), u1 = __shfl(U1, w.owner), u2 = __shfl(U2, w.owner);
                if (CORR) fv = __shfl(fvi, w.owner);
                if (FP32 && KNODE) ow = __shfl(own, w.owner);
            }
            const uint32_t e = w.on ? w.word : kEntBroken;
            const bool live = !(e & kEntBroken), soft = EXT && live && (e & kEntSoft) != 0;
            const uint32_t idx = live ? e & kEntIdx : 0u;
            const NodeRec r = staged_record(lrec, idx);
            MidTerm<Real> m;
            if constexpr (FP32) {
                m = slot_mid32<2>(r, x0, x1, x2, v0, v1, v2);
            } else if constexpr (EXT) {  // (softened slots are within the series, all but a few)
                m = slot_mid<1>(r, x0, x1, x2, u0, u1, u2, mc);
                if (__builtin_amdgcn_ballot_w64(!(fabs(m.d) < 4.0 * kWideRange)) != 0)
                    m = slot_mid<2>(r, x0, x1, x2, u0, u1, u2, mc);
            } else {
                m = slot_mid<2>(r, x0, x1, x2, u0, u1, u2, mc);
            }
            Real q = m.q;
            double coef = live ? static_cast<double>(m.coef) : 0.0;
            auto exact = [&] { return stretch_exact_rec(r.p0, r.p1, r.p2, x0, x1, x2, u0, u1, u2); };  // FP64 build
            double s = 0.0;  // the stretch, where damage laws may ask for it
            if constexpr (EXT) {
                if constexpr (FP32) {
                    s = stretch_of(static_cast<double>(q));
                } else if (fabs(m.d) < 4.0 * kWideRange) {
                    // 1 + s = ((1 + d) / (1 - d))^(1/2) = (1 + d) (1 - d^2)^(-1/2): a slot within
                    // the series needs no root and no division
                    const double d = 0.25 * m.d, z = d * d;
                    double p = __builtin_fma(scalar_const(63.0 / 256.0), z, scalar_const(35.0 / 128.0));
                    p = __builtin_fma(p, z, scalar_const(5.0 / 16.0));
                    p = __builtin_fma(p, z, scalar_const(3.0 / 8.0));
                    p = __builtin_fma(p, z, 0.5) * z;
                    s = __builtin_fma(d, p, d + p);
                    q = __builtin_fma(s, s, s + s);
                } else {
                    s = stretch_of(q);
                }
            }
            const bool over = !(q < (FP32 ? static_cast<Real>(q0f) : static_cast<Real>(P.q0)));
            BondWeight bw;
            if constexpr (EXT) {
                if (live && (BREAKS ? (over || soft) : soft))
                    bw = bond_weight<MODE, FP32>(A, P, w.ds, static_cast<double>(q), s, (e & kEntNoFail) != 0, soft, w.sold, exact);
            } else if (BREAKS && live && over) {
                bw.broke = FP32 ? q >= static_cast<Real>(q0f) : exact() >= P.s0;
            }
            coef = bw.broke || bw.share == 0.0 ? 0.0 : coef * bw.share;
            double f0 = 0.0, f1 = 0.0, f2 = 0.0;
            if (coef != 0.0) {
                if (WEIGHT) coef *= static_cast<double>(weight(idx, w.k, m.L2, fv, ow));
                f0 = coef * static_cast<double>(m.y0);
                f1 = coef * static_cast<double>(m.y1);
                f2 = coef * static_cast<double>(m.y2);
            }
            asm volatile("" : "+v"(wn.word), "+v"(wn.sold));
            if (STIFF) asm volatile("" : "+v"(wn.k));
            if (bw.broke) {  // irreversible; the pass is recorded
                A.ent[w.ds] = static_cast<uint16_t>(e | kEntBroken);
                A.bstep[w.ds] = static_cast<int32_t>(*A.step_base + A.step_local);
            } else if (EXT && bw.newly_soft) {
                A.ent[w.ds] = static_cast<uint16_t>(e | kEntSoft);
            }
            if (EXT && bw.grew) A.smax[w.ds] = bw.smax;
            // back to the owners
            if (w.m == 1) {
                S0 += f0;
                S1 += f1;
                S2 += f2;
            } else {
#pragma unroll 1
                for (int j = 0; __builtin_amdgcn_ballot_w64(j < w.n) != 0; ++j) {
                    const double g0 = __shfl(f0, w.at + j), g1 = __shfl(f1, w.at + j), g2 = __shfl(f2, w.at + j);
                    S0 += j < w.n ? g0 : 0.0;
                    S1 += j < w.n ? g1 : 0.0;
                    S2 += j < w.n ? g2 : 0.0;
                }
            }
            w = wn;
        }
        return true;
    };
    // The sentinel's term is exactly zero as long as its distance does not round; a node beyond
    // that takes its slots at level 2 from the start.
    constexpr double kFar = FP32 ? 1e15 : 1e80;
    auto near = [&](double x) { return fabs(x) < kFar; };
    const bool moderate = near(X0) && near(X1) && near(X2) && (FP32 ? near(Uf0) && near(Uf1) && near(Uf2) : near(U0) && near(U1) && near(U2));
    const int first = __builtin_amdgcn_ballot_w64(!moderate) != 0 ? 2 : 0;
    auto share_rows = [&](int2 pr) {  // after fetch(pr.x)
        int t = pr.x, level = first, usual = first > 1 ? 2 : 1;
        base = pr.x;
#pragma unroll 1
        for (;;) {
            const int stop = min(pr.y, base + 32);
            if (level == 2) {
                t = rows_general(t, stop);
                level = usual;
            } else {
                if (level == 0)
                    t = rows(t, stop, std::integral_constant<int, 0>{});
                else if (BREAKS && level == kMark)
                    t = rows(t, stop, std::integral_constant<int, kMark>{});
                else
                    t = rows(t, stop, std::integral_constant<int, 1>{});
                if (t < stop) {
                    level = need;
                    if (level == kMark) usual = kMark;
                    fetch(t);
                }
            }
            if (t < stop) continue;
            const bool settled = settle();
            base = t;
            if (t >= pr.y) break;
            if (settled) fetch(t);  // (not kept in registers meanwhile)
        }
    };
    auto stage_phase = [&](int ph) {  // a later phase
        const int2 pd = phases[T.phase + ph];
        __syncthreads();  // the records before are no longer read
        stage_records(A.rec_in, list + pd.x, pd.y, tl.wv, lane, lrec);
        if (NODEW) stage_doubles(wsrc, list + pd.x, pd.y, tl.wv, lane, lw);
    };

    if (NODEW && T.nphases > 0) stage_doubles(wsrc, list + T.list, T.n, tl.wv, lane, lw);
    int2 pr = int2{0, 0};
#pragma unroll 1
    for (int ph = 0; ph < T.nphases; ++ph) {
        if (ph > 0) stage_phase(ph);
        pr = tl.pairs(T, segs, ph);
        fetch(pr.x);
        tile_staged();
        __builtin_amdgcn_s_setprio(0);
        if (pr.x < pr.y) share_rows(pr);
        __builtin_amdgcn_s_setprio(3);
    }
    double G[3] = {F0 + E0, F1 + E1, F2 + E2};
    tile_reduce(tl, reinterpret_cast<double*>(lds), G);
    if (tl.sub > 0 || !tl.has) return;
    const double share = FP32 ? kMidScale32 * (!WEIGHT || CORR ? P.c * P.volume : 1.0)
                              : kMidScale * (CORR ? 0.25 * P.cr_2v0 : 1.0) *
                                    (KNODE ? A.na[node] : STIFF ? (VOLN ? 1.0 : P.volume) : VOLN ? P.c : P.c * P.volume);
    node_update<MODE, FP32>(A, P, node, U0, U1, U2, share * G[0], share * G[1], share * G[2]);
}

// ---------------------------------------------------------------- launch templates

template <int G, bool STIFF, bool VOLN, bool KNODE, bool EXT>
hipError_t launch_step_gsv(const StepArgs& a, int mode, hipStream_t s)
{
    const dim3 grid(static_cast<unsigned>((a.nslices + 3) / 4)), block(kBlock);
    switch (mode) {
#define PD_L(M) hipLaunchKernelGGL((step_f64<G, M, STIFF, VOLN, KNODE, EXT>), grid, block, 0, s, a)
    case kModeEC: PD_L(kModeEC); break;
    case kModeVV: PD_L(kModeVV); break;
    case kModeVVInit: PD_L(kModeVVInit); break;
    case kModeFE: PD_L(kModeFE); break;
    case kModeForce: PD_L(kModeForce); break;
#undef PD_L
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int G, bool EXT>
hipError_t launch_step_g(const StepArgs& a, int mode, bool stiff, hipStream_t s)
{
    const bool voln = a.vol != nullptr;
    if (a.nw) return launch_step_gsv<G, false, false, true, EXT>(a, mode, s);  // per-node stiffness
    if (stiff)
        return voln ? launch_step_gsv<G, true, true, false, EXT>(a, mode, s)
                    : launch_step_gsv<G, true, false, false, EXT>(a, mode, s);
    return voln ? launch_step_gsv<G, false, true, false, EXT>(a, mode, s)
                : launch_step_gsv<G, false, false, false, EXT>(a, mode, s);
}

template <bool FP32, int MODE, bool STIFF, bool VOLN, bool KNODE, bool EXT, int CORR>
hipError_t launch_staged_m(const StepArgs& a, hipStream_t s)
{
    auto* kernel = &step_staged<FP32, MODE, STIFF, VOLN, KNODE, EXT, CORR>;
    const size_t bytes = tile_lds(a.stage_max, 48 + (VOLN || KNODE || CORR != kCorrNone ? 8 : 0), kTileWaves * kWave * sizeof(uint16_t));
    const hipError_t e = tile_room(reinterpret_cast<const void*>(kernel), bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(a.ntiles)), dim3(kTileWaves * kWave), bytes, s, a, a.tiles,
                       a.phases, a.segs, a.list);
    return hipGetLastError();
}

template <bool FP32, bool STIFF, bool VOLN, bool KNODE, bool EXT, int CORR = kCorrNone>
hipError_t launch_staged_sv(const StepArgs& a, int mode, hipStream_t s)
{
    switch (mode) {
    case kModeEC: return launch_staged_m<FP32, kModeEC, STIFF, VOLN, KNODE, EXT, CORR>(a, s);
    case kModeVV: return launch_staged_m<FP32, kModeVV, STIFF, VOLN, KNODE, EXT, CORR>(a, s);
    case kModeVVInit: return launch_staged_m<FP32, kModeVVInit, STIFF, VOLN, KNODE, EXT, CORR>(a, s);
    case kModeFE: return launch_staged_m<FP32, kModeFE, STIFF, VOLN, KNODE, EXT, CORR>(a, s);
    case kModeForce: return launch_staged_m<FP32, kModeForce, STIFF, VOLN, KNODE, EXT, CORR>(a, s);
    default: return hipErrorInvalidValue;
    }
}

template <bool FP32, bool EXT>
hipError_t launch_staged_n(const StepArgs& a, int mode, hipStream_t s)
{
    const bool stiff = a.kslot != nullptr, voln = a.vol != nullptr;
    if (a.cfv)  // corrections per slot
        return a.partial ? launch_staged_sv<FP32, false, false, false, EXT, kCorrPartial>(a, mode, s)
                         : launch_staged_sv<FP32, false, false, false, EXT, kCorrPlain>(a, mode, s);
    if (a.nw) return launch_staged_sv<FP32, false, false, true, EXT>(a, mode, s);  // per-node stiffness
    if (stiff)
        return voln ? launch_staged_sv<FP32, true, true, false, EXT>(a, mode, s)
                    : launch_staged_sv<FP32, true, false, false, EXT>(a, mode, s);
    return voln ? launch_staged_sv<FP32, false, true, false, EXT>(a, mode, s)
                : launch_staged_sv<FP32, false, false, false, EXT>(a, mode, s);
}

}  // namespace
}  // namespace pdmi
