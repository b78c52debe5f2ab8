// pdmi_osb.hip -- the ordinary state-based linear solid (Sec. 8.2): two kernels per time
// step on the staged layout.
//
// The bond force of this model depends on the dilation of both end nodes, a sum over each
// node's whole family, so one pass over the bonds cannot both form and use it (Sec. 8.2:
// two loops, hence two kernels).
//
//   pass 1 (osb_staged<0, ...>): every slot forms its stretch; a slot at or over the
//     critical stretch breaks (outside no-failure zones, not in a force evaluation); the
//     node sums |xi| e V over its intact bonds into the dilation theta_i = 3 V / m_i sum and
//     writes the node pair {a_i, b_i - a_i}, a = (3K - 5G) theta / m, b = 15 G / m (a force
//     evaluation for the dilation readout: theta alone).
//   pass 2 (osb_staged<1, ...>): every intact slot adds
//       (t_ij + t_ji) y / |y| V,   t_ij + t_ji = |xi| [(3K - 5G)(A_i + A_j) + 15 G s (B_i + B_j)]
//     with A = theta / m, B = 1 / m, s = e / |xi| the stretch, then the node integrates
//     (the same tail as the bond-based step kernels).
//
// Both passes use the tiles of the bond-based step (pdmi_tile.h): a slice of 64 nodes, one
// lane a node, the records that the tile's bonds reach in LDS; pass 2 copies the node pairs
// beside them.  Influence function 1; a uniform node volume per instance, or per-node
// volumes copied into LDS beside the records (V_j enters the dilation sum and the force
// term).  FP64, or the FP32 build: bond arithmetic in single precision from the f32
// displacements of the records and the f64 coordinates, the node pairs and the integration
// (f64 master displacement) as in FP64.
//
// Per slot, with S = |y|^2 + |xi|^2, tq = |y|^2 - |xi|^2 and d = tq / S (as in the bond-based
// kernels; z = d^2):
//   pass 1: |xi| e = |xi| (|y| - |xi|) = (tq / 2) [1 - d (1/2 + z/8 + z^2/16 + ...)];
//   pass 2: g = 1 - |xi|/|y| = d - (1 - d) (z/2 + 3z^2/8 + 5z^3/16 + ...), and with
//     (s / (1 + s)) = g the force term is
//     (t_ij + t_ji) V y / |y| = V [(a_i + a_j) + g ((b_i - a_i) + (b_j - a_j))] y,
//     the |xi| of the scalar state cancelling the 1 / |xi| of y / |y|.
// A share of rows goes by short series (|d| < kMidRange, FP32 build kMidRange32) up to the
// first block with a slot beyond them or at the decision edge, then by longer ones, and a
// blocks with slots beyond those too slot by slot.
#include "pdmi_step.h"

namespace pdmi {
namespace {

// sqrt(1+q) - 1 without cancellation, any q.
template <typename Real>
__device__ __forceinline__ Real sqrt1p_minus1(Real q)
{
    if constexpr (std::is_same_v<Real, float>) {
        return q * __builtin_amdgcn_rcpf(1.0f + __builtin_sqrtf(1.0f + q));
    } else {
        const double r = rsq64<2>(1.0 + q);
        return q * rcp64(__builtin_fma(1.0 + q, r, 1.0));
    }
}

// One slot: its bond vectors and d.
template <typename Real>
struct OsbTerm {
    Real y0, y1, y2, L2, tq, d;
};

__device__ __forceinline__ OsbTerm<double> osb_term(const NodeRec& n, double X0, double X1, double X2, double U0, double U1,
                                                    double U2)
{
    const double xi0 = n.p0.x - X0, xi1 = n.p0.y - X1, xi2 = n.p1.x - X2;
    const double e0 = n.p1.y - U0, e1 = n.p2.x - U1, e2 = n.p2.y - U2;
    OsbTerm<double> m;
    m.y0 = xi0 + e0;
    m.y1 = xi1 + e1;
    m.y2 = xi2 + e2;
    m.L2 = __builtin_fma(xi2, xi2, __builtin_fma(xi1, xi1, xi0 * xi0));
    const double Y2 = __builtin_fma(m.y2, m.y2, __builtin_fma(m.y1, m.y1, m.y0 * m.y0));
    m.tq = Y2 - m.L2;
    const double S = Y2 + m.L2;
    const double r = __builtin_amdgcn_rcp(S);
    const double d = m.tq * r;
    m.d = __builtin_fma(d, __builtin_fma(-S, r, 1.0), d);
    return m;
}

__device__ __forceinline__ OsbTerm<float> osb_term32(const NodeRec& n, double X0, double X1, double X2, float U0, float U1,
                                                     float U2)
{
    const float xi0 = static_cast<float>(n.p0.x - X0), xi1 = static_cast<float>(n.p0.y - X1),
                xi2 = static_cast<float>(n.p1.x - X2);
    const uint64_t b1 = __double_as_longlong(n.p1.y), b2 = __double_as_longlong(n.p2.x);
    const float e0 = __uint_as_float(static_cast<uint32_t>(b1)) - U0, e1 = __uint_as_float(static_cast<uint32_t>(b1 >> 32)) - U1,
                e2 = __uint_as_float(static_cast<uint32_t>(b2)) - U2;
    OsbTerm<float> m;
    m.y0 = xi0 + e0;
    m.y1 = xi1 + e1;
    m.y2 = xi2 + e2;
    const float z0 = xi0 + m.y0, z1 = xi1 + m.y1, z2 = xi2 + m.y2;
    m.tq = __builtin_fmaf(e2, z2, __builtin_fmaf(e1, z1, e0 * z0));
    m.L2 = __builtin_fmaf(xi2, xi2, __builtin_fmaf(xi1, xi1, xi0 * xi0));
    m.d = m.tq * __builtin_amdgcn_rcpf(__builtin_fmaf(2.0f, m.L2, m.tq));
    return m;
}

// 2 |xi| e / tq = 1 - (1 - sqrt(1 - d^2)) / d and g = d P - (P - 1), P = (1 - d^2)^(-1/2), by their
// series (WIDE: to kWideRange, with the further terms left out where |d| < kMidRange: a
// slot's form follows from its own d alone, so that a bond's two slots agree).
template <typename Real>
__device__ __forceinline__ bool osb_short(Real d)
{
    if constexpr (std::is_same_v<Real, float>)
        return fabsf(d) < static_cast<float>(kMidRange32);
    else
        return fabs(d) < kMidRange;
}
template <bool WIDE, typename Real>
__device__ __forceinline__ Real osb_extension(Real d)
{
    constexpr bool FP32 = std::is_same_v<Real, float>;
    const Real z = d * d;
    Real p = FP32 ? Real(1.0 / 8.0) : Real(1.0 / 16.0);
    if constexpr (WIDE) {
        Real t = __builtin_elementwise_fma(Real(7.0 / 256.0), z, Real(5.0 / 128.0));
        if constexpr (FP32) t = __builtin_elementwise_fma(t, z, Real(1.0 / 16.0));
        t = osb_short(d) ? Real(0) : t;
        p = __builtin_elementwise_fma(t, z, p);
    }
    if constexpr (!FP32) p = __builtin_elementwise_fma(p, z, Real(1.0 / 8.0));
    p = __builtin_elementwise_fma(p, z, Real(0.5));
    return __builtin_elementwise_fma(-d, p, Real(1));
}
template <bool WIDE, typename Real>
__device__ __forceinline__ Real osb_g(Real d)
{
    constexpr bool FP32 = std::is_same_v<Real, float>;
    const Real z = d * d;
    Real p = FP32 ? Real(3.0 / 8.0) : Real(5.0 / 16.0);
    if constexpr (WIDE) {
        Real t = __builtin_elementwise_fma(Real(63.0 / 256.0), z, Real(35.0 / 128.0));
        if constexpr (FP32) t = __builtin_elementwise_fma(t, z, Real(5.0 / 16.0));
        t = osb_short(d) ? Real(0) : t;
        p = __builtin_elementwise_fma(t, z, p);
    }
    if constexpr (!FP32) p = __builtin_elementwise_fma(p, z, Real(3.0 / 8.0));
    p = __builtin_elementwise_fma(p, z, Real(0.5));
    p *= z;  // P - 1
    return __builtin_elementwise_fma(d, p, d - p);
}

template <bool FP32, int PASS, int MODE, bool VOLN>
__global__ __launch_bounds__(kTileWaves * kWave, 4) void osb_staged(StepArgs A, const TileRec* __restrict__ tiles,
                                                                    const int2* __restrict__ phases,
                                                                    const int2* __restrict__ segs,
                                                                    const int32_t* __restrict__ list)
{
    using Real = std::conditional_t<FP32, float, double>;
    extern __shared__ double2 lds[];
    constexpr int B = kPairsAhead;
    constexpr bool BREAKS = PASS == 0 && MODE != kModeForce;
    __builtin_amdgcn_s_setprio(3);  // a tile's staging before another's rows
    const TileRec T = tiles[wave_uniform(xcd_remap(blockIdx.x, gridDim.x))];
    const TileLane tl(T);
    const int lane = tl.lane;
    double2* const lrec = lds;
    double2* const lpair = lrec + 3 * (A.stage_max + 1);  // pass 2: node pairs
    double* const lvol = reinterpret_cast<double*>(lpair + (PASS == 1 ? A.stage_max + 1 : 0));
    if (T.nphases > 0) stage_records(A.rec_in, list + T.list, T.n, tl.wv, lane, lrec);
    const InstParams& P = A.params[T.inst];
    const int64_t node = tl.node(T);
    const double2* __restrict__ rin = reinterpret_cast<const double2*>(A.rec_in);
    const double2 o0 = rin[3 * node], o1 = rin[3 * node + 1], o2 = rin[3 * node + 2];
    const double X0 = o0.x, X1 = o0.y, X2 = o1.x;
    const double U0 = o1.y, U1 = o2.x, U2 = o2.y;  // FP64 build
    const uint64_t ub1 = __double_as_longlong(o1.y), ub2 = __double_as_longlong(o2.x);
    const float Uf0 = __uint_as_float(static_cast<uint32_t>(ub1)), Uf1 = __uint_as_float(static_cast<uint32_t>(ub1 >> 32)),
                Uf2 = __uint_as_float(static_cast<uint32_t>(ub2));  // FP32 build
    const uint32_t* __restrict__ ent = reinterpret_cast<const uint32_t*>(A.ent) + lane;
    const double2* __restrict__ pairs_in = A.osb;
    const double2 own = PASS == 1 ? pairs_in[node] : double2{0.0, 0.0};
    const Real Pa = static_cast<Real>(own.x), Pd = static_cast<Real>(own.y);
    const float q0f = static_cast<float>(P.q0);
    // where a slot's series end, as high words of its d (hi_edge is of 4 d: two exponents more)
    const int32_t edge = !BREAKS ? std::numeric_limits<int32_t>::max() : FP32 ? P.hi_edge32 : max(P.hi_edge, 0x00200000) - 0x00200000;
    constexpr uint32_t range = range_bits<FP32>(0.25 * kMidRange, kMidRange32), wrange = range_bits<FP32>(0.25 * kWideRange, kWideRange32);
    const int32_t hi_pos = min(static_cast<int32_t>(range), edge), hi_wpos = min(static_cast<int32_t>(wrange), edge);
    constexpr uint32_t hi_neg = 0x80000000u | range, hi_wneg = 0x80000000u | wrange;

    // sentinel record, its pair and volume zero
    if (threadIdx.x < 3) lrec[threadIdx.x] = sentinel_part<FP32>(threadIdx.x);
    if (PASS == 1 && threadIdx.x == 0) lpair[0] = double2{0.0, 0.0};
    if (VOLN && threadIdx.x == 0) lvol[0] = 0.0;

    Real D = 0;                  // pass 1: sum of 2 |xi| e (V_j) over intact bonds
    Real F0 = 0, F1 = 0, F2 = 0;  // pass 2: force density (uniform volume: without the factor V)
    auto term = [&](const NodeRec& r) {
        if constexpr (FP32)
            return osb_term32(r, X0, X1, X2, Uf0, Uf1, Uf2);
        else
            return osb_term(r, X0, X1, X2, U0, U1, U2);
    };
    // adds the term of a slot: v = 2 |xi| e in pass 1, g in pass 2
    auto add = [&](const OsbTerm<Real>& m, uint32_t idx, Real v) {
        const Real vj = VOLN ? static_cast<Real>(lvol[idx]) : Real(1);
        if (PASS == 0) {
            D = VOLN ? __builtin_elementwise_fma(vj, v, D) : D + v;
        } else {
            const double2 pj = lpair[idx];
            Real c = __builtin_elementwise_fma(v, Pd + static_cast<Real>(pj.y), Pa + static_cast<Real>(pj.x));
            c = idx != 0 ? c : Real(0);  // padding and broken slots
            const Real coef = VOLN ? vj * c : c;
            F0 = __builtin_elementwise_fma(coef, m.y0, F0);
            F1 = __builtin_elementwise_fma(coef, m.y1, F1);
            F2 = __builtin_elementwise_fma(coef, m.y2, F2);
        }
    };
    auto series = [&](const OsbTerm<Real>& m, auto wide) {
        return PASS == 0 ? m.tq * osb_extension<decltype(wide)::value>(m.d) : osb_g<decltype(wide)::value>(m.d);
    };
    auto high = [&](const OsbTerm<Real>& m) {
        if constexpr (FP32)
            return static_cast<int32_t>(__float_as_uint(m.d));
        else
            return static_cast<int32_t>(__double_as_longlong(m.d) >> 32);
    };
    auto one = [&](const NodeRec& r, uint32_t idx, auto wide) {
        const OsbTerm<Real> m = term(r);
        add(m, idx, series(m, wide));
        return high(m);
    };
    auto ent_at = [&](int t) { return ent[static_cast<int64_t>(t) * kWave]; };
    // One block or more from pair t on, with a look at every slot at the decision edge or beyond the
    // long series; goes on as long as blocks have slots beyond it.
    auto rows_apart = [&](int t, int end, bool always) {
        int block = t + B;
        bool far = false;
        uint32_t e2 = ent_at(t), en = t + 1 < end ? ent_at(t + 1) : 0x80008000u;
        NodeRec r = staged_record(lrec, live_indices<true>(e2) & 0xffffu);
        int h = 0;
#pragma unroll 1
        while (t < end) {
            const uint32_t e = h ? e2 >> 16 : e2 & 0xffffu;
            const NodeRec rn = staged_record(lrec, h ? live_indices<true>(en) & 0xffffu : live_indices<true>(e2) >> 16);
            const OsbTerm<Real> m = term(r);
            Real v = series(m, std::true_type{});
            bool live = !(e & kEntBroken);
            const int32_t hi = high(m);
            const bool beyond = live && (hi >= hi_wpos || static_cast<uint32_t>(hi) >= hi_wneg);
            far |= live && (hi >= static_cast<int32_t>(wrange) || static_cast<uint32_t>(hi) >= hi_wneg);
            if (__builtin_amdgcn_ballot_w64(beyond) != 0 && beyond) {
                Real q;
                if constexpr (FP32)
                    q = m.tq * __builtin_amdgcn_rcpf(m.L2);
                else
                    q = m.tq * rcp64(m.L2);
                if (BREAKS && !(e & kEntNoFail) && !(q < (FP32 ? static_cast<Real>(q0f) : static_cast<Real>(P.q0)))) {
                    if (FP32 ? q >= static_cast<Real>(q0f) : stretch_exact_rec(r.p0, r.p1, r.p2, X0, X1, X2, U0, U1, U2) >= P.s0) {
                        const int64_t ds = static_cast<int64_t>(t) * (2 * kWave) + 2 * lane + h;
                        A.ent[ds] = static_cast<uint16_t>(e | kEntBroken);
                        A.bstep[ds] = static_cast<int32_t>(*A.step_base + A.step_local);
                        live = false;
                    }
                }
                if (!(__builtin_elementwise_abs(m.d) < static_cast<Real>(FP32 ? kWideRange32 : kWideRange))) {
                    if (PASS == 0)
                        v = Real(2) * m.L2 * sqrt1p_minus1(q);
                    else if constexpr (FP32)
                        v = 1.0f - __builtin_amdgcn_rsqf(1.0f + q);
                    else
                        v = one_minus_rsqrt1p(q, series_coef_sregs());
                }
            }
            if (live) add(m, e & kEntIdx, v);
            r = rn;
            h ^= 1;
            if (h == 0) {
                ++t;
                e2 = en;
                en = t + 1 < end ? ent_at(t + 1) : 0x80008000u;
                if (t == block) {
                    if (!always && __builtin_amdgcn_ballot_w64(far) == 0) break;
                    far = false;
                    block += B;
                }
            }
        }
        return t;
    };
    uint32_t en[B];  // the next block's entries
    auto fetch = [&](int t) {
#pragma unroll
        for (int u = 0; u < B; ++u) en[u] = (ent + static_cast<int64_t>(t) * kWave)[u * kWave];
    };
    // The pairs [t, end), after fetch(t), block by block by the short or the long series, up to
    // the first block with a slot that it does not cover; that block is taken back (covered: the
    // long series does).
    bool covered = true;
    auto rows = [&](int t, int end, auto wide) {
        const int32_t pos = wide ? hi_wpos : hi_pos;
        const uint32_t neg = wide ? hi_wneg : hi_neg;
#pragma unroll 1
        for (; t < end; t += B) {
            uint32_t e[B];
#pragma unroll
            for (int u = 0; u < B; ++u) e[u] = en[u];
            fetch(t + B);
            const Real S = D, S0 = F0, S1 = F1, S2 = F2;
            int32_t himax = std::numeric_limits<int32_t>::min();
            uint32_t himin = 0;
            uint32_t v = live_indices<true>(e[0]);
            NodeRec ra = staged_record(lrec, v & 0xffffu);
#pragma unroll
            for (int u = 0; u < B; ++u) {
                if (t + u >= end) break;
                const uint32_t ia = v & 0xffffu, ib = v >> 16;
                const NodeRec rb = staged_record(lrec, ib);
                // (past the share's end: another share's entry, read but not added)
                if (u + 1 < B) v = live_indices<true>(e[u + 1]);
                __builtin_amdgcn_sched_barrier(0);
                const int32_t ha = one(ra, ia, wide);
                if (u + 1 < B) ra = staged_record(lrec, v & 0xffffu);
                __builtin_amdgcn_sched_barrier(0);
                const int32_t hb = one(rb, ib, wide);
                himax = max(max(himax, ha), hb);
                himin = max(max(himin, static_cast<uint32_t>(ha)), static_cast<uint32_t>(hb));
            }
            if (__builtin_amdgcn_ballot_w64(himax >= pos || himin >= neg) != 0) {
                D = S;
                F0 = S0;
                F1 = S1;
                F2 = S2;
                covered = __builtin_amdgcn_ballot_w64(himax >= hi_wpos || himin >= hi_wneg) == 0;
                return t;
            }
        }
        return end;
    };
    // The sentinel's term is exactly zero as long as its distance does not round; a node beyond
    // that takes its slots apart, where padding and broken ones add nothing.
    constexpr double kFar = FP32 ? 1e15 : 1e80;
    auto near = [&](double x) { return fabs(x) < kFar; };
    const bool moderate = near(X0) && near(X1) && near(X2) && (FP32 ? near(Uf0) && near(Uf1) && near(Uf2) : near(U0) && near(U1) && near(U2));
    const bool apart = __builtin_amdgcn_ballot_w64(!moderate) != 0;
    auto share_rows = [&](int2 pr) {  // after fetch(pr.x)
        if (apart) {
            rows_apart(pr.x, pr.y, true);
            return;
        }
        int t = rows(pr.x, pr.y, std::false_type{});
#pragma unroll 1
        while (t < pr.y) {  // once the short series does not do, the long one for the rest
            if (covered) {
                fetch(t);
                t = rows(t, pr.y, std::true_type{});
                if (t >= pr.y) break;
            }
            t = rows_apart(t, pr.y, false);
            covered = true;
        }
    };
    auto stage_weights = [&](const int32_t* l, int n) {
        if (PASS == 1) stage_pairs(pairs_in, l, n, tl.wv, lane, lpair);
        if (VOLN) stage_doubles(A.vol, l, n, tl.wv, lane, lvol);
    };
    auto stage_phase = [&](int ph) {  // a later phase
        const int2 pd = phases[T.phase + ph];
        __syncthreads();  // the records before are no longer read
        stage_records(A.rec_in, list + pd.x, pd.y, tl.wv, lane, lrec);
        stage_weights(list + pd.x, pd.y);
    };

    if (T.nphases > 0) stage_weights(list + T.list, T.n);
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
    if constexpr (PASS == 0) {
        double E[1] = {D};
        tile_reduce(tl, reinterpret_cast<double*>(lds), E);
        if (tl.sub > 0 || !tl.has) return;
        // theta_i = 3 V sum / m_i (per-node volumes: inside the sum); padding nodes (1/m = 0) write zeros
        const double b = A.minv[node];
        const double theta = VOLN ? 1.5 * E[0] * b : (1.5 * P.volume) * E[0] * b;
        const double a = P.osb_a * (theta * b);
        A.osb[node] = MODE == kModeForce && A.force == nullptr ? double2{theta, 0.0} : double2{a, P.osb_b * b - a};
    } else {
        double G[3] = {F0, F1, F2};
        tile_reduce(tl, reinterpret_cast<double*>(lds), G);
        if (tl.sub > 0 || !tl.has) return;
        const double V = VOLN ? 1.0 : P.volume;
        node_update<MODE, FP32>(A, P, node, U0, U1, U2, V * G[0], V * G[1], V * G[2]);
    }
}

template <bool FP32, int PASS, int MODE, bool VOLN>
hipError_t launch_osb_pmv(const StepArgs& a, hipStream_t s)
{
    auto* kernel = &osb_staged<FP32, PASS, MODE, VOLN>;
    const size_t bytes = tile_lds(a.stage_max, 48 + (PASS == 1 ? 16 : 0) + (VOLN ? 8 : 0));
    const hipError_t e = tile_room(reinterpret_cast<const void*>(kernel), bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(a.ntiles)), dim3(kTileWaves * kWave), bytes, s, a, a.tiles,
                       a.phases, a.segs, a.list);
    return hipGetLastError();
}

template <bool FP32, int PASS, int MODE>
hipError_t launch_osb_pm(const StepArgs& a, hipStream_t s)
{
    return a.vol ? launch_osb_pmv<FP32, PASS, MODE, true>(a, s) : launch_osb_pmv<FP32, PASS, MODE, false>(a, s);
}

template <bool FP32>
hipError_t launch_osb_step_p(const StepArgs& a, int mode, hipStream_t s)
{
    hipError_t e = mode != kModeForce ? launch_osb_pm<FP32, 0, kModeEC>(a, s)
                                      : launch_osb_pm<FP32, 0, kModeForce>(a, s);
    if (e != hipSuccess) return e;
    switch (mode) {
    case kModeEC: return launch_osb_pm<FP32, 1, kModeEC>(a, s);
    case kModeVV: return launch_osb_pm<FP32, 1, kModeVV>(a, s);
    case kModeVVInit: return launch_osb_pm<FP32, 1, kModeVVInit>(a, s);
    case kModeFE: return launch_osb_pm<FP32, 1, kModeFE>(a, s);
    case kModeForce: return launch_osb_pm<FP32, 1, kModeForce>(a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_osb_dilation(const StepArgs& args, bool breaking, bool fp32, hipStream_t s)
{
    StepArgs a = args;
    a.force = nullptr;  // the readout: theta itself
    if (a.ntiles <= 0) return hipSuccess;
    if (fp32)
        return breaking ? launch_osb_pm<true, 0, kModeEC>(a, s) : launch_osb_pm<true, 0, kModeForce>(a, s);
    return breaking ? launch_osb_pm<false, 0, kModeEC>(a, s) : launch_osb_pm<false, 0, kModeForce>(a, s);
}

hipError_t launch_osb_step(const StepArgs& a, int mode, bool fp32, hipStream_t s)
{
    if (a.ntiles <= 0) return hipSuccess;
    return fp32 ? launch_osb_step_p<true>(a, mode, s) : launch_osb_step_p<false>(a, mode, s);
}

}  // namespace pdmi
