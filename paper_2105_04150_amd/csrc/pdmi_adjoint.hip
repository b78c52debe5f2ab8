// pdmi_adjoint.hip -- reverse pass of the Euler-Cromer step with a frozen break schedule.
//
// Forward pass k (Sec. 2, Eq. simpleBond, with the semi-implicit Euler update):
//   v^{k+1} = d v^k + h (F(u^k; k) + A bhat),  u^{k+1} = u^k + dt v^{k+1},
//   then the boundary conditions overwrite prescribed components,
// with h = dt/rho and d = 1 - dt eta/rho.  A slot acts in pass k iff k < bstep (the pass
// in which it broke).  Reverse pass k, given lam_u = dL/du^{k+1} and the adjoint nu of
// the unconstrained v^{k+1} (zero on prescribed components):
//   dL/dk_b += h V_j (s/r)_b (y_b . nu_i)          (f_b = k_b V_j (s/r) y)
//   dL/dA   += h bhat_i . nu_i
//   lam_u    = [0 on displacement-controlled components] lam_u + h J_F^T nu
//   nu'      = d nu + dt lam_u on free components, 0 on prescribed ones (pass k-1)
// The tangent of one slot is k_b K_b with K_b = (1/L - 1/r) I + y y^T / r^3, symmetric and
// even in y.  With symmetric stiffness and schedule, (J_F^T nu)_i is the gather
//   sum over the family of i of k_b K_b (V_i nu_j - V_j nu_i),
// the same shape as the force, so the reverse pass walks the forward slot layout and
// needs no reverse-slot index.  1/L - 1/r = (1/L)(1 - (1+q)^(-1/2)) uses
// q = |y|^2/|xi|^2 - 1 with the numerator formed without cancellation, eta.(xi + y), and
// 1/r is 1/L less that.
#include "pdmi_tile.h"

namespace pdmi {
namespace {

// One slot: adds k_b K_b (V_i nu_j - V_j nu_i) to J and returns the slot's
// stiffness-gradient increment h V_j (s/r) (y . nu_i).  An inactive slot (broken in an
// earlier pass, or padding) evaluates q = 0 with zero weights and adds nothing.
__device__ __forceinline__ double adj_slot(bool active, const double2 p0, const double2 p1, const double2 p2,
                                           double X0, double X1, double X2, double U0, double U1, double U2,
                                           const double nj[3], const double ni[3], double Vi, double Vj, double kb,
                                           double h, double J[3])
{
    const double xi0 = p0.x - X0, xi1 = p0.y - X1, xi2 = p1.x - X2;
    const double e0 = p1.y - U0, e1 = p2.x - U1, e2 = p2.y - U2;
    const double y0 = xi0 + e0, y1 = xi1 + e1, y2 = xi2 + e2;
    const double z0 = xi0 + y0, z1 = xi1 + y1, z2 = xi2 + y2;
    const double tq = __builtin_fma(e2, z2, __builtin_fma(e1, z1, e0 * z0));
    const double L2 = __builtin_fma(xi2, xi2, __builtin_fma(xi1, xi1, xi0 * xi0));
    const double iL = rsq64<1>(L2);
    const double q = active ? tq * (iL * iL) : 0.0;
    const double sr = iL * one_minus_rsqrt1p(q, series_coef_sregs());  // s/r = 1/L - 1/r
    const double ir = iL - sr;                    // 1/r, no cancellation: sr is about |s| of iL
    const double ir3 = ir * ir * ir;
    const double w0 = Vi * nj[0] - Vj * ni[0], w1 = Vi * nj[1] - Vj * ni[1], w2 = Vi * nj[2] - Vj * ni[2];
    const double yw = __builtin_fma(y2, w2, __builtin_fma(y1, w1, y0 * w0));
    const double ka = active ? kb : 0.0;
    const double a = ka * sr, b = ka * (yw * ir3);
    J[0] += a * w0 + b * y0;
    J[1] += a * w1 + b * y1;
    J[2] += a * w2 + b * y2;
    const double yn = __builtin_fma(y2, ni[2], __builtin_fma(y1, ni[1], y0 * ni[0]));
    return active ? h * Vj * sr * yn : 0.0;
}

// Adjoint velocities: nn + 1 pairs (components 0 and 1), then nn + 1 third components (the last
// node, the sentinel, zero): a 16-byte and an 8-byte load a node, also on its way into LDS.
__device__ __forceinline__ void nu_load(const double* nu, int64_t nn, int64_t node, double (&n)[3])
{
    const double2 a = reinterpret_cast<const double2*>(nu)[node];
    n[0] = a.x;
    n[1] = a.y;
    n[2] = nu[2 * (nn + 1) + node];
}
__device__ __forceinline__ void nu_store(double* nu, int64_t nn, int64_t node, const double (&n)[3])
{
    reinterpret_cast<double2*>(nu)[node] = double2{n[0], n[1]};
    nu[2 * (nn + 1) + node] = n[2];
}

// Node tail of a reverse pass: body-force gradient, boundary masks, lam_u and next nu.
__device__ __forceinline__ void adj_node(const AdjArgs& A, const InstParams& P, int64_t node, const double ni[3],
                                         const double J[3], double h)
{
    const int32_t bcid = A.bc_id[node];
    if (bcid == kNodePad) return;
    const int64_t nn = A.nn;
    int code = 0;
    if (bcid >= 0) code = A.bc[bcid].code;
    if (P.has_body)
        A.gacc[node] += h * (A.bhat[node] * ni[0] + A.bhat[nn + node] * ni[1] + A.bhat[2 * nn + node] * ni[2]);
    const double damp = 1.0 - A.dt * P.eta / P.rho;
    double out[3];
    for (int d = 0; d < 3; ++d) {
        const int kind = (code >> (2 * d)) & 3;
        const double lu = A.lam_u[d * nn + node];
        const double ln = (kind == 1 ? 0.0 : lu) + h * J[d];
        A.lam_u[d * nn + node] = ln;
        out[d] = kind == 0 ? damp * ni[d] + A.dt * ln : 0.0;
    }
    nu_store(A.nu_out, nn, node, out);
}

// Per-slot streams of one row (index ds) and the neighbour data they point at.
struct AdjRow {
    int64_t ds;
    bool active;
    double kb, g;
    double2 p0, p1, p2;
    double nj[3];
    double Vj;
};

// Stiffness of a slot: KM = kKUniform (c), kKSlot (per-slot array) or kKNode
// (sqrt(k_i) sqrt(k_j) from per-node factors; ai = sqrt(k_i) of the own node).
constexpr int kKUniform = 0, kKSlot = 1, kKNode = 2;

template <int KM, bool VOLN>
__device__ __forceinline__ void adj_load(const AdjArgs& A, const InstParams& P, double ai, int64_t ds, int64_t j,
                                         AdjRow& r)
{
    const double2* __restrict__ rec = reinterpret_cast<const double2*>(A.rec);
    r.ds = ds;
    r.active = A.k < static_cast<int64_t>(A.bstep[ds]);
    r.p0 = rec[3 * j];
    r.p1 = rec[3 * j + 1];
    r.p2 = rec[3 * j + 2];
    nu_load(A.nu_in, A.nn, j, r.nj);
    r.kb = KM == kKSlot ? A.kslot[ds] : KM == kKNode ? ai * A.na[j] : P.c;
    r.Vj = VOLN ? A.vol[j] : P.volume;
    r.g = A.grad[ds];
}

// Sliced layout: G lanes per node, partial sums meet in a shuffle butterfly.  Two rows
// are loaded before either is computed (every slice's row count is even and the slot
// arrays end with spare rows, so the loads stay in bounds); padding slots point at the
// sentinel record, whose adjoint velocity is zero.
template <int G, int KM, bool VOLN>
__global__ __launch_bounds__(kBlock) void adjoint_sliced(AdjArgs A)
{
    constexpr int W = kWave / G;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t slice =
        wave_uniform(xcd_remap(blockIdx.x, gridDim.x) * (kBlock / kWave) + (threadIdx.x >> 6));
    if (slice >= A.nslices) return;
    const InstParams P = A.params[A.slice_inst[slice]];
    const int w = lane / G, g = lane % G;
    const int64_t node = slice * W + w;
    const double2* __restrict__ rec = reinterpret_cast<const double2*>(A.rec);
    const double2 o0 = rec[3 * node], o1 = rec[3 * node + 1], o2 = rec[3 * node + 2];
    double ni[3];
    nu_load(A.nu_in, A.nn, node, ni);
    const double Vi = VOLN ? A.vol[node] : P.volume;
    const double ai = KM == kKNode ? A.na[node] : 0.0;
    const double h = A.dt / P.rho;
    const int64_t base = wave_uniform(A.slice_ptr[slice]);
    const int T = A.slice_T[slice];
    double J[3] = {0.0, 0.0, 0.0};
    for (int t = 0; t < T; t += 2) {
        AdjRow r[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t ds = base + static_cast<int64_t>(t + u) * kWave + lane;
            const int32_t c = A.col[ds];
            adj_load<KM, VOLN>(A, P, ai, ds, static_cast<int32_t>(col_node(c)), r[u]);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const double d = adj_slot(r[u].active, r[u].p0, r[u].p1, r[u].p2, o0.x, o0.y, o1.x, o1.y, o2.x, o2.y,
                                      r[u].nj, ni, Vi, r[u].Vj, r[u].kb, h, J);
            if (r[u].active) A.grad[r[u].ds] = r[u].g + d;
        }
    }
#pragma unroll
    for (int m = 1; m < G; m <<= 1)
        for (int d = 0; d < 3; ++d) J[d] += __shfl_xor(J[d], m);
    if (g != 0) return;
    adj_node(A, P, node, ni, J, h);
}

typedef int int2v __attribute__((ext_vector_type(2)));
typedef double double2v __attribute__((ext_vector_type(2)));
template <bool NT, typename V>
__device__ __forceinline__ V stream_load(const V* p)
{
    if constexpr (NT)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}

// Staged layout: one workgroup a tile (pdmi_tile.h), one lane a node, 2 to 8 wavefronts
// a slice.  The tile's records (x, u^k), adjoint velocities and per-node weights are copied into LDS
// once; the per-slot streams (entries, break steps, stiffness, gradient: 22 to 30 bytes a
// slot, the pass's bound beside latency) come a row pair ahead, 16 bytes a lane and load.
// Padding entries point at the sentinel (far record, zero adjoint velocity and weights).
// Partial sums of J meet in LDS in a fixed order.
// NT: the streams bypass the caches, for problems whose streams exceed them anyway (they then
// leave the nodes' records in L2; 54M slots: 431 us a pass, 383 with, 5.4M: 42.5 and 48.9).
// With the scalar addresses and three loads a node for its adjoint velocity 5.4M slots take 38.9,
// with six loads and four addresses a lane 42.8.
template <int KM, bool VOLN, bool NT>
__global__ __launch_bounds__(kTileWaves * kWave, 4) void adjoint_lds(AdjArgs A, const TileRec* __restrict__ tiles,
                                                                     const int2* __restrict__ phases,
                                                                     const int2* __restrict__ segs,
                                                                     const int32_t* __restrict__ list)
{
    constexpr bool KNODE = KM == kKNode, STIFF = KM == kKSlot;
    extern __shared__ double2 lds[];
    __builtin_amdgcn_s_setprio(3);  // a tile's staging before another's rows
    const TileRec T = tiles[wave_uniform(xcd_remap(blockIdx.x, gridDim.x))];
    const TileLane tl(T);
    const int lane = tl.lane;
    double2* const lrec = lds;
    const int R = A.stage_max + 1;
    double2* const lnu = lrec + 3 * R;                            // components 0 and 1
    double* const lnu2 = reinterpret_cast<double*>(lnu + R);      // 2
    double* const lvol = lnu2 + R;
    double* const lna = lvol + (VOLN ? R : 0);
    auto stage_weights = [&](const int32_t* l, int n) {
        stage_pairs(reinterpret_cast<const double2*>(A.nu_in), l, n, tl.wv, lane, lnu);
        stage_doubles(A.nu_in + 2 * (A.nn + 1), l, n, tl.wv, lane, lnu2);
        if (VOLN) stage_doubles(A.vol, l, n, tl.wv, lane, lvol);
        if (KNODE) stage_doubles(A.na, l, n, tl.wv, lane, lna);
    };
    if (T.nphases > 0) {
        stage_records(A.rec, list + T.list, T.n, tl.wv, lane, lrec);
        stage_weights(list + T.list, T.n);
    }
    const InstParams& P = A.params[T.inst];
    // the parameters that every slot needs as scalars, once: the kernel's own stores make the
    // compiler load them again for every row pair otherwise
    const auto& Q = *(const __attribute__((address_space(4))) InstParams*)(A.params + T.inst);
    double c = Q.c, volume = Q.volume, h = A.dt / Q.rho;
    asm volatile("" : "+s"(c), "+s"(volume));
    const int64_t node = tl.node(T);
    const double2* __restrict__ rec = reinterpret_cast<const double2*>(A.rec);
    const double2 o0 = rec[3 * node], o1 = rec[3 * node + 1], o2 = rec[3 * node + 2];
    double ni[3];
    nu_load(A.nu_in, A.nn, node, ni);
    const double Vi = VOLN ? A.vol[node] : volume;
    const double ai = KNODE ? A.na[node] : 0.0;

    // sentinels: record far from every node; zero adjoint velocity and weights
    if (threadIdx.x < 3) {
        lrec[threadIdx.x] = threadIdx.x == 0 ? double2{1e10, 1e10} : threadIdx.x == 1 ? double2{1e10, 0.0} : double2{0.0, 0.0};
    }
    if (threadIdx.x == 0) {
        lnu[0] = double2{0.0, 0.0};
        lnu2[0] = 0.0;
    }
    if (VOLN && threadIdx.x == 0) lvol[0] = 0.0;
    if (KNODE && threadIdx.x == 0) lna[0] = 0.0;

    double J[3] = {0.0, 0.0, 0.0};
    const int32_t k = static_cast<int32_t>(A.k);
    struct Streams {
        uint32_t e;
        int2 bs;
        double2 kr, gr;
    };
    // a row pair's words: uniform addresses, the lane as their offset (four addresses a lane are
    // eight registers, which the loop does not have)
    auto pair_of = [&](auto* p, int t) { return p + static_cast<int64_t>(t) * (2 * kWave); };
    auto streams = [&](int t) {
        const int2v bs = stream_load<NT>(reinterpret_cast<const int2v*>(pair_of(A.bstep, t)) + lane);
        const double2v kr = STIFF ? stream_load<NT>(reinterpret_cast<const double2v*>(pair_of(A.kslot, t)) + lane) : double2v{0.0, 0.0};
        const double2v gr = stream_load<NT>(reinterpret_cast<const double2v*>(pair_of(A.grad, t)) + lane);
        return Streams{reinterpret_cast<const uint32_t*>(pair_of(A.ent, t))[lane], int2{bs.x, bs.y}, double2{kr.x, kr.y},
                       double2{gr.x, gr.y}};
    };
    auto slot = [&](const NodeRec& r, uint32_t idx, bool active, double kr) {
        const double2 n01 = lnu[idx];
        const double nj[3] = {n01.x, n01.y, lnu2[idx]};
        const double kb = STIFF ? kr : KNODE ? ai * lna[idx] : c;
        const double Vj = VOLN ? lvol[idx] : volume;
        return adj_slot(active, r.p0, r.p1, r.p2, o0.x, o0.y, o1.x, o1.y, o2.x, o2.y, nj, ni, Vi, Vj, kb, h, J);
    };
#pragma unroll 1
    for (int ph = 0; ph < T.nphases; ++ph) {
        if (ph > 0) {
            const int2 pd = phases[T.phase + ph];
            __syncthreads();  // the records before are no longer read
            stage_records(A.rec, list + pd.x, pd.y, tl.wv, lane, lrec);
            stage_weights(list + pd.x, pd.y);
        }
        const int2 pr = tl.pairs(T, segs, ph);
        Streams a = streams(pr.x);  // spare rows follow the last slice's
        tile_staged();
        __builtin_amdgcn_s_setprio(0);
#pragma unroll 1
        for (int t = pr.x; t < pr.y; ++t) {
            const Streams b = streams(t + 1);
            const uint32_t ia = a.e & kEntIdx, ib = (a.e >> 16) & kEntIdx;
            const double da = slot(staged_record(lrec, ia), ia, k < a.bs.x, a.kr.x);
            __builtin_amdgcn_sched_barrier(0);  // the two interleaved do not fit the registers
            const double db = slot(staged_record(lrec, ib), ib, k < a.bs.y, a.kr.y);
            // inactive slots keep their gradient (the increment is zero)
            double2v* const out = reinterpret_cast<double2v*>(pair_of(A.grad, t)) + lane;
            const double2v sum{a.gr.x + da, a.gr.y + db};
            if constexpr (NT)
                __builtin_nontemporal_store(sum, out);
            else
                *out = sum;
            a = b;
        }
        __builtin_amdgcn_s_setprio(3);
    }
    tile_reduce(tl, reinterpret_cast<double*>(lds), J);
    if (tl.sub > 0 || !tl.has) return;
    adj_node(A, P, node, ni, J, h);
}

__global__ __launch_bounds__(kBlock) void bstep_init_kernel(int32_t* bstep, const int32_t* col, const uint16_t* ent,
                                                            int64_t ns)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= ns) return;
    const bool broken = col ? col[i] < 0 : (ent[i] & kEntBroken) != 0;
    bstep[i] = broken ? kBrokeBefore : kNeverBroke;
}

__global__ __launch_bounds__(kBlock) void flags_at_kernel(const int32_t* bstep, int32_t* col, uint16_t* ent,
                                                          int64_t ns, int64_t step)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= ns) return;
    const bool broken = static_cast<int64_t>(bstep[i]) < step;
    if (col) {
        const int32_t c = col[i], j = c ^ (c >> 31);
        col[i] = broken ? ~j : j;
    } else {
        const uint16_t e = ent[i];
        ent[i] = static_cast<uint16_t>((e & ~kEntBroken) | (broken ? kEntBroken : 0));
    }
}

__global__ void adj_seed_kernel(double* lam_u, int64_t nn, const int64_t* sensors, const double* dldu, int64_t m)
{
    const int d = threadIdx.x;
    if (blockIdx.x != 0 || d >= 3) return;
    for (int64_t p = 0; p < m; ++p) lam_u[d * nn + sensors[p]] += dldu[3 * p + d];
}

__global__ __launch_bounds__(kBlock) void adj_nu0_kernel(double* nu, const double* lam_u, const int32_t* bc_id,
                                                         const BCRec* bc, int64_t nn, double dt)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (i >= nn) return;
    const int32_t id = bc_id[i];
    const int code = id >= 0 ? bc[id].code : 0;
    double out[3];
    for (int d = 0; d < 3; ++d) {
        const bool free_comp = id != kNodePad && ((code >> (2 * d)) & 3) == 0;
        out[d] = free_comp ? dt * lam_u[d * nn + i] : 0.0;
    }
    nu_store(nu, nn, i, out);
}

// Deterministic single-workgroup sum.
__global__ __launch_bounds__(kBlock) void sum_kernel(const double* x, int64_t n, double* out)
{
    __shared__ double part[kBlock];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += kBlock) acc += x[i];
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kBlock / 2; s > 0; s >>= 1) {
        if (static_cast<int>(threadIdx.x) < s) part[threadIdx.x] += part[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = part[0];
}

__global__ void set_i64_kernel(int64_t* p, int64_t v)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

template <int G, int KM, bool VOLN>
void adj_launch_sliced(const AdjArgs& a, hipStream_t s)
{
    hipLaunchKernelGGL((adjoint_sliced<G, KM, VOLN>), dim3(static_cast<unsigned>((a.nslices + 3) / 4)),
                       dim3(kBlock), 0, s, a);
}

constexpr int64_t kCacheBytes = int64_t(256) << 20;  // the memory-side cache
template <int KM, bool VOLN>
hipError_t adj_launch_staged(const AdjArgs& a, hipStream_t s)
{
    const bool nt = a.ns * (2 + 4 + 8 + (KM == kKSlot ? 8 : 0)) > kCacheBytes;
    auto* kernel = nt ? &adjoint_lds<KM, VOLN, true> : &adjoint_lds<KM, VOLN, false>;
    const size_t bytes = tile_lds(a.stage_max, 48 + 24 + (VOLN ? 8 : 0) + (KM == kKNode ? 8 : 0));
    const hipError_t e = tile_room(reinterpret_cast<const void*>(kernel), bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(a.ntiles)), dim3(kTileWaves * kWave), bytes, s, a, a.tiles,
                       a.phases, a.segs, a.list);
    return hipGetLastError();
}

template <int KM, bool VOLN>
hipError_t adj_launch_kv(const AdjArgs& a, bool staged, int lanes, hipStream_t s)
{
    if (staged) return adj_launch_staged<KM, VOLN>(a, s);
    switch (lanes) {
    case 1: adj_launch_sliced<1, KM, VOLN>(a, s); break;
    case 4: adj_launch_sliced<4, KM, VOLN>(a, s); break;
    case 16: adj_launch_sliced<16, KM, VOLN>(a, s); break;
    case 64: adj_launch_sliced<64, KM, VOLN>(a, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int KM>
hipError_t adj_launch_k(const AdjArgs& a, bool staged, int lanes, hipStream_t s)
{
    return a.vol ? adj_launch_kv<KM, true>(a, staged, lanes, s) : adj_launch_kv<KM, false>(a, staged, lanes, s);
}

unsigned blocks_for(int64_t n) { return static_cast<unsigned>((n + kBlock - 1) / kBlock); }

}  // namespace

hipError_t launch_adjoint(const AdjArgs& a, bool staged, int lanes, hipStream_t s)
{
    if (a.nslices <= 0) return hipSuccess;
    if (a.kslot) return adj_launch_k<kKSlot>(a, staged, lanes, s);
    if (a.na) return adj_launch_k<kKNode>(a, staged, lanes, s);
    return adj_launch_k<kKUniform>(a, staged, lanes, s);
}

hipError_t launch_bstep_init(int32_t* bstep, const int32_t* col, const uint16_t* ent, int64_t ns, hipStream_t s)
{
    if (ns <= 0) return hipSuccess;
    hipLaunchKernelGGL(bstep_init_kernel, dim3(blocks_for(ns)), dim3(kBlock), 0, s, bstep, col, ent, ns);
    return hipGetLastError();
}

hipError_t launch_flags_at(const int32_t* bstep, int32_t* col, uint16_t* ent, int64_t ns, int64_t step, hipStream_t s)
{
    if (ns <= 0) return hipSuccess;
    hipLaunchKernelGGL(flags_at_kernel, dim3(blocks_for(ns)), dim3(kBlock), 0, s, bstep, col, ent, ns, step);
    return hipGetLastError();
}

hipError_t launch_adj_seed(double* lam_u, int64_t nn, const int64_t* sensors, const double* dldu, int64_t m,
                           hipStream_t s)
{
    if (m <= 0) return hipSuccess;
    hipLaunchKernelGGL(adj_seed_kernel, dim3(1), dim3(kWave), 0, s, lam_u, nn, sensors, dldu, m);
    return hipGetLastError();
}

hipError_t launch_adj_nu0(double* nu, const double* lam_u, const int32_t* bc_id, const BCRec* bc, int64_t nn,
                          double dt, hipStream_t s)
{
    if (nn <= 0) return hipSuccess;
    hipLaunchKernelGGL(adj_nu0_kernel, dim3(blocks_for(nn)), dim3(kBlock), 0, s, nu, lam_u, bc_id, bc, nn, dt);
    return hipGetLastError();
}

hipError_t launch_sum(const double* x, int64_t n, double* out, hipStream_t s)
{
    hipLaunchKernelGGL(sum_kernel, dim3(1), dim3(kBlock), 0, s, x, n, out);
    return hipGetLastError();
}

hipError_t launch_set_i64(int64_t* p, int64_t value, hipStream_t s)
{
    hipLaunchKernelGGL(set_i64_kernel, dim3(1), dim3(kWave), 0, s, p, value);
    return hipGetLastError();
}

}  // namespace pdmi
