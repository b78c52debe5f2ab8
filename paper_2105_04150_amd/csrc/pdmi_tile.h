// pdmi_tile.h -- staging of a tile's records in LDS, shared by the step, state-based and
// adjoint kernels of the staged layout.
//
// A tile is one workgroup of eight wavefronts serving one to four slices of 64 nodes.  All
// records that the tile's bonds reach are copied into LDS once (about six a node for 256
// nodes at horizon 3.015, ten for 64), then every slot reads its neighbour there.  A
// slot's record is 48 bytes, read as three 16-byte words.
#pragma once

#include "pdmi_device.h"

#include <mutex>
#include <set>
#include <utility>

namespace pdmi {
namespace {

typedef __attribute__((address_space(3))) void* lds_ptr;

// A wavefront's place in its tile: S of them share a slice's row pairs.
struct TileLane {
    int wv, lane;  // wavefront of the workgroup, lane
    int sh, S;     // wavefronts per slice, log2 and number: 8 for one slice, 4 for two, 2 for three or four
    int k, sub;    // slice of the tile, share of the slice's row pairs
    bool has;      // the slice exists (three slices leave two wavefronts over)
    __device__ __forceinline__ explicit TileLane(const TileRec& t)
    {
        wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
        lane = threadIdx.x & (kWave - 1);
        sh = t.nslices == 1 ? 3 : t.nslices == 2 ? 2 : 1;
        S = 1 << sh;
        k = wv >> sh;
        sub = wv & (S - 1);
        has = k < t.nslices;
    }
    __device__ __forceinline__ int64_t node(const TileRec& t) const
    {
        return static_cast<int64_t>(t.slice + (has ? k : 0)) * kWave + lane;
    }
    // The wavefront's row pairs of a phase: [first, last) of the slice's, split evenly.
    __device__ __forceinline__ int2 pairs(const TileRec& t, const int2* __restrict__ segs, int ph) const
    {
        const int2 g = segs[t.seg + ph * t.nslices + (has ? k : 0)];
        const int n = has ? g.y : 0;
        return int2{g.x + (n * sub >> sh), g.x + (n * (sub + 1) >> sh)};
    }
};

// Sums N values a lane over the S wavefronts of each slice, in a fixed order, through the LDS
// that the staged records leave (every wavefront of the workgroup calls it); the sums end
// up in the slice's first wavefront.
template <int N>
__device__ __forceinline__ void tile_reduce(const TileLane& tl, double* lds, double (&v)[N])
{
    __syncthreads();  // the records are no longer read
    double* r = lds + tl.wv * N * kWave + tl.lane;
    if (tl.sub > 0)
#pragma unroll
        for (int d = 0; d < N; ++d) r[d * kWave] = v[d];
    __syncthreads();
    if (tl.sub > 0) return;
#pragma unroll 1
    for (int s = 1; s < tl.S; ++s) {
        r += N * kWave;
#pragma unroll
        for (int d = 0; d < N; ++d) v[d] += r[d * kWave];
    }
}

// Dynamic LDS of a tile kernel with `per` bytes a record: the phase's records and the
// sentinel and `more` bytes, at least the partial sums of tile_reduce.
inline size_t tile_lds(int32_t stage_max, size_t per, size_t more = 0)
{
    const size_t b = (static_cast<size_t>(stage_max) + 1) * per + more, red = kTileWaves * 3 * kWave * sizeof(double);
    return b > red ? b : red;
}

// Copies SIZE * CH bytes of each of the n listed nodes to consecutive places at dst with direct
// global-to-LDS loads of SIZE bytes a lane; the caller waits.  A wavefront takes blocks of 64
// nodes, each as CH loads, so that a lane's place in the block is fixed; the list entries
// of three blocks (a whole tile of up to 1536 records) are in flight together.
template <int SIZE, int CH>
__device__ __forceinline__ void stage(const void* src, const int32_t* __restrict__ list, int n, int wv, int lane, void* dst)
{
    constexpr int Q = 3, W = kTileWaves * kWave;
    const char* const base = static_cast<const char*>(src);
    uint32_t r[CH], part[CH];  // record of the block, and byte within it, of chunk 64 j + lane
#pragma unroll
    for (int j = 0; j < CH; ++j) {
        r[j] = static_cast<uint32_t>(kWave * j + lane) / static_cast<uint32_t>(CH);
        part[j] = SIZE * (static_cast<uint32_t>(kWave * j + lane) - CH * r[j]);
    }
#pragma unroll 1
    for (int b0 = wv * kWave; b0 < n; b0 += Q * W) {
        int32_t idx[Q][CH];
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int j = 0; j < CH; ++j) idx[q][j] = list[min(b0 + q * W + static_cast<int>(r[j]), n - 1)];
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int j = 0; j < CH; ++j)
                if (b0 + q * W + static_cast<int>(r[j]) < n)
                    __builtin_amdgcn_global_load_lds(
                        base + (__umul24(idx[q][j], SIZE * CH) + part[j]),
                        (lds_ptr)(static_cast<char*>(dst) + (b0 + q * W) * (SIZE * CH) + kWave * SIZE * j), SIZE, 0, 0);
    }
}

// The listed nodes' records to lrec's record 1 on; a double, a pair each to dst's second on.  (No templates: the host's pass of a kernel would check the load's size against
// the host's features.)
__device__ __forceinline__ void stage_records(const double* rec, const int32_t* __restrict__ list, int n, int wv, int lane,
                                              double2* lrec)
{
    stage<16, 3>(rec, list, n, wv, lane, lrec + 3);
}
__device__ __forceinline__ void stage_doubles(const double* src, const int32_t* __restrict__ list, int n, int wv, int lane,
                                              double* dst)
{
    stage<4, 2>(src, list, n, wv, lane, dst + 1);
}
__device__ __forceinline__ void stage_pairs(const double2* src, const int32_t* __restrict__ list, int n, int wv, int lane,
                                            double2* dst)
{
    stage<16, 1>(src, list, n, wv, lane, dst + 1);
}
// After the copies: every wavefront's loads have landed (s_waitcnt vmcnt = 0) and all see them.
__device__ __forceinline__ void tile_staged()
{
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
}

// Sentinel record (index 0; three 16-byte parts) of padding and broken slots: a bond to a far
// node, reflected: y = -xi, so that xi + y and with it the change of the squared length
// are exactly zero, whatever the lane's own position and displacement.
template <bool FP32>
__device__ __forceinline__ double2 sentinel_part(int j)
{
    const double far = FP32 ? static_cast<double>(1e25f) : 1e100;
    if (j == 0) return double2{far, far};
    if (!FP32) return j == 1 ? double2{far, -2.0 * far} : double2{-2.0 * far, -2.0 * far};
    const uint64_t u = __float_as_uint(-2.0f * 1e25f);
    return j == 1 ? double2{far, __longlong_as_double(static_cast<int64_t>(u << 32 | u))}
                  : double2{__longlong_as_double(static_cast<int64_t>(u)), 0.0};
}

// Record indices of a lane's row pair from its two entries (low and high half); broken and
// padding entries (sign bit) become record 0, the sentinel.  FLAGS: entries may carry the
// no-failure bit and the softened one, which leads to the sentinel too.
typedef short short2v __attribute__((ext_vector_type(2)));
template <bool FLAGS>
__device__ __forceinline__ uint32_t live_indices(uint32_t e2)
{
    if (FLAGS) e2 = (e2 | (e2 & 0x20002000u) << 2) & 0x8fff8fffu;
    short2v v;
    __builtin_memcpy(&v, &e2, sizeof v);
    const short2v zero = {0, 0};
    v = __builtin_elementwise_max(v, zero);
    uint32_t r;
    __builtin_memcpy(&r, &v, sizeof r);
    return r;
}

// One staged node record.
struct NodeRec {
    double2 p0, p1, p2;
};
__device__ __forceinline__ NodeRec staged_record(const double2* lrec, uint32_t idx)
{
    const char* const q = reinterpret_cast<const char*>(lrec) + __umul24(idx, 48u);
    return NodeRec{*reinterpret_cast<const double2*>(q), *reinterpret_cast<const double2*>(q + 16),
                   *reinterpret_cast<const double2*>(q + 32)};
}

// Room for `bytes` of dynamic LDS in a kernel's workgroups (asked for once per kernel and
// device: the largest a tile can need).
inline hipError_t tile_room(const void* kernel, size_t bytes)
{
    if (bytes <= 64 * 1024) return hipSuccess;
    static std::mutex mu;
    static std::set<std::pair<int, const void*>> done;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    if (done.count({dev, kernel})) return hipSuccess;
    hipFuncAttributes at{};
    e = hipFuncGetAttributes(&at, kernel);
    if (e == hipSuccess)
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kLdsBytes - static_cast<int>(at.sharedSizeBytes));
    if (e == hipSuccess) done.insert({dev, kernel});
    return e;
}

}  // namespace
}  // namespace pdmi
