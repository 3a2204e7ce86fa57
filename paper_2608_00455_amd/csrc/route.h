// Device-side routing of delta entries through a transfer plan (paper
// sec. 4.2.2): segment lookup, unravel (eq. canonical_unravel), containment
// and ravel (eq. receiver_local_remapping).  Shared by the remap kernel and
// the extract kernel's routing flush; not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dte_internal.h"

namespace dte {
namespace rt {

__device__ __forceinline__ int lane_prefix(uint64_t mask)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Containment a_s <= u < a_s + e of coordinate u in operation o, without
// branches (u < a_s wraps to a large value).  kNd > 0: the segment's
// dimension count, known at compile time; kNd == 0: o.ndim (wave-uniform).
template <int kNd>
__device__ __forceinline__ bool inside(const DevOp& o, const uint32_t* u)
{
    bool in = true;
#pragma unroll
    for (int d = 0; d < DTE_MAX_DIMS; ++d)
        if (kNd > 0 ? d < kNd : d < o.ndim) in = in & (u[d] - o.src_origin[d] < o.extent[d]);
    return in;
}

// Receiver offset of a contained coordinate: u - a_s + a_r raveled over the
// receiver view n_r, plus the view's base (eq. receiver_local_remapping).
template <int kNd>
__device__ __forceinline__ int64_t ravel(const DevOp& o, const uint32_t* u)
{
    uint64_t j = 0;
#pragma unroll
    for (int d = 0; d < DTE_MAX_DIMS; ++d)
        if (kNd > 0 ? d < kNd : d < o.ndim)
            j = j * o.dst_shape[d] + (uint32_t)(u[d] - o.src_origin[d] + o.dst_origin[d]);
    return o.dst_base + (int64_t)j;
}

__device__ __forceinline__ int64_t readlane64(int64_t x, int lane)
{
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)x, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)((uint64_t)x >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The plan's tables are read-only while kernels run: through the constant
// address space, uniform indexes become scalar loads.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* constant(const T* p)
{
    return (const __attribute__((address_space(4))) T*)(uint64_t)p;
}

__device__ __forceinline__ int64_t uniform64(int64_t x) { return readlane64(x, 0); }

// Wave-uniform description of the current segment (scalar registers).
struct SegInfo {
    int64_t lo, hi;      // flat range [lo, hi); empty before the first lookup
    int32_t seg, k0, k1; // operations [k0, k1)
    int32_t nd;          // dimensions of the segment's shape
    uint32_t shape[DTE_MAX_DIMS];
};

// Segment holding the uniform flat offset i0 (0 <= i0 < total).
__device__ __forceinline__ SegInfo find_segment(const PlanView& pl, int64_t i0)
{
    i0 = uniform64(i0);
    const auto begin = constant(pl.seg_begin);
    int32_t s = constant(pl.lookup)[i0 >> pl.shift];
    while (begin[s + 1] <= i0) ++s;
    SegInfo g;
    g.lo = begin[s];
    g.hi = begin[s + 1];
    g.seg = s;
    g.k0 = constant(pl.seg_ops)[s];
    g.k1 = constant(pl.seg_ops)[s + 1];
    g.nd = constant(pl.seg_ndim)[s];
#pragma unroll
    for (int d = 0; d < DTE_MAX_DIMS; ++d)
        g.shape[d] = constant(pl.seg_shape)[(int64_t)s * DTE_MAX_DIMS + d];
    return g;
}

// One operation, wave-uniform (scalar registers).
__device__ __forceinline__ DevOp load_op(const DevOp* ops, int32_t k)
{
    const auto w = constant(reinterpret_cast<const uint32_t*>(ops + __builtin_amdgcn_readfirstlane(k)));
    DevOp o;
    uint32_t* d = reinterpret_cast<uint32_t*>(&o);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(DevOp) / 4); ++i) d[i] = w[i];
    return o;
}

// Rank out.first + r's bucket and shard (r wave-uniform: scalar registers).
struct Bucket {
    int64_t* off;
    uint16_t* val;
    int64_t cap;
    uint16_t* shard;
    int64_t numel;
};

__device__ __forceinline__ Bucket bucket(const RankSlice& out, int r)
{
    return Bucket{out.off[r], out.val[r], out.cap[r], out.shard[r], out.numel[r]};
}

// One routed entry: to position pos < b.cap of its bucket and, where the call
// applies as well, to the rank's shard at once.  The bucket is read once per
// operation: its fields read from the RankSlice for every entry took
// remap_kernel to 102 VGPRs, four waves per SIMD instead of the seven that 72
// allow (remap of 106 M entries 822 -> 686 us, of 17.5 M 173 -> 160, of 6 M in
// odd segments 74 -> 65; without the shard's fields, 64 VGPRs, 697 / 155 / 66).
__device__ __forceinline__ void emit(const Bucket& b, int64_t pos, int64_t j, uint16_t v)
{
    b.off[pos] = j;
    b.val[pos] = v;
    if ((uint64_t)j < (uint64_t)b.numel) __builtin_nontemporal_store(v, b.shard + j);
}

// Unravel a segment-local offset over a row-major shape of nd dimensions
// (eq. canonical_unravel); kNd as for `inside` (kNd == 0: nd).
template <int kNd>
__device__ __forceinline__ void unravel(uint32_t li, int nd, const uint32_t* shape, uint32_t* u)
{
#pragma unroll
    for (int d = DTE_MAX_DIMS - 1; d >= 0; --d) {
        if (kNd > 0 ? d < kNd : d < nd) {
            if (d == 0) {
                u[0] = li;
            } else {
                const uint32_t q = li / shape[d];
                u[d] = li - q * shape[d];
                li = q;
            }
        } else {
            u[d] = 0;
        }
    }
}

// Route one slot lane by lane in groups sharing a segment (used when a
// chunk spans several segments).  Counters: lane r of `runv` holds the
// running count of rank first + r, lane r of `basev` the reserved bucket
// start.  kWrite == false counts outputs; kWrite == true writes them.
// kShapeRegs: unravel over the shape cached in `cache` (else re-read it: the
// caller keeps four scalar registers fewer).
template <bool kWrite, bool kShapeRegs = true>
__device__ __forceinline__ void route_slot(const PlanView& pl, const RankSlice& out, int lane,
                                           int64_t i, uint16_t v, int& runv, int64_t basev,
                                           SegInfo& cache)
{
    bool pending = i >= 0;
    uint64_t pmask = __ballot(pending);
    while (pmask != 0) {
        const int src = __builtin_ctzll(pmask);
        const int64_t i0 = readlane64(i, src);
        if (!(i0 >= cache.lo && i0 < cache.hi)) cache = find_segment(pl, i0);
        const bool mine = pending && i >= cache.lo && i < cache.hi;
        pending = pending && !mine;
        pmask = __ballot(pending);
        uint32_t u[DTE_MAX_DIMS];
        if (kShapeRegs)
            unravel<0>((uint32_t)(i - cache.lo), cache.nd, cache.shape, u);
        else
            unravel<0>((uint32_t)(i - cache.lo),
                       __builtin_amdgcn_readfirstlane(pl.seg_ndim[cache.seg]),
                       pl.seg_shape + (int64_t)cache.seg * DTE_MAX_DIMS, u);
        for (int32_t k = cache.k0; k < cache.k1; ++k) {
            const DevOp o = load_op(pl.ops, k);
            const int r = o.rank - out.first;
            if (r < 0 || r >= out.count) continue;
            const bool in = mine && inside<0>(o, u);
            const uint64_t b = __ballot(in);
            if (b == 0) continue;
            const int start = __builtin_amdgcn_readlane(runv, r);
            if (lane == r) runv += __popcll(b);
            if (kWrite) {
                const int64_t pos = readlane64(basev, r) + start + lane_prefix(b);
                const Bucket dst = bucket(out, r);
                if (in && pos < dst.cap) emit(dst, pos, ravel<0>(o, u), v);
            }
        }
    }
}

}  // namespace rt
}  // namespace dte
