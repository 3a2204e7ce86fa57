// Delta extraction for gfx950: AdamW inversion (paper sec. 4.1,
// eq. adamw_inverse), BF16 quantisation and bit comparison (sec. 4.2.1,
// eq. canonical_delta_detection) and stream compaction of the changed
// elements, fused in one streaming pass over theta, m, v.
//
// Design (HBM-bound: 12 bytes read per element, ~10 bytes written per
// changed element):
//  - persistent grid of one block of 12 waves per CU (three per SIMD: the
//    block's queues and staging areas take the CU's whole LDS; the 47 to 124
//    VGPRs would allow four and more); each wave owns one contiguous range of
//    256-element slots (one float4 per lane), ranges ascending with the global
//    wave number, so every wave's entries leave in ascending order; in the
//    unordered call over 48 slots per wave and more the static ranges leave
//    out the last 1/16 of the slots, which blocks then take 8 or 32 slots per
//    wave at a time from a counter (the CUs do not stream at one rate, and a
//    static split leaves the fast ones idle at the end);
//    a wave keeps two slots of p, m and v in flight, reloading each slot's
//    registers as soon as it is tested;
//  - proof of "unchanged" before exact arithmetic: with DECAY == 1 the
//    reconstruction is ph = RN(p + u), where u has the sign of m and
//    |u| <= B; B comes from the hardware square root and reciprocal (about
//    1 ulp each), inflated by 2^-16, plus 2^-126; RN and BF16 rounding are
//    monotone, so if RN(p + sign(m) B) has the BF16 pattern of p, so has ph.
//    (DECAY != 1: the same interval is pushed through the division with a
//    bracketing reciprocal of DECAY.)  Lanes without that proof
//    (candidates, about as many as the changed elements) queue
//    (p, m, v, position) in LDS; a wave evaluates 64 queued candidates at a
//    time with the correctly rounded inverse.  The result is bit-identical
//    to evaluating every element exactly.  When theta_hat is requested every
//    element takes the exact path;
//  - the predicate of one float4 slot of the wave (256 consecutive
//    elements) is four ballots; an element's position among the slot's
//    selected elements is the sum of mbcnt over the four ballots (lanes
//    before it) plus its own selected predecessors in the lane, so
//    candidates are queued, and changed entries (32-bit position +
//    BF16 value) staged in LDS, in ascending element order: every wave's
//    output is ascending.  In the unordered call the waves of a block meet
//    every one to four passes over the ring and, once they hold enough
//    entries, reserve output space for all of them with one atomicAdd on the
//    64-bit cursor (block_round below); each wave writes its run after those
//    of the waves before it, coalesced.  A wave whose staging area (kWaveStage entries)
//    fills between two meetings flushes exactly kWaveStage entries on its
//    own with one atomicAdd;
//  - ordered mode: the waves of a block still meet every four passes (a
//    barrier alone), which keeps them in step; each wave writes its
//    flushes to a region of the workspace of its own (no atomics) and,
//    once that is full, to a shared
//    area, recording (position, entries of the wave before it, count,
//    wave); a scan of the wave totals and a copy of the regions and
//    recorded runs then give the entries in ascending offset order
//    (order_scan_kernel, order_copy_kernel below), deterministic whatever
//    the timing of the atomics.
#include <hip/hip_runtime.h>

#include "dte_internal.h"
#include "route.h"

#pragma clang fp contract(off)

namespace dte {
namespace {

constexpr int kWaves = 12;                    // waves per block, one block per CU
// float4 slots in flight per lane and array.  Measured with 8 / 4 / 3 / 2 (386
// M elements, us): lr 1e-6 698 / 691 / 689 / 678, 1e-5 767 / 759 / 762 /
// 757, 1e-4 906 / 894 / 890 / 883; 44 M elements in 13 odd ranges 330 / 299
// / 296 / 285: the code of a pass grows with it, and 12 waves keep the HBM
// queues full with two.
constexpr int kVec = 2;
constexpr int kSlot = 256;                    // elements of one slot of a wave (a float4 per lane)
constexpr int kQueue = 320;                   // queued candidates per wave (16 bytes each)
constexpr int kDrain = 64;                    // queued candidates that are drained after a slot
// Slots per wave before another block is added: every block ends with one
// atomicAdd on the caller's cursor, and 256 of these in a row take about
// 10 us.  2 M elements (zeroing the cursor and the call, between events):
// 33.8 us with 1 slot per wave (256 blocks), 34.1 with 2, 28.8 with 4
// (163 blocks), 29.3 with 8; 1e5 elements 22.8 / 23.0 / 23.8 / 25.0.
constexpr int kMinSlots = 4;
// what is left undrained (fewer than kDrain) and a slot's 4 x 64 elements
// must fit the queue; the part of a slot left after one flush of the
// staging area must fit the emptied area
static_assert(kQueue >= kDrain - 1 + kSlot, "a slot's candidates must fit the queue");
static_assert(kWaveStage >= kSlot, "a slot's changed entries must fit after one flush");

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));   // element-aligned
typedef const __attribute__((address_space(1))) f32x4_any* global_f32x4;
typedef const __attribute__((address_space(1))) float* global_f32;

constexpr int kForwardBlock = 256;
constexpr int64_t kForwardBlocks = (int64_t)1 << 23;   // 2^31 threads, within a launch's limit
// Elements above which the forward step goes past the caches: the last-level
// cache (256 MB) holds the four arrays up to 2^24.  Through / past the
// caches, us: 8 M 31.9 / 38.5, 16 M 60.6 / 82.5, 25 M 136 / 118, 50 M 269 /
// 240, 193 M 984 / 891.
constexpr int64_t kForwardStream = (int64_t)1 << 24;

// Adaptive step term u = (lrb1*m) / (sqrt(v*rbc2) + eps): four binary32
// operations, each rounded once (sqrt and divide correctly rounded).
__device__ __forceinline__ float step_term(float m, float v, float lrb1, float rbc2, float eps)
{
    const float vh = v * rbc2;
    const float sq = __builtin_sqrtf(vh);
    const float den = sq + eps;
    const float num = lrb1 * m;
    return num / den;
}

// The same term in the literal order of eq. adamw_inverse:
// lr * ((m / bc1) / (sqrt(v / bc2) + eps)), six binary32 operations.
__device__ __forceinline__ float step_term_literal(float m, float v, float lr, float bc1, float bc2,
                                                   float eps)
{
    const float mh = m / bc1;
    const float vq = v / bc2;
    const float sq = __builtin_sqrtf(vq);
    const float d = sq + eps;
    const float r = mh / d;
    return lr * r;
}

// BF16 pattern of x: round to nearest even on the binary32 pattern; any NaN
// gives 0x7FC0.  (For non-NaN x the 32-bit sum cannot wrap.)
__device__ __forceinline__ uint32_t bf16_bits(float x)
{
    const uint32_t u = __float_as_uint(x);
    const uint32_t r = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    return (x != x) ? 0x7FC0u : r;
}

using rt::lane_prefix;   // set lanes of the mask below this lane

// True only if b(ph) == b(p) is proven without the exact inverse (see the
// header).  B bounds |u| from above: hardware sqrt / reciprocal (about one
// ulp each) and two roundings, covered by the factor 1 + 2^-16; flushed or
// overflowing intermediates make B non-finite or too large, never too small,
// except a reciprocal flushed to zero, covered by the floor 2^-126 (a |u|
// below it cannot move a |p| >= 2^-100, and a smaller |p| fails the test).
//
// Literal order: the same B bounds the literal u when every intermediate of
// both evaluations is a normal number (each then carries one rounding of
// relative error, about ten in all, far inside 2^-16).  The host allows the
// proof only when eps >= 2^-40, lr <= 2^20 and both bias corrections are
// >= 2^-20.  Then d = sqrt(v/bc2) + eps >= 2^-40, so a subnormal v/bc2
// moves d by at most 2^-75 (relative 2^-35); subnormal m/bc1, lrb1*m or
// m/bc1/d move u by at most 2^-125/eps in all, the floor (`floor`, set by
// the host) used instead of 2^-126; |m| <= 2^64 keeps m/bc1 and m/bc1/d
// finite (other elements take the exact path); v*rbc2 is clamped to the
// largest finite value so that it cannot overflow where v/bc2 does not
// (a NaN stays NaN).
//
// DECAY != 1: theta_hat = RN(w / DECAY) for some w between p and hi, so it
// lies between the smallest and the largest of p, hi, p / DECAY and
// hi / DECAY.  Where p and hi have one sign (else hi's pattern differs) the
// two outer ones of these are, for DECAY < 1, the smaller magnitude of p
// and hi themselves and the larger magnitude times an upper bracket of
// 1 / DECAY; for DECAY > 1 the larger magnitude itself and the smaller
// times a lower bracket.  p has its own pattern, so testing hi and that
// product tests both ends.  `rd` is the bracket; the median of (p, hi,
// far) as unsigned patterns is the larger magnitude for far = 2^32 - 1 and
// the smaller for far = 0.
template <bool kDecayOne, bool kLit>
__device__ __forceinline__ bool proven_unchanged(float p, float m, float v, const StepScalars& a)
{
    const float num = a.lrb1 * m;
    float vh = v * a.rbc2;
    if (kLit) vh = vh > 0x1.fffffep127f ? 0x1.fffffep127f : vh;
    const bool in_range = !kLit || (__float_as_uint(m) & 0x7FFFFFFFu) <= 0x5F800000u;
    const float den = __builtin_amdgcn_sqrtf(vh) + a.eps;
    const float q = __builtin_fabsf(num) * __builtin_amdgcn_rcpf(den);
    const float b = __builtin_fmaf(q, 1.0000153f, kLit ? a.floor : 0x1p-126f);   // NaN stays NaN
    const float hi = p + __builtin_copysignf(b, m);
    const uint32_t up = __float_as_uint(p), uh = __float_as_uint(hi);
    const uint32_t rp = up + 0x7FFFu + ((up >> 16) & 1u);
    const uint32_t rh = uh + 0x7FFFu + ((uh >> 16) & 1u);
    if (kDecayOne) return in_range & ((rp ^ rh) < 0x10000u);
    const uint32_t small = up < uh ? up : uh, large = up < uh ? uh : up;
    const uint32_t capped = large < a.far ? large : a.far;
    const uint32_t outer = small > capped ? small : capped;      // median
    const uint32_t uy = __float_as_uint(__uint_as_float(outer) * a.rd);
    const uint32_t ry = uy + 0x7FFFu + ((uy >> 16) & 1u);
    return in_range & (((rp ^ rh) | (rp ^ ry)) < 0x10000u);
}

// Exact inverse and change test of one element (sec. 4.1 / 4.2.1).
template <bool kDecayOne, bool kLit>
__device__ __forceinline__ float exact_prev(float p, float m, float v, const StepScalars& a)
{
    const float u = kLit ? step_term_literal(m, v, a.lr, a.bc1, a.bc2, a.eps)
                         : step_term(m, v, a.lrb1, a.rbc2, a.eps);
    const float num = p + u;
    return kDecayOne ? num : num / a.decay;
}

constexpr int64_t kDenseRatio = 64;             // see write_staged

// Dynamic tail of the unordered call: when the waves have at least
// kTailSlots slots each, the last total / kTailDiv slots (at most 2^23, so
// that an element's offset from the tail's start fits a staging key; the
// partial slot among them) go to blocks chunk_slots per wave per grab.  A grab adds
// 2^kGrabShift to the caller's cursor, whose bits below kGrabShift count the
// entries (a delta never reaches 2^36 entries): the old value's high bits
// number the chunk, every reservation masks them off, and the block whose
// grab is the last of all (each block's last grab finds no chunk) takes
// them out again.
// Where the line lies: the tail evens out the blocks' ends but costs each of
// them a meeting and at least one more grab.  With the tail / without, us: 25
// M elements (32 slots per wave) lr 1e-6 54.0 / 51.0, 1e-4 65.3 / 61.6, with
// theta_hat 91.6 / 87.6, six runs 71.5 / 65.2; 30 M (38) 61.1 / 57.9, 73.9 /
// 71.1, 106.9 / 103.5, 78.9 / 74.7; 40 M (51) 78.3 / 76.0, 93.2 / 94.0, 132 /
// 139, 98.4 / 97.3; 60 M (76) 111.5 / 110.7, 136.8 / 140.3, 200 / 206, 141.7 /
// 143.5; 110 M (140) 195 / 202, 256 / 267; 200 M (254) 350 / 363, 454 / 473.
constexpr int64_t kTailDiv = 16;
constexpr int64_t kTailSlots = 48;
constexpr int64_t kMaxTailSlots = (int64_t)1 << 23;
// Slots per wave of one grab: few (one meeting's passes) let the blocks end
// together, but a wave's entries from the tail are then short pieces far
// apart, and where a delta is sparse and the plan has many segments remap
// routes them lane by lane.  With 8 / 16 / 32 / 64: extract of 38 M elements
// 74.5 / 78.1 / 87.9 / 110.8 us, of 320 M 562 / 564 / 568 / 576, of 772 M 1328
// / 1327 / 1329 / 1339; remap of 787 M elements in ten layers of 64 experts, lr 1e-6
// 78 / 65 / 63 / -, of twelve Qwen3-30B-A3B layers (7477 M, 0.087 % change) 314
// / 196 / 140 / 139, their extract 13430 / 13424 / 13364 / 13337, remap of
// sixteen Qwen3-8B layers (3104 M) 201 / 198 / 189 / 174.  In between both show:
// 289 M elements extract 525 / 527 / 526 and remap 62 / 60 / 44 in six equal
// layers, 512 / 515 / 516 and 39 / 40 / 42 in three layers of another layout.
// So the longer grabs where the tail has kLongTail slots per wave (604 M
// elements in all), where they cost extract nothing.
constexpr int64_t kChunkSlots = 8, kLongChunkSlots = 32;
constexpr int64_t kLongTail = 48;
constexpr int kGrabShift = 36;
constexpr unsigned long long kCountMask = (1ull << kGrabShift) - 1;

__device__ inline int64_t tail_slots(int64_t slots, int64_t waves)
{
    const int64_t d = slots >= kTailSlots * waves ? slots / kTailDiv : 0;
    return d < kMaxTailSlots ? d : kMaxTailSlots;
}

__device__ inline int64_t chunk_slots(int64_t tail, int64_t waves)
{
    return tail >= kLongTail * waves ? kLongChunkSlots : kChunkSlots;
}

// Per-wave LDS areas.  Keys are element offsets from element `base` of the
// range: the wave's first element, in the dynamic tail the tail's.
struct WaveStage {
    uint32_t* key;    // output staging: changed entries awaiting a flush
    uint16_t* val;
    f32x4* queue;     // candidates, elements without an "unchanged" proof: p, m, v, key
    int64_t base;
    int32_t wave;     // global wave number
};

// Wave-uniform output state: entries staged in LDS, entries flushed so far;
// ordered mode: entries written to the wave's region, and whether the region
// is exhausted (then every later flush goes to the shared area).
struct Staging {
    int staged;
    int64_t flushed;
    int64_t met;        // entries staged in all at the block's last meeting
    int64_t in_region;
    int spilled;
};

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Write staged entries [0, staged) to out_idx / out_val from position
// base, dropping those at or beyond capacity; kStream: offsets with
// non-temporal stores.
template <bool kStream>
__device__ __forceinline__ void write_out(const ExtractParams& a, const WaveStage& st, int64_t base,
                                          int staged, int lane)
{
    const int64_t x0 = a.index_base + st.base;
    for (int i = lane; i < staged; i += 64) {
        const int64_t pos = base + i;
        if (pos < a.capacity) {
            const int64_t x = x0 + (int64_t)st.key[i];
            if (kStream)
                __builtin_nontemporal_store(x, a.out_idx + pos);
            else
                a.out_idx[pos] = x;
            a.out_val[pos] = st.val[i];
        }
    }
}

// Write a wave's staged entries (so.staged > 0) to positions base, base + 1,
// ...  A wave that has so far found more than one changed element per
// kDenseRatio elements scanned writes its offsets with non-temporal stores
// (measured faster on deltas of several percent of the state, slower on
// sparse ones); the choice is wave-uniform.
__device__ __forceinline__ void write_staged(const ExtractParams& a, const WaveStage& st,
                                             Staging& so, int64_t base, int lane)
{
    const int staged = so.staged;
    const uint32_t last = __builtin_amdgcn_readfirstlane(st.key[staged - 1]);
    const int64_t scanned = (int64_t)last + 1;
    if ((so.flushed + staged) * kDenseRatio > scanned)
        write_out<true>(a, st, base, staged, lane);
    else
        write_out<false>(a, st, base, staged, lane);
    so.flushed += staged;
    so.staged = 0;
    wave_sync();   // the staging area is rewritten next: finish these reads first
}

// Copy a wave's staged LDS entries to the reserved global range (and, in
// ordered mode, record the run).  Routing mode: route them through the plan
// into the receiver buckets instead (count, one reservation per rank, write).
template <bool kRoute>
__device__ void flush_wave(const ExtractParams& a, const WaveStage& st, Staging& so, int lane)
{
    const int staged = so.staged;
    wave_sync();   // every lane's LDS stores visible to the other lanes
    if (kRoute) {
        rt::SegInfo cache{};
        int runv = 0;                            // lane r: entries for rank out.first + r
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {
            int64_t basev = 0;
            if (pass == 1) {
                if (lane < a.out.count && runv > 0)
                    basev = (int64_t)atomicAdd(reinterpret_cast<unsigned long long*>(
                                                   &a.rank_count[a.out.first + lane]),
                                               (unsigned long long)runv);
                runv = 0;
            }
#pragma unroll 1
            for (int g = 0; g < staged; g += 64) {
                const int i = g + lane;
                int64_t x = -1;
                uint16_t y = 0;
                if (i < staged) {
                    x = a.index_base + st.base + (int64_t)st.key[i];
                    y = st.val[i];
                    if (x >= a.plan.total) x = -1;
                }
                if (pass == 0)
                    rt::route_slot<false, false>(a.plan, a.out, lane, x, y, runv, 0, cache);
                else
                    rt::route_slot<true, false>(a.plan, a.out, lane, x, y, runv, basev, cache);
            }
        }
        so.flushed += staged;
        so.staged = 0;
        wave_sync();
        return;
    }
    if (a.runs && !so.spilled) {
        if (so.flushed + staged <= a.region_size) {
            // ordered mode: the wave's own region, no atomics (reservations
            // that every wave takes from one address slow the whole stream)
            const int64_t r0 = (int64_t)st.wave * a.region_size + so.flushed;
            for (int i = lane; i < staged; i += 64) {
                a.region_idx[r0 + i] = a.index_base + st.base + (int64_t)st.key[i];
                a.region_val[r0 + i] = st.val[i];
            }
            so.flushed += staged;
            so.in_region = so.flushed;
            so.staged = 0;
            wave_sync();
            return;
        }
        so.spilled = 1;
    }
    unsigned long long base = 0;
    if (lane == 0) {
        base = atomicAdd(reinterpret_cast<unsigned long long*>(a.cursor),
                         (unsigned long long)staged) & kCountMask;
        if (a.runs) {
            const unsigned long long r =
                atomicAdd(reinterpret_cast<unsigned long long*>(a.run_cursor), 1ull);
            if ((int64_t)r < a.max_runs) {
                OrderRun run;
                run.src = (int64_t)base;
                run.woff = so.flushed;
                run.count = staged;
                run.wave = st.wave;
                a.runs[r] = run;
            }
        }
    }
    base = __shfl(base, 0);
    write_staged(a, st, so, (int64_t)base, lane);
}

// Selection of the four elements of each lane's float4 slot (256
// consecutive elements per wave): one ballot per element of the float4 and
// the slot's count.
struct Slot4 {
    uint64_t ball[4];
    int count;
};

__device__ __forceinline__ Slot4 select4(const bool (&sel)[4])
{
    Slot4 r;
    r.count = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        r.ball[c] = __ballot(sel[c]);
        r.count += __popcll(r.ball[c]);
    }
    return r;
}

// Selected elements of the slot in lanes below this one: the position of
// this lane's first selected element; its others follow in element order.
__device__ __forceinline__ int lanes_before(const Slot4& r)
{
    uint32_t before = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        before = __builtin_amdgcn_mbcnt_hi((uint32_t)(r.ball[k] >> 32),
                                           __builtin_amdgcn_mbcnt_lo((uint32_t)r.ball[k], before));
    return (int)before;
}

// Stage one ballot of changed entries (at most 64), flushing first when the
// staging area would overflow.  Wave-uniform control flow.
template <bool kRoute>
__device__ __forceinline__ void stage_changed(const ExtractParams& a, const WaveStage& st,
                                              Staging& so, int lane, bool changed,
                                              uint32_t key, uint16_t val)
{
    const uint64_t k = __ballot(changed);
    if (k == 0) return;
    const int cnt = __popcll(k);
    const int before = so.staged;
    const int pos = before + lane_prefix(k);
    if (changed && pos < kWaveStage) {
        st.key[pos] = key;
        st.val[pos] = val;
    }
    if (before + cnt < kWaveStage) {
        so.staged = before + cnt;
        return;
    }
    // the staging area is full: flush exactly kWaveStage entries (so every
    // flush but a wave's last is one full, aligned block), then stage the rest
    so.staged = kWaveStage;
    flush_wave<kRoute>(a, st, so, lane);
    if (changed && pos >= kWaveStage) {
        st.key[pos - kWaveStage] = key;
        st.val[pos - kWaveStage] = val;
    }
    so.staged = before + cnt - kWaveStage;
}

// Combined flushes of the unordered call.  Every kRound passes over the ring
// (fewer in dense ranges), and once at the end, the waves of a block meet at a
// barrier; when they hold at least kFlushPerWave entries per wave (at the end:
// any), one atomicAdd on the cursor reserves room for all of them and each
// wave writes its entries after those of the waves before it.  Every wave of the device reserving
// its own space from the one cursor address is what slows the stream (the
// atomics, not the stores), so fewer, larger reservations are the point; a
// wave whose staging area fills between two meetings still flushes on its
// own.  Block-uniform control flow; the two LDS slots alternate, so a slot
// is rewritten only after every wave has passed a later barrier.
constexpr int kRound = 4;
constexpr int kFlushPerWave = 768;            // block flush threshold per wave
// Entries that a wave finds between two meetings: those of kRound passes, of
// candidates left in the queue before them and of the range's partial slot.
constexpr int kMaxFound = kRound * kVec * kSlot + kDrain - 1 + kSlot;
static_assert(kMaxFound < 1 << 15 && kWaveStage < 1 << 16, "block_round packs both in one int");

// Returns the number of passes until the next meeting: as many (up to
// kRound) as leave room for what the block's waves found per pass since the
// last one on top of kFlushPerWave entries, so that dense deltas rarely
// make a wave flush on its own.
__device__ int block_round(const ExtractParams& a, const WaveStage& st, Staging& so, int lane,
                           int wave, int (*s_cnt)[kWaves], unsigned long long* s_base, int slot,
                           int passes, bool last_round)
{
    const int64_t all = so.flushed + so.staged;
    if (lane == 0) s_cnt[slot][wave] = so.staged | ((int)(all - so.met) << 16);
    so.met = all;
    __syncthreads();
    int total = 0, before = 0, found = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = s_cnt[slot][w];
        const int staged = c & 0xFFFF;
        total += staged;
        found += c >> 16;
        before += w < wave ? staged : 0;
    }
    total = __builtin_amdgcn_readfirstlane(total);   // scalar: keeps the control flow uniform
    found = __builtin_amdgcn_readfirstlane(found);
    constexpr int kRoom = kWaves * (kWaveStage - kFlushPerWave);
    int next = kRound;
    while (next > 1 && next * found > kRoom * passes) next >>= 1;
    if (total == 0 || (!last_round && total < kWaves * kFlushPerWave)) return next;
    if (threadIdx.x == 0)
        s_base[slot] = atomicAdd(reinterpret_cast<unsigned long long*>(a.cursor),
                                 (unsigned long long)total) & kCountMask;
    __syncthreads();
    if (so.staged > 0) write_staged(a, st, so, (int64_t)s_base[slot] + before, lane);
    return next;
}

// Exact inverse of the first `count` queued candidates, 64 per pass; changed
// ones are staged.  The rest (fewer than 64) move to the queue's front.
template <bool kDecayOne, bool kLit, bool kRoute>
__device__ void drain_queue(const ExtractParams& a, const StepScalars& k, const WaveStage& st,
                            int& queued, int count, Staging& so, int lane)
{
    wave_sync();
    for (int base = 0; base < count; base += 64) {
        const int i = base + lane;
        bool changed = false;
        uint32_t key = 0;
        uint16_t bn = 0;
        if (i < count) {
            const f32x4 c = st.queue[i];
            const float ph = exact_prev<kDecayOne, kLit>(c.x, c.y, c.z, k);
            bn = (uint16_t)bf16_bits(c.x);
            changed = bf16_bits(ph) != bn;
            key = __float_as_uint(c.w);
        }
        stage_changed<kRoute>(a, st, so, lane, changed, key, bn);
    }
    queued -= count;
    if (queued > 0) {
        f32x4 c = {};
        if (lane < queued) c = st.queue[count + lane];
        wave_sync();
        if (lane < queued) st.queue[lane] = c;
    }
    wave_sync();
}

// What a wave loads in place of a slot beyond its last one.
__device__ const f32x4 g_pad = {};

// The float4 of each lane in the whole slot at element e0 of the range, or
// (one request for the wave) the pad: loads are issued on every path, so that
// the number of loads in flight behind a slot's own is known where the slot is
// tested.  Element alignment is enough for 16-byte global loads.
__device__ __forceinline__ void load_slot(const ExtractParams& a, bool valid, int64_t e0, int lane,
                                          f32x4& P, f32x4& M, f32x4& V)
{
    // addresses as integers, cast to the global address space: a choice of
    // two pointers would become flat loads, which wait for LDS as well
    const uint64_t pad = (uint64_t)&g_pad, at = (uint64_t)e0 * sizeof(float);
    const uint64_t p = valid ? (uint64_t)a.p + at : pad;
    const uint64_t m = valid ? (uint64_t)a.m + at : pad;
    const uint64_t v = valid ? (uint64_t)a.v + at : pad;
    const int off = lane * 4 & (valid ? -1 : 0);
    P = __builtin_nontemporal_load((global_f32x4)((global_f32)p + off));
    M = __builtin_nontemporal_load((global_f32x4)((global_f32)m + off));
    V = __builtin_nontemporal_load((global_f32x4)((global_f32)v + off));
}

// Stage the slot's selected elements that land in [from, to) of the staging
// area when counted from `first`, at their place - from.
__device__ __forceinline__ void stage_slot(const WaveStage& st, int first, int from, int to,
                                           const Slot4& r, const bool (&sel)[4], uint32_t key,
                                           const f32x4& P)
{
    int pos = first + lanes_before(r);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if (sel[c] && pos >= from && pos < to) {
            st.key[pos - from] = key + c;
            st.val[pos - from] = (uint16_t)bf16_bits(P[c]);
        }
        pos += sel[c] ? 1 : 0;
    }
}

// One slot, at element e0 of the range.  kPrev: the exact inverse of every
// element, theta_hat written and changed elements staged; else the elements
// without a proof join the queue, which is drained of whole groups of 64.
// kEdge: of the slot's elements only those in [lo, hi) count.
template <bool kEdge, bool kDecayOne, bool kPrev, bool kLit, bool kRoute>
__device__ __forceinline__ void test_slot(const ExtractParams& a, const StepScalars& k,
                                          const WaveStage& st, Staging& so, int& queued, int lane,
                                          int64_t e0, const f32x4& P, const f32x4& M,
                                          const f32x4& V, int64_t lo, int64_t hi)
{
    const int64_t e = e0 + lane * 4;
    const uint32_t key = (uint32_t)(e0 - st.base) + lane * 4;
    bool sel[4];
    f32x4 prev;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if (kPrev) {
            prev[c] = exact_prev<kDecayOne, kLit>(P[c], M[c], V[c], k);
            sel[c] = bf16_bits(prev[c]) != bf16_bits(P[c]);
        } else {
            sel[c] = (kLit && !k.lit_filter) ||
                     !proven_unchanged<kDecayOne, kLit>(P[c], M[c], V[c], k);
        }
        if (kEdge) sel[c] = sel[c] && e + c >= lo && e + c < hi;
    }
    const Slot4 r = select4(sel);
    if (kPrev) {
        if (r.count != 0) {
            const int first = so.staged, end = first + r.count;
            stage_slot(st, first, 0, kWaveStage, r, sel, key, P);
            so.staged = end;
            if (end >= kWaveStage) {   // flush exactly kWaveStage entries, then stage the rest
                so.staged = kWaveStage;
                flush_wave<kRoute>(a, st, so, lane);
                stage_slot(st, first, kWaveStage, end, r, sel, key, P);
                so.staged = end - kWaveStage;
            }
        }
        if (!kEdge) {
            __builtin_nontemporal_store(prev, reinterpret_cast<f32x4_any*>(a.out_prev + e));
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (e + c >= lo && e + c < hi) a.out_prev[e + c] = prev[c];
        }
    } else if (r.count != 0) {
        int pos = queued + lanes_before(r);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (sel[c]) st.queue[pos] = f32x4{P[c], M[c], V[c], __uint_as_float(key + c)};
            pos += sel[c] ? 1 : 0;
        }
        queued += r.count;
        if (queued >= kDrain)
            drain_queue<kDecayOne, kLit, kRoute>(a, k, st, queued, queued & ~63, so, lane);
    }
}

// The run of a wave's current slot: elements [.., end) of the range and their
// scalars (wave-uniform).  Lane k holds run k's end and scalars, so that a
// look-up costs a ballot and a few register reads, no memory latency.
struct CurrentRun {
    int64_t end;
    StepScalars step;
    int64_t lane_end;
    uint32_t lane_step[sizeof(StepScalars) / 4];
};

__device__ __forceinline__ void load_runs(const ExtractParams& a, CurrentRun& r, int lane)
{
    const int k = lane < a.nruns ? lane : a.nruns - 1;
    r.end = 0;
    r.lane_end = lane < a.nruns ? a.table.end[k] : INT64_MAX;
    const uint32_t* w = reinterpret_cast<const uint32_t*>(&a.table.step[k]);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(StepScalars) / 4); ++i) r.lane_step[i] = w[i];
}

// The run of element e < n.
__device__ __forceinline__ void find_run(CurrentRun& r, int64_t e)
{
    const int k = __popcll(__ballot(r.lane_end <= e));
    r.end = rt::readlane64(r.lane_end, k);
    uint32_t* w = reinterpret_cast<uint32_t*>(&r.step);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(StepScalars) / 4); ++i)
        w[i] = __builtin_amdgcn_readlane(r.lane_step[i], k);
}

// Slot [e0, end) that is not all of the current run's.  Before the run
// changes the queue is emptied, as its candidates are evaluated with one
// run's scalars; a wave's slots ascend, so runs are only ever left behind.
template <bool kPrev, bool kLit, bool kRoute>
__device__ __forceinline__ void test_slot_runs(const ExtractParams& a, CurrentRun& run,
                                               const WaveStage& st, Staging& so, int& queued,
                                               int lane, int64_t e0, int64_t end, const f32x4& P,
                                               const f32x4& M, const f32x4& V)
{
#pragma unroll 1
    for (int64_t lo = e0; lo < end;) {
        if (lo >= run.end) {
            if (queued > 0)
                drain_queue<false, kLit, kRoute>(a, run.step, st, queued, queued, so, lane);
            find_run(run, lo);
        }
        const int64_t hi = end < run.end ? end : run.end;
        test_slot<true, false, kPrev, kLit, kRoute>(a, run.step, st, so, queued, lane, e0, P, M, V,
                                                    lo, hi);
        lo = hi;
    }
}

// One launch covers the range.  kFull: n is a multiple of kSlot.  kOneGroup:
// one set of step scalars; else the runs of a.table.
//
// Bound by HBM (12 bytes read an element).  A wave streams its slots through
// a ring of kVec slots in registers: as soon as slot s is tested, the loads
// of slot s + kVec replace it, so loads stay in flight while the wave
// computes.  (Loading eight slots, waiting for all and then testing all left
// the memory idle while dense ranges computed, and tested the last slots of
// odd ranges in a second launch.)  386 M elements of Qwen3-8B layers, before
// -> now: lr 1e-6 697 -> 678 us, 1e-5 (2.3 % change) 805 -> 757, 1e-4 (13.8
// %) 968 -> 883, odd bases 2285 -> 720.  Draining the queue after every slot
// keeps room for any slot; the alternative, putting off and reloading slots
// that find no room, took 2120 us at lr 1e-3 against 1338.
template <bool kFull, bool kOneGroup, bool kDecayOne, bool kWritePrev, bool kLit, bool kRoute>
__global__ __launch_bounds__(64 * kWaves) void extract_kernel(ExtractParams a)
{
    __shared__ uint32_t s_key[kWaves][kWaveStage];
    __shared__ uint16_t s_val[kWaves][kWaveStage];
    __shared__ f32x4 s_queue[kWaves][kQueue];
    __shared__ int s_cnt[2][kWaves];
    __shared__ unsigned long long s_base[2];
    __shared__ unsigned long long s_chunk;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t g = (int64_t)blockIdx.x * kWaves + wave;
    const int64_t nw = (int64_t)gridDim.x * kWaves;
    // unordered output: combined flushes (block_round); every wave of the
    // block runs the same iterations, so the barriers match
    const bool combine = !kRoute && a.runs == nullptr;
    // wave g owns slots [g per, (g+1) per) of the static part [0, s_last);
    // the tail [s_last, slots) is dynamic
    const int64_t slots = (a.n + kSlot - 1) / kSlot, whole = a.n / kSlot;
    const int64_t tail = combine ? tail_slots(slots, nw) : 0;
    const int64_t s_last = slots - tail;
    const int64_t per = (s_last + nw - 1) / nw;
    Staging so{0, 0, 0, 0, 0};
    WaveStage st{s_key[wave], s_val[wave], s_queue[wave], g * per * kSlot, (int32_t)g};
    int queued = 0;
    CurrentRun run;
    if (!kOneGroup) load_runs(a, run, lane);
    const StepScalars& step = kOneGroup ? a.step : run.step;
    int round = 0;                               // block_round calls so far (LDS slot parity)
    int passes = kRound, togo = kRound;          // passes between meetings, until the next
    bool in_tail = false;
    int64_t first = g * per;
    int64_t last = first + per < s_last ? first + per : s_last;
    int64_t iters = (per + kVec - 1) / kVec;     // passes over the ring
    int64_t it = -1;                             // pass -1 only fills it
    f32x4 P[kVec], M[kVec], V[kVec];
    for (;;) {
        const int64_t s0 = first + it * kVec;
        const int64_t rest = (last < whole ? last : whole) - s0;
        const int left = (int)(rest < 2 * kVec ? rest : 2 * kVec);   // whole slots from s0
        // a pass whose slots are not all of one run is tested by a loop of
        // its own: copies of the test in the stream below made the code of a
        // pass longer and dense ranges 1 to 2 % slower
        const int here = it < 0 ? 0 : left < kVec ? left : kVec;
        const bool split = !kOneGroup && here > 0 && (s0 + here) * kSlot > run.end;
        if (split) {
#pragma unroll 1
            for (int j = 0; j < here; ++j) {
                const int64_t e0 = (s0 + j) * kSlot;
                f32x4 p = P[0], m = M[0], v = V[0];
#pragma unroll
                for (int i = 1; i < kVec; ++i) {
                    p = j == i ? P[i] : p;
                    m = j == i ? M[i] : m;
                    v = j == i ? V[i] : v;
                }
                test_slot_runs<kWritePrev, kLit, kRoute>(a, run, st, so, queued, lane, e0,
                                                         e0 + kSlot, p, m, v);
            }
        }
#pragma unroll
        for (int j = 0; j < kVec; ++j) {
            const int64_t e0 = (s0 + j) * kSlot;
            if (!split && j < here)
                test_slot<false, kDecayOne, kWritePrev, kLit, kRoute>(
                    a, step, st, so, queued, lane, e0, P[j], M[j], V[j], 0, 0);
            load_slot(a, j + kVec < left, e0 + kVec * kSlot, lane, P[j], M[j], V[j]);
        }
        ++it;
        if (it > 0 && --togo == 0) {
            togo = kRound;
            if (combine)
                togo = passes = block_round(a, st, so, lane, wave, s_cnt, s_base, (round++) & 1,
                                            passes, false);
            else if (!kRoute)
                __syncthreads();   // ordered: keeps the block's waves in step
        }
        if (it < iters) continue;
        if (!kFull && first <= whole && whole < last) {      // the range's partial slot
            f32x4 p = {}, m = {}, v = {};
            const int64_t e = whole * kSlot + lane * 4;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (e + c < a.n) {
                    p[c] = a.p[e + c];
                    m[c] = a.m[e + c];
                    v[c] = a.v[e + c];
                }
            }
            if (kOneGroup)
                test_slot<true, kDecayOne, kWritePrev, kLit, kRoute>(
                    a, step, st, so, queued, lane, whole * kSlot, p, m, v, INT64_MIN, a.n);
            else
                test_slot_runs<kWritePrev, kLit, kRoute>(a, run, st, so, queued, lane,
                                                         whole * kSlot, a.n, p, m, v);
        }
        if (tail == 0) break;
        if (!in_tail) {
            // staged keys count from the stage's base: empty the queue and
            // the staging areas, then count from the tail's start
            if (queued > 0) drain_queue<kDecayOne, kLit, kRoute>(a, step, st, queued, queued, so, lane);
            togo = passes = block_round(a, st, so, lane, wave, s_cnt, s_base, (round++) & 1,
                                        passes, true);
            st.base = s_last * kSlot;
            in_tail = true;
        }
        const int64_t wave_chunk = chunk_slots(tail, nw), block_chunk = kWaves * wave_chunk;
        if (threadIdx.x == 0)
            s_chunk = atomicAdd(reinterpret_cast<unsigned long long*>(a.cursor),
                                1ull << kGrabShift) >> kGrabShift;
        __syncthreads();
        const int64_t chunk = rt::readlane64((int64_t)s_chunk, 0);   // block-uniform
        __syncthreads();                                     // s_chunk is rewritten next
        if (chunk * block_chunk >= tail) {
            // chunks and one empty grab per block: the last of them clears
            // the grab count
            const int64_t grabs = (tail + block_chunk - 1) / block_chunk + gridDim.x;
            if (threadIdx.x == 0 && chunk == grabs - 1)
                atomicAdd(reinterpret_cast<unsigned long long*>(a.cursor),
                          0ull - ((unsigned long long)grabs << kGrabShift));
            break;
        }
        first = s_last + chunk * block_chunk + wave * wave_chunk;
        last = first + wave_chunk < slots ? first + wave_chunk : slots;
        iters = wave_chunk / kVec;
        it = -1;
    }
    if (queued > 0) drain_queue<kDecayOne, kLit, kRoute>(a, step, st, queued, queued, so, lane);
    if (combine)
        block_round(a, st, so, lane, wave, s_cnt, s_base, (round++) & 1, passes, true);
    else if (so.staged > 0)
        flush_wave<kRoute>(a, st, so, lane);
    if (kRoute) {   // one addition of the entry count per block, not one per flush
        if (lane == 0) s_cnt[0][wave] = (int)so.flushed;
        __syncthreads();
        if (wave == 0) {
            unsigned long long n = lane < kWaves ? (unsigned)s_cnt[0][lane] : 0u;
            for (int d = 8; d > 0; d >>= 1) n += __shfl_down(n, d);
            if (lane == 0 && n > 0)
                atomicAdd(reinterpret_cast<unsigned long long*>(a.cursor), n);
        }
    }
    if (a.runs && lane == 0) {
        a.wave_count[st.wave] = so.flushed;
        a.region_count[st.wave] = so.in_region;
    }
}

// One AdamW step.  Bound by HBM (16 bytes read, 12 written an element).  A
// float4 of each array per lane, whatever the alignment, and as many blocks
// as that takes: blocks that come and go keep reads and writes mixed, where a
// persistent grid of 8 blocks per CU took 1231 us on 193 M elements against
// 986 us, 891 us with loads and stores past the caches (kStream); 2 or 4
// float4 per lane 951 / 932 us, contiguous ranges per block 1041-1095 us.
template <bool kStream>
__global__ __launch_bounds__(kForwardBlock) void adamw_forward_kernel(ForwardParams a)
{
    const auto load = [&](const float* x, int64_t e) {
        f32x4 r = {};
        if (e + 3 < a.n) {
            const global_f32x4 q = (global_f32x4)(x + e);
            r = kStream ? __builtin_nontemporal_load(q) : *q;
        } else {
#pragma unroll
            for (int c = 0; c < 3; ++c)
                if (e + c < a.n) r[c] = x[e + c];
        }
        return r;
    };
    const auto store = [&](float* x, int64_t e, const f32x4& y) {
        if (e + 3 < a.n) {
            if (kStream)
                __builtin_nontemporal_store(y, reinterpret_cast<f32x4_any*>(x + e));
            else
                *reinterpret_cast<f32x4_any*>(x + e) = y;
        } else {
#pragma unroll
            for (int c = 0; c < 3; ++c)
                if (e + c < a.n) x[e + c] = y[c];
        }
    };
    const int64_t stride = (int64_t)gridDim.x * kForwardBlock * 4;
    for (int64_t e = ((int64_t)blockIdx.x * kForwardBlock + threadIdx.x) * 4; e < a.n;
         e += stride) {
        f32x4 P = load(a.p, e), M = load(a.m, e), V = load(a.v, e);
        const f32x4 G = load(a.g, e);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float g = G[c];
            const float m1 = a.b1 * M[c];
            const float m2 = a.omb1 * g;
            const float mt = m1 + m2;
            const float g2 = g * g;
            const float v1 = a.b2 * V[c];
            const float v2 = a.omb2 * g2;
            const float vt = v1 + v2;
            const float u = a.literal ? step_term_literal(mt, vt, a.lr, a.bc1, a.bc2, a.eps)
                                      : step_term(mt, vt, a.lrb1, a.rbc2, a.eps);
            const float dp = a.decay * P[c];
            P[c] = dp - u;
            M[c] = mt;
            V[c] = vt;
        }
        store(a.p, e, P);
        store(a.m, e, M);
        store(a.v, e, V);
    }
}

template <bool F, bool D, bool L, bool R>
void launch_kernel(const ExtractParams& a, dim3 grid, hipStream_t s)
{
    const dim3 block(64 * kWaves);
    if (R)   // routing mode: no theta_hat output
        hipLaunchKernelGGL((extract_kernel<F, true, D, false, L, R>), grid, block, 0, s, a);
    else if (a.out_prev)
        hipLaunchKernelGGL((extract_kernel<F, true, D, true, L, false>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((extract_kernel<F, true, D, false, L, false>), grid, block, 0, s, a);
}

// Blocks of one call: as many as get kMinSlots slots per wave, rounded up
// (the last block may get fewer), one per CU at most.
int64_t blocks_of(int64_t n, int cus)
{
    const int64_t slots = (n + kSlot - 1) / kSlot;
    const int64_t b = (slots + kWaves * kMinSlots - 1) / (kWaves * kMinSlots);
    const int64_t cap = cus < kMaxWaves / kWaves ? cus : kMaxWaves / kWaves;
    return b < cap ? b : cap;
}

template <bool L, bool R>
void launch_runs(const ExtractParams& a, int cus, hipStream_t s)
{
    const dim3 grid((unsigned)blocks_of(a.n, cus)), block(64 * kWaves);
    if (!R && a.out_prev)
        hipLaunchKernelGGL((extract_kernel<false, false, false, true, L, false>), grid, block, 0, s,
                           a);
    else
        hipLaunchKernelGGL((extract_kernel<false, false, false, false, L, R>), grid, block, 0, s,
                           a);
}

template <bool D, bool L, bool R>
void launch_range(const ExtractParams& a, int cus, hipStream_t s)
{
    const dim3 grid((unsigned)blocks_of(a.n, cus));
    if (a.n % kSlot == 0) {
        launch_kernel<true, D, L, R>(a, grid, s);
    } else if constexpr (R && !D) {   // the kernel over runs does the same work for one run
        ExtractParams one = a;
        one.table.end[0] = a.n;
        one.table.step[0] = a.step;
        launch_runs<L, true>(one, cus, s);
    } else {
        launch_kernel<false, D, L, R>(a, grid, s);
    }
}

// ---- ordered mode: runs to ascending positions ----------------------------

// One block: wave_base = *cursor + exclusive prefix of the wave totals; then
// the cursor advances by their sum, the true total of the call.
__global__ __launch_bounds__(1024) void order_scan_kernel(OrderParams o)
{
    constexpr int kThreads = 1024;
    constexpr int kPer = kMaxOrderedWaves / kThreads;
    __shared__ int64_t part[kThreads];
    const int tid = threadIdx.x;
    const int lo = tid * kPer;
    int64_t sum = 0;
    for (int i = 0; i < kPer; ++i)
        if (lo + i < o.waves) sum += o.wave_count[lo + i];
    part[tid] = sum;
    __syncthreads();
    for (int d = 1; d < kThreads; d <<= 1) {      // inclusive scan of the partial sums
        const int64_t x = (tid >= d) ? part[tid - d] : 0;
        __syncthreads();
        part[tid] += x;
        __syncthreads();
    }
    const int64_t c0 = *o.cursor;
    int64_t run = c0 + part[tid] - sum;
    for (int i = 0; i < kPer; ++i) {
        if (lo + i < o.waves) {
            o.wave_base[lo + i] = run;
            run += o.wave_count[lo + i];
        }
    }
    __syncthreads();                              // every thread has read the cursor
    if (tid == 0) *o.cursor = c0 + part[kThreads - 1];
}

constexpr int kCopyBlock = 256;
constexpr int kCopySlots = 8;                  // entries per lane per copy chunk
constexpr int kCopyChunk = 64 * kCopySlots;

// Regions: the waves take chunks of kCopyChunk entries (chunk c of extract
// wave g's region: its entries c kCopyChunk + i, which move to wave_base[g]
// + c kCopyChunk + i), all loads of a chunk before its stores.  Then whole
// recorded runs: entry i of a run moves from src + i to wave_base[wave] +
// woff + i.
__global__ __launch_bounds__(kCopyBlock) void order_copy_kernel(OrderParams o)
{
    const int lane = threadIdx.x & 63;
    const int64_t w = (int64_t)blockIdx.x * (kCopyBlock / 64) + (threadIdx.x >> 6);
    const int64_t nw = (int64_t)gridDim.x * (kCopyBlock / 64);
    const int64_t per_region = (o.region_size + kCopyChunk - 1) / kCopyChunk;
    const int64_t chunks = (int64_t)o.waves * per_region;
    const int64_t* __restrict__ ridx = o.region_idx;
    const uint16_t* __restrict__ rval = o.region_val;
    for (int64_t k = w; k < chunks; k += nw) {
        const int64_t g = k / per_region;
        const int64_t c0 = (k - g * per_region) * kCopyChunk;
        const int64_t cnt = o.region_count[g];
        if (c0 >= cnt) continue;
        const int64_t src0 = g * o.region_size + c0;
        const int64_t dst0 = o.wave_base[g] + c0;
        int64_t x[kCopySlots];
        uint16_t y[kCopySlots];
#pragma unroll
        for (int j = 0; j < kCopySlots; ++j) {
            const int64_t i = j * 64 + lane;
            x[j] = c0 + i < cnt ? ridx[src0 + i] : 0;
            y[j] = c0 + i < cnt ? rval[src0 + i] : (uint16_t)0;
        }
#pragma unroll
        for (int j = 0; j < kCopySlots; ++j) {
            const int64_t i = j * 64 + lane;
            if (c0 + i < cnt && dst0 + i < o.capacity) {
                o.out_idx[dst0 + i] = x[j];
                o.out_val[dst0 + i] = y[j];
            }
        }
    }
    int64_t nruns = *o.run_cursor;
    if (nruns > o.max_runs) nruns = o.max_runs;
    for (int64_t r = w; r < nruns; r += nw) {
        const OrderRun run = o.runs[r];
        const int64_t dst0 = o.wave_base[run.wave] + run.woff;
        for (int i = lane; i < run.count; i += 64) {
            const int64_t src = run.src + i;
            const int64_t dst = dst0 + i;
            if (src < o.src_capacity && dst < o.capacity) {
                o.out_idx[dst] = o.src_idx[src];
                o.out_val[dst] = o.src_val[src];
            }
        }
    }
}

}  // namespace

hipError_t launch_order(const OrderParams& o, int cus, hipStream_t stream)
{
    if (o.waves <= 0) return hipSuccess;
    hipLaunchKernelGGL(order_scan_kernel, dim3(1), dim3(1024), 0, stream, o);
    hipLaunchKernelGGL(order_copy_kernel, dim3((unsigned)cus * 8), dim3(kCopyBlock), 0, stream, o);
    return hipGetLastError();
}

int64_t extract_waves(int64_t n, int cus) { return n > 0 ? blocks_of(n, cus) * kWaves : 0; }

hipError_t launch_extract(const ExtractParams& a, int cus, hipStream_t stream)
{
    if (a.n <= 0) return hipSuccess;
    const bool one = a.step.decay == 1.0f;
    if (a.nruns > 1) {
        if (a.route)
            a.literal ? launch_runs<true, true>(a, cus, stream)
                      : launch_runs<false, true>(a, cus, stream);
        else
            a.literal ? launch_runs<true, false>(a, cus, stream)
                      : launch_runs<false, false>(a, cus, stream);
    } else if (a.route) {
        if (a.literal)
            one ? launch_range<true, true, true>(a, cus, stream)
                : launch_range<false, true, true>(a, cus, stream);
        else
            one ? launch_range<true, false, true>(a, cus, stream)
                : launch_range<false, false, true>(a, cus, stream);
    } else if (a.literal) {
        one ? launch_range<true, true, false>(a, cus, stream)
            : launch_range<false, true, false>(a, cus, stream);
    } else {
        one ? launch_range<true, false, false>(a, cus, stream)
            : launch_range<false, false, false>(a, cus, stream);
    }
    return hipGetLastError();
}

hipError_t launch_adamw_forward(const ForwardParams& a, hipStream_t stream)
{
    if (a.n <= 0) return hipSuccess;
    const int64_t quads = (a.n + 3) / 4;
    const int64_t blocks = (quads + kForwardBlock - 1) / kForwardBlock;
    const dim3 grid((unsigned)(blocks < kForwardBlocks ? blocks : kForwardBlocks));
    if (a.n > kForwardStream)
        hipLaunchKernelGGL(adamw_forward_kernel<true>, grid, dim3(kForwardBlock), 0, stream, a);
    else
        hipLaunchKernelGGL(adamw_forward_kernel<false>, grid, dim3(kForwardBlock), 0, stream, a);
    return hipGetLastError();
}

}  // namespace dte
