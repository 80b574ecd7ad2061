// gfx950 kernels of the eager-SGD round: partial-allreduce arithmetic with stale-gradient
// carry (paper Section 5, walk-through of Fig. 7), the 1/P average (Algorithm 2 line 6)
// and the momentum-SGD update rule (lines 7-8) in ONE pass over HBM.
//
// The path is a pure stream: per element <= 2P adds, one multiply and two FMAs against
// >= 4P bytes, so HBM bandwidth is the only roofline that matters and there is no
// contraction for the matrix cores.  Design for CDNA4:
//   * the host compacts the round into a list of streams ("slots") that must be read, in
//     summation order, each with one action; a wavefront takes one tile of 256 elements, a lane
//     4 consecutive elements of every stream, so a 64-lane wavefront reads or writes one
//     contiguous KiB per fp32 stream and instruction;
//   * burst_kernel, for runs that stream from HBM: many wavefronts per CU, two loads in flight
//     in each; occupancy is capped so that the bytes in flight match what the memory side holds;
//   * short_kernel (eager_short.h), for runs that latency bounds and lists of up to 16 streams: the whole list and its
//     arguments in flight at once, no cap; chunk_kernel (eager_chunk.h) for longer lists there, beside by-products and
//     for launch options: up to 16 or 32 loads in flight per lane;
//   * which streams exist and what is done with each is decided on the host: empty send buffers
//     cost no bytes, the send buffer of an on-time process is "cleared" by a flag on the host,
//     not by writing zeros; burst_kernel applies the actions with scalar bit masks, the other two
//     with a branch per slot;
//   * the accumulator stays in fp32 registers; in fixed-order mode contributions are added
//     in ascending rank order from +0.0f with contraction off, so the result is defined
//     bit for bit; fast mode keeps two partial sums that take the streams in turn (in small runs two of
//     fp32 streams and two of bf16 streams);
//   * carry_kernel: the send-buffer rewrite of late processes as a plain pair-by-pair
//     copy, when a round is split;
//   * optional per-bucket norms as by-products of the same pass: DPP sums inside wavefronts,
//     one record per tile (the helpers live in eager_device.h, the kernels that finish
//     them in eager_aux_kernels.hip).
#include "eager_device.h"
#include "eager_rules.h"

#include <algorithm>

namespace eager {
namespace {

// A wavefront owns one tile of 64 lane-vectors (a lane-vector = 4 elements), so that each load or
// store instruction covers one contiguous kilobyte of an fp32 stream.  With bf16 gradients (BF16)
// a lane's 4 gradient elements are 8 bytes, one half of an aligned 16-byte piece: lanes 2k and
// 2k+1 load the same piece and each keeps its half.  That way every load is the same 16-byte
// instruction whatever the type of its stream - the type, like the action, is a scalar select and
// never a branch around a load.
//
// Addresses are a uniform base (stream + first element of the tile that belongs to the run) plus a 32-bit
// offset of the lane.  Lanes beyond the last lane-vector or before the first repeat it: their loads stay inside the run
// and their results are never stored (see place_lane).
struct Lanes {
    long long e0;          // first element of the run in the tile (arena index), uniform
    unsigned off;          // byte offset of the lane-vector in an fp32 stream
    unsigned off_bf;       // byte offset of the 16-byte piece of a bf16 stream that holds it
    bool odd;              // the lane-vector is the upper half of that piece
    bool in;               // the lane-vector belongs to the run
    bool held;             // it does, or stands in front of it
};

// 16 bytes of a slot's stream (raw: a bf16 stream is widened by slot_value).  For a SKIP every
// lane loads one and the same piece: hardly any traffic.
template <bool BF16>
__device__ __forceinline__ f32x4 ld_slot_or_skip(unsigned long long slot, const Lanes &L)
{
    const bool skip = (slot & (kKindMask | kSlotCopy)) == kSkip;
    const bool is_bf = BF16 && (slot & kSlotBf16);
    const char *base = reinterpret_cast<const char *>(slot & ~static_cast<unsigned long long>(kSlotTag)) +
                       L.e0 * (is_bf ? 2 : 4);
    const unsigned off = L.off, off_bf = L.off_bf;
    return ld_at<true>(base, (is_bf ? off_bf : off) & (skip ? 0u : ~0u));
}

template <bool BF16>
__device__ __forceinline__ f32x4 slot_value(f32x4 plain, bool is_bf, bool odd)
{
    if (!BF16) return plain;
    const u32x4 raw = __builtin_bit_cast(u32x4, plain);
    const unsigned a = odd ? raw.z : raw.x, b = odd ? raw.w : raw.y;
    f32x4 wide;
    wide.x = __uint_as_float(a << 16);
    wide.y = __uint_as_float(a & 0xffff0000u);
    wide.z = __uint_as_float(b << 16);
    wide.w = __uint_as_float(b & 0xffff0000u);
    return is_bf ? wide : plain;
}

__device__ __forceinline__ f32x4 masked(f32x4 x, unsigned m)
{
    return __builtin_bit_cast(f32x4, __builtin_bit_cast(u32x4, x) & m);
}

// The partial sums of a wavefront.  term: what the slot before would add (a HOLD is always
// directly followed by its PAIR).
struct Sums {
    f32x4 s, s2, term;     // s2: the second partial sum of fast mode
};

// Add one slot's values.  The action is applied with bit masks built from scalar conditions,
// never with a branch: if a path existed on which a load is not consumed, the compiler would
// have to drain all memory operations before its registers could be reused.
//   fixed order:  term = x + (term & pair) ;  s = s + (term & adds)
// pair = all ones for a PAIR slot, adds = all ones for ADD and PAIR.  A masked-out term is +0.0f,
// and adding +0.0f changes nothing here: s starts at +0.0f and a sum of two floats is -0.0f only
// if both are, so s is never -0.0f; and x + 0.0f differs from x only for x = -0.0f, which adds
// the same as +0.0f to an s that is not -0.0f, directly or as a part of a pair.
template <bool BF16, bool FAST>
__device__ __forceinline__ void add_slot(unsigned long long slot, f32x4 raw, const Lanes &L, Sums &S,
                                         bool second)
{
    const unsigned tag = static_cast<unsigned>(slot);
    const unsigned lo = tag & 1u, hi = (tag >> 1) & 1u;
    const f32x4 x = slot_value<BF16>(raw, BF16 && (tag & kSlotBf16), L.odd);
    if (FAST) {
        // any order: two interleaved partial sums; everything but SKIP
        f32x4 &s = second ? S.s2 : S.s;
        s = s + masked(x, ~(0u - (lo & hi)));
    } else {
        S.term = x + masked(S.term, 0u - (hi & ~lo & 1u));       // PAIR
        S.s = S.s + masked(S.term, 0u - (~lo & 1u));             // ADD or PAIR
    }
}

// What follows the sum: average, receive buffer, by-products, update rule.
// NTS: parameters, momentum and the receive buffer are streamed with the nontemporal hint
// too (right when they are too large to stay in the last-level cache until the next round).
template <bool FAST, bool NTS, bool OPT, bool STATS>
__device__ __forceinline__ void finish_tile(const SlotHead &h, const Lanes &L, const Sums &S, f32x4 vo,
                                            f32x4 wo, int n_valid, LaneStats &ls)
{
    const long long base = L.e0 * 4;
    f32x4 sum = S.s;
    if (FAST) sum = sum + S.s2;
    const f32x4 avg = sum * h.inv_P;
    if (STATS) {
        stats_vector<OPT>(ls, avg, wo, n_valid);
    }
    f32x4 vn, wn;
    if (OPT) {
        const UpdateRule rule = {h.neg_lr, h.mu, h.wd, h.nesterov};
        update_rule<FAST>(rule, avg, vo, wo, vn, wn);
    }
    if (L.in) {
        if (h.recv) st_at<NTS>(reinterpret_cast<char *>(h.recv) + base, L.off, avg);
        if (OPT) {
            st_at<NTS>(reinterpret_cast<char *>(h.v) + base, L.off, vn);
            st_at<NTS>(reinterpret_cast<char *>(h.w) + base, L.off, wn);
        }
    }
}

// one element of a slot's stream
template <bool BF16>
__device__ __forceinline__ float ld_slot_element(unsigned long long slot, long long i)
{
    typedef const float __attribute__((address_space(1))) GF;
    typedef const unsigned short __attribute__((address_space(1))) GH;
    const unsigned long long base = slot & ~static_cast<unsigned long long>(kSlotTag);
    if (BF16 && (slot & kSlotBf16))
        return __uint_as_float(static_cast<unsigned>(((GH *)base)[i]) << 16);
    return ((GF *)base)[i];
}

// Ragged tail: at most 3 (7 with bf16 gradients) elements per launch, one lane each, by a
// wavefront that has nothing else to do; fixed order in both modes.  The loads of 8 slots are
// issued together: one at a time, a round of 16 streams waited 16 times for memory.
template <bool BF16, bool STATS>
__device__ __forceinline__ void slot_tail_element(KSlotArgs &a, const SlotHead &h, long long i)
{
    float s = 0.0f, term = 0.0f;
    constexpr int C = kSlotFill;          // what is read beyond the list are SKIPs
    for (int k0 = 0; k0 < h.n_sum; k0 += C) {
        float x[C];
#pragma unroll
        for (int j = 0; j < C; ++j) x[j] = ld_slot_element<BF16>(a.slot[k0 + j], i);
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const int kind = static_cast<int>(a.slot[k0 + j] & kKindMask);
            term = kind == kPair ? term + x[j] : x[j];
            s = kind == kAdd || kind == kPair ? s + term : s;
        }
    }
    for (int c0 = 0; c0 < h.n_copy; c0 += C) {
        float x[C];
#pragma unroll
        for (int j = 0; j < C; ++j) x[j] = ld_slot_element<BF16>(a.slot[h.n_sum + c0 + j], i);
#pragma unroll
        for (int j = 0; j < C; ++j)
            if (c0 + j < h.n_copy) a.dst[h.n_sum + c0 + j][i] = x[j];
    }
    const float avg = s * h.inv_P;
    if (h.recv) h.recv[i] = avg;
    if (STATS) {
        // a handful of single elements per launch: one record each, in the block after the
        // last bucket's
        const long long *tbl = a.stats.table;
        LaneStats ls = {0.0, 0.0, 0u, find_bucket(tbl, a.stats.n_buckets, i)};
        if (i < tbl[2 * ls.bucket + 1]) stats_add(ls, avg, h.w ? h.w[i] : 0.0f, h.w != nullptr);
        else ls.bucket = -2;                                   // padding
        const StatsRecord mine = {ls.ssu, ls.ssw, ls.bucket, ls.nf, 0};
        a.stats.lane_records[static_cast<long long>(a.stats.n_buckets) * 64 + (threadIdx.x & 63u)] = mine;
    }
    if (h.w) {
        const UpdateRule rule = {h.neg_lr, h.mu, h.wd, h.nesterov};
        float v = h.v[i], w = h.w[i];
        update_rule_scalar(rule, avg, v, w);
        h.v[i] = v;
        h.w[i] = w;
    }
}

// The head of the arguments, all of it requested at once and waited for here: read where it is
// used, one field after the other, a wavefront starts with four or five trips to the argument
// segment in a row.
__device__ __forceinline__ SlotHead read_head(KSlotArgs &a)
{
    SlotHead h;
    __builtin_memcpy(&h, (const void __attribute__((address_space(4))) *)&a.h, sizeof h);
    asm volatile("" : "+s"(h.e0), "+s"(h.n), "+s"(h.n_sum), "+s"(h.n_copy), "+s"(h.waves_per_block),
                 "+s"(h.xcd_blocks), "+s"(h.w), "+s"(h.v), "+s"(h.recv), "+s"(h.inv_P), "+s"(h.neg_lr),
                 "+s"(h.mu), "+s"(h.wd), "+s"(h.nesterov), "+s"(h.skip));
    return h;
}

// Index of the wavefront in the grid.  Workgroups are dealt to the 8 XCDs round robin; xcd_blocks
// gives every XCD one contiguous eighth of the run instead of every eighth tile (a launch
// option, for A/B).  (The grid's shape comes with the arguments: the built-in blockDim is a load
// from memory that every wavefront would have to wait for.)
__device__ __forceinline__ unsigned wave_index(const SlotHead &h)
{
    unsigned bid = blockIdx.x;
    const unsigned per = static_cast<unsigned>(h.xcd_blocks);
    if (per && bid < per * 8u) bid = (bid % 8u) * per + bid / 8u;
    const unsigned wave = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)));
    return bid * static_cast<unsigned>(h.waves_per_block) + wave;
}

__device__ __forceinline__ Lanes place_lanes(const SlotHead &h, unsigned tile, unsigned nvec)
{
    const LanePlace p = place_lane(threadIdx.x & 63u, tile, nvec - tile * 64u, static_cast<unsigned>(h.skip));
    Lanes L;
    L.e0 = h.e0 + p.first * 4ll;
    L.held = p.held;
    L.in = p.in;
    L.off = p.at * 16u;
    L.off_bf = (p.at >> 1) * 16u;
    L.odd = (p.at & 1u) != 0;
    return L;
}

// By-products: bucket of the lane-vector and how many of its elements lie inside.
__device__ __forceinline__ int place_stats(KSlotArgs &a, const Lanes &L, LaneStats &ls)
{
    const long long e = L.e0 + (L.off >> 2);
    long long end;
    const int b = tile_bucket(a.stats.table, a.stats.b_lo, a.stats.b_hi, L.e0, e, end);
    ls = {0.0, 0.0, 0u, L.held ? b : -1};       // (in front of the run: the bucket of its first element)
    return L.in ? inside(e, end) : 0;
}

// The round as a stream of bursts: a wavefront (one tile) requests kBurst = 2 slots, waits for both,
// adds them, and goes on to the next two; w and v come last.  What bounds it is the memory
// side, and the memory side wants FEW bytes in flight: about 26 KiB per CU is the product of its
// latency and its rate, more only queues up and loses row locality.  Many wavefronts with little
// in flight each do that best: with 16 streams of 268 MB, w and v updated, 2 loads by 12 wavefronts
// move 6.4-6.6 TB/s where 16 loads by 8 wavefronts move 6.0-6.2 (32 streams: 6.2-6.3 and 5.7-5.9;
// both depend on where the arenas lie).  Two or four tiles per wavefront reach 6.7 with some
// placements and 5.2 with others, a rolling window of 2-4 loads is 2 % slower than bursts.
// Copies (late gradients of a fused round) follow the sum in the same way.  Whole rounds, before
// (16 loads at once) and now: 16 processes, 67 M elements, everybody on time 882 -> 841 us; 2
// processes, 20 M: 84.5 -> 78.5; 16 processes, 1 M, 15 late: 38.9 -> 34.8.
template <bool BF16, bool FAST, bool NTS, bool OPT, bool STATS>
__global__ __launch_bounds__(256) void burst_kernel(const SlotArgs)
{
    constexpr int D = kBurst;
    KSlotArgs &a = kernarg<SlotArgs>();
    const SlotHead h = read_head(a);
    constexpr unsigned kRagged = BF16 ? 7u : 3u;          // (slot_nvec in 32 bits, see place_lane)
    const unsigned nvec = static_cast<unsigned>((static_cast<unsigned long long>(h.n) & ~static_cast<unsigned long long>(kRagged)) >> 2);
    const unsigned tile = wave_index(h);
    if (tile * 64u >= nvec) {
        // the grid's last wavefront: the ragged tail
        const unsigned t = threadIdx.x & 63u;
        if (tile * 64u < nvec + 64u && t < (static_cast<unsigned>(h.n) & kRagged))
            slot_tail_element<BF16, STATS>(a, h, h.e0 + nvec * 4ll + t);
        return;
    }
    const Lanes L = place_lanes(h, tile, nvec);
    Sums S;
    S.s = S.s2 = S.term = (f32x4)(0.0f);
    const int n_sum = h.n_sum, n = n_sum + h.n_copy;
    unsigned long long slot[D];
    f32x4 x[D];
    auto request = [&](int k) {
#pragma unroll
        for (int j = 0; j < D; ++j) slot[j] = a.slot[k + j];
#pragma unroll
        for (int j = 0; j < D; ++j) x[j] = ld_slot_or_skip<BF16>(slot[j], L);
    };
    // Everything in flight has arrived before it is used and before the next burst is requested:
    // the empty statements hold the compiler to that order.
    auto arrived = [&]() {
#pragma unroll
        for (int j = 0; j < D; ++j) asm volatile("" : "+v"(x[j]) : : "memory");
    };
    LaneStats ls;
    int n_valid = 0;
    if (n_sum > 0) {
        request(0);
        if (STATS) n_valid = place_stats(a, L, ls);
        for (int k = D;; k += D) {
            arrived();
#pragma unroll
            for (int j = 0; j < D; ++j) add_slot<BF16, FAST>(slot[j], x[j], L, S, j & 1);
            asm volatile("" : "+v"(S.s), "+v"(S.s2), "+v"(S.term) : : "memory");
            if (k >= n_sum) break;
            request(k);
        }
    } else if (STATS) {
        n_valid = place_stats(a, L, ls);
    }
    f32x4 vo = (f32x4)(0.0f), wo = vo;
    if (OPT) {
        vo = ld_at<NTS>(reinterpret_cast<const char *>(h.v) + L.e0 * 4, L.off);
        wo = ld_at<NTS>(reinterpret_cast<const char *>(h.w) + L.e0 * 4, L.off);
    }
    finish_tile<FAST, NTS, OPT, STATS>(h, L, S, vo, wo, n_valid, ls);
    for (int k = n_sum; k < n; k += D) {
        request(k);
        arrived();
#pragma unroll
        for (int j = 0; j < D; ++j)
            if (k + j < n) {
                char *dst = reinterpret_cast<char *>(a.dst[k + j]) + L.e0 * 4;
                if (L.in) st_at<true>(dst, L.off, slot_value<BF16>(x[j], BF16, L.odd));
            }
    }
    if (STATS) stats_commit(a.stats.records, a.stats.lane_records, ls, tile);
}

// R_p <- G_p for the late processes, as a plain copy: pair after pair (blockIdx.y is the
// pair, and workgroups are dealt out x first), so that at any time the device streams one
// source and one destination.  A copy of few streams runs near the read-only rate on MI355X,
// whereas the same bytes written as 8-31 interleaved streams next to the reduction's reads
// cost 10-15 %.  A lane owns 4 elements: every store instruction of a wavefront writes one
// contiguous kilobyte (a bf16 source is read 8 bytes per lane and widened).  No loop and no
// division: a wavefront lives for one load and one store, so whatever stands before its load
// counts (bf16 source, 1.1e9 elements per pair: 6.73 TB/s in this form, 6.62 with the pair
// taken from blockIdx.x by a division, 6.46 with a striding loop around the body).
// BACK: the first tile begins in front of the run (a.skip).
template <bool BF16, int V, bool BACK>
__global__ __launch_bounds__(256) void carry_kernel(const CarryArgs a)
{
    const unsigned pair = blockIdx.y;
    const long long nvec = a.n / 4;
    const char *src = static_cast<const char *>(a.src[pair]);
    float *dst = a.dst[pair];
    // a workgroup copies V * blockDim consecutive lane-vectors: all loads first, then the stores
    const long long base = static_cast<long long>(blockIdx.x) * blockDim.x * V + threadIdx.x;
    f32x4 x[V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const long long vi = base + static_cast<long long>(k) * blockDim.x;
        if ((!BACK || vi >= a.skip) && vi < nvec) {
            const long long e = a.e0 + vi * 4;
            if (BF16) {
                const u32x2 g = __builtin_nontemporal_load(
                    reinterpret_cast<const u32x2 *>(src + e * 2));
                x[k].x = __uint_as_float(g.x << 16);
                x[k].y = __uint_as_float(g.x & 0xffff0000u);
                x[k].z = __uint_as_float(g.y << 16);
                x[k].w = __uint_as_float(g.y & 0xffff0000u);
            } else {
                x[k] = ld_f4<true>(reinterpret_cast<const float *>(src + e * 4));
            }
        }
    }
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const long long vi = base + static_cast<long long>(k) * blockDim.x;
        if ((!BACK || vi >= a.skip) && vi < nvec) st_f4<true>(dst + a.e0 + vi * 4, x[k]);
    }
    const long long rem = a.n - nvec * 4;
    if (blockIdx.x == 0 && static_cast<long long>(threadIdx.x) < rem) {
        const long long i = a.e0 + nvec * 4 + threadIdx.x;
        dst[i] = load_grad_scalar<BF16>(src, i);
    }
}

// ---- the stream list of a round from the rank masks
void build_slots(const RoundArgs &a, SlotArgs &s)
{
    const bool bf16 = a.elem_bytes == 2;
    int n = 0;
    auto push = [&](const void *src, unsigned kind, bool is_bf) {
        s.slot[n++] = reinterpret_cast<unsigned long long>(src) | kind |
                      (is_bf ? kSlotBf16 : 0u);
    };
    for (int p = 0; p < a.P; ++p) {
        const bool on_time = (a.active >> p) & 1ull, has_stale = (a.valid >> p) & 1ull;
        if (has_stale) push(a.r[p], on_time ? kHold : kAdd, false);
        if (on_time) push(a.g[p], has_stale ? kPair : kAdd, bf16);
    }
    // A SKIP is the last stream again (or, where there is none, any readable memory of the run):
    // loaded where slots are taken several at a time, and not added.
    const void *any = a.w ? a.w : a.recv;
    const unsigned long long none = (n > 0 ? s.slot[n - 1] & ~static_cast<unsigned long long>(kKindMask)
                                           : reinterpret_cast<unsigned long long>(any)) | kSkip;
    while (n % kBurst) s.slot[n++] = none;
    s.h.n_sum = n;
    s.h.n_copy = 0;
    for (int p = 0; p < a.P; ++p)
        if ((a.store >> p) & 1ull) {
            s.dst[n] = a.r[p];
            push(a.g[p], kSkip | kSlotCopy, bf16);
            ++s.h.n_copy;
        }
    const unsigned long long skip = s.h.n_copy ? s.slot[n - 1] & ~static_cast<unsigned long long>(kSlotCopy) : none;
    for (int k = 0; k < kSlotFill; ++k) s.slot[n + k] = skip;
    s.h.w = a.w;
    s.h.v = a.v;
    s.h.recv = a.recv;
    const long long back = run_back(a.e0, a.n);
    s.h.e0 = a.e0 - back;
    s.h.n = a.n + back;
    s.h.skip = static_cast<int>(back / 4);
    s.h.inv_P = a.inv_P;
    s.h.neg_lr = a.neg_lr;
    s.h.mu = a.mu;
    s.h.wd = a.wd;
    s.h.nesterov = a.nesterov;
    s.stats = a.stats;
}

template <bool BF16, bool FAST, bool NTS, bool OPT>
hipError_t launch_slots(SlotArgs &s, long long model, const Launch &cfg, hipStream_t st)
{
    const long long tiles = (slot_nvec<BF16>(s.h.n) + 63) / 64;
    const int per = cfg.block / 64;                    // wavefronts per workgroup
    const long long g = round_workgroups(s.h.n, BF16, cfg.block);
    if (g * cfg.block > kMaxRoundThreads) return hipErrorInvalidValue;     // (no run of a call is as long)
    const dim3 grid(static_cast<unsigned>(g));
    s.h.waves_per_block = per;
    s.h.xcd_blocks = cfg.xcd_map ? static_cast<int>(g / 8) : 0;
    const long long per_element = round_bytes(s, OPT);
    const bool small = small_round(s, per_element), plain = model * per_element <= kPlainRoundBytes;
    int bpc = cfg.blocks_per_cu;
    if (bpc == 0) {
        const int w = small || cfg.chunk != 0 ? -1 : burst_waves(s, tiles, s.stats.stats != nullptr, OPT, NTS);
        bpc = w < 0 ? -1 : (w + per - 1) / per;
    }
    const bool stats = s.stats.stats != nullptr;
    // The receive buffer may be a late process's gradient buffer: that gradient has to be carried
    // before the result is stored over it, which is the order of the chunk kernel.  (Copies before
    // the update in the burst kernel too: 0.4 % slower over all rounds with copies, up to 1.5 %.)
    bool late_in_recv = false;
    for (int k = s.h.n_sum; !small && k < s.h.n_sum + s.h.n_copy; ++k)
        late_in_recv |= (s.slot[k] & ~static_cast<unsigned long long>(kSlotTag)) ==
                        reinterpret_cast<unsigned long long>(s.h.recv);
    if (cfg.chunk == 0 && !small && !late_in_recv)
        return stats ? launch_capped(burst_kernel<BF16, FAST, NTS, OPT, true>, s, bpc, cfg, grid, st)
                     : launch_capped(burst_kernel<BF16, FAST, NTS, OPT, false>, s, bpc, cfg, grid, st);
    // (launch options are for the general kernel)
    if (cfg.chunk == 0 && small && cfg.block == 64 && !cfg.xcd_map && bpc < 0 && !NTS && short_round(s) &&
        short_pays(s, BF16, FAST, !plain, OPT)) {
        ShortLauncher *const f = BF16 ? (FAST ? launch_short_bf16_fast : launch_short_bf16)
                                      : (FAST ? launch_short_f32_fast : launch_short_f32);
        return f(s, !plain, st);
    }
    // (8-slot chunks with by-products serve the rule's own choice of short lists; as a launch option
    // that pair has always been refused, by the caller with a message of its own)
    if (stats && cfg.chunk == 8) return hipErrorInvalidValue;
    const bool few = cfg.chunk == 8 || (cfg.chunk == 0 && s.h.n_sum + s.h.n_copy <= 8);
    ChunkLauncher *const fixed = BF16 ? (stats ? launch_chunk_bf16_stats : launch_chunk_bf16)
                                      : (stats ? launch_chunk_f32_stats : launch_chunk_f32);
    ChunkLauncher *const any = BF16 ? (stats ? launch_chunk_bf16_fast_stats : launch_chunk_bf16_fast)
                                    : (stats ? launch_chunk_f32_fast_stats : launch_chunk_f32_fast);
    return (FAST ? any : fixed)(s, !plain, NTS, few, bpc, cfg, st);
}

template <bool BF16, bool FAST>
hipError_t launch_slots(const RoundArgs &a, const Launch &cfg, hipStream_t st)
{
    SlotArgs s;
    build_slots(a, s);
    // w, v (and recv) of a run that cannot stay in the 256 MiB last-level cache until the
    // next round are streamed; smaller ones are left to the cache
    const long long state_bytes = s.h.n * 4 * ((s.h.w ? 2 : 0) + (s.h.recv ? 1 : 0));
    const bool nts = cfg.nt_state < 0 ? state_bytes > kStateCacheBytes : cfg.nt_state != 0;
    if (s.h.w) return nts ? launch_slots<BF16, FAST, true, true>(s, a.model, cfg, st)
                        : launch_slots<BF16, FAST, false, true>(s, a.model, cfg, st);
    return nts ? launch_slots<BF16, FAST, true, false>(s, a.model, cfg, st)
               : launch_slots<BF16, FAST, false, false>(s, a.model, cfg, st);
}

}  // namespace

hipError_t launch_round(const RoundArgs &a, bool bf16, bool fast, const Launch &cfg,
                        hipStream_t stream)
{
    if (a.n <= 0) return hipSuccess;
    if (bf16)
        return fast ? launch_slots<true, true>(a, cfg, stream)
                    : launch_slots<true, false>(a, cfg, stream);
    return fast ? launch_slots<false, true>(a, cfg, stream)
                : launch_slots<false, false>(a, cfg, stream);
}

template <bool BF16, int V>
hipError_t launch_carry_v(const CarryArgs &a, const Launch &cfg, hipStream_t stream)
{
    const long long nvec = a.n / 4;
    const long long tile = static_cast<long long>(cfg.carry_block) * V;
    long long bpp = (nvec + tile - 1) / tile;     // workgroups per pair: they cover it
    if (bpp < 1) bpp = 1;
    // A grid may hold fewer than 2^32 threads in all: the pairs go into as many launches as it
    // takes.  (One pair always fits: a call covers at most 2^33 elements per run.)
    const long long limit = kMaxGridThreads / cfg.carry_block;
    if (bpp > limit) return hipErrorInvalidValue;
    long long pairs_per_launch = std::min<long long>(limit / bpp, 65535);
    Launch l = cfg;
    l.block = cfg.carry_block;
    for (int first = 0; first < a.count; first += static_cast<int>(pairs_per_launch)) {
        CarryArgs part = a;
        part.count = static_cast<int>(std::min<long long>(pairs_per_launch, a.count - first));
        for (int k = 0; k < part.count; ++k) {
            part.src[k] = a.src[first + k];
            part.dst[k] = a.dst[first + k];
        }
        const dim3 grid(static_cast<unsigned>(bpp), static_cast<unsigned>(part.count));
        const hipError_t e = part.skip ? launch_capped(carry_kernel<BF16, V, true>, part, cfg.carry_blocks_per_cu, l, grid, stream)
                                       : launch_capped(carry_kernel<BF16, V, false>, part, cfg.carry_blocks_per_cu, l, grid, stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <bool BF16>
hipError_t launch_carry_t(const CarryArgs &a, const Launch &cfg, hipStream_t stream)
{
    switch (cfg.carry_vec) {
    case 1: return launch_carry_v<BF16, 1>(a, cfg, stream);
    case 2: return launch_carry_v<BF16, 2>(a, cfg, stream);
    case 4: return launch_carry_v<BF16, 4>(a, cfg, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_carry(const CarryArgs &args, bool bf16, const Launch &cfg, hipStream_t stream)
{
    if (args.n <= 0 || args.count <= 0) return hipSuccess;
    CarryArgs a = args;
    const long long back = run_back(a.e0, a.n);
    a.e0 -= back;
    a.n += back;
    a.skip = static_cast<int>(back / 4);
    return bf16 ? launch_carry_t<true>(a, cfg, stream) : launch_carry_t<false>(a, cfg, stream);
}

long long slot_records(long long n, bool bf16, int)
{
    const long long nvec = bf16 ? slot_nvec<true>(n) : slot_nvec<false>(n);
    return (nvec + 63) / 64;
}

int slot_tail(long long n, bool bf16)
{
    return static_cast<int>(n - (bf16 ? slot_nvec<true>(n) : slot_nvec<false>(n)) * 4);
}

}  // namespace eager
