// gfx950 kernel of the round for small runs, whose time is the one from launch to the last store:
// a launch, one trip to the arguments, one trip to the streams.  Lists of up to 16 streams have a kernel of their own
// (eager_short.h); this one takes the longer ones, those that short_pays leaves to it, rounds with by-products and the launch options.  Included by the files that
// instantiate it, one per gradient type and order, with and without by-products (compiled side by side).
#pragma once

#include "eager_device.h"

#include <algorithm>
#include <type_traits>

namespace eager {
namespace {

// What a lane owns: W consecutive elements, 4 or 1, lane-vector number `at` of the launch.
template <int W> struct Width;
template <> struct Width<4> { typedef f32x4 type; };
template <> struct Width<1> { typedef float type; };

template <bool NT>
__device__ __forceinline__ float ld_one(const char *base, unsigned off)
{
    asm("" : "+v"(off));
    typedef const float __attribute__((address_space(1))) GF;
    GF *p = (GF *)(base + off);
    if (NT) return __builtin_nontemporal_load(p);
    return *p;
}
template <bool NT>
__device__ __forceinline__ float ld_half(const char *base, unsigned off)      // 16 bits, in the lower half
{
    asm("" : "+v"(off));
    typedef const unsigned short __attribute__((address_space(1))) GH;
    GH *p = (GH *)(base + off);
    const unsigned short x = NT ? __builtin_nontemporal_load(p) : *p;
    return __uint_as_float(static_cast<unsigned>(x));
}
template <bool NT>
__device__ __forceinline__ void st_one(char *base, unsigned off, float x)
{
    asm("" : "+v"(off));
    typedef float __attribute__((address_space(1))) GFw;
    GFw *p = (GFw *)(base + off);
    if (NT) __builtin_nontemporal_store(x, p);
    else *p = x;
}
template <int W, bool NT>
__device__ __forceinline__ typename Width<W>::type ld_vec(const void *base, unsigned off)
{
    const char *p = static_cast<const char *>(base);
    if constexpr (W == 4) return ld_at<NT>(p, off);
    else return ld_one<NT>(p, off);
}
template <int W, bool NT>
__device__ __forceinline__ void st_vec(void *base, unsigned off, typename Width<W>::type x)
{
    char *p = static_cast<char *>(base);
    if constexpr (W == 4) st_at<NT>(p, off, x);
    else st_one<NT>(p, off, x);
}

// A bf16 stream's values as loaded -> fp32.  W = 4: of the 16-byte piece that two lanes share the
// upper half belongs to the odd one.
__device__ __forceinline__ f32x4 widen(f32x4 raw, bool odd)
{
    const u32x4 r = __builtin_bit_cast(u32x4, raw);
    const unsigned a = odd ? r.z : r.x, b = odd ? r.w : r.y;
    f32x4 x;
    x.x = __uint_as_float(a << 16);
    x.y = __uint_as_float(a & 0xffff0000u);
    x.z = __uint_as_float(b << 16);
    x.w = __uint_as_float(b & 0xffff0000u);
    return x;
}
__device__ __forceinline__ float widen(float raw) { return __uint_as_float(__float_as_uint(raw) << 16); }

__device__ __forceinline__ void apply_rule(const UpdateRule &r, f32x4 u, f32x4 vo, f32x4 wo, f32x4 &vn, f32x4 &wn)
{
    update_rule<false>(r, u, vo, wo, vn, wn);
}
__device__ __forceinline__ void apply_rule(const UpdateRule &r, float u, float vo, float wo, float &vn, float &wn)
{
    vn = vo;
    wn = wo;
    update_rule_scalar(r, u, vn, wn);
}

// Copies out of the argument segment.
__device__ __forceinline__ ChunkHead read(const ChunkHead __attribute__((address_space(4))) &from)
{
    ChunkHead h;
    __builtin_memcpy(&h, (const void __attribute__((address_space(4))) *)&from, sizeof h);
    return h;
}
__device__ __forceinline__ ChunkBits read(const ChunkBits __attribute__((address_space(4))) &from)
{
    ChunkBits b;
    __builtin_memcpy(&b, (const void __attribute__((address_space(4))) *)&from, sizeof b);
    return b;
}

__device__ __forceinline__ int form_of(const ChunkHead &h) { return h.form & ((1 << kFormBits) - 1); }

// A word that the compiler must not connect with an earlier look at it: it would bring a load down to
// where its value is used, next to the other branch that asks for the same slot.
// (W, as a remark in the assembly, keeps the two widths' statements apart.)
template <int W, typename T>
__device__ __forceinline__ T opaque(T x)
{
    asm volatile("; %1" : "+s"(x) : "n"(W));
    return x;
}

// f(0), f(1), ... f(n - 1), at most CH of them, by number: one branch per step, one way out.
template <int CH, int J = 0, typename F>
__device__ __forceinline__ void first_of(int n, const F &f)
{
    if constexpr (J < CH) {
        if (__builtin_expect(n > J, 1)) {
            f(std::integral_constant<int, J>());
            first_of<CH, J + 1>(n, f);
        }
    }
}

// s_waitcnt vmcnt(0) and nothing else
constexpr int kStoresArrived = 0x0f70;

// What one wavefront does: lane-vectors [at0, at0 + 64) of W elements, up to `end`, with CH slots in
// flight.  What bounds it is how many instructions a wavefront issues between its trips to memory - a
// wavefront on its own issues one in 4 cycles or more, 600 of them are a microsecond - so nothing is done
// for a slot that is not there, and what is done with one is a branch on a bit: a load is one
// instruction, an ADD one per element.  (All loads are waited for together, before the first branch
// that depends on a slot's kind: the registers of a slot that was not read are never looked at.)
template <int W, int CH, bool BF16, bool FAST, bool NT, bool NTS, bool OPT, bool STATS, int READ, typename K>
__device__ __forceinline__ void chunk_body(K &a, const ChunkHead &h, const unsigned long long (&slot)[READ], unsigned at0,
                                           unsigned end, long long record)
{
    typedef typename Width<W>::type V;
    const unsigned lane = threadIdx.x & 63u, mine = at0 + lane;
    const unsigned begin = (static_cast<unsigned>(h.form) >> kFormBits) / W;       // (inside the first tile)
    const unsigned up = mine > begin ? mine : begin, at = up < end ? up : end - 1u;
    const bool in = at == mine;
    const unsigned off = at * (4u * W);
    const unsigned off_bf = W == 4 ? (at >> 1) * 16u : at * 2u;
    const bool odd = (at & 1u) != 0u;

    // (FAST: no pairs, but two sums that take the fp32 streams in turn, s and s2, and two of the bf16 streams, s3 and
    // s4, in which hardly anything is rounded.  Every second process with a pending buffer, bf16 gradients, error against
    // 64 bits relative to two sums of all: 0.89 with 2 processes, 0.74 with 4, 0.66 with 16, 0.59 with 64.)
    V s = (V)(0.0f), s2 = s, s3 = s, s4 = s, held = s, x[CH];
    // (W = 1: loads of 2 and of 4 bytes into registers of their own, or the one on the other branch
    // waits for the one before it)
    V half[W == 1 && BF16 ? CH : 1];
    auto request = [&](int k0, const ChunkBits &b, auto address) {
        first_of<CH>(h.n_slots - k0, [&](auto J) {
            constexpr int j = decltype(J)::value;
            const char *base = reinterpret_cast<const char *>(address(J));
            if constexpr (!BF16) x[j] = ld_vec<W, NT>(base, off);
            else if constexpr (W == 4) x[j] = ld_vec<W, NT>(base, b.bf >> j & 1u ? off_bf : off);
            else if (b.bf >> j & 1u) half[j] = ld_half<NT>(base, off_bf);
            else x[j] = ld_vec<W, NT>(base, off);
        });
    };
    // the sum, then the copies, of the slots in flight
    auto consume = [&](int k0, ChunkBits b) {
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            if constexpr (W == 1 && BF16) asm volatile("; %2" : "+v"(x[j]), "+v"(half[j]) : "n"(W) : "memory");
            else asm volatile("; %1" : "+v"(x[j]) : "n"(W) : "memory");
        }
        int sums = opaque<W>(h.n_sum) - k0;
        if (BF16) {
            b.bf = opaque<W>(b.bf);
            // (FAST: these go into sums of their own, and the fp32 streams stand before them)
            const unsigned apart = !FAST || sums <= 0 ? 0u : sums < CH ? b.bf & ((1u << sums) - 1u) : b.bf & (~0u >> (32 - CH));
#pragma unroll
            for (int j = 0; j < CH; ++j)
                if (b.bf >> j & 1u) {
                    if constexpr (W == 1) x[j] = widen(half[j]);
                    else x[j] = widen(x[j], odd);
                    if (FAST && (apart >> j & 1u)) {
                        V &part = j & 1 ? s4 : s3;
                        part = part + x[j];
                        asm volatile("; %1" : "+v"(part) : "n"(W));
                    }
                }
            if (FAST) sums = (sums < CH ? sums : CH) - __builtin_popcount(apart);
        }
        if constexpr (!FAST) {
            b.pair = opaque<W>(b.pair);
#pragma unroll
            for (int g = 0; g < CH; g += 8)
                if (b.pair >> g & 255u) {
#pragma unroll
                    for (int j = g; j < g + 8; ++j)
                        if (b.pair >> j & 1u) {
                            V &before = j ? x[j ? j - 1 : 0] : held;
                            x[j] = before + x[j];
                            before = (V)(0.0f);           // (nothing more to add: s is never -0.0f)
                            asm volatile("; %2" : "+v"(x[j]), "+v"(before) : "n"(W));     // (a branch, not 8 selects)
                        }
                }
            if (sums > CH && (b.hold >> (CH - 1) & 1u)) {
                held = x[CH - 1];
                x[CH - 1] = (V)(0.0f);
            }
        }
        first_of<CH>(sums, [&](auto J) {
            constexpr int j = decltype(J)::value;
            V &part = FAST && j & 1 ? s2 : s;
            part = part + x[j];
            asm volatile("; %1" : "+v"(part) : "n"(W));
        });
        // Stores stay behind the adds: moved ahead of them, the in-order memory counter would make
        // every add wait for the acknowledgement of a store instead of for its load.
        asm volatile("; %1" : "+v"(s) : "n"(W) : "memory");
        if constexpr (FAST) asm volatile("; %1" : "+v"(s2) : "n"(W) : "memory");
        if constexpr (FAST && BF16) asm volatile("; %2" : "+v"(s3), "+v"(s4) : "n"(W) : "memory");
        b.copy = opaque<W>(b.copy);
        if (b.copy && in) {
#pragma unroll
            for (int g = 0; g < CH; g += 8)
                if (b.copy >> g & 255u) {
                    auto *dst = &a.dst[k0 + g - h.dst_first];
                    float *to[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) to[j] = dst[j];
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (b.copy >> (g + j) & 1u) {
                            st_vec<W, NT>(to[j], off, x[g + j]);
                            if (NT && W == 4 && CH == 16 && form_of(h) == kPaced) __builtin_amdgcn_s_waitcnt(kStoresArrived);
                        }
                }
        }
    };

    V vo = (V)(0.0f), wo = vo;
    if (OPT) {
        vo = ld_vec<W, NTS>(h.v, off);
        wo = ld_vec<W, NTS>(h.w, off);
    }
    // w and v go first (16 processes on time, bf16, 72 MiB moved: 10.8 us, 15.7 with them last)
    request(0, h.first, [&](auto J) {
        constexpr int j = decltype(J)::value;
        if constexpr (j < READ) return slot[j];
        else return a.slot[j];
    });
    LaneStats ls = {0.0, 0.0, 0u, -1};
    int n_valid = 0;
    if constexpr (STATS) {
        const long long e = a.first + static_cast<long long>(at) * W;
        if constexpr (W == 4) {
            long long stop;
            const int b = tile_bucket(a.stats.table, a.stats.b_lo, a.stats.b_hi, a.first + at0 * 4ll, e, stop);
            if (mine < end) ls.bucket = b;             // (in front of the run: the bucket of its first element)
            if (in) n_valid = inside(e, stop);
        } else {
            ls.bucket = find_bucket(a.stats.table, a.stats.n_buckets, e);
            if (e < a.stats.table[2 * ls.bucket + 1]) n_valid = 1;
            else ls.bucket = -2;                                   // padding
        }
    }
    consume(0, h.first);
    // (the first chunk stands apart: at the head of a loop the compiler waits for everything in
    // flight, w and v among it, before the first slot is requested)
    for (int k0 = CH; k0 < h.n_slots; k0 += CH) {
        ChunkBits b = read(a.bits[k0 / kChunkWord]);
        const int shift = k0 % kChunkWord;
        b.pair >>= shift;
        b.hold >>= shift;
        b.copy >>= shift;
        b.bf >>= shift;
        request(k0, b, [&](auto J) { return a.slot[k0 + decltype(J)::value]; });
        consume(k0, b);
    }

    if constexpr (FAST) s = s + s2;
    if constexpr (FAST && BF16) s = s + (s3 + s4);
    const V avg = s * h.inv_P;
    if constexpr (STATS) {
        if constexpr (W == 4) {
            stats_vector<OPT>(ls, avg, wo, n_valid);
        } else if (n_valid) {
            stats_add(ls, avg, OPT ? wo : 0.0f, OPT);
        }
    }
    V vn, wn;
    if (OPT) {
        const UpdateRule rule = {h.neg_lr, h.mu, h.wd, h.nesterov};
        apply_rule(rule, avg, vo, wo, vn, wn);
    }
    if (in) {
        if (h.recv) st_vec<W, NTS>(h.recv, off, avg);
        if (OPT) {
            st_vec<W, NTS>(h.v, off, vn);
            st_vec<W, NTS>(h.w, off, wn);
        }
        if constexpr (STATS && W == 1) {
            // the ragged tail: one record per element, in the block after the last bucket's
            const StatsRecord rec = {ls.ssu, ls.ssw, ls.bucket, ls.nf, 0};
            a.stats.lane_records[static_cast<long long>(a.stats.n_buckets) * 64 + lane] = rec;
        }
    }
    if constexpr (STATS && W == 4) stats_commit(a.stats.records, a.stats.lane_records, ls, record);
}

// One tile of 64 lane-vectors per wavefront, 4 elements to a lane, and the ragged tail (at most 3
// elements, 7 with bf16 gradients) by a wavefront of its own, one element to a lane.  A very small run
// is taken one element to a lane altogether: a quarter of the arithmetic in each of four times as many
// wavefronts, for which there is room.
template <bool BF16, bool FAST, bool NT, bool NTS, bool OPT, bool STATS, int CH, typename ARGS>
__global__ __launch_bounds__(256) void chunk_kernel(const ARGS)
{
    const ARGS __attribute__((address_space(4))) &a = kernarg<ARGS>();
    // The head, the first slots and a word of the lines that follow are requested at once - all lines of the
    // short block; of the long one slots up to 63 and destinations up to 24 -: read where they are used, each is
    // a trip of its own (32 processes, 16 late, 64 elements: 5.37 us with the lines of a short list only, 4.80 with
    // these).
    ChunkHead h = read(a.h);
    unsigned long long slot[CH];
#pragma unroll
    for (int j = 0; j < CH; ++j) slot[j] = a.slot[j];
    typedef const unsigned __attribute__((address_space(4))) Word;
    constexpr int far = ARGS::kSlots > kChunkWord ? kChunkWord : 0, step = far / 4;
    const unsigned line[] = {*(Word *)&a.slot[16], *(Word *)&a.slot[24], *(Word *)&a.dst[0], *(Word *)&a.dst[8],
                             *(Word *)&a.dst[16], *(Word *)&a.slot[far], *(Word *)&a.slot[far + step],
                             *(Word *)&a.slot[far + 2 * step], *(Word *)&a.slot[far + 3 * step],
                             *(Word *)&a.dst[3 * step], *(Word *)&a.bits[far / kChunkWord]};
    if constexpr (far > 0)
        asm volatile("" : "+s"(h.w), "+s"(slot[0]), "+s"(slot[CH - 1]) : "s"(line[0]), "s"(line[1]), "s"(line[2]),
                     "s"(line[3]), "s"(line[4]), "s"(line[5]), "s"(line[6]), "s"(line[7]), "s"(line[8]),
                     "s"(line[9]), "s"(line[10]));
    else
        asm volatile("" : "+s"(h.w), "+s"(slot[0]), "+s"(slot[CH - 1]) : "s"(line[0]), "s"(line[1]), "s"(line[2]),
                     "s"(line[3]), "s"(line[4]));
    asm volatile("" : "+s"(h.v), "+s"(h.recv), "+s"(h.n), "+s"(h.n_sum), "+s"(h.n_slots));
    asm volatile("" : "+s"(h.dst_first), "+s"(h.form), "+s"(h.waves_per_block), "+s"(h.xcd_blocks),
                 "+s"(h.inv_P), "+s"(h.neg_lr), "+s"(h.mu), "+s"(h.wd), "+s"(h.nesterov));
    asm volatile("" : "+s"(h.first.pair), "+s"(h.first.hold), "+s"(h.first.copy), "+s"(h.first.bf));
#pragma unroll
    for (int j = 1; j < CH - 1; ++j) asm volatile("" : "+s"(slot[j]));
    // Workgroups are dealt to the 8 XCDs round robin; xcd_blocks gives every XCD one contiguous
    // eighth of the launch instead (a launch option, for A/B).
    unsigned bid = blockIdx.x;
    const unsigned per = static_cast<unsigned>(h.xcd_blocks);
    if (per && bid < per * 8u) bid = (bid % 8u) * per + bid / 8u;
    const unsigned wave = bid * static_cast<unsigned>(h.waves_per_block) +
                          static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)));
    unsigned first = wave * 64u;
    if (form_of(h) != kNarrow) {
        const unsigned nvec = BF16 ? h.n / 8u * 2u : h.n / 4u, tiles = (nvec + 63u) / 64u;
        if (wave < tiles) {
            chunk_body<4, CH, BF16, FAST, NT, NTS, OPT, STATS>(a, h, slot, first, nvec, wave);
            return;
        }
        first = wave == tiles ? nvec * 4u : h.n;
    }
    if (first < h.n) chunk_body<1, STATS ? 16 : 32, BF16, FAST, NT, NTS, OPT, STATS>(a, h, slot, first, h.n, 0);
}

template <typename A>
int kernel_waves(void (*kernel)(A))
{
    hipFuncAttributes of;
    if (hipFuncGetAttributes(&of, reinterpret_cast<const void *>(kernel)) == hipSuccess) return resident_waves(of.numRegs);
    (void)hipGetLastError();
    return 0;
}

template <bool BF16, bool FAST, bool NT, bool NTS, bool OPT, bool STATS, int CH, typename A>
hipError_t launch_segments(const SlotArgs &s, A &a, int bpc, const Launch &cfg, hipStream_t st)
{
    const int per = cfg.block / 64;                    // wavefronts per workgroup
    for (long long first = 0; first < s.h.n; first += kChunkElements) {
        const long long n = std::min(s.h.n - first, kChunkElements);
        fill_chunk(s, FAST, first, n, a);
        const bool narrow = chunk_narrow(s.h.n, a.h.n_slots, s.h.n_copy, BF16, STATS, cfg.chunk);
        a.h.form |= narrow ? kNarrow : kWide;
        if constexpr (NT && CH == 16)
            if (!narrow && chunk_paced(s, a.h.n_slots, BF16, OPT, 32)) {
                // (the kernel is asked for its registers once, and only where all else speaks for it)
                static const int resident = kernel_waves(chunk_kernel<BF16, FAST, NT, NTS, OPT, STATS, CH, A>);
                if (chunk_paced(s, a.h.n_slots, BF16, OPT, resident)) a.h.form |= kPaced;
            }
        const long long g = narrow ? (n + cfg.block - 1) / cfg.block : round_workgroups(n, BF16, cfg.block);
        a.h.waves_per_block = per;
        a.h.xcd_blocks = cfg.xcd_map ? static_cast<int>(g / 8) : 0;
        if constexpr (STATS) {
            a.first = s.h.e0 + first;
            a.stats = s.stats;
            a.stats.records += first / 256;
        }
        const hipError_t e = launch_capped(chunk_kernel<BF16, FAST, NT, NTS, OPT, STATS, CH, A>, a, bpc, cfg,
                                           dim3(static_cast<unsigned>(g)), st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <bool BF16, bool FAST, bool NT, bool NTS, bool OPT, bool STATS, int CH>
hipError_t launch_sized(const SlotArgs &s, int bpc, const Launch &cfg, hipStream_t st)
{
    // (w, v and recv are streamed in runs too long for the shorter block to matter)
    if constexpr (!NTS)
        if (chunk_fits(s, kChunkFewSlots, kChunkFewCopies)) {
            ChunkArgs<kChunkFewSlots, kChunkFewCopies, STATS> a;
            return launch_segments<BF16, FAST, NT, false, OPT, STATS, CH>(s, a, bpc, cfg, st);
        }
    ChunkArgs<kMaxSlots, kMaxP, STATS> a;
    return launch_segments<BF16, FAST, NT, NTS, OPT, STATS, CH>(s, a, bpc, cfg, st);
}

template <bool BF16, bool FAST, bool OPT, bool STATS, int CH>
hipError_t launch_hints(const SlotArgs &s, bool nt, bool nts, int bpc, const Launch &cfg, hipStream_t st)
{
    if (nts) return nt ? launch_sized<BF16, FAST, true, true, OPT, STATS, CH>(s, bpc, cfg, st)
                       : launch_sized<BF16, FAST, false, true, OPT, STATS, CH>(s, bpc, cfg, st);
    return nt ? launch_sized<BF16, FAST, true, false, OPT, STATS, CH>(s, bpc, cfg, st)
              : launch_sized<BF16, FAST, false, false, OPT, STATS, CH>(s, bpc, cfg, st);
}

template <bool BF16, bool FAST, bool STATS>
hipError_t launch_kind(const SlotArgs &s, bool nt, bool nts, bool eight, int bpc, const Launch &cfg,
                       hipStream_t st)
{
    if (s.h.w) return eight ? launch_hints<BF16, FAST, true, STATS, 8>(s, nt, nts, bpc, cfg, st)
                            : launch_hints<BF16, FAST, true, STATS, 16>(s, nt, nts, bpc, cfg, st);
    return eight ? launch_hints<BF16, FAST, false, STATS, 8>(s, nt, nts, bpc, cfg, st)
                 : launch_hints<BF16, FAST, false, STATS, 16>(s, nt, nts, bpc, cfg, st);
}

}  // namespace
}  // namespace eager
