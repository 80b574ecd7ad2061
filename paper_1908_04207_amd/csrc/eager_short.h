// gfx950 kernel of the round for small runs with a short list: up to 16 streams, which is every round of up to 8
// processes.  Included by the files that instantiate it, one per gradient type and order.
//
// What bounds such a run is a launch, one trip to the arguments and one to the streams, and the trip to the arguments
// depends on how many lines they are: 64 elements, 8 processes, 4 late, one launch after another 2.13 us with
// chunk_kernel (552 bytes, 9 lines asked for), 2.02 with 256 bytes in 4 lines, 2.26 with 320 in 5.  The host copies
// fewer bytes too (hipLaunchKernel with arguments of 24, 552 and 1716 bytes: 2.5, 3.1, 3.8 us).  Chunks and this, one call
// per bucket: 16 k elements 2.82 and 2.68, 131 k 3.92 and 3.75, 262 k 5.70 and 5.43; 4 processes, 2 late, 16 k 2.64 and 2.52.
#pragma once

#include "eager_chunk.h"

namespace eager {
namespace {

// What one wavefront does: lane-vectors [at0, at0 + 64) of W elements, up to `end`, the whole list in flight at once.
// What `h` holds is in scalar registers; a slot is a load and a branch, see chunk_body.
template <int W, int CH, bool BF16, bool FAST, bool NT, bool OPT>
__device__ __forceinline__ void short_body(const ShortArgs<CH> &h, unsigned at0, unsigned end)
{
    typedef typename Width<W>::type V;
    constexpr int kHalf = ShortArgs<CH>::kHalf;
    const unsigned lane = threadIdx.x & 63u, mine = at0 + lane;
    const unsigned begin = (h.shape >> kShortSkip) / W;                  // (inside the first tile)
    const unsigned up = mine > begin ? mine : begin, at = up < end ? up : end - 1u;
    const bool in = at == mine;
    unsigned off = at * (4u * W), off_bf = W == 4 ? (at >> 1) * 16u : at * 2u;
    const bool odd = (at & 1u) != 0u;
    const int n_sum = static_cast<int>(h.shape & 255u), n_last = static_cast<int>(h.shape >> 8 & 255u);

    V s = (V)(0.0f), s2 = s, s3 = s, s4 = s, x[CH];
    V half[W == 1 && BF16 ? CH : 1];
    V vo = (V)(0.0f), wo = vo;
    if (OPT) {
        vo = ld_vec<W, false>(h.v, off);
        wo = ld_vec<W, false>(h.w, off);
    }
    auto request = [&](auto J) {
        constexpr int j = decltype(J)::value;
        const char *base = reinterpret_cast<const char *>(h.slot[j]);
        if constexpr (!BF16) x[j] = ld_vec<W, NT>(base, off);
        else if constexpr (W == 4) x[j] = ld_vec<W, NT>(base, h.bits >> (16 + j) & 1u ? off_bf : off);
        else if (h.bits >> (16 + j) & 1u) half[j] = ld_half<NT>(base, off_bf);
        else x[j] = ld_vec<W, NT>(base, off);
    };
    // (Two ways into one register make the compiler wait for all that is on its way before the second: the copies
    // loaded from the back of the sum's slots were 0.25 us slower where there are any.)
    if constexpr (CH == 16) first_of<8>(n_sum, request);
    first_of<8>(n_last, [&](auto J) { request(std::integral_constant<int, kHalf + decltype(J)::value>()); });
#pragma unroll
    for (int j = 0; j < CH; ++j) {
        if constexpr (W == 1 && BF16) asm volatile("; %2" : "+v"(x[j]), "+v"(half[j]) : "n"(W) : "memory");
        else asm volatile("; %1" : "+v"(x[j]) : "n"(W) : "memory");
    }
    int sums = opaque<W>(n_sum);
    const unsigned bits = opaque<W>(h.bits), copies = opaque<W>(h.copies);
    if (BF16) {
#pragma unroll
        for (int j = 0; j < CH; ++j)
            if (bits >> (16 + j) & 1u) {
                if constexpr (W == 1) x[j] = widen(half[j]);
                else x[j] = widen(x[j], odd);
                if (FAST && j < sums) {           // (sums of their own, and the fp32 streams stand before them)
                    V &part = j & 1 ? s4 : s3;
                    part = part + x[j];
                    asm volatile("; %1" : "+v"(part) : "n"(W));
                }
            }
        if (FAST) sums -= __builtin_popcount(bits >> 16 & ~copies);
    }
    if constexpr (!FAST) {
        if (bits & 0xffffu) {
#pragma unroll
            for (int j = 1; j < CH; ++j)
                if (bits >> j & 1u) {
                    x[j] = x[j - 1] + x[j];
                    x[j - 1] = (V)(0.0f);                 // (nothing more to add: s is never -0.0f)
                    asm volatile("; %2" : "+v"(x[j]), "+v"(x[j - 1]) : "n"(W));     // (a branch, not 8 selects)
                }
        }
    }
    first_of<CH>(sums, [&](auto J) {
        constexpr int j = decltype(J)::value;
        V &part = FAST && j & 1 ? s2 : s;
        part = part + x[j];
        asm volatile("; %1" : "+v"(part) : "n"(W));
    });
    // (stores stay behind the adds, see chunk_body)
    asm volatile("; %1" : "+v"(s) : "n"(W) : "memory");
    if constexpr (FAST) asm volatile("; %1" : "+v"(s2) : "n"(W) : "memory");
    if constexpr (FAST && BF16) asm volatile("; %2" : "+v"(s3), "+v"(s4) : "n"(W) : "memory");
    if (copies && in) {
#pragma unroll
        for (int j = kHalf; j < CH; ++j)
            if (copies >> j & 1u) st_vec<W, NT>(h.dst[j - kHalf], off, x[j]);
    }
    if constexpr (FAST) s = s + s2;
    if constexpr (FAST && BF16) s = s + (s3 + s4);
    const V avg = s * h.inv_P;
    V vn, wn;
    if (OPT) {
        const UpdateRule rule = {h.neg_lr, h.mu, h.wd, static_cast<int>(h.shape >> 16 & 1u)};
        apply_rule(rule, avg, vo, wo, vn, wn);
    }
    if (in) {
        if (h.recv) st_vec<W, false>(h.recv, off, avg);
        if (OPT) {
            st_vec<W, false>(h.v, off, vn);
            st_vec<W, false>(h.w, off, wn);
        }
    }
}

// The tiles of chunk_kernel.  All of the arguments are asked for at once.
template <bool BF16, bool FAST, bool NT, bool OPT, int CH>
__global__ __launch_bounds__(64) void short_kernel(const ShortArgs<CH>)
{
    ShortArgs<CH> h;
    __builtin_memcpy(&h, (const void __attribute__((address_space(4))) *)&kernarg<ShortArgs<CH>>(), sizeof h);
    asm volatile("" : "+s"(h.w), "+s"(h.v), "+s"(h.recv), "+s"(h.n), "+s"(h.shape), "+s"(h.bits), "+s"(h.copies), "+s"(h.inv_P),
                 "+s"(h.neg_lr), "+s"(h.mu), "+s"(h.wd));
#pragma unroll
    for (int j = 0; j < CH; ++j) asm volatile("" : "+s"(h.slot[j]));
#pragma unroll
    for (int j = 0; j < kShortCopies; ++j) asm volatile("" : "+s"(h.dst[j]));
    const unsigned wave = blockIdx.x;
    unsigned first = wave * 64u;
    if ((h.shape >> kShortForm & 3u) != kNarrow) {
        const unsigned nvec = BF16 ? h.n / 8u * 2u : h.n / 4u, tiles = (nvec + 63u) / 64u;
        if (wave < tiles) {
            short_body<4, CH, BF16, FAST, NT, OPT>(h, first, nvec);
            return;
        }
        first = wave == tiles ? nvec * 4u : h.n;
    }
    if (first < h.n) short_body<1, CH, BF16, FAST, NT, OPT>(h, first, h.n);
}

template <bool BF16, bool FAST, bool NT, bool OPT, int CH>
hipError_t launch_short_sized(const SlotArgs &s, int slots, hipStream_t st)
{
    const bool narrow = chunk_narrow(s.h.n, slots, s.h.n_copy, BF16, false, 0);
    ShortArgs<CH> a;
    fill_short(s, FAST, narrow ? kNarrow : kWide, a);
    const long long g = narrow ? (s.h.n + 63) / 64 : round_workgroups(s.h.n, BF16, 64);
    return launch(short_kernel<BF16, FAST, NT, OPT, CH>, dim3(static_cast<unsigned>(g)), dim3(64), 0, st, a);
}

template <bool BF16, bool FAST>
hipError_t launch_short(const SlotArgs &s, bool nt, hipStream_t st)
{
    const int slots = sum_terms(s) + s.h.n_copy;
    switch ((slots <= 8 ? 4 : 0) | (nt ? 2 : 0) | (s.h.w ? 1 : 0)) {
    case 0: return launch_short_sized<BF16, FAST, false, false, 16>(s, slots, st);
    case 1: return launch_short_sized<BF16, FAST, false, true, 16>(s, slots, st);
    case 2: return launch_short_sized<BF16, FAST, true, false, 16>(s, slots, st);
    case 3: return launch_short_sized<BF16, FAST, true, true, 16>(s, slots, st);
    case 4: return launch_short_sized<BF16, FAST, false, false, 8>(s, slots, st);
    case 5: return launch_short_sized<BF16, FAST, false, true, 8>(s, slots, st);
    case 6: return launch_short_sized<BF16, FAST, true, false, 8>(s, slots, st);
    default: return launch_short_sized<BF16, FAST, true, true, 8>(s, slots, st);
    }
}

}  // namespace
}  // namespace eager
