// Device-side helpers shared by the kernel files: vector types and nontemporal accesses, the
// update rule, the per-bucket statistics (DPP wavefront sums, records) and the launch helper that
// caps occupancy.  Everything here has internal linkage; not part of the public ABI.
#pragma once

#include "eager_internal.h"
#include "eager_rules.h"

#include <mutex>
#include <set>

namespace eager {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Kernel arguments are read straight from the kernel-argument segment (constant address
// space, scalar loads).  Going through the by-value parameter instead makes the compiler
// keep a private copy of the whole struct in scratch memory as soon as it is indexed
// dynamically in more places than its copy-elision looks at.
typedef const SlotArgs __attribute__((address_space(4))) KSlotArgs;
template <typename T>
__device__ __forceinline__ const T __attribute__((address_space(4))) &kernarg()
{
    return *(const T __attribute__((address_space(4))) *)__builtin_amdgcn_kernarg_segment_ptr();
}

template <bool NT>
__device__ __forceinline__ f32x4 ld_f4(const float *p)
{
    if (NT) return __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
    return *reinterpret_cast<const f32x4 *>(p);
}
template <bool NT>
__device__ __forceinline__ void st_f4(float *p, f32x4 x)
{
    if (NT) __builtin_nontemporal_store(x, reinterpret_cast<f32x4 *>(p));
    else *reinterpret_cast<f32x4 *>(p) = x;
}
template <bool NT>
__device__ __forceinline__ u32x4 ld_u4(const void *p)
{
    if (NT) return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return *reinterpret_cast<const u32x4 *>(p);
}

// An access as a uniform base and a 32-bit byte offset of the lane.
typedef const f32x4 __attribute__((address_space(1))) GF4;
typedef f32x4 __attribute__((address_space(1))) GF4w;

// (the empty statement keeps the widening of the offset next to the access, where it folds into
// the instruction's scalar-base form; hoisted out of it, every stream would hold a 64-bit address
// per lane)
template <bool NT>
__device__ __forceinline__ f32x4 ld_at(const char *base, unsigned off)
{
    asm("" : "+v"(off));
    GF4 *p = (GF4 *)(base + off);
    if (NT) return __builtin_nontemporal_load(p);
    return *p;
}
template <bool NT>
__device__ __forceinline__ void st_at(char *base, unsigned off, f32x4 x)
{
    asm("" : "+v"(off));
    GF4w *p = (GF4w *)(base + off);
    if (NT) __builtin_nontemporal_store(x, p);
    else *p = x;
}

// The update rule U of Algorithm 2, lines 7-8, for one element or one vector of 4:
//   g = u + wd*w  (only if wd != 0);  v' = mu*v + g;  step = nesterov ? g + mu*v' : v';
//   w' = w - lr*step
// every line one fused multiply-add (single rounding) in fixed-order mode.  wd and nesterov
// are uniform over the grid; with wd = 0 and nesterov = 0 this is plain heavy-ball momentum.
struct UpdateRule {
    float neg_lr, mu, wd;
    int nesterov;
};

__device__ __forceinline__ float fma1(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ f32x4 fma4(float a, f32x4 b, f32x4 c)
{
    f32x4 r;
    r.x = __builtin_fmaf(a, b.x, c.x);
    r.y = __builtin_fmaf(a, b.y, c.y);
    r.z = __builtin_fmaf(a, b.z, c.z);
    r.w = __builtin_fmaf(a, b.w, c.w);
    return r;
}

template <bool FAST>
__device__ __forceinline__ void update_rule(const UpdateRule &r, f32x4 u, f32x4 vo, f32x4 wo,
                                            f32x4 &vn, f32x4 &wn)
{
    if (FAST) {
#pragma clang fp contract(fast)
        f32x4 g = u;
        if (r.wd != 0.0f) g = r.wd * wo + u;
        vn = r.mu * vo + g;
        f32x4 step = vn;
        if (r.nesterov) step = r.mu * vn + g;
        wn = r.neg_lr * step + wo;
    } else {
        f32x4 g = u;
        if (r.wd != 0.0f) g = fma4(r.wd, wo, u);
        vn = fma4(r.mu, vo, g);
        f32x4 step = vn;
        if (r.nesterov) step = fma4(r.mu, vn, g);
        wn = fma4(r.neg_lr, step, wo);
    }
}

__device__ __forceinline__ void update_rule_scalar(const UpdateRule &r, float u, float &v, float &w)
{
    float g = u;
    if (r.wd != 0.0f) g = fma1(r.wd, w, u);
    const float vn = fma1(r.mu, v, g);
    float step = vn;
    if (r.nesterov) step = fma1(r.mu, vn, g);
    v = vn;
    w = fma1(r.neg_lr, step, w);
}

// One gradient element of a ragged tail (fewer elements than a vector; scalar code, at most 7
// elements per launch).
template <bool BF16>
__device__ __forceinline__ float load_grad_scalar(const void *g, long long i)
{
    if (BF16) {
        const unsigned short h = static_cast<const unsigned short *>(g)[i];
        return __uint_as_float(static_cast<unsigned>(h) << 16);
    }
    return static_cast<const float *>(g)[i];
}

// Per-bucket by-products (optional): sum of squares of the averaged update and of the
// parameters, count of non-finite elements.  They are reductions ACROSS elements, the one
// place on this path where cross-lane work belongs: a lane sums its 4 elements, the 64 lanes
// of a wavefront are combined with DPP moves inside rows of 16 lanes and lane reads across
// the 4 rows, and one lane writes one record per wavefront.  A wavefront whose elements lie in
// several buckets leaves one record per lane instead.  A finishing kernel adds the records of a bucket,
// combining the wavefronts of its workgroup through LDS and several workgroups through memory.  Fixed trees, whoever
// arrives last: the result is reproducible bit for bit.
struct LaneStats {
    double ssu, ssw;   // squares of the update / of the old parameters
    unsigned nf;       // non-finite elements of the update
    int bucket;        // -1: the lane holds no element
};

// DPP controls: quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror, row_mirror.  Applied
// in this order every lane ends with the sum over its row of 16; all lanes must be active.
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;
constexpr int kDppRotate4 = 0x124, kDppRotate8 = 0x128;      // row_ror

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(b), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(b >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (static_cast<unsigned long long>(static_cast<unsigned>(hi)) << 32) |
                                          static_cast<unsigned>(lo));
}
template <int CTRL>
__device__ __forceinline__ unsigned dpp_u32(unsigned x)
{
    return static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ double readlane_f64(double x, int lane)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = __builtin_amdgcn_readlane(static_cast<int>(b), lane);
    const unsigned hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), lane);
    return __builtin_bit_cast(double, (static_cast<unsigned long long>(hi) << 32) | lo);
}
// sum over the 64 lanes of the wavefront, the same value in every lane (uniform)
__device__ __forceinline__ double wave_sum(double x)
{
    x = x + dpp_f64<kDppXor1>(x);
    x = x + dpp_f64<kDppXor2>(x);
    x = x + dpp_f64<kDppHalfMirror>(x);
    x = x + dpp_f64<kDppMirror>(x);
    return (readlane_f64(x, 0) + readlane_f64(x, 16)) + (readlane_f64(x, 32) + readlane_f64(x, 48));
}
// The sums of two values at once: after the first step even lanes go on with a and odd lanes with b,
// so that the other steps are taken once (rotations by 4 and 8 inside a row of 16 keep even and odd apart).
__device__ __forceinline__ void wave_sums(double &a, double &b)
{
    const bool odd = (threadIdx.x & 1u) != 0u;
    const double keep = odd ? b : a, give = odd ? a : b;
    double x = keep + dpp_f64<kDppXor1>(give);
    x = x + dpp_f64<kDppXor2>(x);
    x = x + dpp_f64<kDppRotate4>(x);
    x = x + dpp_f64<kDppRotate8>(x);
    a = (readlane_f64(x, 0) + readlane_f64(x, 16)) + (readlane_f64(x, 32) + readlane_f64(x, 48));
    b = (readlane_f64(x, 1) + readlane_f64(x, 17)) + (readlane_f64(x, 33) + readlane_f64(x, 49));
}
__device__ __forceinline__ unsigned wave_sum(unsigned x)
{
    x = x + dpp_u32<kDppXor1>(x);
    x = x + dpp_u32<kDppXor2>(x);
    x = x + dpp_u32<kDppHalfMirror>(x);
    x = x + dpp_u32<kDppMirror>(x);
    return static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(x), 0)) +
           static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(x), 16)) +
           static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(x), 32)) +
           static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(x), 48));
}

// the bucket that holds element e: the last one that starts at or before e
__device__ __forceinline__ int find_bucket(const long long *tbl, int nb, long long e)
{
    int lo = 0, hi = nb;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (tbl[2 * mid] <= e) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The bucket of a lane's 4 elements e .. e+3 inside the tile of 256 elements that begins at `first`
// (starts are multiples of 4, so they never straddle one), and where it ends.  Everything looked
// up is uniform over the wavefront: the table is read with scalar loads, which do not wait behind
// the streams; buckets that begin inside the tile are gone through one by one.
typedef const long long __attribute__((address_space(4))) KLong;
__device__ __forceinline__ int tile_bucket(const long long *table, int b_lo, int b_hi, long long first,
                                           long long e, long long &end)
{
    KLong *tbl = (KLong *)reinterpret_cast<unsigned long long>(table);
    int lo = b_lo, hi = b_hi;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (tbl[2 * mid] <= first) lo = mid;
        else hi = mid;
    }
    int b = lo;
    end = tbl[2 * lo + 1];
    for (int k = lo + 1; k < b_hi; ++k) {
        const long long k_start = tbl[2 * k], k_end = tbl[2 * k + 1];
        if (k_start >= first + 256) break;
        if (e >= k_start) {
            b = k;
            end = k_end;
        }
    }
    return b;
}
// how many of the lane's 4 elements lie inside the bucket (the rest is padding)
__device__ __forceinline__ int inside(long long e, long long end)
{
    const long long left = end - e;
    return left >= 4 ? 4 : left > 0 ? static_cast<int>(left) : 0;
}

__device__ __forceinline__ void stats_add(LaneStats &ls, float u, float w_old, bool has_w)
{
    // the square of an fp32 value is exact in fp64, so the fused form rounds exactly like a
    // product followed by a sum
    const double ud = static_cast<double>(u), wd = static_cast<double>(w_old);
    if (__builtin_isfinite(u)) ls.ssu = __builtin_fma(ud, ud, ls.ssu);
    else ls.nf += 1u;
    if (has_w && __builtin_isfinite(w_old)) ls.ssw = __builtin_fma(wd, wd, ls.ssw);
}

// The squares of a lane's 4 elements, the first n_valid of which lie inside their bucket; the others count as
// zeros.  Squares of finite fp32 values add up to finite fp64 sums and one that is not finite makes its sum so:
// where every lane's sums are finite nothing is looked at element by element (the same sums).
// With the two sums of a wavefront reduced together: norms_kernel on 25.6 M elements in 161 buckets 42.5 us
// before, 38.8 now.  (Sums taken twice where a tile has padding, once without a look and once element by element, made the
// layer-wise step on 16 M elements in buckets of 255 169.6 us; 167.3 with zeros in the place of padding.)
template <bool HAS_W>
__device__ __forceinline__ void stats_vector(LaneStats &ls, f32x4 u, f32x4 w_old, int n_valid)
{
    if (__builtin_amdgcn_ballot_w64(n_valid < 4) != 0ull) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            u[k] = n_valid > k ? u[k] : 0.0f;
            if (HAS_W) w_old[k] = n_valid > k ? w_old[k] : 0.0f;
        }
    }
    double su = ls.ssu, sw = ls.ssw;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double ud = static_cast<double>(u[k]);
        su = __builtin_fma(ud, ud, su);
        if (HAS_W) {
            const double wd = static_cast<double>(w_old[k]);
            sw = __builtin_fma(wd, wd, sw);
        }
    }
    const bool finite = __builtin_isfinite(su) && __builtin_isfinite(sw);
    if (__builtin_amdgcn_ballot_w64(!finite) == 0ull) {
        ls.ssu = su;
        ls.ssw = sw;
        return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) stats_add(ls, u[k], HAS_W ? w_old[k] : 0.0f, HAS_W);
}

// Called by every lane of a wavefront (all active).  The lanes that hold elements are a
// prefix of the wavefront and buckets ascend with the lane, so a mixed wavefront is the only
// one whose first lane lies in bucket b0 while a later lane does not: block b0 of the lane
// records is its own.
__device__ __forceinline__ void stats_commit(StatsRecord *records, StatsRecord *lane_records,
                                             const LaneStats &ls, long long wave_index,
                                             long long flag = 0)
{
    const int b0 = __builtin_amdgcn_readfirstlane(ls.bucket);
    const bool mixed = __builtin_amdgcn_ballot_w64(ls.bucket != b0) != 0ull;
    StatsRecord rec = {0.0, 0.0, b0 >= 0 ? b0 : -2, 0u, flag};
    if (mixed) {
        const StatsRecord mine = {ls.ssu, ls.ssw, ls.bucket, ls.nf, 0};
        lane_records[static_cast<long long>(b0) * 64 + (threadIdx.x & 63u)] = mine;
        rec.bucket = -1;
        rec.nf = static_cast<unsigned>(b0);
    } else if (b0 >= 0) {
        rec.ssu = ls.ssu;
        rec.ssw = ls.ssw;
        wave_sums(rec.ssu, rec.ssw);
        if (__builtin_amdgcn_ballot_w64(ls.nf != 0u) != 0ull) rec.nf = wave_sum(ls.nf);
    }
    if ((threadIdx.x & 63u) == 0u) records[wave_index] = rec;
}

// A kernel with arguments of the types that it declares: what is handed over is an array of addresses, from which
// the runtime copies as many bytes as the kernel takes.  (The runtime's own call: the configuration stack and the
// look at the last error behind a <<<>>> launch are 0.15 of 2.35 us, and a small round is bound by what it costs
// the host.)
template <typename... A>
hipError_t launch(void (*kernel)(A...), dim3 grid, dim3 block, unsigned lds, hipStream_t st, const A &...a)
{
    void *args[] = {const_cast<A *>(&a)...};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, args, lds, st);
    if (e != hipSuccess) (void)hipGetLastError();        // reported here, and nowhere again
    return e;
}

// LDS is not used by the kernels; a dynamic allocation only caps how many workgroups a CU
// holds at once.  A stream that mixes reads and writes is fastest on MI355X with about 26 KiB
// of loads in flight per CU; beyond it HBM throughput falls again.  (LDS is handed out in units,
// see eager_rules.h for the counts that this can realise.)
// Parameters and momentum above this size are streamed past the caches (see finish_tile).
constexpr long long kStateCacheBytes = 256ll << 20;

template <typename A>
hipError_t launch_capped(void (*kernel)(A), const A &a, int bpc, const Launch &cfg, dim3 grid,
                         hipStream_t st)
{
    unsigned lds = 0;
    if (bpc > 0) {
        lds = static_cast<unsigned>(kLdsPerCu / bpc / kLdsUnit * kLdsUnit);
        // Kernels of one signature share this function, so the flag is kept per kernel
        // address (a handful of entries; a context is not used from several threads, the
        // mutex covers several contexts).
        static std::mutex mu;
        static std::set<const void *> raised;
        const void *fn = reinterpret_cast<const void *>(kernel);
        std::lock_guard<std::mutex> lock(mu);
        if (!raised.count(fn)) {
            hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                               kLdsPerCu);
            if (e != hipSuccess) return e;
            raised.insert(fn);
        }
    }
    return launch(kernel, grid, dim3(cfg.block), lds, st, a);
}

inline unsigned grid_for(long long nvec, long long per_block, int max_blocks)
{
    long long g = (nvec + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (max_blocks > 0 && g > max_blocks) g = max_blocks;
    // the kernels stride, so a cap is safe; workgroups have at most 256 threads
    if (g > kMaxGridThreads / 256) g = kMaxGridThreads / 256;
    return static_cast<unsigned>(g);
}

}  // namespace
}  // namespace eager
