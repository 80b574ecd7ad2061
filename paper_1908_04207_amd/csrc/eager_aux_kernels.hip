// gfx950 kernels around the round: the finishing of the per-bucket statistics, the update
// rule alone on a receive buffer (plain, or with a layer-wise rate per bucket: norms pass, rate,
// update pass), and what processes that lag by more than one round need - a late gradient
// stashed into a send buffer, the update of several weight views from one read of the result, the
// model average (paper Section 5, last paragraph).  All of them are HBM streams: a lane owns 4 consecutive elements, 64-thread
// workgroups, nontemporal accesses, occupancy chosen for the bytes in flight.
#include "eager_device.h"

namespace eager {
namespace {

// The finishing kernels come with two workgroup sizes, see finish_threads.
//
// Adds the plain records (one per tile whose elements all lie in one bucket) with index in
// [lo, hi) that belong to bucket b: 8 independent loads per thread in flight, wavefront sums by
// DPP, the wavefronts of the workgroup through LDS.  The totals arrive in wavefront 0.  What
// bounds it is latency, so that the number of trips counts: the 832 threads that add records of 1024 take
// 6656 records in one, 256 threads 2048; of norms_kernel's groups of records half as many, each 8 tiles.
// Records of norms_kernel come in groups of kNormsTiles: the first of a group holds the sums of
// all, unless it is flagged - then every tile of the group has a record of its own.
// All of a record has been asked for before any of it is looked at: left alone the compiler moves the
// loads of the sums behind the branch on the bucket, a trip to memory after the other.
__device__ __forceinline__ void whole(StatsRecord &r)
{
    asm volatile("" : "+v"(r.ssu), "+v"(r.ssw), "+v"(r.bucket), "+v"(r.nf));
}

// The numbers among the arguments of the finishing kernels, asked for at once with the first pointers.
// (A pointer that went through a statement would be a flat one.)
__device__ __forceinline__ StatsArgs at_once(const StatsArgs &from)
{
    StatsArgs a = from;
    asm volatile("" : "+s"(a.e0), "+s"(a.n_records), "+s"(a.b_lo), "+s"(a.n_buckets), "+s"(a.tail_count),
                 "+s"(a.want_rate), "+s"(a.trust), "+s"(a.eps), "+s"(a.wd));
    return a;
}

template <int THREADS, bool GROUPED>
__device__ __forceinline__ void add_records(const StatsRecord *records, long long lo, long long hi,
                                            int b, double &su, double &sw, double &nf)
{
    constexpr int K = GROUPED ? 4 : 8, G = GROUPED ? kNormsTiles : 1;
    auto add = [&](const StatsRecord &r) {
        if (r.bucket == b) {
            su += r.ssu;
            sw += r.ssw;
            nf += r.nf;
        }
    };
    const long long g0 = lo / G, g1 = (hi + G - 1) / G;
    for (long long gb = g0 + threadIdx.x; gb < g1; gb += static_cast<long long>(THREADS) * K) {
        StatsRecord r[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const long long g = gb + static_cast<long long>(k) * THREADS;
            r[k].flag = 0;
            if (g < g1) r[k] = records[g * G];
            else r[k].bucket = -2;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (GROUPED && r[k].flag) {
                const long long t = (gb + static_cast<long long>(k) * THREADS) * G;
#pragma unroll
                for (int j = 0; j < G; ++j)
                    if (t + j >= lo && t + j < hi) add(records[t + j]);
            } else {
                add(r[k]);
            }
        }
    }
}

// (the count travels as a double: integers below 2^53 add exactly, and a 32-bit sum could
// overflow on a bucket of billions of elements)
template <int THREADS>
__device__ __forceinline__ void workgroup_sum(double &su, double &sw, double &nf)
{
    constexpr unsigned kWaves = THREADS / 64;
    __shared__ double part[3][kWaves];
    wave_sums(su, sw);
    if (__builtin_amdgcn_ballot_w64(nf != 0.0) != 0ull) nf = wave_sum(nf);
    const unsigned wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    if (lane == 0u) {
        part[0][wave] = su;
        part[1][wave] = sw;
        part[2][wave] = nf;
    }
    __syncthreads();
    if constexpr (kWaves == 4) {
        su = (part[0][0] + part[0][1]) + (part[0][2] + part[0][3]);
        sw = (part[1][0] + part[1][1]) + (part[1][2] + part[1][3]);
        nf = (part[2][0] + part[2][1]) + (part[2][2] + part[2][3]);
    } else if (wave == 0) {              // the totals are needed there
        const bool has = lane < kWaves;
        su = wave_sum(has ? part[0][lane] : 0.0);
        sw = wave_sum(has ? part[1][lane] : 0.0);
        nf = wave_sum(has ? part[2][lane] : 0.0);
    }
}

// A value that another workgroup reads or has written in the same launch.
__device__ __forceinline__ void put(double *p, double x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double get(const double *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// records of bucket b: [w0, w1)
__device__ __forceinline__ void bucket_records(const StatsArgs &a, int b, long long &w0, long long &w1)
{
    KLong *tbl = (KLong *)reinterpret_cast<unsigned long long>(a.table);
    const long long start = tbl[2 * b], end = tbl[2 * b + 1];
    w0 = (start - a.e0) / 256;
    w1 = (end - a.e0 + 255) / 256;
    if (w1 > a.n_records) w1 = a.n_records;
}

// fp64 square roots and division, one rounding to fp32 at the end
__device__ __forceinline__ float layer_rate(const StatsArgs &a, double su, double sw)
{
    const double nu = __builtin_sqrt(su), nw = __builtin_sqrt(sw);
    return nu > 0.0 && nw > 0.0
               ? static_cast<float>(static_cast<double>(a.trust) * nw /
                                    (nu + static_cast<double>(a.wd) * nw + static_cast<double>(a.eps)))
               : 1.0f;
}

// The sums of a bucket: the records of the wavefronts whose 256 elements touch the bucket (they are
// consecutive) - a uniform wavefront's sums, a mixed wavefront's lane records of this bucket - and the records of the
// ragged tail; one thread writes the bucket's totals.  One workgroup per bucket (blockIdx.x) and slice of its records
// (blockIdx.y, see launch_stats_finish).  Where there are several, each leaves a partial, and the last to arrive adds
// them, in the order of the slices: the totals do not depend on who that is.  Partials and count are written
// and read past the caches of an XCD (agent scope); a partial has arrived in memory before its workgroup counts itself.
template <bool GROUPED, int THREADS, bool SLICED>
__global__ __launch_bounds__(THREADS) void stats_finish_kernel(const StatsArgs args)
{
    const StatsArgs a = at_once(args);
    const int b = a.b_lo + static_cast<int>(blockIdx.x), slice = SLICED ? static_cast<int>(blockIdx.y) : 0;
    long long lo, hi, w0, w1;
    bucket_records(a, b, w0, w1);
    lo = w0;
    hi = w1;
    int slices = 1;
    if constexpr (SLICED) {               // (a run has at most 2^25 records)
        // slices begin at whole groups of records
        const long long head = w0 / kNormsTiles * kNormsTiles;
        const unsigned per = static_cast<unsigned>(a.per_slice), count = (static_cast<unsigned>(w1 - head) + per - 1u) / per;
        slices = static_cast<int>(count < 1u ? 1u : count < static_cast<unsigned>(a.slices) ? count : a.slices);
        if (slice >= slices) return;
        if (slice > 0) lo = head + static_cast<long long>(slice) * a.per_slice;
        if (slice + 1 < slices) hi = head + (slice + 1ll) * a.per_slice;
    }
    double su = 0.0, sw = 0.0, nf = 0.0;
    // Only the first and the last wavefront of the bucket can be mixed.  The lane records of the
    // first, those of the last and the ragged tail are read by a wavefront each (one lane per
    // record); in the larger workgroup these are wavefronts of their own, so that their dependent
    // loads run beside the others' and not after them.
    constexpr bool kApart = THREADS > 256;
    constexpr int kPlain = kApart ? THREADS - 3 * 64 : THREADS;
    const int wave = static_cast<int>(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int which = kApart ? wave - kPlain / 64 : wave;
    if (!kApart || which < 0) add_records<kPlain, GROUPED>(a.records, lo, hi, b, su, sw, nf);
    if (slice == 0 && (which == 0 || which == 1)) {
        const long long t = which == 0 ? w0 : w1 - 1;
        // Tile t has lane records where this bucket or the next begins inside it, or where the run ends there.
        // (Asked for without a look at that, those of buckets that have their tiles to themselves were 2 KiB a bucket
        // that nobody needs: 16 M elements in buckets of 255, round with norms 164 and 148 us, layer-wise step 169 and 156.)
        KLong *tbl = (KLong *)reinterpret_cast<unsigned long long>(a.table);
        const long long tile = a.e0 + t * 256, beyond = tbl[2 * b + (b + 1 < a.b_hi ? 2 : 1)];
        const bool before = tile < tbl[2 * b], behind = beyond < tile + 256;
        // (in a group that is not flagged only the first record has been written)
        if (w1 > w0 && (which == 0 || t != w0) && (before || behind)) {
            // A mixed wavefront's lane records stand in the block of its first lane's bucket: this one, or
            // nearly always the one before where the tile begins in front of this bucket.  They are asked
            // for beside the record that says so, not after it (with all of either: layer-wise steps of 0.6 to
            // 45 M elements, two finishing launches each, 0.5 to 1 us less).
            const int guess = before && b > 0 ? b - 1 : b;
            const long long flag = GROUPED ? a.records[t / kNormsTiles * kNormsTiles].flag : 1;
            StatsRecord r = a.records[t], lr = a.lane_records[static_cast<long long>(guess) * 64 + lane];
            whole(r);
            whole(lr);
            if (flag && r.bucket == -1) {
                if (static_cast<int>(r.nf) != guess) lr = a.lane_records[static_cast<long long>(r.nf) * 64 + lane];
                if (lr.bucket == b) {
                    su += lr.ssu;
                    sw += lr.ssw;
                    nf += lr.nf;
                }
            }
        }
    } else if (slice == 0 && which == 2 && lane < a.tail_count) {
        StatsRecord tr = a.lane_records[static_cast<long long>(a.n_buckets) * 64 + lane];
        whole(tr);
        if (tr.bucket == b) {
            su += tr.ssu;
            sw += tr.ssw;
            nf += tr.nf;
        }
    }
    workgroup_sum<THREADS>(su, sw, nf);
    if (SLICED && wave != 0) return;
    if (SLICED && slices > 1) {
        StatsRecord *part = a.partials + static_cast<long long>(b) * kStatsMaxSlices;
        unsigned before = 0u;
        if (lane == 0) {
            put(&part[slice].ssu, su);
            put(&part[slice].ssw, sw);
            put(reinterpret_cast<double *>(&part[slice].bucket), nf);     // (the count of a partial, in 64 bits)
            asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
            // (it begins again at zero by itself)
            before = __builtin_amdgcn_atomic_inc32(reinterpret_cast<unsigned *>(&part->flag), static_cast<unsigned>(slices) - 1u,
                                                   __ATOMIC_RELAXED, "agent");
        }
        if (__builtin_amdgcn_readfirstlane(static_cast<int>(before)) != slices - 1) return;
        asm volatile("" : : : "memory");
        const bool has = lane < slices;
        su = has ? get(&part[lane].ssu) : 0.0;
        sw = has ? get(&part[lane].ssw) : 0.0;
        nf = has ? get(reinterpret_cast<const double *>(&part[lane].bucket)) : 0.0;
        wave_sums(su, sw);
        if (__builtin_amdgcn_ballot_w64(nf != 0.0) != 0ull) nf = wave_sum(nf);
    }
    if (threadIdx.x == 0) {
        BucketStats out;
        out.sumsq_update = su;
        out.sumsq_params = sw;
        out.nonfinite = static_cast<unsigned long long>(nf);
        out.rate = a.want_rate ? layer_rate(a, su, sw) : 0.0f;
        out.reserved = 0u;
        a.stats[b] = out;
    }
}

// A late gradient outside a round (a process that lags by more than one round, last
// paragraph of Section 5): R <- G, or R <- R + G if the send buffer still holds an
// undelivered gradient.  A plain stream, a lane owns 4 elements.
// STRIDE: the grid does not cover the range and every lane loops.  Where it does cover it the
// body stands alone: a wavefront then ends right after its store instead of reaching a loop
// end first, and such short-lived wavefronts are measurably faster that way.
template <bool BF16, bool STRIDE>
__global__ __launch_bounds__(64) void stash_kernel(const StashArgs a)
{
    const long long nvec = a.n / 4;
    const char *src = static_cast<const char *>(a.g);
    auto body = [&](long long vi) {
        const long long e = a.e0 + vi * 4;
        f32x4 x;
        if (BF16) {
            const u32x2 g = __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(src + e * 2));
            x.x = __uint_as_float(g.x << 16);
            x.y = __uint_as_float(g.x & 0xffff0000u);
            x.z = __uint_as_float(g.y << 16);
            x.w = __uint_as_float(g.y & 0xffff0000u);
        } else {
            x = ld_f4<true>(reinterpret_cast<const float *>(src + e * 4));
        }
        if (a.accumulate) x = ld_f4<true>(a.r + e) + x;
        st_f4<true>(a.r + e, x);
    };
    const long long first = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
    if constexpr (STRIDE) {
        const long long stride = static_cast<long long>(gridDim.x) * blockDim.x;
        for (long long vi = first; vi < nvec; vi += stride) body(vi);
    } else {
        if (first < nvec) body(first);
    }
    const long long rem = a.n - nvec * 4;
    if (blockIdx.x == 0 && static_cast<long long>(threadIdx.x) < rem) {
        const long long i = a.e0 + nvec * 4 + threadIdx.x;
        const float g = load_grad_scalar<BF16>(src, i);
        a.r[i] = a.accumulate ? a.r[i] + g : g;
    }
}

// ---------------------------------------------------------------------------------------
// Weight views (one per process).  Both kernels: a lane owns 4 elements, the pointer table is
// read from the kernel-argument segment, views are taken in chunks whose loads are all issued
// before the first use, the last chunk has its exact size.
typedef const ViewsArgs __attribute__((address_space(4))) KViewsArgs;

// the update rule on C views from one value of u: 2C loads, then the arithmetic, then 2C stores
template <bool FAST, int C>
__device__ __forceinline__ void views_sgd_chunk(KViewsArgs &a, int p0, long long e, f32x4 u)
{
    f32x4 wo[C], vo[C];
#pragma unroll
    for (int j = 0; j < C; ++j) {
        vo[j] = ld_f4<true>(a.v[p0 + j] + e);
        wo[j] = ld_f4<true>(a.w[p0 + j] + e);
    }
    const UpdateRule rule = {a.neg_lr, a.mu, a.wd, a.nesterov};
    f32x4 vn[C], wn[C];
#pragma unroll
    for (int j = 0; j < C; ++j) update_rule<FAST>(rule, u, vo[j], wo[j], vn[j], wn[j]);
#pragma unroll
    for (int j = 0; j < C; ++j) {
        st_f4<true>(a.v[p0 + j] + e, vn[j]);
        st_f4<true>(a.w[p0 + j] + e, wn[j]);
    }
}
template <bool FAST, int R>
__device__ __forceinline__ void views_sgd_rest(KViewsArgs &a, int p0, int rem, long long e, f32x4 u)
{
    if constexpr (R >= 1) {
        if (rem == R) views_sgd_chunk<FAST, R>(a, p0, e, u);
        else views_sgd_rest<FAST, R - 1>(a, p0, rem, e, u);
    }
}

template <bool FAST>
__global__ __launch_bounds__(64) void views_sgd_kernel(const ViewsArgs)
{
    KViewsArgs &a = kernarg<ViewsArgs>();
    constexpr int CH = 8;
    const long long nvec = a.n / 4;
    const long long vi = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (vi < nvec) {
        const long long e = a.e0 + vi * 4;
        const f32x4 u = ld_f4<true>(a.u + e);
        const int V = a.n_views;
#pragma unroll
        for (int c = 0; c < kMaxP / CH; ++c)
            if ((c + 1) * CH <= V) views_sgd_chunk<FAST, CH>(a, c * CH, e, u);
        views_sgd_rest<FAST, CH - 1>(a, V / CH * CH, V % CH, e, u);
    }
    const long long rem = a.n - nvec * 4;
    if (blockIdx.x == 0 && static_cast<long long>(threadIdx.x) < rem) {
        const long long i = a.e0 + nvec * 4 + threadIdx.x;
        const UpdateRule rule = {a.neg_lr, a.mu, a.wd, a.nesterov};
        const float u = a.u[i];
        for (int p = 0; p < a.n_views; ++p) {
            float v = a.v[p][i], w = a.w[p][i];
            update_rule_scalar(rule, u, v, w);
            a.v[p][i] = v;
            a.w[p][i] = w;
        }
    }
}

// model synchronisation: every view <- (sum of the views in ascending order from +0.0f) * 1/V,
// the arithmetic of a round in which everybody is on time with an empty send buffer
template <int C>
__device__ __forceinline__ f32x4 views_sum_chunk(KViewsArgs &a, int p0, long long e, f32x4 s)
{
    f32x4 x[C];
#pragma unroll
    for (int j = 0; j < C; ++j) x[j] = ld_f4<true>(a.w[p0 + j] + e);
#pragma unroll
    for (int j = 0; j < C; ++j) s = s + x[j];
    return s;
}
template <int R>
__device__ __forceinline__ f32x4 views_sum_rest(KViewsArgs &a, int p0, int rem, long long e, f32x4 s)
{
    if constexpr (R >= 1) {
        if (rem == R) return views_sum_chunk<R>(a, p0, e, s);
        return views_sum_rest<R - 1>(a, p0, rem, e, s);
    }
    return s;
}

__global__ __launch_bounds__(64) void views_average_kernel(const ViewsArgs)
{
    KViewsArgs &a = kernarg<ViewsArgs>();
    constexpr int CH = 16;
    const long long nvec = a.n / 4;
    const long long vi = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
    const int V = a.n_views;
    if (vi < nvec) {
        const long long e = a.e0 + vi * 4;
        f32x4 s = (f32x4)(0.0f);
#pragma unroll
        for (int c = 0; c < kMaxP / CH; ++c)
            if ((c + 1) * CH <= V) s = views_sum_chunk<CH>(a, c * CH, e, s);
        s = views_sum_rest<CH - 1>(a, V / CH * CH, V % CH, e, s);
        const f32x4 mean = s * a.inv_views;
        for (int p = 0; p < V; ++p) st_f4<true>(a.w[p] + e, mean);
    }
    const long long rem = a.n - nvec * 4;
    if (blockIdx.x == 0 && static_cast<long long>(threadIdx.x) < rem) {
        const long long i = a.e0 + nvec * 4 + threadIdx.x;
        float s = 0.0f;
        for (int p = 0; p < V; ++p) s = s + a.w[p][i];
        const float mean = s * a.inv_views;
        for (int p = 0; p < V; ++p) a.w[p][i] = mean;
    }
}

// The two for up to 16 views, whose pointers every wavefront has in registers before it asks for the first of them: read where
// they are used, line after line of an argument block for 64, they are trips of their own, and the host copies the block with
// every launch.  Average and update, pointers as they come and this: 20 k elements, 8 views 3.0 3.5 and 2.6 3.3 us, 200 k 3.8 6.3
// and 3.7 5.3, 10 views 4.0 8.1 and 4.2 6.2; 25.6 M, 6 views 214 417 and 186 411 (which views are updated
// with the pointers as they come: launch_views_sgd).
// An access is a view's base with the tile's first element, uniform, and the lane's offset.  NT: the views are streamed.
template <bool NT>
__device__ __forceinline__ f32x4 ld_view(const float *view, long long first, unsigned off)
{
    return ld_at<NT>(reinterpret_cast<const char *>(view + first), off);
}
template <bool NT>
__device__ __forceinline__ void st_view(float *view, long long first, unsigned off, f32x4 x)
{
    st_at<NT>(reinterpret_cast<char *>(view + first), off, x);
}
template <int N, bool MOMENTUM>
__device__ __forceinline__ FewViewsArgs<N, MOMENTUM> read_views()
{
    FewViewsArgs<N, MOMENTUM> a;
    __builtin_memcpy(&a, (const void __attribute__((address_space(4))) *)&kernarg<FewViewsArgs<N, MOMENTUM>>(), sizeof a);
    asm volatile("" : "+s"(a.e0), "+s"(a.n), "+s"(a.n_views));
#pragma unroll
    for (int j = 0; j < N; ++j) asm volatile("" : "+s"(a.w[j]));
#pragma unroll
    for (int j = 0; MOMENTUM && j < N; ++j) asm volatile("" : "+s"(a.v[j]));
    return a;
}
template <bool FAST, bool NT, int N, int P0, int R>
__device__ __forceinline__ void few_sgd(const FewViewsArgs<N, true> &a, int rem, long long first, unsigned off, f32x4 u)
{
    if constexpr (R >= 1) {
        if (rem != R) {
            few_sgd<FAST, NT, N, P0, R - 1>(a, rem, first, off, u);
            return;
        }
        f32x4 wo[R], vo[R], vn[R], wn[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            vo[j] = ld_view<NT>(a.v[P0 + j], first, off);
            wo[j] = ld_view<NT>(a.w[P0 + j], first, off);
        }
        const UpdateRule rule = {a.neg_lr, a.mu, a.wd, a.nesterov};
#pragma unroll
        for (int j = 0; j < R; ++j) update_rule<FAST>(rule, u, vo[j], wo[j], vn[j], wn[j]);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            st_view<NT>(a.v[P0 + j], first, off, vn[j]);
            st_view<NT>(a.w[P0 + j], first, off, wn[j]);
        }
    }
}
template <bool FAST, bool NT, int N>
__global__ __launch_bounds__(64) void few_views_sgd_kernel(const FewViewsArgs<N, true>)
{
    const FewViewsArgs<N, true> a = read_views<N, true>();
    const long long nvec = a.n / 4;
    const long long vi = static_cast<long long>(blockIdx.x) * 64 + threadIdx.x;
    if (vi < nvec) {
        const long long first = a.e0 + static_cast<long long>(blockIdx.x) * 256;
        const unsigned off = threadIdx.x * 16u;
        const f32x4 u = ld_view<NT>(a.u, first, off);
        if constexpr (N == 16) {
            few_sgd<FAST, NT, N, 0, 8>(a, 8, first, off, u);
            few_sgd<FAST, NT, N, 8, 8>(a, a.n_views - 8, first, off, u);
        } else {
            few_sgd<FAST, NT, N, 0, N>(a, a.n_views, first, off, u);
        }
    }
    const long long rem = a.n - nvec * 4;
    if (blockIdx.x == 0 && static_cast<long long>(threadIdx.x) < rem) {
        const long long i = a.e0 + nvec * 4 + threadIdx.x;
        const UpdateRule rule = {a.neg_lr, a.mu, a.wd, a.nesterov};
        const float u = a.u[i];
        const FewViewsArgs<N, true> __attribute__((address_space(4))) &k = kernarg<FewViewsArgs<N, true>>();
        for (int p = 0; p < a.n_views; ++p) {
            float v = k.v[p][i], w = k.w[p][i];
            update_rule_scalar(rule, u, v, w);
            k.v[p][i] = v;
            k.w[p][i] = w;
        }
    }
}
template <bool NT, int N, int R>
__device__ __forceinline__ void few_average(const FewViewsArgs<N, false> &a, int views, float inv, long long first, unsigned off)
{
    if constexpr (R >= 1) {
        if (views != R) {
            few_average<NT, N, R - 1>(a, views, inv, first, off);
            return;
        }
        f32x4 x[R], s = (f32x4)(0.0f);
#pragma unroll
        for (int j = 0; j < R; ++j) x[j] = ld_view<NT>(a.w[j], first, off);
#pragma unroll
        for (int j = 0; j < R; ++j) s = s + x[j];
        const f32x4 mean = s * inv;
#pragma unroll
        for (int j = 0; j < R; ++j) st_view<NT>(a.w[j], first, off, mean);
    }
}
template <bool NT, int N>
__global__ __launch_bounds__(64) void few_views_average_kernel(const FewViewsArgs<N, false>)
{
    const FewViewsArgs<N, false> a = read_views<N, false>();
    const long long nvec = a.n / 4;
    const long long vi = static_cast<long long>(blockIdx.x) * 64 + threadIdx.x;
    if (vi < nvec)
        few_average<NT, N, N>(a, a.n_views, a.inv_views, a.e0 + static_cast<long long>(blockIdx.x) * 256, threadIdx.x * 16u);
    const long long rem = a.n - nvec * 4;
    if (blockIdx.x == 0 && static_cast<long long>(threadIdx.x) < rem) {
        const long long i = a.e0 + nvec * 4 + threadIdx.x;
        const FewViewsArgs<N, false> __attribute__((address_space(4))) &k = kernarg<FewViewsArgs<N, false>>();
        float s = 0.0f;
        for (int p = 0; p < k.n_views; ++p) s = s + k.w[p][i];
        const float mean = s * k.inv_views;
        for (int p = 0; p < k.n_views; ++p) k.w[p][i] = mean;
    }
}

// NT: w and v are too large to stay in the last-level cache until they are touched again
// STRIDE: as in stash_kernel
template <bool FAST, bool NT, bool STRIDE>
__global__ __launch_bounds__(256) void sgd_kernel(const SgdArgs a)
{
    const long long nvec = a.n / 4;
    auto body = [&](long long vi) {
        const long long i = a.e0 + vi * 4;
        const f32x4 u = ld_f4<true>(a.u + i);
        const f32x4 vo = ld_f4<NT>(a.v + i);
        const f32x4 wo = ld_f4<NT>(a.w + i);
        f32x4 vn, wn;
        const UpdateRule rule = {a.neg_lr, a.mu, a.wd, a.nesterov};
        update_rule<FAST>(rule, u, vo, wo, vn, wn);
        st_f4<NT>(a.v + i, vn);
        st_f4<NT>(a.w + i, wn);
    };
    const long long first = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
    if constexpr (STRIDE) {
        const long long stride = static_cast<long long>(gridDim.x) * blockDim.x;
        for (long long vi = first; vi < nvec; vi += stride) body(vi);
    } else {
        if (first < nvec) body(first);
    }
    const long long rem = a.n - nvec * 4;
    if (blockIdx.x == 0 && static_cast<long long>(threadIdx.x) < rem) {
        const long long i = a.e0 + nvec * 4 + threadIdx.x;
        const UpdateRule rule = {a.neg_lr, a.mu, a.wd, a.nesterov};
        float v = a.v[i], w = a.w[i];
        update_rule_scalar(rule, a.u[i], v, w);
        a.v[i] = v;
        a.w[i] = w;
    }
}

// ---- update rule with a rate per bucket (layer-wise adaptive rate scaling) ------------------
// Two passes, because the norms of a bucket must be complete before its first element moves (or one, where a
// workgroup holds its bucket: lars_bucket_kernel):
// norms_kernel leaves the same per-wavefront records as a round with statistics (finished by
// stats_finish_kernel, which also forms the rate), lars_kernel applies
//     g = rate_b * (u + wd*w);  v' = mu*v + g;  step = nesterov ? g + mu*v' : v';  w' = w - lr*step
// One lane-vector per lane in both, so that record k belongs to elements [256k, 256k + 256).

// A wavefront takes one tile of 256 elements and leaves its record, or a record per lane where several
// buckets share it.  What bounds it are the reads of u and w, which stay in the last-level cache for
// the update right after where they fit (25.6 M elements, 161 buckets: norms, finish and update 114
// us, 119 in groups, 124 with four tiles per wavefront).
// GROUPED: K consecutive tiles, for large models of large buckets (see norms_grouped).  Where they
// all lie inside one bucket the wavefront requests u and w of one tile after the other, squares and
// sums in its lanes, and combines the lanes once at the end: one record instead of K, and K times
// fewer cross-lane steps in fp64.  Other groups leave a record per tile or per lane, tile after tile.
template <bool GROUPED>
__global__ __launch_bounds__(64) void norms_kernel(const SgdArgs a, const StatsArgs st)
{
    constexpr int K = kNormsTiles, T = GROUPED ? K : 1;      // tiles of the wavefront
    constexpr bool NT = GROUPED;
    KLong *tbl = (KLong *)reinterpret_cast<unsigned long long>(st.table);
    const long long nvec = a.n / 4;
    const long long tile0 = static_cast<long long>(blockIdx.x) * T;
    const unsigned lane = threadIdx.x & 63u;
    bool whole = false;
    if constexpr (GROUPED) {
        const long long first = a.e0 + tile0 * 256, last = first + K * 256;
        const f32x4 *up = reinterpret_cast<const f32x4 *>(a.u + first) + lane;
        const f32x4 *wp = reinterpret_cast<const f32x4 *>(a.w + first) + lane;
        whole = (tile0 + K) * 64 <= nvec;
        f32x4 u, w;
        if (whole) {
            u = ld_f4<NT>(reinterpret_cast<const float *>(up));
            w = ld_f4<NT>(reinterpret_cast<const float *>(wp));
        }
        int bucket = st.b_lo;
        for (int hi = st.b_hi; hi - bucket > 1;) {
            const int mid = (bucket + hi) >> 1;
            if (tbl[2 * mid] <= first) bucket = mid;
            else hi = mid;
        }
        whole = whole && tbl[2 * bucket + 1] >= last;
        if (whole) {
            LaneStats ls = {0.0, 0.0, 0u, bucket};
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const f32x4 x = u, y = w;
                if (k + 1 < K) {
                    u = ld_f4<NT>(reinterpret_cast<const float *>(up + (k + 1) * 64));
                    w = ld_f4<NT>(reinterpret_cast<const float *>(wp + (k + 1) * 64));
                }
                stats_vector<true>(ls, x, y, 4);
            }
            double su = ls.ssu, sw = ls.ssw;
            wave_sums(su, sw);
            unsigned nf = 0u;
            if (__builtin_amdgcn_ballot_w64(ls.nf != 0u) != 0ull) nf = wave_sum(ls.nf);
            if (lane == 0u) {
                const StatsRecord rec = {su, sw, bucket, nf, 0};
                st.records[tile0] = rec;
            }
        }
    }
    for (int k = 0; k < T && !whole; ++k) {
        const long long vi = (tile0 + k) * 64 + lane;
        LaneStats ls = {0.0, 0.0, 0u, -1};
        if (vi < nvec) {
            const long long e = a.e0 + vi * 4;
            const f32x4 u = ld_f4<NT>(a.u + e), w = ld_f4<NT>(a.w + e);
            long long end;
            ls.bucket = tile_bucket(st.table, st.b_lo, st.b_hi, a.e0 + (tile0 + k) * 256, e, end);
            stats_vector<true>(ls, u, w, inside(e, end));
        }
        stats_commit(st.records, st.lane_records, ls, tile0 + k, (tile0 + k) % K == 0 ? 1 : 0);
    }
    const long long rem = a.n - nvec * 4;
    if (blockIdx.x == 0 && static_cast<long long>(threadIdx.x) < rem) {
        const long long i = a.e0 + nvec * 4 + threadIdx.x;
        LaneStats t = {0.0, 0.0, 0u, find_bucket(st.table, st.n_buckets, i)};
        if (i < st.table[2 * t.bucket + 1]) stats_add(t, a.u[i], a.w[i], true);
        else t.bucket = -2;
        const StatsRecord mine = {t.ssu, t.ssw, t.bucket, t.nf, 0};
        st.lane_records[static_cast<long long>(st.n_buckets) * 64 + threadIdx.x] = mine;
    }
}

template <bool FAST>
__device__ __forceinline__ f32x4 scaled_gradient(float rate, float wd, f32x4 u, f32x4 w)
{
    if (FAST) {
#pragma clang fp contract(fast)
        f32x4 g = u;
        if (wd != 0.0f) g = wd * w + u;
        return rate * g;
    }
    f32x4 g = u;
    if (wd != 0.0f) g = fma4(wd, w, u);
    return rate * g;
}

// NT: w, v and their new values are streamed.  The old w and u have just been read by norms_kernel
// and are in the last-level cache where they fit; writing w and v past it leaves nothing there
// that the next kernels would have to write back first.
template <bool FAST, bool NT>
__global__ __launch_bounds__(64) void lars_kernel(const SgdArgs a, const StatsArgs st)
{
    KLong *tbl = (KLong *)reinterpret_cast<unsigned long long>(st.table);
    const long long nvec = a.n / 4;
    const long long vi = static_cast<long long>(blockIdx.x) * 64 + threadIdx.x;
    const long long first = a.e0 + static_cast<long long>(blockIdx.x) * 256;
    // the decay is part of the scaled gradient, so the plain rule follows with wd = 0
    const UpdateRule rule = {a.neg_lr, a.mu, 0.0f, a.nesterov};
    if (vi < nvec) {
        const long long e = a.e0 + vi * 4;
        const f32x4 u = ld_f4<true>(a.u + e);
        const f32x4 vo = ld_f4<NT>(a.v + e);
        const f32x4 wo = ld_f4<NT>(a.w + e);
        // bucket of the wavefront's first element and the rates of it and of those that begin
        // inside the tile: uniform, scalar loads beside the streams
        int b = st.b_lo;
        for (int hi = st.b_hi; hi - b > 1;) {
            const int mid = (b + hi) >> 1;
            if (tbl[2 * mid] <= first) b = mid;
            else hi = mid;
        }
        typedef const float __attribute__((address_space(4))) KFloat;
        KFloat *rates = (KFloat *)reinterpret_cast<unsigned long long>(&st.stats[0].rate);
        constexpr int kStep = sizeof(BucketStats) / sizeof(float);
        float rate = rates[static_cast<long long>(b) * kStep];
        for (++b; b < st.b_hi; ++b) {
            const long long start = tbl[2 * b];
            const float r = rates[static_cast<long long>(b) * kStep];
            if (start >= first + 256) break;
            if (e >= start) rate = r;
        }
        f32x4 vn, wn;
        update_rule<FAST>(rule, scaled_gradient<FAST>(rate, a.wd, u, wo), vo, wo, vn, wn);
        st_f4<NT>(a.v + e, vn);
        st_f4<NT>(a.w + e, wn);
    }
    const long long rem = a.n - nvec * 4;
    if (blockIdx.x == 0 && static_cast<long long>(threadIdx.x) < rem) {
        const long long i = a.e0 + nvec * 4 + threadIdx.x;
        const float rate = st.stats[find_bucket(st.table, st.n_buckets, i)].rate;
        float v = a.v[i], w = a.w[i];
        float g = a.u[i];
        if (a.wd != 0.0f) g = fma1(a.wd, w, g);
        update_rule_scalar(rule, rate * g, v, w);
        a.v[i] = v;
        a.w[i] = w;
    }
}

// The layer-wise rule where every bucket is small: a workgroup per bucket, V lane-vectors to a lane, which wait in
// registers while the workgroup adds their squares and forms the rate.  What bounds it is latency: a launch, the table,
// one trip to u, w and v, the sums, the rate's divisions.
template <bool FAST, bool NT, int THREADS, int V>
__global__ __launch_bounds__(THREADS) void lars_bucket_kernel(const SgdArgs a, const StatsArgs st)
{
    KLong *tbl = (KLong *)reinterpret_cast<unsigned long long>(st.table);
    const int b = st.b_lo + static_cast<int>(blockIdx.x);
    const long long start = tbl[2 * b], end = tbl[2 * b + 1], stop = tbl[2 * b + (b + 1 < st.b_hi ? 2 : 1)];
    const int n = static_cast<int>(end - start), nvec = n / 4, lane = static_cast<int>(threadIdx.x);
    const float *up = a.u + start;
    float *wp = a.w + start, *vp = a.v + start;
    f32x4 u[V], w[V], v[V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
        u[k] = w[k] = v[k] = (f32x4)(0.0f);
        const int vi = k * THREADS + lane;
        if (vi < nvec) {
            u[k] = ld_f4<NT>(up + vi * 4);
            w[k] = ld_f4<NT>(wp + vi * 4);
            v[k] = ld_f4<NT>(vp + vi * 4);
        }
    }
    // up to 3 elements behind the last lane-vector, one to a lane, and the padding up to the run's next bucket
    // (kBucketEnd elements at most)
    const int last = nvec * 4 + lane, behind = static_cast<int>(stop - start);
    float ue = 0.0f, we = 0.0f, ve = 0.0f;
    if (last < behind) {
        ue = up[last];
        we = wp[last];
        ve = vp[last];
    }
    LaneStats ls = {0.0, 0.0, 0u, b};
#pragma unroll
    for (int k = 0; k < V; ++k) stats_vector<true>(ls, u[k], w[k], 4);
    if (last < n) stats_add(ls, ue, we, true);
    double su = ls.ssu, sw = ls.ssw, nf = ls.nf;
    __shared__ float shared_rate;
    workgroup_sum<THREADS>(su, sw, nf);
    if (threadIdx.x < 64u) {
        const float rate = layer_rate(st, su, sw);
        if (threadIdx.x == 0u) {
            const BucketStats out = {su, sw, static_cast<unsigned long long>(nf), rate, 0u};
            st.stats[b] = out;
            shared_rate = rate;
        }
    }
    __syncthreads();
    const float rate = shared_rate;
    // the decay is part of the scaled gradient, so the plain rule follows with wd = 0
    const UpdateRule rule = {a.neg_lr, a.mu, 0.0f, a.nesterov};
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int vi = k * THREADS + lane;
        if (vi < nvec) {
            f32x4 vn, wn;
            update_rule<FAST>(rule, scaled_gradient<FAST>(rate, a.wd, u[k], w[k]), v[k], w[k], vn, wn);
            st_f4<NT>(vp + vi * 4, vn);
            st_f4<NT>(wp + vi * 4, wn);
        }
    }
    if (last < behind) {
        float g = ue;
        if (a.wd != 0.0f) g = fma1(a.wd, we, g);
        update_rule_scalar(rule, rate * g, ve, we);
        vp[last] = ve;
        wp[last] = we;
    }
}

}  // namespace

hipError_t launch_stats_finish(const StatsArgs &a, hipStream_t stream)
{
    const int n = a.b_hi - a.b_lo;
    if (n <= 0 || a.want_rate == kRateByBucket) return hipSuccess;
    if (a.slices > kStatsMaxSlices || a.slices < 1) return hipErrorInvalidValue;
    const bool grouped = a.want_rate && norms_grouped(a.n_records, n), wide = finish_threads(n) == 1024;
    const dim3 grid(static_cast<unsigned>(n), static_cast<unsigned>(a.slices)), threads(wide ? 1024 : 256);
    switch ((a.slices > 1 ? 4 : 0) | (grouped ? 2 : 0) | (wide ? 1 : 0)) {
    case 0: return launch(stats_finish_kernel<false, 256, false>, grid, threads, 0, stream, a);
    case 1: return launch(stats_finish_kernel<false, 1024, false>, grid, threads, 0, stream, a);
    case 2: return launch(stats_finish_kernel<true, 256, false>, grid, threads, 0, stream, a);
    case 3: return launch(stats_finish_kernel<true, 1024, false>, grid, threads, 0, stream, a);
    case 4: return launch(stats_finish_kernel<false, 256, true>, grid, threads, 0, stream, a);
    case 5: return launch(stats_finish_kernel<false, 1024, true>, grid, threads, 0, stream, a);
    case 6: return launch(stats_finish_kernel<true, 256, true>, grid, threads, 0, stream, a);
    default: return launch(stats_finish_kernel<true, 1024, true>, grid, threads, 0, stream, a);
    }
}

hipError_t launch_stash(const StashArgs &a, bool bf16, hipStream_t stream)
{
    if (a.n <= 0) return hipSuccess;
    long long g = (a.n / 4 + 63) / 64;
    if (g < 1) g = 1;
    const bool stride = g > kMaxGridThreads / 64;
    if (stride) g = kMaxGridThreads / 64;
    const dim3 grid(static_cast<unsigned>(g)), block(64);
    if (bf16)
        return stride ? launch(stash_kernel<true, true>, grid, block, 0, stream, a)
                      : launch(stash_kernel<true, false>, grid, block, 0, stream, a);
    return stride ? launch(stash_kernel<false, true>, grid, block, 0, stream, a)
                  : launch(stash_kernel<false, false>, grid, block, 0, stream, a);
}

namespace {
template <typename A>
hipError_t launch_views(void (*kernel)(A), const A &a, const Launch &cfg, int auto_waves, hipStream_t stream)
{
    const long long g = views_tiles(a.n);
    if (g * 64 > kMaxGridThreads) return hipErrorInvalidValue;    // these kernels do not stride
    Launch l = cfg;
    l.block = 64;
    const int bpc = cfg.blocks_per_cu == 0 ? auto_waves : cfg.blocks_per_cu;
    return launch_capped(kernel, a, bpc, l, static_cast<unsigned>(g), stream);
}
template <int N, bool MOMENTUM>
FewViewsArgs<N, MOMENTUM> few_views(const ViewsArgs &a)
{
    FewViewsArgs<N, MOMENTUM> few;
    few.u = a.u;
    few.e0 = a.e0;
    few.n = a.n;
    few.neg_lr = a.neg_lr;
    few.mu = a.mu;
    few.wd = a.wd;
    few.inv_views = a.inv_views;
    few.nesterov = a.nesterov;
    few.n_views = a.n_views;
    for (int p = 0; p < a.n_views; ++p) few.w[p] = a.w[p];
    for (int p = 0; MOMENTUM && p < a.n_views; ++p) few.v[p] = a.v[p];
    return few;
}
template <bool FAST, int N>
hipError_t launch_few_sgd(const ViewsArgs &a, bool nt, const Launch &cfg, int waves, hipStream_t stream)
{
    return nt ? launch_views(few_views_sgd_kernel<FAST, true, N>, few_views<N, true>(a), cfg, waves, stream)
              : launch_views(few_views_sgd_kernel<FAST, false, N>, few_views<N, true>(a), cfg, waves, stream);
}
template <int N>
hipError_t launch_few_average(const ViewsArgs &a, bool nt, const Launch &cfg, int waves, hipStream_t stream)
{
    return nt ? launch_views(few_views_average_kernel<true, N>, few_views<N, false>(a), cfg, waves, stream)
              : launch_views(few_views_average_kernel<false, N>, few_views<N, false>(a), cfg, waves, stream);
}
}  // namespace

hipError_t launch_views_sgd(const ViewsArgs &a, bool fast, const Launch &cfg, hipStream_t stream)
{
    if (a.n <= 0 || a.n_views <= 0) return hipSuccess;
    const int waves = views_sgd_waves(a.n_views, a.n);
    const bool nt = a.n * (4 + 16ll * a.n_views) > kPlainRoundBytes;
    if (a.n_views <= 4)
        return fast ? launch_few_sgd<true, 4>(a, nt, cfg, waves, stream) : launch_few_sgd<false, 4>(a, nt, cfg, waves, stream);
    // (streamed, 7, 8 and 16 views are faster with the pointers read as they come: 25.6 M elements 471 541 1104 us, with all at once
    // 479 562 1123; 6, 9 and 12 views 413 620 844 and 408 616 830)
    if (a.n_views <= (nt ? 6 : 8))
        return fast ? launch_few_sgd<true, 8>(a, nt, cfg, waves, stream) : launch_few_sgd<false, 8>(a, nt, cfg, waves, stream);
    if (a.n_views > 8 && a.n_views <= (nt ? 12 : 16))
        return fast ? launch_few_sgd<true, 16>(a, nt, cfg, waves, stream) : launch_few_sgd<false, 16>(a, nt, cfg, waves, stream);
    return fast ? launch_views(views_sgd_kernel<true>, a, cfg, waves, stream)
                : launch_views(views_sgd_kernel<false>, a, cfg, waves, stream);
}

hipError_t launch_views_average(const ViewsArgs &a, const Launch &cfg, hipStream_t stream)
{
    if (a.n <= 0 || a.n_views <= 0) return hipSuccess;
    const int waves = views_average_waves(a.n_views, a.n);
    const bool nt = views_average_streamed(a.n_views, a.n);
    if (a.n_views <= 4) return launch_few_average<4>(a, nt, cfg, waves, stream);
    if (a.n_views <= 8) return launch_few_average<8>(a, nt, cfg, waves, stream);
    if (a.n_views <= 16) return launch_few_average<16>(a, nt, cfg, waves, stream);
    return launch_views(views_average_kernel, a, cfg, waves, stream);
}

hipError_t launch_sgd(const SgdArgs &a, bool fast, const Launch &cfg, hipStream_t stream)
{
    if (a.n <= 0) return hipSuccess;
    // 64-thread workgroups, one lane-vector per lane unless the grid is capped (measured on
    // 355 M elements: 1.12 ms against 1.22 ms with 256-thread workgroups and cached state)
    const long long nvec = a.n / 4;
    const dim3 grid(grid_for(nvec, 64, 0)), block(64);
    const bool stride = static_cast<long long>(grid.x) * 64 < nvec;
    const bool nt = a.n * 8 > kStateCacheBytes;
    switch ((fast ? 4 : 0) | (nt ? 2 : 0) | (stride ? 1 : 0)) {
    case 0: return launch(sgd_kernel<false, false, false>, grid, block, 0, stream, a);
    case 1: return launch(sgd_kernel<false, false, true>, grid, block, 0, stream, a);
    case 2: return launch(sgd_kernel<false, true, false>, grid, block, 0, stream, a);
    case 3: return launch(sgd_kernel<false, true, true>, grid, block, 0, stream, a);
    case 4: return launch(sgd_kernel<true, false, false>, grid, block, 0, stream, a);
    case 5: return launch(sgd_kernel<true, false, true>, grid, block, 0, stream, a);
    case 6: return launch(sgd_kernel<true, true, false>, grid, block, 0, stream, a);
    default: return launch(sgd_kernel<true, true, true>, grid, block, 0, stream, a);
    }
}

// tiles of 256 elements that the norms kernel leaves a record for
long long norms_records(long long n)
{
    long long g = (n / 4 + 64 * kNormsTiles - 1) / (64 * kNormsTiles);
    return (g < 1 ? 1 : g) * kNormsTiles;
}

hipError_t launch_norms(const SgdArgs &a, const StatsArgs &st, hipStream_t stream)
{
    if (a.n <= 0 || st.want_rate == kRateByBucket) return hipSuccess;
    const long long tiles = norms_records(a.n);
    const bool grouped = norms_grouped(tiles, st.b_hi - st.b_lo);
    const long long g = grouped ? tiles / kNormsTiles : tiles;
    if (g * 64 > kMaxGridThreads) return hipErrorInvalidValue;    // the kernel does not stride
    const dim3 grid(static_cast<unsigned>(g)), block(64);
    // (the grouped form is for runs whose u and w do not fit the last-level cache; elsewhere they are
    // left there for the update right after)
    return grouped ? launch(norms_kernel<true>, grid, block, 0, stream, a, st)
                   : launch(norms_kernel<false>, grid, block, 0, stream, a, st);
}

namespace {
template <int THREADS, int V>
hipError_t launch_by_bucket(const SgdArgs &a, const StatsArgs &st, bool fast, bool nt, hipStream_t stream)
{
    const dim3 grid(static_cast<unsigned>(st.b_hi - st.b_lo)), block(THREADS);
    if (fast)
        return nt ? launch(lars_bucket_kernel<true, true, THREADS, V>, grid, block, 0, stream, a, st)
                  : launch(lars_bucket_kernel<true, false, THREADS, V>, grid, block, 0, stream, a, st);
    return nt ? launch(lars_bucket_kernel<false, true, THREADS, V>, grid, block, 0, stream, a, st)
              : launch(lars_bucket_kernel<false, false, THREADS, V>, grid, block, 0, stream, a, st);
}
}  // namespace

hipError_t launch_sgd_lars(const SgdArgs &a, const StatsArgs &st, bool fast, hipStream_t stream)
{
    if (st.want_rate == kRateByBucket) {
        const bool nt = a.n * 20 > kPlainRoundBytes;
        if (st.n_records <= 1024) return launch_by_bucket<256, 1>(a, st, fast, nt, stream);
        if (st.n_records <= 4096) return launch_by_bucket<256, 4>(a, st, fast, nt, stream);
        return launch_by_bucket<1024, 4>(a, st, fast, nt, stream);
    }
    if (a.n <= 0) return hipSuccess;
    long long g = (a.n / 4 + 63) / 64;                            // one lane-vector per lane
    if (g < 1) g = 1;
    if (g * 64 > kMaxGridThreads) return hipErrorInvalidValue;
    // w and v are streamed unless u, w and v stay in the last-level cache until the next step
    // (norms, rate and update on 10 M elements: 98 us streamed, 99 not; 4 M: 55.9 and 54.0; 25.6 M after
    // a round: 117 and 136)
    const bool nt = a.n * 12 > 96ll << 20;
    const dim3 grid(static_cast<unsigned>(g)), block(64);
    if (fast)
        return nt ? launch(lars_kernel<true, true>, grid, block, 0, stream, a, st)
                  : launch(lars_kernel<true, false>, grid, block, 0, stream, a, st);
    return nt ? launch(lars_kernel<false, true>, grid, block, 0, stream, a, st)
              : launch(lars_kernel<false, false>, grid, block, 0, stream, a, st);
}

}  // namespace eager
