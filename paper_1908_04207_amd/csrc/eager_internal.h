// Internal interface between the host side of the library (argument checking, context
// state, run building) and the gfx950 kernels.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace eager {

constexpr int kMaxP = 64;

// Lane-vectors (groups of 4 elements) of a run that the vector path of a round covers.  With bf16
// gradients two lanes share one 16-byte piece, so the vector path ends at a multiple of 8
// elements and never reads beyond the run.
template <bool BF16>
__host__ __device__ inline long long slot_nvec(long long n)
{
    return BF16 ? (n / 8) * 2 : n / 4;
}

// Optional by-products of a round, per bucket (same layout as eager_bucket_stats of the public
// header): squared norm of the averaged update and of the parameters before the update (finite
// elements only), number of non-finite elements of the update.
struct BucketStats {
    double sumsq_update;
    double sumsq_params;
    unsigned long long nonfinite;
    float rate;
    unsigned reserved;
};

// What one wavefront of the round kernel leaves for the finishing kernel: the sums over its
// 256 elements if they all lie in one bucket (bucket >= 0); bucket = -1 if they lie in several
// (then every lane has left a record of its own in block `nf` of the lane records); bucket =
// -2 if the wavefront holds no element.  Lane records and the records of the ragged tail
// (at most 7 single elements, in the block after the last bucket's) have the same layout.
struct StatsRecord {
    double ssu, ssw;
    int bucket;
    unsigned nf;
    long long flag;              // norms_kernel: the tiles of the group have records of their own
};

struct StatsArgs {
    const long long *table;      // device: start, end of every bucket (2 per bucket)
    BucketStats *stats;          // device: one per bucket
    StatsRecord *records;        // device: one per wavefront of the round kernel
    StatsRecord *lane_records;   // device: (n_buckets + 1) blocks of 64
    int tail_count;              // elements of the run's ragged tail (0..7)
    int per_slice;               // (here it needs no room of its own: 8 bytes more are 0.2 us a launch)
    long long e0;                // first element of the run
    long long n_records;         // wavefronts the round kernel was launched with; with kRateByBucket the
                                 // elements of the largest bucket
    int b_lo, b_hi;              // buckets of the run
    int n_buckets;
    // layer-wise rate, written next to the totals when want_rate is set:
    // trust * |w| / (|u| + wd * |w| + eps), or 1 where a norm is zero
    int want_rate;               // kRateByBucket: by the update kernel itself, which takes a bucket per workgroup
    float trust, wd, eps;
    // A bucket with many records is added up by several workgroups, at most `slices`, of `per_slice` records each, worked out
    // from the records of the largest bucket (finish_slices): one
    // partial each (partials[bucket * kStatsMaxSlices + slice]), and the last of them to arrive adds these.  The bucket's
    // first partial counts the arrivals in its `flag`, zero between launches.
    StatsRecord *partials;
    int slices;
    int largest;                 // records of the run's largest bucket
};
constexpr int kRate = 1, kRateByBucket = 2;
constexpr int kStatsMaxSlices = 64;
// The workspace: bucket table (16 bytes each), a record for each of `stats_tiles` tiles, (n_buckets + 1) blocks of 64 lane
// records, kStatsMaxSlices partials per bucket, the first of which counts arrivals.
inline long long stats_tiles(long long first, long long end) { return (end - first) / 256 + 8; }
constexpr long long kStatsRecordsPerSlice = 4096;

// Capacity of the entry point that allocates nothing: its statistics workspace is a fixed
// device array inside the library (bucket table, one record per 256 elements, lane records,
// partials - the layout of the caller-provided workspace, see stats_tiles), so the context may hold at most this
// many buckets and span at most this many elements.
constexpr int kStaticMaxBuckets = 512;
constexpr long long kStaticMaxElements = 1ll << 27;
constexpr long long kStaticMaxRecords = kStaticMaxElements / 256 + 8;
constexpr long long kStaticScratchBytes =
    kStaticMaxBuckets * 16ll +
    (kStaticMaxRecords + (kStaticMaxBuckets + 1ll) * 64 + kStaticMaxBuckets * 1ll * kStatsMaxSlices) * 32;

// Bucket table entries handed to the device in one kernel-argument block.
constexpr int kTableChunk = 120;
struct TableArgs {
    long long *table;            // device: start, end of every bucket
    int first, count;            // buckets [first, first + count) are written
    StatsRecord *partials;       // their counts of arrivals are cleared
    long long start_end[2 * kTableChunk];
};

// Everything one launch of the round kernel needs, passed by value in the kernel
// argument segment: the P gradient and send-buffer bases stay in scalar registers and
// every per-rank decision is uniform across the grid.
struct RoundArgs {
    const void *g[kMaxP];        // G_p arena bases (fp32 or bf16)
    float *r[kMaxP];             // R_p arena bases (fp32)
    unsigned long long active;   // bit p: process p is on time in this round
    unsigned long long valid;    // bit p: R_p holds an undelivered gradient
    unsigned long long gload;    // bit p: this launch reads G_p (every process that has a gradient
                                 // when fused; only on-time processes when the carry runs as
                                 // its own kernel); follows from active and store, for recorders of
                                 // launches
    unsigned long long store;    // bit p: this launch stores G_p into R_p (late processes when
                                 // fused; none otherwise)
    float *w;                    // parameters (NULL: no update rule)
    float *v;                    // momentum
    float *recv;                 // receive buffer (NULL: not wanted)
    long long e0;                // first element of the run (arena index)
    long long n;                 // elements in the run
    long long model;             // elements of the whole model (first bucket start to last end)
    int P;
    int elem_bytes;              // bytes per gradient element: 4 (fp32) or 2 (bf16)
    float inv_P;                 // 1.0f / (float)P
    float neg_lr;                // -lr
    float mu;
    float wd;                    // weight decay (0: none)
    int nesterov;                // 1: Nesterov momentum
    StatsArgs stats;             // stats.stats == NULL: no by-products
};

// The same round as the kernels take it: a list of streams.  Slot k is one stream and one
// action; slots are listed in the order in which they enter the sum (ascending rank, send
// buffer before gradient):
//   ADD    s = s + x                       (a pending R_p of a late process, or the G_p
//                                           of an on-time process with an empty buffer)
//   HOLD   c = x                           (R_p of an on-time process ...)
//   PAIR   s = s + (c + x)                 (... followed by its G_p)
//   SKIP   nothing                         (fills the list up)
// Streams that need not be read do not appear at all, so no load is wasted.  A stream is
// fp32 (send buffers; fp32 gradients) or bf16 (bf16 gradients); a lane owns 4 consecutive
// elements of every stream either way.  The list goes on with the late gradients that the launch
// copies into their send buffers (COPY, fused rounds; the destinations are listed apart) and
// ends in SKIPs.  A slot is ONE scalar load for the kernel: the arena base, whose low four bits are
// zero, with the action and the type in those bits.  What every wavefront reads first stands first.
constexpr int kMaxSlots = 2 * kMaxP;
constexpr int kBurst = 2;              // slots in flight per wavefront of the burst kernel
constexpr int kSlotFill = 8;           // SKIPs behind the list: its ragged tail takes slots 8 at a time
enum SlotKind : unsigned {
    kAdd = 0, kHold = 1, kPair = 2, kSkip = 3, kKindMask = 3,
    kSlotBf16 = 4,                     // the stream is bf16
    kSlotCopy = 8,                     // with kSkip: a copy
    kSlotTag = 15
};
struct SlotHead {
    long long e0, n;
    int n_sum, n_copy;                 // slots of the sum (a multiple of kBurst), copies
    int waves_per_block, xcd_blocks;   // xcd_blocks: 0, or workgroups per XCD when every XCD takes
                                       // a contiguous eighth of the run
    float *w, *v, *recv;
    float inv_P, neg_lr, mu, wd;
    int nesterov;
    int skip;                          // lane-vectors of the first tile that stand before the run (run_back)
};
struct SlotArgs {
    SlotHead h;
    unsigned long long slot[kMaxSlots + kSlotFill + kBurst];   // a process has at most two slots
    float *dst[kMaxSlots + kSlotFill + kBurst];                // of slot k where it is a copy
    StatsArgs stats;
};

// A round as the kernel for small runs takes it: what a wavefront would have to work out from the
// slots is worked out by the host.  The bases are those of the first element of the launch, so that
// an access is the base and a 32-bit offset; what is done with slot k is bit k of a word each.  The
// list holds the sum, then the copies, and nothing to fill it up; the destination of slot k stands at
// dst[k - dst_first], dst_first being a multiple of 8 at or below the first copy.
//   pair   the slot completes the one before it (a HOLD)     hold   it waits for the next one
//          (neither is looked at where the order is free; there all fp32 streams stand before the bf16 ones)
//   copy   it is stored to its destination                   bf     the stream is bf16
struct ChunkBits {
    unsigned pair, hold, copy, bf;
};
constexpr int kChunkWord = 32;            // slots that a ChunkBits covers
constexpr long long kChunkElements = 1ll << 29;   // of one launch, for the 32-bit offsets
enum ChunkForm : int {
    kWide,                                // a lane owns four elements
    kNarrow,                              // one
    kPaced,                               // four, and a copy's store waits for the one before it
    kFormBits = 2
};
struct ChunkHead {
    float *w, *v, *recv;
    unsigned n;                           // elements
    int n_sum, n_slots, dst_first;
    int form;                             // ChunkForm; above its bits, the elements of the first tile that stand
                                          // before the run (a word of their own moved all that follows by 8
                                          // bytes: 0.2 us more for each launch of 12 slots or more)
    int waves_per_block, xcd_blocks;
    float inv_P, neg_lr, mu, wd;
    int nesterov;
    ChunkBits first;                      // of slots 0..31
};
// The arguments travel to the device with every launch and the host pays by the byte, so lists of up to
// 32 slots and 16 copies (8 processes always, 16 in most rounds) have a block of their own size.
template <int SLOTS, int COPIES, bool STATS>
struct ChunkArgs;
template <int SLOTS, int COPIES>
struct ChunkArgs<SLOTS, COPIES, false> {
    static constexpr int kSlots = SLOTS, kCopies = COPIES;
    ChunkHead h;
    unsigned long long slot[SLOTS];
    float *dst[COPIES + 8];
    ChunkBits bits[SLOTS / kChunkWord];
};
template <int SLOTS, int COPIES>
struct ChunkArgs<SLOTS, COPIES, true> : ChunkArgs<SLOTS, COPIES, false> {
    long long first;                      // arena index of the launch's first element
    StatsArgs stats;                      // records: those of the launch
};
constexpr int kChunkFewSlots = 32, kChunkFewCopies = 16;

// A small round whose list is short, as its own kernel takes it (eager_short.h): all that a wavefront needs is 192 or
// 256 bytes, whole lines of the scalar cache that a few loads bring into registers, and the host copies no more than
// that to the device.  Bases are those of the launch's first element and the sum stands before the copies as in
// ChunkArgs.  Of 8 slots, slot k is copied to dst[k]; of 16, the copies stand in the second half - right behind the sum, or
// from slot 8 on where it is shorter - and slot k is copied to dst[k - 8]: every index is one that the compiler knows.
//   shape   slots of the sum, from bit 8 all slots (of 8) or those of the second half (of 16), Nesterov bit 16, ChunkForm from
//           bit 17, from bit 24 on the elements of the first tile that stand before the run
//   bits    of slot k: bit k as `pair`, bit 16 + k as `bf` of ChunkBits
//   copies  bit k: slot k is copied
constexpr int kShortForm = 17, kShortSkip = 24, kShortCopies = 8;
template <int SLOTS>
struct alignas(64) ShortArgs {
    static constexpr int kHalf = SLOTS - 8;    // slot k is copied to dst[k - kHalf]
    float *w, *v, *recv;
    unsigned n, shape, bits, copies;
    float inv_P, neg_lr, mu, wd;
    unsigned unused[2];
    unsigned long long slot[SLOTS];
    float *dst[kShortCopies];
};
static_assert(sizeof(ShortArgs<8>) == 192 && sizeof(ShortArgs<16>) == 256, "whole lines");

// The carry as a kernel of its own: R_p <- G_p for every late process, one (source,
// destination) pair after the other.
struct CarryArgs {
    const void *src[kMaxP];      // G_p arena bases of the late processes
    float *dst[kMaxP];           // their R_p arena bases
    int count;                   // number of pairs
    long long e0;                // first element of the run
    long long n;                 // elements in the run
    int skip;                    // (launcher) lane-vectors at e0 that stand before it, see run_back
};

// A gradient finished after its round: R <- G (empty send buffer) or R <- R + G.
struct StashArgs {
    const void *g;               // gradient arena base of the process
    float *r;                    // its send-buffer arena base
    long long e0, n;             // run
    int accumulate;              // 1: the send buffer holds an undelivered gradient
};

// Several weight views at once (a weight view per process, for processes that lag by more
// than one round): the update rule applied to every listed view from one read of u, or
// every view replaced by the average of all of them.
struct ViewsArgs {
    float *w[kMaxP];             // parameter views
    float *v[kMaxP];             // momentum views (update rule only)
    const float *u;              // averaged update (update rule only)
    int n_views;
    long long e0, n;
    float neg_lr, mu, wd, inv_views;
    int nesterov;
};

// The same for up to N views, N = 4, 8 or 16, without momentum where it is not needed: whole lines of the scalar cache that
// a few loads bring into registers.
template <int N, bool MOMENTUM>
struct alignas(64) FewViewsArgs {
    const float *u;
    long long e0, n;
    float neg_lr, mu, wd, inv_views;
    int nesterov, n_views;
    float *w[N];
    float *v[MOMENTUM ? N : 1];
};

struct SgdArgs {
    const float *u;
    float *w;
    float *v;
    long long e0;
    long long n;
    float neg_lr;
    float mu;
    float wd;
    int nesterov;
};

struct Launch {
    int block = 64;        // threads per workgroup
    int chunk = 0;         // slots whose loads are in flight together; 0: chosen from the run
    int split = 0;         // 0: chosen from the round; 1: one fused kernel; 2: reduce+update
                           // kernel followed by a carry (copy) kernel
    int blocks_per_cu = 0; // 0: chosen from the round; -1: no cap; else max workgroups resident per CU
    int nt_state = -1;     // w, v, recv nontemporal: -1 chosen from their size, 0 no, 1 yes
    int xcd_map = 0;       // round kernels: 1 = contiguous eighth of the run per XCD
    int carry_block = 64;  // carry kernel: threads per workgroup
    int carry_vec = 1;     // carry kernel: lane-vectors per thread and iteration (1, 2, 4)
    int round_stats = 1;           // 0: rounds skip the by-products although statistics are attached
    int carry_blocks_per_cu = -1;  // carry kernel: -1 no cap, else max workgroups per CU
};

hipError_t launch_round(const RoundArgs &a, bool bf16, bool fast, const Launch &cfg,
                        hipStream_t stream);
// the round in chunks of 16 slots (eight: of 8); nt: streams nontemporal, nts: w, v and recv too
typedef hipError_t ChunkLauncher(const SlotArgs &s, bool nt, bool nts, bool eight, int bpc, const Launch &cfg,
                                 hipStream_t st);
ChunkLauncher launch_chunk_f32, launch_chunk_f32_stats, launch_chunk_bf16, launch_chunk_bf16_stats;
ChunkLauncher launch_chunk_f32_fast, launch_chunk_f32_fast_stats, launch_chunk_bf16_fast, launch_chunk_bf16_fast_stats;
// the round with a short list (see short_round), bursts of 8 slots or 16; nt: streams nontemporal
typedef hipError_t ShortLauncher(const SlotArgs &s, bool nt, hipStream_t st);
ShortLauncher launch_short_f32, launch_short_f32_fast, launch_short_bf16, launch_short_bf16_fast;
hipError_t launch_carry(const CarryArgs &a, bool bf16, const Launch &cfg, hipStream_t stream);
hipError_t launch_stats_finish(const StatsArgs &a, hipStream_t stream);
long long slot_records(long long n, bool bf16, int block);   // tiles of a round, one record each
                                                             // (whatever the workgroups)
int slot_tail(long long n, bool bf16);                       // elements of its ragged tail
hipError_t launch_stash(const StashArgs &a, bool bf16, hipStream_t stream);
hipError_t launch_views_sgd(const ViewsArgs &a, bool fast, const Launch &cfg, hipStream_t stream);
hipError_t launch_views_average(const ViewsArgs &a, const Launch &cfg, hipStream_t stream);
hipError_t launch_sgd(const SgdArgs &a, bool fast, const Launch &cfg, hipStream_t stream);
// norms of update and parameters per bucket (records for launch_stats_finish), then the update
// rule with the rate of each element's bucket read from st.stats
hipError_t launch_norms(const SgdArgs &a, const StatsArgs &st, hipStream_t stream);
hipError_t launch_sgd_lars(const SgdArgs &a, const StatsArgs &st, bool fast, hipStream_t stream);
long long norms_records(long long n);
// This device's copy of the library's fixed scratch array (kStaticScratchBytes bytes, 256-byte
// aligned); the address is looked up once per device.  launch_table_fill writes the bucket
// table there with a kernel, so that the call needs no host-to-device copy.
hipError_t static_scratch(char **ptr);
hipError_t launch_table_fill(long long *table, const long long *start_end, int n_buckets,
                             hipStream_t stream);
hipError_t launch_copy(void *dst, const void *src, long long nbytes, hipStream_t stream);
hipError_t launch_read(const void *src, long long nbytes, float *sink, hipStream_t stream);

// A plain kernel with a round's mix of streams (calibration): n_read streams are summed per
// lane-vector and the sum is written to n_write streams.
constexpr int kMixMaxRead = 80, kMixMaxWrite = 80;
struct MixArgs {
    const void *src[kMixMaxRead];
    void *dst[kMixMaxWrite];
    unsigned long long half;     // bit j: read stream j holds 8 bytes per lane-vector, not 16
    void *sink;                  // 4 writable bytes (only touched when nothing is written)
    int n_read, n_write;
    long long nvec;              // lane-vectors per stream
};
hipError_t launch_mix(const MixArgs &a, int waves_per_cu, hipStream_t stream);

}  // namespace eager
