// Host runtime shared by the C ABI translation units (runtime.cpp, adaptive.cpp,
// server.cpp).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <cstdarg>
#include <cstdint>
#include <exception>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <tuple>
#include <type_traits>
#include <vector>

#include <rocprofiler-sdk-roctx/roctx.h>

#include "bfi.h"
#include "host_pool.h"
#include "internal.h"
#include "is_internal.h"
#include "sph_internal.h"

namespace bfi {

bfi_status fail(bfi_status s, const char *fmt, ...);
bfi_status hip_fail(hipError_t e, const char *what);
void clear_error();

#define BFI_HIP(call)                                 \
    do {                                              \
        hipError_t bfi_e_ = (call);                   \
        if (bfi_e_ != hipSuccess)                     \
            return ::bfi::hip_fail(bfi_e_, #call);    \
    } while (0)

#define BFI_TRY(call)                                 \
    do {                                              \
        bfi_status bfi_s_ = (call);                   \
        if (bfi_s_ != BFI_OK)                         \
            return bfi_s_;                            \
    } while (0)

bool shape_compiled(int nx, int nt);
// BFI_FP64, BFI_FP32_SHIFTED or BFI_FP64_SHIFTED
inline bool known_precision(int prec)
{
    return prec == BFI_FP64 || prec == BFI_FP32_SHIFTED || prec == BFI_FP64_SHIFTED;
}
// Dispatch to the kernels compiled for lattice shape (nx, nt).
hipError_t launch_mc(int nx, int nt, const LaunchSpec &spec, const McArgs &args, hipStream_t st);
hipError_t kernel_info(int nx, int nt, const LaunchSpec &spec, KernelInfo *info);
// Gaussian-proposal sampler kernels of shape (nx, nt).
hipError_t launch_is(int nx, int nt, const LaunchSpec &spec, const IsArgs &args, hipStream_t st);
hipError_t is_kernel_info(int nx, int nt, const LaunchSpec &spec, KernelInfo *info);
hipError_t launch_is_debug(int nx, int nt, const IsDebugArgs &args, hipStream_t st);
// Spherical-coordinate sampler kernels of shape (nx, nt).
hipError_t launch_sph(int nx, int nt, const LaunchSpec &spec, const SphArgs &args, hipStream_t st);
hipError_t sph_kernel_info(int nx, int nt, const LaunchSpec &spec, KernelInfo *info);
hipError_t launch_sph_debug(int nx, int nt, const SphDebugArgs &args, hipStream_t st);
bfi_status check_lattice(const bfi_lattice *lat);
bfi_status check_subvolumes(const bfi_lattice *lat, const bfi_subvolumes *subs);
ActionCoef make_coef(const bfi_lattice &lat);

// Owned copy of a subvolume list.
struct SubList {
    std::vector<uint64_t> id, n, offset;
    std::vector<double> lo, hi;  // count x d
    int d = 0;
    size_t size() const { return id.size(); }
    bfi_subvolumes view() const
    {
        return bfi_subvolumes{id.size(), id.data(), lo.data(), hi.data(), n.data(), offset.data()};
    }
};

// Uniform bisection of a box: 2^k leaves, level t halves dim t mod d at
// 0.5 (lo + hi); heap ids 2^k + b; budget split floor(B/2^k) + (b < B mod 2^k).
SubList uniform_split(int d, const double *box_lo, const double *box_hi, int k, uint64_t budget);

struct TuneKey {
    int nx, nt, prec;
    int pairs = 0;  // antithetic pairs: a kernel of its own, tuned apart
    int obs = 0;    // observable (anchored or averaged), likewise
    bool operator<(const TuneKey &o) const
    {
        return std::tie(nx, nt, prec, pairs, obs) < std::tie(o.nx, o.nt, o.prec, o.pairs, o.obs);
    }
};
struct TuneEntry {
    bfi_launch launch;
    double evals_per_s;
};

// Runs the body of a C ABI entry point: C++ exceptions (host allocation
// failure above all) become status codes, so nothing unwinds into a C caller.
template <class F>
bfi_status guarded(F &&body) noexcept
{
    try {
        return body();
    } catch (const std::bad_alloc &) {
        return fail(BFI_ENOMEM, "host allocation failed");
    } catch (const std::exception &e) {
        return fail(BFI_EINVAL, "%s", e.what());
    } catch (...) {
        return fail(BFI_EINVAL, "unexpected exception");
    }
}

// A named range of host work on the calling thread, visible to rocprofv3
// --marker-trace (roctx); without a tool attached the calls return at once.
struct TraceRange {
    explicit TraceRange(const char *name) { roctxRangePushA(name); }
    ~TraceRange() { roctxRangePop(); }
    TraceRange(const TraceRange &) = delete;
    TraceRange &operator=(const TraceRange &) = delete;
};
// Consecutive phases of one loop body: next() closes the current range and
// opens the following one; leaving the scope closes the last.
struct TracePhases {
    explicit TracePhases(const char *first) { roctxRangePushA(first); }
    void next(const char *name)
    {
        roctxRangePop();
        roctxRangePushA(name);
    }
    ~TracePhases() { roctxRangePop(); }
    TracePhases(const TracePhases &) = delete;
    TracePhases &operator=(const TracePhases &) = delete;
};

// Resolve a requested launch (zeros = tuned or default) for a lattice.
bfi_launch resolve_launch(const bfi_context *ctx, const bfi_lattice &lat, int prec, bool split,
                          const bfi_launch *req);

// Whether an evaluation's work items may be made smaller than its launch shape
// says, to fill the chip: the caller left samples_per_thread open, and the form
// is plain FP64.  The shifted forms keep the launch shape's items at every
// size: a thread's shift is set by the samples that it takes, and with it the
// rounding of their weights (in FP32) and the scale of the record.
inline bool spread_items(int prec, const bfi_launch *req)
{
    return prec == kFP64 && !(req && req->samples_per_thread > 0);
}
// Work items of n samples in chunks, without an integer division: exact below 2^48
// samples of chunks below 2^31 (the quotient, raised by 2^-49, lies above the true
// one and by less than 1/chunk).  A list's size is asked for up to six times:
// 10^4 subvolumes 0.15 -> 0.05 ms.
struct ItemCount {
    double inverse;
    explicit ItemCount(uint64_t chunk) : inverse((1.0 + 0x1p-49) / static_cast<double>(chunk)) {}
    uint64_t operator()(uint64_t n) const
    {
        if (n == 0)
            return 0;
        return static_cast<uint64_t>(
                   static_cast<int64_t>(static_cast<double>(static_cast<int64_t>(n - 1)) * inverse)) +
               1;
    }
};
// Samples per work item of a list of sample counts, at most the launch shape's
// samples_per_thread x block.  The tuned shapes are those of long runs, whose
// items hold 2^16 samples and more; a list of fewer than eight rounds of such
// items over the `resident` blocks leaves blocks without work (2^6 subvolumes
// of 46875 samples made 64 items for 512 blocks) and ends on a round that is
// partly empty.  With `spread`, such a list is cut into about one to eight
// rounds of shorter items, as many as an estimate of the finishing time prefers.
// Measured, launch shape's items -> these, whole calls: 10x2 FP64, 3e6
// evaluations over 64 subvolumes 416 -> 291 us; 301 uneven leaves of 2^10 ..
// 2^17 samples with split statistics 925 -> 501 us; spherical sampler, 2^24
// over 64 shells in two passes 2.16 -> 1.60 ms; 2^27 evaluations of 8x2 as pairs,
// one round of 512 items -> four of a quarter of them, 1.04 -> 0.98 ms.  From
// eight rounds on the
// launch shape's items are as fast and there are fewer records to merge (2^30
// evaluations of 10x2: the same 4096 items, 11.8 ms).
uint64_t item_samples(const bfi_launch &l, bool spread, bool split, const uint64_t *n, size_t nsub,
                      uint64_t resident);

// A list's items: their size, how many there are, how many its largest subvolume
// has.
struct ItemCut {
    uint64_t chunk, nitems, most;
};
ItemCut cut_items(const bfi_launch &l, bool spread, bool split, const uint64_t *n, size_t nsub,
                  uint64_t resident);
// The items of a list of lattice subvolumes, for every entry point alike: shorter
// ones (spread) unless only the launch shape's fit the allocation-free entry
// point's array, so that its records are those of the others on every list that
// it takes.
ItemCut cut_lattice_items(const bfi_launch &l, bool spread, bool split, int d, int rec_len,
                          const uint64_t *n, size_t nsub, uint64_t resident);
// Bytes of that array for a list (noalloc.hip).
size_t noalloc_bytes(size_t nsub, int d, int rec_len, uint64_t nitems, bool split);

// Rounds of items over the resident blocks from which a list counts as long: the
// last round and the start no longer matter.
constexpr uint64_t kRounds = 8;
// Whether the items are drained through a queue or each has a block of its own
// (the records are the same): as asked, or where the caller left it open, as the
// launch shape has it for long lists and long items.  Every block's first item
// and each short one costs the queue's counter 10 ns of its own, all blocks one
// after another: 4x2 FP64, 1984 items of 6 samples per thread took 41 us through
// the queue, 25 as blocks; 10x2, 1024 items of 12 samples 53 and 48; from 64
// samples per thread on both are equal, and on the longest lists the queue is
// ahead (2^30 of 10x2 FP64 11.74 ms, 11.84 as blocks).
inline bool item_queue(const bfi_launch &l, const bfi_launch *req, uint64_t chunk, uint64_t nitems,
                       uint64_t resident)
{
    if (!l.persistent || (req && req->persistent >= 0))
        return l.persistent != 0;
    const bool brief = chunk <= 64 * static_cast<uint64_t>(l.block);
    return nitems >= kRounds * resident || (nitems > resident && !brief);
}

// Work items of a list: record slots in list order (sub_first: first slot of each
// subvolume, nsub + 1 entries), the items themselves in the order in which blocks
// shall take them, whole ones first and then the subvolumes' rests by falling
// length (in 64ths of a whole one), so that the last round ends on the shortest.
// (The records do not depend on the order.)  Measured, list order -> this, whole calls: 2^26
// evaluations of the Gaussian-proposal sampler over 512 streams 1.38 -> 1.33 ms,
// 301 uneven leaves with split statistics 257 -> 250 us.  The order is a count's,
// not a sort's, since long lists gain nothing by it: 10^4 ragged leaves are listed
// in 0.07 ms (a stable sort of the rests 0.7), 10^6 in 7 (120).
void list_items(uint64_t chunk, const uint64_t *n, size_t nsub, const EvalParams *params,
                double *item_rec, int rec_len, uint32_t *sub_first, WorkItem *items);

// Host finalize of partial records (see bfi_finalize).
// evals_per_sample: integrand evaluations behind one record sample (2 for
// antithetic pairs), for n_evals.  leaf_var (nsub doubles, or NULL) gets each
// subvolume's contribution to the variance of C, sum_r [Var N_s - 2 C Cov_s +
// C^2 Var Z_s] / Z^2, clamped at 0.  Large lists are summed in parallel chunks
// whose sums combine in a fixed order (the result does not depend on threads).
// volumes (nsub doubles, or NULL): the products of the extents, when the caller
// keeps them (they must equal the product over dimensions in order).
bfi_status finalize_records(int nx, int d, size_t nsub, const double *lo, const double *hi,
                            const double *partials, bfi_result *out, int evals_per_sample = 1,
                            double *leaf_var = nullptr, const double *volumes = nullptr);

// Evaluates work lists that change from call to call (adaptive rounds) with
// resident buffers: entries are written into pinned staging, run() uploads them,
// builds items and point maps on the device, drains them with the persistent
// kernel, merges and downloads one record (and split statistics) per entry,
// all as one captured graph updated in place from call to call.  Buffers grow
// geometrically and are freed by the destructor.  Blocking on the context's
// stream; not thread-safe.
class ResidentEval {
public:
    ResidentEval() = default;
    ~ResidentEval();
    ResidentEval(const ResidentEval &) = delete;
    ResidentEval &operator=(const ResidentEval &) = delete;
    // split: accumulate split statistics (256-thread blocks, d <= 32)
    bfi_status init(bfi_context *ctx, const bfi_lattice &lat, int prec, bool split,
                    const bfi_launch *launch);
    // stage(count) sizes the list, then set() fills entry i: samples [offset,
    // offset + n) of stream `id` over [lo, hi) (entries may be set from several
    // threads)
    bfi_status stage(size_t count);
    void set(size_t i, uint64_t id, uint64_t offset, uint64_t n, const double *lo,
             const double *hi)
    {
        set_counts(i, id, offset, n);
        set_box(i, lo, hi);
    }
    // the two halves of set: prepare reads the counts; the boxes are read only
    // when the replay copies them to the device, so they may be written after
    // prepare and before launch
    void set_counts(size_t i, uint64_t id, uint64_t offset, uint64_t n)
    {
        h_id_[i] = id;
        h_off_[i] = offset;
        h_n_[i] = n;
    }
    void set_box(size_t i, const double *lo, const double *hi)
    {
        const size_t d = static_cast<size_t>(d_);
        std::copy(lo, lo + d, h_lo_ + i * d);
        std::copy(hi, hi + d, h_hi_ + i * d);
    }
    size_t size() const { return count_; }
    // evaluate the pushed entries (then cleared): rec_out gets count x
    // BFI_PARTIAL_LEN(nx) records, split_out count x BFI_SPLIT_LEN(d) (split
    // only); device_ms the replay's duration from events around it
    bfi_status run(uint64_t seed, double *rec_out, double *split_out, double *device_ms);
    // the same in three steps, so that several evaluators' replays can be queued
    // back to back on the context's stream (all prepared before any launch: a
    // capture never begins while one of them is in flight) and the host reads
    // one's records while the next runs: prepare captures (or updates) the
    // replay, launch queues it, finish waits for it and copies the records out
    bfi_status prepare(uint64_t seed);
    bfi_status launch();
    bfi_status finish(double *rec_out, double *split_out, double *device_ms);
    // the last finished list's records and split statistics in the pinned
    // buffers the replay copied them to (finish with NULL outputs skips the
    // copy), valid until the next prepare; with record copies on only
    const double *records() const { return h_rec_; }
    const double *split_records() const { return h_split_; }
    // whether a replay copies its records to the host (default yes), set
    // before prepare; without, they stay in device memory for a consumer queued
    // after the replay on the context's stream, valid until the next prepare
    void set_copy_records(bool on) { copy_records_ = on; }
    const double *device_records() const { return d_sub_rec_; }
    const double *device_split_records() const { return d_sub_split_; }
    int instantiations() const { return instantiations_; }
    int updates() const { return updates_; }

private:
    bfi_status enqueue(size_t nsub, uint64_t nitems, hipStream_t st);
    void release();

    bfi_context *ctx_ = nullptr;
    bfi_lattice lat_{};
    int prec_ = 0, d_ = 0, rec_len_ = 0, split_len_ = 0;
    bool split_ = false, copy_records_ = true;
    int asked_ = -1;  // 1, 0: the caller chose the queue or a block per item; -1: item_queue
    bfi_launch launch_{};
    uint64_t chunk_ = 0, resident_blocks_ = 0;
    size_t count_ = 0;
    // What the host writes for a list, one block in pinned memory and its copy in
    // device memory: parameters, queue head (0), then ids, counts, offsets and the
    // boxes, each from a multiple of 256 bytes.
    struct Staged {
        size_t head, id, n, off, lo, hi, bytes;
        Staged(size_t count, int d);
    };
    char *h_stage_ = nullptr, *d_stage_ = nullptr;
    size_t cap_h_stage_ = 0, cap_d_stage_ = 0;
    // pieces of h_stage_ for the staged count
    uint64_t *h_id_ = nullptr, *h_n_ = nullptr, *h_off_ = nullptr;
    double *h_lo_ = nullptr, *h_hi_ = nullptr;
    double *h_rec_ = nullptr, *h_split_ = nullptr;
    size_t cap_h_rec_ = 0, cap_h_split_ = 0;
    // device
    double *d_base64_ = nullptr, *d_scale64_ = nullptr;
    float *d_base32_ = nullptr, *d_scale32_ = nullptr;
    uint32_t *d_sub_first_ = nullptr;
    WorkItem *d_items_ = nullptr;
    double *d_item_rec_ = nullptr, *d_item_split_ = nullptr, *d_sub_rec_ = nullptr,
           *d_sub_split_ = nullptr;
    size_t cap_d_sub_[3] = {}, cap_d_map_[4] = {}, cap_d_items_[3] = {};
    hipGraphExec_t exec_ = nullptr;
    hipEvent_t ev_start_ = nullptr, ev_stop_ = nullptr;
    int instantiations_ = 0, updates_ = 0;
    size_t prepared_ = 0;   // entries of the replay prepared and not yet finished
    bool launched_ = false;
};

// Take the device address of the allocation-free entry point's scratch array on
// `device` (which must be current); once per device, later calls return at once.
bfi_status noalloc_setup(int device);

}  // namespace bfi

struct bfi_context {
    int device = 0;
    int cu_count = 0;
    hipStream_t stream = nullptr;
    std::string arch;
    std::map<bfi::TuneKey, bfi::TuneEntry> tuned;
    // blocking calls' memory (CallScratch), one call at a time
    std::mutex scratch_busy;
    char *scratch_dev = nullptr, *scratch_host = nullptr;
    size_t scratch_dev_cap = 0, scratch_host_cap = 0;
    // blocks per CU of the kernel variants asked for so far
    std::mutex occupancy_mutex;
    std::map<std::array<int, 8>, int> occupancy;
};

// A resident evaluation: descriptors, work items and buffers on the device.
struct bfi_plan {
    bfi_context *ctx = nullptr;
    int kind = 0;  // 0: lattice action (mc_kernel), 1: N-sphere test integrand,
                   // 2: Gaussian-proposal sampler (is_kernel) over streams
    bfi_lattice lat{};
    int prec = 0;
    int d = 0, nx = 0, rec_len = 0;
    bool split = false;
    size_t nsub = 0;
    bfi_launch launch{};
    uint32_t nitems = 0, most_items = 0;  // of the list, and of its largest subvolume
    bool direct = false;  // d_sub_rec, d_sub_split in the call's pinned block
    bool queue = false;  // items through the queue (item_queue)
    bool fixed_order = false;  // merged in one run: sums in the launch shape's order
    uint32_t grid = 0;
    uint64_t n_evals = 0;

    // the plan's own device memory (null where a call lends it), and its pieces
    char *d_block = nullptr;
    bfi::EvalParams *d_params = nullptr;
    bfi::EvalParams params{};  // host copy of *d_params
    bfi::WorkItem *d_items = nullptr;
    double *d_item_rec = nullptr, *d_item_split = nullptr;
    uint32_t *d_sub_first = nullptr;
    double *d_sub_rec = nullptr, *d_sub_split = nullptr;
    uint32_t *d_head = nullptr;
    bfi::IsTable *d_is_table = nullptr;  // kind 2

    // captured replays (queue reset, kernel, merge, copy to the destination), one
    // per (stream, destination) pair, the kMaxReplays used last kept (ordered by
    // last use): alternating output buffers replays without capturing again
    struct Replay {
        hipGraphExec_t exec = nullptr;
        hipGraph_t def = nullptr;
        hipStream_t stream = nullptr;
        double *dst = nullptr;
    };
    static constexpr size_t kMaxReplays = 4;
    std::vector<Replay> replays;
    hipStream_t last_stream = nullptr;
    // bracket the Monte Carlo kernel of every run (timing of the hot kernel)
    hipEvent_t ev_start = nullptr, ev_stop = nullptr;
};

namespace bfi {
// Device and pinned host memory of one blocking call on the context's stream:
// the context's, kept from call to call, or -- while another call holds it, or
// beyond kScratchLimit -- the call's own.  Given back by the destructor, which
// first waits for the stream unless wait() has (an error path's copies may
// still read the host block).
//
// A call used to allocate and free its 14 device buffers, copy nine arrays from
// pageable memory and create two events: of 225 us for 2^16 evaluations of 4x2
// the kernels were 21.  With one block and one copy each way it takes 44 us;
// 2^26 evaluations of the Gaussian-proposal sampler over 512 streams 1.67 ->
// 1.42 ms, 3.2e7 of the N-sphere integrand 544 -> 338 us.
class CallScratch {
public:
    static constexpr size_t kScratchLimit = size_t(64) << 20;
    CallScratch() = default;
    ~CallScratch();
    CallScratch(const CallScratch &) = delete;
    CallScratch &operator=(const CallScratch &) = delete;
    bfi_status take(bfi_context *ctx, size_t host_bytes, size_t dev_bytes);
    char *host() const { return host_; }
    char *dev() const { return dev_; }
    // Whether kernels may write `bytes` of results straight into the host block
    // (pinned, the context's own): up to 64 KiB, which the bus takes within the
    // merge's own time.  A copy apart cost a call 2 to 7 us (2^16 evaluations of
    // 4x2 44 us with it, 42 without; 3e6 of 10x2 92 and 85).
    bool direct(size_t bytes) const { return held_.owns_lock() && bytes <= (size_t(64) << 10); }
    // copy the first `bytes` of the host block to the device block
    bfi_status upload(size_t bytes);
    // copy `bytes` of the device block from `from` to the host block's start and
    // wait for them
    bfi_status download(size_t from, size_t bytes);
    // wait for what is queued
    bfi_status wait();

private:
    bfi_context *ctx_ = nullptr;
    std::unique_lock<std::mutex> held_;
    std::vector<char> own_host_;
    char *own_dev_ = nullptr, *host_ = nullptr, *dev_ = nullptr;
    bool queued_ = false;
};

// Blocks of one kernel variant that fill the chip once (kind as in bfi_plan, with
// the N-sphere's dimension as nx; 3: the sampler in spherical coordinates).
bfi_status resident_blocks(bfi_context *ctx, int kind, const bfi_lattice &lat,
                           const LaunchSpec &spec, uint64_t *blocks);

bfi_status plan_build(bfi_context *ctx, const bfi_lattice &lat, int prec,
                      const bfi_subvolumes &subs, const bfi_launch *launch, bfi_plan **out);
// One blocking evaluation of a list on the context's stream: records to
// `partials`, split statistics to `split` when non-NULL.
//   eval_once: the lattice action over boxes.  fixed_order: items of the launch
//     shape and a merge in one run, for callers that decide by the split
//     statistics.  Where a few samples carry a subvolume's weight, two
//     dimensions' spreads are equal but for the last bits of the sums, and
//     another order of summation would suggest another dimension.
//   eval_once_nsphere: the N-sphere integrand over `dim`-dimensional boxes
//     (FP64, split statistics always on, 256-thread blocks, fixed order);
//     records have nx = 0.
//   eval_once_is: the Gaussian-proposal sampler; `streams` lists stream ids (bit
//     63: uniform component), sample counts and offsets (lo, hi unused).
bfi_status eval_once(bfi_context *ctx, const bfi_lattice &lat, int prec, uint64_t seed,
                     const bfi_subvolumes &subs, const bfi_launch *launch, double *partials,
                     double *split, bool fixed_order = false);
bfi_status eval_once_nsphere(bfi_context *ctx, int dim, uint64_t seed, const bfi_subvolumes &subs,
                             const bfi_launch *launch, double *partials, double *split);
bfi_status eval_once_is(bfi_context *ctx, const bfi_lattice &lat, int prec, uint64_t seed,
                        const bfi_subvolumes &streams, const IsTable &table,
                        const bfi_launch *launch, double *partials);
// timed: record the plan's events around the Monte Carlo kernel (not inside a
// graph capture, where recorded events carry no timestamps)
bfi_status plan_enqueue(bfi_plan *p, uint64_t seed, double *dst, hipStream_t stream, bool timed);
bfi_status plan_free(bfi_plan *p);
// Write the seed into the plan's device parameters (waits for earlier runs).
bfi_status plan_set_seed(bfi_plan *p, uint64_t seed);
}  // namespace bfi
