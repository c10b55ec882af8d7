// Resident evaluation of work lists that change from call to call (the rounds of
// adaptive refinement): device buffers and pinned host staging sized once and
// grown geometrically, the whole device sequence captured in a hipGraph.
//
// One call: the list staged in pinned memory is copied to the device (one block,
// the zeroed queue head in it), the point maps and work items are built there
// (launch_build_items), the persistent Monte Carlo kernel drains the items, the
// merge kernel folds them into per-entry records, and the records (and split
// statistics) are copied back to pinned memory.  That sequence is captured on
// the context's stream and applied to the executable graph of the previous
// call with hipGraphExecUpdate (same nodes, new sizes and arguments); only when
// the update is refused is the graph instantiated again.  No device allocation
// happens unless a list outgrows every list before it.  (Six arrays copied apart
// and a kernel that reset the queue head cost each of a round's two replays some
// 30 us, and each run the pinning of twice eight buffers: a run of 2^28
// evaluations over 8 rounds 9.7 -> 8.2 ms without them.)
#include "launch_limits.h"
#include "runtime.h"

#include <algorithm>
#include <cstring>

namespace bfi {

namespace {

template <class T>
hipError_t grow_device(T **p, size_t *cap, size_t need)
{
    if (need <= *cap && *p)
        return hipSuccess;
    const size_t n = std::max<size_t>({need, 2 * *cap, 64});
    if (*p) {
        hipError_t e = hipFree(*p);
        if (e != hipSuccess)
            return e;
        *p = nullptr;
    }
    *cap = 0;
    hipError_t e = hipMalloc(reinterpret_cast<void **>(p), n * sizeof(T));
    if (e == hipSuccess)
        *cap = n;
    return e;
}

// Pinned memory; its contents are dropped when it grows.
template <class T>
hipError_t grow_pinned(T **p, size_t *cap, size_t need)
{
    if (need <= *cap && *p)
        return hipSuccess;
    const size_t n = std::max<size_t>({need, 2 * *cap, 64});
    if (*p)
        (void)hipHostFree(*p);
    *p = nullptr;
    *cap = 0;
    hipError_t e = hipHostMalloc(reinterpret_cast<void **>(p), n * sizeof(T), hipHostMallocDefault);
    if (e == hipSuccess)
        *cap = n;
    return e;
}

}  // namespace

ResidentEval::Staged::Staged(size_t count, int d)
{
    size_t at = 0;
    auto region = [&](size_t size) {
        const size_t here = at;
        at += (size + 255) & ~size_t(255);
        return here;
    };
    region(sizeof(EvalParams));
    head = region(sizeof(uint32_t));
    id = region(count * 8);
    n = region(count * 8);
    off = region(count * 8);
    lo = region(count * static_cast<size_t>(d) * 8);
    hi = region(count * static_cast<size_t>(d) * 8);
    bytes = at;
}

ResidentEval::~ResidentEval() { release(); }

void ResidentEval::release()
{
    // a replay may still be queued (an error between launch and finish): let it
    // end before its graph and buffers go
    if (ctx_)
        (void)hipStreamSynchronize(ctx_->stream);
    if (exec_)
        (void)hipGraphExecDestroy(exec_);
    exec_ = nullptr;
    prepared_ = 0;
    launched_ = false;
    void *dev[] = {d_stage_, d_base64_, d_scale64_, d_base32_, d_scale32_, d_sub_first_, d_items_,
                   d_item_rec_, d_item_split_, d_sub_rec_, d_sub_split_};
    for (void *p : dev)
        if (p)
            (void)hipFree(p);
    void *host[] = {h_stage_, h_rec_, h_split_};
    if (ev_start_)
        (void)hipEventDestroy(ev_start_);
    if (ev_stop_)
        (void)hipEventDestroy(ev_stop_);
    ev_start_ = ev_stop_ = nullptr;
    for (void *p : host)
        if (p)
            (void)hipHostFree(p);
    h_stage_ = d_stage_ = nullptr;
    h_id_ = h_n_ = h_off_ = nullptr;
    h_lo_ = h_hi_ = h_rec_ = h_split_ = nullptr;
    d_base64_ = d_scale64_ = nullptr;
    d_base32_ = d_scale32_ = nullptr;
    d_sub_first_ = nullptr;
    d_items_ = nullptr;
    d_item_rec_ = d_item_split_ = d_sub_rec_ = d_sub_split_ = nullptr;
}

bfi_status ResidentEval::init(bfi_context *ctx, const bfi_lattice &lat, int prec, bool split,
                              const bfi_launch *launch)
{
    ctx_ = ctx;
    lat_ = lat;
    prec_ = prec;
    split_ = split;
    d_ = lat.nx * lat.nt;
    rec_len_ = BFI_PARTIAL_LEN(lat.nx);
    split_len_ = BFI_SPLIT_LEN(d_);
    launch_ = resolve_launch(ctx, lat, prec, split, launch);
    launch_.use_graph = 1;
    launch_.persistent = 1;
    asked_ = launch && launch->persistent >= 0 ? launch->persistent != 0 : -1;
    if (!mc_block_ok(launch_.block))
        return fail(BFI_EINVAL, "block must be 64, 128, 256, 512 or 1024 (got %d)", launch_.block);
    if (launch_.samples_per_thread < 1 || launch_.samples_per_thread > (1 << 20))
        return fail(BFI_EINVAL, "samples_per_thread out of range");
    chunk_ = static_cast<uint64_t>(launch_.samples_per_thread) * launch_.block;
    if (chunk_ > 0x7FFFFFFFull)
        return fail(BFI_EINVAL, "samples per work item exceed 2^31");
    LaunchSpec spec{prec, launch_.block, split ? 1 : 0, 1, 0, lat.observable, lat.antithetic};
    KernelInfo info{};
    BFI_HIP(kernel_info(lat.nx, lat.nt, spec, &info));
    resident_blocks_ = static_cast<uint64_t>(std::max(info.blocks_per_cu, 1)) *
                       std::max(ctx->cu_count, 1);
    count_ = 0;
    return BFI_OK;
}

bfi_status ResidentEval::stage(size_t count)
{
    count_ = 0;
    const Staged at(count, d_);
    BFI_HIP(grow_pinned(&h_stage_, &cap_h_stage_, at.bytes));
    h_id_ = reinterpret_cast<uint64_t *>(h_stage_ + at.id);
    h_n_ = reinterpret_cast<uint64_t *>(h_stage_ + at.n);
    h_off_ = reinterpret_cast<uint64_t *>(h_stage_ + at.off);
    h_lo_ = reinterpret_cast<double *>(h_stage_ + at.lo);
    h_hi_ = reinterpret_cast<double *>(h_stage_ + at.hi);
    count_ = count;
    return BFI_OK;
}

bfi_status ResidentEval::run(uint64_t seed, double *rec_out, double *split_out, double *device_ms)
{
    BFI_TRY(prepare(seed));
    BFI_TRY(launch());
    return finish(rec_out, split_out, device_ms);
}

bfi_status ResidentEval::prepare(uint64_t seed)
{
    prepared_ = 0;
    const size_t nsub = count_;
    if (nsub == 0)
        return BFI_OK;
    if (nsub >= 0xFFFFFFFFull)
        return fail(BFI_EINVAL, "too many entries in one list");
    const size_t d = static_cast<size_t>(d_);
    uint64_t nitems = 0;
    for (size_t s = 0; s < nsub; ++s) {
        nitems += h_n_[s] / chunk_ + (h_n_[s] % chunk_ != 0);
        if (nitems > 0x7FFFFFFFull)
            return fail(BFI_EINVAL, "more than 2^31 work items; raise samples_per_thread");
    }
    // device capacity (a buffer that moves is a new argument of its nodes, which
    // the graph update below takes like any other)
    const Staged at(nsub, d_);
    BFI_HIP(grow_device(&d_stage_, &cap_d_stage_, at.bytes));
    BFI_HIP(grow_device(&d_sub_first_, &cap_d_sub_[0], nsub + 1));
    BFI_HIP(grow_device(&d_base64_, &cap_d_map_[0], nsub * d));
    BFI_HIP(grow_device(&d_scale64_, &cap_d_map_[1], nsub * d));
    BFI_HIP(grow_device(&d_base32_, &cap_d_map_[2], nsub * d));
    BFI_HIP(grow_device(&d_scale32_, &cap_d_map_[3], nsub * d));
    BFI_HIP(grow_device(&d_items_, &cap_d_items_[0], nitems));
    BFI_HIP(grow_device(&d_item_rec_, &cap_d_items_[1], nitems * rec_len_));
    BFI_HIP(grow_device(&d_sub_rec_, &cap_d_sub_[1], nsub * rec_len_));
    // pinned room for the records only when they come back (at a million
    // leaves that is hundreds of megabytes, slow to pin)
    if (copy_records_)
        BFI_HIP(grow_pinned(&h_rec_, &cap_h_rec_, nsub * rec_len_));
    if (split_) {
        BFI_HIP(grow_device(&d_item_split_, &cap_d_items_[2], nitems * 2 * d));
        BFI_HIP(grow_device(&d_sub_split_, &cap_d_sub_[2], nsub * split_len_));
        if (copy_records_)
            BFI_HIP(grow_pinned(&h_split_, &cap_h_split_, nsub * split_len_));
    }
    const EvalParams P{d_base64_, d_scale64_, d_base32_, d_scale32_,
                       reinterpret_cast<const uint64_t *>(d_stage_ + at.id),
                       reinterpret_cast<const uint64_t *>(d_stage_ + at.off), make_coef(lat_),
                       static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32)};
    std::memcpy(h_stage_, &P, sizeof(P));
    std::memset(h_stage_ + at.head, 0, sizeof(uint32_t));

    hipStream_t st = ctx_->stream;
    BFI_HIP(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
    bfi_status s = enqueue(nsub, nitems, st);
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(st, &g);
    if (s != BFI_OK) {
        if (g)
            (void)hipGraphDestroy(g);
        return s;
    }
    BFI_HIP(e);
    if (exec_) {
        hipGraphNode_t bad = nullptr;
        hipGraphExecUpdateResult why = hipGraphExecUpdateSuccess;
        e = hipGraphExecUpdate(exec_, g, &bad, &why);
        if (e != hipSuccess || why != hipGraphExecUpdateSuccess) {
            (void)hipGetLastError();  // a refused update is not an error of the call
            (void)hipGraphExecDestroy(exec_);
            exec_ = nullptr;
        } else {
            ++updates_;
        }
    }
    if (!exec_) {
        e = hipGraphInstantiate(&exec_, g, nullptr, nullptr, 0);
        if (e != hipSuccess) {
            exec_ = nullptr;
            (void)hipGraphDestroy(g);
            return hip_fail(e, "hipGraphInstantiate");
        }
        ++instantiations_;
    }
    (void)hipGraphDestroy(g);
    if (!ev_start_) {
        BFI_HIP(hipEventCreate(&ev_start_));
        BFI_HIP(hipEventCreate(&ev_stop_));
    }
    prepared_ = nsub;
    return BFI_OK;
}

bfi_status ResidentEval::launch()
{
    if (prepared_ == 0)
        return BFI_OK;
    hipStream_t st = ctx_->stream;
    BFI_HIP(hipEventRecord(ev_start_, st));
    BFI_HIP(hipGraphLaunch(exec_, st));
    BFI_HIP(hipEventRecord(ev_stop_, st));
    launched_ = true;
    return BFI_OK;
}

bfi_status ResidentEval::finish(double *rec_out, double *split_out, double *device_ms)
{
    if (device_ms)
        *device_ms = 0.0;
    const size_t nsub = prepared_;
    if (nsub == 0) {
        count_ = 0;
        return BFI_OK;
    }
    if (!launched_)
        return fail(BFI_EINVAL, "finish before launch");
    launched_ = false;
    prepared_ = 0;
    BFI_HIP(hipEventSynchronize(ev_stop_));
    if (device_ms) {
        float ms = 0.0f;
        BFI_HIP(hipEventElapsedTime(&ms, ev_start_, ev_stop_));
        *device_ms = ms;
    }
    if (rec_out || split_out)
        if (!copy_records_)
            return fail(BFI_EINVAL, "records kept on the device");
    if (rec_out)
        std::memcpy(rec_out, h_rec_, nsub * rec_len_ * sizeof(double));
    if (split_ && split_out)
        std::memcpy(split_out, h_split_, nsub * split_len_ * sizeof(double));
    count_ = 0;
    return BFI_OK;
}

bfi_status ResidentEval::enqueue(size_t nsub, uint64_t nitems, hipStream_t st)
{
    const Staged at(nsub, d_);
    auto *params = reinterpret_cast<EvalParams *>(d_stage_);
    BFI_HIP(hipMemcpyAsync(d_stage_, h_stage_, at.bytes, hipMemcpyHostToDevice, st));
    BuildArgs ba{reinterpret_cast<const double *>(d_stage_ + at.lo),
                 reinterpret_cast<const double *>(d_stage_ + at.hi),
                 reinterpret_cast<const uint64_t *>(d_stage_ + at.n), d_sub_first_, d_base64_,
                 d_scale64_, d_base32_, d_scale32_, d_items_, params, d_item_rec_, chunk_,
                 static_cast<uint32_t>(nsub), d_, rec_len_};
    BFI_HIP(launch_build_items(ba, st));
    // (a block per item as asked, as far as a launch reaches)
    const bool queue = asked_ < 0 ? item_queue(launch_, nullptr, chunk_, nitems, resident_blocks_)
                                  : asked_ == 1 || nitems * launch_.block > kMaxThreads;
    LaunchSpec spec{prec_, launch_.block, split_ ? 1 : 0, queue ? 1 : 0,
                    static_cast<uint32_t>(
                        queue ? std::min<uint64_t>(resident_blocks_, nitems) : nitems),
                    lat_.observable, lat_.antithetic};
    McArgs a{};
    a.items = d_items_;
    a.item_rec = d_item_rec_;
    a.item_split = split_ ? d_item_split_ : nullptr;
    a.queue_head = queue ? reinterpret_cast<uint32_t *>(d_stage_ + at.head) : nullptr;
    a.nitems = static_cast<uint32_t>(nitems);
    a.samples_per_thread = static_cast<uint32_t>(launch_.samples_per_thread);
    BFI_HIP(launch_mc(lat_.nx, lat_.nt, spec, a, st));
    MergeArgs m{};
    m.item_rec = d_item_rec_;
    m.item_split = split_ ? d_item_split_ : nullptr;
    m.sub_first = d_sub_first_;
    m.sub_rec = d_sub_rec_;
    m.sub_split = split_ ? d_sub_split_ : nullptr;
    m.nsub = static_cast<uint32_t>(nsub);
    // nitems and most stay 0, so every subvolume is one run (sums that decide keep one
    // order) and every list takes the same kernel: another one from round to round
    // could not be updated in place
    m.nx = lat_.nx;
    m.d = d_;
    BFI_HIP(launch_merge(m, st));
    if (!copy_records_)
        return BFI_OK;
    BFI_HIP(hipMemcpyAsync(h_rec_, d_sub_rec_, nsub * rec_len_ * 8, hipMemcpyDeviceToHost, st));
    if (split_)
        BFI_HIP(hipMemcpyAsync(h_split_, d_sub_split_, nsub * split_len_ * 8,
                               hipMemcpyDeviceToHost, st));
    return BFI_OK;
}

}  // namespace bfi
