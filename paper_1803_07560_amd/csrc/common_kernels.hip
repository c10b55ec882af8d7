// Shape-independent kernels: work items and point maps built on the device, queue
// reset, the ordered per-subvolume merge of work-item records, and the
// point-emitting test hook.
#include <algorithm>
#include <type_traits>

#include "bfi.h"
#include "device.hpp"
#include "launch_limits.h"

namespace bfi {
namespace {

// First work item of every subvolume: an exclusive prefix sum of
// ceil(n_s / chunk) in tiles of the block, one block for the whole list.
constexpr int kScanBlock = 1024;
__global__ void __launch_bounds__(kScanBlock)
    first_items_kernel(const uint64_t *n, uint32_t nsub, uint64_t chunk, uint32_t *sub_first)
{
    __shared__ uint32_t tile[kScanBlock];
    uint32_t carry = 0;
    const uint32_t t = threadIdx.x;
    for (uint32_t base = 0; base < nsub; base += kScanBlock) {
        const uint32_t s = base + t;
        const uint32_t cnt =
            s < nsub ? static_cast<uint32_t>(n[s] / chunk + (n[s] % chunk != 0)) : 0u;
        tile[t] = cnt;
        __syncthreads();
        // inclusive Hillis-Steele scan of the tile
        for (uint32_t off = 1; off < kScanBlock; off <<= 1) {
            const uint32_t add = t >= off ? tile[t - off] : 0u;
            __syncthreads();
            tile[t] += add;
            __syncthreads();
        }
        if (s < nsub)
            sub_first[s] = carry + tile[t] - cnt;
        const uint32_t tile_total = tile[kScanBlock - 1];
        __syncthreads();  // every read of the tile done before the next one is written
        carry += tile_total;
    }
    if (t == 0)
        sub_first[nsub] = carry;
}

// Point maps (scale = (hi - lo) 2^-32, base = lo + scale/2, then the FP32
// copies) and work items of each subvolume: block b takes subvolumes b, b +
// grid, ...  The arithmetic is the host's in bfi_eval, operation for operation.

__global__ void __launch_bounds__(256) build_kernel(BuildArgs a)
{
    for (uint32_t s = blockIdx.x; s < a.nsub; s += gridDim.x) {
        const size_t row = static_cast<size_t>(s) * a.d;
        for (int k = threadIdx.x; k < a.d; k += blockDim.x) {
            const double scale = (a.hi[row + k] - a.lo[row + k]) * 0x1p-32;
            const double base = __dadd_rn(a.lo[row + k], 0.5 * scale);
            a.scale64[row + k] = scale;
            a.base64[row + k] = base;
            a.scale32[row + k] = static_cast<float>(scale);
            a.base32[row + k] = static_cast<float>(base);
        }
        const uint32_t i0 = a.sub_first[s], i1 = a.sub_first[s + 1];
        const uint64_t n = a.n[s];
        for (uint32_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
            const uint64_t start = static_cast<uint64_t>(i - i0) * a.chunk;
            const uint64_t cnt = n - start < a.chunk ? n - start : a.chunk;
            a.items[i] = WorkItem{a.params, a.item_rec + static_cast<size_t>(i) * a.rec_len, start,
                                  s, static_cast<uint32_t>(cnt)};
        }
    }
}

__global__ void reset_head_kernel(uint32_t *head)
{
    if (blockIdx.x == 0 && threadIdx.x == 0)
        *head = 0u;
}

// One block per subvolume: its items in consecutive runs, as many as their number
// says (merge_runs) and no matter what is merged beside them, so that a
// subvolume's record does not depend on the rest of its list.  Thread f of a
// wavefront merges field f over a run in item order with Neumaier compensation,
// after moving every item to the smallest shift of the subvolume (factor
// exp(sigma_min - sigma_item) for first-order sums, its square for second-order
// sums; 1 in FP64 form); the runs' sums and compensations then merge in order.
// Items are read kMergeBatch at a time, all loads of a batch issued before its
// arithmetic (the sums keep item order).  What bounds it is latency: a wavefront
// takes about a microsecond per batch, so the wavefronts of a block share the
// runs (launch_merge).  Measured, whole calls: spherical sampler, 2^24 over 64
// shells of up to some thousand items, one wavefront and batches of 8 695 us, by
// the rule 623 us, batches of 16 601 us; 301 uneven leaves with split statistics
// 250 -> 237 us by the longer batches.
constexpr uint32_t kMergeBatch = 16;
constexpr int kMergeMaxFields = BFI_PARTIAL_LEN(BFI_MAX_NX) + 2 * 32;

// One run for a batch of items, four for up to four batches, else sixteen.
__host__ __device__ inline uint32_t merge_runs(uint64_t items)
{
    const uint64_t batches = (items + kMergeBatch - 1) / kMergeBatch;
    return batches <= 1 ? 1 : batches <= 4 ? 4 : 16;
}

struct Compensated {
    double sum = 0.0, comp = 0.0;
    __device__ __forceinline__ void add(double v)
    {
        const double t = sum + v;
        comp += fabs(sum) >= fabs(v) ? (sum - t) + v : (v - t) + sum;
        sum = t;
    }
};

template <int WAVES>
__device__ __forceinline__ void merge_subvolume(const MergeArgs &m, uint32_t s)
{
    extern __shared__ double part[];  // runs x fields x (sum, compensation)
    __shared__ double low[WAVES];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const int nx = m.nx, d = m.d;
    const int rec_len = 4 + 3 * nx;
    const int fields = rec_len + (m.item_split ? 2 * d : 0);
    const uint32_t i0 = m.sub_first[s], i1 = m.sub_first[s + 1];

    // the smallest shift: items over the threads
    double sigma = __builtin_inf();
    for (uint32_t i = i0 + threadIdx.x; i < i1; i += 64 * WAVES)
        sigma = fmin(sigma, m.item_rec[static_cast<size_t>(i) * rec_len + 1]);
    sigma = dev::wave_min(sigma);
    if constexpr (WAVES > 1) {
        if (lane == 0)
            low[wave] = sigma;
        __syncthreads();
#pragma unroll
        for (int g = 0; g < WAVES; ++g)
            sigma = fmin(sigma, low[g]);
    }
    if (i0 == i1)
        sigma = 0.0;

    const uint32_t runs = m.most ? merge_runs(i1 - i0) : 1, per = (i1 - i0 + runs - 1) / runs;
    double *out = m.sub_rec + static_cast<size_t>(s) * rec_len;
    auto store = [&](int f, const Compensated &c) {
        if (f < rec_len)
            out[f] = c.sum + c.comp;
        else
            m.sub_split[static_cast<size_t>(s) * (1 + 2 * d) + 1 + (f - rec_len)] = c.sum + c.comp;
    };
    // tasks: a run of 64 fields each, the runs of the same fields next to each other
    Compensated total;  // one wavefront: over the runs of its fields
    for (uint32_t task = wave; task < runs * ((fields + 63) / 64); task += WAVES) {
        const uint32_t run = task % runs;
        const int f = static_cast<int>(task / runs * 64 + lane);
        if (f >= fields || f == 1)
            continue;
        int order;
        if (f < rec_len)
            order = f == 0 ? 0 : f == 2 ? 1 : f == 3 ? 2 : f < 4 + nx ? 1 : 2;
        else
            order = (f - rec_len) < d ? 1 : 2;
        const uint32_t a = i0 + run * per < i1 ? i0 + run * per : i1;
        const uint32_t b = i1 - a < per ? i1 : a + per;
        Compensated c;
        for (uint32_t i = a; i < b; i += kMergeBatch) {
            double vb[kMergeBatch], sb[kMergeBatch];
#pragma unroll
            for (uint32_t j = 0; j < kMergeBatch; ++j) {
                if (i + j < b) {
                    const double *rec = m.item_rec + static_cast<size_t>(i + j) * rec_len;
                    vb[j] = f < rec_len ? rec[f]
                                        : m.item_split[static_cast<size_t>(i + j) * (2 * d) +
                                                       (f - rec_len)];
                    sb[j] = rec[1];
                }
            }
#pragma unroll
            for (uint32_t j = 0; j < kMergeBatch; ++j) {
                if (i + j < b) {
                    double v = vb[j];
                    const double by = sigma - sb[j];
                    if (order != 0 && by != 0.0) {  // (a factor of 1 left out)
                        const double f1 = exp(by);
                        v *= order == 1 ? f1 : f1 * f1;
                    }
                    c.add(v);
                }
            }
        }
        if (runs == 1) {
            store(f, c);
        } else if constexpr (WAVES > 1) {
            double *p = part + (static_cast<size_t>(run) * fields + f) * 2;
            p[0] = c.sum;
            p[1] = c.comp;
        } else {
            if (run == 0)
                total = Compensated();
            total.add(c.sum);
            total.add(c.comp);
            if (run + 1 == runs)
                store(f, total);
        }
    }
    if (WAVES > 1 && runs > 1) {
        __syncthreads();
        for (int f = static_cast<int>(threadIdx.x); f < fields; f += 64 * WAVES) {
            if (f == 1)
                continue;
            Compensated c;
#pragma unroll 4
            for (uint32_t run = 0; run < runs; ++run) {
                const double *p = part + (static_cast<size_t>(run) * fields + f) * 2;
                c.add(p[0]);
                c.add(p[1]);
            }
            store(f, c);
        }
    }
    if (threadIdx.x == 0) {
        out[1] = sigma;
        if (m.sub_split)
            m.sub_split[static_cast<size_t>(s) * (1 + 2 * d)] = sigma;
    }
}

template <int WAVES>
__global__ void __launch_bounds__(64 * WAVES) merge_kernel(MergeArgs m)
{
    merge_subvolume<WAVES>(m, blockIdx.x);
}

// Several lists in one launch, their arguments in the kernel's own: list r's
// subvolumes are blocks first[r] .. first[r + 1] - 1.  A burst of 16 served
// requests (2^16 .. 2^22 evaluations) ended on 15 merges and as many copies one
// after another, 22 us a pair, most of it between the launches: 1.18 .. 1.22 ->
// 1.06 .. 1.13 ms for the burst with one launch that writes the records to host
// memory.
constexpr uint32_t kMergeLists = 16;
struct MergeLists {
    MergeArgs list[kMergeLists];
    uint32_t first[kMergeLists + 1];
    uint32_t n;
};

template <int WAVES>
__global__ void __launch_bounds__(64 * WAVES) merge_lists_kernel(MergeLists l)
{
    uint32_t r = 0;
    while (r + 1 < l.n && blockIdx.x >= l.first[r + 1])
        ++r;
    merge_subvolume<WAVES>(l.list[r], blockIdx.x - l.first[r]);
}

// The N-sphere integrand of the paper's examples (section 3, Listings 1 and 2):
// half the volume of the unit (dim+1)-ball as the integral of sqrt(1 - |x|^2).
// Same points as the lattice kernels (Philox words, fma map); FP64 sums of f and
// f^2, and of both over the upper half of the box along each dimension.

// Square root of a in [2^-53, 1]: Goldschmidt's coupled iteration for sqrt(a) and
// 1 / (2 sqrt(a)) from the hardware's reciprocal root, then one correction by the
// exact residual a - g^2.  No range to scale or special value to keep, which
// is half of what the general square root does.
__device__ __forceinline__ double sqrt_unit(double a)
{
    const double y = __builtin_amdgcn_rsq(a);
    double g = a * y, h = 0.5 * y;
    double e = __fma_rn(-h, g, 0.5);
    g = __fma_rn(g, e, g);
    h = __fma_rn(h, e, h);
    e = __fma_rn(-g, g, a);
    g = __fma_rn(e, h, g);
    e = __fma_rn(-g, g, a);
    return __fma_rn(e, h, g);
}

// One kernel per dimension: the loop over coordinates, its Philox blocks and the
// 2 + 2 DIM sums are unrolled, the point map stays in registers (offsets
// scalar, scales in vector registers), and the item's share of Philox is
// computed once.  What bounds it is instruction issue.  A kernel for any
// dimension up to 16 kept 34 sums whatever the dimension, read the map from
// memory for every coordinate and masked the unused ones: a call of 3.2e7
// samples in 6 dimensions took 338 us with it, 201 us with this (164 with the
// block launch and merge batches of today; its items are the launch shape's).
template <int DIM>
__global__ void __launch_bounds__(256) nsphere_kernel(McArgs a)
{
    constexpr int kBlock = 256, kWaves = kBlock / 64, NB = (DIM + 3) / 4, NF = 2 + 2 * DIM;
    __shared__ double red[kWaves][NF];
    __shared__ uint32_t next_item;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;

    uint32_t it;
    if (a.queue_head) {
        if (tid == 0)
            next_item = atomicAdd(a.queue_head, 1u);
        __syncthreads();
        it = __builtin_amdgcn_readfirstlane(next_item);
    } else {
        it = blockIdx.x;
    }
    while (it < a.nitems) {
        const WorkItem wi = dev::load_uniform(a.items + it);
        const EvalParams P = dev::load_uniform(wi.params);
        const uint64_t id = P.ids[wi.sub];
        const uint64_t first_index = P.offsets[wi.sub] + wi.start;
        const uint32_t id_lo = static_cast<uint32_t>(id), id_hi = static_cast<uint32_t>(id >> 32);
        const double *base_g = P.base64 + static_cast<size_t>(wi.sub) * DIM;
        const double *scale_g = P.scale64 + static_cast<size_t>(wi.sub) * DIM;
        double base[DIM], scale[DIM];
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            base[k] = dev::load_uniform(base_g + k);
            scale[k] = scale_g[k];
        }
        double acc[NF];
#pragma unroll
        for (int i = 0; i < NF; ++i)
            acc[i] = 0.0;

        // counters q = index NB + block; where they keep one upper word, part of
        // Philox is the item's (PhiloxItem)
        const uint64_t q_first = first_index * NB;
        const uint64_t q_end = (first_index + wi.count) * NB;  // host: no wrap
        const dev::PhiloxItem pitem = dev::philox_item(static_cast<uint32_t>(q_first >> 32), id_lo,
                                                       id_hi, P.seed_lo, P.seed_hi);
        auto samples = [&](auto same_hi_tag) {
            constexpr bool kSameHi = decltype(same_hi_tag)::value;
            for (uint32_t k = 0; k < a.samples_per_thread; ++k) {
                const uint32_t local = k * kBlock + tid;
                if (local >= wi.count)
                    break;
                const uint64_t q0 = q_first + static_cast<uint64_t>(local) * NB;
                uint32_t w[4 * NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    if constexpr (kSameHi)
                        dev::philox_block_item(static_cast<uint32_t>(q0) + j, pitem, w + 4 * j);
                    else
                        dev::philox_block(q0 + j, id_lo, id_hi, P.seed_lo, P.seed_hi, w + 4 * j);
                }
                double r2 = 0.0;
#pragma unroll
                for (int kk = 0; kk < DIM; ++kk) {
                    const double u = dev::map_word(w[kk], scale[kk], base[kk]);
                    r2 = __fma_rn(u, u, r2);
                }
                // outside the ball every term is 0: a wavefront wholly outside
                // (most of them from 10 dimensions on) skips the sums
                if (r2 < 1.0) {
                    const double f = sqrt_unit(1.0 - r2);
                    const double f2 = f * f;
                    acc[0] += f;
                    acc[1] += f2;
#pragma unroll
                    for (int kk = 0; kk < DIM; ++kk) {
                        // the half as 0 or 1: the sum gains f or exactly nothing
                        const double up = static_cast<double>(w[kk] >> 31);
                        acc[2 + kk] = __fma_rn(up, f, acc[2 + kk]);
                        acc[2 + DIM + kk] = __fma_rn(up, f2, acc[2 + DIM + kk]);
                    }
                }
            }
        };
        if ((q_first >> 32) == ((q_end - 1) >> 32))
            samples(std::true_type{});
        else
            samples(std::false_type{});

        dev::wave_sums<NF>([&](int i) { return acc[i]; }, red[wave], lane);
        __syncthreads();
        if (tid < NF) {
            double total = 0.0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w)
                total += red[w][tid];
            if (tid < 2)
                wi.rec[2 + tid] = total;
            else
                a.item_split[static_cast<size_t>(wi.rec - a.item_rec) / BFI_PARTIAL_LEN(0) * (2 * DIM) +
                             (tid - 2)] = total;
        }
        if (tid == 0) {
            wi.rec[0] = static_cast<double>(wi.count);
            wi.rec[1] = 0.0;
        }
        if (!a.queue_head)
            break;
        __syncthreads();
        if (tid == 0)
            next_item = atomicAdd(a.queue_head, 1u);
        __syncthreads();
        it = __builtin_amdgcn_readfirstlane(next_item);
    }
}

// f(DIM as a compile-time constant) for the run-time dimension.
template <class F>
hipError_t by_dim(int dim, F &&f)
{
    switch (dim) {
#define BFI_DIM(D) \
    case D:        \
        return f(std::integral_constant<int, D>{});
        BFI_DIM(1) BFI_DIM(2) BFI_DIM(3) BFI_DIM(4) BFI_DIM(5) BFI_DIM(6) BFI_DIM(7) BFI_DIM(8)
        BFI_DIM(9) BFI_DIM(10) BFI_DIM(11) BFI_DIM(12) BFI_DIM(13) BFI_DIM(14) BFI_DIM(15)
        BFI_DIM(16)
#undef BFI_DIM
    default:
        return hipErrorInvalidValue;
    }
}
static_assert(kMaxNsphereDim == 16, "one kernel per dimension");

__global__ void __launch_bounds__(256) debug_points_kernel(DebugPointArgs a)
{
    const uint64_t i = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= a.n)
        return;
    const int d = a.d;
    const int nb = (d + 3) / 4;
    const uint64_t q0 = a.index[i] * static_cast<uint64_t>(nb);
    const uint32_t id_lo = static_cast<uint32_t>(a.id), id_hi = static_cast<uint32_t>(a.id >> 32);
    for (int j = 0; j < nb; ++j) {
        uint32_t blk[4];
        dev::philox_block(q0 + j, id_lo, id_hi, a.seed_lo, a.seed_hi, blk);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int k = 4 * j + t;
            if (k >= d)
                break;
            a.out[i * d + k] =
                a.prec != kFP32Shifted
                    ? dev::map_word(blk[t], a.scale64[k], a.base64[k])
                    : static_cast<double>(dev::map_word(blk[t], a.scale32[k], a.base32[k]));
        }
    }
}

}  // namespace

hipError_t launch_build_items(const BuildArgs &args, hipStream_t stream)
{
    if (args.nsub == 0)
        return hipSuccess;
    hipLaunchKernelGGL(first_items_kernel, dim3(1), dim3(kScanBlock), 0, stream, args.n, args.nsub,
                       args.chunk, args.sub_first);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    const uint32_t grid = args.nsub < 4096 ? args.nsub : 4096u;
    hipLaunchKernelGGL(build_kernel, dim3(grid), dim3(256), 0, stream, args);
    return hipGetLastError();
}

hipError_t launch_reset_head(uint32_t *head, hipStream_t stream)
{
    hipLaunchKernelGGL(reset_head_kernel, dim3(1), dim3(64), 0, stream, head);
    return hipGetLastError();
}

hipError_t launch_nsphere(const NsphereArgs &args, uint32_t grid, hipStream_t stream)
{
    if (!args.mc.item_split)
        return hipErrorInvalidValue;
    if (grid == 0)
        return hipSuccess;
    return by_dim(args.dim, [&](auto dim) {
        hipLaunchKernelGGL((nsphere_kernel<decltype(dim)::value>), dim3(grid), dim3(256), 0, stream,
                           args.mc);
        return hipGetLastError();
    });
}

hipError_t nsphere_kernel_info(int dim, KernelInfo *info)
{
    return by_dim(dim, [&](auto tag) {
        int blocks = 0;
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &blocks, nsphere_kernel<decltype(tag)::value>, 256, 0);
        info->blocks_per_cu = blocks;
        return e;
    });
}

namespace {

int merge_fields(const MergeArgs &args)
{
    return 4 + 3 * args.nx + (args.item_split ? 2 * args.d : 0);
}

// Wavefronts per subvolume: one for one batch of items, four for up to four,
// else sixteen.  The largest subvolume decides while the blocks fit the chip
// together (2048 of up to 16 wavefronts are four rounds); of longer lists the
// average does, whose few large subvolumes end beside the others; and lists too long
// for a launch of so many take fewer.  (The runs, and with them the sums, do not
// depend on it.)
int merge_waves(const MergeArgs &args)
{
    if (!args.most)
        return 1;
    const uint64_t items =
        args.nsub <= 2048 ? args.most : static_cast<uint64_t>(args.nitems) / args.nsub;
    return fitting_waves(args.nsub, static_cast<int>(merge_runs(items)));
}

// LDS that the runs' sums of the list's largest subvolume take.
uint32_t merge_lds(const MergeArgs &args, int waves)
{
    return waves == 1 ? 0 : merge_runs(args.most) * merge_fields(args) * 2 * sizeof(double);
}

}  // namespace

hipError_t launch_merge(const MergeArgs &args, hipStream_t stream)
{
    if (args.nsub == 0)
        return hipSuccess;
    if (merge_fields(args) > kMergeMaxFields)
        return hipErrorInvalidValue;
    const int waves = merge_waves(args);
    const uint32_t lds = merge_lds(args, waves);
    const dim3 grid(args.nsub), block(64 * waves);
    if (waves == 1)
        hipLaunchKernelGGL(merge_kernel<1>, grid, block, lds, stream, args);
    else if (waves == 4)
        hipLaunchKernelGGL(merge_kernel<4>, grid, block, lds, stream, args);
    else
        hipLaunchKernelGGL(merge_kernel<16>, grid, block, lds, stream, args);
    return hipGetLastError();
}

hipError_t launch_merges(const MergeArgs *args, size_t n, hipStream_t stream)
{
    for (const int waves : {1, 4, 16}) {
        MergeLists l{};
        uint32_t lds = 0;
        auto flush = [&]() -> hipError_t {
            if (l.n == 0)
                return hipSuccess;
            const dim3 grid(l.first[l.n]), block(64 * waves);
            if (waves == 1)
                hipLaunchKernelGGL(merge_lists_kernel<1>, grid, block, lds, stream, l);
            else if (waves == 4)
                hipLaunchKernelGGL(merge_lists_kernel<4>, grid, block, lds, stream, l);
            else
                hipLaunchKernelGGL(merge_lists_kernel<16>, grid, block, lds, stream, l);
            l.n = 0;
            lds = 0;
            return hipGetLastError();
        };
        for (size_t i = 0; i < n; ++i) {
            const MergeArgs &m = args[i];
            if (m.nsub == 0 || merge_waves(m) != waves)
                continue;
            if (merge_fields(m) > kMergeMaxFields)
                return hipErrorInvalidValue;
            const uint64_t most_blocks = kMaxThreads / (64 * waves);
            if (l.n == kMergeLists || (l.n && uint64_t(l.first[l.n]) + m.nsub > most_blocks)) {
                const hipError_t e = flush();
                if (e != hipSuccess)
                    return e;
            }
            l.list[l.n] = m;
            l.first[l.n + 1] = l.first[l.n] + m.nsub;
            ++l.n;
            lds = std::max(lds, merge_lds(m, waves));
        }
        const hipError_t e = flush();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

hipError_t launch_debug_points(const DebugPointArgs &args, hipStream_t stream)
{
    const unsigned grid = static_cast<unsigned>((args.n + 255) / 256);
    if (grid == 0)
        return hipSuccess;
    hipLaunchKernelGGL(debug_points_kernel, dim3(grid), dim3(256), 0, stream, args);
    return hipGetLastError();
}

}  // namespace bfi
