// Leaf records of an adaptive run in device memory: the fold of a round's
// records into the leaves and the analysis of every leaf (the finalize's two
// passes over the records, paper section 2's estimators of Z and C(r) with
// their delta-method errors, and the refinement's split choice, section 3).
// The arithmetic is the host's (finalize_records, merge_shifted, split_choice)
// operation for operation, without contraction into fused multiply-adds; only
// the order of the sums over leaves differs (tree sums per wavefront, groups of
// wavefronts in order with Neumaier compensation).
#include "device.hpp"
#include "launch_limits.h"

#pragma clang fp contract(off)

namespace bfi {
namespace {

// Field classes of a record: 0 the count, 1 the shift, 2 first-order sums
// (scaled by the shift factor), 3 second-order sums (by its square).
__device__ __forceinline__ int rec_class(int f, int nx)
{
    return f == 0 ? 0 : f == 1 ? 1 : f == 2 ? 2 : f == 3 ? 3 : f < 4 + nx ? 2 : 3;
}
// Split statistics: the shift, then d first-order and d second-order sums.
__device__ __forceinline__ int split_class(int f, int d)
{
    return f == 0 ? 1 : f <= d ? 2 : 3;
}

// Field value a merged with b (disjoint samples of one leaf, shifts sa and sb),
// both moved to the smaller shift; counts add, a shift becomes the smaller one.
__device__ __forceinline__ double merge_field(double a, double b, double sa, double sb, int cls)
{
    const double sig = sb < sa ? sb : sa;
    if (cls == 1)
        return sig;
    if (cls == 0)
        return a + b;
    const double fa = exp(sig - sa), fb = exp(sig - sb);
    return cls == 2 ? fa * a + fb * b : fa * fa * a + fb * fb * b;
}

// One wavefront per entry, a lane per field (every entry has a leaf of its own),
// so that an entry's records are read and written in whole lines; with a thread
// per entry the rows of 34 to 41 doubles went through 64 lines at a time and a
// record in scratch memory.  What bounds it is latency.  Measured, 512 to 1024
// entries of 10x2: 26 us with a thread per entry, 4.3 us with a wavefront.
constexpr int kFoldBlock = 256;

__global__ void __launch_bounds__(kFoldBlock) fold_kernel(FoldArgs a)
{
    const uint32_t i = blockIdx.x * (kFoldBlock / 64) + (threadIdx.x >> 6);
    const int lane = static_cast<int>(threadIdx.x & 63u);
    if (i >= a.count)
        return;
    const FoldEntry en = a.entries[i];
    const int nx = a.nx, d = a.d, rec_len = 4 + 3 * nx, split_len = 1 + 2 * d;
    const bool has_w = en.wpos >= 0, has_p = en.opos >= 0;
    const double *w = a.with_rec + static_cast<size_t>(has_w ? en.wpos : 0) * rec_len;
    const double *sp = a.with_split + static_cast<size_t>(has_w ? en.wpos : 0) * split_len;
    const double *p = a.plain_rec + static_cast<size_t>(has_p ? en.opos : 0) * rec_len;
    double *lrec = a.leaf_rec + static_cast<size_t>(en.dst) * rec_len;
    double *lsplit = a.leaf_split + static_cast<size_t>(en.dst) * split_len;
    double *lbase = a.leaf_base + static_cast<size_t>(en.dst) * rec_len;
    // counts and shifts first: the stores below replace the leaf's
    const double wn = has_w ? w[0] : 0.0, ws = has_w ? w[1] : 0.0;
    const double pn = has_p ? p[0] : 0.0, ps = has_p ? p[1] : 0.0;
    // the record of the entry's samples from its two parts (either may be absent):
    // the first part, then the second merged in (a part with no samples adds
    // nothing)
    const bool only_w = !has_p || pn == 0, only_p = !only_w && wn == 0;
    auto part = [&](int f) -> double {
        const double x = has_w ? w[f] : 0.0;
        if (only_w)
            return x;
        return only_p ? p[f] : merge_field(x, p[f], ws, ps, rec_class(f, nx));
    };
    if (en.kind == 0) {
        const double rs = only_w ? ws : only_p ? ps : ps < ws ? ps : ws;
        const double ls = lrec[1], ss = lsplit[0], bs = lbase[1], sps = has_w ? sp[0] : 0.0;
        for (int f = lane; f < rec_len; f += 64)
            lrec[f] = merge_field(lrec[f], part(f), ls, rs, rec_class(f, nx));
        if (has_w && wn > 0) {
            // the continuation still lies below the split statistics' cut
            for (int f = lane; f < split_len; f += 64)
                lsplit[f] = merge_field(lsplit[f], sp[f], ss, sps, split_class(f, d));
            for (int f = lane; f < rec_len; f += 64)
                lbase[f] = merge_field(lbase[f], w[f], bs, ws, rec_class(f, nx));
        }
        return;
    }
    for (int f = lane; f < rec_len; f += 64) {
        lrec[f] = part(f);
        lbase[f] = has_w ? w[f] : 0.0;
    }
    for (int f = lane; f < split_len; f += 64)
        lsplit[f] = has_w ? sp[f] : 0.0;
    if (lane == 0)
        a.leaf_vol[en.dst] = en.vol;
}

// ---- analysis ----------------------------------------------------------------

// Leaves are summed in fixed groups whatever the launch: 64 leaves by a
// wavefront's butterfly, 16 of those sums in order (a group of kAnalysisBlock
// leaves), the groups in order with Neumaier compensation.  A block holds four
// wavefronts, so that a few thousand leaves use more than a few CUs; what bounds
// each of these kernels at such sizes is latency.  Measured, 1024 to 2048 leaves
// of 10x2, blocks of 1024 threads with LDS permutes and the split choices in the
// same threads -> this: first pass 11.5 -> 6.1 us, second pass and choices 36
// -> 6.1 us.
constexpr int kPassBlock = 256;
constexpr int kGroupWaves = kAnalysisBlock / 64;

// scratch layout (doubles): per group the smallest shift, then per wavefront the
// first pass's 4 + nx sums and the second pass's nx sums; then [sigma, z, 1/z^2,
// C(r)]
__device__ __forceinline__ size_t ngroups_of(uint32_t count)
{
    return (static_cast<size_t>(count) + kAnalysisBlock - 1) / kAnalysisBlock;
}
__device__ __forceinline__ size_t nwaves_of(uint32_t count)
{
    return (static_cast<size_t>(count) + 63) / 64;
}
struct Scratch {
    double *shift, *first, *second, *scal;
    __device__ __forceinline__ explicit Scratch(const LeafAnalysisArgs &a)
    {
        const size_t ng = ngroups_of(a.count), nw = nwaves_of(a.count);
        shift = a.scratch;
        first = shift + ng;
        second = first + nw * (4 + a.nx);
        scal = second + nw * a.nx;
    }
};

__global__ void __launch_bounds__(kAnalysisBlock) shift_kernel(LeafAnalysisArgs a)
{
    __shared__ double m[kAnalysisBlock];
    const uint32_t s = blockIdx.x * kAnalysisBlock + threadIdx.x;
    const int rec_len = 4 + 3 * a.nx;
    m[threadIdx.x] = s < a.count ? a.rec[static_cast<size_t>(s) * rec_len + 1] : __builtin_inf();
    __syncthreads();
    for (int k = kAnalysisBlock / 2; k > 0; k >>= 1) {
        if (threadIdx.x < k) {
            const double x = m[threadIdx.x + k];
            // the smaller of the two, a NaN never taken (the host's std::min)
            if (x < m[threadIdx.x])
                m[threadIdx.x] = x;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0)
        a.scratch[blockIdx.x] = m[0];
}

// The smallest shift of the groups; with DIRECT of the leaves themselves (short
// lists: one launch less).
template <bool DIRECT>
__global__ void __launch_bounds__(kAnalysisBlock) shift_reduce_kernel(LeafAnalysisArgs a)
{
    __shared__ double m[kAnalysisBlock];
    const size_t n = DIRECT ? a.count : ngroups_of(a.count);
    const int rec_len = 4 + 3 * a.nx;
    double sig = __builtin_inf();
    for (size_t b = threadIdx.x; b < n; b += kAnalysisBlock) {
        const double x = DIRECT ? a.rec[b * rec_len + 1] : a.scratch[b];
        if (x < sig)
            sig = x;
    }
    m[threadIdx.x] = sig;
    __syncthreads();
    for (int k = kAnalysisBlock / 2; k > 0; k >>= 1) {
        if (threadIdx.x < k && m[threadIdx.x + k] < m[threadIdx.x])
            m[threadIdx.x] = m[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        Scratch(a).scal[0] = m[0];
        a.out_totals[0] = m[0];
    }
}
constexpr uint32_t kDirectShift = 8 * kAnalysisBlock;

__global__ void __launch_bounds__(kPassBlock) first_pass_kernel(LeafAnalysisArgs a)
{
    const Scratch sc(a);
    const int nx = a.nx, rec_len = 4 + 3 * nx, nt = 4 + nx;
    const double sig = sc.scal[0];
    const uint32_t s = blockIdx.x * kPassBlock + threadIdx.x;
    const int lane = static_cast<int>(threadIdx.x & 63u);
    const bool on = s < a.count;
    const double *rec = a.rec + static_cast<size_t>(on ? s : 0) * rec_len;
    double n = 1.0, vol = 0.0, aa = 0.0, sw = 0.0, sw2 = 0.0;
    if (on) {
        n = rec[0];
        vol = a.vol[s];
        aa = exp(sig - rec[1]);
        sw = aa * rec[2];
        sw2 = aa * aa * rec[3];
    }
    // the finalize's sums: Z, Var Z, squared weights, samples, N(r); lane j keeps
    // sum j
    double mine = 0.0;
    for (int j = 0; j < nt; ++j) {
        double t = 0.0;
        if (on) {
            if (j == 0)
                t = vol * sw / n;
            else if (j == 1)
                t = vol * vol * (sw2 - sw * sw / n) / (n * (n - 1.0));
            else if (j == 2)
                t = (vol / n) * (vol / n) * sw2;
            else if (j == 3)
                t = n;
            else
                t = vol * aa * rec[j] / n;
        }
        const double v = dev::wave_sum(t);
        mine = lane == j ? v : mine;
    }
    const size_t wave = s >> 6;
    if (lane < nt && wave < nwaves_of(a.count))
        sc.first[wave * nt + lane] = mine;
}

// Totals of `stride` sums from the wavefronts' (nw x stride): groups of
// kGroupWaves in order, the groups with Neumaier compensation.  The block's 16
// wavefronts take a group each, all its loads ahead of the additions, then
// thread j adds the 16 groups' sums; total j is returned to thread j.
constexpr int kMaxSums = 4 + kMaxAnalysisNx;
__device__ double ordered_total(const double *part, size_t nw, int stride)
{
    __shared__ double sums[kGroupWaves][kMaxSums];
    const int j = static_cast<int>(threadIdx.x & 63u);
    const size_t mine = threadIdx.x >> 6, ng = (nw + kGroupWaves - 1) / kGroupWaves;
    double sum = 0.0, comp = 0.0;
    for (size_t g0 = 0; g0 < ng; g0 += kGroupWaves) {
        const size_t w0 = (g0 + mine) * kGroupWaves;
        if (j < stride && w0 < nw) {
            double x[kGroupWaves];
#pragma unroll
            for (int k = 0; k < kGroupWaves; ++k)
                x[k] = w0 + k < nw ? part[(w0 + k) * stride + j] : 0.0;
            double t = 0.0;
#pragma unroll
            for (int k = 0; k < kGroupWaves; ++k)
                t += x[k];
            sums[mine][j] = t;
        }
        __syncthreads();
        if (threadIdx.x < static_cast<uint32_t>(stride)) {
            for (size_t k = 0; k < kGroupWaves && g0 + k < ng; ++k) {
                const double x = sums[k][j];
                const double t = sum + x;
                comp += fabs(sum) >= fabs(x) ? (sum - t) + x : (x - t) + sum;
                sum = t;
            }
        }
        __syncthreads();
    }
    return sum + comp;
}

__global__ void __launch_bounds__(kAnalysisBlock) first_reduce_kernel(LeafAnalysisArgs a)
{
    __shared__ double tot[kMaxSums];
    const Scratch sc(a);
    const int nx = a.nx, nt = 4 + nx, j = static_cast<int>(threadIdx.x);
    const double t = ordered_total(sc.first, nwaves_of(a.count), nt);
    if (j < nt) {
        tot[j] = t;
        a.out_totals[1 + j] = t;
    }
    __syncthreads();
    const double z = tot[0];
    if (j == 0) {
        sc.scal[1] = z;
        sc.scal[2] = z > 0 ? 1.0 / (z * z) : 0.0;
    }
    if (j < nx)
        sc.scal[3 + j] = tot[4 + j] / z;
}

// A leaf's split choice from its split statistics and the record of the samples
// they cover (the host's split_choice): lane j of half a wavefront takes
// dimension j, the smallest spread wins, the lower dimension among equals.
__device__ void split_choice(const LeafAnalysisArgs &a, uint32_t s, int j)
{
    const int d = a.d;
    const double *sp = a.split + static_cast<size_t>(s) * (1 + 2 * d);
    const double *base = a.base + static_cast<size_t>(s) * (4 + 3 * a.nx);
    const double S = base[2], Q = base[3], m = base[0], half = 0.5 * m;
    double best = __builtin_inf();
    if (j < d) {
        const double su = sp[1 + j], qu = sp[1 + d + j];
        const double sl = S - su, ql = Q - qu;
        const double vu0 = qu / half - (su / half) * (su / half);
        const double vl0 = ql / half - (sl / half) * (sl / half);
        const double vu = vu0 < 0.0 ? 0.0 : vu0, vl = vl0 < 0.0 ? 0.0 : vl0;
        const double sj = sqrt(vu) + sqrt(vl);
        best = sj < best ? sj : best;  // (a NaN never wins)
    }
    int best_j = j;
    for (int off = 16; off >= 1; off >>= 1) {
        const double x = __shfl_xor(best, off, 32);
        const int k = __shfl_xor(best_j, off, 32);
        if (x < best || (x == best && k < best_j)) {
            best = x;
            best_j = k;
        }
    }
    if (j == 0) {
        const double v = Q / m - (S / m) * (S / m);
        const double sigma = sqrt(v < 0.0 ? 0.0 : v);
        a.best[s] = best_j;
        a.gain[s] = sigma > 0 ? best / (2.0 * sigma) : 1.0;
    }
}

// The first `sum_blocks` blocks sum the second pass, a thread per leaf; the
// others make the split choices from leaf `first` on, half a wavefront per leaf.
__global__ void __launch_bounds__(kPassBlock) second_pass_kernel(LeafAnalysisArgs a,
                                                                 uint32_t sum_blocks,
                                                                 uint32_t first)
{
    const int lane = static_cast<int>(threadIdx.x & 63u);
    if (blockIdx.x >= sum_blocks) {
        const uint32_t s =
            first + (blockIdx.x - sum_blocks) * (kPassBlock / 32) + (threadIdx.x >> 5);
        if (s < a.count)
            split_choice(a, s, lane & 31);
        return;
    }
    const Scratch sc(a);
    const int nx = a.nx, rec_len = 4 + 3 * nx;
    const double sig = sc.scal[0], inv_z2 = sc.scal[2];
    const uint32_t s = blockIdx.x * kPassBlock + threadIdx.x;
    const bool on = s < a.count;
    const double *rec = a.rec + static_cast<size_t>(on ? s : 0) * rec_len;
    double n = 1.0, v2 = 0.0, nn = 1.0, aa = 0.0, a2 = 0.0, sw = 0.0, var_z = 0.0;
    if (on) {
        n = rec[0];
        const double vol = a.vol[s];
        v2 = vol * vol;
        nn = n * (n - 1.0);
        aa = exp(sig - rec[1]);
        a2 = aa * aa;
        sw = aa * rec[2];
        const double sw2 = a2 * rec[3];
        var_z = v2 * (sw2 - sw * sw / n) / nn;
    }
    double e = 0.0, mine = 0.0;
    for (int r = 0; r < nx; ++r) {
        double t = 0.0;
        if (on) {
            const double C = sc.scal[3 + r];
            const double spw = aa * rec[4 + r], spw2 = a2 * rec[4 + nx + r],
                         spww = a2 * rec[4 + 2 * nx + r];
            const double var_n = v2 * (spw2 - spw * spw / n) / nn;
            const double cov = v2 * (spww - spw * sw / n) / nn;
            t = var_n - 2.0 * C * cov + C * C * var_z;
            e += t;
        }
        const double v = dev::wave_sum(t);
        mine = lane == r ? v : mine;
    }
    const size_t wave = s >> 6;
    if (lane < nx && wave < nwaves_of(a.count))
        sc.second[wave * nx + lane] = mine;
    if (!on)
        return;
    // the host's max(e, 0) / Z^2, read back as a contribution (NaN counts 0)
    const double c = (e < 0.0 ? 0.0 : e) * inv_z2;
    a.e[s] = c >= 0.0 ? c : 0.0;
}

__global__ void __launch_bounds__(kAnalysisBlock) second_reduce_kernel(LeafAnalysisArgs a)
{
    const double t = ordered_total(Scratch(a).second, nwaves_of(a.count), a.nx);
    if (static_cast<int>(threadIdx.x) < a.nx)
        a.out_totals[1 + 4 + a.nx + threadIdx.x] = t;
}

}  // namespace

hipError_t launch_fold(const FoldArgs &args, hipStream_t stream)
{
    if (args.count == 0)
        return hipSuccess;
    if (args.nx < 1 || args.nx > kMaxAnalysisNx || args.d < 1 || args.d > 32)
        return hipErrorInvalidValue;
    return for_slices(args.count, kFoldSlice, hipSuccess, [&](uint32_t first, uint32_t n) {
        FoldArgs part = args;
        part.entries += first;
        part.count = n;
        const uint32_t per_block = kFoldBlock / 64;
        hipLaunchKernelGGL(fold_kernel, dim3((n + per_block - 1) / per_block), dim3(kFoldBlock), 0,
                           stream, part);
        return hipGetLastError();
    });
}

size_t analysis_scratch_doubles(uint32_t count, int nx)
{
    const size_t ng = (static_cast<size_t>(count) + kAnalysisBlock - 1) / kAnalysisBlock;
    const size_t nw = (static_cast<size_t>(count) + 63) / 64;
    return ng + nw * (4 + 2 * static_cast<size_t>(nx)) + 3 + static_cast<size_t>(nx);
}

hipError_t launch_leaf_analysis(const LeafAnalysisArgs &args, hipStream_t stream)
{
    if (args.count == 0 || args.count > kMaxLeaves || args.nx < 1 || args.nx > kMaxAnalysisNx ||
        args.d < 1 || args.d > 32)
        return hipErrorInvalidValue;
    auto blocks = [&](size_t threads, size_t block) {
        return static_cast<uint32_t>((threads + block - 1) / block);
    };
    const size_t count = args.count;
    if (args.count <= kDirectShift) {
        hipLaunchKernelGGL(shift_reduce_kernel<true>, dim3(1), dim3(kAnalysisBlock), 0, stream, args);
    } else {
        hipLaunchKernelGGL(shift_kernel, dim3(blocks(count, kAnalysisBlock)), dim3(kAnalysisBlock), 0,
                           stream, args);
        hipLaunchKernelGGL(shift_reduce_kernel<false>, dim3(1), dim3(kAnalysisBlock), 0, stream,
                           args);
    }
    const uint32_t sums = blocks(count, kPassBlock);
    hipLaunchKernelGGL(first_pass_kernel, dim3(sums), dim3(kPassBlock), 0, stream, args);
    hipLaunchKernelGGL(first_reduce_kernel, dim3(1), dim3(kAnalysisBlock), 0, stream, args);
    // sums and choices in one launch, or apart where that is too long for one
    const uint32_t beside = args.count <= kChoiceSlice ? sums : 0;
    if (!beside)
        hipLaunchKernelGGL(second_pass_kernel, dim3(sums), dim3(kPassBlock), 0, stream, args, sums,
                           0u);
    const hipError_t e =
        for_slices(args.count, kChoiceSlice, hipSuccess, [&](uint32_t first, uint32_t n) {
            hipLaunchKernelGGL(second_pass_kernel,
                               dim3(beside + blocks(32 * static_cast<size_t>(n), kPassBlock)),
                               dim3(kPassBlock), 0, stream, args, beside, first);
            return hipGetLastError();
        });
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(second_reduce_kernel, dim3(1), dim3(kAnalysisBlock), 0, stream, args);
    return hipGetLastError();
}

}  // namespace bfi
