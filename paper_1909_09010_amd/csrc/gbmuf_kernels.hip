// gbmuf_kernels.hip -- gfx950 kernels of libgbmuf besides the fused one (gbmuf_sync.hip): the neighbour
// sampler, the final model average and the placement change of Algorithm 1 (arXiv 1909.09010); and the
// launches of all of them.
#include "gbmuf_device.h"

#include "../../include/gbmuf.h"

#include <algorithm>

#pragma clang fp contract(off)

namespace gbmuf {

namespace {

// ---------------------------------------------------------------------------------------
// Neighbour sampler: one thread per (component, worker).  Up to kFewDraws neighbours are drawn in
// registers; for more, the thread's copy of the candidate list lives in LDS, interleaved so that
// thread t owns words t, t+TB, t+2TB...
// ---------------------------------------------------------------------------------------
struct LdsPerm {
    int32_t *base;
    int stride;
    __device__ int32_t &operator()(int32_t x) const { return base[x * stride]; }
};

__global__ void sample_kernel(SampleArgs a)
{
    extern __shared__ int32_t perm_lds[];
    const int tb = blockDim.x;
    const int64_t idx = static_cast<int64_t>(blockIdx.x) * tb + threadIdx.x;
    if (idx >= a.pairs) return;                       // no barrier below
    const int64_t pair = a.first_pair + idx;
    const uint32_t comp = static_cast<uint32_t>(pair / a.K);
    const int32_t w = static_cast<int32_t>(pair - static_cast<int64_t>(comp) * a.K);
    if (a.check_periods && a.step % static_cast<uint64_t>(a.comp[comp].period) != 0) return;   // not due
    const int32_t q = a.mixed ? a.comp[comp].q : a.q;
    const DrawKey key{a.key0, a.key1, a.round0, a.round1};
    int32_t *row = a.out + pair * a.width;
    if (a.q <= kFewDraws) {                           // a.q: the largest of all components
        int32_t v[8], picked[kFewDraws];
        draw_few(picked, a.K, a.p, a.C, q, key, comp, w);
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = j < q && j < kFewDraws ? picked[j < kFewDraws ? j : 0] : 0x7fffffff;
        sort_few(v);
#pragma unroll
        for (int j = 0; j < kFewDraws; ++j)
            if (j < a.width) row[j] = j < q ? v[j] : -1;
        return;
    }
    LdsPerm perm{perm_lds + threadIdx.x, tb};
    draw_many(perm, a.K, a.p, a.C, q, key, comp, w);
    for (int32_t j = 0; j < q; ++j) row[j] = perm(j);
    for (int32_t j = q; j < a.width; ++j) row[j] = -1;
}

// ---------------------------------------------------------------------------------------
// A work list of the fused kernel, one thread per tile.  Tile boundaries sit at multiples of T columns counted from the row
// start, not from the component start: with rows aligned to T*16 bytes every interior tile then covers whole
// cache lines (a component that starts mid-line only gets a short first tile), and no tile
// crosses a block of a blocked state.  Tiles that straddle lines cost a quarter of the bandwidth on MI355X.
//
// With `apart` (aligned rows, see tiles_apart on the host) the whole tiles of a component are dealt anew among as many: 64 tiles, or the 64 KB
// worth of tiles that are left, share the columns they cover in stretches of 512 bytes.  A tile's stretches lie in pairs
// 32 KB apart, so that each instruction of a wave, 1 KB, accesses both of a pair; the pairs follow each other every 64 KB (64 tiles), or are spread
// evenly over 32 KB (64 KB of tiles).  HBM takes such writes better, it seems because a memory page holds the same 512 bytes of
// neighbouring 32 KB.  16 or 32 rows in turns of 4 KB, in-place: 5.8, 5.7 TB/s, with 4 stretches 32 KB apart 6.5, 6.1, with whole runs of 64 KB in one row 6.3, 6.4;
// reads alone 7.5 whatever the order.  Stretches of 256 bytes or 1 KB and distances of 8, 16, 64 or 128 KB gain nothing in the fused kernel, nor do pairs of
// different waves.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void tile_kernel(TileArgs a)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= a.n) return;
    int32_t lo = 0, hi = a.m;                             // the last component that begins at or before tile i
    while (hi - lo > 1) {
        const int32_t mid = lo + (hi - lo) / 2;
        if (a.start[mid] <= i) lo = mid;
        else hi = mid;
    }
    const int64_t begin = a.off[lo], end = a.off[lo + 1], T = static_cast<int64_t>(1) << a.logT;
    const int64_t g = ((begin >> 2) >> a.logT) + (i - a.start[lo]);
    int64_t first = max(g * T * 4, begin);
    const int64_t last = min((g + 1) * T * 4, end), n = last - first;
    int kind = kOneStretch;
    if (a.apart) {
        const int64_t whole = (begin + 4 * T - 1) >> (a.logT + 2), wholes = max((end >> (a.logT + 2)) - whole, int64_t{0}), j = g - whole;
        const int64_t wide = wholes >> 6 << 6, narrow = 1 << (kLogApart + 1 - a.logT), left = (wholes - wide) / narrow * narrow;
        if (j >= 0 && j < wide) {
            first = ((whole + (j >> 6 << 6)) * T + ((j & 63) << kLogStretch)) * 4;
            kind = kApartWide;
        } else if (j >= wide && j < wide + left) {
            const int64_t in = (j - wide) % narrow;
            first = ((g - in) * T + (in << kLogStretch)) * 4;
            kind = kApartNarrow;
        }
    }
    a.out[i] = TileDesc{first, static_cast<uint16_t>(n), static_cast<uint16_t>(a.comp[lo].q | kind << kTileKind), lo};
}

// ---------------------------------------------------------------------------------------
// Final model average (Algorithm 1, RETURN): out[e] = fl(1/K) * (theta[0][e] + theta[1][e] + ...),
// summed in ascending worker id.  One thread per 16-byte column, one wave per workgroup; rows may start
// at any 4-byte address; 4(K+1) bytes per parameter.
//
// Bound by HBM reads, and by the latency of the caches where they hold the rows: what counts is how many loads a CU has
// in flight, and beyond the caches that there are no more than HBM takes; the host chooses both by the size of the sum
// and says with which figures.
// ---------------------------------------------------------------------------------------
// s plus the last n <= B rows, all their loads in flight; a row that is not there is read as the last one.  No load of
// an average is behind a branch: a guard on each cost a wait for those before it.  1024 workers x 36.5 K plain:
// 93 us guarded, 70 now, the last P % 4 elements by one thread 333.
template <int B, class V, class Load>
__device__ __forceinline__ V add_last(V s, const float *col, int n, int64_t stride, Load load)
{
    if constexpr (B > 1)
        if (n <= B / 2) return add_last<B / 2>(s, col, n, stride, load);
    V v[B];
#pragma unroll
    for (int j = 0; j < B; ++j) v[j] = load(col + static_cast<int64_t>(min(j, n - 1)) * stride);
#pragma unroll
    for (int j = 0; j < B; ++j)
        if (j < n) s = s + v[j];
    return s;
}

template <int B, class V, class Load>
__device__ __forceinline__ V worker_mean(const float *col, int K, int64_t stride, float inv, Load load)
{
    V s = load(col);
    int k = 1;
    for (; k + B <= K; k += B) {                           // B rows in flight, then added in ascending order
        V v[B];
#pragma unroll
        for (int j = 0; j < B; ++j) v[j] = load(col + static_cast<int64_t>(k + j) * stride);
#pragma unroll
        for (int j = 0; j < B; ++j) s = s + v[j];
    }
    if (k < K) s = add_last<B>(s, col + static_cast<int64_t>(k) * stride, K - k, stride, load);
    return s * inv;
}

template <int B, int POL>
__global__ __launch_bounds__(64) void final_average_kernel(const float *theta, Placement at, int K, int64_t P,
                                                           float inv, float *out, int xcd_log, int rotate)
{
    // as in the fused kernel, XCD r takes the r-th run of 2^xcd_log workgroups in every group of 8 runs
    const unsigned lg = static_cast<unsigned>(xcd_log), whole = (gridDim.x >> (3 + lg)) << (3 + lg);
    unsigned b = blockIdx.x;
    if (b < whole) {
        const unsigned i = b >> 3, group = i >> lg, r = (b + (rotate ? group >> 3 : 0u)) & 7u;
        b = (((group << 3) | r) << lg) | (i & ((1u << lg) - 1u));
    }
    const int64_t i = static_cast<int64_t>(b) * 64 + threadIdx.x;
    const int64_t n4 = P >> 2;
    if (i < n4) {
        const float *col = theta + placed(at, i << 2);
        store4<POL>(out + (i << 2), worker_mean<B, v4f>(col, K, at.stride, inv, [](const float *p) { return load4<POL>(p); }));
    } else if (static_cast<int64_t>(b) * 64 >= n4 && threadIdx.x < (P & 3)) {
        // the last P % 4 elements, one thread each of a wave that holds no columns, for which they would wait
        const int64_t e = (n4 << 2) + threadIdx.x;
        out[e] = worker_mean<B, float>(theta + placed(at, e), K, at.stride, inv, [](const float *p) { return *p; });
    }
}

// ---------------------------------------------------------------------------------------
// Copy of up to three state arrays between two placements, one 16-byte column
// per thread, one load and one store in flight each: more of either per thread is slower here (5.6
// against 6.2 TB/s on a plain copy).  The rows are cut into pieces of 256 columns (4 KB); the pieces
// are walked in runs of run_len pieces of one worker, then the same run of the next worker, and of `fold` arrays one after the
// other before the next run; blockIdx.z counts the arrays that are not folded.  Columns are counted from
// the destination row's 128-byte line, so that stores cover whole lines; the loads take any 4-byte address.
//
// Bound by HBM, which takes two long streams best.  Stores go through the L2 at once, and beyond the caches loads leave it
// first (choose_policy on the host says why; 1 M values 5.0 us, plain stores 5.7).  The host chooses the walk.
// ---------------------------------------------------------------------------------------
template <int LOADS>
__global__ __launch_bounds__(256) void state_copy_kernel(CopyArgs a)
{
    const uint32_t i = blockIdx.y * gridDim.x + blockIdx.x, K = static_cast<uint32_t>(a.K), rows = K * a.fold;
    const uint32_t run = i / a.run_len, group = run / rows, row = run - group * rows, array = row / K, w = row - array * K;
    const int64_t piece = static_cast<int64_t>(group) * a.run_len + (i - run * a.run_len);
    const float *src = a.src[blockIdx.z + array] + w * a.sa.stride;
    float *dst = a.dst[blockIdx.z + array] + w * a.da.stride;
    const int64_t head = static_cast<int64_t>((reinterpret_cast<uintptr_t>(dst) >> 2) & 31u);
    const int64_t e = (piece * 256 + threadIdx.x) * 4 - head;
    if (e >= a.P) return;
    // four floats that neither side cuts at a block edge
    if (e >= 0 && e + 4 <= a.P && ((e ^ (e + 3)) >> a.sa.logB) == 0 && ((e ^ (e + 3)) >> a.da.logB) == 0) {
        store4<kStreamed>(dst + placed(a.da, e), load4<LOADS>(src + placed(a.sa, e)));
        return;
    }
    for (int c = 0; c < 4; ++c)
        if (e + c >= 0 && e + c < a.P) dst[placed(a.da, e + c)] = src[placed(a.sa, e + c)];
}

// Plain streaming copy of n 16-byte words (calibration of HBM counters and a reference for
// the bandwidth a 1:1 read/write stream reaches on this device).
__global__ __launch_bounds__(256) void copy_probe_kernel(v4f *dst, const v4f *src, int64_t n, int flags)
{
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
        const v4f v = (flags & 2) ? __builtin_nontemporal_load(src + i) : src[i];
        if (flags & 1) __builtin_nontemporal_store(v, dst + i);
        else dst[i] = v;
    }
}

}  // namespace

int launch_final_average(const float *theta, const Placement &at, int K, int64_t P, float inv, float *out,
                         const AverageShape &shape, hipStream_t stream)
{
    if (P <= 0) return GBMUF_OK;
    size_t lds_floor = shape.lds_floor < 60 * 1024 ? shape.lds_floor : 60 * 1024;   // stays below what needs a raised limit
    const int64_t blocks = ((P >> 2) + 63) / 64 + ((P & 3) != 0);
    if (blocks > 0x7fffffffLL) return GBMUF_EUNSUPPORTED;
    Placement pl = at;
    int xcd_log = shape.xcd_log, rotate = shape.rotate ? 1 : 0;
    void *argv[] = {&theta, &pl, &K, &P, &inv, &out, &xcd_log, &rotate};
    const bool streamed = shape.policy == kStreamed;
    using Fn = void (*)(const float *, Placement, int, int64_t, float, float *, int, int);
    const Fn kernel = shape.rows_in_flight <= 4   ? (streamed ? final_average_kernel<4, kStreamed> : final_average_kernel<4, kPlain>)
                      : shape.rows_in_flight <= 8 ? final_average_kernel<8, kPlain>
                                                  : (streamed ? final_average_kernel<16, kStreamed> : final_average_kernel<16, kPlain>);
    const void *fn = reinterpret_cast<const void *>(kernel);
    const hipError_t err = hipLaunchKernel(fn, dim3(static_cast<unsigned>(blocks)), dim3(64), argv, lds_floor, stream);
    return err == hipSuccess ? GBMUF_OK : hip_failed("hipLaunchKernel(final average)", err, GBMUF_EDEVICE);
}

// The walk of a copy.  Rows to rows are copied whole, array by array: two long streams.  A blocked side is one stretch of memory where
// the arrays of a run follow each other.  us for three arrays, now / runs of 4 KB to 128 KB or whole rows, array by array, at their best:
//   blocked to blocked, 32 KB, folded, 400 M values: 3 workers 1420 / 1625, 44 workers 1418 / 1751, 300 workers 1411 / 1463.
//   rows to blocked, folded, up to 32 workers 128 KB: 3 x 133 M odd rows 1528 / 1713, 24 x 16.7 M 1602 / 1633; up to 200 workers 64 KB: 40 x
//     0.75 M odd rows 117 / 32 KB 120, whole rows 130; 64 x 0.94 M padded 241 / 279, 252; 64 x 6.2 M 1504 / 1581, 1703; more workers 32 KB: 256 x 1.6
//     M 1566 / 64 KB 1689, whole rows 1717 (128 x 3.1 M 1582 / 1565, 1726).  33 to 60 workers and up to 15 M values, and more workers and up to 40 M, whole
//     rows: 64 x 0.47 M 120 / 64 KB 127.  Single sizes differ by 5 to 10 % either way, by where the arrays lie.
//   blocked to rows, array by array: aligned rows of up to 16 workers 32 KB, 12 x 33 M 1469 / whole rows 1505, of more whole rows, 44 x 9.1 M
//     1513 / 1631; rows that share lines of up to 48 workers 4 KB, 24 x 16.7 M 1629 / whole rows 1710, 44 x 9.1 M 1745 / 1782, of
//     more whole rows, 100 x 4 M 1673 / 4 KB 1860.
//   Up to 4 M values the caches hold them: whole rows, which stay there.
int launch_state_copy(const CopyArgs &c, int arrays, hipStream_t stream)
{
    if (c.P <= 0 || c.K <= 0 || arrays <= 0) return GBMUF_OK;
    CopyArgs args = c;
    const int64_t pieces = (c.P + 31 + 1023) / 1024, values = c.P * c.K;       // 31: the largest head
    const bool from = c.sa.logB != 62, to = c.da.logB != 62, streamed = values > 4000000;
    int64_t run = pieces;
    bool fold = false;
    if (streamed && to && (from || c.K <= 32 || values > (c.K <= 60 ? 15000000 : 40000000))) {
        run = from || c.K > 200 ? 8 : c.K <= 32 ? 32 : 16;
        fold = true;
    } else if (streamed && from && !to) {
        bool shared = c.K > 1 && c.da.stride % 32 != 0;
        for (int n = 0; n < arrays; ++n) shared = shared || reinterpret_cast<uintptr_t>(c.dst[n]) % 128 != 0;
        if (c.K <= (shared ? 48 : 16)) run = shared ? 1 : 8;
    }
    // runs of equal length: the last one of a row is filled up by workgroups that have nothing to do
    const int64_t runs = (pieces + run - 1) / run, len = (pieces + runs - 1) / runs;
    int64_t blocks = runs * len * c.K;
    if (fold && blocks * arrays > (static_cast<int64_t>(511) << 23)) fold = false;
    args.run_len = static_cast<uint32_t>(len);
    args.fold = fold ? static_cast<uint32_t>(arrays) : 1u;
    blocks *= args.fold;
    // a grid holds fewer than 2^32 threads along x: the rest goes along y
    const int64_t x = blocks < (1 << 23) ? blocks : (1 << 23), y = (blocks + x - 1) / x;
    if (y > 511) return GBMUF_EUNSUPPORTED;                // 17 TB: the kernel counts pieces in 32 bits
    const unsigned z = fold ? 1u : static_cast<unsigned>(arrays);
    void *argv[] = {&args};
    const auto kernel = streamed ? state_copy_kernel<kStreamed> : state_copy_kernel<kPlain>;
    const hipError_t err = hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3(static_cast<unsigned>(x), static_cast<unsigned>(y), z),
                                           dim3(256), argv, 0, stream);
    return err == hipSuccess ? GBMUF_OK : hip_failed("hipLaunchKernel(state copy)", err, GBMUF_EDEVICE);
}

int launch_copy_probe(float *dst, const float *src, int64_t n_floats, int flags, int blocks, hipStream_t stream)
{
    int64_t n = n_floats / 4;
    if (n <= 0) return GBMUF_OK;
    v4f *d = reinterpret_cast<v4f *>(dst);
    const v4f *s = reinterpret_cast<const v4f *>(src);
    void *argv[] = {&d, &s, &n, &flags};
    const hipError_t err = hipLaunchKernel(reinterpret_cast<const void *>(copy_probe_kernel), dim3(blocks), dim3(256),
                                           argv, 0, stream);
    return err == hipSuccess ? GBMUF_OK : hip_failed("hipLaunchKernel(copy probe)", err, GBMUF_EDEVICE);
}

// ---------------------------------------------------------------------------------------
// The fused kernel's shapes, LDS and launch.
// ---------------------------------------------------------------------------------------
namespace {
constexpr Variant kVariants[] = {
    {256, 8, 8}, {512, 8, 8}, {512, 4, 4}, {256, 16, 16}, {1024, 4, 4}, {256, 4, 4},
    {256, 2, 2}, {512, 2, 2}, {1024, 2, 2}, {1024, 1, 1}, {512, 1, 1}, {256, 1, 1},
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

KernelFn pick_kernel(const Variant &v, int policy, int q, bool mixed)
{
    static constexpr PickFn *parts[3][5] = {
        {GBMUF_PICK_NAME(0, 0), GBMUF_PICK_NAME(1, 0), GBMUF_PICK_NAME(2, 0), GBMUF_PICK_NAME(3, 0), GBMUF_PICK_NAME(4, 0)},
        {GBMUF_PICK_NAME(0, 1), GBMUF_PICK_NAME(1, 1), GBMUF_PICK_NAME(2, 1), GBMUF_PICK_NAME(3, 1), GBMUF_PICK_NAME(4, 1)},
        {GBMUF_PICK_NAME(0, 2), GBMUF_PICK_NAME(1, 2), GBMUF_PICK_NAME(2, 2), GBMUF_PICK_NAME(3, 2), GBMUF_PICK_NAME(4, 2)}};
    for (PickFn *pick : parts[policy])
        if (KernelFn k = pick(v, q, mixed)) return k;
    return nullptr;
}

size_t perm_bytes(int K, int C) { return static_cast<size_t>(K) * static_cast<size_t>(C) * sizeof(int32_t); }

}  // namespace

// Workgroups can draw their own neighbour rows when the candidates of all workers fit 8 KB of LDS.
bool can_sample_inline(int K, int C) { return perm_bytes(K, C) <= 8192; }

// Rows of at most kFewDraws neighbours are drawn in registers.
bool draws_in_registers(int q) { return q <= kFewDraws; }

const Variant *variant_table(int *count)
{
    *count = kNumVariants;
    return kVariants;
}

// Dynamic LDS one workgroup of the fused kernel needs: the theta tile, the merged neighbour
// rows (q = the largest q_i) and, when it draws them itself, the candidate copies.
size_t sync_lds_bytes(const Variant &v, int K, int q, bool mixed, int C, bool in_kernel_sampling)
{
    return static_cast<size_t>(v.threads) * v.slots * sizeof(float4) + ids_words(K, ids_pitch(kernel_q1(q, mixed), q)) * sizeof(uint16_t) +
           (in_kernel_sampling && !draws_in_registers(q) ? perm_bytes(K, C) : 0);
}

// Raises the dynamic-LDS limit of a kernel this plan may launch to the device's maximum
// (so that plans with different needs can share a kernel) and says whether workgroups can
// draw their own neighbour rows.  GBMUF_EUNSUPPORTED if one workgroup's LDS exceeds the device.
int prepare_kernel(const Variant &v, int policy, int K, int q, bool mixed, int C, bool *can_sample_in_kernel)
{
    const bool inl = can_sample_inline(K, C);
    *can_sample_in_kernel = inl;
    const size_t lds = sync_lds_bytes(v, K, q, mixed, C, inl);
    int dev = 0, max_lds = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return hip_failed("hipGetDevice", err, GBMUF_EDEVICE);
    err = hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (err != hipSuccess) return hip_failed("hipDeviceGetAttribute(MaxSharedMemoryPerBlock)", err, GBMUF_EDEVICE);
    if (lds > static_cast<size_t>(max_lds)) return GBMUF_EUNSUPPORTED;
    KernelFn k = pick_kernel(v, policy, q, mixed);
    if (!k) return GBMUF_EINVAL;
    err = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, max_lds);
    if (err != hipSuccess) return hip_failed("hipFuncSetAttribute(fused kernel)", err, GBMUF_EDEVICE);
    return GBMUF_OK;
}

// lds_floor: the workgroup asks for at least this much dynamic LDS, which bounds how many
// workgroups a compute unit holds at once (0 = only what it needs).
int launch_sync(const Variant &v, int policy, const SyncArgs &a, int64_t n_tiles, size_t lds_floor, hipStream_t stream)
{
    if (n_tiles <= 0) return GBMUF_OK;
    if (n_tiles > 0x7fffffffLL) return GBMUF_EUNSUPPORTED;
    const bool mixed = (a.flags & kFlagMixedQ) != 0;
    KernelFn k = pick_kernel(v, policy, a.q, mixed);
    if (!k) return GBMUF_EINVAL;
    if (a.nbr == nullptr && !draws_in_registers(a.q) && !can_sample_inline(a.K, a.C)) return GBMUF_EINVAL;
    size_t lds = sync_lds_bytes(v, a.K, a.q, mixed, a.C, a.nbr == nullptr);
    if (lds < lds_floor) lds = lds_floor;
    SyncArgs args = a;
    void *argv[] = {&args};
    // the launch's own status: an earlier, unrelated error of the process is not ours to report
    const hipError_t err = hipLaunchKernel(reinterpret_cast<const void *>(k), dim3(static_cast<unsigned>(n_tiles)),
                                           dim3(v.threads), argv, lds, stream);
    return err == hipSuccess ? GBMUF_OK : hip_failed("hipLaunchKernel(sync)", err, GBMUF_EDEVICE);
}

int launch_tiles(const TileArgs &a, hipStream_t stream)
{
    if (a.n <= 0) return GBMUF_OK;
    const int64_t blocks = (a.n + 255) / 256;
    if (blocks > 0x7fffffffLL) return GBMUF_EUNSUPPORTED;
    TileArgs args = a;
    void *argv[] = {&args};
    const hipError_t err = hipLaunchKernel(reinterpret_cast<const void *>(tile_kernel), dim3(static_cast<unsigned>(blocks)), dim3(256), argv, 0,
                                           stream);
    return err == hipSuccess ? GBMUF_OK : hip_failed("hipLaunchKernel(tile list)", err, GBMUF_EDEVICE);
}

int launch_sampler(const SampleArgs &a, hipStream_t stream)
{
    if (a.pairs <= 0 || a.width <= 0) return GBMUF_OK;
    // beyond kFewDraws each thread keeps C ints in LDS: as many threads as fit 48 KB, at most 64
    const size_t per_thread = draws_in_registers(a.q) ? 0 : static_cast<size_t>(a.C) * sizeof(int32_t);
    int tb = 64;
    while (tb > 1 && tb * per_thread > 48 * 1024) tb >>= 1;
    if (tb * per_thread > 48 * 1024) return GBMUF_EUNSUPPORTED;
    const int64_t blocks = (a.pairs + tb - 1) / tb;
    if (blocks > 0x7fffffffLL) return GBMUF_EUNSUPPORTED;
    SampleArgs args = a;
    void *argv[] = {&args};
    const hipError_t err = hipLaunchKernel(reinterpret_cast<const void *>(sample_kernel),
                                           dim3(static_cast<unsigned>(blocks)), dim3(tb), argv,
                                           tb * per_thread, stream);
    return err == hipSuccess ? GBMUF_OK : hip_failed("hipLaunchKernel(sampler)", err, GBMUF_EDEVICE);
}

}  // namespace gbmuf
