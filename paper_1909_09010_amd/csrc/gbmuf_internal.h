// gbmuf_internal.h -- types shared by the host and device halves of libgbmuf.
// Not part of the public interface (that is include/gbmuf.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace gbmuf {

// One workgroup's share of a sync: n elements of component `comp`, for all K workers, the first of them `lo`.  A tile of kind kOneStretch holds the
// elements [lo, lo + n), which never cross a component boundary and lie inside one run of tile_columns 16-byte columns (a column is 4 elements whose first
// index is a multiple of 4).  The n = 4 * tile_columns elements of the other kinds lie in stretches of 2^kLogStretch columns, the first of which begins at lo;
// the two of a pair begin 2^kLogApart columns from each other, and the last ends up to 64 tiles' worth of columns, or 64 KB, behind lo (tile_kernel).  The low bits
// of q are the number of neighbours this component draws, the two above (from kTileKind on) the tile's kind.
struct TileDesc {
    int64_t lo;
    uint16_t n;
    uint16_t q;
    int32_t comp;
};
constexpr int kTileKind = 14;            // the bit of q where the kind begins
enum : int { kOneStretch = 0, kApartWide = 1, kApartNarrow = 2 };
constexpr int kLogStretch = 5, kLogApart = 11;     // 512 bytes, 32 KB
static_assert(sizeof(TileDesc) == 16, "one 16-byte load per workgroup");

// Per-component constants on the device.
struct CompDesc {
    float inv;               // 1/(q_i + 1), rounded once on the host
    int32_t period;          // sync period H_i (1 if the plan has none)
    int32_t q;               // neighbours drawn for this component
    int32_t reserved;
};
static_assert(sizeof(CompDesc) == 16, "one 16-byte load");

// Placement of one state array's elements: element e of worker w is at
//   base + w * stride + e + (e >> logB) * block_extra
// Rows: logB = 62 and block_extra = 0.  Blocked: 2^logB floats per block and
// block_extra = block_stride - 2^logB.
struct Placement {
    int64_t stride;
    int64_t block_extra;
    int32_t logB;
    int32_t reserved;
};

// Arguments of the fused gather-average-momentum kernels.
struct SyncArgs {
    const TileDesc *tiles;
    const int32_t *nbr;      // [m][K][width], device; nullptr: the workgroup draws its rows itself
    const CompDesc *comp;    // [m]
    float *theta, *omega, *delta;
    Placement at;
    int32_t K, q;            // q: neighbours per component (the largest q_i when they differ)
    int32_t logT;            // log2(columns per tile)
    int32_t xcd_log;         // log2(consecutive tiles that one XCD takes)
    int32_t mode;            // GBMUF_MODE_*
    float eta, zeta, inv;    // inv = 1/(q+1), rounded once on the host (plans with one q)
    int32_t flags;           // bit 3: walk the tile list backwards, bit 4: components draw different q (read the
                             // tile's q and the component's inv), bit 5: skip components whose
                             // period does not divide `step`, bit 6: rotate the XCDs (tile_of_block),
                             // bit 7: the library's sampler wrote nbr (not a caller)
    // in-kernel sampling (nbr == nullptr): same bits as the sampler kernel, drawn from the key below
    int32_t p, C;            // ring degree, candidates per worker
    uint32_t key0, key1, round0, round1;
    uint64_t step;           // with flag bit 5: component i syncs iff step % H_i == 0
};

enum : int32_t {
    kFlagBackwards = 8,
    kFlagMixedQ = 16,
    kFlagCheckPeriods = 32,
    kFlagRotate = 64,
    kFlagSampledTable = 128,
};

// Arguments of the neighbour-sampling kernel: pairs [first_pair, first_pair + pairs) of the
// (component, worker) grid, pair = component * K + worker.
struct SampleArgs {
    const CompDesc *comp;    // [m]
    int32_t *out;            // [m][K][width]; entries beyond a component's q are set to -1
    int64_t first_pair, pairs;
    int32_t K, p, C;         // ring degree, candidates per worker
    int32_t q, width;        // q is every component's unless `mixed`, the largest otherwise
    int32_t mixed;           // components draw different q: take comp[i].q
    int32_t check_periods;   // skip components whose period does not divide `step`
    uint32_t key0, key1;     // seed low / high
    uint32_t round0, round1; // round low / high
    uint64_t step;
};

// Arguments of the placement change: up to three arrays, all from placement `sa` to `da`.
struct CopyArgs {
    float *dst[3];
    const float *src[3];
    Placement da, sa;
    int64_t P;
    int32_t K;
    uint32_t run_len;        // pieces of one worker that follow each other (set by the launch)
    uint32_t fold;           // arrays whose runs follow each other (set by the launch)
};

// One tile shape of the fused kernel: threads per workgroup and 16-byte slots per thread.
// A tile holds threads*slots slots = K worker rows of tile_columns columns each.  depth: how many
// slots of omega and Delta a thread holds at a time (depth < slots: for many workers).
struct Variant {
    int threads;
    int slots;
    int depth;
};
// shapes that only the library's own rules take (aligned_shape, shared_variant)
constexpr Variant kSixtyFour = {1024, 2, 1};
constexpr Variant kMany = {1024, 4, 2};
constexpr Variant kVeryMany = {512, 16, 4};
constexpr size_t kLdsPerWorkgroup = 160 * 1024;    // gfx950

// Which instance of the fused kernel a component's neighbour count takes (gbmuf_sync.hip), and the
// layout of its neighbour rows in LDS.
constexpr int kFewDraws = 7;                       // up to so many neighbours are drawn in registers
constexpr int kUpTo8 = 8, kMixed = 9, kAnyQ = 0;
constexpr int kernel_q1(int q, bool mixed) { return q > kFewDraws ? kAnyQ : mixed ? kMixed : q > 4 ? kUpTo8 : q + 1; }
// uint16 per row, and in all rows (padded to 16 bytes)
__host__ __device__ constexpr int ids_pitch(int Q1, int q) { return Q1 == kAnyQ ? q + 1 : Q1 <= 4 ? 4 : 8; }
__host__ __device__ constexpr size_t ids_words(int K, int pitch)
{
    return (static_cast<size_t>(K) * static_cast<size_t>(pitch) + 7) & ~static_cast<size_t>(7);
}

using KernelFn = void (*)(SyncArgs);

// How the accesses of state use the caches (load4, store4): plainly, or loads that leave the L2 first and stores that go
// through it at once.  kApart: streamed, and whole tiles may lie in stretches (tile_kernel).  Kernels of their own, because what these take
// is paid where no tile does: with the code for them in the streamed kernels those of gossip-MA waited for their neighbour table before
// the first load of theta, and of what is then in flight some shapes have too little (blocked, us, apart / together: 5 x 380 M 2492 / 2685, 6 x 150 M
// 1066 / 1127, 40 x 22 M 1068 / 1102).
enum : int { kPlain = 0, kStreamed = 1, kApart = 2 };

// The shapes of gbmuf_sync.hip in each part and policy, or nullptr.
#define GBMUF_PICK_NAME2(part, policy) pick_kernel_##part##_##policy
#define GBMUF_PICK_NAME(part, policy) GBMUF_PICK_NAME2(part, policy)
using PickFn = KernelFn(const Variant &v, int q, bool mixed);
PickFn GBMUF_PICK_NAME(0, 0), GBMUF_PICK_NAME(1, 0), GBMUF_PICK_NAME(2, 0), GBMUF_PICK_NAME(3, 0), GBMUF_PICK_NAME(4, 0);
PickFn GBMUF_PICK_NAME(0, 1), GBMUF_PICK_NAME(1, 1), GBMUF_PICK_NAME(2, 1), GBMUF_PICK_NAME(3, 1), GBMUF_PICK_NAME(4, 1);
PickFn GBMUF_PICK_NAME(0, 2), GBMUF_PICK_NAME(1, 2), GBMUF_PICK_NAME(2, 2), GBMUF_PICK_NAME(3, 2), GBMUF_PICK_NAME(4, 2);

// Remembers the most recent failing HIP call of this thread (what gbmuf_last_error_detail
// returns) and maps it to a status.
int hip_failed(const char *what, hipError_t err, int status);

// Arguments of the kernel that writes a tile list.
struct TileArgs {
    const int64_t *off;      // m+1 component offsets
    const int64_t *start;    // m+1: first tile of every component
    const CompDesc *comp;
    TileDesc *out;
    int64_t n;               // tiles
    int32_t m, logT;
    int32_t apart;           // whole tiles lie in stretches
};

// gbmuf_kernels.hip
int launch_tiles(const TileArgs &a, hipStream_t stream);
int launch_sampler(const SampleArgs &a, hipStream_t stream);
struct AverageShape {
    int rows_in_flight;      // 16-byte loads a thread keeps in flight: 4, 8 or 16
    size_t lds_floor;        // bounds the resident one-wave workgroups per compute unit like in launch_sync
    int xcd_log;             // log2 of the consecutive workgroups that one XCD takes
    bool rotate;             // see the fused kernel's tile_of_block
    int policy;              // kPlain or kStreamed
};
int launch_final_average(const float *theta, const Placement &at, int K, int64_t P, float inv, float *out,
                         const AverageShape &shape, hipStream_t stream);
int launch_state_copy(const CopyArgs &c, int arrays, hipStream_t stream);
int launch_copy_probe(float *dst, const float *src, int64_t n_floats, int flags, int blocks, hipStream_t stream);
int launch_sync(const Variant &v, int policy, const SyncArgs &a, int64_t n_tiles, size_t lds_floor, hipStream_t stream);
size_t sync_lds_bytes(const Variant &v, int K, int q, bool mixed, int C, bool in_kernel_sampling);
int prepare_kernel(const Variant &v, int policy, int K, int q, bool mixed, int C, bool *can_sample_in_kernel);
bool can_sample_inline(int K, int C);
bool draws_in_registers(int q);
const Variant *variant_table(int *count);          // the shapes a plan description can name

}  // namespace gbmuf
