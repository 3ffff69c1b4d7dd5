// gbmuf_plan.hip -- host half of libgbmuf: plan construction (partition, ring topology,
// tile lists), the host sampler, argument checks and the C entry points of include/gbmuf.h.
#include "gbmuf_internal.h"

#include "../../include/gbmuf.h"

#include <algorithm>
#include <array>
#include <cstddef>
#include <cstdio>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

using namespace gbmuf;

namespace {

// Work list of the fused kernel for one tile width, in component order.
struct TileSet {
    int32_t logT = 0;
    bool apart = false;                // see tile_kernel
    std::vector<int64_t> tile_start;   // m+1: first tile of every component, and how many there are
    TileDesc *d_tiles = nullptr;       // in gbmuf_plan_s::d_tiles
};

// How the fused kernel runs on one kind of state placement.
struct LayoutCfg {
    Variant variant{256, 8, 8};
    int32_t policy = 0;                // how state is loaded and stored (load4, store4)
    int32_t logT = 0;
    int32_t set = 0;                   // which TileSet
    int32_t workgroups_per_cu = 0;     // 0 = no bound
    int32_t xcd_columns_log = 0;       // log2 of the columns of a row that one XCD takes in one run (if more than a tile)
    bool rotate = false;               // see tile_of_block
    bool apart = false;                // see tile_kernel
};

// kShared: rows of which some start inside a 128-byte line, so that neighbouring tiles share lines.
// kFine: aligned rows, most of whose floats are in short components (rows_layout).
enum { kRows = 0, kBlocked = 1, kShared = 2, kFine = 3, kLayouts = 4 };
enum { kBmuf = 0, kMa = 1, kBranches = 2 };   // the three-array update, or the gossip-MA branch (theta only)
// How much one launch updates.  With sync periods that differs from call to call by orders of magnitude, so
// everything that depends on it is chosen per launch, from the components that are due.
enum { kTiny = 0, kSmall = 1, kCompact = 2, kMiddle = 3, kLarge = 4, kSizes = 5 };
constexpr int kMaxTileSets = kLayouts * kBranches * kSizes;

// Whether tiles in stretches 32 KB apart (tile_kernel) pay in the component [a, b) of aligned rows: shorter ones have few of them and, in the wide shapes that
// go with stretches, more tiles that their ends cut.  us in components of one size, as if they were short / stretches: 12 x 58 M of 16 K floats (15872) 2790 / 3194, of 140 K 2811 / 2886, of
// 160 K 2805 / 2760; gossip-MA 6 x 117 M of 140 K 863 / 910, of 200 K 865 / 851; 2 x 150 M of 16 K 1120 / 1276, of 100 K 1113 / 1091; 13 x 23 M of 23 K 1196 / 1268, of 50 K 1202 / 1181; 32 x 9.4 M of 32 K
// 1325 / 1340, of 50 K 1333 / 1234; 48 x 0.6 M of 5 K 103 / 107, of 50 K 103 / 102; 8 x 19 M of 102400 610 / 560, 8 x 87 M of 76800 2754 / 2891; 3 x 10 M of 51200 97.4 / 95.4, gossip-MA 6 x 50 M of
// 51200 361 / 373.  Short ones that begin on a tile and are, but for a twentieth, 64 KB or a multiple long have
// nothing else: 12 x 12.5 M of 16384 606 / 530, 8 x 19 M of 65536 610 / 550, 2 x 350 M of 49152 gossip-MA 890 / 822, 32 x 22 M of 16384 3152 / 2881, at worst 4 x 175 M of 102400 2687 / 2784.
bool long_component(int K, int what, bool large, int64_t a, int64_t b)
{
    const int64_t n = b - a, tile = K <= 2 ? 4096 : 1024;
    int64_t least = K <= 2 ? 1 << 17 : K <= 12 ? 10 << 14 : 1 << 15;
    if (K == 3 || K == 4 || K == 8 || (K > 4 && K < 8 && what == kBmuf)) least = large && K > 4 ? 10 << 14 : 3 << 14;
    return n >= least || (n >= 1 << 14 && a % tile == 0 && n % (1 << 14) <= n / 20);
}

// What launches on aligned rows update in long components, by branch and in launches of up to and of more than kLargeValues.
struct LongValues {
    int64_t of[kBranches][2] = {};
    void add(int K, int64_t a, int64_t b)
    {
        for (int what = 0; what < kBranches; ++what)
            for (int large = 0; large < 2; ++large)
                if (long_component(K, what, large != 0, a, b)) of[what][large] += K * (b - a);
    }
};

}  // namespace

struct gbmuf_plan_s {
    int32_t m = 0, K = 0, q = 0, p = 0, C = 0;
    uint64_t seed = 0;
    int64_t P = 0;
    bool mixed_q = false, has_periods = false;
    std::vector<int64_t> off;        // m+1 component offsets
    std::vector<int32_t> qv;         // m: neighbours per component
    std::vector<int32_t> periods;    // m: sync period H_i (all 1 without periods)
    std::vector<int32_t> cand;       // [K][C] ring candidates, order of Definition 1
    std::vector<CompDesc> comp;      // m: per-component constants of the kernels
    LongValues long_values;
    LayoutCfg cfg[kLayouts][kBranches][kSizes];
    int32_t min_block_logT = 0;      // blocks hold at least 4 << min_block_logT floats
    TileSet sets[kMaxTileSets];      // one per distinct tile width among the configurations that calls can take
    int32_t n_sets = 0;
    float inv = 1.0f;                // 1/(q+1), rounded once (plans with one q)
    int32_t sampling = GBMUF_SAMPLING_AUTO;   // as asked for
    bool launch_bound = false;       // with AUTO: workgroups always draw their own neighbour rows
    bool named_shape = false;        // the plan description names the tile shape
    bool alternate = true;           // odd rounds walk the tile list backwards (see tile_of_block)

    bool has_device = false;
    int device = -1;
    int32_t lds_per_cu = 0, cus = 0;
    CompDesc *d_comp = nullptr;
    int64_t *d_starts = nullptr;     // off, then tile_start of every set
    TileDesc *d_tiles = nullptr;     // the lists of all sets
    int32_t *d_nbr = nullptr;        // neighbour scratch of gbmuf_sync, [m][K][q]
};

// ---------------------------------------------------------------------------------------
// Neighbour table of gbmuf_sync_static: device memory that exists without any allocation call.
// Every GPU the library runs on holds its own copy of this array (2 MiB) until the process
// ends.  In host code the array's name is only a handle for hipGetSymbolAddress: the device
// address is looked up once per device, with that device current, when a plan is made there,
// and kernels and copies are only ever given that address.
// ---------------------------------------------------------------------------------------
static __device__ __align__(256) int32_t scratch[GBMUF_STATIC_TABLE_ENTRIES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
int32_t *g_scratch_ptr[kMaxDevices] = {};

// Looks up this device's copy of `scratch`; `device` must be the current device.
int resolve_scratch(int device)
{
    if (device < 0 || device >= kMaxDevices) return GBMUF_OK;       // gbmuf_sync_static will refuse this device
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[device]) return GBMUF_OK;
    void *p = nullptr;
    const hipError_t err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (err != hipSuccess || !p) return gbmuf::hip_failed("hipGetSymbolAddress(scratch)", err, GBMUF_EDEVICE);
    g_scratch_ptr[device] = static_cast<int32_t *>(p);
    return GBMUF_OK;
}

int32_t *scratch_of(int device)
{
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    return g_scratch_ptr[device];
}
}  // namespace

namespace gbmuf {
static thread_local char g_detail[256] = "";
int hip_failed(const char *what, hipError_t err, int status)
{
    std::snprintf(g_detail, sizeof(g_detail), "%s: %s (%d)", what, hipGetErrorString(err), static_cast<int>(err));
    return status;
}
}  // namespace gbmuf

namespace {

// Section 3.3: p = log2(n) - 1, here floor(log2 K) - 1 and at least 1.
int32_t default_degree(int32_t K)
{
    int32_t lg = 0;
    while ((static_cast<int64_t>(2) << lg) <= K) ++lg;
    return lg - 1 > 1 ? lg - 1 : 1;
}

// Definition 1: (w-1)%K .. (w-p)%K, then (w+1)%K .. (w+p)%K; first occurrence kept, w dropped.
void ring_of(int32_t w, int32_t K, int32_t p, std::vector<int32_t> &out)
{
    out.clear();
    std::vector<char> taken(static_cast<size_t>(K), 0);
    taken[static_cast<size_t>(w)] = 1;
    for (int dir = -1; dir <= 1; dir += 2)
        for (int32_t d = 1; d <= p; ++d) {
            int64_t v = (static_cast<int64_t>(w) + static_cast<int64_t>(dir) * d) % K;
            if (v < 0) v += K;
            if (!taken[static_cast<size_t>(v)]) {
                taken[static_cast<size_t>(v)] = 1;
                out.push_back(static_cast<int32_t>(v));
            }
        }
}

// ---------------------------------------------------------------------------------------
// Host writing of the sampler (the device has its own in gbmuf_device.h; the tests
// require the two, and the reference implementation, to agree bit for bit).
// ---------------------------------------------------------------------------------------
using Words4 = std::array<uint32_t, 4>;

// Philox-4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds, each one multiplying words
// 0 and 2 by the two round constants and mixing the high halves with the neighbouring words
// and the key, which advances by the two Weyl increments.
Words4 philox_block(Words4 ctr, uint32_t key_lo, uint32_t key_hi)
{
    for (int round = 0; round < 10; ++round) {
        const uint64_t prod0 = static_cast<uint64_t>(ctr[0]) * 0xD2511F53u;
        const uint64_t prod2 = static_cast<uint64_t>(ctr[2]) * 0xCD9E8D57u;
        ctr = Words4{static_cast<uint32_t>(prod2 >> 32) ^ ctr[1] ^ key_lo, static_cast<uint32_t>(prod2),
                     static_cast<uint32_t>(prod0 >> 32) ^ ctr[3] ^ key_hi, static_cast<uint32_t>(prod0)};
        key_lo += 0x9E3779B9u;
        key_hi += 0xBB67AE85u;
    }
    return ctr;
}

// Algorithm 1, sync branch, first statement, for worker `w` and component `comp` in sync
// `round`: q ids out of the worker's C candidates, uniformly without replacement, ascending.
// Draw j uses word j mod 4 of the block with counter (round lo, round hi, comp, w + 65536 * (j div 4))
// and exchanges pool[j] with pool[j + floor(word * (C - j) / 2^32)].
void host_pick(const int32_t *cand, int32_t C, int32_t q, uint64_t seed, uint64_t round, uint32_t comp, uint32_t w,
               std::vector<int32_t> &pool, int32_t *out)
{
    pool.assign(cand, cand + C);
    Words4 words{};
    for (int32_t j = 0; j < q; ++j) {
        if (j % 4 == 0)
            words = philox_block(Words4{static_cast<uint32_t>(round), static_cast<uint32_t>(round >> 32), comp,
                                        w + (static_cast<uint32_t>(j / 4) << 16)},
                                 static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32));
        const uint64_t remaining = static_cast<uint64_t>(C - j);
        const size_t pick = static_cast<size_t>(j) + static_cast<size_t>((words[static_cast<size_t>(j % 4)] * remaining) >> 32);
        std::swap(pool[static_cast<size_t>(j)], pool[pick]);
    }
    std::sort(pool.begin(), pool.begin() + q);
    std::copy_n(pool.begin(), q, out);
}

// ---------------------------------------------------------------------------------------
// Tile shapes
// ---------------------------------------------------------------------------------------
bool find_variant(int threads, int slots, Variant *out)
{
    int count = 0;
    const Variant *tab = variant_table(&count);
    for (int i = 0; i < count; ++i)
        if (tab[i].threads == threads && tab[i].slots == slots) {
            *out = tab[i];
            return true;
        }
    return false;
}

// Bounds of the sizes, in values (K times the elements that are due).  Up to kTinyValues passes over a few states in turn
// stay in the caches, and loads that leave them early lose (choose_policy).  From kSmallValues on there are enough tiles of
// any shape for all CUs.  Up to kCompactValues something is left in the 256 MB memory-side cache from one sync to the next;
// for rows that share lines that is all that counts (three arrays, or theta alone).  Above kLargeValues a launch's rows are
// drawn in a kernel of their own (draws_itself), but gossip-MA's from kLargeValuesMa on.
constexpr int64_t kTinyValues = 2000000, kSmallValues = 5000000, kCompactValues = 20000000, kCompactValuesSharedMa = 60000000;
constexpr int64_t kLargeValues = 500000000, kLargeValuesMa = 130000000, kLargeValuesSharedMa = 149000000;

int size_of_launch(int64_t values, int layout, int what)
{
    const bool shared = layout == kShared;
    if (!shared && values <= kTinyValues) return kTiny;
    if (!shared && values <= kSmallValues) return kSmall;
    if (values <= (shared && what == kMa ? kCompactValuesSharedMa : kCompactValues)) return kCompact;
    return values <= (shared && what == kMa ? kLargeValuesSharedMa : kLargeValues) ? kMiddle : kLarge;
}

// Whether most of what a launch on aligned rows updates is in short components.  Above 64 workers stretches pay whatever the components (128 x 2.3 M
// of 15 K floats 1456 / 1463, of 23 K 1467 / 1389), as they do with 3 above 500 M values (3 x 200 M of 16 K 2530 / 2358, 3 x 233 M of 32 K 2930 / 2997), and 33 to 39 leave
// kMany's slots empty (33 x 0.9 M of 16 K 113, in stretches 111).  Up to 20 M values, much of which comes from the caches, it is the pages that a state has got that decide
// (side by side / in stretches, 4 x 3.8 M gossip-MA 25.2 / 18.2 or 17.2 / 18.1, 12 x 0.67 M 26.2 / 27.8 or 28.0 / 26.1).
int rows_layout(int K, int what, int size, int64_t values, const LongValues &in)
{
    if (size <= kCompact || (K == 3 && size == kLarge) || (K > 32 && K < 40) || K > 64) return kRows;
    return 2 * in.of[what][size == kLarge] < values ? kFine : kRows;
}

// Which sizes a call of this plan can have: without periods a call updates everything.
bool size_occurs(const gbmuf_plan_s &pl, int layout, int what, int size)
{
    const int64_t values = pl.K * pl.P;
    const int all = size_of_launch(values, layout, what), least = size_of_launch(0, layout, what);
    if (layout == kRows || layout == kFine) {
        // with periods parts that are all short or all long may be due
        const int64_t in_long = pl.long_values.of[what][size == kLarge];
        const bool part = pl.has_periods && (layout == kFine ? rows_layout(pl.K, what, size, 1, LongValues{}) == kFine && in_long < values : in_long > 0);
        if (rows_layout(pl.K, what, size, values, pl.long_values) != layout && !part) return false;
    }
    return size == all || (pl.has_periods && size < all && size >= least);
}

// Rows that share lines, launches that the caches hold: bound by latency.  One slot per thread, and no more threads than
// make a tile of 16 columns; more workers than that take 1024 x 4 [10 % from the best of every point]: the wider kVeryMany leaves
// most CUs without a tile.  Gossip-MA, with a third of the loads, takes two slots [3 %; one 6 %].
Variant cached_variant(int K, int what)
{
    Variant v{1024, 4, 4};
    if (what == kMa) {
        if (K <= 64) find_variant(K <= 32 ? 256 : 512, 2, &v);
        else if (K <= 128) find_variant(512, 4, &v);
    } else if (K <= 64) {
        find_variant(K <= 16 ? 512 : 1024, K <= 32 ? 1 : 2, &v);
    }
    return v;
}

// log2 of the largest power of two T with K * T <= the shape's slots.
int32_t widest_tile(const Variant &v, int K)
{
    int32_t lg = 0;
    while ((static_cast<int64_t>(K) << (lg + 1)) <= static_cast<int64_t>(v.threads) * v.slots) ++lg;
    return lg;
}

// Rows that share lines: whether 3 to 16 workers take 1024 x 1, whose slots K rows fill to 7/8 up to 8 workers, above 500 M values to
// 3/4, and to 15/16 from 9 on (6 x 133 M 1024 x 1 3639 us, 512 x 1 3720; 14 x 57 M 3857 / 3749; 14 x 7.1 M 480 / 474).
bool shared_wide(int K, int size)
{
    const int rows = K << widest_tile({1024, 1, 1}, K);
    return K == 3 || (K <= 16 && rows >= (K > 8 ? 960 : size == kLarge ? 768 : 896));
}

// Rows that share lines, beyond the caches: 3K address streams, of which each access touches one line more than it needs.  All wide
// shapes end within 5 % of each other: 5.4 TB/s with 4 workers, 5.1 to 5.8 with 16, by placement, and 4.9 from 64 on.
//   BMUF: up to 2 workers 512 x 2, one per CU (2 x 350 M 3069 us, 256 x 1 3250), up to 16 1024 x 1 where K rows fill its slots (8 x 75 M 2735,
//     kSixtyFour 2870; 16 x 37.5 M 2819 / 2873), and with 3 workers (3 x 233 M 3132, 512 x 1 3179), else 512 x 1 (6 x 33 M
//     914, kSixtyFour 931; 12 x 16.7 M 927 / 938), up to 64 kSixtyFour (32 x
//     18.8 M 2887, 1024 x 2 2948; 48 x 12.5 M 2885 / 2965), but 33 to 39 kMany, one per CU (33 x 24 M 3792, kSixtyFour 3954; 36 x 8.3 M 1435 / 1462), above 1024 x 4 (200 x 3 M 2970, kVeryMany 2988), large up to 128 kMany (96 x 6.2 M 2929,
//     1024 x 4 3008; 128 x 0.5 M 366 / 356), large above 256 kVeryMany (300 x 2 M 3100), above 512 at all sizes (1024 x 4 20 to 50 % more).
//   gossip-MA: 2 and 4 workers 256 x 4, three per CU (2 x 40 M 111 us, 512 x 2 114; 4 x 30 M 166 / 174), 1 and 3 512 x 2, above 149 M values 1024
//     x 4 (4 x 75 M 428, 256 x 4 445), 2 workers 512 x 8, two per CU (2 x 150 M 415, 1024 x 4 424, 256 x 4 441), up to 16 256 x 2 (16 x 25 M 600, 256 x 4 609), up to 32 256 x 4, up to
//     64 512 x 4 (64 x 6.2 M 629, 1024 x 4 632), up to 128 1024 x 4, above kVeryMany (200 x 2 M 657, 1024 x 4 710).
Variant shared_variant(int K, int what, int size, bool few)
{
    Variant v{1024, 4, 4};
    const bool large = size == kLarge;
    if (size == kCompact) return cached_variant(K, what);
    if (what == kMa) {
        if (few && K > 128) return kVeryMany;
        if ((K == 2 || K == 4) && !large) find_variant(256, 4, &v);
        else if (K <= 4 && !large) find_variant(512, 2, &v);
        else if (K == 2) find_variant(512, 8, &v);
        else if (K > 4 && K <= 32) find_variant(256, K <= 16 ? 2 : 4, &v);
        else if (K > 32 && K <= 64) find_variant(512, 4, &v);
    } else {
        if (few && (K > 512 || (K > 256 && large))) return kVeryMany;
        if (K <= 2) find_variant(512, 2, &v);
        else if (shared_wide(K, size)) find_variant(1024, 1, &v);
        else if (K <= 16) find_variant(512, 1, &v);
        else if (K <= 32 || (K >= 40 && K <= 64)) v = kSixtyFour;
        else if (K < 40 || (K <= 128 && large)) v = kMany;
    }
    return v;
}

// Gossip-MA on aligned rows beyond the caches: whether components that draw more than 4 neighbours, whose averages take longer, need more workgroups per CU
// than the wide shapes leave (33 to 64 workers: one), or tiles side by side.  us, shapes for few neighbours / smaller ones: 6 neighbours, 64 x 0.9 M 91.3 / 78.0, 40 x 0.55 M
// 42.7 / 35.9, 20 x 30 M 926 / 858, 12 x 50 M 840 / 772; 5, 2 and 7 in turn, 48 x 0.9 M 78.5 / 62.7, 8 x 7.5 M 75.9 / 69.7; 9, 28 x 5.4 M 272.5 / 257; but 6, 28 x 5.4 M 204.5 / 214.8, and 5, 6 x 10 M 71.9 / 76.7.
bool long_averages(int K, int q) { return q > 4 && K > 6 && (K <= 24 || (K > 32 && K <= 64) || !draws_in_registers(q)); }

// Rows that are so long that tiles of 64 columns in stretches lose where there are more than 16 of them: each then lies in address ranges of its own that have to be
// translated.  us, side by side / in stretches, by the floats of a row, 50 M values of them due: 66 workers 20 M 197.5 / 202.8, 28 M 200 / 220, 42 M 198 / 238; 128 workers 20 M 198.7 / 199.9, 28 M
// 198 / 212, 42 M 199 / 227; all of 96 workers' 12 M 5181 / 4860, 20 M 9275 / 8539 or 7407 / 7555, 34 M 12567 / 14402; gossip-MA of all of 66 workers' 16 M 1557 / 1588, 24 M 2228 / 2529, 42 M 4065 / 5280.
bool far_rows(int64_t P) { return P > 22000000; }

// How the fused kernel runs where no line is shared, by K, layout, branch and size of the launch: the shape, the resident
// workgroups per CU (0: as many as fit) and which XCD takes which tiles (tile_of_block).  Each rule holds over a whole range
// of K and is what came out best or within 1 to 3 % of it in sweeps of all built-in shapes, bounds and runs on K = 2 .. 400,
// 1 M .. 1.5 G values; TB/s of the rule, then the nearest rival.
//   Tiny and small launches want many tiles: up to 64 workers as few slots as give tiles of 8 columns and more (64 workers, 1 M values
//     5.6 us, 1024 slots 5.9, 4096 9.5; 3 M 12.7, 13.0, 14.4). Of more workers small ones stream omega and Delta (kMany: 128 x 20 K 10.9, 1024 x 4 12.1; 200 x 24 K 18.8, 20.2); tiny ones
//     do not, which would be 6 to 16 % faster up to 512 workers and 8 to 15 % slower for 600 (128 x 9 K 9.7, 1024 x 4 11.3; 600 x 2.3 K 16.3, 13.9).
//   Blocked state is one stretch of memory, and every tile shape that keeps 512 bytes to 1 KB of a row together is fast: 6.7 to 6.85
//     up to 64 workers.  An XCD takes 1 KB of each row in one run (xcd 6): 8 x 300 M / 8 1045 us, tile by tile 1065; from 33 to 128
//     workers, and beyond the caches up to 256 and above 512, one tile, and these move on from block to block (rotate), without which an
//     XCD sees the same addresses modulo 4 KB in every block: 64 x 23.4 M 5356 us, not rotated 5425 (1 KB) and more; 160 x 1.9 M 1091, 1100; but 257 to 512,
//     whose tiles hold 256 bytes of a row (300 x 1 M 1244, one tile moving on 1314; 400 x 1.8 M 2976 / 3129),
//     481 to 512 in tiles of 128 bytes, which they fill, and runs of 4 KB (512 x 0.6 M 1378, kVeryMany 1411).
//     No bound of the residency helps above 4 workers; up to 2 three per CU (2 x 300 M 2165 us, six 2517), 3 and 4 six
//     (3 x 333 M 3511, four 3727, unbounded 3553; 4 x 250 M 3554, 3492, 3562), but five where components draw different numbers of neighbours, whose
//     tiles load sooner (4 x 225 M 3153, six 3187), and then two with 17 to 32 workers (24 x 4.2 M 356, unbounded 359).  Up to 8 workers 256 x 1, 9-16 512 x 1 where K rows fill its
//     slots to 7/8, else 256 x 2, whose threads idle in whole slots (12 x 25 M 1051 us; 512 x 1 1080), 17-32 512 x 2, 33-64 kSixtyFour (40 x
//     7.5 M 1070 us, 512 x 4 1092; 44 x 9.1 M 1422, 1459; 64 x 4.7 M 1070, 1085), 65-128 kMany, above kVeryMany (160 x 1.9 M 1092, kMany
//     1290; 300 x 1 M 1244, 1250; 300 x 4.3 M 5467, 5737), 5 to 20 M values kSixtyFour (200 x 0.1 M 84 us, kMany 88).
//   Aligned rows are 3K address streams: 6.4 with 4 workers, 5.8 with 32, 5.5 with 128, in tiles whose stretches lie 32 KB apart (tiles_apart), the more of them
//     the better until one tile is all that a CU holds.  1, 2 and 4 256 x 2, two per CU (4 x 112 M 1670 us; 1024 x 1 1670, 256 x 1 1720), 3 512 x 1 (3 x 8.3 M 94.6;
//     256 x 1 98.3; kSixtyFour 94.8, but 96.9 in 87 components, whose ends cut its wide tiles, 512 x 1 94), 5-8 kSixtyFour (8 x 56 M 1693, 1024 x 2 1706), 9-32 kMany (24 x 42 M 4014, 1024 x 4 4039, kSixtyFour 4536; 12 x 58 M 2676,
//     kSixtyFour 2738), but 13-16 kSixtyFour (16 x 28 M 1744, kMany 1779; 14 x 50 M in components of 300 K floats 2726, kMany 2777), 33-128 kVeryMany (48 x 21 M 4240, 1024 x 4 4252; 64 x 15.6 M 4206, kMany 4298), tile by tile (64 x 15.6 M 4206, 4 KB
//     per XCD 4288), above 128 too, where a stretch is all of a tile and 4 KB of a row go to one XCD (300 x 0.8 M 1209, tile by tile 1259).
//     In short components (rows_layout) tiles lie side by side and are smaller: up to 4 256 x 1, four per CU (4 x 75 M 1127, 256 x 2 in stretches 1273), 5 and 6 512 x 1 (6 x 117 M 2710, 256 x 2
//     2785, kSixtyFour in stretches 2915), 7 and 8 256 x 2, two per CU (8 x 87 M 2774, 512 x 1 2955, kSixtyFour in stretches 3063), 9-32 kSixtyFour (12 x 58 M 2790, kMany in stretches 3194); 40-64 in stretches still, kMany (48 x 0.6 M 103.3 us,
//     kVeryMany 107.5), of rows far from each other (far_rows) 512 x 4 side by side
//     (64 x 0.5 M of rows of 60 M 112.2, kMany 117.6), large kVeryMany (48 x 14.6 M 3184, kMany 3289); 65-128 workers' rows far from each other side by side too, 512 x 4, large kVeryMany.
//     5 to 20 M values: up to 8 256 x 1, four per CU (2 x 6 M 46.8 us, 512 x 1 47.1; 8 x 0.75 M 21.9, 1024 x 1 22.5; 5 x 1.6 M 30.9, 34.7), up to 32 kSixtyFour (16 x 0.75 M 50.7,
//     256 x 4 52.3), above 1024 x 4 (40 x 0.3 M 55.2, kMany 55.9), 4 KB per XCD from 17 on.
//   Gossip-MA has a third of the loads and takes more slots per thread.  Blocked: up to 2 workers 256 x 1, but 2 of
//     more than 500 M values 512 x 2, two per CU (2 x 650 M 1610 us, 256 x 1 1817), 4 512 x 2 (4 x 175 M 848, 256 x 2 898; two per CU 837, but 4 x 5.2 M 6 %
//     more), up to 16 256 x 2 where K rows
//     fill it to 7/8 (8 x 75 M 723 us; 512 x 2 748), and 5 and 6 (5 x 140 M 923, 256 x 4 1050; 6 x 50 M 362 / 402), of 7 and more
//     workers six per CU (16 x 119 M, three states in turn, 2224 us, unbounded 2246, five 2244, four 2404; 7 x 271 M 2495 / 2580; 14 x 136 M 2277 / 2338; 5 x 380 M 2580 / 2496; with 5 neighbours
//     16 x 119 M 2311 / 2314, five 2446), else 256 x 4, up to 32 256 x 4 (725; 512 x 2 735), 33-64 512 x 4, above 1024 x 4, large of
//     more than 256 workers kVeryMany (300 x 2 M 947; 956).  Rows, in stretches: up to 8 512 x 2 where K rows fill 1024 slots to 7/8 (4 x 100 M 481, 512 x 4 488), up to
//     24 512 x 4 (12 x 33 M 499, 512 x 2 513; 6 x 17 M 124, 512 x 2 129), up to 32 kMany (32 x 12.5 M 528, 512 x 4 545), above kVeryMany (64 x 15.6 M 1340, kMany 1379; 300 x 2 M 1003,
//     1024 x 4 1089); smaller ones where averages are long (long_averages); 3 side by side, 256 x 2 (3 x 20 M 64.1; 256 x 4 in stretches 67.1; but 3 x 100 M 368 / 358), short components up to 8 256 x 2 (6 x 50 M 364; 512 x 4 in stretches 439), up to
//     24 256 x 4 (12 x 25 M 380; 512 x 4 413).  5 to 20 M values: 256 x 2 up to 64 workers, up to 128 512 x 2.
void aligned_shape(int K, int64_t P, int layout, int what, int size, int q, bool mixed, LayoutCfg &cfg)
{
    Variant &v = cfg.variant;
    int &bound = cfg.workgroups_per_cu, &run = cfg.xcd_columns_log;
    v = Variant{1024, 4, 4};
    bound = 0; run = 0; cfg.rotate = false;
    const bool blocked = layout == kBlocked, few = draws_in_registers(q), smaller = (layout == kFine && K <= 32) || (!blocked && long_averages(K, q));
    const auto fills = [K](int slots) { return (K << widest_tile({slots, 1, 1}, K)) * 8 >= slots * 7; };
    if (what == kMa) {
        if (size <= kSmall) v = cached_variant(K, what);
        else if (size <= kCompact) find_variant(K <= 64 ? 256 : K <= 128 ? 512 : 1024, K <= 128 ? 2 : 4, &v);
        else if (blocked && (K == 4 || (K == 2 && size == kLarge))) {
            find_variant(512, 2, &v);
            if (K == 2) bound = 2;
        }
        else if (blocked && K <= 2) find_variant(256, 1, &v);
        else if (smaller) {
            if (K <= 24) find_variant(256, K <= 8 ? 2 : 4, &v);
        }
        else if (!blocked) {
            if (K == 3) find_variant(256, 2, &v);
            else if (K <= 24) find_variant(512, K <= 8 && fills(1024) ? 2 : 4, &v);
            else if (K <= 32) v = kMany;
            else if (few) v = kVeryMany;
        }
        else if (K == 5 || K == 6 || (K <= 16 && fills(512))) {
            find_variant(256, 2, &v);
            if (K > 6) bound = 6;
        }
        else if (K <= 32) find_variant(256, 4, &v);
        else if (K <= 64) find_variant(512, 4, &v);
        else if (few && (K > 512 || (K > 256 && size == kLarge))) v = kVeryMany;
    } else if (size <= kSmall) {
        if (K <= 64) find_variant(K <= 16 && (blocked || K > 2) ? 256 : 512, 1, &v);
        else if (size == kSmall) v = kMany;
    } else if (blocked) {
        if (K <= 8) find_variant(256, 1, &v);
        else if (K <= 16 && fills(512)) find_variant(512, 1, &v);
        else if (K <= 16) find_variant(256, 2, &v);
        else if (K <= 32) find_variant(512, 2, &v);
        else if (K <= 64) v = kSixtyFour;
        else if (K <= 128) v = kMany;
        else if (size == kCompact && K <= 256) v = kSixtyFour;
        else if (size != kCompact && few && !(K > 480 && K <= 512)) v = kVeryMany;
        else if (size != kCompact && few) find_variant(512, 8, &v);
        else v = kMany;
        if (K <= 4) bound = K <= 2 ? 3 : mixed ? 5 : 6;
        else if (mixed && K > 16 && K <= 32) bound = 2;
    } else {
        if (size == kCompact) {
            if (K <= 8) find_variant(256, 1, &v);
            else if (K <= 32) v = kSixtyFour;
            if (K <= 8) bound = 4;
        } else if (layout == kFine && (K <= 32 || size != kLarge)) {
            if (K <= 4) find_variant(256, 1, &v);
            else if (K <= 6) find_variant(512, 1, &v);
            else if (K <= 8) find_variant(256, 2, &v);
            else if (K > 32 && far_rows(P)) find_variant(512, 4, &v);
            else v = K <= 32 ? kSixtyFour : kMany;
            if (K <= 4) bound = 4;
            else if (K == 7 || K == 8) bound = 2;
        } else {
            if (K <= 2 || K == 4) find_variant(256, 2, &v);
            else if (K == 3) find_variant(512, 1, &v);
            else if (K <= 8 || (K > 12 && K <= 16)) v = kSixtyFour;
            else if (K <= 32) v = kMany;
            else if (K > 64 && K <= 128 && size != kLarge && far_rows(P)) find_variant(512, 4, &v);
            else if (few) v = kVeryMany;
            if (K <= 2 || K == 4) bound = 2;
        }
    }
    if (size <= kSmall) return;
    if (blocked) {
        cfg.rotate = K > 32 && (what == kMa || K <= 128 || (size != kCompact && (K <= 256 || K > 512)));
        run = cfg.rotate ? 0 : K > 480 && K <= 512 && size != kCompact ? 8 : 6;
    } else {
        run = K > (size == kCompact || (what == kMa && (smaller || (K > 64 && far_rows(P)))) ? 16 : 128) ? 8 : 0;
    }
}
// Small plans with rows of more than 7 neighbours draw them through LDS in every workgroup (launch_bound), a thread a
// row: a chain that is hidden by many workgroups, not by large ones, and paid per tile.  9 neighbours, us, these
// shapes / the default ones: 36 workers x 0.33 M blocked 112 / 167, rows 85 / 166; 17 x 0.71 M blocked 107 / 135.
Variant lds_drawing_variant(int K, int layout)
{
    Variant v{1024, 4, 4};
    if (layout == kBlocked && K > 4) {
        if (K <= 64) find_variant(512, K <= 16 ? 1 : K <= 32 ? 2 : 4, &v);
    } else if (K <= 32) {
        find_variant(256, K <= 8 ? 1 : K <= 16 ? 2 : 4, &v);
    }
    return v;
}

// Rows that share lines: one workgroup per CU with up to 2 workers (2 x 350 M 3069 us, two 3200) and of kMany (96 x 6.2 M 2929, two 2976), four of 512 x
// 1, else two.  A state that stays in the cache has nothing to gain from a bound, and gossip-MA moves too little to need one but
// in the wide tiles of 2 and 4 workers (see above).
int shared_workgroups_per_cu(int K, int what, int size)
{
    if (size == kCompact) return 0;
    if (what == kMa) return size == kMiddle ? (K == 2 || K == 4 ? 3 : 0) : K == 2 ? 2 : 0;
    if (K <= 2 || (K > 32 && K < 40) || (K > 64 && K <= 128 && size == kLarge)) return 1;
    return K > 4 && K <= 16 && !shared_wide(K, size) ? 4 : 2;
}

// What a plan that names its shape gets if it does not name a bound: no bound on rows, few on blocked state.
int32_t named_workgroups_per_cu(int K, int layout, int what)
{
    if (layout == kRows || layout == kFine) return 0;
    if (what == kMa) return K <= 16 ? 4 : 2;
    return K <= 4 ? 4 : K <= 32 ? 2 : 1;
}

// Streamed: loads leave the L2 first, stores go through it at once.  Lines that were read are dead, and unless they leave first
// they push lines that were written out in an order that HBM takes worse: three arrays of 2 GB updated in place 5810
// GB/s, 5450 with plain accesses, either half alone 5420 to 5550.  Not where neighbouring tiles share lines, whose halves the L2 would
// no longer join (16 x 43.8 M odd rows 4023 us, plain 3255; tiles of 64 bytes, 1024 x 3 K 24 / 12), and not where all of a launch comes from the caches.  A plan's
// cache_hints ask for it at any size.
int choose_policy(int layout, int size, int logT, int hints)
{
    return layout != kShared && logT >= 3 && (size != kTiny || hints != 0) ? kStreamed : kPlain;
}

// Whether a launch's tiles lie in stretches 32 KB apart (tile_kernel): aligned rows whose tiles hold 64 columns and more, but for short components of
// up to 32 workers, gossip-MA of 3, some of its long averages, and more than 64 rows that are far from each other.  us on rows padded to 4 KB, each in the better of its shapes,
// stretches / side by side: 8 x 37 M 1107 / 1226, 16 x 18 M 1151 / 1286, 32 x 9.4 M 1221 / 1342, 64 x 4.7 M 1262 / 1400, 64 x 119 M 32121 / 35654, 128 x 2.3 M 1350 / 1463; gossip-MA 8 x 37 M 360 / 374,
// 24 x 12 M 356 / 426, 64 x 4.7 M 388 / 425.  Up to 5 M values all comes from the caches (2 x 3 M 21.2 / 21.9, 32 x 0.19 M 21.3 / 21.4), up to 20 M much: 16 x 0.75 M 38.1 / 41.6, of rows of 100 M 38.9 / 45.2,
// but above 16 workers, whose tiles hold 64 columns, as much is lost as gained (24 x 0.58 M 42.6 / 47.7, 24 x 0.25 M 24.1 / 22.3, 64 x 0.28 M 65.7 / 60.8) and a third of rows that are far from each other
// (32 x 0.33 M of rows of 53 M 51.0 / 39.3, 64 x 0.22 M of rows of 34 M 70.1 / 54.1).  Blocks of 32 KB have the pairs by themselves: a wave takes neighbouring workers' blocks.
bool tiles_apart(int K, int64_t P, int q, int layout, int what, int size, int logT, bool named)
{
    if (named || logT <= kLogStretch || logT > kLogApart) return false;
    if (layout == kFine ? K <= 32 : layout != kRows) return false;
    if (size <= kCompact) return size == kCompact && (what == kMa || K <= 16);
    if (K > 64 && far_rows(P)) return false;
    return what != kMa || (K != 3 && !(long_averages(K, q) && (K > 24 || !draws_in_registers(q))));
}

// Tiles of a component [a, b) at T columns each.
int64_t tiles_of(int64_t a, int64_t b, int64_t T) { return a < b ? (((b + 3) >> 2) + T - 1) / T - (a >> 2) / T : 0; }

int64_t count_tiles(const gbmuf_plan_s &pl, int32_t logT)
{
    int64_t count = 0;
    for (int32_t i = 0; i < pl.m; ++i)
        count += tiles_of(pl.off[static_cast<size_t>(i)], pl.off[static_cast<size_t>(i) + 1], static_cast<int64_t>(1) << logT);
    return count;
}

// Small plans draw in the kernel whatever q is, so that their syncs may run on several streams at once
// (gbmuf_info_t.in_kernel_sampling).  Small is 8192 tiles of about 32 columns, not of whatever width the rows
// shape has: rows of more than 7 neighbours are drawn through LDS, and that is slow.  In the kernel / separate,
// 16 workers, 8 neighbours, us: 1.0 M parameters (drawn in the kernel) 116 / 78, 2.1 M (separate) 229 / 154.
bool is_launch_bound(const gbmuf_plan_s &pl, const gbmuf_plan_desc_t *desc)
{
    const int slots = pl.named_shape ? desc->tile_threads * desc->tile_slots : pl.K <= 8 ? 256 : pl.K <= 16 ? 512 : pl.K <= 32 ? 1024 : 4096;
    return can_sample_inline(pl.K, pl.C) && pl.K <= slots && count_tiles(pl, widest_tile(Variant{slots, 1, 1}, pl.K)) <= 8192;
}

// Split every component into runs of at most T 16-byte columns (the fused kernel's work list).  Here only where every
// component's tiles begin; the list itself is written on the GPU (tile_kernel).
void build_tiles(const gbmuf_plan_s &pl, TileSet &ts)
{
    ts.tile_start.assign(static_cast<size_t>(pl.m) + 1, 0);
    for (int32_t i = 0; i < pl.m; ++i)
        ts.tile_start[static_cast<size_t>(i) + 1] = ts.tile_start[static_cast<size_t>(i)] +
            tiles_of(pl.off[static_cast<size_t>(i)], pl.off[static_cast<size_t>(i) + 1], static_cast<int64_t>(1) << ts.logT);
}

void free_device(gbmuf_plan_s &pl)
{
    if (pl.d_comp) (void)hipFree(pl.d_comp);
    if (pl.d_starts) (void)hipFree(pl.d_starts);
    if (pl.d_tiles) (void)hipFree(pl.d_tiles);
    if (pl.d_nbr) (void)hipFree(pl.d_nbr);
    for (TileSet &ts : pl.sets) ts.d_tiles = nullptr;
    pl.d_comp = nullptr; pl.d_starts = nullptr; pl.d_tiles = nullptr; pl.d_nbr = nullptr;
}

template <class T>
int upload(T **dst, const std::vector<T> &src)
{
    const size_t bytes = (src.empty() ? 1 : src.size()) * sizeof(T);
    hipError_t err = hipMalloc(reinterpret_cast<void **>(dst), bytes);
    if (err != hipSuccess) { *dst = nullptr; return hip_failed("hipMalloc(plan table)", err, GBMUF_ENOMEM); }
    if (!src.empty()) {
        err = hipMemcpy(*dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice);
        if (err != hipSuccess) return hip_failed("hipMemcpy(plan table)", err, GBMUF_EDEVICE);
    }
    return GBMUF_OK;
}

const LayoutCfg &cfg_of_all(const gbmuf_plan_s &pl, int layout, int what)
{
    return pl.cfg[layout][what][size_of_launch(pl.K * pl.P, layout, what)];
}

int make_device_state(gbmuf_plan_s &pl, int32_t sampling)
{
    int ndev = 0;
    hipError_t err = hipGetDeviceCount(&ndev);
    if (err != hipSuccess || ndev < 1) {
        hip_failed("hipGetDeviceCount", err, GBMUF_OK);
        (void)hipGetLastError();
        return GBMUF_OK;                                   // host-only plan
    }
    err = hipGetDevice(&pl.device);
    if (err != hipSuccess) return hip_failed("hipGetDevice", err, GBMUF_EDEVICE);
    int max_lds = 0;
    err = hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, pl.device);
    if (err != hipSuccess) return hip_failed("hipDeviceGetAttribute(MaxSharedMemoryPerBlock)", err, GBMUF_EDEVICE);
    pl.lds_per_cu = max_lds;                               // on this GPU one workgroup may take a CU's whole LDS
    err = hipDeviceGetAttribute(&pl.cus, hipDeviceAttributeMultiprocessorCount, pl.device);
    if (err != hipSuccess) return hip_failed("hipDeviceGetAttribute(MultiprocessorCount)", err, GBMUF_EDEVICE);
    {
        const int rc0 = resolve_scratch(pl.device);
        if (rc0 != GBMUF_OK) return rc0;
    }
    bool can = false;
    int rc = GBMUF_OK;
    std::vector<LayoutCfg> done;                            // every kernel that a call can launch, once
    for (int l = 0; l < kLayouts * kBranches * kSizes && rc == GBMUF_OK; ++l) {
        const int layout = l / kSizes / kBranches, what = l / kSizes % kBranches, size = l % kSizes;
        if (!size_occurs(pl, layout, what, size)) continue;
        for (int policy : {static_cast<int>(kPlain), pl.cfg[layout][what][size].policy}) {       // blocks may share lines: plain
            LayoutCfg c = pl.cfg[layout][what][size];
            c.policy = policy;
            if ((layout == kRows || layout == kFine) && policy != pl.cfg[layout][what][size].policy) continue;
            bool seen = false;
            for (const LayoutCfg &d : done)
                seen = seen || (d.policy == c.policy && d.variant.threads == c.variant.threads && d.variant.slots == c.variant.slots &&
                                d.variant.depth == c.variant.depth);
            if (seen || rc != GBMUF_OK) continue;
            done.push_back(c);
            rc = prepare_kernel(c.variant, c.policy, pl.K, pl.q, pl.mixed_q, pl.C, &can);
        }
    }
    if (rc != GBMUF_OK) return rc;
    if (sampling == GBMUF_SAMPLING_IN_KERNEL && !can) return GBMUF_EUNSUPPORTED;
    pl.sampling = sampling;
    if ((rc = upload(&pl.d_comp, pl.comp)) != GBMUF_OK) return rc;
    // The tile lists, 16 bytes a tile and millions of tiles for a large model, are written where they are used: 74 us for a
    // plan of 8 x 19.8 M, 156 of 16 x 278.6 M; built here and copied 684 and 21076.
    std::vector<int64_t> starts(pl.off);
    int64_t tiles = 0;
    for (int s = 0; s < pl.n_sets; ++s) {
        starts.insert(starts.end(), pl.sets[s].tile_start.begin(), pl.sets[s].tile_start.end());
        tiles += pl.sets[s].tile_start.back();
    }
    if ((rc = upload(&pl.d_starts, starts)) != GBMUF_OK) return rc;
    err = hipMalloc(reinterpret_cast<void **>(&pl.d_tiles), static_cast<size_t>(tiles ? tiles : 1) * sizeof(TileDesc));
    if (err != hipSuccess) {
        pl.d_tiles = nullptr;
        return hip_failed("hipMalloc(tile lists)", err, GBMUF_ENOMEM);
    }
    TileDesc *next = pl.d_tiles;
    for (int s = 0; s < pl.n_sets; ++s) {
        TileSet &ts = pl.sets[s];
        ts.d_tiles = next;
        next += ts.tile_start.back();
        rc = launch_tiles(TileArgs{pl.d_starts, pl.d_starts + static_cast<int64_t>(s + 1) * (pl.m + 1), pl.d_comp, ts.d_tiles,
                                   ts.tile_start.back(), pl.m, ts.logT, ts.apart ? 1 : 0}, nullptr);
        if (rc != GBMUF_OK) return rc;
    }
    err = hipStreamSynchronize(nullptr);                   // calls may come on any stream
    if (err != hipSuccess) return hip_failed("hipStreamSynchronize(tile lists)", err, GBMUF_EDEVICE);
    const size_t n = static_cast<size_t>(pl.m) * pl.K * pl.q;
    err = hipMalloc(reinterpret_cast<void **>(&pl.d_nbr), (n ? n : 1) * sizeof(int32_t));
    if (err != hipSuccess) {
        pl.d_nbr = nullptr;
        return hip_failed("hipMalloc(neighbour scratch)", err, GBMUF_ENOMEM);
    }
    pl.has_device = true;
    return GBMUF_OK;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Device calls need the plan's GPU to be the current one: its tables live there.
int check_device(const gbmuf_plan_s *pl)
{
    if (!pl->has_device) return GBMUF_EDEVICE;
    int dev = -1;
    const hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return hip_failed("hipGetDevice", err, GBMUF_EDEVICE);
    if (dev != pl->device) return hip_failed("current device is not the plan's device", hipErrorInvalidDevice, GBMUF_EDEVICE);
    return GBMUF_OK;
}

// Do the floats two arrays of one state cover intersect?  Array X covers, for every worker w
// (and block g), `run` floats from X + g*group + w*stride.  Two such sets meet iff some
// combination d + dg*group + dw*stride lies within (-run, run); the nearest candidates decide
// because the rows of one block group do not reach into the next (validated by the caller).
bool arrays_overlap(const float *x, const float *y, int64_t K, int64_t stride, int64_t run, int64_t groups,
                    int64_t group)
{
    if (!x || !y || run <= 0) return false;
    const std::ptrdiff_t d_bytes = reinterpret_cast<const char *>(y) - reinterpret_cast<const char *>(x);
    const double d = static_cast<double>(d_bytes) / 4.0;      // in floats; a fraction still orders correctly
    auto near = [](double target, double step, int64_t limit, int64_t out[3]) {
        int64_t c = step > 0 ? static_cast<int64_t>(target / step + (target >= 0 ? 0.5 : -0.5)) : 0;
        int n = 0;
        for (int64_t k = c - 1; k <= c + 1; ++k) out[n++] = k < -limit ? -limit : (k > limit ? limit : k);
    };
    int64_t gs[3] = {0, 0, 0};
    if (groups > 1) near(-d, static_cast<double>(group), groups - 1, gs);
    for (int64_t dg : gs) {
        const double d2 = d + static_cast<double>(dg) * static_cast<double>(group);
        int64_t ws[3] = {0, 0, 0};
        if (K > 1) near(-d2, static_cast<double>(stride), K - 1, ws);
        for (int64_t dw : ws) {
            const double d3 = d2 + static_cast<double>(dw) * static_cast<double>(stride);
            if (d3 > -static_cast<double>(run) && d3 < static_cast<double>(run)) return true;
        }
    }
    return false;
}

// Validates a state description for this plan and turns it into the kernels' placement.
int check_state(const gbmuf_plan_s *pl, const gbmuf_state_t *st, bool need_slots, Placement *at, int *layout)
{
    if (!pl || !st || !st->theta) return GBMUF_EINVAL;
    if (need_slots && (!st->omega || !st->delta)) return GBMUF_EINVAL;
    int64_t run = pl->P, groups = 1, group = 0;
    if (st->block_floats == 0) {
        if (st->worker_stride < pl->P) return GBMUF_EINVAL;
        *at = Placement{st->worker_stride, 0, 62, 0};
        *layout = kRows;
    } else {
        const int64_t B = st->block_floats;
        if (B < 0 || (B & (B - 1)) != 0 || B > (static_cast<int64_t>(1) << 30)) return GBMUF_EINVAL;
        if (B < (static_cast<int64_t>(4) << pl->min_block_logT)) return GBMUF_EINVAL;
        if (st->worker_stride < B) return GBMUF_EINVAL;
        if (st->block_stride < static_cast<int64_t>(pl->K - 1) * st->worker_stride + B) return GBMUF_EINVAL;
        int32_t lg = 0;
        while ((static_cast<int64_t>(1) << lg) < B) ++lg;
        *at = Placement{st->worker_stride, st->block_stride - B, lg, 0};
        *layout = kBlocked;
        run = B; groups = (pl->P + B - 1) / B; group = st->block_stride;
    }
    const float *arr[3] = {st->theta, need_slots ? st->omega : nullptr, need_slots ? st->delta : nullptr};
    for (int a = 0; a < 3; ++a)
        for (int b = a + 1; b < 3; ++b)
            if (arrays_overlap(arr[a], arr[b], pl->K, st->worker_stride, run, groups, group)) return GBMUF_EINVAL;
    return GBMUF_OK;
}

gbmuf_state_t rows_state(float *theta, float *omega, float *delta, int64_t stride)
{
    gbmuf_state_t st{};
    st.theta = theta; st.omega = omega; st.delta = delta;
    st.worker_stride = stride;
    return st;
}

// Groups of 8 runs that a launch on rows that share lines has at least, its runs being halved for it: tiles beyond the last whole group go
// to the XCDs one by one, and with 32 KB a run those are all of a row of less than 256 KB.  us, runs of 32 KB / halved: gossip-MA 128 x
// 12 K 8.6 / 6.2, 128 x 47 K 14.8 / 11.9; BMUF 16 x 50 K 6.9 / 5.3, 128 x 47 K 29.2 / 26.5.  With 8 or 16 groups 1 and 3 % more.
constexpr int64_t kLeastGroups = 4;

// Whether rows or blocks start inside 128-byte lines, so that neighbouring tiles share lines: unless both are taken by one XCD its
// L2 cannot join the halves, and every shared line is fetched twice and written in two pieces.  One XCD takes 32 KB of a
// row then, and one line in 256 is shared.  16 workers x 35.0 M in plain tensors, an earlier kernel: 3944 GB/s at 512 B, 4984 at 4 KB, 5073 at
// 16 KB; 64 workers x 26.9 M: 3880 at 1 KB, 4405 at 4 KB, 5163 at 32 KB.  (The stride of a single
// worker is no distance between rows: 1 x 600 M, odd stride, 2497 us; by 32 KB 2694.)
bool shares_lines(const Placement &at, const gbmuf_state_t *st, int32_t mode, int K)
{
    uintptr_t low = reinterpret_cast<uintptr_t>(st->theta) | (static_cast<uintptr_t>((K > 1 ? at.stride : 0) | at.block_extra) << 2);
    if (mode != GBMUF_MODE_GOSSIP_MA)
        low |= reinterpret_cast<uintptr_t>(st->omega) | reinterpret_cast<uintptr_t>(st->delta);
    return (low & 127u) != 0;
}

// The dynamic LDS a workgroup asks for so that at most `workgroups_per_cu` of them fit a CU.
size_t lds_floor(const gbmuf_plan_s *pl, const LayoutCfg &cfg)
{
    const int n = cfg.workgroups_per_cu;
    if (n <= 0 || n > 8 || pl->lds_per_cu <= 0) return 0;
    const int64_t share = pl->lds_per_cu / n - 2048;         // margin for the allocation granule
    return share > 0 ? static_cast<size_t>(share) : 0;
}

// How many resident one-wave workgroups per CU take `n` of them best, of which `aim` is best for very many.  The last round takes
// as long as 0.6 of a full one however few it has: 6, 7, 8 or, up to 14, all at once are taken so that it is not nearly empty; above
// 24 workgroups per CU it hardly counts.  128 x 0.59 M (8.9 per CU), odd rows: 8 resident 59.6 us, 6 52.1, 16 47.0; 96 x 0.94 M
// (14.3), padded: 8 54.1, 6 59.1; 256 x 0.47 M (7.2), blocked: 6 92.3, 8 70.7; 65 x 1.2 M (17.6), padded: 8 50.4, 6 43.7; 200 x 6.5 M (99),
// blocked: 6 747, 8 775.
int average_waves(double n, int aim)
{
    if (n > 24) return aim;
    int best = 16;
    double least = n <= 14 ? 1.02 * n : 1e30;
    for (int w = 6; w <= 8; ++w) {
        const double rounds = n / w, whole = std::floor(rounds), rest = rounds - whole;
        const double cost = (whole + (rest > 0 ? std::max(rest, 0.6) : 0)) * w * (1 + 0.005 * std::abs(w - aim));
        if (cost < least) { least = cost; best = w; }
    }
    return best;
}

// Rows in flight per thread, resident one-wave workgroups per CU (32: as many as fit), who reads what and how, for a final
// average.  us on MI355X, in the order of the rules:
//   sums of up to 20 M values come from the caches, which plain loads leave them in (64 x 0.16 M 7.4, streamed 8.1), and of up to 22 M
//     (theta 88 MB, of three states in turn) rows and blocks of up to 16 workers (8 x 2.6 M padded 15.4, 16.9; 5 x 4.2 M odd rows 16.2, 17.9; 7 x 3 M
//     blocked 15.8, 16.7; 48 x 0.44 M blocked 14.2, 13.6; from 25 M on 2 to 13 % the other way).  More waves hide their latency, with enough
//     rows per thread that few workers take one pass: 8 x 4.2 M padded 25 (16 rows x 3 waves 33), 1024 x 36 K 66 (8 rows 87).
//     More than 64 workers up to 35 M (300 x 83 K 22.7, streamed 24.0).
//   beyond, streamed: 8 x 25 M blocked 127, plain 145; 64 x 15.6 M padded 607, plain 674; also rows that share lines, of which nothing is written (8 x
//     5 M odd rows 30.4, plain 32.5; 200 x 1.5 M 179, 191).  Up to 60 M, and where rows are of up
//     to 4 workgroups per CU, without bound and with 16 rows of more than 64 workers in flight (1024 x 195 K 122, 4 rows x 6 waves 157).
//   one worker is a copy: 590 M 746, 16 waves 770, 8 waves 1303.
//   larger sums take 4 rows at a time, and the fewer waves the more workers there are, above 16 by the workgroups too
//     (average_waves): blocked 4 x 50 M 142 (12 waves), 64 x 3.1 M 119 (6; 8 rows x 4 125), 128 x 7.8 M 577 (6; 16 rows x 3 591); padded 16 x 62
//     M 630 (8).  Blocked 14 to 16
//     workers, who fill a batch of 16 rows: 16 x 4 (16 x 62 M 591, 4 x 8 603; 10 x 50 M 379, 4 x 8 315).  4 KB per XCD where rows share lines (2 x 100 M 185, workgroup by
//     workgroup 191) and for 9 to 64 workers of blocked state (32 x 116 M 2092 / 2130), but 33 to 64 of more than 500 M
//     values move on by an XCD from block to block as in the fused kernel (64 x 57.8 M 2177, 4 KB per XCD 2250; 64 x 3.1 M 121 / 119).
AverageShape average_shape(const gbmuf_plan_s *pl, int layout, bool shared_lines)
{
    const int K = pl->K;
    const int64_t values = static_cast<int64_t>(K) * pl->P;
    AverageShape s{};
    int waves = 32;
    const double groups = pl->cus > 0 ? static_cast<double>(pl->P) / 256 / pl->cus : 1e6;      // workgroups per CU
    const bool short_rows = groups <= 4;
    const int64_t cached = K > 64 ? 35000000 : K <= 2 || (layout == kBlocked && K > 16) ? kCompactValues : 22000000;
    if (values <= cached) {
        s.rows_in_flight = K <= 4 ? 4 : K <= 16 ? 8 : 16;
        s.xcd_log = K > 1 ? 2 : 0;
    } else {
        s.policy = kStreamed;
        s.rows_in_flight = K <= 64 || (values > 60000000 && !short_rows) ? 4 : 16;
        s.xcd_log = (K > 1 && shared_lines) || (layout == kBlocked && K > 8 && K <= 64) ? 2 : 0;
        if (values > 60000000 && !short_rows) {
            if (layout == kBlocked) {
                waves = K <= 3 ? 32 : K <= 7 ? 12 : K <= 13 ? 8 : K <= 16 ? 4 : average_waves(groups, 6);
                if (K > 13 && K <= 16) s.rows_in_flight = 16;
                s.rotate = K > 32 && K <= 64 && values > kLargeValues;
                if (s.rotate) s.xcd_log = 0;
            } else {
                waves = K == 1 ? 32 : K <= 3 ? 16 : K <= 7 ? 12 : K <= 16 ? 8 : average_waves(groups, K <= 128 ? 8 : 6);
            }
        }
    }
    if (waves < 32 && pl->lds_per_cu > 0) s.lds_floor = static_cast<size_t>(std::max(0, pl->lds_per_cu / waves - 2048));
    return s;
}

// What one call updates.
struct Due {
    int64_t values = 0;                                       // K times the elements of the components that are due
    LongValues long_values;
    int32_t first = 0, last = -1;                             // the first and the last component with elements among them
    bool one_run = true;                                      // they lie side by side, with none in between that is not due
};

Due due_all(const gbmuf_plan_s *pl) { return Due{pl->K * pl->P, pl->long_values, 0, pl->m - 1, true}; }

// The components that are due at this step, on the host: empty ones do not matter.
Due due_at(const gbmuf_plan_s *pl, uint64_t step)
{
    Due d;
    int64_t end = 0;
    for (int32_t i = 0; i < pl->m; ++i) {
        const int64_t a = pl->off[static_cast<size_t>(i)], b = pl->off[static_cast<size_t>(i) + 1];
        if (a == b || step % static_cast<uint64_t>(pl->periods[static_cast<size_t>(i)]) != 0) continue;
        if (d.last < 0) d.first = i;
        else if (a != end) d.one_run = false;
        d.last = i;
        end = b;
        d.values += pl->K * (b - a);
        d.long_values.add(pl->K, a, b);
    }
    return d;
}

// Whether a launch's workgroups draw its neighbour rows themselves.  That saves the sampler launch, about
// 5 us of a sync, and costs about 1 % of it where the rows are drawn in registers.  Measured, in the kernel /
// separate, us: 16 workers x 6.2 M 395 / 402, 20.6 M 1365 / 1373, 35.0 M 2045 / 2032, 166.1 M 10050 / 9880,
// 278.6 M 16715 / 16295; 8 x 20.6 M 639 / 643; 64 x 5.4 M 1311 / 1315, 9.3 M 2274 / 2277.  Gossip-MA moves a third
// of the bytes: 4 x 84.8 M 422 / 409, 18 x 4.3 M 157 / 164.  Rows of more than 7 neighbours are drawn through
// LDS, which only launch-bound plans do.
bool draws_itself(const gbmuf_plan_s *pl, int32_t mode, int64_t values)
{
    if (pl->sampling != GBMUF_SAMPLING_AUTO) return pl->sampling == GBMUF_SAMPLING_IN_KERNEL;
    return pl->launch_bound ||
           (draws_in_registers(pl->q) && values <= (mode == GBMUF_MODE_GOSSIP_MA ? kLargeValuesMa : kLargeValues));
}

int enqueue_sync(const gbmuf_plan_s *pl, const int32_t *nbr_dev, const gbmuf_state_t *st, const Placement &at,
                 int layout, float eta, float zeta, int32_t mode, hipStream_t stream, uint64_t round, const Due &due,
                 bool callers_table = false)
{
    const int what = mode == GBMUF_MODE_GOSSIP_MA ? kMa : kBmuf;
    const bool shared = shares_lines(at, st, mode, pl->K);
    if (layout == kRows)
        layout = shared ? kShared : rows_layout(pl->K, what, size_of_launch(due.values, kRows, what), due.values, due.long_values);
    const LayoutCfg &cfg = pl->cfg[layout][what][size_of_launch(due.values, layout, what)];
    const TileSet &ts = pl->sets[cfg.set];
    // One run of components is launched as exactly its tiles (the list is in component order); for several
    // runs one launch covers all tiles, and the workgroups of components that are not due return at once.
    const int64_t first = due.one_run && due.last >= 0 ? ts.tile_start[static_cast<size_t>(due.first)] : 0;
    const int64_t end = due.one_run && due.last >= 0 ? ts.tile_start[static_cast<size_t>(due.last) + 1]
                                                     : ts.tile_start.back();
    SyncArgs a{};
    a.tiles = ts.d_tiles + first;
    a.nbr = nbr_dev;
    a.comp = pl->d_comp;
    a.theta = st->theta; a.omega = st->omega; a.delta = st->delta;
    a.at = at;
    a.K = pl->K; a.q = pl->q; a.logT = cfg.logT; a.mode = mode;
    a.eta = eta; a.zeta = zeta; a.inv = pl->inv;
    a.flags = ((pl->alternate && (round & 1)) ? kFlagBackwards : 0) | (pl->mixed_q ? kFlagMixedQ : 0) |
              (due.one_run ? 0 : kFlagCheckPeriods) | (cfg.rotate ? kFlagRotate : 0) |
              (nbr_dev != nullptr && !callers_table ? kFlagSampledTable : 0);
    a.p = pl->p; a.C = pl->C;                               // used only when nbr_dev == nullptr
    a.key0 = static_cast<uint32_t>(pl->seed); a.key1 = static_cast<uint32_t>(pl->seed >> 32);
    a.round0 = static_cast<uint32_t>(round); a.round1 = static_cast<uint32_t>(round >> 32);
    a.step = round;
    a.xcd_log = std::max(0, (shared ? 11 : cfg.xcd_columns_log) - cfg.logT);
    while (shared && a.xcd_log > 0 && (end - first) >> (3 + a.xcd_log) < kLeastGroups) --a.xcd_log;
    return launch_sync(cfg.variant, shared ? kPlain : cfg.policy, a, end - first, lds_floor(pl, cfg), stream);
}

SampleArgs sample_args(const gbmuf_plan_s *pl, uint64_t round, int32_t *out)
{
    SampleArgs s{};
    s.comp = pl->d_comp;
    s.out = out;
    s.first_pair = 0;
    s.pairs = static_cast<int64_t>(pl->m) * pl->K;
    s.K = pl->K; s.p = pl->p; s.C = pl->C; s.q = pl->q; s.width = pl->q;
    s.mixed = pl->mixed_q ? 1 : 0;
    s.check_periods = 0;
    s.key0 = static_cast<uint32_t>(pl->seed); s.key1 = static_cast<uint32_t>(pl->seed >> 32);
    s.round0 = static_cast<uint32_t>(round); s.round1 = static_cast<uint32_t>(round >> 32);
    s.step = round;
    return s;
}

int check_mode(int32_t mode)
{
    return (mode < GBMUF_MODE_NO_RESTART || mode > GBMUF_MODE_GOSSIP_MA) ? GBMUF_EINVAL : GBMUF_OK;
}

// Argument checks shared by the sync entry points; argument errors come before device errors.
int check_sync(const gbmuf_plan_s *pl, const gbmuf_state_t *st, int32_t mode, Placement *at, int *layout)
{
    if (!pl || !st) return GBMUF_EINVAL;
    if (check_mode(mode) != GBMUF_OK) return GBMUF_EINVAL;
    const int rc = check_state(pl, st, mode != GBMUF_MODE_GOSSIP_MA, at, layout);
    if (rc != GBMUF_OK) return rc;
    return check_device(pl);
}

}  // namespace

extern "C" {

int gbmuf_plan_create(gbmuf_plan_t **out, const gbmuf_plan_desc_t *desc)
{
    if (!out) return GBMUF_EINVAL;
    *out = nullptr;
    if (!desc || desc->struct_size < sizeof(gbmuf_plan_desc_t)) return GBMUF_EINVAL;
    const int32_t m = desc->m, K = desc->K, p = desc->p;
    const int64_t *comp_offsets = desc->comp_offsets;
    if (!comp_offsets || m < 0 || K < 1 || desc->q < 0 || p < -1) return GBMUF_EINVAL;
    if (comp_offsets[0] != 0) return GBMUF_EINVAL;
    for (int32_t i = 0; i < m; ++i)
        if (comp_offsets[i + 1] < comp_offsets[i]) return GBMUF_EINVAL;
    if (desc->sampling < GBMUF_SAMPLING_AUTO || desc->sampling > GBMUF_SAMPLING_SEPARATE) return GBMUF_EINVAL;
    if (desc->sweep < GBMUF_SWEEP_AUTO || desc->sweep > GBMUF_SWEEP_FORWARD) return GBMUF_EINVAL;
    if (desc->cache_hints < 0 || desc->cache_hints > 3 || desc->workgroups_per_cu < 0) return GBMUF_EINVAL;
    if ((desc->tile_threads == 0) != (desc->tile_slots == 0)) return GBMUF_EINVAL;
    for (int32_t i = 0; desc->periods && i < m; ++i)
        if (desc->periods[i] < 1) return GBMUF_EINVAL;
    for (int32_t i = 0; desc->q_per_component && i < m; ++i)
        if (desc->q_per_component[i] < 0) return GBMUF_EINVAL;
    if (K > GBMUF_MAX_K) return GBMUF_EUNSUPPORTED;

    gbmuf_plan_s *pl = new (std::nothrow) gbmuf_plan_s;
    if (!pl) return GBMUF_ENOMEM;
    int rc = GBMUF_OK;
    try {
        pl->m = m; pl->K = K; pl->seed = desc->seed;
        // Beyond K-1 the listing of Definition 1 reaches nobody new (its first half alone has
        // passed every other worker), so larger degrees are the same topology.
        const int32_t want = p == 0 ? default_degree(K) : (p < 0 ? K / 2 : p);
        pl->p = want > K - 1 ? K - 1 : want;
        pl->off.assign(comp_offsets, comp_offsets + m + 1);
        pl->P = pl->off.back();
        if (desc->q_per_component) pl->qv.assign(desc->q_per_component, desc->q_per_component + m);
        else pl->qv.assign(static_cast<size_t>(m), desc->q);
        pl->q = desc->q_per_component ? 0 : desc->q;
        for (int32_t qi : pl->qv) {
            pl->q = std::max(pl->q, qi);
            if (qi != pl->qv.front()) pl->mixed_q = true;
        }
        pl->has_periods = desc->periods != nullptr;
        if (desc->periods) pl->periods.assign(desc->periods, desc->periods + m);
        else pl->periods.assign(static_cast<size_t>(m), 1);
        pl->inv = 1.0f / static_cast<float>(pl->q + 1);
        pl->comp.resize(static_cast<size_t>(m));
        for (int32_t i = 0; i < m; ++i)
            pl->comp[static_cast<size_t>(i)] = CompDesc{1.0f / static_cast<float>(pl->qv[static_cast<size_t>(i)] + 1),
                                                       pl->periods[static_cast<size_t>(i)],
                                                       pl->qv[static_cast<size_t>(i)], 0};
        for (int32_t i = 0; i < m; ++i) pl->long_values.add(K, comp_offsets[i], comp_offsets[i + 1]);

        std::vector<int32_t> ring;
        ring_of(0, K, pl->p, ring);
        pl->C = static_cast<int32_t>(ring.size());
        if (pl->q > pl->C) rc = GBMUF_EINVAL;              // the paper requires q <= 2p
        if (rc == GBMUF_OK) {
            pl->cand.resize(static_cast<size_t>(K) * pl->C);
            for (int32_t w = 0; w < K; ++w) {
                ring_of(w, K, pl->p, ring);
                if (pl->C > 0)
                    std::memcpy(pl->cand.data() + static_cast<size_t>(w) * pl->C, ring.data(),
                                sizeof(int32_t) * static_cast<size_t>(pl->C));
            }
            pl->named_shape = desc->tile_threads != 0;
            pl->alternate = desc->sweep == GBMUF_SWEEP_AUTO;
            pl->launch_bound = is_launch_bound(*pl, desc);
            const bool through_lds = !draws_in_registers(pl->q) && !pl->named_shape &&
                                     (desc->sampling == GBMUF_SAMPLING_IN_KERNEL || (desc->sampling == GBMUF_SAMPLING_AUTO && pl->launch_bound));
            for (int l = 0; l < kLayouts * kBranches * kSizes && rc == GBMUF_OK; ++l) {
                const int layout = l / kSizes / kBranches, what = l / kSizes % kBranches, size = l % kSizes;
                LayoutCfg &cfg = pl->cfg[layout][what][size];
                const bool few = draws_in_registers(pl->q);
                if (pl->named_shape) {
                    if (!find_variant(desc->tile_threads, desc->tile_slots, &cfg.variant) ||
                        K > cfg.variant.threads * cfg.variant.slots) { rc = GBMUF_EINVAL; break; }
                    pl->min_block_logT = widest_tile(cfg.variant, K);
                    cfg.workgroups_per_cu = named_workgroups_per_cu(K, layout, what);
                } else {
                    if (layout == kShared) {
                        cfg.variant = shared_variant(K, what, size, few);
                        cfg.workgroups_per_cu = shared_workgroups_per_cu(K, what, size);
                    } else {
                        aligned_shape(K, pl->P, layout, what, size, pl->q, pl->mixed_q, cfg);
                    }
                    if (through_lds) {
                        cfg.variant = lds_drawing_variant(K, layout);
                        cfg.workgroups_per_cu = 0;
                    }
                    // where the neighbour rows do not fit beside the widest tile, the next smaller one
                    if (sync_lds_bytes(cfg.variant, K, pl->q, pl->mixed_q, pl->C, can_sample_inline(K, pl->C)) > kLdsPerWorkgroup)
                        find_variant(1024, 4, &cfg.variant);
                    // Blocks may be narrower than a tile: the kernel looks an element's block up column by column
                    // (where a thread keeps its column, T <= threads, which holds for all shapes of more than 2 workers).
                    pl->min_block_logT = widest_tile(Variant{K <= 16 ? 1024 : K <= 64 ? 2048 : 4096, 1, 1}, K);
                }
                cfg.logT = widest_tile(cfg.variant, K);
                cfg.policy = choose_policy(layout, size, cfg.logT, desc->cache_hints);
                cfg.apart = tiles_apart(K, pl->P, pl->q, layout, what, size, cfg.logT, pl->named_shape);
                if (cfg.apart) cfg.policy = kApart;
                if (desc->workgroups_per_cu != 0) cfg.workgroups_per_cu = desc->workgroups_per_cu;
            }
            if (rc == GBMUF_OK) {
                // one tile list per distinct tile width
                for (int l = 0; l < kLayouts * kBranches * kSizes; ++l) {
                    const int layout = l / kSizes / kBranches, what = l / kSizes % kBranches, size = l % kSizes;
                    if (!size_occurs(*pl, layout, what, size)) continue;
                    LayoutCfg &cfg = pl->cfg[layout][what][size];
                    int found = -1;
                    for (int s2 = 0; s2 < pl->n_sets; ++s2)
                        if (pl->sets[s2].logT == cfg.logT && pl->sets[s2].apart == cfg.apart) found = s2;
                    if (found < 0) {
                        found = pl->n_sets++;
                        pl->sets[found].logT = cfg.logT;
                        pl->sets[found].apart = cfg.apart;
                        build_tiles(*pl, pl->sets[found]);
                    }
                    cfg.set = found;
                }
                rc = make_device_state(*pl, desc->sampling);
            }
        }
    } catch (const std::bad_alloc &) {
        rc = GBMUF_ENOMEM;
    }
    if (rc != GBMUF_OK) {
        free_device(*pl);
        delete pl;
        return rc;
    }
    *out = pl;
    return GBMUF_OK;
}

int gbmuf_plan(gbmuf_plan_t **out, const int64_t *comp_offsets, int32_t m, int32_t K, int32_t q, int32_t p,
               uint64_t seed)
{
    gbmuf_plan_desc_t d;
    std::memset(&d, 0, sizeof(d));
    d.struct_size = sizeof(d);
    d.m = m; d.K = K; d.q = q; d.p = p; d.seed = seed;
    d.comp_offsets = comp_offsets;
    return gbmuf_plan_create(out, &d);
}

int gbmuf_plan_destroy(gbmuf_plan_t *plan)
{
    if (!plan) return GBMUF_OK;
    int rc = GBMUF_OK;
    if (plan->has_device) {
        if (hipDeviceSynchronize() != hipSuccess) rc = GBMUF_EDEVICE;
        free_device(*plan);
    }
    delete plan;
    return rc;
}

int gbmuf_plan_info(const gbmuf_plan_t *plan, gbmuf_info_t *info)
{
    if (!plan || !info) return GBMUF_EINVAL;
    std::memset(info, 0, sizeof(*info));
    info->m = plan->m; info->K = plan->K; info->q = plan->q; info->p = plan->p; info->C = plan->C;
    info->has_device = plan->has_device ? 1 : 0;
    info->P = plan->P;
    const int64_t values = plan->K * plan->P;
    const int layout = rows_layout(plan->K, kBmuf, size_of_launch(values, kRows, kBmuf), values, plan->long_values);
    const LayoutCfg &rows = cfg_of_all(*plan, layout, kBmuf), &blocked = cfg_of_all(*plan, kBlocked, kBmuf);
    info->n_tiles = plan->sets[rows.set].tile_start.back();
    info->tile_columns = 1 << rows.logT;
    info->threads = rows.variant.threads;
    info->seed = plan->seed;
    info->mixed_q = plan->mixed_q ? 1 : 0;
    info->has_periods = plan->has_periods ? 1 : 0;
    info->in_kernel_sampling = plan->has_device && draws_itself(plan, GBMUF_MODE_PAPER, values) &&      // then any part is, too
                                       draws_itself(plan, GBMUF_MODE_GOSSIP_MA, values) ? 1 : 0;
    info->tile_columns_blocked = 1 << blocked.logT;
    info->threads_blocked = blocked.variant.threads;
    info->workgroups_per_cu_blocked = blocked.workgroups_per_cu;
    info->tile_columns_blocked_ma = 1 << cfg_of_all(*plan, kBlocked, kMa).logT;
    info->min_block_floats = 4 << plan->min_block_logT;
    return GBMUF_OK;
}

int gbmuf_candidates_host(const gbmuf_plan_t *plan, int32_t w, int32_t *out_host)
{
    if (!plan || w < 0 || w >= plan->K || (!out_host && plan->C > 0)) return GBMUF_EINVAL;
    if (plan->C > 0)
        std::memcpy(out_host, plan->cand.data() + static_cast<size_t>(w) * plan->C,
                    sizeof(int32_t) * static_cast<size_t>(plan->C));
    return GBMUF_OK;
}

int gbmuf_neighbours_host(const gbmuf_plan_t *plan, uint64_t round, int32_t *out_host)
{
    if (!plan) return GBMUF_EINVAL;
    const int32_t width = plan->q, C = plan->C, K = plan->K;
    if (width == 0 || plan->m == 0) return GBMUF_OK;
    if (!out_host) return GBMUF_EINVAL;
    try {
        std::vector<int32_t> pool;
        pool.reserve(static_cast<size_t>(C));
        for (int32_t i = 0; i < plan->m; ++i) {
            const int32_t qi = plan->qv[static_cast<size_t>(i)];
            for (int32_t w = 0; w < K; ++w) {
                int32_t *row = out_host + (static_cast<size_t>(i) * K + w) * width;
                host_pick(plan->cand.data() + static_cast<size_t>(w) * C, C, qi, plan->seed, round,
                          static_cast<uint32_t>(i), static_cast<uint32_t>(w), pool, row);
                std::fill(row + qi, row + width, -1);
            }
        }
    } catch (const std::bad_alloc &) {
        return GBMUF_ENOMEM;
    }
    return GBMUF_OK;
}

int gbmuf_neighbours_device(const gbmuf_plan_t *plan, uint64_t round, int32_t *out_dev, void *stream)
{
    if (!plan) return GBMUF_EINVAL;
    const int rc = check_device(plan);
    if (rc != GBMUF_OK) return rc;
    if (plan->q == 0 || plan->m == 0) return GBMUF_OK;
    if (!out_dev) return GBMUF_EINVAL;
    return launch_sampler(sample_args(plan, round, out_dev), static_cast<hipStream_t>(stream));
}

int gbmuf_sync_state(const gbmuf_plan_t *plan, const gbmuf_state_t *state, float eta, float zeta, int32_t nesterov,
                     uint64_t round, void *stream)
{
    Placement at{};
    int layout = kRows;
    int rc = check_sync(plan, state, nesterov, &at, &layout);
    if (rc != GBMUF_OK) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const Due due = due_all(plan);
    if (draws_itself(plan, nesterov, due.values))
        return enqueue_sync(plan, nullptr, state, at, layout, eta, zeta, nesterov, s, round, due);
    rc = launch_sampler(sample_args(plan, round, plan->d_nbr), s);
    if (rc != GBMUF_OK) return rc;
    return enqueue_sync(plan, plan->d_nbr, state, at, layout, eta, zeta, nesterov, s, round, due);
}

int gbmuf_sync_static(const gbmuf_plan_t *plan, const gbmuf_state_t *state, float eta, float zeta, int32_t nesterov,
                      uint64_t round, void *stream)
{
    Placement at{};
    int layout = kRows;
    int rc = check_sync(plan, state, nesterov, &at, &layout);
    if (rc != GBMUF_OK) return rc;
    const int64_t entries = static_cast<int64_t>(plan->m) * plan->K * plan->q;
    if (entries > GBMUF_STATIC_TABLE_ENTRIES) {
        std::snprintf(gbmuf::g_detail, sizeof(gbmuf::g_detail),
                      "gbmuf_sync_static: the neighbour table has %lld entries, the static table holds %d",
                      static_cast<long long>(entries), GBMUF_STATIC_TABLE_ENTRIES);
        return GBMUF_EUNSUPPORTED;
    }
    int32_t *table = scratch_of(plan->device);
    if (!table) return hip_failed("no static table on this device", hipErrorInvalidDevice, GBMUF_EDEVICE);
    hipStream_t s = static_cast<hipStream_t>(stream);
    // the sampler fills every row the fused kernel reads, so nothing of an earlier call is seen
    rc = launch_sampler(sample_args(plan, round, table), s);
    if (rc != GBMUF_OK) return rc;
    return enqueue_sync(plan, table, state, at, layout, eta, zeta, nesterov, s, round, due_all(plan));
}

int gbmuf_sync(const gbmuf_plan_t *plan, float *replicas, float *global, float *delta, int64_t worker_stride,
               float eta, float zeta, int32_t nesterov, uint64_t round, void *stream)
{
    const gbmuf_state_t st = rows_state(replicas, global, delta, worker_stride);
    return gbmuf_sync_state(plan, &st, eta, zeta, nesterov, round, stream);
}

int gbmuf_sync_step_state(const gbmuf_plan_t *plan, const gbmuf_state_t *state, float eta, float zeta,
                          int32_t nesterov, uint64_t step, void *stream)
{
    Placement at{};
    int layout = kRows;
    int rc = check_sync(plan, state, nesterov, &at, &layout);
    if (rc != GBMUF_OK) return rc;
    if (!plan->has_periods) return gbmuf_sync_state(plan, state, eta, zeta, nesterov, step, stream);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const Due due = due_at(plan, step);
    if (due.last < 0) return GBMUF_OK;
    const int32_t *nbr = nullptr;                           // nullptr: workgroups draw their own rows
    if (!draws_itself(plan, nesterov, due.values)) {
        // only the components that are due are sampled: the launch spans first..last of them and
        // the threads of components in between that are not due leave without drawing
        SampleArgs sa = sample_args(plan, step, plan->d_nbr);
        sa.first_pair = static_cast<int64_t>(due.first) * plan->K;
        sa.pairs = static_cast<int64_t>(due.last - due.first + 1) * plan->K;
        sa.check_periods = 1;
        rc = launch_sampler(sa, s);
        if (rc != GBMUF_OK) return rc;
        nbr = plan->d_nbr;
    }
    return enqueue_sync(plan, nbr, state, at, layout, eta, zeta, nesterov, s, step, due);
}

int gbmuf_sync_step(const gbmuf_plan_t *plan, float *replicas, float *global, float *delta, int64_t worker_stride,
                    float eta, float zeta, int32_t nesterov, uint64_t step, void *stream)
{
    const gbmuf_state_t st = rows_state(replicas, global, delta, worker_stride);
    return gbmuf_sync_step_state(plan, &st, eta, zeta, nesterov, step, stream);
}

int gbmuf_sync_table_state(const gbmuf_plan_t *plan, const int32_t *nbr_dev, const gbmuf_state_t *state, float eta,
                           float zeta, int32_t nesterov, void *stream)
{
    Placement at{};
    int layout = kRows;
    if (plan && !nbr_dev && plan->q > 0 && plan->m > 0) return GBMUF_EINVAL;
    const int rc = check_sync(plan, state, nesterov, &at, &layout);
    if (rc != GBMUF_OK) return rc;
    return enqueue_sync(plan, nbr_dev ? nbr_dev : plan->d_nbr, state, at, layout, eta, zeta, nesterov,
                        static_cast<hipStream_t>(stream), 0, due_all(plan), nbr_dev != nullptr);
}

int gbmuf_sync_table(const gbmuf_plan_t *plan, const int32_t *nbr_dev, float *replicas, float *global,
                     float *delta, int64_t worker_stride, float eta, float zeta, int32_t nesterov, void *stream)
{
    const gbmuf_state_t st = rows_state(replicas, global, delta, worker_stride);
    return gbmuf_sync_table_state(plan, nbr_dev, &st, eta, zeta, nesterov, stream);
}

int gbmuf_final_average_state(const gbmuf_plan_t *plan, const gbmuf_state_t *state, float *out_dev, void *stream)
{
    if (!plan || !state || !out_dev) return GBMUF_EINVAL;
    Placement at{};
    int layout = kRows;
    int rc = check_state(plan, state, false, &at, &layout);
    if (rc != GBMUF_OK) return rc;
    if ((rc = check_device(plan)) != GBMUF_OK) return rc;
    const int K = plan->K;
    const AverageShape shape = average_shape(plan, layout, at.stride % 32 != 0 || reinterpret_cast<uintptr_t>(state->theta) % 128 != 0);
    return launch_final_average(state->theta, at, K, plan->P, 1.0f / static_cast<float>(K), out_dev, shape,
                                static_cast<hipStream_t>(stream));
}

int gbmuf_final_average(const gbmuf_plan_t *plan, const float *replicas, int64_t worker_stride, float *out_dev,
                        void *stream)
{
    const gbmuf_state_t st = rows_state(const_cast<float *>(replicas), nullptr, nullptr, worker_stride);
    return gbmuf_final_average_state(plan, &st, out_dev, stream);
}

int gbmuf_state_copy(const gbmuf_plan_t *plan, const gbmuf_state_t *dst, const gbmuf_state_t *src, int32_t which,
                     void *stream)
{
    if (!plan || !dst || !src || which < 0 || which > 7) return GBMUF_EINVAL;
    float *const d[3] = {dst->theta, dst->omega, dst->delta};
    const float *const s[3] = {src->theta, src->omega, src->delta};
    gbmuf_state_t dsel = *dst, ssel = *src;                 // only the selected arrays take part in the checks
    float **dp[3] = {&dsel.theta, &dsel.omega, &dsel.delta};
    float **sp[3] = {&ssel.theta, &ssel.omega, &ssel.delta};
    int first = -1;
    for (int a = 0; a < 3; ++a) {
        if (which & (1 << a)) {
            if (!d[a] || !s[a]) return GBMUF_EINVAL;
            if (first < 0) first = a;
        } else {
            *dp[a] = nullptr; *sp[a] = nullptr;
        }
    }
    if (first < 0) return GBMUF_OK;
    // check_state wants theta: validate the geometry with the first selected array in its place
    gbmuf_state_t dgeo = dsel, sgeo = ssel;
    dgeo.theta = d[first]; sgeo.theta = const_cast<float *>(s[first]);
    Placement dat{}, sat{};
    int dl = kRows, sl = kRows;
    int rc = check_state(plan, &dgeo, false, &dat, &dl);
    if (rc != GBMUF_OK) return rc;
    if ((rc = check_state(plan, &sgeo, false, &sat, &sl)) != GBMUF_OK) return rc;
    if ((rc = check_device(plan)) != GBMUF_OK) return rc;
    CopyArgs c{};
    int n = 0;
    for (int a = 0; a < 3; ++a) {
        if (!(which & (1 << a))) continue;
        c.dst[n] = d[a];
        c.src[n++] = s[a];
    }
    c.da = dat; c.sa = sat;
    c.P = plan->P; c.K = plan->K;
    return launch_state_copy(c, n, static_cast<hipStream_t>(stream));
}

int gbmuf_recommend_layout(const gbmuf_plan_t *plan, int64_t P, int32_t K, int32_t kind, gbmuf_layout_t *out)
{
    if (!out || P < 0 || K < 1 || (kind != GBMUF_LAYOUT_ROWS && kind != GBMUF_LAYOUT_BLOCKED)) return GBMUF_EINVAL;
    if (plan && (plan->K != K || plan->P != P)) return GBMUF_EINVAL;
    std::memset(out, 0, sizeof(*out));
    if (kind == GBMUF_LAYOUT_ROWS) {
        const int64_t row = (P + 1023) / 1024 * 1024;      // rows start on 4 KB: tiles cover whole cache lines
        out->worker_stride = 3 * row;
        out->omega_offset = row;
        out->delta_offset = 2 * row;
        out->arena_floats = static_cast<int64_t>(K) * 3 * row;
        return GBMUF_OK;
    }
    // 32 KB blocks: K = 16 runs within a point of its best (8-32 KB), K = 64 at its best; 64 KB
    // blocks lose 7-10 points for both.  A plan with very wide tiles needs more.
    int64_t B = 8192;
    if (plan)
        while (B < (static_cast<int64_t>(4) << plan->min_block_logT)) B <<= 1;
    const int64_t blocks = (P + B - 1) / B;
    out->worker_stride = B;
    out->block_floats = B;
    out->block_stride = static_cast<int64_t>(3) * K * B;
    out->omega_offset = static_cast<int64_t>(K) * B;
    out->delta_offset = static_cast<int64_t>(2) * K * B;
    out->arena_floats = blocks * out->block_stride;
    return GBMUF_OK;
}

int gbmuf_probe_copy(float *dst_dev, const float *src_dev, int64_t n_floats, int32_t flags, void *stream)
{
    if (!dst_dev || !src_dev || n_floats < 0 || (n_floats & 3)) return GBMUF_EINVAL;
    if (!aligned16(dst_dev) || !aligned16(src_dev)) return GBMUF_EINVAL;
    return launch_copy_probe(dst_dev, src_dev, n_floats, flags, 256 * 16, static_cast<hipStream_t>(stream));
}

const char *gbmuf_last_error_detail(void) { return gbmuf::g_detail; }

const char *gbmuf_strerror(int code)
{
    switch (code) {
        case GBMUF_OK: return "ok";
        case GBMUF_EINVAL: return "invalid argument";
        case GBMUF_ENOMEM: return "out of host or device memory";
        case GBMUF_EDEVICE: return "no usable GPU or a HIP call failed";
        case GBMUF_EUNSUPPORTED: return "beyond the limits of this library";
        default: return "unknown status";
    }
}

}  // extern "C"
