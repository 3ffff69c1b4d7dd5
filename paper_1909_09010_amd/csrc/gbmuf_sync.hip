// gbmuf_sync.hip -- the fused gather-average-momentum kernel of libgbmuf (Algorithm 1, sync branch, of
// arXiv 1909.09010) in all its shapes.  Compiled once per GBMUF_PART, each with a part of the shapes
// (they take minutes one after the other).
//
// Fused kernel, in one sentence: a workgroup owns a tile of T 16-byte columns of one
// component for ALL K workers, parks the K x T block of theta in LDS (so every worker's
// average reads its neighbours from LDS, and all reads of theta happen before any write:
// the in-place update keeps snapshot semantics), and streams omega and Delta through
// registers; every state byte is read once and written once.  Where an element lives is a
// Placement: plain rows, or blocks of 2^logB floats whose same-index blocks of all workers lie
// together (a thread looks the block of its column up once).

#include "gbmuf_device.h"
#include "gbmuf_cut.h"

#include "../../include/gbmuf.h"

#pragma clang fp contract(off)

namespace gbmuf {

namespace {

// ---------------------------------------------------------------------------------------
// The block-momentum filter and the restart for one element (Algorithm 1, gossip-BMUF
// statements): G = avg - theta_{t-H};  Delta' = eta*Delta + zeta*G;  omega' = omega +
// Delta';  theta' = omega' + eta*Delta'.  theta_{t-H} is omega + eta*Delta in the paper's
// mode (what the previous restart wrote), omega otherwise.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void filter(float avg, float om, float de, float eta, float zeta, int mode,
                                       float &th_out, float &om_out, float &de_out)
{
    const float t = eta * de;
    const float start = (mode == GBMUF_MODE_PAPER) ? om + t : om;
    const float G = avg - start;
    const float zg = zeta * G;
    const float dn = t + zg;
    const float on = om + dn;
    float tn = on;
    if (mode != GBMUF_MODE_NO_RESTART) {
        const float r = eta * dn;
        tn = on + r;
    }
    th_out = tn; om_out = on; de_out = dn;
}

// Keeps the compiler from moving the computation of a uniform value into a branch, or its load apart.
__device__ __forceinline__ void hold(uint32_t &x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "+s"(x));
#endif
}

// Which tile this workgroup takes.  Workgroups are dealt round-robin to the 8 XCDs (blockIdx mod 8);
// the list is cut into groups of 8 * 2^xcd_log consecutive tiles, and in every group XCD r takes the
// r-th run of 2^xcd_log tiles; with the rotate flag the runs move on by one XCD every 8 groups
// (aligned_shape and shares_lines on the host say when and why).  With the backwards flag (set on odd
// rounds unless the plan asked for forward sweeps) the list is walked backwards, so that what the
// previous sync wrote last is read first, while it may still be in the 256 MB memory-side cache (it
// is for states of up to a few GB; larger states neither gain nor lose); the XCD of a tile stays the
// same up to the rotation.  Tiles beyond the last whole group are taken in order.
//
// This and the load of the descriptor stand before a workgroup's first access of state and are not hidden where one or two
// workgroups fill a CU: nothing here branches, so that all arguments are fetched at once, and the descriptor is one scalar load.
__device__ __forceinline__ unsigned tile_of_block(const SyncArgs &a)
{
    const unsigned n = gridDim.x, lg = static_cast<unsigned>(a.xcd_log), b = blockIdx.x;
    const unsigned back = (a.flags & kFlagBackwards) ? ~0u : 0u;  // a mask: x ^ back is x or -1 - x
    const unsigned whole = (n >> (3 + lg)) << (3 + lg);           // tiles in whole groups
    const unsigned rest = back & (n - whole);                     // backwards the others come first
    const unsigned i = (back & (whole >> 3)) + (((b - rest) >> 3) ^ back);
    const unsigned group = i >> lg;
    const unsigned r = (b + ((a.flags & kFlagRotate) ? group >> 3 : 0u)) & 7u;
    unsigned in_group = (((group << 3) | r) << lg) | (i & ((1u << lg) - 1u)), alone = (back & n) + (b ^ back);
    hold(in_group);
    hold(alone);
    return b - rest < whole ? in_group : alone;                   // backwards b < rest wraps to beyond whole
}

// kApart: the tile's kind besides; other lists have none.
template <int POL>
__device__ __forceinline__ TileDesc load_tile(const TileDesc *p, int &kind)
{
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    const v4u v = *reinterpret_cast<const v4u *>(p);
    uint32_t w[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
    for (int i = 0; i < 4; ++i) hold(w[i]);                       // else it is taken apart into loads of each field
    kind = POL == kApart ? static_cast<int>(w[2] >> (16 + kTileKind)) : kOneStretch;
    return TileDesc{static_cast<int64_t>(w[0] | (static_cast<uint64_t>(w[1]) << 32)), static_cast<uint16_t>(w[2] & 0xFFFFu),
                    static_cast<uint16_t>(POL == kApart ? (w[2] >> 16) & ((1u << kTileKind) - 1u) : w[2] >> 16), static_cast<int32_t>(w[3])};
}

// ---------------------------------------------------------------------------------------
// The neighbour rows of a tile's component in LDS: worker w's row holds the q+1 ids whose values it
// averages, its own among them, ascending.  Kernels are built for these Q1:
//   1..5         every component draws Q1 - 1 neighbours: sums fully unrolled
//   kUpTo8       5 to 7 neighbours
//   kMixed       up to 7 neighbours, a different number per component: a workgroup takes the path of
//                its component's number at the start (a run-time count costs 2 % on 16 workers)
//   kAnyQ        any number
// All but the last keep rows of 4 or 8 uint16, which a thread gets in one read.
// ---------------------------------------------------------------------------------------
// Sorts worker w into its q neighbours (v[0..q)) and stores the row.
template <int Q1>
__device__ __forceinline__ void put_row(uint16_t *dst, int32_t (&v)[Q1], int w, int q)
{
#pragma unroll
    for (int j = 0; j < Q1 - 1; ++j) v[j] = j < q ? v[j] : 0xFFFF;
    v[Q1 - 1] = w;
    sort_few(v);
    uint32_t word[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < Q1; ++j) word[j / 2] |= static_cast<uint32_t>(v[j]) << (16 * (j % 2));
    if (Q1 <= 2) *reinterpret_cast<uint32_t *>(dst) = word[0];
    else if (Q1 <= 4) *reinterpret_cast<uint2 *>(dst) = make_uint2(word[0], word[1]);
    else *reinterpret_cast<uint4 *>(dst) = make_uint4(word[0], word[1], word[2], word[3]);
}

// Worker w's row of the table in memory.  Ids are clamped into [0, K) so that a bad caller table
// cannot index outside the tile.
template <int Q1>
__device__ __forceinline__ void load_row(int32_t (&v)[Q1], const SyncArgs &a, int comp, int w, int q)
{
    const int32_t *row = a.nbr + (static_cast<int64_t>(comp) * a.K + w) * a.q;
#pragma unroll
    for (int j = 0; j < Q1 - 1; ++j)
        if (j < q) v[j] = row[j];
}

template <int Q1>
__device__ __forceinline__ void clamp_row(int32_t (&v)[Q1], int K)
{
#pragma unroll
    for (int j = 0; j < Q1 - 1; ++j) v[j] = min(max(v[j], 0), K - 1);
}

struct LdsRow {
    int32_t *base;
    __device__ int32_t &operator()(int32_t x) const { return base[x]; }
};

// The rows of one tile.  begin() is called before the tile's loads are issued, finish() after.
// a.nbr == nullptr: thread w draws for worker w.
template <int NT, int Q1>
struct Rows {
    int32_t v[Q1];
    __device__ __forceinline__ void begin(const SyncArgs &a, const TileDesc &td)
    {
        const int q = Q1 == kUpTo8 ? td.q : Q1 - 1;
        if (a.nbr != nullptr && static_cast<int>(threadIdx.x) < a.K) load_row<Q1>(v, a, td.comp, threadIdx.x, q);
    }
    __device__ __forceinline__ void put(const SyncArgs &a, const TileDesc &td, uint16_t *ids, int w, int q)
    {
        if (a.nbr != nullptr) {
#if defined(__HIP_DEVICE_COMPILE__)
            // the row is first looked at here: the compiler would move the clamping up to its load and wait for it
            // before the tile's loads are issued
#pragma unroll
            for (int j = 0; j < Q1 - 1; ++j) asm volatile("" : "+v"(v[j]));
#endif
            clamp_row<Q1>(v, a.K);
        } else if constexpr (Q1 > 1) {
            int32_t picked[Q1 - 1];
            draw_few<Q1 - 1>(picked, a.K, a.p, a.C, q, DrawKey{a.key0, a.key1, a.round0, a.round1},
                             static_cast<uint32_t>(td.comp), w);
#pragma unroll
            for (int j = 0; j < Q1 - 1; ++j) v[j] = picked[j];
        }
        put_row<Q1>(ids + w * ids_pitch(Q1, 0), v, w, q);
    }
    __device__ __forceinline__ void finish(const SyncArgs &a, const TileDesc &td, uint16_t *ids)
    {
        const int K = a.K, q = Q1 == kUpTo8 ? td.q : Q1 - 1, first = threadIdx.x;
        if (first < K) put(a, td, ids, first, q);
        for (int w = first + NT; w < K; w += NT) {
            if (a.nbr != nullptr) load_row<Q1>(v, a, td.comp, w, q);
            put(a, td, ids, w, q);
        }
    }
};

// Any number of neighbours.  Rows that the library's sampler wrote are ascending, distinct and without the
// worker: an entry's place follows from itself and its successor, and all threads place entries side by side.  A
// caller's row may hold anything; a thread sorts it by insertion, a chain of LDS accesses for which the
// whole workgroup waits.  9 neighbours, placed / sorted, us: 16 workers x 3.75 M 239 / 320 (7 neighbours, in
// registers: 232), gossip-MA 10 x 6 M 110 / 182 (91); 20 neighbours, 24 x 2.5 M 287 / 412.
template <int NT>
struct Rows<NT, kAnyQ> {
    __device__ __forceinline__ void begin(const SyncArgs &, const TileDesc &) {}
    __device__ __forceinline__ void finish(const SyncArgs &a, const TileDesc &td, uint16_t *ids)
    {
        const int K = a.K, q = td.q, pitch = ids_pitch(kAnyQ, a.q);
        const int32_t *table = a.nbr + static_cast<int64_t>(td.comp) * K * a.q;
        if ((a.flags & kFlagSampledTable) && 4 * K <= NT) { // with more workers every thread has a row to sort
            const int places = max(q, 1);                   // a component without neighbours: the worker itself
            for (int i = threadIdx.x; i < K * places; i += NT) {
                const int w = i / places, j = i - w * places;
                const int32_t *row = table + static_cast<int64_t>(w) * a.q;
                uint16_t *dst = ids + w * pitch;
                const int v = q > 0 ? min(max(row[j], 0), K - 1) : K, next = j + 1 < q ? row[j + 1] : K;
                if (q > 0) dst[v < w ? j : j + 1] = static_cast<uint16_t>(v);
                if (v < w && w < next) dst[j + 1] = static_cast<uint16_t>(w);
                if (j == 0 && w < v) dst[0] = static_cast<uint16_t>(w);
            }
            return;
        }
        int32_t *perm = reinterpret_cast<int32_t *>(ids + ids_words(K, pitch));
        for (int w = threadIdx.x; w < K; w += NT) {
            uint16_t *dst = ids + w * pitch;
            if (a.nbr != nullptr) {
                const int32_t *row = table + static_cast<int64_t>(w) * a.q;
                dst[0] = static_cast<uint16_t>(w);
                for (int j = 0; j < q; ++j) {
                    const int v = min(max(row[j], 0), K - 1);
                    int b = j;
                    while (b >= 0 && dst[b] > v) { dst[b + 1] = dst[b]; --b; }
                    dst[b + 1] = static_cast<uint16_t>(v);
                }
            } else {
                int32_t *mine = perm + w * a.C;
                draw_many(LdsRow{mine}, K, a.p, a.C, q, DrawKey{a.key0, a.key1, a.round0, a.round1},
                          static_cast<uint32_t>(td.comp), w);
                int j = 0, o = 0;                           // mine[0..q) ascending; insert w
                while (j < q && mine[j] < w) dst[o++] = static_cast<uint16_t>(mine[j++]);
                dst[o++] = static_cast<uint16_t>(w);
                while (j < q) dst[o++] = static_cast<uint16_t>(mine[j++]);
            }
        }
    }
};

// ---------------------------------------------------------------------------------------
// The fused kernel.  A column is 4 consecutive floats, loaded and stored as one 16-byte access
// wherever the row starts: global memory takes 16-byte accesses at any 4-byte address, and what a
// misaligned row costs is only the cache lines that two tiles share (shares_lines on the host).
// Slot s of the tile (s = tid + n*NT) is worker s >> logT, column s & (T-1).
//
// Bound by HBM.  Measured on 16 workers x 35.0 M parameters (6.7 GB) in plain [K, P] tensors with an
// odd P: 2300 to 2480 us (5.4 to 5.8 TB/s); with 4-byte accesses, tiles dealt to the XCDs one by one: 3230 us.
// ---------------------------------------------------------------------------------------
// A column of which only the floats in `mk` are this tile's (at least one).  Of a cut column
// the floats outside are read as copies of the nearest one inside, so that its four loads depend on nothing: a
// vector filled float by float made every array's load wait for the one before, three memory latencies in
// a row in each cut tile.  48 components of one cut tile each, 100 workers, 1024 x 4: 9.6 us, that way 12.7;
// edges between columns 7.3.
__device__ __forceinline__ v4f load_col(const float *p, unsigned mk)
{
    if (mk == 0xFu) return load4<kPlain>(p);
    const int first = __builtin_ctz(mk), last = 31 - __builtin_clz(mk);
    v4f v;
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = p[min(max(c, first), last)];
    return v;
}

__device__ __forceinline__ void store_col(float *p, v4f v, unsigned mk)
{
    if (mk == 0xFu) {
        store4<kPlain>(p, v);
        return;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (mk & (1u << c)) p[c] = v[c];
}

// The average of one column: sum over the worker and its neighbours, ascending worker id, then * 1/(q+1).
template <int Q1>
__device__ __forceinline__ v4f average(const v4f *tile, const uint16_t *row, int q1, int logT, int col, float inv)
{
    v4f s;
    if constexpr (Q1 != kAnyQ) {
        uint32_t word[4];
        if (Q1 <= 2) {
            word[0] = *reinterpret_cast<const uint32_t *>(row);
        } else if (Q1 <= 4) {
            const uint2 v = *reinterpret_cast<const uint2 *>(row);
            word[0] = v.x; word[1] = v.y;
        } else {
            const uint4 v = *reinterpret_cast<const uint4 *>(row);
            word[0] = v.x; word[1] = v.y; word[2] = v.z; word[3] = v.w;
        }
#pragma unroll
        for (int j = 0; j < Q1; ++j) {
            if (Q1 == kUpTo8 && j >= q1) break;
            const uint32_t id = (j & 1) ? word[j / 2] >> 16 : word[j / 2] & 0xFFFFu;
            const v4f x = tile[(id << logT) + col];
            s = j == 0 ? x : s + x;
        }
    } else {
        s = tile[(static_cast<int>(row[0]) << logT) + col];
        for (int j = 1; j < q1; ++j) s = s + tile[(static_cast<int>(row[j]) << logT) + col];
    }
    return s * inv;
}

// MIXED (up to 7 neighbours, whose path the workgroup has taken): 1/(q+1) of the tile's component is a constant, because a load of it
// is waited for before the tile's own are issued.  us, loaded / constant: gossip-MA on blocks 24 x 8 M 240 / 232, 48 x 19 M 1127 / 1073, 12 x 0.46 M
// 8.6 / 8.1; BMUF 16 x 29 M 1649 / 1636, 128 x 14 K 14.2 / 13.6 (up to 7 neighbours), but 4 x 50 M 700 / 702.
template <int Q1>
__device__ __forceinline__ constexpr float inverse_of(int q)
{
    return Q1 != kUpTo8 ? 1.0f / Q1 : q == 5 ? 1.0f / 6 : q == 6 ? 1.0f / 7 : 1.0f / 8;
}

// A tile that a component edge cuts, all arrays in flight at once.  Slot n of a thread is worker w0 + wn(n), column col0 + cn(n) with
// the same wn, cn for all threads: with T <= NT a thread keeps its column and visits every (NT/T)-th worker, with T > NT (few
// workers in a wide shape) slot n is one stretch of one worker's row.
template <int NT, int SLOTS, int Q1, bool MIXED>
__device__ __forceinline__ void do_tile(const SyncArgs &a, const TileDesc &td, v4f *tile, uint16_t *ids)
{
    const int tid = threadIdx.x, K = a.K, logT = a.logT, T = 1 << logT, mode = a.mode;
    const float inv = MIXED ? inverse_of<Q1>(td.q) : (a.flags & kFlagMixedQ) ? a.comp[td.comp].inv : a.inv;
    const bool slots_too = mode != GBMUF_MODE_GOSSIP_MA;
    const int col0 = tid & (T - 1), w0 = tid >> logT;
    auto wn = [&](int n) { return (n * NT) >> logT; };
    auto cn = [&](int n) { return (n * NT) & (T - 1); };
    const int64_t e0 = ((td.lo >> 2) + col0) << 2;
    const int64_t at0 = static_cast<int64_t>(w0) * a.at.stride + placed(a.at, e0);
    auto at = [&](int n) { return at0 + static_cast<int64_t>(wn(n)) * a.at.stride + 4 * cn(n); };
    // which of the 4 floats of slot n are this tile's (0: none, or no such worker)
    auto mask = [&](int n) {
        unsigned mk = 0;
        if (w0 + wn(n) < K) {
            const int64_t e = e0 + 4 * cn(n);
#pragma unroll
            for (int c = 0; c < 4; ++c) mk |= (e + c >= td.lo && e + c < td.lo + td.n) ? (1u << c) : 0u;
        }
        return mk;
    };

    Rows<NT, Q1> rows;
    rows.begin(a, td);
    v4f th[SLOTS], om[SLOTS], de[SLOTS];
#pragma unroll
    for (int n = 0; n < SLOTS; ++n) {
        const unsigned mk = mask(n);
        if (mk == 0u) continue;
        th[n] = load_col(a.theta + at(n), mk);
        if (slots_too) {
            om[n] = load_col(a.omega + at(n), mk);
            de[n] = load_col(a.delta + at(n), mk);
        }
    }
    rows.finish(a, td, ids);
#pragma unroll
    for (int n = 0; n < SLOTS; ++n)
        if (mask(n)) tile[tid + n * NT] = th[n];
    __syncthreads();

    const int pitch = ids_pitch(Q1, a.q);
#pragma unroll
    for (int n = 0; n < SLOTS; ++n) {
        const unsigned mk = mask(n);
        if (mk == 0u) continue;
        v4f tn = average<Q1>(tile, ids + (w0 + wn(n)) * pitch, td.q + 1, logT, col0 + cn(n), inv);
        if (slots_too) {
            const v4f avg = tn, o = om[n], d = de[n];
            v4f on, dn;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float t1, o1, d1;
                filter(avg[c], o[c], d[c], a.eta, a.zeta, mode, t1, o1, d1);
                tn[c] = t1; on[c] = o1; dn[c] = d1;
            }
            store_col(a.omega + at(n), on, mk);
            store_col(a.delta + at(n), dn, mk);
        }
        store_col(a.theta + at(n), tn, mk);
    }
}

// A tile whose columns are loaded as they are.  The same slots, but no load stands behind a branch: where one may have been left out
// the compiler cannot count how many are under way, and waits for all of them instead of the oldest, which took
// the streamed omega and Delta their depth.  T is the widest power of two, so that more than SLOTS / 2 slots hold rows for every thread.
// Where all arrays are in flight at once the slots beyond the N that hold rows are left out; where omega and Delta are
// streamed, blocks of DEPTH slots are left out in front, so that the stream ends in the same slots for any K.  A thread
// that has no row in a slot loads the tile's first column of row K - 1, one line for the whole wave, and stores nothing.
// kApart: bits 5 and up of a column's number say where its stretch lies in the row if the tile has several (tile_kernel).
// CUT (T <= NT): component edges cut the tile, which is not thin.  A column that is not the tile's at all is treated like a missing row.
// Of a cut column the four floats nearest to it that are the tile's are loaded and moved, and its own are stored one by one (cut_column).
template <int NT, int SLOTS, int DEPTH, int Q1, bool MIXED, int POL, bool MA, bool CUT>
struct WholeTile {
    static constexpr bool APART = POL == kApart && !CUT;
    const SyncArgs &a;
    const TileDesc &td;
    v4f *tile;
    uint16_t *ids;
    int N, skipped, w0, col0;                                     // slots with rows; DEPTH < SLOTS: the first slot that is used
    int beyond;                                                   // APART: where in a row bits 6 and up of a column's number go
    int64_t col_at, spare;                                        // where the thread's first column lies in row 0; what is loaded without a row
    float inv;
    unsigned mine;                                                // CUT: which floats of the thread's column are the tile's
    int from;                                                     // CUT: where its load starts, counted from it
    v4f om[DEPTH], de[DEPTH];

    __device__ __forceinline__ WholeTile(const SyncArgs &args, const TileDesc &desc, v4f *lds, uint16_t *rows)
        : a(args), td(desc), tile(lds), ids(rows) {}
    __device__ __forceinline__ int worker(int n) const { return w0 + (((n - skipped) * NT) >> a.logT); }
    __device__ __forceinline__ int column(int n) const { return ((n - skipped) * NT) & ((1 << a.logT) - 1); }
    // slots that may be unused, or hold no row for some threads
    static __device__ __forceinline__ constexpr bool may_lack(int n) { return n >= (DEPTH == SLOTS ? SLOTS / 2 : SLOTS - DEPTH); }
    __device__ __forceinline__ bool used(int n) const
    {
        return DEPTH == SLOTS ? n <= SLOTS / 2 || n < N : n >= SLOTS / 2 || n >= skipped;
    }
    __device__ __forceinline__ int64_t at(int n) const
    {
        int64_t p = col_at + static_cast<int64_t>(worker(n)) * a.at.stride;
        if constexpr (APART) p += column(n) >> 6 << (beyond + 2);
        else p += 4 * column(n);
        return (!may_lack(n) || worker(n) < a.K) && (!CUT || mine) ? p : spare;
    }
    // The floats of a column as they were loaded, in their places.
    __device__ __forceinline__ v4f moved(v4f v) const
    {
        if (!CUT) return v;
        const bool one = from & 1, two = from & 2;                // turned by `from`: float c comes from c - from, modulo 4
        const v4f h = {one ? v[3] : v[0], one ? v[0] : v[1], one ? v[1] : v[2], one ? v[2] : v[3]};
        return v4f{two ? h[2] : h[0], two ? h[3] : h[1], two ? h[0] : h[2], two ? h[1] : h[3]};
    }
    __device__ __forceinline__ void store(float *p, v4f v) const
    {
        if (!CUT || mine == 0xFu) {
            store4<POL>(p, v);
            return;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (mine & (1u << c)) p[c - from] = v[c];
    }
    __device__ __forceinline__ void load_slots(int n) { load_slots(n, n % DEPTH); }
    __device__ __forceinline__ void load_slots(int n, int to)
    {
        if (MA) return;
        om[to] = load4<POL>(a.omega + at(n));
        de[to] = load4<POL>(a.delta + at(n));
    }
    // Slot n; `next`: the slot whose omega and Delta take its registers, or 0.  GUARD: some threads may have no row.
    template <bool GUARD>
    __device__ __forceinline__ void slot(int n, int next)
    {
        const v4f o = moved(om[n % DEPTH]), d = moved(de[n % DEPTH]);
        if (next) load_slots(next);
        const int w = GUARD ? min(worker(n), a.K - 1) : worker(n);
        const int64_t p = at(n);
        v4f tn = average<Q1>(tile, ids + w * ids_pitch(Q1, a.q), td.q + 1, a.logT, col0 + column(n), inv), on, dn;
        if (!MA) {
            const v4f avg = tn;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float t1, o1, d1;
                filter(avg[c], o[c], d[c], a.eta, a.zeta, a.mode, t1, o1, d1);
                tn[c] = t1; on[c] = o1; dn[c] = d1;
            }
        }
        if ((!GUARD || worker(n) < a.K) && (!CUT || mine)) {
            if (!MA) {
                store(a.omega + p, on);
                store(a.delta + p, dn);
            }
            store(a.theta + p, tn);
        }
    }
    __device__ __forceinline__ void run(int kind)
    {
        const int tid = threadIdx.x, T = 1 << a.logT;
        N = ((a.K << a.logT) + NT - 1) / NT;
        skipped = DEPTH == SLOTS ? 0 : (SLOTS - N) / DEPTH * DEPTH;
        col0 = tid & (T - 1);
        w0 = tid >> a.logT;
        inv = MIXED ? inverse_of<Q1>(td.q) : (a.flags & kFlagMixedQ) ? a.comp[td.comp].inv : a.inv;
        int in_row = col0;
        if constexpr (APART) {
            const int apart = kind == kOneStretch ? kLogStretch : kLogApart;
            beyond = kind == kOneStretch ? kLogStretch + 1 : kind == kApartWide ? kLogApart + 1 : kLogApart + 6 - a.logT;
            in_row = (col0 & 31) | (((col0 >> 5) & 1) << apart) | (col0 >> 6 << beyond);
        }
        const int64_t first = td.lo & ~static_cast<int64_t>(3), e = first + 4 * in_row;
        const CutColumn cut = CUT ? cut_column(e, td.lo, td.n) : CutColumn{0xFu, 0};
        mine = cut.mine;
        from = cut.from;
        col_at = placed(a.at, e + from);
        spare = placed(a.at, td.lo) + static_cast<int64_t>(a.K - 1) * a.at.stride;
        // Nothing is under way here, but the compiler, to which the paths join where the program ends, cannot know: it waited for one slot's
        // theta before the next one's load (gossip-MA 25 x 16 M 519 us, 577).  Two kinds of wait, or it would move one in front of both paths.
        if constexpr (APART) __builtin_amdgcn_s_waitcnt(MA ? 0x0070 : 0x0F70);          // vmcnt(0) and, MA, lgkmcnt(0)
        Rows<NT, Q1> rows;
        rows.begin(a, td);
        // Gossip-MA, more than 4 neighbours, drawn here: behind a full set of theta's loads drawing takes longest, and it goes first (blocked, us, after / before them, 6 neighbours:
        // 64 x 1.2 M 104.2 / 91.3, 32 x 3.8 M 167.0 / 144.8; but with a slot less 48 x 0.6 M 39.8 / 41.6, 24 x 5 M 150.6 / 158.6, and in 1024 x 4 100 x 0.3 M 44.9 / 46.8).
        constexpr bool MAY_DRAW_FIRST = MA && POL == kStreamed && !CUT && Q1 == kUpTo8 && SLOTS == 4 && DEPTH == SLOTS && NT <= 512;
        const bool drawn = MAY_DRAW_FIRST && a.nbr == nullptr && N == SLOTS;
        if (MAY_DRAW_FIRST && drawn) rows.finish(a, td, ids);
        v4f th[SLOTS];
#pragma unroll
        for (int n = 0; n < SLOTS; ++n)
            if (used(n)) th[n] = load4<POL>(a.theta + at(n));
        // kSixtyFour: omega and Delta on top of theta would be more in flight per CU than HBM takes best, although from 2 neighbours on the scalar registers
        // leave one workgroup per CU.  With / without the wait, us, blocked 40 x 62 M 2 neighbours 8850 / 9142, 4 8834 / 8994, 64 x 39 M none;
        // aligned rows 16 x 44 M 3 neighbours 2741 / 2774.  With 5 to 7 it gains as much on rows and 3 % of 40 x 62 M, but costs 1 to 2 % of 40 x 7.5 M and 0.5 % of 64 x 39 M;
        // with more it costs 1 to 4 % (40 x 7.5 M 1268 / 1215).
        if (DEPTH == 1 && SLOTS == 2 && Q1 >= 1 && Q1 <= 5) __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0)
        if constexpr (DEPTH == SLOTS) {
#pragma unroll
            for (int n = 0; n < SLOTS; ++n)
                if (used(n)) load_slots(n);
        } else {
#pragma unroll
            for (int n = 0; n < DEPTH; ++n) load_slots(skipped + n, n);
        }
        if (!MAY_DRAW_FIRST || !drawn) rows.finish(a, td, ids);
#pragma unroll
        for (int n = 0; n < SLOTS; ++n)
            if (used(n)) tile[tid + (n - skipped) * NT] = moved(th[n]);
        __syncthreads();
#pragma unroll
        for (int n = 0; n < SLOTS; ++n) {
            if (!used(n)) continue;
            if (may_lack(n)) slot<true>(n, 0);
            else slot<false>(n, n + DEPTH < SLOTS ? n + DEPTH : 0);
        }
    }
};

// A cut tile of the streamed shapes whose columns are not loaded whole (is_thin): one column of one worker at a time, only those that
// hold floats of the tile.  One or two as a rule, of which a thread has few: its first one's loads are all issued before the barrier.
template <int NT, int Q1, bool MIXED>
__device__ __forceinline__ void thin_tile(const SyncArgs &a, const TileDesc &td, v4f *tile, uint16_t *ids)
{
    const float inv = MIXED ? inverse_of<Q1>(td.q) : (a.flags & kFlagMixedQ) ? a.comp[td.comp].inv : a.inv;
    const bool slots_too = a.mode != GBMUF_MODE_GOSSIP_MA;
    const int64_t first = td.lo & ~static_cast<int64_t>(3);
    const int columns = static_cast<int>((td.lo + td.n - 1 - first) >> 2) + 1;
    const int lg = columns == 1 ? 0 : columns == 2 ? 1 : a.logT, end = a.K << lg;
    auto column = [&](int i) { return i & ((1 << lg) - 1); };
    auto at = [&](int i) { return placed(a.at, first + 4 * column(i)) + static_cast<int64_t>(i >> lg) * a.at.stride; };
    auto mask = [&](int i) { return i < end ? cut_column(first + 4 * column(i), td.lo, td.n).mine : 0u; };
    Rows<NT, Q1> rows;
    rows.begin(a, td);
    const int i0 = threadIdx.x;
    const unsigned mine = mask(i0);
    v4f t, o, d;
    if (mine) {
        t = load_col(a.theta + at(i0), mine);
        if (slots_too) {
            o = load_col(a.omega + at(i0), mine);
            d = load_col(a.delta + at(i0), mine);
        }
    }
    rows.finish(a, td, ids);                                      // drawn while the loads are under way
    if (mine) tile[((i0 >> lg) << a.logT) + column(i0)] = t;
#pragma unroll 1
    for (int i = i0 + NT; i < end; i += NT)
        if (const unsigned mk = mask(i)) tile[((i >> lg) << a.logT) + column(i)] = load_col(a.theta + at(i), mk);
    __syncthreads();
#pragma unroll 1
    for (int i = i0; i < end; i += NT) {
        const unsigned mk = mask(i);
        if (mk == 0u) continue;
        v4f tn = average<Q1>(tile, ids + (i >> lg) * ids_pitch(Q1, a.q), td.q + 1, a.logT, column(i), inv);
        if (slots_too) {
            const v4f avg = tn;
            v4f on, dn;
            if (i != i0) {
                o = load_col(a.omega + at(i), mk);
                d = load_col(a.delta + at(i), mk);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float t1, o1, d1;
                filter(avg[c], o[c], d[c], a.eta, a.zeta, a.mode, t1, o1, d1);
                tn[c] = t1; on[c] = o1; dn[c] = d1;
            }
            store_col(a.omega + at(i), on, mk);
            store_col(a.delta + at(i), dn, mk);
        }
        store_col(a.theta + at(i), tn, mk);
    }
}

template <int NT, int SLOTS, int DEPTH, int Q1, bool MIXED, int POL>
__device__ __forceinline__ void any_tile(const SyncArgs &a, const TileDesc &td, int kind, v4f *tile, uint16_t *ids)
{
    // Cut tiles take plain accesses: they share lines, and a store that goes through the L2 is counted as under way until memory has
    // it, for which loads issued behind it wait (128 workers x 54 K in 9 components 50 us, with plain ones below 29).
    // Each path ends the program: did they meet, to the compiler one path's loads could still be under way where another
    // begins, and it would wait there for the registers they share, between one array's loads and the next.
    const bool cut = ((td.lo & 3) | (td.n & ~(4 << a.logT))) != 0;      // n is less than T columns
    if (cut) {
        if constexpr (DEPTH == SLOTS) {
            do_tile<NT, SLOTS, Q1, MIXED>(a, td, tile, ids);
        } else if (is_thin(td.lo, td.n, a.at.logB)) {
            thin_tile<NT, Q1, MIXED>(a, td, tile, ids);
        } else if (a.mode == GBMUF_MODE_GOSSIP_MA) {
            WholeTile<NT, SLOTS, DEPTH, Q1, MIXED, kPlain, true, true>(a, td, tile, ids).run(kOneStretch);
            __builtin_amdgcn_endpgm();
        } else {
            WholeTile<NT, SLOTS, DEPTH, Q1, MIXED, kPlain, false, true>(a, td, tile, ids).run(kOneStretch);
        }
        __builtin_amdgcn_endpgm();
    }
    if (a.mode == GBMUF_MODE_GOSSIP_MA) {
        WholeTile<NT, SLOTS, DEPTH, Q1, MIXED, POL, true, false>(a, td, tile, ids).run(kind);
        __builtin_amdgcn_endpgm();
    }
    WholeTile<NT, SLOTS, DEPTH, Q1, MIXED, POL, false, false>(a, td, tile, ids).run(kind);
    __builtin_amdgcn_endpgm();
}

// DEPTH < SLOTS is for many workers.  A tile holds theta of all K workers, so its width is what K
// leaves of the 160 KB LDS; narrow tiles touch each row in pieces of 256 bytes and less, which HBM
// answers at two thirds of the rate of 512-byte pieces.  So the tile takes up to 128 KB, all of theta is
// loaded and parked first, and omega and Delta, whose values no other worker needs, are not held for
// the whole tile but streamed through DEPTH slots of registers.  256 workers x 6.2 M (19 GB, blocked),
// T = 32: 5890 us (6450 GB/s), 6290 with plain accesses; T = 16, all that the registers hold of three arrays, 7576.
template <int NT, int SLOTS, int DEPTH, int Q1, int POL>
__global__ __launch_bounds__(NT) void sync_kernel(SyncArgs a)
{
    extern __shared__ float4 lds4[];
    v4f *tile = reinterpret_cast<v4f *>(lds4);
    uint16_t *ids = reinterpret_cast<uint16_t *>(lds4 + NT * SLOTS);
    uint32_t logB = static_cast<uint32_t>(a.at.logB);
    hold(logB);                                                   // fetched with the other arguments, not after the descriptor
    a.at.logB = static_cast<int32_t>(logB);
    int kind;
    const TileDesc td = load_tile<POL>(a.tiles + tile_of_block(a), kind);
    if ((a.flags & kFlagCheckPeriods) && a.step % static_cast<uint64_t>(a.comp[td.comp].period) != 0)
        return;                                                   // not due: the whole workgroup leaves
    if constexpr (Q1 == kMixed) {
        switch (td.q) {
            case 0: return any_tile<NT, SLOTS, DEPTH, 1, true, POL>(a, td, kind, tile, ids);
            case 1: return any_tile<NT, SLOTS, DEPTH, 2, true, POL>(a, td, kind, tile, ids);
            case 2: return any_tile<NT, SLOTS, DEPTH, 3, true, POL>(a, td, kind, tile, ids);
            case 3: return any_tile<NT, SLOTS, DEPTH, 4, true, POL>(a, td, kind, tile, ids);
            case 4: return any_tile<NT, SLOTS, DEPTH, 5, true, POL>(a, td, kind, tile, ids);
            default: return any_tile<NT, SLOTS, DEPTH, kUpTo8, true, POL>(a, td, kind, tile, ids);
        }
    } else {
        any_tile<NT, SLOTS, DEPTH, Q1, false, POL>(a, td, kind, tile, ids);
    }
}

template <int NT, int SLOTS, int DEPTH>
KernelFn pick_q(int Q1)
{
    switch (Q1) {
        case 1: return sync_kernel<NT, SLOTS, DEPTH, 1, GBMUF_POLICY>;
        case 2: return sync_kernel<NT, SLOTS, DEPTH, 2, GBMUF_POLICY>;
        case 3: return sync_kernel<NT, SLOTS, DEPTH, 3, GBMUF_POLICY>;
        case 4: return sync_kernel<NT, SLOTS, DEPTH, 4, GBMUF_POLICY>;
        case 5: return sync_kernel<NT, SLOTS, DEPTH, 5, GBMUF_POLICY>;
        case kUpTo8: return sync_kernel<NT, SLOTS, DEPTH, kUpTo8, GBMUF_POLICY>;
        case kMixed: return sync_kernel<NT, SLOTS, DEPTH, kMixed, GBMUF_POLICY>;
        default: return sync_kernel<NT, SLOTS, DEPTH, kAnyQ, GBMUF_POLICY>;
    }
}

}  // namespace

#define GBMUF_CASE(NT, SL, D) \
    if (v.threads == NT && v.slots == SL && v.depth == D) return pick_q<NT, SL, D>(kernel_q1(q, mixed));
// shapes that tiles in stretches never take
#if GBMUF_POLICY == 2
#define GBMUF_CASE_SIDE_BY_SIDE(NT, SL, D)
#else
#define GBMUF_CASE_SIDE_BY_SIDE(NT, SL, D) GBMUF_CASE(NT, SL, D)
#endif

#if GBMUF_PART == 0
KernelFn GBMUF_PICK_NAME(0, GBMUF_POLICY)(const Variant &v, int q, bool mixed)
{
    GBMUF_CASE_SIDE_BY_SIDE(256, 16, 16)
    GBMUF_CASE(256, 2, 2)
    GBMUF_CASE(256, 1, 1)
    return nullptr;
}
#elif GBMUF_PART == 1
KernelFn GBMUF_PICK_NAME(1, GBMUF_POLICY)(const Variant &v, int q, bool mixed)
{
    GBMUF_CASE(512, 16, 4)
    GBMUF_CASE(512, 1, 1)
    GBMUF_CASE(512, 2, 2)
    return nullptr;
}
#elif GBMUF_PART == 2
KernelFn GBMUF_PICK_NAME(2, GBMUF_POLICY)(const Variant &v, int q, bool mixed)
{
    GBMUF_CASE_SIDE_BY_SIDE(256, 8, 8)
    GBMUF_CASE(256, 4, 4)
    GBMUF_CASE_SIDE_BY_SIDE(1024, 1, 1)
    GBMUF_CASE(1024, 2, 1)
    return nullptr;
}
#elif GBMUF_PART == 3
KernelFn GBMUF_PICK_NAME(3, GBMUF_POLICY)(const Variant &v, int q, bool mixed)
{
    GBMUF_CASE_SIDE_BY_SIDE(512, 8, 8)
    GBMUF_CASE_SIDE_BY_SIDE(1024, 2, 2)
    GBMUF_CASE(512, 4, 4)
    return nullptr;
}
#elif GBMUF_PART == 4
KernelFn GBMUF_PICK_NAME(4, GBMUF_POLICY)(const Variant &v, int q, bool mixed)
{
    GBMUF_CASE(1024, 4, 4)
    GBMUF_CASE(1024, 4, 2)
    return nullptr;
}
#endif

}  // namespace gbmuf
