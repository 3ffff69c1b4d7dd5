// gbmuf_device.h -- device code shared by libgbmuf's kernels: the sampler core and 16-byte access.
#pragma once

#include "gbmuf_internal.h"

// Every multiply and add below is rounded on its own: the reference arithmetic has no
// fused multiply-add.  (The build also passes -ffp-contract=off.)
#pragma clang fp contract(off)

namespace gbmuf {
namespace {

// ---------------------------------------------------------------------------------------
// Device writing of the sampler.  (The host has its own, separately written one.)
// ---------------------------------------------------------------------------------------
// Philox-4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): counter (c0..c3), key (k0, k1).
__device__ inline void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                     uint32_t k0, uint32_t k1, uint32_t out[4])
{
    const uint64_t mul_a = 0xD2511F53ull, mul_b = 0xCD9E8D57ull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t pa = mul_a * c0;
        const uint64_t pb = mul_b * c2;
        const uint32_t x0 = static_cast<uint32_t>(pb >> 32) ^ c1 ^ k0;
        const uint32_t x2 = static_cast<uint32_t>(pa >> 32) ^ c3 ^ k1;
        c1 = static_cast<uint32_t>(pb);
        c3 = static_cast<uint32_t>(pa);
        c0 = x0;
        c2 = x2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// Candidate x of worker w, 0 <= x < C = min(2p, K-1) (Definition 1: (w-1)%K .. (w-p)%K, then (w+1)%K ..
// (w+p)%K, repeats dropped).  With p <= K-1 the first p are distinct, and of the others w+d repeats
// one of them exactly when d >= K-p: what is left is d = 1 .. C-p, in order.
__device__ __forceinline__ int32_t ring_candidate(int32_t w, int32_t x, int32_t p, int32_t K)
{
    int32_t v = x < p ? w - 1 - x : w + 1 + (x - p);
    v = v < 0 ? v + K : v;
    return v >= K ? v - K : v;
}

struct DrawKey {
    uint32_t key0, key1, round0, round1;
};

// The random pick of q neighbours (Algorithm 1, sync branch, first statement) for one
// (component, worker): partial Fisher-Yates shuffle of the worker's C candidates.  Draw j takes
// 32-bit word j%4 of the Philox block whose counter is (round low, round high, component,
// worker + 65536*(j/4)) under the key (seed low, seed high) and swaps position j with
// j + floor(word * (C-j) / 2^32).  Integer arithmetic only.
//
// draw_few: up to kFewDraws neighbours, in registers, unsorted: instead of the shuffled list it keeps
// what the swaps so far moved (position -> id), which is all that a later draw can see of them.  No
// memory is read: 16 workers' rows cost one wave under half a microsecond, which the tile's loads hide.
template <int MOST>
__device__ __forceinline__ void draw_few(int32_t (&picked)[MOST], int32_t K, int32_t p, int32_t C, int32_t q,
                                         const DrawKey &k, uint32_t component, int32_t worker)
{
    int32_t moved_to[MOST], moved_id[MOST];
    uint32_t u[4];
#pragma unroll
    for (int j = 0; j < MOST; ++j) {
        if (j >= q) break;
        if (j % 4 == 0)
            philox4x32_10(k.round0, k.round1, component, static_cast<uint32_t>(worker) + 65536u * (j / 4), k.key0, k.key1, u);
        const int32_t r = j + static_cast<int32_t>(__umulhi(u[j % 4], static_cast<uint32_t>(C - j)));
        int32_t at_j = ring_candidate(worker, j, p, K), at_r = ring_candidate(worker, r, p, K);
#pragma unroll
        for (int i = 0; i < j; ++i) {                  // later swaps override earlier ones
            at_j = moved_to[i] == j ? moved_id[i] : at_j;
            at_r = moved_to[i] == r ? moved_id[i] : at_r;
        }
        picked[j] = at_r;
        moved_to[j] = r;
        moved_id[j] = at_j;
    }
}

// draw_many: any q, on a list of C ids in LDS that `perm(x)` exposes; afterwards positions [0, q)
// hold the pick, ascending.
template <class Perm>
__device__ inline void draw_many(Perm perm, int32_t K, int32_t p, int32_t C, int32_t q, const DrawKey &k,
                                 uint32_t component, int32_t worker)
{
    for (int32_t x = 0; x < C; ++x) perm(x) = ring_candidate(worker, x, p, K);
    uint32_t u[4] = {0u, 0u, 0u, 0u};
    for (int32_t j = 0; j < q; ++j) {
        const int lane = j & 3;
        if (lane == 0)
            philox4x32_10(k.round0, k.round1, component, static_cast<uint32_t>(worker) + 65536u * static_cast<uint32_t>(j >> 2),
                          k.key0, k.key1, u);
        const uint32_t word = lane == 0 ? u[0] : lane == 1 ? u[1] : lane == 2 ? u[2] : u[3];
        const int32_t r = j + static_cast<int32_t>(__umulhi(word, static_cast<uint32_t>(C - j)));
        const int32_t a = perm(j), b = perm(r);
        perm(j) = b;
        perm(r) = a;
    }
    for (int32_t a = 1; a < q; ++a) {           // insertion sort of the q chosen ids
        const int32_t v = perm(a);
        int32_t b = a - 1;
        while (b >= 0 && perm(b) > v) { perm(b + 1) = perm(b); --b; }
        perm(b + 1) = v;
    }
}

// Ascending order of N <= 8 values by the shortest sorting networks (Knuth, TAOCP vol. 3, 5.3.4).
template <int N>
__device__ __forceinline__ void sort_few(int32_t (&v)[N])
{
    constexpr int count = N <= 1 ? 0 : N == 2 ? 1 : N == 3 ? 3 : N == 4 ? 5 : N == 5 ? 9 : 19;
    constexpr int net3[3][2] = {{0, 2}, {0, 1}, {1, 2}};
    constexpr int net4[5][2] = {{0, 1}, {2, 3}, {0, 2}, {1, 3}, {1, 2}};
    constexpr int net5[9][2] = {{0, 3}, {1, 4}, {0, 2}, {1, 3}, {0, 1}, {2, 4}, {1, 2}, {3, 4}, {2, 3}};
    constexpr int net8[19][2] = {{0, 1}, {2, 3}, {4, 5}, {6, 7}, {0, 2}, {1, 3}, {4, 6}, {5, 7}, {1, 2}, {5, 6},
                                 {0, 4}, {1, 5}, {2, 6}, {3, 7}, {2, 4}, {3, 5}, {1, 2}, {3, 4}, {5, 6}};
    static_assert(N <= 5 || N == 8, "no network for this size");
#pragma unroll
    for (int i = 0; i < count; ++i) {
        const int x = N == 2 ? 0 : N == 3 ? net3[i % 3][0] : N == 4 ? net4[i % 5][0] : N == 5 ? net5[i % 9][0] : net8[i][0];
        const int y = N == 2 ? 1 : N == 3 ? net3[i % 3][1] : N == 4 ? net4[i % 5][1] : N == 5 ? net5[i % 9][1] : net8[i][1];
        const int32_t lo = min(v[x], v[y]), hi = max(v[x], v[y]);
        v[x] = lo;
        v[y] = hi;
    }
}

// ---------------------------------------------------------------------------------------
// 16-byte access at any 4-byte address, and where an element of a worker's row lies.
// ---------------------------------------------------------------------------------------
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));

template <int POL>
__device__ __forceinline__ v4f load4(const float *p)
{
    const v4f_any *q = reinterpret_cast<const v4f_any *>(p);
    if constexpr (POL != kPlain) return __builtin_nontemporal_load(q);
    else return *q;
}

template <int POL>
__device__ __forceinline__ void store4(float *p, v4f v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (POL != kPlain) {
        typedef unsigned v4u __attribute__((ext_vector_type(4)));
        typedef unsigned v4u_any __attribute__((ext_vector_type(4), aligned(4)));      // any 4-byte address, as above
        __builtin_amdgcn_global_store_b128((__attribute__((address_space(1))) v4u_any *)p, __builtin_bit_cast(v4u, v), "agent");
        return;
    }
#endif
    *reinterpret_cast<v4f_any *>(p) = v;
}

__device__ __forceinline__ int64_t placed(const Placement &at, int64_t e)
{
    return e + (e >> at.logB) * at.block_extra;
}

}  // namespace
}  // namespace gbmuf
