// Adjacency lists of the row sweeps and the group sweep, and their walks.
//
// A node's list is idx[list.x .. list.x + list.y), and once more in one 16-byte
// word: its entries as eight 16-bit numbers, kNone past the last; with more than
// eight, kMore in the last place.  One load then gives the list of nearly every
// node, where start, length and entries are a chain of three.
#pragma once

#include "cfpq_internal.h"

namespace cfpq {

constexpr uint32_t kNone = 0xFFFF, kMore = 0xFFFE;  // nodes are below 16384
constexpr int32_t kLongList = 32;                   // entries a lane walks itself

__device__ __forceinline__ uint32_t entry(const uint4& v, int u) {
    const uint32_t w = u < 2 ? v.x : u < 4 ? v.y : u < 6 ? v.z : v.w;
    return u & 1 ? w >> 16 : w & 0xFFFFu;
}
__device__ __forceinline__ bool has_more(const uint4& v) { return v.w >> 16 == kMore; }

// The 16-byte form as its entries come: the nth entry k of a list of `count`.
__device__ __forceinline__ void put_near(uint16_t* near, int32_t nth, int32_t count, int32_t k) {
    if (nth < 7 || (nth == 7 && count == 8)) near[nth] = static_cast<uint16_t>(k);
    if (nth == 7 && count > 8) near[7] = static_cast<uint16_t>(kMore);
}

// The OR of in[k] over node i's list: in[k] lies at word (k % 64, k / 64).
__device__ __forceinline__ uint64_t gather_words(const uint64_t* buf, int stride, int lane, bool have, int64_t i,
                                                 const uint4* __restrict__ near, const int2* __restrict__ list,
                                                 const int32_t* __restrict__ idx) {
    uint64_t acc = 0;
    auto word = [&](int32_t k) { return buf[(k & 63) * stride + (k >> 6)]; };
    const uint4 v = have ? near[i] : make_uint4(~0u, ~0u, ~0u, ~0u);
    const bool more = has_more(v);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const uint32_t k = entry(v, u);
        if (__ballot(k < kMore) == 0) break;  // uniform: no lane has more than u entries
        if (k < kMore) acc |= word(static_cast<int32_t>(k));
    }
    if (__ballot(more) == 0) return acc;
    const int2 l = more ? list[i] : make_int2(0, 0);
    for (int32_t e = 7, m = min(l.y, kLongList); e < m; ++e) acc |= word(idx[l.x + e]);
    for (uint64_t m = __ballot(l.y > kLongList); m != 0; m &= m - 1) {
        const int who = __ffsll(static_cast<unsigned long long>(m)) - 1;
        const int32_t ls = __builtin_amdgcn_readlane(l.x, who), lc = __builtin_amdgcn_readlane(l.y, who);
        uint64_t w = 0;
        for (int32_t e = kLongList + lane; e < lc; e += 64) w |= word(idx[ls + e]);
        for (int o = 32; o > 0; o >>= 1)
            w |= static_cast<uint64_t>(__shfl_xor(static_cast<unsigned long long>(w), o, 64));
        if (lane == who) acc |= w;
    }
    return acc;
}

// Sets, in this lane's LDS row x, the bits of node i's list.
__device__ __forceinline__ void scatter_list(const uint4& v, bool have, int64_t i, const int2* __restrict__ list,
                                             const int32_t* __restrict__ idx, uint32_t* lds, int32_t x, int lane) {
    const bool more = have && has_more(v);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const uint32_t j = have ? entry(v, u) : kNone;
        if (__ballot(j < kMore) == 0) break;
        if (j < kMore) atomicOr(lds + x + (j >> 5), 1u << (j & 31));
    }
    if (__ballot(more) == 0) return;
    const int2 l = more ? list[i] : make_int2(0, 0);
    for (int32_t e = 7, m = min(l.y, kLongList); e < m; ++e) {
        const int32_t j = idx[l.x + e];
        atomicOr(lds + x + (j >> 5), 1u << (j & 31));
    }
    for (uint64_t m = __ballot(l.y > kLongList); m != 0; m &= m - 1) {
        const int who = __ffsll(static_cast<unsigned long long>(m)) - 1;
        const int32_t ls = __builtin_amdgcn_readlane(l.x, who), lc = __builtin_amdgcn_readlane(l.y, who);
        const int32_t xw = __builtin_amdgcn_readlane(x, who);
        for (int32_t e = kLongList + lane; e < lc; e += 64) {
            const int32_t j = idx[ls + e];
            atomicOr(lds + xw + (j >> 5), 1u << (j & 31));
        }
    }
}

// The same for the lists of base + k, every bit k of f; two bits a step.
__device__ __forceinline__ void scatter_word(uint64_t f, int64_t base, const uint4* __restrict__ near,
                                             const int2* __restrict__ list, const int32_t* __restrict__ idx,
                                             uint32_t* lds, int32_t x, int lane) {
    while (__ballot(f != 0) != 0) {
        uint4 v[2];
        bool have[2];
        int64_t k[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            have[u] = f != 0;
            k[u] = base + (have[u] ? __ffsll(static_cast<unsigned long long>(f)) - 1 : 0);
            f &= f - 1;  // 0 stays 0
            v[u] = have[u] ? near[k[u]] : make_uint4(~0u, ~0u, ~0u, ~0u);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) scatter_list(v[u], have[u], k[u], list, idx, lds, x, lane);
    }
}

}  // namespace cfpq
