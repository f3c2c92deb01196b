// Single-path semantics (section 5): a path length for every triple of the
// relational closure.
//
// The closure runs Algorithm 1's simultaneous step.  Every cell that is in
// T_A carries a length L_A(i, j) >= 1: 1 for the edge-derived cells of the
// initialisation, and l_B(i, k) + l_C(k, j) for a cell that a step first adds
// through a rule A -> B C and a middle node k, both operand cells being from
// the previous step.  A cell keeps its length afterwards.  When one step
// offers several (rule, k) choices the smallest sum is kept (the section does
// not choose; the smallest makes the result unique).
//
// One loop on the device:
//  1. Boolean step: Y = X | OR_rules X_B x X_C (fp4 MFMA or ROWS products),
//     flags per nonterminal;
//  2. the new cells D_A = Y_A & ~X_A, counted (cells, 64 x 64 tiles holding
//     one), with L_A = kInf on them;
//  3. for every rule A -> B C whose A gained cells, for each new cell (i, j)
//        L_A(i, j) = min(L_A(i, j), min_k L_B(i, k) + L_C(k, j))
//     over the k where X_B(i, k) and X_C(k, j) are set (cells of the previous
//     step only: a new cell of B written by this loop is never read).  A rule
//     whose B is a fixed sparse edge matrix walks the set bits of B's rows
//     (minplus_rows_kernel); one whose C is, C's columns through a column
//     index built once (minplus_cols_kernel); the others take the row walk,
//     minplus_kernel over the 64 x 64 output tiles that hold new cells of
//     A (split along k when they are few), while the lengths are at most 16
//     minplus_pow_kernel on the matrix cores, or while they are at most 127
//     minplus_cells_kernel by single cells, whichever a cost model from the
//     counts prefers;
//  4. X = Y.
// Lengths are uint32 in cells of a |N| x npad x npad array (0 = absent); sums
// stay below 2^31 - 1 or the call reports CFPQ_ERANGE.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <string>
#include <type_traits>
#include <unordered_map>
#include <vector>

#include "cfpq_internal.h"
#include "rowor_device.h"

namespace cfpq {
namespace {

constexpr uint32_t kInf = 0x7FFFFFFFu;  // absent operand; kInf + kInf does not wrap

// L = 1 where the bit matrices are set, 0 elsewhere (all |N| matrices).
__global__ void lengths_from_bits_kernel(const uint64_t* __restrict__ T, uint32_t* __restrict__ L,
                                         int64_t total_words) {
    for (int64_t w = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; w < total_words;
         w += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const uint64_t bits = T[w];
        uint4* dst = reinterpret_cast<uint4*>(L + w * 64);
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const uint32_t b = static_cast<uint32_t>(bits >> (4 * q));
            dst[q] = make_uint4(b & 1u, (b >> 1) & 1u, (b >> 2) & 1u, (b >> 3) & 1u);
        }
    }
}

// D = Y & ~X over one matrix.
// The step's new cells of every nonterminal (blockIdx.y = A): D_A = Y_A & ~X_A,
// with per nonterminal the number of new cells (dcount) and of 64 x 64 tiles
// holding one (tiles, from the flags tflag[A][tile]), and L_A = kInf on every
// new cell: the min-plus kernels lower it, and a new cell still at kInf after
// them had no finite sum.
__global__ __launch_bounds__(256) void delta_all_kernel(const uint64_t* __restrict__ Y,
                                                        const uint64_t* __restrict__ X, uint64_t* __restrict__ D,
                                                        uint32_t* __restrict__ lengths, int64_t W, int64_t npad,
                                                        unsigned long long* dcount, int32_t* tflag, int32_t* tiles) {
    // one wavefront per 64 consecutive words at a time (npad * W is a
    // multiple of 64): lanes form the words, then each new word's cells get
    // kInf in one coalesced masked store
    const int lane = threadIdx.x & 63;
    const int64_t a = blockIdx.y;
    const int64_t words = npad * W;
    const uint64_t* y = Y + a * words;
    const uint64_t* x = X + a * words;
    uint64_t* d = D + a * words;
    uint32_t* la = lengths + a * npad * npad;
    int32_t* tf = tflag + a * W * W;
    unsigned long long c = 0;
    uint32_t first = 0;  // tiles this thread flagged first
    const int64_t waves = static_cast<int64_t>(gridDim.x) * (blockDim.x >> 6);
    for (int64_t base = (static_cast<int64_t>(blockIdx.x) * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 64;
         base < words; base += waves * 64) {
        const int64_t w = base + lane;
        const uint64_t v = y[w] & ~x[w];
        d[w] = v;
        if (v) {
            c += __popcll(v);
            int32_t* f = tf + (w / W >> 6) * W + w % W;
            if (*f == 0 && atomicOr(f, 1) == 0) ++first;
        }
        for (uint64_t nz = __ballot(v != 0); nz; nz &= nz - 1) {
            const int src = __ffsll(static_cast<unsigned long long>(nz)) - 1;
            const int64_t ws = base + src;
            if ((rowor::readlane64(v, src) >> lane) & 1ull) la[(ws / W) * npad + 64 * (ws % W) + lane] = kInf;
        }
    }
    // one atomic per workgroup and counter (same-address atomics queue)
    for (int off = 32; off > 0; off >>= 1) {
        c += __shfl_down(c, off, 64);
        first += __shfl_down(first, off, 64);
    }
    __shared__ unsigned long long pc[4];
    __shared__ uint32_t pf[4];
    if (lane == 0) {
        pc[threadIdx.x >> 6] = c;
        pf[threadIdx.x >> 6] = first;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned long long tc = pc[0] + pc[1] + pc[2] + pc[3];
        const uint32_t tn = pf[0] + pf[1] + pf[2] + pf[3];
        if (tc) atomicAdd(dcount + a, tc);
        if (tn) atomicAdd(tiles + a, static_cast<int32_t>(tn));
    }
}

// Chunks of 32 k whose skip mask one pass builds (LDS bits).
constexpr int32_t kSegChunks = 1024;

// First chunk >= from (< n) whose bit is set in m, or -1.  Every thread of
// the workgroup gets the same answer (m is in LDS).
__device__ __forceinline__ int32_t next_chunk(const uint32_t* m, int32_t from, int32_t n) {
    for (int32_t c = from; c < n;) {
        const uint32_t w = m[c >> 5] >> (c & 31);
        if (w) {
            const int32_t r = c + __ffs(w) - 1;
            return r < n ? r : -1;
        }
        c = (c | 31) + 1;
    }
    return -1;
}

// One workgroup per 64 x 64 output tile; 16 x 16 threads, 4 x 4 cells each.
// Operand chunks of 32 k are staged in LDS k-major, already masked to kInf
// where the previous step's bit is clear.  A first pass over the tile's row
// block of X_B and column word of X_C marks the chunks where both operand
// blocks hold bits (segments of kSegChunks chunks); only those are staged
// and multiplied.  (Prefetching the next chunk into registers while the
// current one is multiplied needed 154 VGPRs and ran slower: occupancy,
// not the staging latency, hides the loads.)
//
// kNarrow: every operand length is at most 2^14 - 1, so lengths and their
// sums fit 16 bits below kInf16 and two cells go through each VALU
// instruction (v_pk_add_u16, v_pk_min_u16: one instruction per term instead
// of the 32-bit loop's add per term and three-way min per two).  L_B is
// staged with its value in both halves of a dword, L_C as 16-bit pairs along
// j; the sums are the same integers, so the lengths are identical.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
constexpr uint32_t kInf16 = 0x7FFFu;  // absent operand in the narrow kernel; kInf16 + kInf16 does not wrap
constexpr int64_t kNarrowMaxLength = (1 << 14) - 1;

template <bool kNarrow>
__global__ __launch_bounds__(256) void minplus_kernel(const uint64_t* __restrict__ D, const uint64_t* __restrict__ XB,
                                                      const uint64_t* __restrict__ XC, const uint32_t* LB,
                                                      const uint32_t* LC, uint32_t* LA, int64_t W, int64_t npad,
                                                      int32_t kchunks, const int32_t* __restrict__ tflag,
                                                      int32_t ksplit, unsigned long long* cells) {
    const int64_t tile = blockIdx.x / ksplit;
    if (!tflag[tile]) return;  // no new cell in this tile
    const int32_t per = ((kchunks + ksplit - 1) / ksplit + 1) & ~1;  // even: the marks read chunk pairs
    const int32_t c_begin = static_cast<int32_t>(blockIdx.x % ksplit) * per;
    const int32_t c_end = min(kchunks, c_begin + per);
    if (c_begin >= c_end) return;
    const int64_t ti = tile / W, tj = tile % W;  // W tiles per side (64 cells each)
    const int64_t i0 = ti * 64, jw = tj;  // j0 = 64 * jw
    const int t = threadIdx.x;
    __shared__ __align__(16) uint32_t As[32][64 + 4];  // As[kk][i] (narrow: the 16-bit value twice)
    __shared__ __align__(16) uint32_t Bs[32][64 + 4];  // Bs[kk][j] (narrow: 16-bit, first half of each row)
    __shared__ uint32_t bmask[kSegChunks / 32], cmask[kSegChunks / 32];
    int32_t done_chunks = 0;
    const int tx = t & 15, ty = t >> 4;
    uint32_t acc[4][4];  // narrow: acc[r][0..1] hold the four cells as 16-bit pairs
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] = 0xFFFFFFFFu;
    for (int32_t seg0 = c_begin; seg0 < c_end; seg0 += kSegChunks) {
        const int32_t seg_n = min(kSegChunks, c_end - seg0);
        // ---- chunk marks: bit c = chunk seg0 + c has bits in both operand blocks
        __syncthreads();  // the previous segment's marks and buffers are no longer read
        if (t < kSegChunks / 32) {
            bmask[t] = 0;
            cmask[t] = 0;
        }
        __syncthreads();
        const int32_t bwords = (seg_n + 1) / 2;  // 64-bit k-words of X_B rows (two chunks each)
        for (int32_t e = t; e < 64 * bwords; e += 256) {
            const int32_t r = e / bwords, wq = e % bwords;
            const uint64_t x = XB[(i0 + r) * W + seg0 / 2 + wq];  // seg0 is even
            const uint32_t two = (static_cast<uint32_t>(x) != 0 ? 1u : 0u) | ((x >> 32) != 0 ? 2u : 0u);
            if (two) atomicOr(&bmask[(2 * wq) >> 5], two << ((2 * wq) & 31));
        }
        for (int32_t e = t; e < seg_n * 32; e += 256) {
            const int64_t k = static_cast<int64_t>(seg0) * 32 + e;  // < 32 * kchunks <= npad
            if (XC[k * W + jw]) atomicOr(&cmask[(e >> 5) >> 5], 1u << ((e >> 5) & 31));
        }
        __syncthreads();
        if (t < kSegChunks / 32) bmask[t] &= cmask[t];
        __syncthreads();
        // ---- the marked chunks
        for (int32_t c = next_chunk(bmask, 0, seg_n); c >= 0; c = next_chunk(bmask, c + 1, seg_n)) {
            const int64_t k0 = static_cast<int64_t>(seg0 + c) * 32;
            // stage: 64 x 32 of L_B (rows i, cols k) and 32 x 64 of L_C (rows k,
            // cols j); thread t takes rows i0 + t/32 + 8q of column k0 + t%32 of
            // L_B and rows k0 + t/64 + 4q of column 64 jw + t%64 of L_C, q < 8
            // (all below npad: k0 + 31 < 32 * kchunks <= npad)
            const int bi = t >> 5, bk = t & 31, ck = t >> 6, cj = t & 63;
            const int64_t bcol = k0 + bk;
            const uint32_t* lbp = LB + (i0 + bi) * npad + bcol;
            const uint64_t* xbp = XB + (i0 + bi) * W + (bcol >> 6);
            const uint32_t* lcp = LC + (k0 + ck) * npad + 64 * jw + cj;
            const uint64_t* xcp = XC + (k0 + ck) * W + jw;
            const int bsh = static_cast<int>(bcol & 63);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const bool set = (xbp[q * 8 * W] >> bsh) & 1ull;
                const bool cset = (xcp[q * 4 * W] >> cj) & 1ull;
                if (kNarrow) {
                    const uint32_t a = set ? lbp[q * 8 * npad] : kInf16;
                    As[bk][bi + 8 * q] = a | (a << 16);
                    reinterpret_cast<uint16_t*>(&Bs[ck + 4 * q][0])[cj] =
                        static_cast<uint16_t>(cset ? lcp[q * 4 * npad] : kInf16);
                } else {
                    As[bk][bi + 8 * q] = set ? lbp[q * 8 * npad] : kInf;
                    Bs[ck + 4 * q][cj] = cset ? lcp[q * 4 * npad] : kInf;
                }
            }
            __syncthreads();
            if (kNarrow) {
#pragma unroll 8
                for (int kk = 0; kk < 32; ++kk) {
                    const uint4 a = *reinterpret_cast<const uint4*>(&As[kk][ty * 4]);
                    const uint2 b = reinterpret_cast<const uint2*>(&Bs[kk][0])[tx];  // j = 4 tx .. 4 tx + 3
                    const uint32_t av[4] = {a.x, a.y, a.z, a.w};
                    const u16x2 b0 = __builtin_bit_cast(u16x2, b.x), b1 = __builtin_bit_cast(u16x2, b.y);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const u16x2 a2 = __builtin_bit_cast(u16x2, av[r]);
                        const u16x2 m0 = __builtin_elementwise_min(__builtin_bit_cast(u16x2, acc[r][0]), a2 + b0);
                        const u16x2 m1 = __builtin_elementwise_min(__builtin_bit_cast(u16x2, acc[r][1]), a2 + b1);
                        acc[r][0] = __builtin_bit_cast(uint32_t, m0);
                        acc[r][1] = __builtin_bit_cast(uint32_t, m1);
                    }
                }
            } else {
#pragma unroll 8
                for (int kk = 0; kk < 32; ++kk) {
                    const uint4 a = *reinterpret_cast<const uint4*>(&As[kk][ty * 4]);
                    const uint4 b = *reinterpret_cast<const uint4*>(&Bs[kk][tx * 4]);
                    const uint32_t av[4] = {a.x, a.y, a.z, a.w};
                    const uint32_t bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int q = 0; q < 4; ++q) acc[r][q] = min(acc[r][q], av[r] + bv[q]);
                }
            }
            ++done_chunks;
            __syncthreads();  // every thread is done with the chunk before the next is staged
        }
    }
    if (t == 0 && done_chunks) atomicAdd(cells, static_cast<unsigned long long>(done_chunks) * 32 * 64 * 64);
    // new cells only: min with what an earlier rule of this loop stored
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t i = i0 + ty * 4 + r;
        const uint64_t drow = D[i * W + jw];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int jj = tx * 4 + c;
            if (!((drow >> jj) & 1ull)) continue;
            const uint32_t v = kNarrow ? (acc[r][c >> 1] >> (16 * (c & 1))) & 0xFFFFu : acc[r][c];
            // kInf (kInf16 and above when narrow: a sum with an absent operand):
            // this rule (or this k range) offered no k for the cell
            if (v < (kNarrow ? kInf16 : kInf)) atomicMin(LA + i * npad + 64 * jw + jj, v);
        }
    }
}

// ---- min-plus on the matrix cores, while every operand length is at most 16
//
// A length l becomes the power of two 2^(67 - 8 l), an absent cell 0.  A
// product of two is 2^(134 - 8 s), s the sum of the lengths, so over 128 k the
// sum of the products lies in [2^(134 - 8 s), 128 * 2^(134 - 8 s)], s being the
// smallest sum: at most 7 of the 8 exponent steps to the next smaller sum are
// used up, and the exponent alone gives s.  Powers of two, their products
// (exponents -122 .. 118 for s = 32 .. 2) and every rounding of sums of positive
// terms keep those bounds, so the lengths are exact.  Every 128 k are
// combined by a maximum: the larger sum has the smaller s.
//
// In bf16 such a power has no mantissa and, with an odd bias, an even biased
// exponent, so its low byte is 0: the operands are kept as the high bytes
// (length_bytes_kernel), a quarter of the uint32 lengths, and spread by one
// v_perm_b32 per two cells on the way to LDS.
constexpr int32_t kPowMaxLength = 16;
constexpr int kPowStep = 8, kPowBias = 67;
constexpr uint32_t kCellsMaxLength = 127;  // of minplus_cells_kernel, below
constexpr int kCellsWords = 16;
typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));

// The high byte of bf16 2^(kPowBias - kPowStep * l), 0 unless 1 <= l <= 16.
__device__ __forceinline__ uint32_t power_byte(uint32_t l) {
    return l - 1u < static_cast<uint32_t>(kPowMaxLength) ? (kPowBias + 127 - kPowStep * l) >> 1 : 0u;
}

// Operand bytes of one matrix of lengths, cells without the previous step's
// bit X left out: rows[i][k] as it lies, cols[j][k] transposed (either may be
// null).  kPowers: powers of two as above; else the lengths themselves, 255 for
// an absent cell, and only rows and columns in whose tiles a new cell lies
// (tflag).  One workgroup per 64 x 64 tile; thread t holds 16 cells of row t / 4.
template <bool kPowers>
__global__ __launch_bounds__(256) void length_bytes_kernel(const uint32_t* __restrict__ L,
                                                           const uint64_t* __restrict__ X, uint8_t* __restrict__ rows,
                                                           uint8_t* __restrict__ cols, int64_t W, int64_t npad,
                                                           const int32_t* __restrict__ tflag) {
    __shared__ uint32_t tile[64][17];  // 64 bytes a row, padded
    const int t = threadIdx.x;
    const int64_t ti = blockIdx.x / W, tj = blockIdx.x % W;
    if (!kPowers) {  // rows and columns in which no new cell lies stay out
        bool in_row = false, in_col = false;
        for (int64_t x = t; x < W; x += 256) {
            in_row = in_row || tflag[ti * W + x] != 0;
            in_col = in_col || tflag[x * W + tj] != 0;
        }
        if (!__syncthreads_or(rows != nullptr && in_row)) rows = nullptr;
        if (!__syncthreads_or(cols != nullptr && in_col)) cols = nullptr;
        if (rows == nullptr && cols == nullptr) return;
    }
    const int r = t >> 2, c = (t & 3) * 16;
    const int64_t i = ti * 64 + r;
    const uint32_t bits = static_cast<uint32_t>(X[i * W + tj] >> c) & 0xFFFFu;
    const uint4* src = reinterpret_cast<const uint4*>(L + i * npad + tj * 64 + c);
    constexpr uint32_t kAbsent = kPowers ? 0u : 0xFFu;
    uint32_t out[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) out[q] = kAbsent * 0x01010101u;
    if (bits != 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint4 v = src[q];
            const uint32_t l[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t b = kPowers ? power_byte(l[u]) : l[u] & 0xFFu;
                out[q] ^= ((bits >> (4 * q + u)) & 1u ? b ^ kAbsent : 0u) << (8 * u);
            }
        }
    }
    if (rows != nullptr)
        *reinterpret_cast<uint4*>(rows + i * npad + tj * 64 + c) = make_uint4(out[0], out[1], out[2], out[3]);
    if (cols == nullptr) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) tile[r][(t & 3) * 4 + q] = out[q];
    __syncthreads();
    // row j = t / 4 of the transpose, its bytes k = c .. c + 15
    const uint8_t* tb = reinterpret_cast<const uint8_t*>(tile);
    uint32_t o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        o[q] = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) o[q] |= static_cast<uint32_t>(tb[(c + 4 * q + u) * 68 + r]) << (8 * u);
    }
    *reinterpret_cast<uint4*>(cols + (tj * 64 + r) * npad + ti * 64 + c) = make_uint4(o[0], o[1], o[2], o[3]);
}

// L_A = min(L_A, min-plus product) on the new cells, 128 x 128 cells a
// workgroup: four wavefronts of 64 x 64 (2 x 2 blocks of 32 x 32), chunks of
// 64 k staged in two LDS buffers, the next chunk's bytes loaded while one is
// multiplied; two chunks are summed before the maximum.  Workgroups without a new cell return at once.
//
// What bounds it: LDS reads (16 KiB a wavefront and chunk for 16 MFMAs, even
// with the matrix pipe, and as much again in stores for two).  A full product at
// n = 4096 (6.9e10 terms) takes 224 us = 307 T terms/s (258 with the maximum and
// cleared accumulators every 64 k); the VALU kernel took 2750 us for the same
// step (25 T terms/s).  The closure of ER Dyck n = 4096
// went from 9.7 to 4.5 ms with it and the column kernel below.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr int kPowTile = 128, kPowChunk = 64, kPowStride = kPowChunk + 8;  // LDS rows of 144 bytes: no bank conflicts

__global__ __launch_bounds__(256) void minplus_pow_kernel(const uint8_t* __restrict__ B, const uint8_t* __restrict__ CT,
                                                          const uint64_t* __restrict__ D, uint32_t* LA, int64_t W,
                                                          int64_t npad, int32_t chunks,
                                                          const int32_t* __restrict__ tflag,
                                                          unsigned long long* cells) {
    const int64_t side = npad / kPowTile;
    const int64_t ti = blockIdx.x / side, tj = blockIdx.x % side;
    const int32_t* f = tflag + ti * 2 * W + tj * 2;
    if (!(f[0] | f[1] | f[W] | f[W + 1])) return;
    __shared__ __align__(16) uint16_t As[2][kPowTile][kPowStride], Bs[2][kPowTile][kPowStride];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int g = lane >> 5, r32 = lane & 31;
    const int wi = (wave >> 1) * 64, wj = (wave & 1) * 64;
    // staging: thread t takes 32 bytes (half a row) of each operand
    const int sr = t >> 1, sh = (t & 1) * 32;
    const uint8_t* bp = B + (ti * kPowTile + sr) * npad + sh;
    const uint8_t* cp = CT + (tj * kPowTile + sr) * npad + sh;
    uint4 ab[2], cb[2];
    auto load = [&](int c) {
        const uint4* x = reinterpret_cast<const uint4*>(bp + static_cast<int64_t>(c) * kPowChunk);
        const uint4* y = reinterpret_cast<const uint4*>(cp + static_cast<int64_t>(c) * kPowChunk);
        ab[0] = x[0];
        ab[1] = x[1];
        cb[0] = y[0];
        cb[1] = y[1];
    };
    // four bytes b0..b3 -> bf16 pairs (b0 << 8, b1 << 8), (b2 << 8, b3 << 8)
    auto spread = [](uint32_t v, uint32_t* o) {
        o[0] = __builtin_amdgcn_perm(v, v, 0x010C000Cu);
        o[1] = __builtin_amdgcn_perm(v, v, 0x030C020Cu);
    };
    auto store = [&](uint16_t* row, const uint4 (&v)[2]) {
        uint4* dst = reinterpret_cast<uint4*>(row + sh);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            uint32_t o[8];
            spread(v[q].x, o);
            spread(v[q].y, o + 2);
            spread(v[q].z, o + 4);
            spread(v[q].w, o + 6);
            dst[2 * q] = make_uint4(o[0], o[1], o[2], o[3]);
            dst[2 * q + 1] = make_uint4(o[4], o[5], o[6], o[7]);
        }
    };
    f32x16 best[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) best[a][b][e] = 0.0f;
    f32x16 acc[2][2];
    const f32x16 zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    // chunk c of an even (first) or odd index: LDS buffer 0 or 1
    auto multiply = [&](int32_t c, auto first) {
        constexpr int cur = decltype(first)::value ? 0 : 1;
        const bool more = c + 1 < chunks;
        if (more) load(c + 1);
#pragma unroll
        for (int s = 0; s < kPowChunk / 16; ++s) {
            bf16x8 af[2], bf[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                af[a] = *reinterpret_cast<const bf16x8*>(&As[cur][wi + 32 * a + r32][16 * s + 8 * g]);
                bf[a] = *reinterpret_cast<const bf16x8*>(&Bs[cur][wj + 32 * a + r32][16 * s + 8 * g]);
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        af[a], bf[b], s == 0 && cur == 0 ? zero : acc[a][b], 0, 0, 0);
        }
        if (more) {
            store(As[cur ^ 1][sr], ab);  // last read a barrier ago
            store(Bs[cur ^ 1][sr], cb);
        }
        __syncthreads();
    };
    load(0);
    store(As[0][sr], ab);
    store(Bs[0][sr], cb);
    __syncthreads();
    for (int32_t c = 0; c < chunks; c += 2) {
        multiply(c, std::true_type());
        if (c + 1 < chunks) multiply(c + 1, std::false_type());
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int e = 0; e < 16; ++e) best[a][b][e] = fmaxf(best[a][b][e], acc[a][b][e]);
    }
    if (t == 0) atomicAdd(cells, static_cast<unsigned long long>(chunks) * kPowChunk * kPowTile * kPowTile);
    // accumulator e of lane (g, r32): row 8 (e / 4) + 4 g + e % 4, column r32 of its block
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int64_t i = ti * kPowTile + wi + 32 * a + 8 * (e / 4) + 4 * g + (e % 4);
            const int64_t jw = (tj * kPowTile + wj) / 64;
            const uint64_t drow = D[i * W + jw];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const float v = best[a][b][e];
                if (v <= 0.0f || !((drow >> (32 * b + r32)) & 1ull)) continue;
                const int ex = static_cast<int>(__float_as_uint(v) >> 23) - 127;
                const uint32_t s = static_cast<uint32_t>(2 * kPowBias - ex + kPowStep - 1) / kPowStep;
                uint32_t* cell = LA + i * npad + jw * 64 + 32 * b + r32;
                if (s < *cell) *cell = s;
            }
        }
}

// Row by column min-plus of single new cells, operands as bytes holding the
// lengths themselves (length_bytes_kernel<false>).  A wavefront holds 4096 k of row i in registers, each byte in
// 16 bits of its own, and for every new cell (i, j) of its word of D reads the
// same k of column j; absent cells are 255, so with lengths of at most
// kCellsMaxLength a sum with one is at least 256 and none is masked.  A workgroup
// takes kCellsWords words of D, apart by the number of workgroups (new cells
// crowd in few rows), and its four wavefronts share the cells of each word.
//
// For steps of few new cells in many tiles, which the tile kernels take whole.
// What bounds it: the columns from L2 (10 M cells at n = 4096 in 2.9 ms, 14
// TB/s) while cells are many, the latency of a row and a column a word when few.
// ER Dyck n = 4096, the step after a length passed 16 (35000 to 70000 new cells
// in 700 to 1400 of 4096 tiles): 1206 -> 120 us; the closure 3.85 -> 3.43 ms
// (degree 3: 8.4 -> 4.4).  Tried: the common k from the bit rows, 16-bit columns
// behind them (287 us), taken word by word (702); eight wavefronts a workgroup
// (141) and the next column loaded ahead (146).
__global__ __launch_bounds__(256) void minplus_cells_kernel(const uint64_t* __restrict__ D,
                                                            const uint8_t* __restrict__ B,
                                                            const uint8_t* __restrict__ CT, uint32_t* LA, int64_t W,
                                                            int64_t npad, int64_t words) {
    constexpr uint32_t kEven = 0x00FF00FFu, kNone = 0xFFFFFFFFu;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t step = gridDim.x;
    for (int64_t w0 = blockIdx.x; w0 < words; w0 += kCellsWords * step) {
        const int64_t at = w0 + lane * step;
        const uint64_t dw = lane < kCellsWords && at < words ? D[at] : 0;
        for (uint64_t nz = __ballot(dw != 0); nz; nz &= nz - 1) {
            const int src = __ffsll(static_cast<unsigned long long>(nz)) - 1;
            const uint64_t all = rowor::readlane64(dw, src);
            if (__popcll(all) <= ((wave - src) & 3)) continue;  // fewer cells than wavefronts
            const int64_t w = w0 + src * step;
            const int64_t i = w / W, j0 = 64 * (w % W);
            for (int64_t k0 = 16 * lane; k0 - 16 * lane < npad; k0 += 4096) {
                uint32_t even[16], odd[16];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t k = k0 + 1024 * q;
                    uint4 v = make_uint4(kNone, kNone, kNone, kNone);
                    if (k < npad) v = *reinterpret_cast<const uint4*>(B + i * npad + k);
                    const uint32_t x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        even[4 * q + u] = x[u] & kEven;
                        odd[4 * q + u] = (x[u] >> 8) & kEven;
                    }
                }
                int turn = src;
                for (uint64_t cells = all; cells; cells &= cells - 1, ++turn) {
                    if ((turn & 3) != wave) continue;
                    const int64_t j = j0 + __ffsll(static_cast<unsigned long long>(cells)) - 1;
                    uint4 c[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int64_t k = k0 + 1024 * q;
                        c[q] = make_uint4(kNone, kNone, kNone, kNone);
                        if (k < npad) c[q] = *reinterpret_cast<const uint4*>(CT + j * npad + k);
                    }
                    ushort2v best = {0xFFFF, 0xFFFF};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t x[4] = {c[q].x, c[q].y, c[q].z, c[q].w};
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const uint32_t e = even[4 * q + u] + (x[u] & kEven);
                            const uint32_t o = odd[4 * q + u] + ((x[u] >> 8) & kEven);
                            best = __builtin_elementwise_min(best, __builtin_bit_cast(ushort2v, e));
                            best = __builtin_elementwise_min(best, __builtin_bit_cast(ushort2v, o));
                        }
                    }
                    uint32_t s = min<uint32_t>(best.x, best.y);
                    for (int o = 32; o > 0; o >>= 1)
                        s = min(s, static_cast<uint32_t>(__shfl_xor(static_cast<int>(s), o, 64)));
                    if (lane == 0 && s <= 2 * kCellsMaxLength) atomicMin(LA + i * npad + j, s);
                }
            }
        }
    }
}

// Row walk min-plus: L_A(i, j) = min over the set bits k of X_B's row i of
// L_B(i, k) + L_C(k, j), for the new cells (i, j) where X_C(k, j) is set.
// A work item is (row i, group of kGatherWords words of X_B's row): long rows
// spread over many wavefronts.  The k of an item form a wave-uniform stream;
// for each, the lanes take the columns j, 64 at a time, where X_C(k, j) and
// D_A(i, j) are both set.  Items of one row can meet at a cell, so cells are
// lowered with atomicMin (a new cell holds kInf until a finite sum lowers it).
constexpr int kGatherWords = 8;

__global__ __launch_bounds__(256) void minplus_rows_kernel(const uint64_t* __restrict__ D,
                                                           const uint64_t* __restrict__ XB,
                                                           const uint64_t* __restrict__ XC, const uint32_t* LB,
                                                           const uint32_t* LC, uint32_t* LA, int64_t W, int64_t npad,
                                                           int32_t nrows) {
    const int lane = threadIdx.x & 63;
    const int64_t waves = static_cast<int64_t>(gridDim.x) * (blockDim.x >> 6);
    const int64_t groups = (W + kGatherWords - 1) / kGatherWords;
    for (int64_t item = static_cast<int64_t>(blockIdx.x) * (blockDim.x >> 6) + (threadIdx.x >> 6);
         item < nrows * groups; item += waves) {
        const int64_t i = item / groups, kw0 = (item % groups) * kGatherWords;
        const uint64_t bw = lane < kGatherWords && kw0 + lane < W ? XB[i * W + kw0 + lane] : 0;
        uint64_t nz = __ballot(bw != 0);
        if (!nz) continue;
        const uint64_t* drow = D + i * W;
        bool any = false;
        for (int64_t w0 = 0; w0 < W && !any; w0 += 64) any = __ballot(w0 + lane < W && drow[w0 + lane] != 0) != 0;
        if (!any) continue;
        for (; nz; nz &= nz - 1) {
            const int src = __ffsll(static_cast<unsigned long long>(nz)) - 1;
            for (uint64_t kb = rowor::readlane64(bw, src); kb; kb &= kb - 1) {
                const int64_t k = (kw0 + src) * 64 + (__ffsll(static_cast<unsigned long long>(kb)) - 1);
                const uint32_t lb = LB[i * npad + k];
                const uint64_t* crow = XC + k * W;
                for (int64_t jw0 = 0; jw0 < W; jw0 += 64) {
                    const uint64_t m = jw0 + lane < W ? (crow[jw0 + lane] & drow[jw0 + lane]) : 0;
                    for (uint64_t mz = __ballot(m != 0); mz; mz &= mz - 1) {
                        const int s2 = __ffsll(static_cast<unsigned long long>(mz)) - 1;
                        if (!((rowor::readlane64(m, s2) >> lane) & 1ull)) continue;
                        const int64_t j = (jw0 + s2) * 64 + lane;
                        const uint32_t v = lb + LC[k * npad + j];
                        if (v < kInf) atomicMin(LA + i * npad + j, v);
                    }
                }
            }
        }
    }
}

// Column index of a fixed sparse bit matrix (compressed columns): cnt[j] =
// set bits of column j; then ptr = exclusive prefix sums of cnt (ptr[npad] =
// total); then idx[ptr[j] ...] = the rows k of column j's bits, in any order.
__global__ void csc_count_kernel(const uint64_t* __restrict__ M, int64_t W, int64_t words, int32_t* cnt) {
    for (int64_t w = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; w < words;
         w += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        uint64_t x = M[w];
        const int64_t j0 = 64 * (w % W);
        for (; x; x &= x - 1) atomicAdd(cnt + j0 + __ffsll(static_cast<unsigned long long>(x)) - 1, 1);
    }
}

// One workgroup of 1024 threads: ptr[0..n] = exclusive scan of cnt[0..n),
// and cursor = ptr[0..n) for the fill.
__global__ __launch_bounds__(1024) void csc_scan_kernel(const int32_t* __restrict__ cnt, int32_t* ptr,
                                                        int32_t* cursor, int64_t n) {
    __shared__ int32_t part[1024];
    __shared__ int32_t carry;
    const int t = threadIdx.x;
    if (t == 0) carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < n; base += 1024) {
        const int32_t v = base + t < n ? cnt[base + t] : 0;
        part[t] = v;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {  // inclusive Hillis-Steele scan
            const int32_t add = t >= off ? part[t - off] : 0;
            __syncthreads();
            part[t] += add;
            __syncthreads();
        }
        const int32_t excl = carry + part[t] - v;
        if (base + t < n) {
            ptr[base + t] = excl;
            cursor[base + t] = excl;
        }
        __syncthreads();
        if (t == 1023) carry += part[1023];
        __syncthreads();
    }
    if (t == 0) ptr[n] = carry;
}

__global__ void csc_fill_kernel(const uint64_t* __restrict__ M, int64_t W, int64_t words, int32_t* cursor,
                                int32_t* idx) {
    for (int64_t w = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; w < words;
         w += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        uint64_t x = M[w];
        const int64_t k = w / W, j0 = 64 * (w % W);
        for (; x; x &= x - 1) {
            const int32_t pos = atomicAdd(cursor + j0 + __ffsll(static_cast<unsigned long long>(x)) - 1, 1);
            idx[pos] = static_cast<int32_t>(k);
        }
    }
}

// Min-plus of a rule whose right operand C is a fixed sparse matrix, given
// its column index: one wavefront per row i at a time, lanes over the new
// cells (i, j) 64 columns at a time; lane j takes the rows k of column j of C
// where X_B(i, k) is set.
__device__ __forceinline__ void cols_cell(int64_t i, int64_t j, const uint64_t* __restrict__ brow,
                                          const int32_t* __restrict__ cptr, const int32_t* __restrict__ cidx,
                                          const uint32_t* LB, const uint32_t* LC, uint32_t* LA, int64_t npad) {
    uint32_t best = kInf;
    for (int32_t q = cptr[j], e = cptr[j + 1]; q < e; ++q) {
        const int64_t k = cidx[q];
        if (!((brow[k >> 6] >> (k & 63)) & 1ull)) continue;
        best = min(best, LB[i * npad + k] + LC[k * npad + j]);
    }
    uint32_t* dst = LA + i * npad + j;  // kInf until a finite sum lowers it
    if (best < *dst) *dst = best;
}

__global__ __launch_bounds__(256) void minplus_cols_kernel(const uint64_t* __restrict__ D,
                                                           const uint64_t* __restrict__ XB,
                                                           const int32_t* __restrict__ cptr,
                                                           const int32_t* __restrict__ cidx, const uint32_t* LB,
                                                           const uint32_t* LC, uint32_t* LA, int64_t W, int64_t npad,
                                                           int32_t nrows) {
    // a work item is (row i, group of kGatherWords words of D_A's row); lane
    // l takes word l / 8 of the group and its bits b with b % 8 == l % 8, so
    // a lane walks at most 8 new cells and each cell has one owner
    const int lane = threadIdx.x & 63;
    const int64_t waves = static_cast<int64_t>(gridDim.x) * (blockDim.x >> 6);
    const int64_t groups = (W + kGatherWords - 1) / kGatherWords;
    const int64_t w_in = lane >> 3;
    const uint64_t phase = 0x0101010101010101ull << (lane & 7);
    for (int64_t item = static_cast<int64_t>(blockIdx.x) * (blockDim.x >> 6) + (threadIdx.x >> 6);
         item < nrows * groups; item += waves) {
        const int64_t i = item / groups, w = (item % groups) * kGatherWords + w_in;
        uint64_t bits = w < W ? (D[i * W + w] & phase) : 0;
        if (!__ballot(bits != 0)) continue;
        for (; bits; bits &= bits - 1)
            cols_cell(i, w * 64 + __ffsll(static_cast<unsigned long long>(bits)) - 1, XB + i * W, cptr, cidx, LB, LC,
                      LA, npad);
    }
}

// The same, a workgroup a row: L_B's row (kInf where X_B is clear) is read once
// into LDS, and each new cell takes the smallest entry of its column's list,
// plus one -- a fixed matrix holds edges only, of length 1.  One coalesced
// read of the row and LDS reads an edge, where the lanes above chase three
// dependent loads per cell and edge (the densest step of ER Dyck n = 4096, 275
// -> 96 us).  For rows that fit LDS, and steps with at
// least kColsRowCells new cells a row on average (fewer do not repay reading
// the row).
constexpr int32_t kColsRowMax = 16384;
constexpr unsigned long long kColsRowCells = 128;
constexpr size_t kColsRowStatic = 256;  // LDS of the workgroup-wide OR

__global__ __launch_bounds__(256) void minplus_cols_row_kernel(const uint64_t* __restrict__ D,
                                                               const uint64_t* __restrict__ XB,
                                                               const int32_t* __restrict__ cptr,
                                                               const int32_t* __restrict__ cidx, const uint32_t* LB,
                                                               uint32_t* LA, int64_t W, int64_t npad, int32_t n) {
    extern __shared__ uint32_t row[];
    const int64_t i = blockIdx.x;
    const uint64_t* drow = D + i * W;
    const uint64_t* brow = XB + i * W;
    bool any = false;
    for (int64_t w = threadIdx.x; w < W; w += 256) any = any || drow[w] != 0;
    if (!__syncthreads_or(any)) return;
    const uint32_t* lb = LB + i * npad;
    for (int32_t k = threadIdx.x; k < n; k += 256) row[k] = (brow[k >> 6] >> (k & 63)) & 1ull ? lb[k] : kInf;
    __syncthreads();
    uint32_t* la = LA + i * npad;
    // four columns a step, so that their list lookups are in flight together
    for (int32_t j0 = threadIdx.x; j0 < n; j0 += 1024) {
        int32_t e[4], e1[4], k[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t j = j0 + 256 * u;
            const bool have = j < n && ((drow[j >> 6] >> (j & 63)) & 1ull);
            e[u] = have ? cptr[j] : 0;
            e1[u] = have ? cptr[j + 1] : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) k[u] = e[u] < e1[u] ? cidx[e[u]] : 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (e[u] >= e1[u]) continue;
            uint32_t best = row[k[u]];
            for (int32_t q = e[u] + 1; q < e1[u]; ++q) best = min(best, row[cidx[q]]);
            const int32_t j = j0 + 256 * u;
            if (best < kInf - 1 && best + 1 < la[j]) la[j] = best + 1;
        }
    }
}

// Overflow check: a new cell that no rule gave a finite sum (still kInf)
// has a length that did not fit (its Boolean product term exists, so some sum
// was >= 2^31 - 1); it goes back to 0 (absent).
// *longest (unless null) gets the largest length of the others.
__global__ __launch_bounds__(256) void check_new_cells_kernel(const uint64_t* __restrict__ D,
                                                              uint32_t* __restrict__ LA, int64_t W, int64_t npad,
                                                              int32_t* overflow, uint32_t* longest) {
    uint32_t most = 0;
    for (int64_t w = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; w < npad * W;
         w += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        uint64_t d = D[w];
        if (!d) continue;
        const int64_t i = w / W, j0 = 64 * (w % W);
        while (d) {
            const int b = __ffsll(static_cast<unsigned long long>(d)) - 1;
            d &= d - 1;
            uint32_t* cell = LA + i * npad + j0 + b;
            const uint32_t l = *cell;
            if (l >= kInf) {
                *cell = 0;
                atomicOr(overflow, 1);
            } else {
                most = max(most, l);
            }
        }
    }
    if (longest == nullptr) return;
    for (int o = 32; o > 0; o >>= 1) most = max(most, static_cast<uint32_t>(__shfl_xor(static_cast<int>(most), o, 64)));
    if ((threadIdx.x & 63) == 0 && most > __hip_atomic_load(longest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(longest, most);
}

// Tile kernel launch shape: split each active tile along k until about
// kTileTarget workgroups have work (eight rounds at 7 per CU: short pieces
// keep the last round's tail small), at most kMaxSplit ways, and with at most
// kMaxTileGrid workgroups in the grid.
constexpr int64_t kTileTarget = 14336, kMaxSplit = 16, kMaxTileGrid = int64_t{1} << 22;

unsigned grid_for(int64_t items, int64_t cap = 65536) {
    return static_cast<unsigned>(std::max<int64_t>(1, std::min<int64_t>((items + 255) / 256, cap)));
}

// Boolean step products: a rule whose left operand heads no binary rule (a
// fixed edge matrix) runs as ROWS when the graph has at most npad^2 / 16
// edges; the others on the fp4 MFMA (right operands kept transposed, rebuilt
// when they change) up to 2^19 nodes, else on the VALU.
struct SpPlan {
    Layout L;
    int32_t n_nt = 0;
    bool mfma = false, any_rows = false;
    std::vector<char> rows_left;     // per nonterminal
    std::vector<int32_t> right_slot;  // per nonterminal: transpose slot or -1
    std::vector<int32_t> csc_slot;    // per nonterminal: column index slot or -1
    int32_t n_right = 0, n_csc = 0;
    size_t off_edges = 0, off_term_off = 0, off_term_lhs = 0, off_flags = 0, off_bad = 0, off_second = 0,
           off_delta = 0, off_trans = 0, off_rowor = 0, off_csc = 0, csc_bytes = 0, off_csc_cursor = 0,
           off_csc_idx = 0, off_tinfo = 0, tinfo_bytes = 0, off_tiles = 0, off_tflag = 0, off_bytes = 0, total = 0;
    bool any_tiles = false;  // a rule without a fixed operand: its min-plus may run on the matrix cores
};

SpPlan sp_plan(const cfpq_graph* g, const cfpq_grammar* gr) {
    SpPlan p;
    p.L = layout_for(g->n_nodes);
    p.n_nt = gr->n_nonterminals;
    const size_t mat = static_cast<size_t>(p.L.mat_words) * 8;
    size_t off = 0;
    p.off_edges = off;
    if (!g->edges_on_device) off += align_up(static_cast<size_t>(g->n_edges) * sizeof(cfpq_edge), 256);
    p.off_term_off = off;
    off += align_up(static_cast<size_t>(gr->n_terminals + 1) * 4, 256);
    p.off_term_lhs = off;
    off += align_up(static_cast<size_t>(std::max(gr->n_term_rules, 1)) * 4, 256);
    p.off_flags = off;
    off += align_up(static_cast<size_t>(p.n_nt) * 4 + 12, 256);  // change flags, overflow, longest length
    p.off_bad = off;
    off += 256;
    p.off_second = off;  // Y
    off += mat * p.n_nt;
    p.off_delta = off;  // D, one per nonterminal
    off += mat * p.n_nt;
    p.mfma = g->n_nodes <= kMfmaMaxNodes;
    p.rows_left.assign(p.n_nt, 0);
    p.right_slot.assign(p.n_nt, -1);
    if (g->n_edges <= p.L.npad * p.L.npad / 16) {
        std::vector<char> heads(p.n_nt, 0);
        for (int32_t r = 0; r < gr->n_bin_rules; ++r) heads[gr->bin_rules[r].lhs] = 1;
        for (int32_t a = 0; a < p.n_nt; ++a) p.rows_left[a] = heads[a] ? 0 : 1;
    }
    p.csc_slot.assign(p.n_nt, -1);
    for (int32_t r = 0; r < gr->n_bin_rules; ++r) {
        const cfpq_bin_rule& br = gr->bin_rules[r];
        if (p.rows_left[br.left]) {
            p.any_rows = true;
            continue;
        }
        if (p.mfma && p.right_slot[br.right] < 0) p.right_slot[br.right] = p.n_right++;
        if (!p.rows_left[br.right]) p.any_tiles = true;
        // min-plus through the column index of a fixed sparse right operand
        // (its cells come from edges, so at most n_edges of them)
        if (p.rows_left[br.right] && p.csc_slot[br.right] < 0 && g->n_edges < INT32_MAX)
            p.csc_slot[br.right] = p.n_csc++;
    }
    p.off_trans = off;
    off += mat * p.n_right;
    p.off_rowor = off;
    if (p.any_rows) off += align_up(rowor_scratch_bytes(p.L), 256);
    // per column index: ptr (npad + 1), cursor / counts (npad), rows (n_edges)
    p.off_csc_cursor = align_up(static_cast<size_t>(p.L.npad + 1) * 4, 256);
    p.off_csc_idx = p.off_csc_cursor + align_up(static_cast<size_t>(p.L.npad) * 4, 256);
    p.csc_bytes = p.off_csc_idx + align_up(static_cast<size_t>(std::max<int64_t>(g->n_edges, 1)) * 4, 256);
    p.off_csc = off;
    off += p.csc_bytes * p.n_csc;
    // per loop: new-cell counts (uint64), active-tile counts and tile flags
    p.off_tinfo = off;
    p.off_tiles = align_up(static_cast<size_t>(p.n_nt) * 8, 256);
    p.off_tflag = p.off_tiles + align_up(static_cast<size_t>(p.n_nt) * 4, 256);
    p.tinfo_bytes = p.off_tflag + align_up(static_cast<size_t>(p.n_nt) * p.L.W * p.L.W * 4, 256);
    off += p.tinfo_bytes;
    p.off_bytes = off;  // operand bytes of a min-plus product: the left one's rows, the right one's columns
    if (p.any_tiles) off += 2 * static_cast<size_t>(p.L.npad) * static_cast<size_t>(p.L.npad);
    p.total = off;
    return p;
}

}  // namespace
}  // namespace cfpq

using namespace cfpq;

extern "C" {

size_t cfpq_lengths_bytes(int32_t n_nodes, int32_t n_nonterminals) {
    if (n_nonterminals < 0) return 0;
    const Layout L = layout_for(n_nodes < 0 ? 0 : n_nodes);
    return static_cast<size_t>(L.npad) * static_cast<size_t>(L.npad) * 4 * static_cast<size_t>(n_nonterminals);
}

cfpq_status cfpq_single_path_workspace_bytes(const cfpq_graph* graph, const cfpq_grammar* grammar, size_t* bytes) {
    clear_last_error();
    if (!bytes) return fail(CFPQ_EINVAL, "bytes is NULL");
    cfpq_status st = validate_grammar(grammar);
    if (st != CFPQ_OK) return st;
    if (!graph) return fail(CFPQ_EINVAL, "graph is NULL");
    if (graph->n_nodes < 0 || graph->n_nodes > CFPQ_MAX_NODES || graph->n_edges < 0)
        return fail(CFPQ_EINVAL, "graph size out of range");
    *bytes = sp_plan(graph, grammar).total;
    return CFPQ_OK;
}

cfpq_status cfpq_single_path(const cfpq_graph* graph, const cfpq_grammar* grammar, int64_t max_iters, void* stream,
                             void* d_workspace, size_t workspace_bytes, uint64_t* d_result, uint32_t* d_lengths,
                             cfpq_stats* stats) {
    clear_last_error();
    cfpq_status st = validate_grammar(grammar);
    if (st != CFPQ_OK) return st;
    st = validate_graph(graph, grammar);
    if (st != CFPQ_OK) return st;
    if (!d_result || !d_lengths) return fail(CFPQ_EINVAL, "d_result or d_lengths is NULL");
    if ((reinterpret_cast<uintptr_t>(d_result) | reinterpret_cast<uintptr_t>(d_lengths) |
         reinterpret_cast<uintptr_t>(d_workspace)) % 16)
        return fail(CFPQ_EINVAL, "d_result, d_lengths and d_workspace must be 16-byte aligned");
    if (max_iters < 0) return fail(CFPQ_EINVAL, "max_iters is negative");
    const SpPlan p = sp_plan(graph, grammar);
    if (!d_workspace || workspace_bytes < p.total)
        return fail(CFPQ_ENOMEM, "workspace too small: need " + std::to_string(p.total) + " bytes");
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(d_workspace);
    const Layout& L = p.L;
    const size_t mw = static_cast<size_t>(L.mat_words);
    const int32_t n_nt = p.n_nt;

    std::vector<int32_t> term_off(grammar->n_terminals + 1, 0), term_lhs(std::max(grammar->n_term_rules, 1), 0);
    for (int32_t r = 0; r < grammar->n_term_rules; ++r) term_off[grammar->term_rules[r].terminal + 1]++;
    for (int32_t x = 0; x < grammar->n_terminals; ++x) term_off[x + 1] += term_off[x];
    {
        std::vector<int32_t> fill(term_off.begin(), term_off.end() - 1);
        for (int32_t r = 0; r < grammar->n_term_rules; ++r)
            term_lhs[fill[grammar->term_rules[r].terminal]++] = grammar->term_rules[r].lhs;
    }
    auto* d_term_off = reinterpret_cast<int32_t*>(ws + p.off_term_off);
    auto* d_term_lhs = reinterpret_cast<int32_t*>(ws + p.off_term_lhs);
    auto* d_flags = reinterpret_cast<int32_t*>(ws + p.off_flags);
    auto* d_overflow = d_flags + n_nt;
    auto* d_longest = reinterpret_cast<uint32_t*>(d_overflow + 1);
    auto* d_bytes = reinterpret_cast<uint8_t*>(ws + p.off_bytes);
    auto* d_bad = reinterpret_cast<int32_t*>(ws + p.off_bad);
    uint64_t* X = d_result;
    uint64_t* Y = reinterpret_cast<uint64_t*>(ws + p.off_second);
    uint64_t* D = reinterpret_cast<uint64_t*>(ws + p.off_delta);
    const cfpq_edge* d_edges = graph->edges;

    hipEvent_t ev0 = nullptr, ev1 = nullptr, mp0 = nullptr, mp1 = nullptr;
    CFPQ_HIP(hipEventCreate(&ev0));
    CFPQ_HIP(hipEventCreate(&ev1));
    CFPQ_HIP(hipEventCreate(&mp0));
    CFPQ_HIP(hipEventCreate(&mp1));
    struct EvGuard {
        hipEvent_t a, b, c, d;
        ~EvGuard() {
            (void)hipEventDestroy(a);
            (void)hipEventDestroy(b);
            (void)hipEventDestroy(c);
            (void)hipEventDestroy(d);
        }
    } guard{ev0, ev1, mp0, mp1};
    auto* d_cells = reinterpret_cast<unsigned long long*>(d_bad + 2);  // in the same 256-byte block
    double minplus_ms = 0.0;
    CFPQ_HIP(hipMemcpyAsync(d_term_off, term_off.data(), term_off.size() * 4, hipMemcpyHostToDevice, s));
    CFPQ_HIP(hipMemcpyAsync(d_term_lhs, term_lhs.data(), term_lhs.size() * 4, hipMemcpyHostToDevice, s));
    if (!graph->edges_on_device && graph->n_edges > 0) {
        auto* dst = reinterpret_cast<cfpq_edge*>(ws + p.off_edges);
        CFPQ_HIP(hipMemcpyAsync(dst, graph->edges, static_cast<size_t>(graph->n_edges) * sizeof(cfpq_edge),
                                hipMemcpyHostToDevice, s));
        d_edges = dst;
    }
    CFPQ_HIP(hipMemsetAsync(d_bad, 0, 16, s));
    CFPQ_HIP(hipMemsetAsync(d_overflow, 0, 8, s));
    CFPQ_HIP(hipEventRecord(ev0, s));
    CFPQ_HIP(launch_zero(X, mw * n_nt, s));
    CFPQ_HIP(launch_init_scatter(d_edges, graph->n_edges, d_term_off, d_term_lhs, grammar->n_terminals,
                                 graph->n_nodes, X, L, d_bad, s));
    if (graph->edges_on_device) {
        int32_t bad = 0;
        CFPQ_HIP(hipMemcpyAsync(&bad, d_bad, 4, hipMemcpyDeviceToHost, s));
        CFPQ_HIP(hipStreamSynchronize(s));
        if (bad) return fail(CFPQ_EINVAL, std::to_string(bad) + " device edges have an id out of range");
    }
    {
        const int64_t words = static_cast<int64_t>(mw) * n_nt;
        lengths_from_bits_kernel<<<dim3(grid_for(words)), dim3(256), 0, s>>>(X, d_lengths, words);
        CFPQ_HIP(hipGetLastError());
    }
    CFPQ_HIP(hipMemcpyAsync(Y, X, mw * 8 * n_nt, hipMemcpyDeviceToDevice, s));
    // column indexes of the fixed right operands (their cells are final now)
    for (int32_t c = 0; c < n_nt; ++c) {
        if (p.csc_slot[c] < 0) continue;
        char* base = ws + p.off_csc + p.csc_bytes * p.csc_slot[c];
        auto* cptr = reinterpret_cast<int32_t*>(base);
        auto* cursor = reinterpret_cast<int32_t*>(base + p.off_csc_cursor);
        auto* cidx = reinterpret_cast<int32_t*>(base + p.off_csc_idx);
        CFPQ_HIP(launch_zero(reinterpret_cast<uint64_t*>(cursor), static_cast<size_t>(L.npad) / 2, s));
        csc_count_kernel<<<dim3(grid_for(static_cast<int64_t>(mw), 4096)), dim3(256), 0, s>>>(
            X + c * mw, L.W, static_cast<int64_t>(mw), cursor);
        CFPQ_HIP(hipGetLastError());
        csc_scan_kernel<<<dim3(1), dim3(1024), 0, s>>>(cursor, cptr, cursor, L.npad);
        CFPQ_HIP(hipGetLastError());
        csc_fill_kernel<<<dim3(grid_for(static_cast<int64_t>(mw), 4096)), dim3(256), 0, s>>>(
            X + c * mw, L.W, static_cast<int64_t>(mw), cursor, cidx);
        CFPQ_HIP(hipGetLastError());
    }

    auto* d_dcount = reinterpret_cast<unsigned long long*>(ws + p.off_tinfo);
    auto* d_tiles = reinterpret_cast<int32_t*>(ws + p.off_tinfo + p.off_tiles);
    auto* d_tflag = reinterpret_cast<int32_t*>(ws + p.off_tinfo + p.off_tflag);
    // set bits of every X_A, kept up to date on the host from the new-cell counts
    std::vector<unsigned long long> xcount(n_nt, 0), dcount(n_nt, 0);
    std::vector<int32_t> tiles(n_nt, 0);
    CFPQ_HIP(launch_zero(reinterpret_cast<uint64_t*>(d_dcount), static_cast<size_t>(n_nt), s));
    CFPQ_HIP(launch_popcount(X, n_nt, L, d_dcount, s));
    CFPQ_HIP(hipMemcpyAsync(xcount.data(), d_dcount, static_cast<size_t>(n_nt) * 8, hipMemcpyDeviceToHost, s));
    CFPQ_HIP(hipStreamSynchronize(s));
    const int64_t nn = graph->n_nodes;
    const int64_t cap = max_iters > 0 ? max_iters : nn * nn * n_nt + 1;
    const size_t lmat = static_cast<size_t>(L.npad) * static_cast<size_t>(L.npad);
    const int32_t kchunks = static_cast<int32_t>((L.n + 31) / 32);
    std::vector<int32_t> flags(n_nt + 2, 0);
    // a loop's read-backs land in pinned memory (new-cell counts, change flags
    // with the overflow flag, new-cell tiles) and one synchronisation waits
    // for all three
    void* pb = nullptr;
    CFPQ_HIP(pinned_readback(static_cast<size_t>(n_nt) * 16 + 8, &pb));
    auto* h_dcount = static_cast<unsigned long long*>(pb);
    auto* h_flags = reinterpret_cast<int32_t*>(h_dcount + n_nt);
    int32_t* h_tiles = h_flags + n_nt + 2;
    int64_t iters = 0, products = 0, sparse = 0;
    bool converged = grammar->n_bin_rules == 0 || graph->n_nodes == 0;
    int32_t overflow = 0;
    uint64_t* TT = reinterpret_cast<uint64_t*>(ws + p.off_trans);
    int32_t* rowor_ws = reinterpret_cast<int32_t*>(ws + p.off_rowor);
    int64_t rowor_calls = 0;  // numbered row-gather calls (launch_rowor_product)
    if (p.any_rows) CFPQ_HIP(launch_rowor_reset(rowor_ws, s));
    bool pending = false;
    while (!converged && iters < cap) {
        // transposed right operands of X: all in the first loop, then those X changed in
        for (int32_t a = 0; a < n_nt; ++a)
            if (p.right_slot[a] >= 0 && (iters == 0 || flags[a]))
                CFPQ_HIP(launch_transpose(X + a * mw, TT + p.right_slot[a] * mw, L, s));
        CFPQ_HIP(hipMemsetAsync(d_flags, 0, static_cast<size_t>(n_nt) * 4, s));
        for (int32_t r = 0; r < grammar->n_bin_rules; ++r) {
            const auto& br = grammar->bin_rules[r];
            // operands the previous step left as they were have been multiplied
            if (iters > 0 && !flags[br.left] && !flags[br.right]) continue;
            int32_t* flag = d_flags + br.lhs;
            if (p.rows_left[br.left]) {
                CFPQ_HIP(launch_rowor_product(X + br.left * mw, X + br.right * mw, Y + br.lhs * mw, L, flag, rowor_ws,
                                              s, nullptr, 1, rowor_calls++));
                ++sparse;
            } else if (p.mfma) {
                CFPQ_HIP(launch_mfma_path(CFPQ_PATH_FP4, X + br.left * mw, TT + p.right_slot[br.right] * mw,
                                          Y + br.lhs * mw, L, flag, s));
            } else {
                CFPQ_HIP(launch_bits_product(X + br.left * mw, X + br.right * mw, Y + br.lhs * mw, L, flag, s, 0));
            }
            ++products;
        }
        // the step's new cells, their counts and tiles, L = kInf on them
        CFPQ_HIP(launch_zero(reinterpret_cast<uint64_t*>(d_dcount), p.tinfo_bytes / 8, s));
        delta_all_kernel<<<dim3(grid_for(static_cast<int64_t>(mw), 256), static_cast<unsigned>(n_nt)), dim3(256), 0,
                           s>>>(Y, X, D, d_lengths, L.W, L.npad, d_dcount, d_tflag, d_tiles);
        CFPQ_HIP(hipGetLastError());
        CFPQ_HIP(hipMemcpyAsync(h_flags, d_flags, static_cast<size_t>(n_nt + 2) * 4, hipMemcpyDeviceToHost, s));
        CFPQ_HIP(hipMemcpyAsync(h_dcount, d_dcount, static_cast<size_t>(n_nt) * 8, hipMemcpyDeviceToHost, s));
        CFPQ_HIP(hipMemcpyAsync(h_tiles, d_tiles, static_cast<size_t>(n_nt) * 4, hipMemcpyDeviceToHost, s));
        CFPQ_HIP(hipStreamSynchronize(s));
        std::copy(h_flags, h_flags + n_nt + 2, flags.begin());
        std::copy(h_dcount, h_dcount + n_nt, dcount.begin());
        std::copy(h_tiles, h_tiles + n_nt, tiles.begin());
        if (pending) {
            // the previous loop's min-plus time, and its overflow check (the
            // flag after the change flags, read back with them): on overflow
            // this loop's Boolean step is dropped (X is untouched)
            float mp_ms = 0.f;
            CFPQ_HIP(hipEventElapsedTime(&mp_ms, mp0, mp1));
            minplus_ms += mp_ms;
            pending = false;
            if (flags[n_nt]) {
                overflow = 1;
                break;
            }
        }
        ++iters;
        bool any = false;
        for (int32_t a = 0; a < n_nt; ++a) any = any || flags[a] != 0;
        if (!any) {
            converged = true;
            break;
        }
        // Min-plus kernel per rule.  A fixed sparse operand: row or column
        // gathers.  Otherwise the row gather when its estimated time is below
        // the tile kernels': about 10 ns per (row with new cells, set bit of
        // X_B in it) pair, against 20 T (i, j, k) terms/s over the active tiles
        // on the VALU or, while no operand length exceeds 16 (the longest so
        // far was read back with the flags), the matrix cores' time.
        // No rule's tiles take as long as the least that the powers or the cell
        // walk take (0.7 tile_ms >= 0.02, see below: from 769 nodes on): neither
        // is asked for, and the longest length is not tracked for them (50 nodes:
        // 370 us a closure against 390).
        const bool others = p.any_tiles && 0.7 * static_cast<double>(L.W * L.W * kchunks) * 131072.0 / 2e10 >= 0.02;
        const bool powers = others && flags[n_nt + 1] <= kPowMaxLength;
        // 128 x 128 tiles, 2 T terms/s a workgroup and at best 500 over the
        // chip, after a pass over the lengths (4 bytes a cell at 3 TB/s)
        auto pow_ms = [&](int32_t active) {
            const double wgs = std::min<double>(active, static_cast<double>(L.W) * L.W / 4);
            const double cells = static_cast<double>(L.npad) * L.npad;
            return std::max(kchunks * 524288.0 / 2e9, wgs * kchunks * 524288.0 / 5e11) + 0.02 + cells * 4 / 3e9;
        };
        // the cell walk: the operand bytes, the words of D, and 0.55 ns a cell
        // at n = 4096 (0.3 to 0.5 where new cells fill words; n = 8192: 0.76)
        const bool cells_fit = others && static_cast<uint32_t>(flags[n_nt + 1]) <= kCellsMaxLength;
        auto cells_walk_ms = [&](unsigned long long cells) {
            return 0.03 + static_cast<double>(L.npad) * L.npad * 3e-9 +
                   static_cast<double>(cells) * (1.4e-7 + 1e-10 * L.npad);
        };
        // a rule's operand bytes: the left one's rows, the right one's columns
        auto bytes = [&](const cfpq_bin_rule& br, bool powers_of_two) {
            const auto kernel = powers_of_two ? length_bytes_kernel<true> : length_bytes_kernel<false>;
            const dim3 grid(static_cast<unsigned>(L.W * L.W));
            const int32_t* f = d_tflag + br.lhs * L.W * L.W;
            const bool same = br.left == br.right;
            kernel<<<grid, dim3(256), 0, s>>>(d_lengths + br.left * lmat, X + br.left * mw, d_bytes,
                                              same ? d_bytes + lmat : nullptr, L.W, L.npad, f);
            if (!same)
                kernel<<<grid, dim3(256), 0, s>>>(d_lengths + br.right * lmat, X + br.right * mw, nullptr,
                                                  d_bytes + lmat, L.W, L.npad, f);
            return hipGetLastError();
        };
        const int64_t gather_items = static_cast<int64_t>(L.n) * ((L.W + kGatherWords - 1) / kGatherWords);
        const unsigned gather_grid = static_cast<unsigned>(std::min<int64_t>((gather_items + 3) / 4, 2048));
        std::vector<char> on_tiles(grammar->n_bin_rules, 0);
        for (int32_t r = 0; r < grammar->n_bin_rules; ++r) {
            const auto& br = grammar->bin_rules[r];
            if (!flags[br.lhs]) continue;
            bool rows = p.rows_left[br.left] != 0;
            if (!rows && p.csc_slot[br.right] < 0) {
                const double n = static_cast<double>(L.n);
                const double active_rows =
                    std::min({n, static_cast<double>(dcount[br.lhs]), 64.0 * tiles[br.lhs]});
                const double rows_ms = active_rows * static_cast<double>(xcount[br.left]) / n * 1e-5;
                const double tile_ms = static_cast<double>(tiles[br.lhs]) * kchunks * 131072.0 / 2e10;
                // (tile_ms counts every chunk; the VALU kernel passes over those
                // without bits, all but a few on a chain of 3000 nodes: 26 us a
                // step, 58 by this estimate, 71 on the matrix cores)
                const bool pow = powers && pow_ms(tiles[br.lhs]) < 0.7 * tile_ms;
                const double best_ms = pow ? pow_ms(tiles[br.lhs]) : tile_ms;
                // (rows_ms is high by up to 6 where rows are short: 27 us
                // against 164 at n = 4096 and 16 k bits)
                if (cells_fit && cells_walk_ms(dcount[br.lhs]) < std::min(0.3 * rows_ms, best_ms)) {
                    CFPQ_HIP(bytes(br, false));
                    const int64_t wgs = (p.L.mat_words + kCellsWords - 1) / kCellsWords;
                    minplus_cells_kernel<<<dim3(static_cast<unsigned>(std::min<int64_t>(wgs, 65536))), dim3(256), 0,
                                           s>>>(D + br.lhs * mw, d_bytes, d_bytes + lmat, d_lengths + br.lhs * lmat,
                                                L.W, L.npad, p.L.mat_words);
                    CFPQ_HIP(hipGetLastError());
                    continue;
                }
                // and the powers of two have to win against 0.6 of it: 3000 nodes,
                // one edge a node, 36 us for the rows (130 by the estimate) and 104
                // for the powers (89); 1000 nodes, few long rows, 95 and 30
                rows = (pow ? 0.6 * rows_ms : rows_ms) < best_ms;
                on_tiles[r] = rows ? 0 : pow ? 2 : 1;
            }
            if (rows) {
                minplus_rows_kernel<<<dim3(gather_grid), dim3(256), 0, s>>>(
                    D + br.lhs * mw, X + br.left * mw, X + br.right * mw, d_lengths + br.left * lmat,
                    d_lengths + br.right * lmat, d_lengths + br.lhs * lmat, L.W, L.npad, L.n);
            } else if (p.csc_slot[br.right] >= 0) {
                const char* base = ws + p.off_csc + p.csc_bytes * p.csc_slot[br.right];
                if (L.n <= kColsRowMax && dcount[br.lhs] >= kColsRowCells * L.n) {
                    const size_t lds = static_cast<size_t>(L.n) * 4;
                    if (lds + kColsRowStatic > 64 * 1024)  // more LDS than a launch gets unasked
                        CFPQ_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&minplus_cols_row_kernel),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     static_cast<int>(lds)));
                    minplus_cols_row_kernel<<<dim3(static_cast<unsigned>(L.n)), dim3(256), lds, s>>>(
                        D + br.lhs * mw, X + br.left * mw, reinterpret_cast<const int32_t*>(base),
                        reinterpret_cast<const int32_t*>(base + p.off_csc_idx), d_lengths + br.left * lmat,
                        d_lengths + br.lhs * lmat, L.W, L.npad, L.n);
                    CFPQ_HIP(hipGetLastError());
                    continue;
                }
                minplus_cols_kernel<<<dim3(gather_grid), dim3(256), 0, s>>>(
                    D + br.lhs * mw, X + br.left * mw, reinterpret_cast<const int32_t*>(base),
                    reinterpret_cast<const int32_t*>(base + p.off_csc_idx), d_lengths + br.left * lmat,
                    d_lengths + br.right * lmat, d_lengths + br.lhs * lmat, L.W, L.npad, L.n);
            } else {
                continue;
            }
            CFPQ_HIP(hipGetLastError());
        }
        // the others on the tile kernel (timed: its terms are counted); with
        // few active tiles each is split along k into ksplit workgroups so
        // that the launch still fills the chip
        CFPQ_HIP(hipEventRecord(mp0, s));
        for (int32_t r = 0; r < grammar->n_bin_rules; ++r) {
            const auto& br = grammar->bin_rules[r];
            if (!on_tiles[r]) continue;
            const int64_t all_tiles = L.W * L.W;
            if (on_tiles[r] == 2) {
                CFPQ_HIP(bytes(br, true));
                const int64_t side = L.npad / kPowTile;
                minplus_pow_kernel<<<dim3(static_cast<unsigned>(side * side)), dim3(256), 0, s>>>(
                    d_bytes, d_bytes + lmat, D + br.lhs * mw, d_lengths + br.lhs * lmat, L.W, L.npad,
                    static_cast<int32_t>((L.n + kPowChunk - 1) / kPowChunk), d_tflag + br.lhs * all_tiles, d_cells);
                CFPQ_HIP(hipGetLastError());
                continue;
            }
            int64_t ksplit = std::max<int64_t>(1, (kTileTarget + tiles[br.lhs] - 1) / std::max(tiles[br.lhs], 1));
            ksplit = std::min<int64_t>({ksplit, kMaxSplit, std::max<int64_t>(1, kchunks / 2),
                                        std::max<int64_t>(1, kMaxTileGrid / all_tiles)});
            // a length of step t is at most 2^t (each step's sums add two
            // lengths of the previous one), so the first 14 steps run narrow
            const bool narrow = iters < 14 && (int64_t{1} << iters) <= kNarrowMaxLength;
            const dim3 grid(static_cast<unsigned>(all_tiles * ksplit));
            if (narrow)
                minplus_kernel<true><<<grid, dim3(256), 0, s>>>(
                    D + br.lhs * mw, X + br.left * mw, X + br.right * mw, d_lengths + br.left * lmat,
                    d_lengths + br.right * lmat, d_lengths + br.lhs * lmat, L.W, L.npad, kchunks,
                    d_tflag + br.lhs * all_tiles, static_cast<int32_t>(ksplit), d_cells);
            else
                minplus_kernel<false><<<grid, dim3(256), 0, s>>>(
                    D + br.lhs * mw, X + br.left * mw, X + br.right * mw, d_lengths + br.left * lmat,
                    d_lengths + br.right * lmat, d_lengths + br.lhs * lmat, L.W, L.npad, kchunks,
                    d_tflag + br.lhs * all_tiles, static_cast<int32_t>(ksplit), d_cells);
            CFPQ_HIP(hipGetLastError());
        }
        CFPQ_HIP(hipEventRecord(mp1, s));
        for (int32_t a = 0; a < n_nt; ++a) {
            if (!flags[a]) continue;
            check_new_cells_kernel<<<dim3(grid_for(static_cast<int64_t>(mw), 4096)), dim3(256), 0, s>>>(
                D + a * mw, d_lengths + a * lmat, L.W, L.npad, d_overflow, cells_fit ? d_longest : nullptr);
            CFPQ_HIP(hipGetLastError());
            CFPQ_HIP(hipMemcpyAsync(X + a * mw, Y + a * mw, mw * 8, hipMemcpyDeviceToDevice, s));
        }
        for (int32_t a = 0; a < n_nt; ++a) xcount[a] += dcount[a];
        pending = true;  // min-plus time and overflow are read at the next synchronisation
    }
    CFPQ_HIP(hipEventRecord(ev1, s));
    CFPQ_HIP(hipEventSynchronize(ev1));
    if (pending) {
        float mp_ms = 0.f;
        CFPQ_HIP(hipEventElapsedTime(&mp_ms, mp0, mp1));
        minplus_ms += mp_ms;
        CFPQ_HIP(hipMemcpy(&overflow, d_overflow, 4, hipMemcpyDeviceToHost));
    }
    float ms = 0.f;
    CFPQ_HIP(hipEventElapsedTime(&ms, ev0, ev1));
    if (stats) {
        unsigned long long cells = 0;
        CFPQ_HIP(hipMemcpy(&cells, d_cells, 8, hipMemcpyDeviceToHost));
        std::memset(stats, 0, sizeof(*stats));
        stats->iterations = iters;
        stats->products = products;
        stats->sparse_products = sparse;  // ROWS products: not counted as bit-operations
        stats->bitops = 2.0 * static_cast<double>(L.npad) * L.npad * L.npad * static_cast<double>(products - sparse);
        stats->device_ms = ms;
        stats->product_ms = minplus_ms;
        stats->path_used = p.mfma ? CFPQ_PATH_FP4 : CFPQ_PATH_BITS;
        stats->converged = converged ? 1 : 0;
        stats->minplus_terms = static_cast<double>(cells);
    }
    if (overflow) return fail(CFPQ_ERANGE, "a path length reached 2^31 - 1");
    if (!converged) return fail(CFPQ_ENOTCONV, "max_iters reached before the fixpoint");
    return CFPQ_OK;
}

int64_t cfpq_witness(const cfpq_graph* graph, const cfpq_grammar* grammar, const uint32_t* lengths, int32_t a,
                     int32_t i, int32_t j, cfpq_edge* path, int64_t max_edges) {
    clear_last_error();
    cfpq_status st = validate_grammar(grammar);
    if (st != CFPQ_OK) return st;
    st = validate_graph(graph, grammar);
    if (st != CFPQ_OK) return st;
    if (graph->edges_on_device) return fail(CFPQ_EINVAL, "cfpq_witness takes host edges");
    if (!lengths || (!path && max_edges > 0) || max_edges < 0) return fail(CFPQ_EINVAL, "NULL pointer");
    const int32_t n = graph->n_nodes;
    if (a < 0 || a >= grammar->n_nonterminals || i < 0 || i >= n || j < 0 || j >= n)
        return fail(CFPQ_EINVAL, "cell out of range");
    const int64_t npad = layout_for(n).npad;
    auto len = [&](int32_t A, int32_t s, int32_t t) -> uint32_t {
        return lengths[(static_cast<int64_t>(A) * npad + s) * npad + t];
    };
    const uint32_t total = len(a, i, j);
    if (total == 0) return fail(CFPQ_EINVAL, "the cell is not in R_A");
    if (static_cast<int64_t>(total) > max_edges) return fail(CFPQ_ENOMEM, "path buffer shorter than the length");
    // edges by (src, dst), and terminal rules by lhs
    std::unordered_map<int64_t, std::vector<int32_t>> labels;
    for (int64_t e = 0; e < graph->n_edges; ++e)
        labels[static_cast<int64_t>(graph->edges[e].src) * n + graph->edges[e].dst].push_back(graph->edges[e].label);
    std::vector<std::vector<int32_t>> terms_of(grammar->n_nonterminals);
    for (int32_t r = 0; r < grammar->n_term_rules; ++r)
        terms_of[grammar->term_rules[r].lhs].push_back(grammar->term_rules[r].terminal);
    struct Cell {
        int32_t A, s, t;
    };
    std::vector<Cell> stack{{a, i, j}};
    int64_t out = 0, budget = 2 * static_cast<int64_t>(total);
    while (!stack.empty()) {
        if (--budget < 0) return fail(CFPQ_EINVAL, "lengths are inconsistent");
        const Cell c = stack.back();
        stack.pop_back();
        const uint32_t l = len(c.A, c.s, c.t);
        if (l == 0) return fail(CFPQ_EINVAL, "lengths are inconsistent");
        if (l == 1) {
            bool found = false;
            auto it = labels.find(static_cast<int64_t>(c.s) * n + c.t);
            if (it != labels.end())
                for (int32_t x : it->second) {
                    if (std::find(terms_of[c.A].begin(), terms_of[c.A].end(), x) != terms_of[c.A].end()) {
                        if (out >= max_edges) return fail(CFPQ_EINVAL, "lengths are inconsistent (path too long)");
                        path[out++] = cfpq_edge{c.s, x, c.t};
                        found = true;
                        break;
                    }
                }
            if (!found) return fail(CFPQ_EINVAL, "lengths are inconsistent (no edge for a length-1 cell)");
            continue;
        }
        bool split = false;
        for (int32_t r = 0; r < grammar->n_bin_rules && !split; ++r) {
            const auto& br = grammar->bin_rules[r];
            if (br.lhs != c.A) continue;
            for (int32_t k = 0; k < n; ++k) {
                const uint32_t lb = len(br.left, c.s, k), lc = len(br.right, k, c.t);
                if (lb && lc && static_cast<uint64_t>(lb) + lc == l) {
                    stack.push_back({br.right, k, c.t});
                    stack.push_back({br.left, c.s, k});
                    split = true;
                    break;
                }
            }
        }
        if (!split) return fail(CFPQ_EINVAL, "lengths are inconsistent (no split)");
    }
    return out;
}

}  // extern "C"
