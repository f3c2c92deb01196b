// The resident sweep (resident.h): one workgroup runs the whole in-place
// fixpoint of a small graph, everything it reads per loop in LDS.
//
// A row of a growing nonterminal belongs to a group of L lanes, 128 bits each.
// Per loop and row: the rows of the changed nodes its lists select are ORed in
// (lf rules), the new bits are stored, and each new bit sets the bits of its
// list in the rows of the rf rules' heads, all in the same group -- so one
// barrier a loop is enough.  A group whose neighbours did not change reads a
// list and a bitmap word.  dd rules (S -> S S) walk the bits of D_B[i] and of
// B[i] at changed rows, or, when the loop has many, the workgroup transposes C
// in LDS and multiplies on the fp4 MFMA.
//
// What bounds it: on long chains the LDS latency of one dependent step (list,
// row, store, scatter), on dense graphs the VALU work around the tiles and the
// LDS bandwidth of the walks.  Measured against the kernel that multiplied
// whole matrices every loop (engine_resident_kernel, still used for the Jacobi
// schedule, for grammars beyond the tables and for lists that do not fit): two
// cycles of 64 and 63 nodes, 4033 loops, 17.9 -> 3.4 ms (0.8 us a loop); Dyck
// on G(450, 1800) 627 -> 233 us; same-generation on 100 nodes 120 -> 48 us.
#include <algorithm>

#include "mfma_tile.h"
#include "resident.h"

namespace cfpq {
namespace {

__device__ __forceinline__ uint4 or4(const uint4& a, const uint4& b) {
    return make_uint4(a.x | b.x, a.y | b.y, a.z | b.z, a.w | b.w);
}
__device__ __forceinline__ uint4 andnot4(const uint4& a, const uint4& b) {
    return make_uint4(a.x & ~b.x, a.y & ~b.y, a.z & ~b.z, a.w & ~b.w);
}
__device__ __forceinline__ bool any4(const uint4& a) { return (a.x | a.y | a.z | a.w) != 0; }

// LDS written by this wavefront's lanes is read back by others of the same
// wavefront: LDS operations of a wavefront complete in order, so only the
// compiler has to keep theirs.
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

constexpr int threads_for(int lanes) { return lanes == 1 ? 128 : lanes == 2 ? 512 : 1024; }

// Bits of the dd masks of a loop from which the product runs on the matrix
// cores: a walked bit costs the LDS of a row of C (64 bytes at four lanes a
// row, about 1.2 cycles), the tiles and the transposes about 20000 cycles
// (four lanes), 5000 (two) or 3000 (one).
template <int L>
constexpr int32_t kTileBits = L == 4 ? 16384 : L == 2 ? 8192 : 4096;

// Bits a row gained, on average, from which a loop's scatters run turned
// (transposed in LDS, columns ORed along the incoming lists, turned back): some
// 5000 cycles a rule (1800 with one lane a row), where a lane scatters four
// bits in about 800 and the longest lane counts.  With 12 bits, a^n b^n on
// G(200, 600) took 210 us and Dyck on G(400, 1200) 289; with 4, 154 and 243;
// with 3 the same.
template <int L>
constexpr int32_t kTurnBits = L == 1 ? 1 : 4;

// Following single facts: while a loop gains only a few bits (two cycles, a
// chain: thousands of loops of one or two), one wavefront applies the rules to
// those instead of to all rows: a bit (i, j) of C gives A -> B C the bits (k, j)
// of the edges k -> i of B, a bit (i, j) of B gives A -> B C the bits (i, k) of
// the edges j -> k of C.  Eight lanes a fact take one entry each of a list's
// 8-byte form, so pulls and scatters are three dependent LDS operations each
// (fact, entry, bit), without a barrier or a loop over entries.  More than
// kFacts bits go back to the rows, whose loops cost the same however many.
//
// Two cycles of 64 and 63 nodes: 1.39 -> 0.83 us a loop (2130 cycles, a quarter
// of them in LDS, the rest some 200 instructions and 30 branches of one
// wavefront).  Keeping a lone fact in scalar registers measured 4% less and was
// not worth its code.
constexpr int32_t kFacts = 32, kRing = 512;
constexpr uint32_t kNoFact = ~0u;
__device__ __forceinline__ uint32_t fact(int h, int i, int j) {
    return static_cast<uint32_t>(h) << 16 | static_cast<uint32_t>(i) << 8 | static_cast<uint32_t>(j);
}

struct FactQueue {
    uint32_t q[kRing];
    int32_t count, capped;
    int64_t loops, products;
};

// A launch with the most dynamic LDS has room for what the kernel declares
// itself: the grammar, resident_solo's state, some 100 bytes of counters, and
// class 0's queue.
static_assert(resident_max_lds(0) + sizeof(ResidentGrammar) + sizeof(SlotState) + 256 + sizeof(FactQueue) <= kLdsBytes &&
              resident_max_lds(1) + sizeof(ResidentGrammar) + sizeof(SlotState) + 256 <= kLdsBytes);

// One wavefront; the facts are in q.q[0, q.count).  Ends with q.count = 0 (the
// fixpoint, or the cap) or with every pending fact's row marked in chg and any.
template <typename Rules>
__device__ __forceinline__ void follow_facts(const Rules& u, FactQueue& q, uint32_t* T, uint32_t* chg, uint32_t* any,
                                             int64_t t, int64_t max_iters) {
    const int lane = threadIdx.x & 63, g = lane >> 3, e = lane & 7;
    const uint64_t below = (1ull << lane) - 1;
    int64_t products = 0;
    // positions in the ring: the pending facts from base on, those a pull can
    // use from `pull_from` on, the next free one
    uint32_t base = 0, at = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(q.count)), pull_from = 0;
    uint32_t heads = 0;  // of the pending facts
    bool lost = false, capped = false;
    uint32_t pulled_heads = 0;  // heads that some lf rule reads
    for (int r = 0; r < u.n_lf; ++r) pulled_heads |= 1u << rs_right(u.lf, r);
    for (uint32_t b = 0; b < at; b += 64) {
        const int h = b + lane < at ? static_cast<int>(q.q[b + lane] >> 16) : 31;
        for (int x = 0; x < u.n_dyn; ++x) heads |= __ballot(h == x) != 0 ? 1u << x : 0;
    }
    auto mark = [&](uint32_t f) {
        const int h = f >> 16, i = (f >> 8) & 255;
        atomicOr(chg + h * u.words + (i >> 5), 1u << (i & 31));
        atomicOr(any, 1u << h);
    };
    // the bits (i, j) of h on the lanes with `on`: the new ones are appended
    auto add = [&](bool on, int h, int i, int j, uint32_t& seen) {
        const uint32_t bit = 1u << (j & 31);
        bool gained = false;
        if (on) gained = !(atomicOr(T + h * u.mat + i * 4 + (j >> 5), bit) & bit);
        const uint64_t m = __ballot(gained);
        if (m == 0) return;
        seen |= 1u << h;
        const uint32_t f = fact(h, i, j);
        const uint32_t more = static_cast<uint32_t>(__popcll(m));
        if (at + more - base <= kRing) {
            if (gained) q.q[(at + static_cast<uint32_t>(__popcll(m & below))) % kRing] = f;
            at += more;
        } else {  // the loop ends the following
            if (gained) mark(f);
            lost = true;
        }
    };
    // put(on, k) for this lane's entry k of list l's node i, then the entries past the eighth
    auto each = [&](bool on, int l, int i, auto put) {
        const int node = l * u.n + i;
        const int k = on ? reinterpret_cast<const uint8_t*>(u.near)[8 * node + e] : 0xFF;
        put(k < 0xFE, k);
        const bool more = k == 0xFE;
        if (__ballot(more) == 0) return;
        uint32_t x = more ? u.end[node] + 7 : 0;
        const uint32_t stop = more ? u.end[node + 1] : 0;
        for (; __ballot(x < stop) != 0; ++x) put(x < stop, x < stop ? static_cast<int>(u.idx[x]) : 0);
    };
    auto take = [&](uint32_t from, uint32_t to) { return from + g < to ? q.q[(from + g) % kRing] : kNoFact; };
    while (true) {
        if (t >= max_iters) {
            capped = true;
            break;
        }
        ++t;
        for (uint32_t m = heads; m != 0; m &= m - 1) products += (u.runs >> (8 * (__ffs(m) - 1))) & 0xFF;
        const uint32_t end0 = at;
        uint32_t seen0 = 0, seen1 = 0;
        for (uint32_t b = pull_from; b < end0; b += 8) {
            const uint32_t f = take(b, end0);
            const int h = f >> 16;
            for (int r = 0; r < u.n_lf; ++r) {
                const bool on = h == rs_right(u.lf, r);
                if (__ballot(on) == 0) continue;
                each(on, static_cast<int>(u.lf_in >> (8 * r)) & 255, (f >> 8) & 255,
                     [&](bool x, int k) { add(x, rs_head(u.lf, r), k, f & 255, seen0); });
            }
        }
        wave_order();
        const uint32_t end1 = at;
        for (uint32_t b = end0; b < end1; b += 8) {
            const uint32_t f = take(b, end1);
            const int h = f >> 16;
            for (int r = 0; r < u.n_rf; ++r) {
                const bool on = h == rs_left(u.rf, r);
                if (__ballot(on) == 0) continue;
                each(on, rs_right(u.rf, r), f & 255,
                     [&](bool x, int k) { add(x, rs_head(u.rf, r), (f >> 8) & 255, k, seen1); });
            }
        }
        wave_order();
        base = end0;
        pull_from = (seen0 & pulled_heads) != 0 ? end0 : end1;
        heads = seen0 | seen1;
        if (heads == 0) break;  // the fixpoint
        if (lost || at - base > kFacts) {
            for (uint32_t x = base + lane; x < at; x += 64) mark(q.q[x % kRing]);
            lost = true;
            break;
        }
    }
    if (lane == 0) {
        q.count = lost ? 1 : 0;
        q.capped = capped ? 1 : 0;
        q.loops = t;
        q.products = products;
    }
}

// kDD: the slots have dd rules.  kTurn: their LDS may hold transposed operands.
// d: the slot's descriptor, grammar: where its rules would be, out: its state.
template <int L, bool kDD, bool kTurn>
__device__ __forceinline__ void resident_closure(const SlotDesc& d, const int32_t* __restrict__ grammar,
                                                 const int32_t* __restrict__ term_tab, SlotState* out) {
    constexpr int kThreads = threads_for(L);
    constexpr int kGroups = kThreads / L;
    constexpr int RW = 4 * L;  // dwords of a row
    constexpr int kPasses = L == 4 ? 2 : 1;  // rows of a group
    constexpr bool kQueue = L == 1 && !kDD && !kTurn;
    constexpr int kKept = 2;  // edges a thread keeps between the two passes over them
    extern __shared__ __align__(16) uint32_t lds[];
    __shared__ ResidentGrammar G;
    __shared__ int32_t wave_tot[16];
    __shared__ uint32_t any_s[3];
    __shared__ int32_t bits_s, bad_s, fed_s[2];  // fed: bits the scatters' operand gained, by loop parity
    const int tid = threadIdx.x;
    const int32_t n = d.n;
    const size_t mdw = static_cast<size_t>(d.npad) * d.W * 2;
    uint32_t* gT = reinterpret_cast<uint32_t*>(d.T);

    cfpq_edge kept[kKept];
#pragma unroll
    for (int u = 0; u < kKept; ++u)
        if (tid + u * kThreads < d.n_edges) kept[u] = d.edges[tid + u * kThreads];
    constexpr int kGramWords = static_cast<int>(sizeof(ResidentGrammar) / 4);
    for (int q = tid; q < kGramWords; q += kThreads)
        reinterpret_cast<int32_t*>(&G)[q] = grammar[q];
    if (tid < 3) any_s[tid] = 0;
    if (tid < 2) fed_s[tid] = 0;
    if (tid == 0) {
        bits_s = 0;
        bad_s = 0;
    }
    __syncthreads();
    const bool turned = kTurn && d.tile != 0;
    const ResidentLds lay = resident_lds(n, G, 0, turned);
    auto uni = [](int32_t x) { return __builtin_amdgcn_readfirstlane(x); };
    auto uni64 = [&](uint64_t x) {
        return static_cast<uint64_t>(static_cast<uint32_t>(uni(static_cast<int32_t>(x)))) |
               static_cast<uint64_t>(static_cast<uint32_t>(uni(static_cast<int32_t>(x >> 32)))) << 32;
    };
    const int n_dyn = uni(G.n_dyn), n_lf = uni(G.n_lf), n_rf = uni(G.n_rf), n_ll = uni(G.n_ll);
    const int n_dd = kDD ? uni(G.n_dd) : 0, d_nt = kDD ? uni(G.d_nt) : -1;
    const uint64_t lf = uni64(G.lf), rf = uni64(G.rf), ll = uni64(G.ll), dd = uni64(G.dd), runs = uni64(G.runs);
    const int src = uni(G.src), n_term = uni(G.n_term);
    // heads whose rows a loop after the first has to look at
    const uint32_t row_heads = static_cast<uint32_t>(uni(G.pull_mask)) | (kDD && d_nt >= 0 ? 1u << d_nt : 0u);
    const int n_lists = G.n_list * n;
    const int mat = lay.mat / 4, words = lay.rows / 32;  // dwords of a matrix, of a bitmap
    uint32_t* T = lds;
    uint32_t* D = lds + lay.off_d / 4;
    uint32_t* TT = lds + lay.off_tt / 4;
    uint32_t* chg = lds + lay.off_chg / 4;  // [3][n_dyn][words]
    uint64_t* near = reinterpret_cast<uint64_t*>(lds) + lay.off_near / 8;
    uint32_t* end = lds + lay.off_end / 4;  // end[q] = start of list q; after the fill its end is end[q + 1]
    uint16_t* idx = reinterpret_cast<uint16_t*>(lds) + lay.off_idx / 2;

    // ---- initialisation
    for (int x = tid; x < lay.off_idx / 16; x += kThreads) reinterpret_cast<uint4*>(lds)[x] = make_uint4(0, 0, 0, 0);
    for (int a = 0; a < d.n_nt; ++a) {
        if (G.dyn[a] >= 0) continue;  // written at the end
        uint4* p = reinterpret_cast<uint4*>(gT + a * mdw);
        for (size_t x = tid; x < mdw / 4; x += kThreads) p[x] = make_uint4(0, 0, 0, 0);
    }
    __threadfence();
    __syncthreads();
    // every terminal rule of an edge's label
    auto each_term = [&](int32_t label, auto use) {
        if (n_term >= 0) {
            for (int q = 0; q < n_term; ++q)
                if ((G.term[q] >> 8) == label) use(G.term[q] & 0xFF);
        } else {
            const int32_t* toff = term_tab + d.term_off;
            for (int32_t q = toff[label]; q < toff[label + 1]; ++q) use(term_tab[d.term_lhs_off + q]);
        }
    };
    auto each_edge = [&](auto use) {
#pragma unroll
        for (int u = 0; u < kKept; ++u)
            if (tid + u * kThreads < d.n_edges) use(kept[u]);
        for (int64_t e = tid + kKept * kThreads; e < d.n_edges; e += kThreads) use(d.edges[e]);
    };
    auto in_range = [&](const cfpq_edge& ed) {
        return ed.src >= 0 && ed.src < n && ed.dst >= 0 && ed.dst < n && ed.label >= 0 && ed.label < d.n_terminals;
    };
    each_edge([&](const cfpq_edge& ed) {
        if (!in_range(ed)) {
            atomicAdd(&bad_s, 1);
            return;
        }
        each_term(ed.label, [&](int a) {
            const uint32_t bit = 1u << (ed.dst & 31);
            if (G.dyn[a] >= 0) {
                atomicOr(T + G.dyn[a] * mat + ed.src * RW + (ed.dst >> 5), bit);
            } else {
                atomicOr(gT + a * mdw + static_cast<size_t>(ed.src) * d.W * 2 + (ed.dst >> 5), bit);
                if (G.list[a] >= 0) atomicAdd(end + G.list[a] * n + ed.src + 1, 1u);
                if (G.in[a] >= 0) atomicAdd(end + G.in[a] * n + ed.dst + 1, 1u);
            }
        });
    });
    __syncthreads();
    {
        // end[q + 1] holds the length of list q: make it the list's start
        const int per = (n_lists + kThreads - 1) / kThreads;
        const int q0 = tid * per, q1 = min(n_lists, q0 + per);
        uint32_t sum = 0;
        for (int q = q0; q < q1; ++q) sum += end[q + 1];
        const int lane = tid & 63, wave = tid >> 6;
        uint32_t x = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wave_tot[wave] = static_cast<int32_t>(x);
        __syncthreads();
        uint32_t at = x - sum;
        for (int w = 0; w < wave; ++w) at += static_cast<uint32_t>(wave_tot[w]);
        for (int q = q0; q < q1; ++q) {
            const uint32_t c = end[q + 1];
            end[q + 1] = at;
            at += c;
        }
    }
    __syncthreads();
    each_edge([&](const cfpq_edge& ed) {
        if (!in_range(ed)) return;
        each_term(ed.label, [&](int a) {
            const int l = G.list[a], li = G.in[a];
            if (l >= 0) idx[atomicAdd(end + l * n + ed.src + 1, 1u)] = static_cast<uint16_t>(ed.dst);
            if (li >= 0) idx[atomicAdd(end + li * n + ed.dst + 1, 1u)] = static_cast<uint16_t>(ed.src);
        });
    });
    const int group = tid / L, sub = tid % L;
    // initial bits: gained "in loop 0"
    for (int i = group; i < n; i += kGroups) {
        for (int h = 0; h < n_dyn; ++h) {
            const uint4 t = reinterpret_cast<const uint4*>(T + h * mat + i * RW)[sub];
            if (kDD && h == d_nt) reinterpret_cast<uint4*>(D + i * RW)[sub] = t;
            if (any4(t)) {
                atomicOr(chg + h * words + (i >> 5), 1u << (i & 31));
                atomicOr(&any_s[0], 1u << h);
            }
        }
    }
    __syncthreads();
    if (kQueue && G.queued)  // read after the first loop's barriers
        for (int q = tid; q < n_lists; q += kThreads) {
            const int c = static_cast<int>(end[q + 1] - end[q]);
            uint64_t v = ~0ull;
            for (int e = 0; e < min(c, 8); ++e)
                v = (v & ~(0xFFull << (8 * e))) | static_cast<uint64_t>(idx[end[q] + e]) << (8 * e);
            if (c > 8) v = (v & ~(0xFFull << 56)) | 0xFEull << 56;
            near[q] = v;
        }
    // the lists of the first two lf rules at this group's rows: start, length, first entry
    uint32_t l0[kPasses][2], ln[kPasses][2];
    int lk[kPasses][2];
#pragma unroll
    for (int ps = 0; ps < kPasses; ++ps)
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int i = group + ps * kGroups;
            const bool have = i < n && r < n_lf;
            const int q = have ? rs_left(lf, r) * n + i : 0;
            l0[ps][r] = end[q];
            ln[ps][r] = have ? end[q + 1] - end[q] : 0;
            lk[ps][r] = ln[ps][r] != 0 ? idx[end[q]] : 0;
        }

    // The bits of f, this lane's part of row i of growing nonterminal h, set
    // the bits of their lists in the rows of the heads of h's rf rules.  Four
    // bits a step, so that their lookups are in flight together.
    auto scatter = [&](int i, int h, const uint4& f, uint32_t* cc, uint32_t& any) {
        for (int r = 0; r < n_rf; ++r) {
            if (rs_left(rf, r) != h) continue;
            const int x = rs_head(rf, r);
            uint32_t* xrow = T + x * mat + i * RW;
            const uint32_t* ends = end + rs_right(rf, r) * n + sub * 128;
            bool gained = false;
            auto put = [&](int j) {
                const uint32_t bit = 1u << (j & 31);
                if (!(atomicOr(xrow + (j >> 5), bit) & bit)) {
                    gained = true;
                    if (kDD && x == d_nt) atomicOr(D + i * RW + (j >> 5), bit);
                }
            };
            uint64_t m[2] = {f.x | static_cast<uint64_t>(f.y) << 32, f.z | static_cast<uint64_t>(f.w) << 32};
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                while (m[w] != 0) {
                    uint32_t e[4], e1[4];
                    int j[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const bool have = m[w] != 0;
                        const int k = have ? 64 * w + __ffsll(static_cast<unsigned long long>(m[w])) - 1 : 0;
                        m[w] &= m[w] - 1;  // 0 stays 0
                        e[u] = ends[k];
                        e1[u] = have ? ends[k + 1] : e[u];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) j[u] = e[u] < e1[u] ? idx[e[u]] : 0;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (e[u] >= e1[u]) continue;
                        put(j[u]);
                        for (uint32_t q = e[u] + 1; q < e1[u]; ++q) put(idx[q]);
                    }
                }
            }
            if (gained) {
                atomicOr(cc + x * words + (i >> 5), 1u << (i & 31));
                any |= 1u << x;
            }
        }
    };

    // ---- the fixpoint: loop t reads the marks of loop t - 1
    int64_t products = 0, t = 0;
    int dense = 0;  // products by tiles
    int capped = 0;
    int prev = 0, cur = 1, next = 2;  // t % 3 of the last, this and the next loop
    bool refeed = false;  // this loop scatters all bits of T, as the first one does
    while (true) {
        if (t >= d.max_iters) {
            capped = 1;
            break;
        }
        ++t;
        const bool first = t == 1 || refeed;
        const uint32_t any_prev = __builtin_amdgcn_readfirstlane(static_cast<int>(any_s[prev]));
        const uint32_t* cp = chg + prev * n_dyn * words;
        uint32_t* cc = chg + cur * n_dyn * words;
        for (int x = tid; x < n_dyn * words; x += kThreads) chg[next * n_dyn * words + x] = 0;
        if (tid == 0) {
            any_s[next] = 0;
            fed_s[(t + 1) & 1] = 0;
        }
        if (first) {
            products += n_lf + n_rf + n_ll + n_dd;
        } else {
            for (uint32_t m = any_prev; m != 0; m &= m - 1) products += (runs >> (8 * (__ffs(m) - 1))) & 0xFF;
            if (kDD)
                for (int r = 0; r < n_dd; ++r)
                    products += ((any_prev >> rs_left(dd, r)) | (any_prev >> rs_right(dd, r))) & 1u;
        }
        uint32_t any = 0;

        if (kDD) {
            // the bits k of row i to take: those B gained, and those whose row of C changed
            int32_t c = 0;
            for (int i = group; i < n; i += kGroups) {
                const uint32_t* brow = T + d_nt * mat + i * RW;
                const uint32_t* drow = D + i * RW;
                for (int r = 0; r < n_dd; ++r) {
                    const uint32_t* marks = cp + rs_right(dd, r) * words;
                    for (int w = sub; w < min(RW, words); w += L) c += __popc(drow[w] | (brow[w] & marks[w]));
                }
            }
            for (int o = 32; o > 0; o >>= 1) c += __shfl_down(c, o, 64);
            if ((tid & 63) == 0 && c != 0) atomicAdd(&bits_s, c);
            __syncthreads();
            const int32_t bits = bits_s;
            if (bits > 0 && (!turned || bits < kTileBits<L>)) {
                for (int i = group; i < n; i += kGroups) {
                    uint32_t* drow = D + i * RW;
                    const uint32_t* brow = T + d_nt * mat + i * RW;
                    uint4 dnew = make_uint4(0, 0, 0, 0);
                    for (int r = 0; r < n_dd; ++r) {
                        const int h = rs_head(dd, r), cn = rs_right(dd, r);
                        const uint32_t* marks = cp + cn * words;
                        const uint4* rows = reinterpret_cast<const uint4*>(T + cn * mat) + sub;
                        uint4 acc = make_uint4(0, 0, 0, 0);
                        for (int w = 0; w < min(RW, words); ++w) {
                            uint32_t m = drow[w] | (brow[w] & marks[w]);
                            const uint4* block = rows + 32 * w * L;
                            while (m != 0) {
                                int kk[4];
                                kk[0] = __ffs(m) - 1;
                                m &= m - 1;
#pragma unroll
                                for (int u = 1; u < 4; ++u) {
                                    kk[u] = m != 0 ? __ffs(m) - 1 : kk[0];
                                    m &= m - 1;  // 0 stays 0
                                }
                                uint4 v[4];
#pragma unroll
                                for (int u = 0; u < 4; ++u) v[u] = block[kk[u] * L];
#pragma unroll
                                for (int u = 0; u < 4; ++u) acc = or4(acc, v[u]);
                            }
                        }
                        uint4* trow = reinterpret_cast<uint4*>(T + h * mat + i * RW) + sub;
                        const uint4 told = *trow;
                        const uint4 nw = andnot4(acc, told);
                        if (any4(nw)) {
                            *trow = or4(told, nw);
                            if (h == d_nt) dnew = or4(dnew, nw);
                            atomicOr(cc + h * words + (i >> 5), 1u << (i & 31));
                            any |= 1u << h;
                        }
                    }
                    wave_order();  // every lane of the group has walked D's row
                    reinterpret_cast<uint4*>(drow)[sub] = dnew;  // from here on: the bits this loop gains
                    wave_order();
                }
            } else if (bits > 0) {
                for (int i = group; i < n; i += kGroups)
                    reinterpret_cast<uint4*>(D + i * RW)[sub] = make_uint4(0, 0, 0, 0);
                // C^T of every right operand, 64 x 64 bits a wavefront at a time
                const int lane = tid & 63, wave = tid >> 6, nb = lay.rows / 64;
                for (int h = 0; h < n_dyn; ++h) {
                    const int slot_tt = G.tt[h];
                    if (slot_tt < 0) continue;
                    const uint32_t* src = T + h * mat;
                    uint32_t* dst = TT + slot_tt * mat;
                    for (int b = wave; b < nb * nb; b += kThreads / 64) {
                        const int br = b / nb, bc = b % nb;
                        uint64_t x = *reinterpret_cast<const uint64_t*>(src + (64 * br + lane) * RW + 2 * bc);
                        x = transpose64(x, lane);
                        *reinterpret_cast<uint64_t*>(dst + (64 * bc + lane) * RW + 2 * br) = x;
                    }
                }
                __syncthreads();
                // tiles of 32 rows i x 128 columns j: the four words of one lane's part of row i
                const int g = lane >> 5, r32 = lane & 31;
                const int ti = (n + 31) / 32, tj = lay.rows / 128;
                dense += n_dd;
                for (int r = 0; r < n_dd; ++r) {
                    const int h = rs_head(dd, r);
                    const uint32_t* Bm = T + d_nt * mat;
                    const uint32_t* CT = TT + G.tt[rs_right(dd, r)] * mat;
                    for (int u = wave; u < ti * tj; u += kThreads / 64) {
                        const int i = (u / tj) * 32 + r32, jc = u % tj;
                        mfma::v16f acc[4];
#pragma unroll
                        for (int jb = 0; jb < 4; ++jb)
#pragma unroll
                            for (int e = 0; e < 16; ++e) acc[jb][e] = 0.0f;
#pragma unroll 1
                        for (int kc = 0; kc < (L + 1) / 2; ++kc) {  // 256 k a chunk: this half's four words
                            // one lane a row: 128 k, the other half multiplies zeros
                            const int at = L == 1 ? 0 : 2 * kc + g;
                            uint4 bv = reinterpret_cast<const uint4*>(Bm + i * RW)[at];
                            if (L == 1 && g == 1) bv = make_uint4(0, 0, 0, 0);
                            uint4 cv[4];
#pragma unroll
                            for (int jb = 0; jb < 4; ++jb)
                                cv[jb] = reinterpret_cast<const uint4*>(CT + (jc * 128 + jb * 32 + r32) * RW)[at];
#pragma unroll
                            for (int s = 0; s < 4; ++s) {
                                const mfma::v4i bb = mfma::spread4(mfma::word_of(bv, s));
#pragma unroll
                                for (int jb = 0; jb < 4; ++jb)
                                    acc[jb] = mfma::mfma_f32_32x32x64_fp4(mfma::spread4(mfma::word_of(cv[jb], s)), bb,
                                                                          acc[jb], mfma::kFmtFp4, mfma::kFmtFp4, 0, 0,
                                                                          0, 0);
                            }
                        }
                        uint32_t word[4];
#pragma unroll
                        for (int jb = 0; jb < 4; ++jb) {
                            uint32_t w = 0;
#pragma unroll
                            for (int e = 0; e < 16; ++e)
                                w |= (acc[jb][e] > 0 ? 1u : 0u) << (8 * (e / 4) + 4 * g + (e % 4));
                            word[jb] = w | static_cast<uint32_t>(__shfl_xor(static_cast<int>(w), 32, 64));
                        }
                        if (g == 0 && i < n) {
                            uint4* trow = reinterpret_cast<uint4*>(T + h * mat + i * RW) + jc;
                            const uint4 told = *trow;
                            const uint4 nw = andnot4(make_uint4(word[0], word[1], word[2], word[3]), told);
                            if (any4(nw)) {
                                *trow = or4(told, nw);
                                if (h == d_nt) {
                                    uint4* drow = reinterpret_cast<uint4*>(D + i * RW) + jc;
                                    *drow = or4(*drow, nw);
                                }
                                atomicOr(cc + h * words + (i >> 5), 1u << (i & 31));
                                any |= 1u << h;
                            }
                        }
                    }
                    __syncthreads();  // the next rule may have the same head; its rows are read below
                }
            }
        }

        // rows: pulls, then scatters -- at once, or where the rows may be
        // turned once the bits of all rows are counted (in the first loop too:
        // a lane that scatters what a rule of two lists gave its row took Dyck
        // on G(128, 2560) 330 us, 161 turned)
        const bool later = turned && src >= 0;
        uint4 held[kPasses];
        int32_t fed = 0;
#pragma unroll
        for (int ps = 0; ps < kPasses; ++ps) {
            held[ps] = make_uint4(0, 0, 0, 0);
            const int i = group + ps * kGroups;
            if (i >= n) continue;
            const uint32_t rbit = 1u << (i & 31);
            uint32_t heads = first ? (1u << n_dyn) - 1 : row_heads;
            for (; heads != 0; heads &= heads - 1) {
                const int h = __ffs(heads) - 1;
                uint32_t* trow = T + h * mat + i * RW;
                uint4 acc = make_uint4(0, 0, 0, 0);
                auto pull = [&](int r, uint32_t e, uint32_t len, int k) {
                    const int c = rs_right(lf, r);
                    const uint32_t* marks = cp + c * words;
                    const uint4* rows = reinterpret_cast<const uint4*>(T + c * mat) + sub;
                    for (uint32_t q = 0; q < len; ++q) {
                        if (q != 0) k = idx[e + q];
                        if ((marks[k >> 5] >> (k & 31)) & 1u) acc = or4(acc, rows[k * L]);
                    }
                };
#pragma unroll
                for (int r = 0; r < 2; ++r)
                    if (r < n_lf && rs_head(lf, r) == h && ((any_prev >> rs_right(lf, r)) & 1u))
                        pull(r, l0[ps][r], ln[ps][r], lk[ps][r]);
                for (int r = 2; r < n_lf; ++r) {
                    if (rs_head(lf, r) != h || !((any_prev >> rs_right(lf, r)) & 1u)) continue;
                    const uint32_t* q = end + rs_left(lf, r) * n + i;
                    if (q[0] < q[1]) pull(r, q[0], q[1] - q[0], idx[q[0]]);
                }
                if (first) {
                    // both operands fixed: the lists of the list's nodes
                    for (int r = 0; r < n_ll; ++r) {
                        if (rs_head(ll, r) != h) continue;
                        const int q = rs_left(ll, r) * n + i;
                        for (uint32_t e = end[q] + sub; e < end[q + 1]; e += L) {
                            const int q2 = rs_right(ll, r) * n + idx[e];
                            for (uint32_t f = end[q2]; f < end[q2 + 1]; ++f) {
                                const int j = idx[f];
                                const uint32_t bit = 1u << (j & 31);
                                if (!(atomicOr(trow + (j >> 5), bit) & bit)) {
                                    if (kDD && h == d_nt) atomicOr(D + i * RW + (j >> 5), bit);
                                    atomicOr(cc + h * words + (i >> 5), rbit);
                                    any |= 1u << h;
                                }
                            }
                        }
                    }
                    wave_order();
                }
                // what this loop gave row i of h feeds the scatters (in the
                // first loop with the initial bits)
                uint4 f = make_uint4(0, 0, 0, 0);
                if (first || any4(acc)) {
                    const uint4 told = reinterpret_cast<const uint4*>(trow)[sub];
                    const uint4 nw = andnot4(acc, told);
                    if (any4(nw)) {
                        reinterpret_cast<uint4*>(trow)[sub] = or4(told, nw);
                        if (kDD && h == d_nt) {
                            uint4* drow = reinterpret_cast<uint4*>(D + i * RW) + sub;
                            *drow = or4(*drow, nw);
                        }
                        atomicOr(cc + h * words + (i >> 5), rbit);
                        any |= 1u << h;
                    }
                    f = first ? or4(told, nw) : nw;
                }
                if (kDD && !first && h == d_nt) f = reinterpret_cast<const uint4*>(D + i * RW)[sub];
                if (!any4(f)) continue;
                if (!later) {
                    scatter(i, h, f, cc, any);
                } else if (h == src) {
                    held[ps] = f;
                    fed += __popc(f.x) + __popc(f.y) + __popc(f.z) + __popc(f.w);
                }
            }
        }
        bool turn = false;
        if (later) {
            if (__ballot(fed != 0) != 0) {
                for (int o = 32; o > 0; o >>= 1) fed += __shfl_down(fed, o, 64);
                if ((tid & 63) == 0) atomicAdd(&fed_s[t & 1], fed);
            }
            __syncthreads();
            turn = uni(fed_s[t & 1]) >= kTurnBits<L> * n;
            if (!turn) {
#pragma unroll
                for (int ps = 0; ps < kPasses; ++ps)
                    if (any4(held[ps])) scatter(group + ps * kGroups, src, held[ps], cc, any);
            }
        }
        if (turn) {
            const int lane = tid & 63, wave = tid >> 6, nb = lay.rows / 64;
            for (int r = 0; r < n_rf; ++r) {
                const int h = rs_left(rf, r), x = rs_head(rf, r);
                const uint32_t* from = T + h * mat;
                __syncthreads();  // T's rows are written, TT is free
                for (int b = wave; b < nb * nb; b += kThreads / 64) {
                    const int br = b / nb, bc = b % nb;
                    uint64_t v = *reinterpret_cast<const uint64_t*>(from + (64 * br + lane) * RW + 2 * bc);
                    v = transpose64(v, lane);
                    *reinterpret_cast<uint64_t*>(TT + (64 * bc + lane) * RW + 2 * br) = v;
                }
                __syncthreads();
                // column j of the result: the columns of its incoming edges; two
                // threads a column, or one
                constexpr int kPer = (L + 1) / 2;
                const int j = L == 1 ? tid : tid / 2, c0 = L == 1 ? 0 : (tid & 1) * kPer;
                uint4 acc[kPer];
#pragma unroll
                for (int q = 0; q < kPer; ++q) acc[q] = make_uint4(0, 0, 0, 0);
                if (j < n) {
                    const uint32_t* e0 = end + G.rf_in[r] * n + j;
                    for (uint32_t e = e0[0]; e < e0[1]; ++e) {
                        const uint4* col = reinterpret_cast<const uint4*>(TT + idx[e] * RW) + c0;
#pragma unroll
                        for (int q = 0; q < kPer; ++q) acc[q] = or4(acc[q], col[q]);
                    }
                }
                __syncthreads();
                if (j < lay.rows) {
#pragma unroll
                    for (int q = 0; q < kPer; ++q) reinterpret_cast<uint4*>(TT + j * RW)[c0 + q] = acc[q];
                }
                __syncthreads();
                for (int b = wave; b < nb * nb; b += kThreads / 64) {
                    const int br = b / nb, bc = b % nb;
                    uint64_t v = *reinterpret_cast<const uint64_t*>(TT + (64 * br + lane) * RW + 2 * bc);
                    v = transpose64(v, lane);
                    const int i = 64 * bc + lane;
                    uint64_t* trow = reinterpret_cast<uint64_t*>(T + x * mat + i * RW) + br;
                    const uint64_t told = *trow;
                    const uint64_t nw = v & ~told;
                    if (nw == 0) continue;
                    *trow = told | nw;
                    if (kDD && x == d_nt) reinterpret_cast<uint64_t*>(D + i * RW)[br] |= nw;
                    atomicOr(cc + x * words + (i >> 5), 1u << (i & 31));
                    any |= 1u << x;
                }
            }
        }
        if (any != 0) atomicOr(&any_s[cur], any);
        __syncthreads();
        if (kDD && tid == 0) bits_s = 0;  // read before the barrier; added to after the next one
        if (any_s[cur] == 0) break;
        if (kDD) __syncthreads();
        const int p = prev;
        prev = cur;
        cur = next;
        next = p;
        refeed = false;
        if (kQueue && t == 1 && G.queued) {
            // the bits of the rows the first loop changed, if they are few: old
            // ones among them add nothing
            __shared__ FactQueue queue;
            uint32_t* marks = chg + prev * n_dyn * words;
            if (tid == 0) queue.count = 0;
            __syncthreads();
            for (int h = 0; h < n_dyn && tid < n; ++h) {
                if (!((marks[h * words + (tid >> 5)] >> (tid & 31)) & 1u)) continue;
                const uint4 row = reinterpret_cast<const uint4*>(T + h * mat + tid * RW)[0];
                const int c = __popc(row.x) + __popc(row.y) + __popc(row.z) + __popc(row.w);
                int at = atomicAdd(&queue.count, c);
                if (at + c > kFacts) continue;
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    for (uint32_t m = w == 0 ? row.x : w == 1 ? row.y : w == 2 ? row.z : row.w; m != 0; m &= m - 1)
                        queue.q[at++] = fact(h, tid, 32 * w + __ffs(m) - 1);
            }
            __syncthreads();
            if (queue.count <= kFacts) {
                for (int x = tid; x < n_dyn * words; x += kThreads) marks[x] = 0;
                if (tid == 0) any_s[prev] = 0;
                __syncthreads();
                if (tid < 64) {
                    struct {
                        const uint64_t* near;
                        const uint32_t* end;
                        const uint16_t* idx;
                        uint64_t lf, rf, runs, lf_in;
                        int n, mat, words, n_dyn, n_lf, n_rf;
                    } u = {near, end, idx, lf, rf, runs, 0, n, mat, words, n_dyn, n_lf, n_rf};
                    for (int r = 0; r < n_lf; ++r) u.lf_in |= static_cast<uint64_t>(uni(G.lf_in[r])) << (8 * r);
                    follow_facts(u, queue, T, marks, &any_s[prev], t, d.max_iters);
                }
                __syncthreads();
                t = queue.loops;
                products += queue.products;
                capped = queue.capped;
                if (queue.count == 0) break;
                refeed = true;  // bits lost to the queue have not been scattered
            }
        }
    }

    // ---- results
    const int w4 = d.W / 2;  // 16-byte pieces of a row of the result
    for (int h = 0; h < n_dyn; ++h) {
        uint4* out = reinterpret_cast<uint4*>(gT + G.dyn_nt[h] * mdw);
        const uint4* in = reinterpret_cast<const uint4*>(T + h * mat);
        for (int x = tid; x < d.npad * w4; x += kThreads) {
            const int i = x / w4, q = x % w4;
            out[x] = i < n && q < L ? in[i * L + q] : make_uint4(0, 0, 0, 0);
        }
    }
    if (tid == 0) {
        out->iterations = t;
        out->products = products;
        out->dense = dense;
        out->capped = capped;
        out->bad_edges = bad_s;
        out->done = 1;
        out->active = 0;
    }
}

template <int L, bool kDD, bool kTurn>
__global__ __launch_bounds__(threads_for(L)) void resident_sweep_kernel(const SlotDesc* __restrict__ descs,
                                                                        SlotState* states,
                                                                        const int32_t* __restrict__ rules_tab,
                                                                        const int32_t* __restrict__ term_tab,
                                                                        const int32_t* __restrict__ ids) {
    const int slot = ids[blockIdx.x];
    const SlotDesc& d = descs[slot];
    resident_closure<L, kDD, kTurn>(d, rules_tab + 3 * d.rule_off, term_tab, states + slot);
}

// One closure by itself: what the host knows comes as kernel arguments, its
// state and clock go to pinned host memory (ResidentReport), so the call takes
// one launch and no copy.
template <int L, bool kDD, bool kTurn>
__global__ __launch_bounds__(threads_for(L)) void resident_solo_kernel(SlotDesc d, ResidentGrammar g,
                                                                       ResidentReport* report) {
    __shared__ SlotState st;
    const uint64_t begin = wall_clock64();
    resident_closure<L, kDD, kTurn>(d, reinterpret_cast<const int32_t*>(&g), nullptr, &st);
    __syncthreads();
    if (threadIdx.x != 0) return;
    report->iterations = st.iterations;
    report->products = st.products;
    if constexpr (kDD) report->dense = st.dense;
    report->capped = st.capped;
    report->bad_edges = st.bad_edges;
    report->ticks = wall_clock64() - begin;
    __threadfence_system();
    __hip_atomic_store(&report->loop, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <int L, bool kDD, bool kTurn = true>
hipError_t launch_solo(const SlotDesc& d, const ResidentPlan& p, ResidentReport* report, hipStream_t s) {
    if (p.lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&resident_solo_kernel<L, kDD, kTurn>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, p.lds);
        if (e != hipSuccess) return e;
    }
    resident_solo_kernel<L, kDD, kTurn><<<dim3(1), dim3(threads_for(L)), static_cast<size_t>(p.lds), s>>>(d, p.g,
                                                                                                      report);
    return hipGetLastError();
}

template <int L, bool kDD, bool kTurn = true>
hipError_t launch(const EngineBuffers& b, const int32_t* ids, int32_t count, int32_t lds, hipStream_t s) {
    if (lds > 64 * 1024) {  // more dynamic LDS than a launch gets unasked
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&resident_sweep_kernel<L, kDD, kTurn>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    resident_sweep_kernel<L, kDD, kTurn><<<dim3(static_cast<unsigned>(count)), dim3(threads_for(L)),
                                    static_cast<size_t>(lds), s>>>(b.descs, b.states, b.rules_tab, b.term_tab, ids);
    return hipGetLastError();
}

}  // namespace

bool resident_rules(const cfpq_grammar* gr, bool queue, ResidentPlan* plan) {
    const int32_t n_bin = gr->n_bin_rules, n_term = gr->n_term_rules;
    if (n_bin < 1 || n_bin > kRsMaxBin) {
        std::memset(&plan->g, 0, sizeof(plan->g));
        return false;
    }
    int32_t rules[3 * kRsMaxBin];
    for (int32_t r = 0; r < n_bin; ++r) {
        rules[3 * r] = gr->bin_rules[r].lhs;
        rules[3 * r + 1] = gr->bin_rules[r].left;
        rules[3 * r + 2] = gr->bin_rules[r].right;
    }
    if (!resident_grammar(rules, n_bin, gr->n_nonterminals, queue, &plan->g)) return false;
    const cfpq_term_rule* term = gr->term_rules;
    int32_t per_edge = 1;
    bool fits = n_term <= kRsMaxTerm;
    for (int32_t r = 0; r < n_term; ++r) {
        int32_t c = 0;
        for (int32_t q = 0; q < n_term; ++q) c += term[q].terminal == term[r].terminal ? 1 : 0;
        per_edge = std::max(per_edge, c);
        fits = fits && term[r].terminal < (1 << 23);
    }
    plan->per_edge = per_edge;
    if (fits) {
        plan->g.n_term = n_term;
        for (int32_t r = 0; r < n_term; ++r) plan->g.term[r] = term[r].terminal << 8 | term[r].lhs;
    }
    return true;
}

bool resident_fits(int32_t n, int64_t n_edges, ResidentPlan* plan) {
    if (n <= 0 || n > kSmallMaxPad) return false;
    const bool one = resident_lanes(n) == 1, sparse = n_edges < 2 * static_cast<int64_t>(n);
    // an edge enters at most two lists (outgoing, incoming) per terminal rule of its label
    const int64_t entries = 2 * n_edges * plan->per_edge;
    // one lane a row: with two edges a node and more.  On sparser graphs a loop
    // sets few bits, and the kernel without the turned code takes a fifth less a
    // loop over rows (two cycles of 64 and 63 nodes, without follow_facts: 5.6
    // against 6.9 ms; same-generation on G(100, 300), where the turned code runs:
    // 265 against 161 us)
    const bool want = (plan->g.n_dd > 0 || plan->g.n_rf > 0) && !(one && sparse);
    const int32_t walked = resident_lanes(n) / 2 + (plan->g.n_dd > 0 ? 3 : 0);  // the class without turned operands
    ResidentLds l = resident_lds(n, plan->g, entries, want);
    plan->cls = one && want ? (plan->g.n_dd > 0 ? 7 : 6) : walked;
    plan->turned = want && l.total <= resident_max_lds(plan->cls) ? 1 : 0;
    if (!plan->turned) {
        plan->cls = walked;
        l = resident_lds(n, plan->g, entries, false);
    }
    if (l.total > resident_max_lds(plan->cls)) return false;
    // Lists are walked entry by entry: dense graphs go to the kernel that
    // multiplies.  The lines, in edges a node, with both sides in us (that
    // kernel, this one): pulls beside scatters or rules of two lists 12 (Dyck,
    // n = 128: 136, 127; 24: 133, 177); pulls alone 24 (103, 94; 40: 106, 136);
    // scatters without turned operands 8 (four heads, n = 512: 999, 732; 10:
    // 685, 696), with products beside them 6 (three heads: 746, 707; 8: 657,
    // 737); scatters from several nonterminals, which are never turned, 2 up
    // to two lanes a row (n = 128: 163, 96; 3: 196, 224) and 5 beyond (n = 512,
    // 6: 828, 793; 8: 613, 581; n = 400, 6: 621, 712).
    const ResidentGrammar& g = plan->g;
    int64_t most = g.n_ll > 0 || (g.n_lf > 0 && g.n_rf > 0) ? 12 : g.n_lf > 0 ? 24 : n_edges;
    if (g.n_rf > 0 && !plan->turned) most = std::min<int64_t>(most, g.n_dd > 0 ? 6 : 8);
    if (g.n_rf > 0 && g.src < 0) most = std::min<int64_t>(most, resident_lanes(n) < 4 ? 2 : 5);
    if (n_edges > most * n) return false;
    plan->lds = l.total;
    return true;
}

hipError_t resident_solo(const SlotDesc& d, const ResidentPlan& p, ResidentReport* report, hipStream_t s) {
    switch (p.cls) {
        case 0: return launch_solo<1, false, false>(d, p, report, s);
        case 1: return launch_solo<2, false>(d, p, report, s);
        case 2: return launch_solo<4, false>(d, p, report, s);
        case 3: return launch_solo<1, true, false>(d, p, report, s);
        case 4: return launch_solo<2, true>(d, p, report, s);
        case 5: return launch_solo<4, true>(d, p, report, s);
        case 6: return launch_solo<1, false>(d, p, report, s);
        default: return launch_solo<1, true>(d, p, report, s);
    }
}

hipError_t resident_sweep(const EngineBuffers& b, const int32_t* ids, int32_t count, int32_t cls, int32_t lds,
                          hipStream_t s) {
    if (count <= 0) return hipSuccess;
    switch (cls) {
        case 0: return launch<1, false, false>(b, ids, count, lds, s);
        case 1: return launch<2, false>(b, ids, count, lds, s);
        case 2: return launch<4, false>(b, ids, count, lds, s);
        case 3: return launch<1, true, false>(b, ids, count, lds, s);
        case 4: return launch<2, true>(b, ids, count, lds, s);
        case 5: return launch<4, true>(b, ids, count, lds, s);
        case 6: return launch<1, false>(b, ids, count, lds, s);
        default: return launch<1, true>(b, ids, count, lds, s);
    }
}

}  // namespace cfpq
