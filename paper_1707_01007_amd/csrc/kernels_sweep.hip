// Kernels of the row sweeps (see sweep.h).
#include <algorithm>

#include "near_list.h"
#include "rowor_device.h"
#include "sweep.h"

namespace cfpq {
namespace {

constexpr int kWaves = 4;             // wavefronts of a sweep_clean_kernel workgroup
constexpr int64_t kMaxBlocks = 2048;  // and its grid: eight workgroups per CU

// T, then the bitmaps, counters and control block (contiguous), cleared in
// one launch.
__global__ __launch_bounds__(256) void sweep_clear_kernel(uint4* __restrict__ a, size_t na, uint4* __restrict__ b,
                                                          size_t nb) {
    const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
    for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < na + nb; i += stride) {
        if (i < na)
            a[i] = make_uint4(0, 0, 0, 0);
        else
            b[i - na] = make_uint4(0, 0, 0, 0);
    }
}

struct InitArgs {
    SweepGrammar::Term term[kSwMaxTerm];
    int32_t n_term, n, n_terminals;
    int64_t W, mat_words;
};

// counter[i * stride] += 1 on the active lanes; the value before it, a different
// one a lane.  Lanes with the first one's i add together when they are many: a
// hub's edges (a star of 16384 nodes spent 200 us a kernel on one counter, now
// 21 in the scatter and 5 in the fill).
__device__ __forceinline__ int32_t count_up(int32_t* counter, int32_t stride, int32_t i) {
    constexpr int kMany = 24;
    int32_t* at = counter + static_cast<int64_t>(i) * stride;
    const bool same = i == __builtin_amdgcn_readfirstlane(i);
    const uint64_t m = __ballot(same);
    if (__popcll(m) < kMany || !same) return atomicAdd(at, 1);
    const int lane = threadIdx.x & 63, who = __ffsll(static_cast<unsigned long long>(m)) - 1;
    int32_t base = 0;
    if (lane == who) base = atomicAdd(at, static_cast<int32_t>(__popcll(m)));
    return __builtin_amdgcn_readlane(base, who) + static_cast<int32_t>(__popcll(m & ((1ull << lane) - 1)));
}

// One thread per edge: the bits of Algorithm 1's matrix initialisation, and
// the lengths of the adjacency lists.  Parallel edges may enter a list twice.
__global__ __launch_bounds__(256) void sweep_scatter_kernel(const cfpq_edge* __restrict__ edges, int64_t m,
                                                            InitArgs a, uint64_t* T, int2* list, SweepCtl* ctl) {
    const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (e >= m) return;
    const cfpq_edge ed = edges[e];
    if (ed.src < 0 || ed.src >= a.n || ed.dst < 0 || ed.dst >= a.n || ed.label < 0 || ed.label >= a.n_terminals) {
        atomicAdd(&ctl->bad_edges, 1);
        return;
    }
    const unsigned long long bit = 1ull << (ed.dst & 63);
    const int64_t off = static_cast<int64_t>(ed.src) * a.W + (ed.dst >> 6);
    for (int32_t q = 0; q < a.n_term; ++q) {
        if (a.term[q].label != ed.label) continue;
        atomicOr(reinterpret_cast<unsigned long long*>(T + a.term[q].nt * a.mat_words + off), bit);
        if (a.term[q].out >= 0) count_up(&list[0].y, 2, a.term[q].out * a.n + ed.src);
        if (a.term[q].in >= 0) count_up(&list[0].y, 2, a.term[q].in * a.n + ed.dst);
    }
}

// Entries from which a list is a hub's.
__host__ __device__ inline int32_t hub_list(int64_t W) { return static_cast<int32_t>(kSwHubWords / W); }

// Lists that would be hubs: the fixed operands of lf and of rf rules (n_rules = 0:
// none are looked for), and their nonterminals.
struct HubArgs {
    uint8_t list[2 * kSwMaxRules], nt[2 * kSwMaxRules];
    int32_t n_rules, n, longest;
};

// Places of the lists in idx: a workgroup's lists are consecutive, the
// workgroups' runs come in any order (one atomic each).
__global__ __launch_bounds__(256) void sweep_place_kernel(int2* list, int32_t* __restrict__ cur,
                                                          uint4* __restrict__ near, int32_t lists, SweepCtl* ctl,
                                                          HubArgs hubs) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __shared__ int32_t wave_tot[4], base_s;
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    const int32_t c = i < lists ? list[i].y : 0;
    int32_t x = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wave_tot[wave] = x;
    __syncthreads();
    if (threadIdx.x == 0) base_s = atomicAdd(&ctl->list_top, wave_tot[0] + wave_tot[1] + wave_tot[2] + wave_tot[3]);
    __syncthreads();
    int32_t at = base_s + x - c;
    for (int w = 0; w < wave; ++w) at += wave_tot[w];
    if (i >= lists) return;
    list[i].x = at;
    if (c >= hubs.longest)
        for (int32_t r = 0; r < hubs.n_rules; ++r)
            if (hubs.list[r] == i / hubs.n) {
                const int32_t q = atomicAdd(&ctl->n_hubs, 1);
                if (q < kSwMaxHubs) ctl->hub[q] = make_int2(r | hubs.nt[r] << 8, i % hubs.n);
            }
    cur[i] = 0;
    near[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
}

__global__ __launch_bounds__(256) void sweep_fill_kernel(const cfpq_edge* __restrict__ edges, int64_t m, InitArgs a,
                                                         const int2* __restrict__ list, int32_t* cur,
                                                         uint4* near, int32_t* __restrict__ idx, int32_t longest) {
    const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (e >= m) return;
    const cfpq_edge ed = edges[e];
    if (ed.src < 0 || ed.src >= a.n || ed.dst < 0 || ed.dst >= a.n || ed.label < 0 || ed.label >= a.n_terminals)
        return;  // counted by the scatter
    auto put = [&](int32_t i, int32_t k) {
        const int2 l = list[i];
        // (hubs' lists come out sorted; the others stay in the order of the
        // atomics, which spreads the bits that a scatter sets together)
        const int32_t nth = l.y >= longest ? count_up(cur, 1, i) : atomicAdd(cur + i, 1);
        idx[l.x + nth] = k;
        put_near(reinterpret_cast<uint16_t*>(near + i), nth, l.y, k);
    };
    for (int32_t q = 0; q < a.n_term; ++q) {
        if (a.term[q].label != ed.label) continue;
        if (a.term[q].out >= 0) put(a.term[q].out * a.n + ed.src, ed.dst);
        if (a.term[q].in >= 0) put(a.term[q].in * a.n + ed.dst, ed.src);
    }
}

struct SweepArgs {
    SweepGrammar g;
    uint64_t* T;
    const uint64_t* Dprev;
    uint64_t* Dcur;
    const uint64_t* P;
    uint64_t* chg;
    SweepCtl* ctl;
    const int32_t* wg_prev;
    int32_t* wg_cur;
    const int2* list;
    const uint4* near;
    const int32_t* idx;
    int64_t W, mat_words;
    int32_t n, t, rows;  // rows of a workgroup: 16, 32 or 64
    uint32_t p_mask;
    int32_t count, dense_dd;
};

// Lists longer than this are pulled by the whole workgroup instead of a wavefront.
constexpr int32_t kLongPull = 256;

// ORs into acc the rows src[k, :] of the lanes' k (kNone: none) for which
// live(k).  Returns whether there was one.  Rows are read four at a time (a
// missing one repeats the last).
template <int WPL, typename Live>
__device__ __forceinline__ bool pull_lanes(const uint64_t* src, int64_t W, const uint32_t (&off)[WPL], uint32_t k,
                                           Live live, uint64_t (&acc)[WPL]) {
    uint64_t m = __ballot(k < kMore && live(static_cast<int32_t>(k)));
    const bool got = m != 0;
    while (m != 0) {
        const uint64_t* row[4];
        int l = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (m != 0) l = __ffsll(static_cast<unsigned long long>(m)) - 1;
            m &= m - 1;
            row[u] = src + static_cast<int64_t>(__builtin_amdgcn_readlane(static_cast<int>(k), l)) * W;
        }
        uint64_t v[4][WPL];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < WPL; ++q) v[u][q] = row[u][off[q]];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < WPL; ++q) acc[q] |= v[u][q];
    }
    return got;
}

// The rows of a whole list: entries part * 64 + [0, 64), then every parts * 64 on.
template <int WPL, typename Live>
__device__ __forceinline__ bool pull_list(const uint64_t* src, int64_t W, const uint32_t (&off)[WPL], int lane, int2 l,
                                          int part, int parts, const int32_t* __restrict__ idx, Live live,
                                          uint64_t (&acc)[WPL]) {
    bool got = false;
    for (int32_t b = part * 64; b < l.y; b += parts * 64)
        got |= pull_lanes<WPL>(src, W, off, b + lane < l.y ? static_cast<uint32_t>(idx[l.x + b + lane]) : kNone, live,
                               acc);
    return got;
}

// One loop.  A workgroup of 16 wavefronts takes `rows` consecutive rows of
// every dynamic nonterminal and is their only writer.
//  1. Pulls, a wavefront a row: per head the changed rows its lists select
//     (in the first loop rows of T, which hold the initial bits, in later ones
//     the last loop's D) and P's row; the new bits are stored at once.  A hub's
//     rows (a list of many entries: up to 32 MiB, which one workgroup takes
//     600 us for) are pulled by all workgroups, 64 entries a wavefront, into
//     an inbox row that its own workgroup takes over a loop later (a star of
//     16384 nodes, S -> A S | a: 1427 -> 208 us with the counters below, 428 by
//     products).
//  2. Scatters, per head of an rf rule: from the bits its operands gained in
//     step 1 (an operand that is itself such a head feeds a loop later, from
//     D; in the first loop T's rows feed).  Few bits are scattered one by one
//     into an LDS row.  Many are turned: the workgroup's rows are transposed
//     64 x 64 bits at a time in LDS, which makes column k one 64-bit word over
//     the rows, and column j of the result is the OR of the words k of its
//     incoming edges -- one LDS read an edge for all rows together, whatever
//     the density, where the scatter takes one atomic an edge and bit (at
//     n = 16384 and three quarters of the bits set, 1700 us).
// T rows are read while other workgroups add to them only in the first loop:
// old or new, they are subsets of the fixpoint that hold the initial bits.
//
// What bounds it: idle rows read their lists and the bitmaps (latency; two or
// more rows in flight a SIMD), active ones move rows of D and T.
template <int WPL, bool kFirst>
__global__ __launch_bounds__(1024) void sweep_kernel(SweepArgs a) {
    extern __shared__ __align__(16) uint64_t buf[];  // 64 rows of W + 1 words, n_dyn bitmaps of W
    __shared__ uint32_t any_s;
    __shared__ unsigned long long gained_s[kSwMaxDyn], rows_s[kSwMaxDyn];  // this loop's bits and changed rows
    __shared__ unsigned long long long_s;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int64_t W = a.W;
    const int stride = static_cast<int>(W) + 1;
    const int n_dyn = a.g.n_dyn;
    const int cur = a.t & 3, prev = (a.t - 1) & 3, next = (a.t + 1) & 3;
    SweepCtl* ctl = a.ctl;
    uint32_t any_prev = kFirst ? ~0u : ctl->any[prev];
    if (kFirst && (WPL <= 2 || ctl->n_hubs == 0 || ctl->n_hubs > kSwMaxHubs)) any_prev &= ~kSwHubsBit;
    const auto hubs = [&] { return WPL > 2 && (any_prev & kSwHubsBit) != 0; };
    if (blockIdx.x == 0) {
        for (int64_t x = threadIdx.x; x < n_dyn * W; x += blockDim.x) a.chg[next * n_dyn * W + x] = 0;
        if (threadIdx.x < kSwMaxDyn) ctl->gained[next][threadIdx.x] = 0;
        if (threadIdx.x == 0) {
            ctl->any[next] = 0;
            if (any_prev != 0) {
                // rules this loop runs: an operand changed in the last one
                int32_t sp = kFirst ? a.g.n_ll : 0, de = 0;
                for (int r = 0; r < a.g.n_lf; ++r) sp += (any_prev >> a.g.lf[r].right) & 1u;
                for (int r = 0; r < a.g.n_rf; ++r) sp += (any_prev >> a.g.rf[r].left) & 1u;
                if (a.dense_dd)
                    for (int r = 0; r < a.g.n_dd; ++r)
                        de += ((any_prev >> a.g.dd[r].left) | (any_prev >> a.g.dd[r].right)) & 1u;
                ctl->loops = a.t;
                ctl->sparse += sp;
                ctl->delta += kFirst ? 0 : sp;
                ctl->dense += de;
                ctl->products += sp + de;
            }
        }
    }
    if (any_prev == 0) return;  // the fixpoint was reached (uniform over the grid)
    if (threadIdx.x == 0) {
        any_s = 0;
        long_s = 0;
    }
    if (threadIdx.x < kSwMaxDyn) {
        gained_s[threadIdx.x] = 0;
        rows_s[threadIdx.x] = 0;
    }
    // the last loop's changed rows
    uint64_t* marks = buf + 64 * stride;
    if (!kFirst)
        for (int64_t x = threadIdx.x; x < n_dyn * W; x += blockDim.x) marks[x] = a.chg[prev * n_dyn * W + x];
    __syncthreads();
    uint64_t* chg_cur = a.chg + cur * n_dyn * W;
    const int32_t row0 = static_cast<int32_t>(blockIdx.x) * a.rows;
    const int32_t nrows = min(a.rows, a.n - row0);
    uint32_t off[WPL];
    bool valid[WPL];
#pragma unroll
    for (int q = 0; q < WPL; ++q) {
        valid[q] = lane + 64 * q < W;
        off[q] = static_cast<uint32_t>(valid[q] ? lane + 64 * q : W - 1);
    }
    auto T_row = [&](int h, int lr) { return a.T + a.g.dyn_nt[h] * a.mat_words + static_cast<int64_t>(row0 + lr) * W; };
    // New bits nw of row lr of head h, by one wavefront: those T lacks are
    // stored, kept as D's row (added to what the loop already put there) and marked.
    auto commit = [&](int h, int lr, uint64_t (&nw)[WPL]) {
        uint64_t* trow = T_row(h, lr);
        uint64_t told[WPL];
        bool mine = false;
#pragma unroll
        for (int q = 0; q < WPL; ++q) told[q] = trow[off[q]];
#pragma unroll
        for (int q = 0; q < WPL; ++q) {
            nw[q] = valid[q] ? nw[q] & ~told[q] : 0;
            mine = mine || nw[q] != 0;
        }
        if (__ballot(mine) == 0) return;
        uint64_t* drow = a.Dcur + h * a.mat_words + static_cast<int64_t>(row0 + lr) * W;
        const bool again = (rows_s[h] >> lr) & 1ull;
        unsigned long long c = 0;
#pragma unroll
        for (int q = 0; q < WPL; ++q) {
            if (!valid[q]) continue;
            if (nw[q] != 0) trow[off[q]] = told[q] | nw[q];
            drow[off[q]] = again ? drow[off[q]] | nw[q] : nw[q];
            c += __popcll(nw[q]);
        }
        for (int o = 32; o > 0; o >>= 1) c += __shfl_down(c, o, 64);
        if (lane == 0) {
            atomicOr(&rows_s[h], 1ull << lr);
            atomicAdd(&gained_s[h], c);
        }
    };
    // this lane's entry of node list i's 16-byte form, and whether there are more
    auto near_entry = [&](int64_t i) -> uint32_t {
        return lane < 8 ? reinterpret_cast<const uint16_t*>(a.near)[8 * i + lane] : kNone;
    };
    auto more_than_near = [&](uint32_t k) {
        return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(k), 7)) == kMore;
    };
    // the rows head h pulls into row lr, but for lists past kLongPull (their rows
    // are noted); or, whole, this wavefront's part of all lists
    bool lng = false;
    auto pull_head = [&](int h, int lr, bool whole, uint64_t (&acc)[WPL]) {
        bool got = false;
        for (int r = 0; r < a.g.n_lf; ++r) {
            const int c = a.g.lf[r].right;
            if (a.g.lf[r].head != h) continue;
            if (kFirst ? !((a.g.init_mask >> c) & 1u) : !((any_prev >> c) & 1u)) continue;
            const int64_t i = static_cast<int64_t>(a.g.lf[r].left) * a.n + row0 + lr;
            const uint64_t* src = kFirst ? a.T + a.g.dyn_nt[c] * a.mat_words : a.Dprev + c * a.mat_words;
            auto live = [&](int32_t k) { return kFirst || ((marks[c * W + (k >> 6)] >> (k & 63)) & 1ull) != 0; };
            const uint32_t k = near_entry(i);
            if (!whole && !more_than_near(k)) {
                got |= pull_lanes<WPL>(src, W, off, k, live, acc);
                continue;
            }
            const int2 l = a.list[i];
            if (hubs() && l.y >= hub_list(W)) continue;
            if (whole || l.y <= kLongPull)
                got |= pull_list<WPL>(src, W, off, lane, l, whole ? wave : 0, whole ? 16 : 1, a.idx, live, acc);
            else
                lng = true;
        }
        return got;
    };

    // ---- 1. pulls
    for (int lr = wave; lr < nrows; lr += 16) {
        lng = false;
        for (int h = 0; h < n_dyn; ++h) {
            uint64_t acc[WPL];
#pragma unroll
            for (int q = 0; q < WPL; ++q) acc[q] = 0;
            bool got = pull_head(h, lr, false, acc);
            if ((a.p_mask >> h) & 1u) {
                const int slot = __popc(a.g.p_mask & ((1u << h) - 1));
                const uint64_t* prow = a.P + slot * a.mat_words + static_cast<int64_t>(row0 + lr) * W;
#pragma unroll
                for (int q = 0; q < WPL; ++q) acc[q] |= prow[off[q]];
                got = true;
            }
            if (got) commit(h, lr, acc);
        }
        if (lng && lane == 0) atomicOr(&long_s, 1ull << lr);  // left to the whole workgroup, below
    }
    __syncthreads();
    for (uint64_t lm = long_s; lm != 0; lm &= lm - 1) {  // uniform over the workgroup
        const int lr = __ffsll(static_cast<unsigned long long>(lm)) - 1;
        for (int h = 0; h < n_dyn; ++h) {
            for (int64_t w = threadIdx.x; w < W; w += blockDim.x) buf[w] = 0;
            __syncthreads();
            uint64_t acc[WPL];
#pragma unroll
            for (int q = 0; q < WPL; ++q) acc[q] = 0;
            if (pull_head(h, lr, true, acc)) {
#pragma unroll
                for (int q = 0; q < WPL; ++q)
                    if (valid[q] && acc[q] != 0)
                        atomicOr(reinterpret_cast<unsigned long long*>(buf + off[q]),
                                 static_cast<unsigned long long>(acc[q]));
            }
            __syncthreads();
            if (wave == 0) {
#pragma unroll
                for (int q = 0; q < WPL; ++q) acc[q] = buf[off[q]];
                commit(h, lr, acc);
            }
            __syncthreads();
        }
    }

    // hubs: what the last loop left in the inbox of this workgroup's rows, then
    // this workgroup's part of their lists, as far as T lacks it
    if (hubs()) {
        const int32_t n_hubs = ctl->n_hubs;
        auto* inbox = reinterpret_cast<uint64_t*>(ctl + 1);  // [2][kSwMaxHubs][W], by loop parity
        for (int q = 0; q < n_hubs; ++q) {  // uniform over the workgroup
            const int lr = ctl->hub[q].y - row0, r = ctl->hub[q].x & 255;
            if (r >= a.g.n_lf) continue;
            if (kFirst || !(any_prev & kSwInboxBit) || lr < 0 || lr >= nrows) continue;
            if (wave == 0) {
                uint64_t* in = inbox + (static_cast<int64_t>(prev & 1) * kSwMaxHubs + q) * W;
                uint64_t acc[WPL];
#pragma unroll
                for (int u = 0; u < WPL; ++u) {
                    acc[u] = in[off[u]];
                    if (valid[u]) in[off[u]] = 0;
                }
                commit(a.g.lf[r].head, lr, acc);
            }
            __syncthreads();
        }
        for (int q = 0; q < n_hubs; ++q) {
            const int r = ctl->hub[q].x & 255;
            if (r >= a.g.n_lf) continue;
            const auto rule = a.g.lf[r];
            const int c = rule.right;
            if (kFirst ? !((a.g.init_mask >> c) & 1u) : !((any_prev >> c) & 1u)) continue;
            const int32_t node = ctl->hub[q].y;
            const int2 l = a.list[static_cast<int64_t>(rule.left) * a.n + node];
            const uint64_t* src = kFirst ? a.T + a.g.dyn_nt[c] * a.mat_words : a.Dprev + c * a.mat_words;
            auto live = [&](int32_t k) { return kFirst || ((marks[c * W + (k >> 6)] >> (k & 63)) & 1ull) != 0; };
            uint64_t acc[WPL];
#pragma unroll
            for (int u = 0; u < WPL; ++u) acc[u] = 0;
            if (!pull_list<WPL>(src, W, off, lane, l, static_cast<int>(blockIdx.x + gridDim.x * wave),
                                static_cast<int>(16 * gridDim.x), a.idx, live, acc))
                continue;
            const uint64_t* trow = a.T + a.g.dyn_nt[rule.head] * a.mat_words + static_cast<int64_t>(node) * W;
            auto* in = reinterpret_cast<unsigned long long*>(
                inbox + (static_cast<int64_t>(cur & 1) * kSwMaxHubs + q) * W);
            bool fresh = false;
#pragma unroll
            for (int u = 0; u < WPL; ++u) {
                const uint64_t nw = valid[u] ? acc[u] & ~trow[off[u]] : 0;
                if (nw == 0) continue;
                fresh = true;
                atomicOr(in + off[u], static_cast<unsigned long long>(nw));
            }
            if (__ballot(fresh) != 0 && lane == 0) atomicOr(&any_s, kSwInboxBit);
        }
    }

    // ---- 2. scatters
    const uint64_t all_rows = nrows == 64 ? ~0ull : (1ull << nrows) - 1;
    // rows of operand h that feed this loop's scatters, and where they are
    auto late = [&](int h) { return ((a.g.rf_mask >> h) & 1u) != 0; };
    auto feed_rows = [&](int h) -> uint64_t {
        if (kFirst) return (a.g.init_mask >> h) & 1u ? all_rows : rows_s[h];
        return late(h) ? (marks[h * W + (row0 >> 6)] >> (row0 & 63)) & all_rows : rows_s[h];
    };
    auto feed_row = [&](int h, int lr) -> const uint64_t* {
        if (kFirst) return T_row(h, lr);
        return (late(h) ? a.Dprev : a.Dcur) + h * a.mat_words + static_cast<int64_t>(row0 + lr) * W;
    };
    // The hubs of rf rule r among the bits f: their lists are rows of the operand's
    // matrix, ORed in whole.  Entry by entry the bits of one word wait for each
    // other: the first loop of a star of 16384 nodes, S -> S A | a, 218 us, and 861
    // with its list in order; 75 so.
    auto hub_bits = [&](int r, uint64_t (&f)[WPL], uint64_t* xrow) {
        for (int q = 0; q < ctl->n_hubs; ++q) {
            if ((ctl->hub[q].x & 255) != a.g.n_lf + r) continue;
            const int32_t k = ctl->hub[q].y;
            bool mine = false;
#pragma unroll
            for (int u = 0; u < WPL; ++u)
                if (lane + 64 * u == k >> 6 && ((f[u] >> (k & 63)) & 1ull)) {
                    mine = true;
                    f[u] &= ~(1ull << (k & 63));
                }
            if (__ballot(mine) == 0) continue;
            const uint64_t* row = a.T + (ctl->hub[q].x >> 8) * a.mat_words + static_cast<int64_t>(k) * W;
#pragma unroll
            for (int u = 0; u < WPL; ++u)
                if (valid[u]) atomicOr(reinterpret_cast<unsigned long long*>(xrow + off[u]),
                                       static_cast<unsigned long long>(row[off[u]]));
        }
    };
    // the first loop's heads of ll rules alone come first: they may feed the others
    const uint32_t only_ll = kFirst ? a.g.ll_mask & ~a.g.rf_mask : 0;
    for (int o = 0; o < 2 * n_dyn; ++o) {
        const int th = o < n_dyn ? o : o - n_dyn;
        if (!(((o < n_dyn ? only_ll : a.g.rf_mask) >> th) & 1u)) continue;
        // the feeding rows and bits of this target's rules (uniform)
        uint64_t fed = 0;
        bool many = false;
        __syncthreads();  // rows_s and gained_s of the heads before th are final, buf is free
        for (int r = 0; r < a.g.n_rf; ++r) {
            if (a.g.rf[r].head != th) continue;
            const int h = a.g.rf[r].left;
            const uint64_t m = feed_rows(h);
            fed |= m;
            // 24 bits a row: a lane scatters four bits a step, some 2 us, the turn takes about 10
            const unsigned long long bits =
                late(h) ? (m != 0 ? a.wg_prev[h * gridDim.x + blockIdx.x] : 0) : gained_s[h];
            many = many || (!kFirst && bits > static_cast<unsigned long long>(24 * nrows));
        }
        bool ll = false;
        if (kFirst)
            for (int r = 0; r < a.g.n_ll; ++r) ll = ll || a.g.ll[r].head == th;
        if (ll) fed = all_rows;
        if (fed == 0) continue;
        __syncthreads();  // every wavefront has read the counts above
        if (!many) {
            for (int lr = wave; lr < nrows; lr += 16) {
                if (!((fed >> lr) & 1ull)) continue;
                uint64_t* xrow = buf + lr * stride;
                uint32_t* lds32 = reinterpret_cast<uint32_t*>(buf);
#pragma unroll
                for (int q = 0; q < WPL; ++q)
                    if (valid[q]) xrow[off[q]] = 0;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                for (int r = 0; r < a.g.n_rf; ++r) {
                    const int h = a.g.rf[r].left;
                    if (a.g.rf[r].head != th || !((feed_rows(h) >> lr) & 1ull)) continue;
                    const uint64_t* frow = feed_row(h, lr);
                    uint64_t f[WPL];
#pragma unroll
                    for (int q = 0; q < WPL; ++q) f[q] = valid[q] ? frow[off[q]] : 0;
                    if (hubs()) hub_bits(r, f, xrow);
                    const int64_t l = static_cast<int64_t>(a.g.rf[r].right) * a.n;
#pragma unroll
                    for (int q = 0; q < WPL; ++q)
                        scatter_word(f[q], l + (lane + 64 * q) * 64, a.near, a.list, a.idx, lds32, lr * stride * 2,
                                     lane);
                }
                if (kFirst) {
                    // A -> B C with both fixed: the edges k -> j of C for the edges row -> k of B
                    for (int r = 0; r < a.g.n_ll; ++r) {
                        if (a.g.ll[r].head != th) continue;
                        const int64_t cb = static_cast<int64_t>(a.g.ll[r].right) * a.n;
                        const int2 l = a.list[static_cast<int64_t>(a.g.ll[r].left) * a.n + row0 + lr];
                        for (int32_t b = 0; b < l.y; b += 64) {
                            const bool have = b + lane < l.y;
                            const int64_t k = cb + (have ? a.idx[l.x + b + lane] : 0);
                            const uint4 v = have ? a.near[k] : make_uint4(~0u, ~0u, ~0u, ~0u);
                            scatter_list(v, have, k, a.list, a.idx, lds32, lr * stride * 2, lane);
                        }
                    }
                }
                // every scatter of this wavefront has reached LDS before its row is read
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                uint64_t nw[WPL];
#pragma unroll
                for (int q = 0; q < WPL; ++q) nw[q] = xrow[off[q]];
                commit(th, lr, nw);
            }
            continue;
        }
        // turned: this wavefront's columns are the 64-column words wave, wave + 16, ...
        uint64_t acc[4 * WPL];
#pragma unroll
        for (int i = 0; i < 4 * WPL; ++i) acc[i] = 0;
        for (int r = 0; r < a.g.n_rf; ++r) {
            if (a.g.rf[r].head != th) continue;
            const int h = a.g.rf[r].left;
            const uint64_t m = feed_rows(h);
            if (m == 0) continue;
            __syncthreads();  // buf is free
            for (int lr = wave; lr < nrows; lr += 16) {
                if (!((m >> lr) & 1ull)) continue;
                const uint64_t* frow = feed_row(h, lr);
#pragma unroll
                for (int q = 0; q < WPL; ++q)
                    if (valid[q]) buf[lr * stride + off[q]] = frow[off[q]];
            }
            __syncthreads();
            const bool have = (m >> lane) & 1ull;
            for (int64_t c = wave; c < W; c += 16) {
                uint64_t x = have ? buf[lane * stride + c] : 0;
                if (__ballot(x != 0) != 0) x = transpose64(x, lane);
                buf[lane * stride + c] = x;
            }
            __syncthreads();
            const int64_t l = static_cast<int64_t>(a.g.rf_in[r]) * a.n;
#pragma unroll
            for (int i = 0; i < 4 * WPL; ++i) {
                const int32_t j = (wave + 16 * i) * 64 + lane;
                acc[i] |= gather_words(buf, stride, lane, j < a.n, l + j, a.near, a.list, a.idx);
            }
        }
        __syncthreads();  // every read of the turned operands is done
#pragma unroll
        for (int i = 0; i < 4 * WPL; ++i) {
            const int64_t c = wave + 16 * i;
            if (c >= W) break;  // uniform over the wavefront
            uint64_t x = acc[i];
            if (__ballot(x != 0) != 0) x = transpose64(x, lane);
            buf[lane * stride + c] = x;
        }
        __syncthreads();
        for (int lr = wave; lr < nrows; lr += 16) {
            uint64_t nw[WPL];
#pragma unroll
            for (int q = 0; q < WPL; ++q) nw[q] = buf[lr * stride + off[q]];
            commit(th, lr, nw);
        }
    }
    __syncthreads();
    // D rows that this loop did not write keep an older loop's bits: where a
    // dd rule reads a whole D matrix they are cleared first (sweep_clean_kernel)
    if (threadIdx.x < n_dyn) {
        const int h = threadIdx.x;
        const uint64_t m = rows_s[h];
        if (m != 0) {
            a.wg_cur[h * gridDim.x + blockIdx.x] = static_cast<int32_t>(gained_s[h]);
            atomicOr(reinterpret_cast<unsigned long long*>(chg_cur + h * W + (row0 >> 6)),
                     static_cast<unsigned long long>(m << (row0 & 63)));
            atomicOr(&any_s, 1u << h);
            if (a.count) atomicAdd(&ctl->gained[cur][h], gained_s[h]);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && any_s != 0) {
        if (hubs()) any_s |= kSwHubsBit;
        const uint32_t have = __hip_atomic_load(&ctl->any[cur], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((any_s & ~have) != 0) atomicOr(&ctl->any[cur], any_s);
    }
}

// Clears the rows of D (npad rows) whose mark is clear; a wavefront a row.
__global__ __launch_bounds__(256) void sweep_clean_kernel(uint64_t* __restrict__ D, const uint64_t* __restrict__ marks,
                                                          int64_t W, int64_t npad) {
    const int lane = threadIdx.x & 63;
    for (int64_t row = static_cast<int64_t>(blockIdx.x) * kWaves + (threadIdx.x >> 6); row < npad;
         row += static_cast<int64_t>(gridDim.x) * kWaves) {
        if ((marks[row >> 6] >> (row & 63)) & 1ull) continue;
        for (int64_t w = lane; w < W; w += 64) D[row * W + w] = 0;
    }
}

// One wavefront: loop t's state to the host.
__global__ void sweep_report_kernel(const SweepCtl* __restrict__ ctl, int32_t t, SweepReport* out) {
    if (threadIdx.x != 0) return;
    out->any = ctl->any[t & 3];
    out->bad_edges = ctl->bad_edges;
    out->loops = ctl->loops;
    out->products = ctl->products;
    out->sparse = ctl->sparse;
    out->delta = ctl->delta;
    out->dense = ctl->dense;
    for (int h = 0; h < kSwMaxDyn; ++h) out->gained[h] = ctl->gained[t & 3][h];
    __threadfence_system();
    __hip_atomic_store(&out->loop, t, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <int WPL, bool kFirst>
hipError_t sweep_launch(const SweepArgs& a, dim3 grid, size_t lds, hipStream_t s) {
    // more than 64 KiB of dynamic LDS has to be asked for
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sweep_kernel<WPL, kFirst>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
        if (e != hipSuccess) return e;
    }
    sweep_kernel<WPL, kFirst><<<grid, dim3(1024), lds, s>>>(a);
    return hipGetLastError();
}

}  // namespace

bool sweep_grammar(const cfpq_grammar* gr, SweepGrammar* result) {
    SweepGrammar g;
    const int32_t n_nt = gr->n_nonterminals;
    if (gr->n_bin_rules < 1 || gr->n_bin_rules > kSwMaxRules || gr->n_term_rules > kSwMaxTerm) return false;
    int8_t dyn[CFPQ_MAX_NONTERMINALS], out[CFPQ_MAX_NONTERMINALS], in[CFPQ_MAX_NONTERMINALS];
    for (auto* x : {dyn, out, in}) std::fill(x, x + CFPQ_MAX_NONTERMINALS, int8_t{-1});
    bool heads[CFPQ_MAX_NONTERMINALS] = {};
    for (int32_t r = 0; r < gr->n_bin_rules; ++r) heads[gr->bin_rules[r].lhs] = true;
    for (int32_t a = 0; a < n_nt; ++a) {
        if (!heads[a]) continue;
        if (g.n_dyn == kSwMaxDyn) return false;
        dyn[a] = static_cast<int8_t>(g.n_dyn);
        g.dyn_nt[g.n_dyn++] = static_cast<uint8_t>(a);
    }
    // lists of a fixed nonterminal, made when a rule first needs them
    auto list = [&](int8_t (&of)[CFPQ_MAX_NONTERMINALS], int32_t a) {
        if (of[a] < 0 && g.n_list < kSwMaxLists) of[a] = static_cast<int8_t>(g.n_list++);
        return of[a];
    };
    bool fits = true;
    for (int32_t r = 0; r < gr->n_bin_rules; ++r) {
        const cfpq_bin_rule& br = gr->bin_rules[r];
        const bool lg = heads[br.left], rg = heads[br.right];  // growing operands
        SweepGrammar::Rule q;
        q.head = static_cast<uint8_t>(dyn[br.lhs]);
        const int8_t l = lg ? dyn[br.left] : list(out, br.left), rt = rg ? dyn[br.right] : list(out, br.right);
        fits = fits && l >= 0 && rt >= 0;
        q.left = static_cast<uint8_t>(l);
        q.right = static_cast<uint8_t>(rt);
        if (lg && rg) {
            g.dd[g.n_dd++] = q;
            g.dd_mask |= (1u << q.left) | (1u << q.right);
            g.p_mask |= 1u << q.head;
        } else if (rg) {
            g.lf[g.n_lf++] = q;
        } else if (lg) {
            const int8_t i = list(in, br.right);
            fits = fits && i >= 0;
            g.rf_in[g.n_rf] = static_cast<uint8_t>(i);
            g.rf[g.n_rf++] = q;
            g.rf_mask |= 1u << q.head;
        } else {
            g.ll[g.n_ll++] = q;
            g.ll_mask |= 1u << q.head;
        }
    }
    if (!fits) return false;
    for (int32_t r = 0; r < gr->n_term_rules; ++r) {
        const cfpq_term_rule& tr = gr->term_rules[r];
        bool seen = false;  // a rule given twice adds nothing
        for (int q = 0; q < g.n_term; ++q) seen = seen || (g.term[q].label == tr.terminal && g.term[q].nt == tr.lhs);
        if (seen) continue;
        g.term[g.n_term++] = {tr.terminal, static_cast<int16_t>(tr.lhs), out[tr.lhs], in[tr.lhs]};
        if (heads[tr.lhs]) g.init_mask |= 1u << dyn[tr.lhs];
    }
    *result = g;
    return true;
}

hipError_t launch_sweep_init(const SweepGrammar& g, const SweepBuffers& b, const Layout& L, const cfpq_edge* edges,
                             int64_t m, int32_t n_nt, int32_t n_terminals, hipStream_t s) {
    // bitmaps, the control block and the lists lie together from chg to cur
    const size_t tq = static_cast<size_t>(L.mat_words) * n_nt / 2;
    const size_t cq = static_cast<size_t>(reinterpret_cast<char*>(b.cur) - reinterpret_cast<char*>(b.chg)) / 16;
    const size_t blocks = std::min<size_t>((tq + cq + 1023) / 1024, 4096);
    sweep_clear_kernel<<<dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s>>>(
        reinterpret_cast<uint4*>(b.T), tq, reinterpret_cast<uint4*>(b.chg), cq);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    InitArgs a;
    std::copy(g.term, g.term + kSwMaxTerm, a.term);
    a.n_term = g.n_term;
    a.n = L.n;
    a.n_terminals = n_terminals;
    a.W = L.W;
    a.mat_words = L.mat_words;
    const dim3 eg(static_cast<unsigned>((m + 255) / 256));
    if (m > 0) sweep_scatter_kernel<<<eg, dim3(256), 0, s>>>(edges, m, a, b.T, b.list, b.ctl);
    if (g.n_list > 0) {
        // also without edges: the sweeps read every node's 16-byte form, written here
        const int32_t lists = g.n_list * L.n;
        HubArgs hubs{};
        hubs.n = L.n;
        hubs.longest = hub_list(L.W);
        for (int r = 0; sweep_hubs(L) && r < g.n_lf + g.n_rf; ++r) {
            const uint8_t l = r < g.n_lf ? g.lf[r].left : g.rf[r - g.n_lf].right;
            hubs.list[hubs.n_rules] = l;
            for (int q = 0; q < g.n_term; ++q)
                if (g.term[q].out == l) hubs.nt[hubs.n_rules] = static_cast<uint8_t>(g.term[q].nt);
            ++hubs.n_rules;
        }
        sweep_place_kernel<<<dim3(static_cast<unsigned>((lists + 255) / 256)), dim3(256), 0, s>>>(b.list, b.cur, b.near,
                                                                                                 lists, b.ctl, hubs);
        const int32_t longest = sweep_hubs(L) ? hub_list(L.W) : INT32_MAX;
        if (m > 0) sweep_fill_kernel<<<eg, dim3(256), 0, s>>>(edges, m, a, b.list, b.cur, b.near, b.idx, longest);
    }
    return hipGetLastError();
}

hipError_t launch_sweep(const SweepGrammar& g, const SweepBuffers& b, const Layout& L, int32_t t, uint32_t p_mask,
                        bool count, bool dense_dd, hipStream_t s) {
    SweepArgs a;
    a.g = g;
    a.T = b.T;
    a.Dprev = b.D[(t + 1) & 1];
    a.Dcur = b.D[t & 1];
    a.P = b.P;
    a.chg = b.chg;
    a.ctl = b.ctl;
    a.list = b.list;
    a.near = b.near;
    a.idx = b.idx;
    a.W = L.W;
    a.mat_words = L.mat_words;
    a.n = L.n;
    a.t = t;
    a.p_mask = p_mask;
    a.count = count ? 1 : 0;
    a.dense_dd = dense_dd ? 1 : 0;
    a.rows = sweep_rows(L.n);
    const int32_t groups = sweep_groups(L.n);
    a.wg_prev = b.wg + static_cast<size_t>((t + 1) & 1) * g.n_dyn * groups;
    a.wg_cur = b.wg + static_cast<size_t>(t & 1) * g.n_dyn * groups;
    const dim3 grid(static_cast<unsigned>(groups));
    const size_t lds = (static_cast<size_t>(64) * (L.W + 1) + static_cast<size_t>(g.n_dyn) * L.W) * 8;
    if (L.W <= 64) return t == 1 ? sweep_launch<1, true>(a, grid, lds, s) : sweep_launch<1, false>(a, grid, lds, s);
    if (L.W <= 128) return t == 1 ? sweep_launch<2, true>(a, grid, lds, s) : sweep_launch<2, false>(a, grid, lds, s);
    return t == 1 ? sweep_launch<4, true>(a, grid, lds, s) : sweep_launch<4, false>(a, grid, lds, s);
}

hipError_t launch_sweep_clean(const SweepGrammar& g, const SweepBuffers& b, const Layout& L, int32_t t, int h,
                              hipStream_t s) {
    const unsigned blocks = static_cast<unsigned>(std::min<int64_t>(L.npad / kWaves, kMaxBlocks));
    sweep_clean_kernel<<<dim3(blocks), dim3(256), 0, s>>>(
        b.D[(t + 1) & 1] + h * L.mat_words,
        b.chg + (static_cast<int64_t>((t - 1) & 3) * g.n_dyn + h) * L.W, L.W, L.npad);
    return hipGetLastError();
}

hipError_t launch_sweep_report(const SweepBuffers& b, int32_t t, SweepReport* report, hipStream_t s) {
    sweep_report_kernel<<<dim3(1), dim3(64), 0, s>>>(b.ctl, t, report);
    return hipGetLastError();
}

}  // namespace cfpq
