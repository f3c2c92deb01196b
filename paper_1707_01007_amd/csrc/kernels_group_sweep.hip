// Kernels of the group sweep (see group_sweep.h).
#include <algorithm>
#include <numeric>

#include "batch_engine.h"
#include "group_sweep.h"
#include "mfma_tile.h"
#include "near_list.h"

namespace cfpq {
namespace {

// ---- initialisation: grid (x, slot)

__global__ __launch_bounds__(256) void group_clear_kernel(const GroupSlot* __restrict__ slots) {
    const GroupSlot& d = slots[blockIdx.y];
    int64_t np = 0;
    for (int h = 0; h < d.g.n_dyn; ++h) np += d.g.p_slot[h] >= 0 ? 1 : 0;
    const int64_t tq = d.mat_words * d.n_nt / 2, pq = d.mat_words * np / 2;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
    const int64_t at = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    uint4* t = reinterpret_cast<uint4*>(d.T);
    uint4* p = reinterpret_cast<uint4*>(d.P);
    for (int64_t i = at; i < tq; i += stride) t[i] = make_uint4(0, 0, 0, 0);
    for (int64_t i = at; i < pq; i += stride) p[i] = make_uint4(0, 0, 0, 0);
    if (at == 0) *d.ctl = GroupCtl{};
}

// Grid (list, slot), one list a workgroup: lengths, places and entries from
// LDS counters; the workgroup after the last list sets the bits of Algorithm
// 1's matrix initialisation.  (With counters in global memory, one workgroup
// an instance took 228 us for 205 instances; this takes 89.)
__global__ __launch_bounds__(512) void group_lists_kernel(const GroupSlot* __restrict__ slots) {
    __shared__ SweepGrammar::Term term[kSwMaxTerm];
    __shared__ int32_t cnt[kGsMaxWords * 64], cur[kGsMaxWords * 64];
    __shared__ int32_t wave_tot[8], base_s;
    const GroupSlot& d = slots[blockIdx.y];
    const int x = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (x > d.g.n_list) return;
    const int32_t n = d.n, n_term = d.g.n_term;
    if (tid < n_term) term[tid] = d.g.term[tid];
    for (int32_t i = tid; i < n; i += 512) cnt[i] = 0;
    __syncthreads();
    auto ok = [&](const cfpq_edge& e) {
        return e.src >= 0 && e.src < n && e.dst >= 0 && e.dst < n && e.label >= 0 && e.label < d.n_terminals;
    };
    if (x == d.g.n_list) {
        for (int64_t e = tid; e < d.n_edges; e += 512) {
            const cfpq_edge ed = d.edges[e];
            if (!ok(ed)) {
                atomicAdd(&d.ctl->bad_edges, 1);
                continue;
            }
            const unsigned long long bit = 1ull << (ed.dst & 63);
            const int64_t off = static_cast<int64_t>(ed.src) * d.W + (ed.dst >> 6);
            for (int32_t q = 0; q < n_term; ++q)
                if (term[q].label == ed.label)
                    atomicOr(reinterpret_cast<unsigned long long*>(d.T + term[q].nt * d.mat_words + off), bit);
        }
        return;
    }
    for (int64_t e = tid; e < d.n_edges; e += 512) {
        const cfpq_edge ed = d.edges[e];
        if (!ok(ed)) continue;
        for (int32_t q = 0; q < n_term; ++q) {
            if (term[q].label != ed.label) continue;
            if (term[q].out == x) atomicAdd(&cnt[ed.src], 1);
            if (term[q].in == x) atomicAdd(&cnt[ed.dst], 1);
        }
    }
    __syncthreads();
    // exclusive sums, 512 nodes a round
    int32_t total = 0;
    for (int32_t i0 = 0; i0 < n; i0 += 512) {
        const int32_t c = i0 + tid < n ? cnt[i0 + tid] : 0;
        int32_t v = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t y = __shfl_up(v, o, 64);
            if (lane >= o) v += y;
        }
        if (lane == 63) wave_tot[wave] = v;
        __syncthreads();
        int32_t at = total + v - c;
        for (int w = 0; w < 8; ++w) {
            at += w < wave ? wave_tot[w] : 0;
            total += wave_tot[w];
        }
        if (i0 + tid < n) cur[i0 + tid] = at;
        __syncthreads();  // wave_tot is written again
    }
    if (tid == 0) base_s = atomicAdd(&d.ctl->list_top, total);
    __syncthreads();
    const int32_t base = base_s;
    int2* list = d.list + static_cast<int64_t>(x) * n;
    auto* near = reinterpret_cast<uint16_t*>(d.near + static_cast<int64_t>(x) * n);
    for (int32_t i = tid; i < n; i += 512) {
        list[i] = make_int2(base + cur[i], cnt[i]);
        d.near[static_cast<int64_t>(x) * n + i] = make_uint4(~0u, ~0u, ~0u, ~0u);
    }
    __syncthreads();
    // an entry: its place in idx, and in the node's first eight if it is one of them
    auto put = [&](int32_t i, int32_t start, int32_t k) {
        const int32_t at = atomicAdd(&cur[i], 1);
        d.idx[base + at] = k;
        put_near(near + 8 * i, at - start, cnt[i], k);
    };
    for (int64_t e = tid; e < d.n_edges; e += 512) {
        const cfpq_edge ed = d.edges[e];
        if (!ok(ed)) continue;
        for (int32_t q = 0; q < n_term; ++q) {
            if (term[q].label != ed.label) continue;
            if (term[q].out == x) put(ed.src, list[ed.src].x - base, ed.dst);
            if (term[q].in == x) put(ed.dst, list[ed.dst].x - base, ed.src);
        }
    }
}

// ---- a loop

__device__ __forceinline__ int head_of(uint32_t r) { return r & 255u; }
__device__ __forceinline__ int left_of(uint32_t r) { return (r >> 8) & 255u; }
__device__ __forceinline__ int right_of(uint32_t r) { return (r >> 16) & 255u; }
__device__ __forceinline__ int in_of(uint32_t r) { return r >> 24; }

// The instance's own number of the group's loop.
__device__ __forceinline__ int32_t own_loop(const GroupSlot& d, uint32_t loop) {
    return static_cast<int32_t>(loop - d.base);
}

// The change mask loop t starts from: before the first loop, what the edges set.
__device__ __forceinline__ uint32_t mask_before(const GroupSlot& d, int32_t t) {
    return t == 1 ? d.g.init_mask : d.ctl->any[(t - 1) & 3];
}

// Transposes of the dd rules' right operands that changed (all of them before
// the first loop: no product reads one that was never made); a wavefront a
// 256 x 256 tile.
__global__ __launch_bounds__(256) void group_transpose_kernel(const GroupSlot* __restrict__ slots,
                                                              const int32_t* __restrict__ map, int32_t count,
                                                              uint32_t loop) {
    const int32_t item = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    if (item >= count) return;
    const int32_t m = map[item];
    const GroupSlot& d = slots[m >> 16];
    const int c = (m >> 8) & 255;
    const int32_t t = own_loop(d, loop);
    if (t > d.max_iters || (t > 1 && !((mask_before(d, t) >> c) & 1u))) return;
    const int64_t br0 = ((m >> 4) & 15) * 4, bc0 = (m & 15) * 4;
    const int lane = threadIdx.x & 63;
    uint64_t* dst = d.TT + d.g.tt_slot[c] * d.mat_words;
    uint64_t x[4][4];
    load_transpose256(d.T + d.g.dyn_nt[c] * d.mat_words, d.W, br0, bc0, lane, x);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        ulonglong2* o = reinterpret_cast<ulonglong2*>(dst + ((bc0 + q) * 64 + lane) * d.W + br0);
        o[0] = make_ulonglong2(x[q][0], x[q][1]);
        o[1] = make_ulonglong2(x[q][2], x[q][3]);
    }
}

// P |= T_B x T_C of a dd rule with a changed operand, a 256 x 256 tile a
// workgroup (eight wavefronts of 64 x 128, two a SIMD: the few chunks of these
// products are latency that the other wavefront hides).
__global__ __launch_bounds__(512) void group_product_kernel(const GroupSlot* __restrict__ slots,
                                                            const int32_t* __restrict__ map, uint32_t loop) {
    const int32_t m = map[blockIdx.x];
    const GroupSlot& d = slots[m >> 16];
    const int32_t t = own_loop(d, loop);
    const uint32_t rule = d.g.rule[d.g.n_lf + d.g.n_rf + d.g.n_ll + ((m >> 8) & 255)];
    const uint32_t before = mask_before(d, t);
    if (t > d.max_iters || !(((before >> left_of(rule)) | (before >> right_of(rule))) & 1u)) return;
    const int wave = threadIdx.x >> 6;
    mfma::mfma4_wave_tile<true, 2, 2>(
        reinterpret_cast<const uint32_t*>(d.T + d.g.dyn_nt[left_of(rule)] * d.mat_words),
        reinterpret_cast<const uint32_t*>(d.TT + d.g.tt_slot[right_of(rule)] * d.mat_words),
        reinterpret_cast<uint32_t*>(d.P + d.g.p_slot[head_of(rule)] * d.mat_words), 2 * d.W, (d.n + 255) / 256,
        ((m >> 4) & 15) * 256 + (wave >> 1) * 64, (m & 15) * 256 + (wave & 1) * 128,
        &d.ctl->spare);  // the sweep finds what changed
}


// Bits a row, on average, from which the turned scatter is taken.
constexpr int32_t kTurnBits = 8;
constexpr uint32_t kPull = kGsPull;  // rows a row of a head pulls from LDS
constexpr int32_t kLongPull = 64;  // entries a row's lanes walk themselves in a pull

struct GroupShared {
    unsigned long long rows[kSwMaxDyn];  // this loop's changed rows
    unsigned long long act[kSwMaxDyn];   // rows with something to pull
    unsigned long long lng;              // rows with a list past kLongPull
    uint32_t gained[kSwMaxDyn];
    uint32_t any;
};

// Loop t of 64 rows of one instance, LPR lanes a row (rows of at most LPR
// words), as in sweep_kernel: pulls, then scatters, each row written by this
// workgroup alone.  Which rows pull at all is found first, a lane a row.
template <int LPR, bool kFirst>
__device__ __forceinline__ void group_rows(const GroupSlot& d, int32_t t, int32_t grp, uint32_t before, uint64_t* buf,
                                           GroupShared& sh) {
    constexpr int kRpw = 64 / LPR, kStep = 4 * kRpw;  // rows at once of a wavefront, of the workgroup
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int sub = lane / LPR, sl = lane % LPR;
    const int W = d.W, stride = W + 1, n_dyn = d.g.n_dyn;
    const bool valid = sl < W;
    const int off = valid ? sl : W - 1;
    const int32_t row0 = grp * kGsRows;
    const int32_t nrows = min(kGsRows, d.n - row0);
    const uint64_t all_rows = nrows == 64 ? ~0ull : (1ull << nrows) - 1;
    const uint64_t* Dprev = d.D[(t + 1) & 1];
    uint64_t* Dcur = d.D[t & 1];
    uint64_t* marks = buf + kGsRows * stride;  // the last loop's changed rows, [n_dyn][W]
    const int32_t n_lf = d.g.n_lf, n_rf = d.g.n_rf, n_ll = d.g.n_ll;
    const uint32_t* lf = d.g.rule;
    const uint32_t* rf = lf + n_lf;
    const uint32_t* llr = rf + n_rf;
    const uint32_t* dd = llr + n_ll;
    const int2* __restrict__ list = d.list;
    const uint4* __restrict__ near = d.near;
    const int32_t* __restrict__ idx = d.idx;
    // what each row of a head pulls: up to kPull rows, dyn << 12 | row
    auto* pulls = reinterpret_cast<uint16_t*>(marks + n_dyn * W);     // [n_dyn][64][kPull]
    auto* n_pull = reinterpret_cast<uint32_t*>(pulls + n_dyn * 64 * kPull);  // [n_dyn][64], the true count
    if (!kFirst) {
        const uint64_t* chg_prev = d.chg + static_cast<int64_t>((t + 1) & 1) * n_dyn * W;
        for (int x = threadIdx.x; x < n_dyn * W; x += 256) marks[x] = chg_prev[x];
    }
    for (int x = threadIdx.x; x < n_dyn * 64; x += 256) n_pull[x] = 0;
    if (threadIdx.x < kSwMaxDyn) {
        sh.rows[threadIdx.x] = 0;
        sh.act[threadIdx.x] = 0;
        sh.gained[threadIdx.x] = 0;
    }
    if (threadIdx.x == 0) {
        sh.lng = 0;
        sh.any = 0;
    }
    __syncthreads();
    auto T_row = [&](int h, int lr) { return d.T + d.g.dyn_nt[h] * d.mat_words + static_cast<int64_t>(row0 + lr) * W; };
    auto live = [&](int c, int32_t k) { return kFirst || ((marks[c * W + (k >> 6)] >> (k & 63)) & 1ull) != 0; };
    auto source = [&](int c) { return kFirst ? d.T + d.g.dyn_nt[c] * d.mat_words : Dprev + c * d.mat_words; };

    // ---- rows that pull, and what: a lane a row, the rules spread over the wavefronts
    for (int r = wave; r < n_lf; r += 4) {
        const uint32_t q = lf[r];
        const int c = right_of(q), h = head_of(q);
        if (!((before >> c) & 1u)) continue;
        bool act = false, lng = false;
        if (lane < nrows) {
            const int64_t i = static_cast<int64_t>(left_of(q)) * d.n + row0 + lane;
            const uint4 v = near[i];
            uint32_t k[8], m = 0;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                k[u] = entry(v, u);
                if (k[u] < kMore && live(c, static_cast<int32_t>(k[u]))) m |= 1u << u;
            }
            uint32_t* count = n_pull + h * 64 + lane;
            if (has_more(v)) {
                const int2 l = list[i];
                lng = l.y > kLongPull;
                act = lng;
                if (!lng)
                    for (int32_t e = 0; e < l.y; ++e) act = act || live(c, idx[l.x + e]);
                if (act) atomicAdd(count, static_cast<uint32_t>(kPull + 1));  // taken from the lists
            } else if (m != 0) {
                act = true;
                uint32_t at = atomicAdd(count, static_cast<uint32_t>(__popc(m)));
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if ((m >> u) & 1u) {
                        if (at < kPull) pulls[(h * 64 + lane) * kPull + at] = static_cast<uint16_t>(c << 12 | k[u]);
                        ++at;
                    }
            }
        }
        const uint64_t am = __ballot(act), lm = __ballot(lng);
        if (lane == 0 && am != 0) atomicOr(&sh.act[h], static_cast<unsigned long long>(am));
        if (lane == 0 && lm != 0) atomicOr(&sh.lng, static_cast<unsigned long long>(lm));
    }
    __syncthreads();

    // New bits nw of row lr of head h (every lane of the wavefront takes part,
    // `on` where its row does): those T lacks are stored, kept as D's row and marked.
    auto commit = [&](int h, int lr, bool on, uint64_t nw, uint64_t told) {
        uint64_t* trow = T_row(h, lr);
        nw = on && valid ? nw & ~told : 0;
        const uint64_t b = __ballot(nw != 0);
        if (b == 0) return;
        const uint64_t mine = LPR == 64 ? b : b >> (sub * LPR) & ((1ull << (LPR & 63)) - 1);
        const bool again = (sh.rows[h] >> lr) & 1ull;
        int c = __popcll(nw);
#pragma unroll
        for (int o = LPR / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
        if (mine == 0) return;
        if (valid) {
            uint64_t* drow = Dcur + h * d.mat_words + static_cast<int64_t>(row0 + lr) * W;
            if (nw != 0) trow[off] = told | nw;
            drow[off] = again ? drow[off] | nw : nw;
        }
        if (sl == 0) {
            atomicOr(&sh.rows[h], 1ull << lr);
            atomicAdd(&sh.gained[h], static_cast<uint32_t>(c));
        }
    };

    // Row lr of head h from its lists themselves (more entries than `pulls` holds).
    auto walk_lists = [&](int h, int lr) -> uint64_t {
        uint64_t acc = 0;
        for (int r = 0; r < n_lf; ++r) {
            const uint32_t q = lf[r];
            const int c = right_of(q);
            if (head_of(q) != h || !((before >> c) & 1u)) continue;
            const int2 l = list[left_of(q) * d.n + row0 + lr];
            const uint64_t* src = source(c);
            for (int32_t e = 0; e < l.y; e += 4) {
                int32_t k[4];
                uint64_t v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) k[u] = idx[l.x + min(e + u, l.y - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = live(c, k[u]) ? src[static_cast<int64_t>(k[u]) * W + off] : 0;
#pragma unroll
                for (int u = 0; u < 4; ++u) acc |= v[u];
            }
        }
        return acc;
    };

    // ---- 1. pulls
    for (int h = 0; h < n_dyn; ++h) {
        bool has_p = false;
        for (int r = 0; r < d.g.n_dd; ++r)
            has_p = has_p || (head_of(dd[r]) == h && (((before >> left_of(dd[r])) | (before >> right_of(dd[r]))) & 1u));
        const uint64_t act = (sh.act[h] & ~sh.lng) | (has_p ? all_rows : 0);
        if (act == 0) continue;
#pragma unroll 1
        for (int st = 0; st < kGsRows; st += kStep) {
            const int lr = st + wave * kRpw + sub;
            const bool on = (act >> lr) & 1ull;
            if (__ballot(on) == 0) continue;
            uint64_t acc = 0, told = 0;
            uint32_t count = 0;
            if (on) {
                told = T_row(h, lr)[off];  // in flight with the rows pulled
                if (has_p) acc = d.P[d.g.p_slot[h] * d.mat_words + static_cast<int64_t>(row0 + lr) * W + off];
                count = n_pull[h * 64 + lr];
            }
            // a longer list is walked itself, or (past kLongPull) by the whole workgroup, below
            if (count > kPull) acc |= (sh.lng >> lr) & 1ull ? 0 : walk_lists(h, lr);
            const uint16_t* from = pulls + (h * 64 + lr) * kPull;
            for (uint32_t e = 0; count <= kPull && e < count; e += 2) {
                uint64_t v[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint32_t x = from[min(e + u, count - 1)];
                    v[u] = source(x >> 12)[static_cast<int64_t>(x & 4095u) * W + off];
                }
                acc |= v[0] | v[1];
            }
            commit(h, lr, on, acc, told);
        }
    }
    __syncthreads();
    for (uint64_t lm = sh.lng; lm != 0; lm &= lm - 1) {  // uniform over the workgroup
        const int lr = __ffsll(static_cast<unsigned long long>(lm)) - 1;
        for (int h = 0; h < n_dyn; ++h) {
            if (!((sh.act[h] >> lr) & 1ull)) continue;
            for (int w = threadIdx.x; w < W; w += 256) buf[w] = 0;
            __syncthreads();
            uint64_t acc = 0;
            for (int r = 0; r < n_lf; ++r) {
                const uint32_t q = lf[r];
                const int c = right_of(q);
                if (head_of(q) != h || !((before >> c) & 1u)) continue;
                const int2 l = list[left_of(q) * d.n + row0 + lr];
                const uint64_t* src = source(c);
                for (int32_t e = wave * kRpw + sub; e < l.y; e += kStep) {
                    const int32_t k = idx[l.x + e];
                    if (live(c, k)) acc |= src[static_cast<int64_t>(k) * W + off];
                }
            }
            if (valid && acc != 0)
                atomicOr(reinterpret_cast<unsigned long long*>(buf + off), static_cast<unsigned long long>(acc));
            __syncthreads();
            if (wave == 0) commit(h, lr, sub == 0, buf[off], sub == 0 ? T_row(h, lr)[off] : 0);
            __syncthreads();
        }
    }

    // ---- 2. scatters, a target at a time.  The first loop scatters the bits of
    // the edges; an operand that is no scatter's target feeds the bits its
    // pulls just gained (in the second loop the first one's as well, which come
    // from the ll rules), the others the last loop's.
    auto late = [&](int h) { return ((d.g.rf_mask >> h) & 1u) != 0; };
    auto from_prev = [&](int h) { return !kFirst && (late(h) || t == 2); };
    auto feed_rows = [&](int h) -> uint64_t {
        if (kFirst) return (d.g.init_mask >> h) & 1u ? all_rows : 0;
        return (late(h) ? 0 : sh.rows[h]) | (from_prev(h) ? marks[h * W + grp] & all_rows : 0);
    };
    auto feed_word = [&](int h, int lr) -> uint64_t {
        const int64_t at = h * d.mat_words + static_cast<int64_t>(row0 + lr) * W + off;
        if (kFirst) return T_row(h, lr)[off];
        uint64_t f = 0;
        if (!late(h) && ((sh.rows[h] >> lr) & 1ull)) f = Dcur[at];
        if (from_prev(h) && ((marks[h * W + grp] >> lr) & 1ull)) f |= Dprev[at];
        return f;
    };
    const int32_t* wg_prev = d.wg + static_cast<int64_t>((t + 1) & 1) * n_dyn * d.groups;
    int32_t* wg_cur = d.wg + static_cast<int64_t>(t & 1) * n_dyn * d.groups;
    const uint32_t targets = d.g.rf_mask | (kFirst ? d.g.ll_mask : 0);
    for (int th = 0; th < n_dyn; ++th) {
        if (!((targets >> th) & 1u)) continue;
        uint64_t fed = 0;
        bool many = false;
        __syncthreads();  // the rows and counts of the heads before th are final, buf is free
        for (int r = 0; r < n_rf; ++r) {
            if (head_of(rf[r]) != th) continue;
            const int h = left_of(rf[r]);
            const uint64_t m = feed_rows(h);
            fed |= m;
            if (kFirst) continue;
            uint32_t bits = late(h) ? 0 : sh.gained[h];
            if (from_prev(h) && marks[h * W + grp] != 0) bits += wg_prev[h * d.groups + grp];
            many = many || bits > static_cast<uint32_t>(kTurnBits * nrows);
        }
        if (kFirst)
            for (int r = 0; r < n_ll; ++r)
                if (head_of(llr[r]) == th) fed = all_rows;
        if (fed == 0) continue;
        __syncthreads();  // every wavefront has read the counts above
        if (!many) {
#pragma unroll 1
            for (int st = 0; st < kGsRows; st += kStep) {
                const int lr = st + wave * kRpw + sub;
                const bool on = (fed >> lr) & 1ull;
                if (__ballot(on) == 0) continue;
                if (valid) buf[lr * stride + off] = 0;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                uint32_t* lds = reinterpret_cast<uint32_t*>(buf);
                const int32_t x = lr * stride * 2;
                for (int r = 0; r < n_rf; ++r) {
                    if (head_of(rf[r]) != th) continue;
                    const int h = left_of(rf[r]);
                    const bool fr = valid && ((feed_rows(h) >> lr) & 1ull);
                    const uint64_t f = fr ? feed_word(h, lr) : 0;
                    scatter_word(f, static_cast<int64_t>(right_of(rf[r])) * d.n + sl * 64, near, list, idx, lds, x,
                                 lane);
                }
                if (kFirst) {
                    // A -> B C with both fixed: the edges k -> j of C for the edges row -> k of B
                    for (int r = 0; r < n_ll; ++r) {
                        if (head_of(llr[r]) != th) continue;
                        const int64_t lb = static_cast<int64_t>(left_of(llr[r])) * d.n + row0 + lr;
                        const int64_t cb = static_cast<int64_t>(right_of(llr[r])) * d.n;
                        const int2 l = on ? list[lb] : make_int2(0, 0);
                        for (int32_t b = sl; __ballot(b < l.y) != 0; b += LPR) {
                            const bool have = b < l.y;
                            const int64_t k = cb + (have ? idx[l.x + b] : 0);
                            const uint4 v = have ? near[k] : make_uint4(~0u, ~0u, ~0u, ~0u);
                            scatter_list(v, have, k, list, idx, lds, x, lane);
                        }
                    }
                }
                // every scatter of this wavefront has reached LDS before its rows are read
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                commit(th, lr, on, buf[lr * stride + off], on ? T_row(th, lr)[off] : 0);
            }
            continue;
        }
        // turned: this wavefront's columns are the 64-column words wave, wave + 4, ...
        uint64_t acc[LPR / 4];
#pragma unroll
        for (int i = 0; i < LPR / 4; ++i) acc[i] = 0;
        for (int r = 0; r < n_rf; ++r) {
            if (head_of(rf[r]) != th) continue;
            const int h = left_of(rf[r]);
            const uint64_t m = feed_rows(h);
            if (m == 0) continue;
            __syncthreads();  // buf is free
#pragma unroll 1
            for (int st = 0; st < kGsRows; st += kStep) {
                const int lr = st + wave * kRpw + sub;
                if (valid) buf[lr * stride + off] = (m >> lr) & 1ull ? feed_word(h, lr) : 0;
            }
            __syncthreads();
            for (int c = wave; c < W; c += 4) {
                uint64_t x = buf[lane * stride + c];
                if (__ballot(x != 0) != 0) x = transpose64(x, lane);
                buf[lane * stride + c] = x;
            }
            __syncthreads();
            const int64_t in = static_cast<int64_t>(in_of(rf[r])) * d.n;
#pragma unroll
            for (int i = 0; i < LPR / 4; ++i) {
                const int32_t j = (wave + 4 * i) * 64 + lane;
                acc[i] |= gather_words(buf, stride, lane, j < d.n, in + j, near, list, idx);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();  // every read of the turned operands is done
#pragma unroll
        for (int i = 0; i < LPR / 4; ++i) {
            const int c = wave + 4 * i;
            if (c >= W) break;  // uniform over the wavefront
            uint64_t x = acc[i];
            if (__ballot(x != 0) != 0) x = transpose64(x, lane);
            buf[lane * stride + c] = x;
        }
        __syncthreads();
#pragma unroll 1
        for (int st = 0; st < kGsRows; st += kStep) {
            const int lr = st + wave * kRpw + sub;
            const bool on = lr < nrows;
            commit(th, lr, on, buf[lr * stride + off], on ? T_row(th, lr)[off] : 0);
        }
    }
    __syncthreads();
    if (threadIdx.x < n_dyn) {
        const int h = threadIdx.x;
        const unsigned long long m = sh.rows[h];
        d.chg[(static_cast<int64_t>(t & 1) * n_dyn + h) * W + grp] = m;
        if (m != 0) {
            wg_cur[h * d.groups + grp] = static_cast<int32_t>(sh.gained[h]);
            atomicOr(&sh.any, 1u << h);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && sh.any != 0) {
        uint32_t* any = &d.ctl->any[t & 3];
        const uint32_t have = __hip_atomic_load(any, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((sh.any & ~have) != 0) atomicOr(any, sh.any);
    }
}

// One loop of every running instance, 64 rows a workgroup.
//
// What bounds it: latency.  A dense loop of the 512-instance batch (205
// instances of 513 to 2048 nodes here) reads 65 and writes 100 MB and issues
// 29 M vector instructions, some 50 us of either, and takes 100 to 130; a
// wavefront waits two thirds of its time, on chains of a list, the rows it
// names and T.  5 to 8 wavefronts a SIMD and 2 to 16 bits a row for the turned
// scatter measured within 3% of each other; instances in falling size, spread
// over the XCDs by words, took a fifth off the loops (59 -> 48 us on average).
//
// kWide: the instances with rows of more than 32 words, in a launch of their
// own: their sixteen columns a lane of the turned scatter take half the
// wavefronts' registers.
template <bool kFirst, bool kWide>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kWide ? 3 : 6))) void group_sweep_kernel(const GroupSlot* __restrict__ slots,
                                                          const int32_t* __restrict__ map, uint32_t loop) {
    extern __shared__ __align__(16) uint64_t buf[];
    __shared__ GroupShared sh;
    const int32_t m = map[blockIdx.x];
    if (m < 0) return;
    const GroupSlot& d = slots[m >> 16];
    const int32_t grp = m & 0xFFFF;
    const int32_t t = own_loop(d, loop);
    GroupCtl* ctl = d.ctl;
    const uint32_t before = mask_before(d, t);
    const bool run = (kFirst || before != 0) && t <= d.max_iters;
    if (grp == 0 && threadIdx.x == 0) {
        ctl->any[(t + 1) & 3] = 0;
        if (run) {
            // rules this loop runs: an operand changed in the last one
            int32_t c = kFirst ? d.g.n_ll : 0;
            const int32_t n_lr = d.g.n_lf + d.g.n_rf;
            for (int r = 0; r < n_lr; ++r) {
                const uint32_t q = d.g.rule[r];
                c += (before >> (r < d.g.n_lf ? right_of(q) : left_of(q))) & 1u;
            }
            int32_t dense = 0;
            for (int r = n_lr + d.g.n_ll; r < n_lr + d.g.n_ll + d.g.n_dd; ++r)
                dense += ((before >> left_of(d.g.rule[r])) | (before >> right_of(d.g.rule[r]))) & 1u;
            ctl->loops = t;
            ctl->products += c + dense;
            ctl->dense += dense;
        } else if (before != 0) {
            ctl->capped = 1;
        }
    }
    if (!run) return;
    if (kWide)
        group_rows<64, kFirst>(d, t, grp, before, buf, sh);
    else if (d.W <= 16)
        group_rows<16, kFirst>(d, t, grp, before, buf, sh);
    else
        group_rows<32, kFirst>(d, t, grp, before, buf, sh);
}

template <bool kWide>
hipError_t sweep_launch(const GroupSlot* slots, const int32_t* map, int32_t blocks, uint32_t loop, bool first,
                        size_t lds, hipStream_t s) {
    if (blocks == 0) return hipSuccess;
    const dim3 grid(static_cast<unsigned>(blocks));
    if (first)
        group_sweep_kernel<true, kWide><<<grid, dim3(256), lds, s>>>(slots, map, loop);
    else
        group_sweep_kernel<false, kWide><<<grid, dim3(256), lds, s>>>(slots, map, loop);
    return hipGetLastError();
}

// One workgroup: how many instances changed in loop t.
__global__ __launch_bounds__(256) void group_report_kernel(const GroupSlot* __restrict__ slots, int32_t count,
                                                           uint32_t loop, GroupReport* out) {
    __shared__ int32_t run_s, dd_s;
    if (threadIdx.x == 0) run_s = dd_s = 0;
    __syncthreads();
    int32_t run = 0, dd = 0;
    for (int32_t i = threadIdx.x; i < count; i += 256) {
        const bool on = slots[i].ctl->any[own_loop(slots[i], loop) & 3] != 0;
        run += on ? 1 : 0;
        dd += on && slots[i].g.n_dd > 0 ? 1 : 0;
    }
    if (run != 0) atomicAdd(&run_s, run);
    if (dd != 0) atomicAdd(&dd_s, dd);
    __syncthreads();
    if (threadIdx.x != 0) return;
    out->running = run_s;
    out->running_dd = dd_s;
    __threadfence_system();
    __hip_atomic_store(&out->loop, static_cast<int32_t>(loop), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(64) void group_finish_kernel(const GroupSlot* __restrict__ slots, int32_t count,
                                                          uint32_t loop, SlotState* states) {
    const int32_t i = blockIdx.x * 64 + threadIdx.x;
    if (i >= count) return;
    const GroupCtl& c = *slots[i].ctl;
    SlotState& st = states[slots[i].slot];
    st.iterations = c.loops;
    st.products = c.products;
    st.dense = c.dense;
    st.capped = c.capped;
    st.bad_edges = c.bad_edges;
    st.done = c.any[own_loop(slots[i], loop) & 3] == 0 ? 1 : 0;
    st.active = 1 - st.done;
}

}  // namespace

bool group_grammar(const cfpq_grammar* gr, int32_t n_nodes, int64_t n_edges, GroupGrammar* out) {
    const Layout L = layout_for(n_nodes);
    if (n_nodes <= 0 || L.npad <= kSmallMaxPad || L.W > kGsMaxWords || n_edges > sweep_max_edges(L)) return false;
    SweepGrammar sg;
    if (!sweep_grammar(gr, &sg)) return false;
    // With several products a loop they decide, and the tile engine takes fewer
    // loops (27 against 21): eight instances of 3000 nodes and two products,
    // us there and here, at 1 edge a node 6367, 4268, at 2.5 16662, 16281, at 4
    // 6526, 7251; of 2048 nodes and 4 edges a node 3309, 3004.
    if (sg.n_dd > 1 && L.W > 32 && n_edges > 2 * static_cast<int64_t>(n_nodes)) return false;
    GroupGrammar g{};
    g.n_dyn = sg.n_dyn;
    g.n_list = sg.n_list;
    g.n_lf = sg.n_lf;
    g.n_rf = sg.n_rf;
    g.n_ll = sg.n_ll;
    g.n_dd = sg.n_dd;
    g.n_term = sg.n_term;
    g.rf_mask = sg.rf_mask;
    g.ll_mask = sg.ll_mask;
    g.init_mask = sg.init_mask;
    int32_t k = 0;
    auto put = [&](const SweepGrammar::Rule& r, uint32_t in) {
        g.rule[k++] = r.head | static_cast<uint32_t>(r.left) << 8 | static_cast<uint32_t>(r.right) << 16 | in << 24;
    };
    for (int r = 0; r < sg.n_lf; ++r) put(sg.lf[r], 0);
    for (int r = 0; r < sg.n_rf; ++r) put(sg.rf[r], sg.rf_in[r]);
    for (int r = 0; r < sg.n_ll; ++r) put(sg.ll[r], 0);
    for (int r = 0; r < sg.n_dd; ++r) put(sg.dd[r], 0);
    std::fill(g.p_slot, g.p_slot + kSwMaxDyn, -1);
    std::fill(g.tt_slot, g.tt_slot + kSwMaxDyn, -1);
    int32_t np = 0, nt = 0;
    for (int r = 0; r < sg.n_dd; ++r) {
        if (g.p_slot[sg.dd[r].head] < 0) g.p_slot[sg.dd[r].head] = np++;
        if (g.tt_slot[sg.dd[r].right] < 0) g.tt_slot[sg.dd[r].right] = nt++;
    }
    for (int h = 0; h < sg.n_dyn; ++h) g.dyn_nt[h] = sg.dyn_nt[h];
    std::copy(sg.term, sg.term + kSwMaxTerm, g.term);
    *out = g;
    return true;
}

GroupSlot group_slot(const GroupGrammar& g, int32_t n_nodes) {
    const Layout L = layout_for(n_nodes);
    GroupSlot d{};
    d.g = g;
    d.mat_words = L.mat_words;
    d.n = n_nodes;
    d.W = static_cast<int32_t>(L.W);
    d.groups = (n_nodes + kGsRows - 1) / kGsRows;
    return d;
}

size_t group_layout(const GroupGrammar& g, int32_t n_nodes, char* ws, GroupSlot* d) {
    const Layout L = layout_for(n_nodes);
    const size_t mat = static_cast<size_t>(L.mat_words) * 8;
    const int32_t groups = (n_nodes + kGsRows - 1) / kGsRows;
    int32_t np = 0, nt = 0, per_edge = 1;
    for (int h = 0; h < g.n_dyn; ++h) {
        np += g.p_slot[h] >= 0 ? 1 : 0;
        nt += g.tt_slot[h] >= 0 ? 1 : 0;
    }
    // an edge enters the lists of its label's (distinct) terminal rules
    for (int32_t q = 0; q < g.n_term; ++q) {
        int32_t c = 0;
        for (int32_t r = 0; r < g.n_term; ++r)
            if (g.term[r].label == g.term[q].label) c += (g.term[r].out >= 0 ? 1 : 0) + (g.term[r].in >= 0 ? 1 : 0);
        per_edge = std::max(per_edge, c);
    }
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align_up(bytes, 256);
        return at;
    };
    const size_t lists = static_cast<size_t>(g.n_list) * n_nodes;
    const size_t d0 = take(mat * g.n_dyn), d1 = take(mat * g.n_dyn), p = take(mat * np), tt = take(mat * nt);
    const size_t chg = take(static_cast<size_t>(2) * g.n_dyn * L.W * 8);
    const size_t ctl = take(sizeof(GroupCtl));
    const size_t wg = take(static_cast<size_t>(2) * g.n_dyn * groups * 4);
    const size_t list = take(lists * 8), near = take(lists * 16);
    const size_t idx = take(static_cast<size_t>(sweep_max_edges(L)) * per_edge * 4);
    if (ws != nullptr) {
        d->D[0] = reinterpret_cast<uint64_t*>(ws + d0);
        d->D[1] = reinterpret_cast<uint64_t*>(ws + d1);
        d->P = reinterpret_cast<uint64_t*>(ws + p);
        d->TT = reinterpret_cast<uint64_t*>(ws + tt);
        d->chg = reinterpret_cast<uint64_t*>(ws + chg);
        d->ctl = reinterpret_cast<GroupCtl*>(ws + ctl);
        d->wg = reinterpret_cast<int32_t*>(ws + wg);
        d->list = reinterpret_cast<int2*>(ws + list);
        d->near = reinterpret_cast<uint4*>(ws + near);
        d->idx = reinterpret_cast<int32_t*>(ws + idx);
    }
    return off;
}

hipError_t group_init(const GroupSlot* slots, int32_t count, int32_t max_lists, hipStream_t s) {
    group_clear_kernel<<<dim3(16, static_cast<unsigned>(count)), dim3(256), 0, s>>>(slots);
    group_lists_kernel<<<dim3(static_cast<unsigned>(max_lists + 1), static_cast<unsigned>(count)), dim3(512), 0, s>>>(
        slots);
    return hipGetLastError();
}

hipError_t group_loop(const GroupSlot* slots, const GroupMaps& m, uint32_t loop, bool first, bool with_dd,
                      hipStream_t s) {
    if (with_dd && m.n_tiles > 0) {
        group_transpose_kernel<<<dim3(static_cast<unsigned>((m.n_trans + 3) / 4)), dim3(256), 0, s>>>(slots, m.trans,
                                                                                                    m.n_trans, loop);
        group_product_kernel<<<dim3(static_cast<unsigned>(m.n_tiles)), dim3(512), 0, s>>>(slots, m.tiles, loop);
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = sweep_launch<false>(slots, m.rows[0], m.n_rows[0], loop, first, m.lds[0], s);
    if (e == hipSuccess) e = sweep_launch<true>(slots, m.rows[1], m.n_rows[1], loop, first, m.lds[1], s);
    return e;
}

hipError_t group_report(const GroupSlot* slots, int32_t count, uint32_t loop, GroupReport* out, hipStream_t s) {
    group_report_kernel<<<dim3(1), dim3(256), 0, s>>>(slots, count, loop, out);
    return hipGetLastError();
}

hipError_t group_finish(const GroupSlot* slots, int32_t count, uint32_t loop, SlotState* states, hipStream_t s) {
    group_finish_kernel<<<dim3(static_cast<unsigned>((count + 63) / 64)), dim3(64), 0, s>>>(slots, count, loop,
                                                                                         states);
    return hipGetLastError();
}

void GroupLists::add(const GroupSlot* slots, int32_t begin, int32_t end) {
    constexpr int kXcds = 8;
    std::vector<int32_t> order(end - begin);
    std::iota(order.begin(), order.end(), begin);
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return slots[a].W > slots[b].W; });
    for (int wide = 0; wide < 2; ++wide) {
        std::vector<int32_t> per[kXcds];
        int64_t words[kXcds] = {};
        lds[wide] = 0;
        for (int32_t k : order) {
            const GroupSlot& d = slots[k];
            if ((d.W > 32) != (wide == 1)) continue;
            const auto x = std::min_element(words, words + kXcds) - words;
            words[x] += static_cast<int64_t>(d.n) * d.W;
            for (int32_t r = 0; r < d.groups; ++r) per[x].push_back(k << 16 | r);
            lds[wide] = std::max(lds[wide], group_lds(d.W, d.g.n_dyn));
        }
        size_t most = 0;
        for (const auto& v : per) most = std::max(most, v.size());
        rows[wide].assign(most * kXcds, -1);
        for (int x = 0; x < kXcds; ++x)
            for (size_t q = 0; q < per[x].size(); ++q) rows[wide][q * kXcds + x] = per[x][q];
    }
    tiles.clear();
    trans.clear();
    for (int32_t k : order) {
        const GroupGrammar& g = slots[k].g;
        const int32_t side = slots[k].W / 4;
        for (int32_t ij = 0; g.n_dd > 0 && ij < side * side; ++ij) {
            const int32_t tile = (ij / side) << 4 | (ij % side);
            for (int32_t r = 0; r < g.n_dd; ++r) tiles.push_back(k << 16 | r << 8 | tile);
            for (int32_t c = 0; c < g.n_dyn; ++c)
                if (g.tt_slot[c] >= 0) trans.push_back(k << 16 | c << 8 | tile);
        }
    }
}

size_t GroupLists::put(int32_t* host, const int32_t* device, GroupMaps* m) const {
    size_t at = 0;
    auto list = [&](const std::vector<int32_t>& v, const int32_t** where, int32_t* count) {
        std::copy(v.begin(), v.end(), host + at);
        *where = device + at;
        *count = static_cast<int32_t>(v.size());
        at += v.size();
    };
    for (int wide = 0; wide < 2; ++wide) {
        list(rows[wide], &m->rows[wide], &m->n_rows[wide]);
        m->lds[wide] = lds[wide];
    }
    list(tiles, &m->tiles, &m->n_tiles);
    list(trans, &m->trans, &m->n_trans);
    return at;
}

}  // namespace cfpq
