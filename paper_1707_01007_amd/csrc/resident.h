// The resident sweep: the whole in-place fixpoint of a small graph in one
// workgroup and its LDS (kernels_resident.hip).
#pragma once

#include <cstddef>
#include <cstdint>
#include <cstring>

#include "batch_engine.h"

namespace cfpq {

constexpr int kRsMaxRules = 5;   // rules per kind, packed in one scalar register pair
constexpr int kRsMaxDyn = 8;     // nonterminals that head a binary rule
constexpr int kRsMaxLists = 16;  // adjacency lists of fixed operands, outgoing and incoming
constexpr int kRsMaxBin = 4 * kRsMaxRules;
constexpr int kRsMaxTerm = 12;   // terminal rules kept beside the grammar

// A rule of a kind: head | left << 3 | right << 7, rule r at bit 11 r -- growing
// nonterminals by their number, fixed operands by their list.
__host__ __device__ inline int rs_head(uint64_t kind, int r) { return static_cast<int>(kind >> (11 * r)) & 7; }
__host__ __device__ inline int rs_left(uint64_t kind, int r) { return static_cast<int>(kind >> (11 * r + 3)) & 15; }
__host__ __device__ inline int rs_right(uint64_t kind, int r) {
    return static_cast<int>((kind >> 7) >> (11 * r)) & 15;
}

// A grammar's rules by kind, as in sweep.h.
struct ResidentGrammar {
    int32_t n_dyn, n_list, n_lf, n_rf, n_ll, n_dd;
    int32_t d_nt;   // growing nonterminal whose gained bits are kept (left operand of the dd rules), or -1
    int32_t n_tt;   // right operands of dd rules
    uint64_t lf, rf, ll, dd;
    uint64_t runs;       // by growing nonterminal, eight bits each: the lf and rf rules that read it
    int32_t pull_mask;   // heads of lf rules
    int32_t src;         // the one left operand of the rf rules, -1 when they differ or there are none
    int32_t n_term;      // terminal rules in term[], -1: too many, in the slot's tables only
    int32_t term[kRsMaxTerm];  // label << 8 | nonterminal
    // by nonterminal, or -1: the growing ones' numbers, the fixed ones' lists (in: of rf operands)
    int8_t dyn[CFPQ_MAX_NONTERMINALS], list[CFPQ_MAX_NONTERMINALS], in[CFPQ_MAX_NONTERMINALS];
    int8_t rf_in[kRsMaxRules];  // by rf rule: its operand's incoming list
    int8_t lf_in[kRsMaxRules];  // and by lf rule, with `queued`
    int8_t queued;              // the kernel may follow single facts (all lf_in exist)
    int8_t dyn_nt[kRsMaxDyn], tt[kRsMaxDyn];                          // by growing nonterminal
};

// Sorts n_rules (lhs, left, right) triples; false when the grammar is beyond
// the kernel: its tables, a scatter head that is itself scattered from, or dd
// rules with different left operands (or a head that is scattered from and is
// not that operand).  queue: with the lists that following single facts takes.
inline bool resident_grammar(const int32_t* rules, int32_t n_rules, int32_t n_nt, bool queue, ResidentGrammar* g) {
    std::memset(g, 0, sizeof(*g));
    g->n_term = -1;
    g->n_dyn = g->n_list = g->n_lf = g->n_rf = g->n_ll = g->n_dd = g->n_tt = 0;
    g->d_nt = -1;
    g->lf = g->rf = g->ll = g->dd = 0;
    for (int a = 0; a < CFPQ_MAX_NONTERMINALS; ++a) g->dyn[a] = g->list[a] = g->in[a] = -1;
    for (int a = 0; a < kRsMaxDyn; ++a) g->dyn_nt[a] = g->tt[a] = -1;
    if (n_rules < 1 || n_rules > kRsMaxBin) return false;
    for (int r = 0; r < n_rules; ++r) g->dyn[rules[3 * r]] = 0;
    for (int a = 0; a < n_nt; ++a) {
        if (g->dyn[a] < 0) continue;
        if (g->n_dyn == kRsMaxDyn) return false;
        g->dyn[a] = static_cast<int8_t>(g->n_dyn);
        g->dyn_nt[g->n_dyn++] = static_cast<int8_t>(a);
    }
    for (int r = 0; r < n_rules; ++r) {
        const int h = g->dyn[rules[3 * r]], b = rules[3 * r + 1], c = rules[3 * r + 2];
        for (int o : {b, c})
            if (g->dyn[o] < 0 && g->list[o] < 0) {
                if (g->n_list == kRsMaxLists) return false;
                g->list[o] = static_cast<int8_t>(g->n_list++);
            }
        const bool bd = g->dyn[b] >= 0, cd = g->dyn[c] >= 0;
        if (bd && !cd) {
            if (g->in[c] < 0) {
                if (g->n_list == kRsMaxLists) return false;
                g->in[c] = static_cast<int8_t>(g->n_list++);
            }
            if (g->n_rf < kRsMaxRules) g->rf_in[g->n_rf] = g->in[c];
        }
        const uint64_t packed = static_cast<uint64_t>(h | (bd ? g->dyn[b] : g->list[b]) << 3 |
                                                      (cd ? g->dyn[c] : g->list[c]) << 7);
        uint64_t* kind = bd ? (cd ? &g->dd : &g->rf) : (cd ? &g->lf : &g->ll);
        int32_t* n = bd ? (cd ? &g->n_dd : &g->n_rf) : (cd ? &g->n_lf : &g->n_ll);
        if (*n == kRsMaxRules) return false;
        *kind |= packed << (11 * (*n)++);
        if (bd && cd) {
            if (g->d_nt >= 0 && g->d_nt != g->dyn[b]) return false;
            g->d_nt = g->dyn[b];
            if (g->tt[static_cast<int>(g->dyn[c])] < 0) g->tt[static_cast<int>(g->dyn[c])] = static_cast<int8_t>(g->n_tt++);
        }
    }
    for (int r = 0; r < g->n_rf; ++r) {
        const int from = rs_left(g->rf, r);
        for (int q = 0; q < g->n_rf; ++q)
            if (rs_head(g->rf, q) == from) return false;
        for (int q = 0; q < g->n_dd; ++q)
            if (rs_head(g->dd, q) == from && from != g->d_nt) return false;
        g->src = r == 0 || g->src == from ? from : -1;
        g->runs += uint64_t{1} << (8 * from);
    }
    if (g->n_rf == 0) g->src = -1;
    for (int r = 0; r < g->n_lf; ++r) {
        g->runs += uint64_t{1} << (8 * rs_right(g->lf, r));
        g->pull_mask |= 1 << rs_head(g->lf, r);
    }
    g->queued = queue && g->n_dd == 0;
    for (int r = 0, lf = 0; r < n_rules && g->queued; ++r) {
        const int b = rules[3 * r + 1];
        if (g->dyn[b] >= 0 || g->dyn[rules[3 * r + 2]] < 0) continue;
        if (g->in[b] < 0 && g->n_list < kRsMaxLists) g->in[b] = static_cast<int8_t>(g->n_list++);
        g->lf_in[lf++] = g->in[b];
        if (g->in[b] < 0) g->queued = 0;
    }
    return true;
}

// Lanes a row: 128 bits each.
__host__ __device__ inline int resident_lanes(int32_t n) { return n <= 128 ? 1 : n <= 256 ? 2 : 4; }

// LDS of a slot in bytes (offsets from the start of the dynamic LDS): T of
// the growing nonterminals, the kept gained bits, transposed operands (with
// `turned`: where there is room), changed-row bitmaps of three
// loops, list ends, with `queued` the lists' first eight entries in 8 bytes, list
// entries.
struct ResidentLds {
    int32_t rows, mat;  // rows of a matrix (a multiple of 128 where it is multiplied by tiles), bytes
    int32_t off_d, off_tt, off_chg, off_end, off_near, off_idx, total;
};
__host__ __device__ inline ResidentLds resident_lds(int32_t n, const ResidentGrammar& g, int64_t entries,
                                                    bool turned) {
    ResidentLds l;
    const int lanes = resident_lanes(n);
    const int round = turned ? (g.n_dd > 0 ? 128 : 64) : 32;
    l.rows = (n + round - 1) / round * round;
    l.mat = l.rows * lanes * 16;
    l.off_d = g.n_dyn * l.mat;
    l.off_tt = l.off_d + (g.d_nt >= 0 ? l.mat : 0);
    l.off_chg = l.off_tt + (turned ? (g.n_tt > 0 ? g.n_tt : 1) * l.mat : 0);
    // every part starts on 16 bytes: the kernel clears up to off_idx in such pieces
    l.off_end = l.off_chg + (3 * g.n_dyn * (l.rows / 32) * 4 + 15) / 16 * 16;
    l.off_near = l.off_end + ((g.n_list * n + 1) * 4 + 15) / 16 * 16;
    l.off_idx = l.off_near + (g.queued ? (g.n_list * n * 8 + 15) / 16 * 16 : 0);
    const int64_t t = l.off_idx + (entries * 2 + 15) / 16 * 16;
    l.total = t > (1 << 30) ? 1 << 30 : static_cast<int32_t>(t);
    return l;
}
// Launch classes: lanes a row (1, 2, 4), without and with dd rules; then one
// lane a row with transposed operands, without and with dd rules.
constexpr int32_t kResidentClasses = 8;

// Most dynamic LDS of a launch.  The rest of the 160 KiB is the kernel's own: at
// most 480 bytes, and in class 0, whose kernel may follow single facts, their
// queue (2544 bytes in all).
constexpr int32_t kLdsBytes = 160 * 1024;
__host__ __device__ constexpr int32_t resident_max_lds(int32_t cls) { return cls == 0 ? 156 * 1024 : 158 * 1024; }

// Whether the resident sweep takes a graph of n nodes and n_edges edges and this
// grammar (tables and lists fit, and the lists are short enough to pay), and for
// its launch: the grammar as the kernel reads it (kept where the slot's rule
// triples would be), class, LDS bytes, and whether those hold transposed
// operands (SlotDesc::tile).
struct ResidentPlan {
    ResidentGrammar g;
    int32_t per_edge;  // the most terminal rules of one label
    int32_t cls, lds, turned;
};
// Graphs that may follow single facts: sparse, one lane a row.
inline bool resident_queues(int32_t n, int64_t n_edges) {
    return resident_lanes(n) == 1 && n_edges < 2 * static_cast<int64_t>(n);
}
// The grammar's part (the same for every graph with the same `queue`), then the
// graph's; resident_plan does both.
bool resident_rules(const cfpq_grammar* gr, bool queue, ResidentPlan* plan);
bool resident_fits(int32_t n, int64_t n_edges, ResidentPlan* plan);
inline bool resident_plan(const cfpq_grammar* gr, int32_t n, int64_t n_edges, ResidentPlan* plan) {
    return resident_rules(gr, resident_queues(n, n_edges), plan) && resident_fits(n, n_edges, plan);
}

// What resident_solo leaves in pinned host memory; loop = 1 comes last.
struct ResidentReport {
    int64_t iterations, products, dense;
    uint64_t ticks;  // of the constant clock, from start to end
    int32_t capped, bad_edges, loop, pad;
};

// One slot by itself, without tables on the device; its terminal rules have to
// be in the grammar (g.n_term >= 0).
hipError_t resident_solo(const SlotDesc& d, const ResidentPlan& p, ResidentReport* report, hipStream_t s);

// One workgroup per listed slot of class cls, with `lds` bytes of LDS (the
// most any of them needs).  It initialises the slot's matrices itself, from
// the edges, and counts edges out of range in the slot's state.
hipError_t resident_sweep(const EngineBuffers& b, const int32_t* ids, int32_t count, int32_t cls, int32_t lds,
                          hipStream_t s);

}  // namespace cfpq
