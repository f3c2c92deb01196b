// Row sweeps: one launch per loop for every rule with an edge-matrix operand.
//
// A nonterminal that heads no binary rule is fixed: its matrix is the edge
// matrix of its terminals, a few bits a row, kept here as adjacency lists.
// For a rule A -> B C with a fixed operand a loop then needs no matrix
// product, only what the last loop added:
//   B fixed:  row i of A gains the rows D_C[k] for the edges i -> k of B,
//             D_C[k] being the bits row k of C gained in the last loop;
//   C fixed:  every bit k that row i of B gains sets the bits of the edges
//             k -> j of C in row i of A: it stays within the row.
// One workgroup takes a few rows of every nonterminal, so each row has one
// writer: it pulls, scatters, stores the new bits into T and into the loop's
// D rows, and marks the rows in the loop's changed-row bitmap.  Rows without
// a changed neighbour cost a few bitmap reads.  The loop's flags stay on the
// device, so the host queues loops ahead of their results.
//
// Measured (in place of the product loops, which took a launch or more per
// rule and loop and whole-matrix passes): a^n b^n on G(7001, 28004), 2480 ->
// 550 us; same-generation on G(1500, 6000), 1870 -> 242 us, and on a
// 4096-node hierarchy, 334 -> 87 us; Dyck on G(16384, 65536), 5540 -> 4070 us.
// A dense a^n b^n loop at 7001 nodes takes about 35 us for some 60 MB.
//
// A rule whose two operands both grow (S -> S S) is multiplied by the product
// kernels into a matrix P of its head, which the sweep ORs in like a pulled
// row.
#pragma once

#include <cstddef>
#include <cstdint>

#include "cfpq_internal.h"

namespace cfpq {

constexpr int kSwMaxRules = 32;      // rules with a fixed operand, per kind
constexpr int kSwMaxDyn = 8;         // nonterminals that head a binary rule
constexpr int kSwMaxLists = 32;      // adjacency lists of fixed operands, outgoing and incoming
constexpr int kSwMaxTerm = 32;       // terminal rules
constexpr int32_t kSwLoopNodes = 8192;  // past them a grammar of growing pairs alone keeps the product loops
constexpr int64_t kSwMaxWords = 256;  // words per row (16384 nodes): 64 rows of them fill 132 of the 160 KiB of LDS

// Edges up to which the adjacency lists are reserved (each edge may enter several).
inline int64_t sweep_max_edges(const Layout& L) { return 16 * L.npad; }

// A grammar's rules by kind.  Dynamic nonterminals (heads of binary rules) are
// numbered 0..n_dyn-1 (dyn_nt gives their ids); a fixed operand is the number
// of its list: row k of an outgoing list holds the j of the edges k -> j, row
// j of an incoming one their k.
struct SweepGrammar {
    int32_t n_dyn = 0, n_list = 0, n_lf = 0, n_rf = 0, n_ll = 0, n_dd = 0, n_term = 0;
    uint8_t dyn_nt[kSwMaxDyn] = {};
    struct Rule {
        uint8_t head, left, right;
    };
    Rule lf[kSwMaxRules] = {};  // head dyn, left fixed, right dyn
    Rule rf[kSwMaxRules] = {};  // head dyn, left dyn, right fixed
    uint8_t rf_in[kSwMaxRules] = {};  // and its incoming list
    Rule ll[kSwMaxRules] = {};  // head dyn, both fixed (first loop only)
    Rule dd[kSwMaxRules] = {};  // all dyn
    struct Term {
        int32_t label;
        int16_t nt;        // nonterminal whose matrix gains the bit
        int8_t out, in;    // its lists, or -1
    };
    Term term[kSwMaxTerm] = {};
    uint32_t rf_mask = 0;    // dyn: head of an rf rule
    uint32_t ll_mask = 0;    // dyn: head of an ll rule
    uint32_t init_mask = 0;    // dyn: has terminal rules, so may hold bits after initialisation
    uint32_t dd_mask = 0;      // dyn: operand of a dd rule
    uint32_t p_mask = 0;       // dyn: head of a dd rule
};

// Rows of a workgroup, and workgroups: 16 rows (one a wavefront) up to 4096
// nodes, 64 (256 workgroups at 16384) from 8192 on.
inline int32_t sweep_rows(int32_t n) { return n <= 4096 ? 16 : n <= 8192 ? 32 : 64; }
inline int32_t sweep_groups(int32_t n) { return (n + sweep_rows(n) - 1) / sweep_rows(n); }

// False when the grammar is beyond the tables above.
bool sweep_grammar(const cfpq_grammar* gr, SweepGrammar* out);

// Hubs: lists whose rows make this many words and more.  They are pulled by all
// workgroups together, or scattered as a row of their matrix (kernels_sweep.hip);
// at most kSwMaxHubs of them, or none is.
constexpr int64_t kSwHubWords = 512 * 1024;
constexpr int kSwMaxHubs = 32;
// In SweepCtl::any beside the mask: rows wait in the inbox; there are hubs (set
// with some other bit only, so that 0 is still the fixpoint).
constexpr uint32_t kSwInboxBit = 1u << 31, kSwHubsBit = 1u << 30;
// Looked for above 8192 nodes: below, a list is at most 8 MiB of rows, and the
// code for them costs the sweeps 2% (dense loops at 7001 nodes 26.6 -> 27.2 us).
inline bool sweep_hubs(const Layout& L) { return L.W > 128; }

// Control block on the device.  Flags and counts of loop t are at index t & 3;
// each loop clears the next one's.
struct alignas(256) SweepCtl {
    uint32_t any[4];                          // mask of the dynamic nonterminals that changed
    unsigned long long gained[4][kSwMaxDyn];  // bits gained (grammars with dd rules)
    int32_t loops;                            // loops executed
    int32_t bad_edges;
    int64_t products, sparse, delta, dense;   // rules run, by kind
    int32_t list_top;                         // bump allocator of the adjacency lists
    int32_t n_hubs;                           // entries of hub that would be used
    int2 hub[kSwMaxHubs];                     // lf rule, or n_lf + rf rule, | fixed operand << 8; node
};

// The inbox follows the control block: [2][kSwMaxHubs][W], by loop parity.
inline size_t sweep_inbox_bytes(const Layout& L) {
    return sweep_hubs(L) ? static_cast<size_t>(2) * kSwMaxHubs * L.W * 8 : 0;
}

// What the host reads while loops are in flight (pinned host memory).
struct SweepReport {
    int32_t loop;   // the last loop a report was made for
    uint32_t any;   // its change mask
    int32_t bad_edges;
    int32_t loops;  // loops executed so far
    int64_t products, sparse, delta, dense;
    unsigned long long gained[kSwMaxDyn];
};

struct SweepBuffers {
    uint64_t* T = nullptr;        // result matrices
    uint64_t* D[2] = {};          // rows gained, by loop parity: n_dyn matrices each
    uint64_t* P = nullptr;        // one matrix per head of a dd rule (slot by p_mask order)
    uint64_t* chg = nullptr;      // changed-row bitmaps [4][n_dyn][W], by loop & 3
    SweepCtl* ctl = nullptr;
    int32_t* wg = nullptr;        // [2][n_dyn][sweep_groups] bits a workgroup's rows gained, by loop parity
    int2* list = nullptr;         // [n_list][n] start and length
    int32_t* cur = nullptr;       // [n_list][n] fill cursors
    uint4* near = nullptr;        // [n_list][n] the 16-byte form (near_list.h)
    int32_t* idx = nullptr;       // targets
};

// Clear T, the control block, bitmaps and counters, set the edges' bits and
// build the adjacency lists.
hipError_t launch_sweep_init(const SweepGrammar& g, const SweepBuffers& b, const Layout& L, const cfpq_edge* edges,
                             int64_t m, int32_t n_nt, int32_t n_terminals, hipStream_t s);

// Loop t (1, 2, ...).  p_mask: heads whose P holds this loop's products.
// count: add the bits gained to ctl->gained.  dense_dd: the dd rules run
// dense on the device's own decision (counted here); otherwise the host
// counts them.  Does nothing when loop t - 1 changed nothing.
hipError_t launch_sweep(const SweepGrammar& g, const SweepBuffers& b, const Layout& L, int32_t t, uint32_t p_mask,
                        bool count, bool dense_dd, hipStream_t s);

// Clears the rows of head h's D matrix that loop t - 1 did not write (and the
// padding rows), so that a product may read the whole matrix in loop t.
hipError_t launch_sweep_clean(const SweepGrammar& g, const SweepBuffers& b, const Layout& L, int32_t t, int h,
                              hipStream_t s);

// Copies loop t's state to *report (device-visible host memory).
hipError_t launch_sweep_report(const SweepBuffers& b, int32_t t, SweepReport* report, hipStream_t s);

// Whether the sweeps may run a closure of this size, grammar and options (they
// do when it has at most sweep_max_edges edges), the workspace they need, and
// the closure itself.
bool sweep_route(const cfpq_graph* g, const cfpq_grammar* gr, const cfpq_options& o);
size_t sweep_workspace(const cfpq_graph* g, const cfpq_grammar* gr);
cfpq_status closure_sweep(const cfpq_graph* graph, const cfpq_grammar* grammar, const cfpq_options& o, void* stream,
                          void* d_workspace, size_t workspace_bytes, uint64_t* d_result, cfpq_stats* stats);

}  // namespace cfpq
