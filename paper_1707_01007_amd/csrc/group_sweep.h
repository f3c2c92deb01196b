// Row sweeps of many instances at once: the batched engine's route for
// instances of 513 to 4096 nodes.
//
// The rules are split as in sweep.h (fixed operands as adjacency lists, deltas
// D of the last loop, rules over two growing operands multiplied into P), but
// one launch a loop serves every instance: a workgroup takes 64 rows of one
// instance, a row is 16, 32 or 64 lanes wide, and what an instance needs (its
// tables, its loop's flags) is data on the device.  An instance that reached
// its fixpoint costs its workgroups a look at its flags.
//
// Measured on the benchmark's batch (512 instances of 64 to 2048 nodes, the
// smaller ones resident beside these): 8.7 -> 4.4 ms, of which 1.4 ms pass in
// the caller.  The tile engine ran rules with an edge matrix on the left by
// rows and the others as products, four launches a loop (135 us a loop while
// the instances were dense, 18 us near the end; now 220 and 5).
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

#include "sweep.h"

namespace cfpq {

constexpr int64_t kGsMaxWords = 64;  // words per row: one a lane (4096 nodes)
constexpr int kGsPull = 16;          // rows a row pulls from a list in LDS
constexpr int kGsRows = 64;          // rows of a workgroup: one word of a changed-row bitmap

// A rule of SweepGrammar, packed: head, left, right and (rf) incoming list.
struct GroupGrammar {
    int32_t n_dyn, n_list, n_lf, n_rf, n_ll, n_dd, n_term;
    uint32_t rf_mask, ll_mask, init_mask;
    uint32_t rule[kSwMaxRules];  // lf, rf, ll, dd
    int32_t dyn_nt[kSwMaxDyn];
    int32_t p_slot[kSwMaxDyn];   // head of a dd rule: its matrix of P, or -1
    int32_t tt_slot[kSwMaxDyn];  // right operand of one: its transpose, or -1
    SweepGrammar::Term term[kSwMaxTerm];
};

struct GroupCtl {
    uint32_t any[4];  // dynamic nonterminals changed by loop t, at t & 3
    int32_t loops, capped, bad_edges;
    int32_t list_top;  // entries of idx in use
    int64_t products, dense;  // dense: of the rules over two growing operands
    int32_t spare;  // change flag nobody reads
};

struct GroupSlot {
    GroupGrammar g;
    uint64_t* T;
    uint64_t* D[2];
    uint64_t* P;
    uint64_t* TT;
    uint64_t* chg;  // [2][n_dyn][W], by loop parity; written whole by every loop
    GroupCtl* ctl;
    int32_t* wg;    // [2][n_dyn][groups]: bits a workgroup's rows gained
    int2* list;     // [n_list][n]: start and length
    uint4* near;    // [n_list][n]: the first entries (group_lists_kernel)
    int32_t* idx;
    const cfpq_edge* edges;
    int64_t n_edges, max_iters, mat_words;
    int32_t n, W, n_nt, n_terminals, groups;
    int32_t slot;   // the engine's slot whose SlotState gets the result
    uint32_t base;  // loops of the group before the instance joined: its own t = loop - base
};

// Work of a launch, a block each: slot << 16 | what (row group, tile), -1: none.
struct GroupMaps {
    const int32_t* rows[2] = {};     // row groups of instances of up to 32 words a row, and of more
    const int32_t* tiles = nullptr;  // 256 x 256 tiles of the dd rules: slot << 16 | rule << 8 | i << 4 | j
    const int32_t* trans = nullptr;  // 256 x 256 tiles of their right operands: slot << 16 | dyn << 8 | i << 4 | j
    int32_t n_rows[2] = {}, n_tiles = 0, n_trans = 0;
    size_t lds[2] = {};
};

// The blocks of slots [begin, end) of a table.  Workgroups go to the eight XCDs
// in turn by their number, so an instance's row groups are placed eight apart:
// the rows they pull from each other then come through one XCD's L2.  The
// widest instances go first, each to the XCD with the fewest words so far.
struct GroupLists {
    std::vector<int32_t> rows[2], tiles, trans;
    size_t lds[2] = {};
    void add(const GroupSlot* slots, int32_t begin, int32_t end);
    size_t size() const { return rows[0].size() + rows[1].size() + tiles.size() + trans.size(); }
    // Writes the lists to host, as they will lie at device; the entries written.
    size_t put(int32_t* host, const int32_t* device, GroupMaps* m) const;
};

// What the host reads while loops are in flight (pinned host memory).
struct GroupReport {
    int32_t loop, running, running_dd, pad;
};

// Whether an instance may run here, its packed grammar, its descriptor without
// pointers, and the workspace it needs from ws on (the pointers of *d into it
// are set when ws is not null).
bool group_grammar(const cfpq_grammar* gr, int32_t n_nodes, int64_t n_edges, GroupGrammar* g);
GroupSlot group_slot(const GroupGrammar& g, int32_t n_nodes);
size_t group_layout(const GroupGrammar& g, int32_t n_nodes, char* ws, GroupSlot* d);

// Clears what must be clear, sets the edges' bits and builds the lists.
hipError_t group_init(const GroupSlot* slots, int32_t count, int32_t max_lists, hipStream_t s);
// Loop `loop` of the group (an instance's own loop is loop - base; first: that is
// 1 for all of them).  with_dd: some slot that still runs has dd rules.
hipError_t group_loop(const GroupSlot* slots, const GroupMaps& m, uint32_t loop, bool first, bool with_dd,
                      hipStream_t s);
hipError_t group_report(const GroupSlot* slots, int32_t count, uint32_t loop, GroupReport* out, hipStream_t s);
// The slots' loops, products, caps and bad edges into the engine's states;
// those that `loop` did not change are done.
struct SlotState;
hipError_t group_finish(const GroupSlot* slots, int32_t count, uint32_t loop, SlotState* states, hipStream_t s);

// LDS bytes of a workgroup for rows of W words.
inline size_t group_lds(int64_t W, int32_t n_dyn) {
    return (static_cast<size_t>(kGsRows) * (W + 1) + static_cast<size_t>(n_dyn) * W) * 8 +
           static_cast<size_t>(n_dyn) * kGsRows * (2 * kGsPull + 4);
}

}  // namespace cfpq
