// cfpq_closure by row sweeps (sweep.h): the in-place closure of grammars
// whose rules mostly have an edge-matrix operand.
//
// Grammars without a rule over two growing operands, and padded sides below
// kHybridMinRows, run without the host: a loop is one sweep (after the dense
// products of the rules over two growing operands, each skipped on the device
// when its operands did not change), loops are queued in groups, and a group's
// report is awaited only after the next group is queued.  From kHybridMinRows
// on a dense product costs more than a round trip, so those rules' products
// are chosen per loop by the cost model from the reported counts.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstring>
#include <string>
#include <vector>

#include "batch_engine.h"
#include "closure_common.h"
#include "sweep.h"

namespace cfpq {
namespace {

// Loops queued per report.  Two groups are in flight, so at most 2 * 4 - 1
// sweeps run past the fixpoint, about 2 us each; shorter groups cost a report
// (3 us) each, and the host's queueing (about 3 us a launch) has to stay ahead.
constexpr int32_t kGroup = 4;

struct SweepPlan {
    SweepGrammar g;
    Layout L;
    size_t off_edges = 0, off_wg = 0, off_chg = 0, off_ctl = 0, off_list = 0, off_cur = 0, off_near = 0, off_idx = 0;
    size_t off_d0 = 0, off_d1 = 0, off_p = 0, off_tt = 0, off_bt = 0, off_pt = 0, off_ct = 0, off_rowor = 0;
    size_t off_flag = 0, total = 0;
    bool hosted = false;  // dd products chosen on the host
    int8_t tt_slot[kSwMaxDyn];
    int32_t n_tt = 0;
};

SweepPlan sweep_plan(const cfpq_graph* gr, const SweepGrammar& g) {
    SweepPlan p;
    p.g = g;
    p.L = layout_for(gr->n_nodes);
    const Layout& L = p.L;
    const size_t mat = static_cast<size_t>(L.mat_words) * 8;
    p.hosted = g.n_dd > 0 && L.npad >= kHybridMinRows;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align_up(bytes, 256);
        return at;
    };
    p.off_edges = take(gr->edges_on_device ? 0 : static_cast<size_t>(gr->n_edges) * sizeof(cfpq_edge));
    const size_t lists = static_cast<size_t>(std::max(g.n_list, 1)) * std::max(L.n, 1);
    p.off_wg = take(static_cast<size_t>(2) * g.n_dyn * sweep_groups(L.n) * 4);
    p.off_chg = take(static_cast<size_t>(4) * g.n_dyn * L.W * 8);
    static_assert(sizeof(SweepCtl) % 256 == 0, "the inbox follows");
    p.off_ctl = take(sizeof(SweepCtl));
    take(sweep_inbox_bytes(L));  // after ctl, where the kernels look for it
    p.off_list = take(lists * 8);
    p.off_cur = take(lists * 4);
    p.off_near = take(lists * 16);
    // an edge enters the lists of its label's (distinct) terminal rules
    int32_t per_edge = 1;
    for (int32_t q = 0; q < g.n_term; ++q) {
        int32_t c = 0;
        for (int32_t r = 0; r < g.n_term; ++r)
            if (g.term[r].label == g.term[q].label) c += (g.term[r].out >= 0 ? 1 : 0) + (g.term[r].in >= 0 ? 1 : 0);
        per_edge = std::max(per_edge, c);
    }
    p.off_idx = take(static_cast<size_t>(sweep_max_edges(L)) * per_edge * 4);
    p.off_d0 = take(mat * g.n_dyn);
    p.off_d1 = take(mat * g.n_dyn);
    p.off_p = take(mat * __builtin_popcount(g.p_mask));
    std::fill(p.tt_slot, p.tt_slot + kSwMaxDyn, int8_t{-1});
    for (int r = 0; r < g.n_dd; ++r) {
        const int c = g.dd[r].right;
        if (p.tt_slot[c] < 0) p.tt_slot[c] = static_cast<int8_t>(p.n_tt++);
    }
    p.off_tt = take(mat * p.n_tt);
    if (p.hosted) {
        p.off_bt = take(mat);
        p.off_pt = take(mat);
        p.off_ct = take(mat);
        p.off_rowor = take(rowor_scratch_bytes(L));
    }
    p.off_flag = take(256);
    p.total = off;
    return p;
}

}  // namespace

// The sweeps pay where the lists are short and 64 rows fit in LDS; the other
// closures (and every option that names a kernel, a schedule or a measurement)
// keep the product loops.
bool sweep_route(const cfpq_graph* g, const cfpq_grammar* gr, const cfpq_options& o) {
    if (o.schedule != CFPQ_SCHEDULE_INPLACE || o.hybrid != CFPQ_HYBRID_AUTO || !o.dirty_worklist || o.profile ||
        o.warm_start != 0 || o.tile != 0)
        return false;
    if (g->n_nodes <= 0) return false;
    const Layout L = layout_for(g->n_nodes);
    if (L.W > kSwMaxWords || L.npad <= kSmallMaxPad) return false;
    SweepGrammar sg;
    if (!sweep_grammar(gr, &sg)) return false;
    if (sg.n_dd > 0 && g->n_nodes > kMfmaMaxNodes) return false;
    // Only rules of two growing operands: a sweep has nothing of its own to add,
    // and its products, which see a loop's bits in the next one, take more
    // loops than the product loops, which work in place.  From 8193 nodes the
    // products are what a closure costs.  S -> S S, times of the sweeps over
    // the loops': chains 0.9 to 1.2 at 8000 nodes, 1.3 to 2.0 from 9000
    // (16000: 10.4 ms against 5.3), grids 1.07 and 1.02 to 1.2, random graphs
    // of 15 edges a node 1.26 and 1.4 to 1.5; trees and components of 20
    // nodes, which end after five cheap loops, 0.8 and 0.9.
    if (sg.n_dd > 0 && sg.n_lf == 0 && sg.n_rf == 0 && g->n_nodes > kSwLoopNodes) return false;
    return true;
}

size_t sweep_workspace(const cfpq_graph* g, const cfpq_grammar* gr) {
    SweepGrammar sg;
    if (!sweep_grammar(gr, &sg)) return 0;
    return sweep_plan(g, sg).total;
}

cfpq_status closure_sweep(const cfpq_graph* graph, const cfpq_grammar* grammar, const cfpq_options& o, void* stream,
                          void* d_workspace, size_t workspace_bytes, uint64_t* d_result, cfpq_stats* stats) {
    SweepGrammar sg;
    if (!sweep_grammar(grammar, &sg)) return fail(CFPQ_EINVAL, "grammar beyond the row sweeps");
    const SweepPlan p = sweep_plan(graph, sg);
    if (!d_workspace) return fail(CFPQ_EINVAL, "d_workspace is NULL");
    if (workspace_bytes < p.total)
        return fail(CFPQ_ENOMEM, "workspace too small: need " + std::to_string(p.total) + " bytes");
    JsonLog jlog;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(d_workspace);
    const Layout& L = p.L;
    const size_t mw = static_cast<size_t>(L.mat_words);
    const int32_t n_nt = grammar->n_nonterminals;
    SweepBuffers b;
    b.T = d_result;
    b.D[0] = reinterpret_cast<uint64_t*>(ws + p.off_d0);
    b.D[1] = reinterpret_cast<uint64_t*>(ws + p.off_d1);
    b.P = reinterpret_cast<uint64_t*>(ws + p.off_p);
    b.chg = reinterpret_cast<uint64_t*>(ws + p.off_chg);
    b.ctl = reinterpret_cast<SweepCtl*>(ws + p.off_ctl);
    b.wg = reinterpret_cast<int32_t*>(ws + p.off_wg);
    b.list = reinterpret_cast<int2*>(ws + p.off_list);
    b.cur = reinterpret_cast<int32_t*>(ws + p.off_cur);
    b.near = reinterpret_cast<uint4*>(ws + p.off_near);
    b.idx = reinterpret_cast<int32_t*>(ws + p.off_idx);
    uint64_t* TT = reinterpret_cast<uint64_t*>(ws + p.off_tt);
    uint64_t* BT = reinterpret_cast<uint64_t*>(ws + p.off_bt);
    uint64_t* PT = reinterpret_cast<uint64_t*>(ws + p.off_pt);
    uint64_t* CTT = reinterpret_cast<uint64_t*>(ws + p.off_ct);
    int32_t* ROWOR = reinterpret_cast<int32_t*>(ws + p.off_rowor);
    int32_t* spare = reinterpret_cast<int32_t*>(ws + p.off_flag);

    float tuned_ms = 0.f;
    int32_t tile = 0, tp = 0, tt = 0;
    const int32_t path = choose_path(L, o.path, &tile);
    if (!(tuned_choice(L, &tp, &tt, &tuned_ms) && tp == path)) tuned_ms = 0.f;
    const bool ct = reads_ct(path);

    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    CFPQ_HIP(hipEventCreate(&ev0));
    CFPQ_HIP(hipEventCreate(&ev1));
    struct EvGuard {
        hipEvent_t a, b;
        ~EvGuard() {
            (void)hipEventDestroy(a);
            (void)hipEventDestroy(b);
        }
    } guard{ev0, ev1};
    const cfpq_edge* d_edges = graph->edges;
    if (!graph->edges_on_device && graph->n_edges > 0) {
        auto* dst = reinterpret_cast<cfpq_edge*>(ws + p.off_edges);
        CFPQ_HIP(hipMemcpyAsync(dst, graph->edges, static_cast<size_t>(graph->n_edges) * sizeof(cfpq_edge),
                                hipMemcpyHostToDevice, s));
        d_edges = dst;
    }
    void* pb = nullptr;
    CFPQ_HIP(pinned_readback(2 * sizeof(SweepReport), &pb));
    auto* rep = static_cast<SweepReport*>(pb);
    rep[0].loop = rep[1].loop = 0;
    Drain drain{s};
    CFPQ_HIP(hipEventRecord(ev0, s));
    CFPQ_HIP(launch_sweep_init(sg, b, L, d_edges, graph->n_edges, n_nt, grammar->n_terminals, s));
    if (sg.p_mask != 0) CFPQ_HIP(launch_zero(b.P, mw * __builtin_popcount(sg.p_mask), s));

    const int64_t nn = graph->n_nodes;
    const int64_t cap = o.max_iters > 0 ? o.max_iters : nn * nn * n_nt + 1;
    auto T_of = [&](int h) { return b.T + sg.dyn_nt[h] * mw; };
    auto P_of = [&](int h) { return b.P + __builtin_popcount(sg.p_mask & ((1u << h) - 1)) * mw; };
    const auto host_t0 = std::chrono::steady_clock::now();
    auto log_t = host_t0;
    auto log_loop = [&](int64_t loop, uint32_t any, int64_t launched, int64_t products, int64_t sparse,
                        int64_t delta) {
        const auto now = std::chrono::steady_clock::now();
        char buf[320];
        std::snprintf(buf, sizeof(buf),
                      "{\"event\": \"loop\", \"loop\": %lld, \"rules_launched\": %lld, \"changed\": %d, "
                      "\"products\": %lld, \"sparse_products\": %lld, \"delta_products\": %lld, "
                      "\"host_ms\": %.4f}",
                      static_cast<long long>(loop), static_cast<long long>(launched),
                      __builtin_popcount(any & ~(kSwInboxBit | kSwHubsBit)),
                      static_cast<long long>(products), static_cast<long long>(sparse), static_cast<long long>(delta),
                      std::chrono::duration<double, std::milli>(now - log_t).count());
        log_t = now;
        jlog.line(buf);
    };

    SweepReport last{};
    int64_t products = 0, sparse = 0, delta = 0, dense = 0;  // the host's part (hosted dd products)
    bool converged = false;
    if (!p.hosted) {
        // queue a group, then look at the report of the one before
        const int32_t group = jlog.f ? 1 : kGroup;
        const bool lag = !jlog.f;
        int64_t t = 0, waiting = 0;  // waiting: the loop of the oldest report not yet read
        int slot = 0;
        int64_t logged = 0;
        bool transposed = false;  // the kept transposes exist
        while (true) {
            int64_t queued_report = 0;
            if (t < cap) {
                const int64_t end = std::min<int64_t>(cap, t + group);
                for (++t; t <= end; ++t) {
                    const int32_t ti = static_cast<int32_t>(t & 0x7FFFFFFF);
                    if (sg.n_dd > 0) {
                        // the last loop's change mask predicates the transposes and products
                        const int32_t* any_prev = reinterpret_cast<const int32_t*>(&b.ctl->any[(t - 1) & 3]);
                        const bool first = t == 1;
                        if (!first || (sg.init_mask & sg.dd_mask) != 0) {
                            for (int c = 0; c < sg.n_dyn && ct; ++c)
                                if (p.tt_slot[c] >= 0)
                                    CFPQ_HIP(launch_transpose(T_of(c), TT + p.tt_slot[c] * mw, L, s,
                                                              transposed ? any_prev : nullptr, -(1 << c)));
                            transposed = true;
                            for (int r = 0; r < sg.n_dd; ++r) {
                                const auto& q = sg.dd[r];
                                const int32_t want = -static_cast<int32_t>((1u << q.left) | (1u << q.right));
                                const int32_t* go = first ? nullptr : any_prev;
                                if (ct)
                                    CFPQ_HIP(launch_mfma_path(path, T_of(q.left), TT + p.tt_slot[q.right] * mw,
                                                              P_of(q.head), L, spare, s, go, want, tile));
                                else
                                    CFPQ_HIP(launch_bits_product(T_of(q.left), T_of(q.right), P_of(q.head), L, spare, s,
                                                                 tile, go, want));
                            }
                        }
                    }
                    CFPQ_HIP(launch_sweep(sg, b, L, ti, sg.p_mask, false, true, s));
                }
                t = end;
                CFPQ_HIP(launch_sweep_report(b, static_cast<int32_t>(t), &rep[slot], s));
                queued_report = t;
                slot ^= 1;
            }
            // read the older report (the newest too, once nothing more is queued)
            if (waiting == 0 && lag && t < cap) {
                waiting = queued_report;
                continue;
            }
            const int64_t want = waiting != 0 ? waiting : queued_report;
            if (want == 0) break;  // cap reached and every report read
            const SweepReport* r = &rep[((want - 1) / group) & 1];
            CFPQ_HIP(await_report(r, static_cast<int32_t>(want), s));
            last = *r;
            waiting = waiting != 0 ? queued_report : 0;
            if (jlog.f && last.loops > logged) {
                log_loop(last.loops, last.any, last.products - products, last.products, last.sparse, last.delta);
                products = last.products;
                logged = last.loops;
            }
            if (last.any == 0) {
                converged = true;
                break;
            }
        }
        products = last.products;
        sparse = last.sparse;
        delta = last.delta;
        dense = last.dense;
    } else {
        const HybridModel model = make_model(L, path, tuned_ms);
        int64_t rowor_calls = 0;
        CFPQ_HIP(launch_rowor_reset(ROWOR, s));
        std::vector<unsigned long long> nnz(kSwMaxDyn, 0), dnnz(kSwMaxDyn, 0);
        bool tt_fresh[kSwMaxDyn] = {};
        if ((sg.init_mask & sg.dd_mask) != 0) {
            // initial bits of the operands (counted in the control block's spare loop slots)
            std::vector<unsigned long long> all(n_nt, 0);
            auto* d_cnt = reinterpret_cast<unsigned long long*>(CTT);
            CFPQ_HIP(launch_zero(CTT, static_cast<size_t>(n_nt), s));
            CFPQ_HIP(launch_popcount(b.T, n_nt, L, d_cnt, s));
            CFPQ_HIP(hipMemcpyAsync(all.data(), d_cnt, static_cast<size_t>(n_nt) * 8, hipMemcpyDeviceToHost, s));
            CFPQ_HIP(hipStreamSynchronize(s));
            for (int h = 0; h < sg.n_dyn; ++h) dnnz[h] = nnz[h] = all[sg.dyn_nt[h]];
        }
        uint32_t any_prev = 0;
        // one product P |= B x C; bt / ctm: transposes that exist, else nullptr
        auto product_by = [&](int32_t mode, const uint64_t* Bm, const uint64_t* bt, const uint64_t* Cm,
                              const uint64_t* ctm, uint64_t* Pm) -> cfpq_status {
            if (mode == kModeRows) {
                CFPQ_HIP(launch_rowor_product(Bm, Cm, Pm, L, spare, ROWOR, s, nullptr, 1, rowor_calls++));
                return CFPQ_OK;
            }
            if ((mode == kModeCols || ct) && !ctm) {
                CFPQ_HIP(launch_transpose(Cm, CTT, L, s));
                ctm = CTT;
            }
            if (mode == kModeCols) {
                if (!bt) {
                    CFPQ_HIP(launch_transpose(Bm, BT, L, s));
                    bt = BT;
                }
                CFPQ_HIP(launch_zero(PT, mw, s));
                CFPQ_HIP(launch_rowor_product(ctm, bt, PT, L, nullptr, ROWOR, s, nullptr, 1, rowor_calls++));
                CFPQ_HIP(launch_transpose_or(PT, Pm, L, spare, s));
            } else if (ct) {
                CFPQ_HIP(launch_mfma_path(path, Bm, ctm, Pm, L, spare, s, nullptr, 1, tile));
            } else {
                CFPQ_HIP(launch_bits_product(Bm, Cm, Pm, L, spare, s, tile));
            }
            return CFPQ_OK;
        };
        for (int64_t t = 1; t <= cap; ++t) {
            uint32_t p_mask = 0;
            int64_t launched = 0;
            const uint64_t* Dm = b.D[(t + 1) & 1];
            uint32_t clean = 0;  // dyn whose last D matrix has its unchanged rows cleared
            for (int r = 0; r < sg.n_dd; ++r) {
                const auto& q = sg.dd[r];
                const double nb = static_cast<double>(nnz[q.left]), nc = static_cast<double>(nnz[q.right]);
                const bool first = t == 1;
                if (first ? nb == 0 || nc == 0 : !((any_prev >> q.left | any_prev >> q.right) & 1u)) continue;
                const bool rows_kept = p.tt_slot[q.left] >= 0 && tt_fresh[q.left];
                const bool right_kept = tt_fresh[q.right];
                const HybridChoice full = hybrid_choice(model, nb, nc, rows_kept, right_kept, ct);
                HybridChoice h1{kModeSkip, 0.0}, h2{kModeSkip, 0.0};
                bool use_delta = false;
                const double db = static_cast<double>(dnnz[q.left]), dc = static_cast<double>(dnnz[q.right]);
                if (!first) {
                    if (db > 0) h1 = hybrid_choice(model, db, nc, false, right_kept, ct);
                    if (dc > 0) h2 = hybrid_choice(model, nb, dc, rows_kept, false, ct);
                    use_delta = h1.us + h2.us < full.us;
                }
                uint64_t* Pm = P_of(q.head);
                p_mask |= 1u << q.head;
                // the kept transpose of an operand, brought up to date when the mode reads it
                auto kept = [&](int h) -> const uint64_t* { return tt_fresh[h] ? TT + p.tt_slot[h] * mw : nullptr; };
                auto refresh = [&](int h) -> cfpq_status {
                    if (p.tt_slot[h] >= 0 && !tt_fresh[h]) {
                        CFPQ_HIP(launch_transpose(T_of(h), TT + p.tt_slot[h] * mw, L, s));
                        tt_fresh[h] = true;
                    }
                    return CFPQ_OK;
                };
                cfpq_status st = CFPQ_OK;
                if (!use_delta) {
                    if (full.mode == kModeCols || (full.mode == kModeDense && ct)) st = refresh(q.right);
                    if (st == CFPQ_OK)
                        st = product_by(full.mode, T_of(q.left), kept(q.left), T_of(q.right), kept(q.right), Pm);
                    if (st != CFPQ_OK) return st;
                    ++products;
                    ++launched;
                    (full.mode == kModeDense ? dense : sparse) += 1;
                } else {
                    for (int h : {static_cast<int>(q.left), static_cast<int>(q.right)})
                        if (!((clean >> h) & 1u)) {
                            CFPQ_HIP(launch_sweep_clean(sg, b, L, static_cast<int32_t>(t & 0x7FFFFFFF), h, s));
                            clean |= 1u << h;
                        }
                    if (h1.mode != kModeSkip) {  // D_B x C
                        if (h1.mode == kModeCols || (h1.mode == kModeDense && ct)) st = refresh(q.right);
                        if (st == CFPQ_OK)
                            st = product_by(h1.mode, Dm + q.left * mw, nullptr, T_of(q.right), kept(q.right), Pm);
                        if (st != CFPQ_OK) return st;
                        ++products;
                        ++launched;
                        ++delta;
                        (h1.mode == kModeDense ? dense : sparse) += 1;
                    }
                    if (h2.mode != kModeSkip) {  // B x D_C
                        if (h2.mode == kModeCols) st = refresh(q.left);
                        if (st == CFPQ_OK)
                            st = product_by(h2.mode, T_of(q.left), kept(q.left), Dm + q.right * mw, nullptr, Pm);
                        if (st != CFPQ_OK) return st;
                        ++products;
                        ++launched;
                        ++delta;
                        (h2.mode == kModeDense ? dense : sparse) += 1;
                    }
                }
            }
            CFPQ_HIP(launch_sweep(sg, b, L, static_cast<int32_t>(t & 0x7FFFFFFF), p_mask, true, false, s));
            CFPQ_HIP(launch_sweep_report(b, static_cast<int32_t>(t & 0x7FFFFFFF), &rep[0], s));
            CFPQ_HIP(await_report(&rep[0], static_cast<int32_t>(t & 0x7FFFFFFF), s));
            const int64_t before = last.products;
            last = rep[0];
            any_prev = last.any;
            for (int h = 0; h < sg.n_dyn; ++h) {
                dnnz[h] = last.gained[h];
                nnz[h] += last.gained[h];
                if ((any_prev >> h) & 1u) tt_fresh[h] = false;
            }
            if (jlog.f)
                log_loop(t, any_prev, last.products - before + launched, last.products + products,
                         last.sparse + sparse, last.delta + delta);
            if (any_prev == 0) {
                converged = true;
                break;
            }
        }
        products += last.products;
        sparse += last.sparse;
        delta += last.delta;
    }
    CFPQ_HIP(hipEventRecord(ev1, s));
    CFPQ_HIP(hipEventSynchronize(ev1));
    drain.armed = false;
    if (last.bad_edges)
        return fail(CFPQ_EINVAL, std::to_string(last.bad_edges) + " device edges have an id out of range");
    float ms = 0.f;
    CFPQ_HIP(hipEventElapsedTime(&ms, ev0, ev1));
    if (stats) {
        std::memset(stats, 0, sizeof(*stats));
        stats->iterations = last.loops;
        stats->products = products;
        const double npad = static_cast<double>(L.npad);
        stats->bitops = 2.0 * npad * npad * npad * static_cast<double>(dense);
        stats->sparse_products = sparse;
        stats->delta_products = delta;
        stats->device_ms = ms;
        stats->path_used = path;
        stats->converged = converged ? 1 : 0;
    }
    if (jlog.f) {
        char buf[512];
        std::snprintf(buf, sizeof(buf),
                      "{\"event\": \"closure\", \"n\": %d, \"edges\": %lld, \"nonterminals\": %d, "
                      "\"path\": \"%s\", \"hybrid\": 1, \"schedule\": \"inplace\", \"captured\": 0, "
                      "\"iterations\": %lld, \"products\": %lld, \"sparse_products\": %lld, "
                      "\"delta_products\": %lld, \"converged\": %d, \"device_ms\": %.4f}",
                      graph->n_nodes, static_cast<long long>(graph->n_edges), n_nt, path_name(path),
                      static_cast<long long>(last.loops), static_cast<long long>(products),
                      static_cast<long long>(sparse), static_cast<long long>(delta), converged ? 1 : 0,
                      static_cast<double>(ms));
        jlog.line(buf);
    }
    if (!converged) return fail(CFPQ_ENOTCONV, "max_iters reached before the fixpoint");
    return CFPQ_OK;
}

}  // namespace cfpq
