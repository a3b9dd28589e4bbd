// bsim_summarize.hip -- host driver of one batch summarization.
//
// Device round trips per call: one after staging (tile and hub counts), two
// in finalize (block and edge counts).  The refinement loop has none on grids
// of up to 16,384 workgroups: the host queues a few launches ahead of what the
// device reports through pinned memory, so a run of thousands of iterations
// (long k-chaining) costs only the kernels themselves plus a few early-exit
// launches.  Past that it has one per level, for the stop test's answer.
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <thread>

#include "bsim_api_internal.h"

namespace bsim {

void validate_params(const bsim_graph& graph, const bsim_params& p, bool directions) {
    if (graph.label_bytes != 2 && graph.label_bytes != 4)
        throw DeviceError{BSIM_E_INVALID, "label_bytes must be 2 or 4"};
    if (graph.mem_kind != BSIM_MEM_HOST && graph.mem_kind != BSIM_MEM_DEVICE)
        throw DeviceError{BSIM_E_INVALID, "unknown mem_kind"};
    if (graph.n_edges >= (1ull << 32))
        throw DeviceError{BSIM_E_UNSUPPORTED, "this library supports fewer than 2^32 edges"};
    if (graph.n_vertices >= 0xFFFFFFFFu)
        throw DeviceError{BSIM_E_UNSUPPORTED, "too many vertices"};
    if (!graph.row_off || !graph.type_off)
        throw DeviceError{BSIM_E_INVALID, "row_off and type_off are required"};
    if (graph.n_edges && (!graph.targets || !graph.labels))
        throw DeviceError{BSIM_E_INVALID, "targets and labels are required"};
    if (!(p.flags & BSIM_STOP_AT_FIXPOINT) && p.k_max > (1u << 24))
        throw DeviceError{BSIM_E_INVALID, "without a fixpoint test k_max must be finite (< 2^24)"};
    if (p.flags & ~(BSIM_STOP_AT_FIXPOINT | BSIM_KEEP_LEVELS | BSIM_UNTYPED | BSIM_RESULT_ON_HOST |
                    BSIM_NO_SUMMARY_EDGES | BSIM_BACKWARD | BSIM_BOTH_DIRECTIONS | BSIM_PREV_LEVEL_EDGES))
        throw DeviceError{BSIM_E_INVALID, "unknown flag bits"};
    if ((p.flags & BSIM_BACKWARD) && (p.flags & BSIM_BOTH_DIRECTIONS))
        throw DeviceError{BSIM_E_INVALID, "BSIM_BACKWARD and BSIM_BOTH_DIRECTIONS exclude each other"};
    if ((p.flags & BSIM_PREV_LEVEL_EDGES) && (p.flags & (BSIM_BACKWARD | BSIM_BOTH_DIRECTIONS)))
        throw DeviceError{BSIM_E_INVALID, "BSIM_PREV_LEVEL_EDGES is defined for the forward direction only"};
    if (!directions && (p.flags & (BSIM_BACKWARD | BSIM_BOTH_DIRECTIONS)))
        throw DeviceError{BSIM_E_UNSUPPORTED, "edge directions other than outgoing are supported by "
                                              "bsim_summarize without a state only"};
}

void upload_graph(const bsim_graph& in, Staged& g, Arena& arena, hipStream_t s, HostStaging* staging) {
    g.n = in.n_vertices;
    g.m = in.n_edges;
    g.label_bytes = in.label_bytes;
    if (in.mem_kind == BSIM_MEM_DEVICE) {
        g.row_off = in.row_off;
        g.tgt = in.targets;
        g.lab = in.labels;
        g.type_off = in.type_off;
        g.type_ids = in.type_ids;
        g.alive = in.alive;
        return;
    }
    const size_t n = in.n_vertices, m = in.n_edges;
    // type_off[n] tells how many type ids follow; read it from the host copy
    const size_t nt = in.type_off[n];
    // (the arrays one after the other, each from a 256-byte boundary)
    const void* from[6] = {in.row_off, in.type_off, in.type_ids, in.targets, in.labels, in.alive};
    const size_t bytes[6] = {(n + 1) * 4, (n + 1) * 4, nt * 4, m * 4, m * in.label_bytes, in.alive ? n : 0};
    size_t at[6], total = 0;
    for (int i = 0; i < 6; i++) {
        at[i] = total;
        total += (bytes[i] + 16 + 255) & ~size_t(255);
    }
    // A small graph goes up in one copy from pinned memory: five copies from
    // pageable memory, each through the runtime's staging, took 110 us of a
    // 1,000-vertex graph's 456.  Past a MiB the extra pass over the host's
    // arrays would cost more than the copies' overhead.
    uint8_t* dev = arena.alloc<uint8_t>(total);
    uint8_t* up = staging && total <= HostStaging::kSmall ? static_cast<uint8_t*>(staging->get_small()) : nullptr;
    if (up) {
        for (int i = 0; i < 6; i++)
            if (bytes[i]) memcpy(up + at[i], from[i], bytes[i]);
        hip_check(hipMemcpyAsync(dev, up, total, hipMemcpyHostToDevice, s), "upload graph");
    } else {
        for (int i = 0; i < 6; i++)
            if (bytes[i]) hip_check(hipMemcpyAsync(dev + at[i], from[i], bytes[i], hipMemcpyHostToDevice, s), "upload graph");
    }
    uint32_t* ro = reinterpret_cast<uint32_t*>(dev + at[0]);
    uint32_t* to = reinterpret_cast<uint32_t*>(dev + at[1]);
    uint32_t* ti = reinterpret_cast<uint32_t*>(dev + at[2]);
    uint32_t* tg = reinterpret_cast<uint32_t*>(dev + at[3]);
    void* lb = dev + at[4];
    uint8_t* al = in.alive ? dev + at[5] : nullptr;
    g.row_off = ro;
    g.type_off = to;
    g.type_ids = ti;
    g.tgt = tg;
    g.lab = lb;
    g.alive = al;
}

LoopResult run_refinement(bsim_ctx* ctx, const Staged& g, const bsim_params& p, RunBuffers& rb,
                          LevelSink* sink, Arena& arena, uint32_t* rep_prev, bool use_timers) {
    hipStream_t s = ctx->stream;
    const bool stop = (p.flags & BSIM_STOP_AT_FIXPOINT) != 0;
    const bool untyped = (p.flags & BSIM_UNTYPED) != 0;
    if (sink && !sink->levels.empty()) rb.h[0] = sink->levels[0];
    launch_init(g, rb, untyped, s);
    if (rb.bc.gid && rb.small.n_small) {
        // the small graphs of a batch go to their stop levels now, each in one
        // workgroup; their per-level counts need history rows up to there
        // (with the fixpoint test a graph of n vertices stops by level max(n, 1))
        const uint64_t depth =
            stop ? std::min<uint64_t>(p.k_max, static_cast<uint64_t>(rb.small.max_n) + 1) : p.k_max;
        const uint64_t need = depth + 2;
        if (need > rb.bc.hist_cap) {
            const size_t G = rb.bc.n_graphs;
            uint32_t* nh = arena.alloc<uint32_t>(need * G);
            hip_check(hipMemsetAsync(nh, 0, need * G * 4, s), "history clear");
            hip_check(hipMemcpyAsync(nh, rb.bc.hist, static_cast<size_t>(rb.bc.hist_cap) * G * 4,
                                     hipMemcpyDeviceToDevice, s), "history copy");
            rb.bc.hist = nh;
            rb.bc.hist_cap = static_cast<uint32_t>(need);
        }
        launch_small_graphs(g, rb, rb.small, p.k_max, stop, s);
    }

    LoopResult lr;
    const bool all = sink && !sink->levels.empty();
    // Launch k tests level k - lag_of(k).  With lag 1 the classes of every level
    // are a launch of their own after its hashes: the next launch knows them,
    // and a run hashes no level past its last.  With lag 2 (always with
    // tail_split_ppm = 0) they are tested beside the next level's hashes, in one
    // launch, and level k_done + 1 is hashed and dropped.  A run past kDeep
    // levels goes over to that: a level of a small graph costs its launches
    // (20,000 vertices in 20,000 levels 253 ms with two, 150 with one), and one
    // more level than 256 hardly shows.  Large grids pay their work, not the
    // launch.
    constexpr uint64_t kDeep = 256;
    constexpr uint32_t kLargeGrid = 16384;
    const uint32_t full_grid = iteration_grid(g, 3, all);
    auto lag_of = [&](uint64_t kk) { return !ctx->tail_split_ppm || (kk > kDeep && full_grid <= kLargeGrid) ? 2u : 1u; };
    const uint64_t k_last = static_cast<uint64_t>(p.k_max) + lag_of(p.k_max + 1ull);
    // The host follows the run through the words that block 0 of every launch
    // writes to pinned memory, and queues at most `ahead` launches past the
    // last one it has seen: enough that the device never waits for the host,
    // few enough that a run of three or four levels does not queue twenty
    // launches that find it over (a check per chunk of launches did: 28
    // launches for three levels, 195 of the 690 us a 1,000-vertex graph
    // kept the device busy).  An early exit still dispatches its whole grid
    // (about 2 ns a workgroup), so past kLargeGrid workgroups, where one
    // would cost more than the host's round trip of some 10 us, the stop test
    // runs as a launch of one workgroup and the host waits for its answer.
    const bool large = full_grid > kLargeGrid || ctx->chunk_max == 1;
    const uint32_t ahead = std::min<uint32_t>(ctx->chunk_max, 4);
    uint64_t* const report = ctx->report_host;
    for (uint32_t i = 0; i < kReportRing; i++) report[i] = 0;
    bool done = false, prev_taken = false;
    uint64_t seen = 0;  // launches whose word the host has read
    auto read_report = [&](uint64_t kk, bool wait) {
        volatile uint64_t* w = &report[kk & (kReportRing - 1)];
        const uint32_t tag = report_tag(static_cast<uint32_t>(kk));
        uint64_t x = 0;
        for (uint32_t spin = 1;; spin++) {
            x = *w;
            if (static_cast<uint32_t>(x >> 32) >> 3 == tag >> 3) break;
            if (!wait) return false;
            if (spin % 64 == 0) std::this_thread::yield();
            if (spin % 16384 == 0) {
                // the device is done (or has failed) without a word
                const hipError_t e = hipStreamQuery(s);
                if (e == hipErrorNotReady) continue;
                hip_check(e, "refinement");
                x = *w;
                if (static_cast<uint32_t>(x >> 32) >> 3 == tag >> 3) break;
                throw DeviceError{BSIM_E_DEVICE, "refinement did not report its stop test"};
            }
        }
        seen = kk;
        const uint32_t flags = static_cast<uint32_t>(x >> 32);
        if (flags & kReportError)
            throw DeviceError{BSIM_E_DEVICE, "a hub hash bucket could not be split to fit its table"};
        const uint32_t lag = lag_of(kk);
        // (launch kDeep + 1 tests the level that the one before it tested)
        if (!rb.bc.gid && kk == lr.blocks_per_iter.size() + lag) lr.blocks_per_iter.push_back(static_cast<uint32_t>(x));
        if (flags & kReportDone) {
            done = true;
            lr.k_done = static_cast<uint32_t>(kk - lag);
            lr.fixpoint = flags & kReportFixpoint ? 1u : 0u;
        }
        return true;
    };
    std::vector<hipEvent_t> timers;  // (start, after hashes, after hubs, after the split) per timed launch
    std::vector<uint32_t> timed_k;   // the launches timed
    struct TimerGuard {
        std::vector<hipEvent_t>& t;
        ~TimerGuard() {
            for (hipEvent_t e : t) (void)hipEventDestroy(e);
        }
    } timer_guard{timers};
    auto issue = [&](uint32_t kk) {
        if (all) {
            // keep every level: iteration kk reads levels[kk-1], writes levels[kk]
            const uint32_t top = static_cast<uint32_t>(sink->levels.size()) - 1;
            rb.h[(kk - 1) & 1] = sink->levels[std::min(kk - 1, top)];
            rb.h[kk & 1] = sink->levels[std::min(kk, top)];
        }
        if (rb.bc.gid && kk + 1ull > rb.bc.hist_cap) {
            // launch kk writes level kk of the per-graph history: grow it
            // while no launch is in flight
            hip_check(hipStreamSynchronize(s), "history sync");
            const uint64_t cap = std::max<uint64_t>(2ull * rb.bc.hist_cap, kk + 1ull);
            const size_t G = rb.bc.n_graphs;
            uint32_t* nh = arena.alloc<uint32_t>(cap * G);
            hip_check(hipMemsetAsync(nh, 0, cap * G * 4, s), "history clear");
            hip_check(hipMemcpyAsync(nh, rb.bc.hist, static_cast<size_t>(rb.bc.hist_cap) * G * 4,
                                     hipMemcpyDeviceToDevice, s), "history copy");
            rb.bc.hist = nh;
            rb.bc.hist_cap = static_cast<uint32_t>(cap);
        }
        const uint32_t lag = lag_of(kk);
        if (rb.bc.gid) launch_graph_stop(rb, kk, lag, p.k_max, stop, s);
        const bool hashes = kk <= p.k_max;
        const bool splits = lag == 2 && kk >= 2 && kk - 1 <= p.k_max;  // level kk-1, whose split launch was left out
        if (!hashes) {
            launch_iteration(g, rb, kk, lag, p.k_max, stop, all, report,
                             splits ? IterParts::kSplit : IterParts::kStopTest, s);
            return;
        }
        if (large) {
            launch_iteration(g, rb, kk, lag, p.k_max, stop, all, report, IterParts::kStopTest, s);
            read_report(kk, true);
            if (done) return;
        }
        hipEvent_t et[4] = {nullptr, nullptr, nullptr, nullptr};
        const bool timed = use_timers && ctx->time_launches && kk % ctx->time_launches == 0;
        auto mark = [&](int i) {
            if (timed) hip_check(hipEventRecord(et[i], s), "event");
        };
        if (timed) {
            timed_k.push_back(kk);
            for (hipEvent_t& e : et) {
                hip_check(hipEventCreate(&e), "event");
                timers.push_back(e);
            }
        }
        mark(0);
        launch_iteration(g, rb, kk, lag, p.k_max, stop, all, large ? nullptr : report,
                         splits ? IterParts::kHashesAndSplit : IterParts::kHashes, s);
        mark(1);
        launch_hubs(g, rb, kk, s);
        mark(2);
        if (rep_prev && kk == p.k_max && g.n) {
            // the (k_max-1)-classes, or the final ones of a run that stopped
            // earlier at a fixpoint
            hip_check(hipMemcpyAsync(rep_prev, rb.rep, static_cast<size_t>(g.n) * 4, hipMemcpyDeviceToDevice, s),
                      "previous classes");
            prev_taken = true;
        }
        if (lag_of(kk + 1ull) == 1) launch_split(g, rb, kk, s);
        mark(3);
        lr.launches++;
        if (lag == 1) lr.split_launches++;
    };
    try {
        for (uint64_t kk = 1; kk <= k_last && !done; kk++) {
            issue(static_cast<uint32_t>(kk));
            while (!done && seen < kk && read_report(seen + 1, seen + ahead <= kk)) {
            }
        }
        while (!done && seen < k_last) read_report(seen + 1, true);
        if (!done) throw DeviceError{BSIM_E_DEVICE, "refinement did not reach its stop test"};
    } catch (...) {
        (void)hipStreamSynchronize(s);
        throw;
    }
    // launches past the last hashed level return at once
    if (!timers.empty()) hip_check(hipStreamSynchronize(s), "launch timers");
    for (size_t i = 0; 4 * i + 3 < timers.size(); i++) {
        if (timed_k[i] > lr.k_done + lag_of(timed_k[i]) - 1) break;
        float t[3] = {0.f, 0.f, 0.f};
        for (int j = 0; j < 3; j++)
            hip_check(hipEventElapsedTime(&t[j], timers[4 * i + j], timers[4 * i + j + 1]), "launch timer");
        lr.ms_kernels += t[0] + t[2];
        lr.ms_hub_kernels += t[1];
        lr.n_timed++;
    }
    // k_max = 0, or a run whose stop was seen before launch k_max: the final
    // classes (level 0, or a fixpoint's)
    if (rep_prev && !prev_taken && g.n)
        hip_check(hipMemcpyAsync(rep_prev, rb.rep, static_cast<size_t>(g.n) * 4, hipMemcpyDeviceToDevice, s),
                  "previous classes");
    if (rb.bc.gid) {  // batched: counts and final buffers are per graph
        lr.h_final = nullptr;
        return lr;
    }
    if (sink && !sink->levels.empty())
        lr.h_final = sink->levels[std::min<size_t>(lr.k_done, sink->levels.size() - 1)];
    else
        lr.h_final = rb.h[lr.k_done & 1];
    return lr;
}

bsim_result* make_result(bsim_ctx* ctx, const Staged& g, const LoopResult& lr, const uint64_t* h,
                         FinalOut& fo, Arena& keep, uint32_t flags, uint64_t* hashes_preset) {
    hipStream_t s = ctx->stream;
    bsim_result* r = new bsim_result();
    ResultPriv* p = new ResultPriv();
    memset(r, 0, sizeof(*r));
    r->priv = p;
    p->device = ctx->device;
    p->stream = s;
    p->blocks_per_iter = lr.blocks_per_iter;
    r->n_vertices = g.n;
    r->k_done = lr.k_done;
    r->fixpoint = lr.fixpoint;
    r->n_blocks = fo.n_blocks;
    r->n_summary_edges = fo.n_se;
    r->n_iter_launches = lr.launches;
    r->ms_iter_kernels = lr.ms_kernels;
    r->ms_hub_kernels = lr.ms_hub_kernels;
    r->n_timed_launches = lr.n_timed;
    r->n_split_launches = lr.split_launches;
    r->blocks_per_iter = p->blocks_per_iter.data();
    uint64_t* hashes = hashes_preset ? hashes_preset : keep.alloc<uint64_t>(g.n);
    if (g.n) hip_check(hipMemcpyAsync(hashes, h, static_cast<size_t>(g.n) * 8, hipMemcpyDeviceToDevice, s),
                       "hashes");
    void* dev[] = {hashes, fo.block_ids, fo.block_sizes, fo.se_src, fo.se_label, fo.se_dst};
    if (flags & BSIM_RESULT_ON_HOST) {
        const size_t sizes[] = {static_cast<size_t>(g.n) * 8, static_cast<size_t>(g.n) * 4,
                                static_cast<size_t>(fo.n_blocks) * 4, fo.n_se * 4, fo.n_se * 4, fo.n_se * 4};
        void* host[6];
        p->host = host_arrays(ctx, dev, sizes, host);
        keep.release();
        r->mem_kind = BSIM_MEM_HOST;
        r->hashes = static_cast<uint64_t*>(host[0]);
        r->block_ids = static_cast<uint32_t*>(host[1]);
        r->block_sizes = static_cast<uint32_t*>(host[2]);
        r->se_src = static_cast<uint32_t*>(host[3]);
        r->se_label = static_cast<uint32_t*>(host[4]);
        r->se_dst = static_cast<uint32_t*>(host[5]);
    } else {
        for (void* q : dev) {
            p->device_ptrs.push_back(q);
            keep.detach(q);
        }
        r->mem_kind = BSIM_MEM_DEVICE;
        r->hashes = hashes;
        r->block_ids = fo.block_ids;
        r->block_sizes = fo.block_sizes;
        r->se_src = fo.se_src;
        r->se_label = fo.se_label;
        r->se_dst = fo.se_dst;
    }
    return r;
}

bsim_result* summarize_graph(bsim_ctx* ctx, const bsim_graph& graph, const bsim_params& p,
                             const std::vector<uint32_t>* labels) {
    validate_params(graph, p, true);
    hipStream_t s = ctx->stream;
    Arena arena(s), keep(s);
    ctx_back_arena(ctx, arena);
    hipEvent_t ev[4];
    for (auto& e : ev) hip_check(hipEventCreate(&e), "event");
    struct EvGuard {
        hipEvent_t* e;
        ~EvGuard() {
            for (int i = 0; i < 4; i++) (void)hipEventDestroy(e[i]);
        }
    } guard{ev};
    hip_check(hipEventRecord(ev[0], s), "event");
    Staged g;
    upload_graph(graph, g, arena, s, &ctx->staging);
    g.hub_table_slots = ctx->hub_table_slots;
    stage_graph(g, ctx->stage_host, arena, s);
    // direction / label parameterizations: refine the view h, take the
    // summary edges from the kept edges f
    const bool view = labels || (p.flags & (BSIM_BACKWARD | BSIM_BOTH_DIRECTIONS));
    DirectedView dv;
    if (view) {
        direction_view(g, p.flags, labels, !(p.flags & BSIM_NO_SUMMARY_EDGES), dv, ctx->stage_host, arena, s);
    }
    const Staged& gr = view ? dv.h : g;
    const Staged& gf = view ? dv.f : g;
    RunBuffers rb;
    alloc_run_buffers(gr, rb, arena, s);
    hip_check(hipEventRecord(ev[1], s), "event");
    const bool prev_edges = (p.flags & BSIM_PREV_LEVEL_EDGES) != 0;
    uint32_t* rep_prev = prev_edges ? arena.alloc<uint32_t>(gr.n + 1) : nullptr;
    LoopResult lr = run_refinement(ctx, gr, p, rb, nullptr, arena, rep_prev);
    hip_check(hipEventRecord(ev[2], s), "event");
    FinalOut fo;
    fo.n_blocks = lr.blocks_per_iter.back();
    // (at a fixpoint the previous level's count is the same)
    fo.n_prev_blocks = lr.blocks_per_iter[lr.k_done && lr.k_done == p.k_max ? lr.k_done - 1 : lr.k_done];
    if (prev_edges)
        finalize_prev_level(gf, rb.rep, rep_prev, !(p.flags & BSIM_NO_SUMMARY_EDGES), fo, ctx->final_host, arena, keep,
                            s);
    else
        finalize(gf, rb.rep, !(p.flags & BSIM_NO_SUMMARY_EDGES), fo, ctx->final_host, arena, keep, s);
    bsim_result* r = make_result(ctx, g, lr, lr.h_final, fo, keep, p.flags);
    hip_check(hipEventRecord(ev[3], s), "event");
    hip_check(hipEventSynchronize(ev[3]), "event");
    (void)hipEventElapsedTime(&r->ms_stage, ev[0], ev[1]);
    (void)hipEventElapsedTime(&r->ms_iterate, ev[1], ev[2]);
    (void)hipEventElapsedTime(&r->ms_finalize, ev[2], ev[3]);
    (void)hipEventElapsedTime(&r->ms_total, ev[0], ev[3]);
    ctx_note_demand(ctx, arena);
    return r;
}

}  // namespace bsim
