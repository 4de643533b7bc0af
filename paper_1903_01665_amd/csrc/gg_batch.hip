// gg_batch.hip -- batched SSSP/BFS over many independent instances
// (declared in include/gg.h).
//
// Instances of one algorithm and one graph class are concatenated into a
// single graph: instance j's vertex v becomes base_j + v and its edges keep
// their heads inside the instance, so every instance is a set of components
// of its own.  One multi-source traversal of the group (one source per
// instance) then computes each instance exactly as a separate call would.
// The group is a regular uploaded graph with its own workspace and stream;
// after its first (eager) run its launch sequence -- init, seed and a fixed
// number of rounds -- is captured in a HIP graph and replayed by later runs.

#include <algorithm>
#include <cstring>
#include <map>
#include <new>
#include <tuple>
#include <vector>

#include "gg_runtime.h"

using namespace gg;

namespace {

struct Group {
    int algo = 0;
    std::vector<int> members;  // instance indices, in order
    std::vector<long long> vbase;
    long long n = 0, m = 0;
    long long out_off = 0;     // first output slot of the group
    gg_graph g = nullptr;
    int* sources = nullptr;    // device, concatenated ids
    int nsrc = 0;
    gg_opts opts{};            // variant the group runs
    hipStream_t stream = nullptr;
    hipEvent_t done = nullptr;
    int* h_ctl = nullptr;      // pinned copy of (done, rounds) after a replay
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    int* graph_out = nullptr;  // output pointer baked into the captured graph
    int r_cap = 0;
    int last_rounds = 0;
};

}  // namespace

struct gg_batch_s {
    std::vector<Group> groups;
    std::vector<int> order;  // of the groups' launches
    std::vector<long long> v_off;
    long long total_n = 0, total_m = 0;
    uint32_t flags = 0;
    hipEvent_t start = nullptr;
};

namespace {

bool valid_instance(const gg_instance& x, int* max_deg) {
    if ((x.algo != GG_ALGO_SSSP && x.algo != GG_ALGO_BFS) || x.n < 1 || x.m < 0 ||
        x.m >= (1LL << 31) || !x.row_ptr || (x.m > 0 && !x.col) || x.source < 0 ||
        x.source >= x.n || (x.algo == GG_ALGO_SSSP && x.m > 0 && !x.w))
        return false;
    if (x.row_ptr[0] != 0 || x.row_ptr[x.n] != x.m) return false;
    int md = 0;
    for (int v = 0; v < x.n; ++v) {
        const int d = x.row_ptr[v + 1] - x.row_ptr[v];
        if (d < 0) return false;
        md = d > md ? d : md;
    }
    *max_deg = md;
    return true;
}

// Whether an instance may be traversed by one workgroup.  Not where even degrees
// (small_even) or, above 2^16 edges, few edges a vertex and no long row make a
// deep graph likely: a 160 x 160 grid takes one workgroup 3.7 ms, the rounds of
// all CUs 2.5.
bool fits_workgroup(const gg_instance& x, int max_deg) {
    int32_t sc = 0, kc = 0, dc = 0;
    gg_class_of(x.m, x.n, max_deg, -1, &sc, &kc, &dc);
    return x.n <= kSmallN && x.m <= kSmallM && (x.m <= 65536 || x.m >= 6LL * x.n || kc > 0) &&
           !small_even(x.n, x.m, max_deg);
}

// Whether `count` instances, m edges in all, are one launch, where the longest of
// those that may hold it up has `longest` (0: none).
//
// A CU needs 7-10 us for the smallest, so beyond some number the rounds of all CUs
// together are faster; in us, rounds / one launch:
//   edges each        250           1000          4000          8000
//   SSSP   64      105 /  86      96 / 105      97 / 200     100 / 324
//        1024      162 /  84     171 / 123     246 / 269     295 / 465
//        4096      206 /  90     304 / 149     516 / 374     783 / 699
//   BFS  1024       77 /  81      82 / 103     123 / 201     172 / 340
//        4096       90 /  84     134 / 115     232 / 242     303 / 443
// A launch lasts as long as its longest instance, so a few large ones are not
// (SSSP of uniform graphs takes long either way: 131,072 edges 216-310 / 255):
//   instances          1             4             8            16
//   SSSP 80000     108 / 136     118 / 137     138 / 137     270 / 137
//       131072     128 / 197     148 / 194     288 / 195     426 / 196
//   BFS  80000      81 /  99      83 / 101      83 / 100     120 / 100
//       131072      85 / 143      91 / 143      89 / 144     103 / 146
// (They cost the batch a launch of their own beside it, so up to 2^16 edges they
// stay: 24 instances of scales 10 and 11, 125 us together, 134 apart.)
constexpr long long kFewEdges = 65536;

bool longest_ok(int algo, long long m, long long longest) {
    return longest <= kFewEdges || m >= (algo == GG_ALGO_SSSP ? 6 : 20) * longest;
}

bool one_launch(int algo, long long count, long long m, long long longest) {
    const double each = (double)m / (double)std::max(1LL, count);
    return m <= kSmallGroupM && longest_ok(algo, m, longest) &&
           (double)count <= (algo == GG_ALGO_SSSP ? 512 + 2.5 * each : each * each / 4096);
}

bool holds_up(const gg_instance& x, int max_deg) {
    int32_t sc = 0, kc = 0, dc = 0;
    gg_class_of(x.m, x.n, max_deg, -1, &sc, &kc, &dc);
    return x.algo == GG_ALGO_BFS || kc > 0;
}

void destroy_group(Group& G) {
    if (G.stream) (void)hipStreamSynchronize(G.stream);
    if (G.exec) (void)hipGraphExecDestroy(G.exec);
    if (G.graph) (void)hipGraphDestroy(G.graph);
    if (G.g) gg_graph_free(G.g);
    if (G.sources) (void)hipFree(G.sources);
    if (G.h_ctl) (void)hipHostFree(G.h_ctl);
    if (G.done) (void)hipEventDestroy(G.done);
    if (G.stream) (void)hipStreamDestroy(G.stream);
    G = Group{};
}

// Capture init, seed and G.r_cap rounds of the group into a HIP graph.
int capture(Group& G, int* out) {
    if (G.exec) (void)hipGraphExecDestroy(G.exec);
    if (G.graph) (void)hipGraphDestroy(G.graph);
    G.exec = nullptr;
    G.graph = nullptr;
    Plan p;
    int rc = plan_make(G.g, nullptr, G.algo, 0, G.sources, G.nsrc, &G.opts, out, G.stream, &p);
    if (rc != GG_OK) return rc;
    hipError_t e;
    // the tag is reserved before the capture begins; every replay uses it
    const int base = reserve_stamps(p.ws, G.stream, (long long)G.r_cap + 1, &e);
    if (e != hipSuccess) return GG_EHIP;
    p.R.epoch = base;
    if (hipStreamBeginCapture(G.stream, hipStreamCaptureModeThreadLocal) != hipSuccess)
        return GG_EHIP;
    e = plan_init(p);
    for (int r = 0; r < G.r_cap && e == hipSuccess; ++r) e = plan_round(p, r);
    hipGraph_t graph = nullptr;
    const hipError_t e2 = hipStreamEndCapture(G.stream, &graph);
    if (e != hipSuccess || e2 != hipSuccess || !graph) {
        if (graph) (void)hipGraphDestroy(graph);
        return GG_EHIP;
    }
    if (hipGraphInstantiate(&G.exec, graph, nullptr, nullptr, 0) != hipSuccess) {
        (void)hipGraphDestroy(graph);
        return GG_EHIP;
    }
    G.graph = graph;
    G.graph_out = out;
    return GG_OK;
}

}  // namespace

extern "C" {

int gg_batch_create(const gg_instance* inst, int32_t count, uint32_t flags, void* stream,
                    gg_batch* out) {
    if (!out) return GG_EINVAL;
    *out = nullptr;
    if (!inst || count < 1) return GG_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    // group key: algorithm and graph class (size, skew) of the instance.  The
    // instances that fit a workgroup are one group per algorithm, which runs as
    // one launch, unless they are too many for that, or too large together for a
    // graph, while those of a class may not be.  Few large ones stay out of it,
    // where no larger instance takes as long anyway.
    std::vector<int> max_deg((size_t)count);
    std::vector<char> fits((size_t)count), holds((size_t)count);
    std::vector<long long> large[2];  // edges of those that may hold the launch up
    long long fit_count[2] = {0, 0}, fit_n[2] = {0, 0}, fit_m[2] = {0, 0};
    bool all_fit = true;
    for (int i = 0; i < count; ++i) {
        if (!valid_instance(inst[i], &max_deg[i])) return GG_EINVAL;
        fits[i] = fits_workgroup(inst[i], max_deg[i]);
        holds[i] = holds_up(inst[i], max_deg[i]);
        all_fit = all_fit && fits[i];
        if (!fits[i]) continue;
        const int a = inst[i].algo;
        fit_count[a]++;
        fit_n[a] += inst[i].n;
        fit_m[a] += inst[i].m;
        if (holds[i]) large[a].push_back(inst[i].m);
    }
    bool one[2];
    long long most[2] = {kSmallM, kSmallM};  // edges of an instance of the one launch
    for (int a = 0; a < 2; ++a) {
        long long n = fit_n[a], m = fit_m[a], left = fit_count[a];
        std::sort(large[a].begin(), large[a].end());
        while (all_fit && !large[a].empty() && !longest_ok(a, m, large[a].back())) {
            most[a] = large[a].back() - 1;
            m -= large[a].back();
            left--;
            large[a].pop_back();
        }
        one[a] = left > 0 && n < (1LL << 31) && one_launch(a, left, m, 0);
    }
    std::map<std::tuple<int, int, int>, std::vector<int>> keys;
    for (int i = 0; i < count; ++i) {
        int32_t sc = 0, kc = 0, dc = 0;
        gg_class_of(inst[i].m, inst[i].n, max_deg[i], -1, &sc, &kc, &dc);
        const int a = inst[i].algo;
        if (flags & GG_BATCH_ONE_GROUP) sc = kc = 0;
        else if (fits[i] && one[a] && !(holds[i] && inst[i].m > most[a])) sc = kc = -1;
        keys[std::make_tuple(a, sc, kc)].push_back(i);
    }
    gg_batch b = new (std::nothrow) gg_batch_s();
    if (!b) return GG_ENOMEM;
    b->flags = flags;
    b->v_off.assign(count, 0);
    auto bail = [&](int code) {
        for (Group& G : b->groups) destroy_group(G);
        if (b->start) (void)hipEventDestroy(b->start);
        delete b;
        return code;
    };
    if (hipEventCreateWithFlags(&b->start, hipEventDisableTiming) != hipSuccess)
        return bail(GG_EHIP);
    long long out_off = 0;
    for (auto& kv : keys) {
        b->groups.emplace_back();
        Group& G = b->groups.back();
        G.algo = std::get<0>(kv.first);
        G.members = kv.second;
        for (int i : G.members) {
            G.vbase.push_back(G.n);
            G.n += inst[i].n;
            G.m += inst[i].m;
        }
        if (G.n >= (1LL << 31) || G.m >= (1LL << 31)) return bail(GG_EINVAL);
        const bool weighted = G.algo == GG_ALGO_SSSP;
        std::vector<int> row((size_t)G.n + 1), col((size_t)std::max(G.m, 1LL));
        std::vector<int> w(weighted ? (size_t)std::max(G.m, 1LL) : 0);
        std::vector<int> src;
        long long eb = 0;
        for (size_t k = 0; k < G.members.size(); ++k) {
            const gg_instance& x = inst[G.members[k]];
            const int vb = (int)G.vbase[k];
            for (int v = 0; v < x.n; ++v) row[vb + v] = (int)(eb + x.row_ptr[v]);
            for (long long e = 0; e < x.m; ++e) col[eb + e] = vb + x.col[e];
            if (weighted && x.m) std::memcpy(&w[eb], x.w, sizeof(int) * (size_t)x.m);
            src.push_back(vb + x.source);
            b->v_off[G.members[k]] = out_off + vb;
            eb += x.m;
        }
        row[G.n] = (int)eb;
        G.out_off = out_off;
        out_off += G.n;
        b->total_m += G.m;
        // the group's traversal starts from a device list of caller ids:
        // kept in the caller's vertex order
        int rc = gg_graph_upload((int)G.n, G.m, row.data(), col.data(),
                                 weighted ? w.data() : nullptr, GG_KEEP_ORDER, stream, &G.g);
        if (rc != GG_OK) return bail(rc);
        G.nsrc = (int)src.size();
        if (dalloc(&G.sources, src.size()) != hipSuccess ||
            hipMemcpyAsync(G.sources, src.data(), sizeof(int) * src.size(),
                           hipMemcpyHostToDevice, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return bail(GG_EHIP);
        if (hipEventCreateWithFlags(&G.done, hipEventDisableTiming) != hipSuccess ||
            hipHostMalloc(reinterpret_cast<void**>(&G.h_ctl), 2 * sizeof(int)) != hipSuccess)
            return bail(GG_EHIP);
        bool fit = true;
        long long longest = 0;
        for (int i : G.members) {
            fit = fit && fits[i];
            if (holds[i] && all_fit) longest = std::max<long long>(longest, inst[i].m);
        }
        if (fit && one_launch(G.algo, (long long)G.members.size(), G.m, longest)) {
            // the longest first, so that none of them starts last
            std::vector<int4> first;
            for (size_t k = 0; k < G.members.size(); ++k) {
                const gg_instance& x = inst[G.members[k]];
                const int vb = (int)G.vbase[k];
                first.push_back(make_int4(vb, vb + x.n, vb + x.source, (int)x.m));
                G.g->inst_lds = std::max(G.g->inst_lds, small_lds(G.algo, x.n, x.m));
            }
            std::stable_sort(first.begin(), first.end(),
                             [](const int4& a, const int4& b) { return a.w > b.w; });
            if (dalloc(&G.g->inst, first.size()) != hipSuccess ||
                hipMemcpyAsync(G.g->inst, first.data(), sizeof(int4) * first.size(),
                               hipMemcpyHostToDevice, s) != hipSuccess ||
                hipStreamSynchronize(s) != hipSuccess)
                return bail(GG_EHIP);
        }
        gg_resolve(G.g, G.algo, nullptr, &G.opts);
        // The table's choice is measured on single-source traversals.  A
        // group is one traversal from hundreds of sources over as many small
        // components: near-far rounds then follow the component that needs
        // the most buckets, while the repeated hub expansions the buckets
        // save belong to large skewed graphs (measured on 512 R-MAT
        // instances of scales 10-18: near-far with long-row deferral 18.4 ms
        // per run, the plain worklist 14.0 ms).  Groups run the worklist.
        if (G.opts.sched == GG_NEARFAR) {
            G.opts.sched = GG_ASYNC;
            G.opts.delta = 0;
            G.opts.far_degree = 0;
            G.opts.hops = 0;
        }
    }
    // The longest groups first: the host takes ~50 us to launch a replay, the
    // streams share four hardware queues, and a run lasts as long as the group
    // that ends last (48 R-MAT instances of scales 10-17: 1.55 ms; by algorithm
    // and ascending class 1.66-1.71).
    auto work = [&](int i) {
        const Group& G = b->groups[i];
        return (G.algo == GG_ALGO_SSSP ? 3 : 1) * G.m;
    };
    for (size_t i = 0; i < b->groups.size(); ++i) b->order.push_back((int)i);
    std::stable_sort(b->order.begin(), b->order.end(),
                     [&](int x, int y) { return work(x) > work(y); });
    for (int i : b->order)
        if (hipStreamCreateWithFlags(&b->groups[i].stream, hipStreamNonBlocking) != hipSuccess)
            return bail(GG_EHIP);
    b->total_n = out_off;
    *out = b;
    return GG_OK;
}

int gg_batch_run(gg_batch b, int32_t* out_dev, void* stream) {
    if (!b || !out_dev) return GG_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const bool graphs = !(b->flags & GG_BATCH_NO_GRAPH);
    if (hipEventRecord(b->start, s) != hipSuccess) return GG_EHIP;
    std::vector<char> replayed(b->groups.size(), 0);
    int status = GG_OK;
    // launch every group: replays go out at once; a group without a graph
    // (first run, other output, or graphs off) runs eagerly and is captured
    for (int i : b->order) {
        Group& G = b->groups[i];
        int* out = out_dev + G.out_off;
        if (hipStreamWaitEvent(G.stream, b->start, 0) != hipSuccess) return GG_EHIP;
        if (graphs && G.exec && G.graph_out == out) {
            Ctl* ctl = G.g->ws0->dev.ctl;
            if (hipGraphLaunch(G.exec, G.stream) != hipSuccess ||
                hipMemcpyAsync(G.h_ctl, ctl, 2 * sizeof(int), hipMemcpyDeviceToHost, G.stream) !=
                    hipSuccess ||
                hipEventRecord(G.done, G.stream) != hipSuccess)
                return GG_EHIP;
            replayed[i] = 1;
            continue;
        }
        int rc = run_multi(G.g, nullptr, G.algo, 0, G.sources, G.nsrc, &G.opts, out, G.stream);
        if (rc != GG_OK) status = rc;
        gg_stats st{};
        if (gg_last_stats(G.g, nullptr, &st) == GG_OK) G.last_rounds = st.iterations;
        if (rc == GG_OK && graphs) {
            // room for the rounds just used and a margin (asynchronous rounds
            // vary a little from run to run)
            G.r_cap = G.last_rounds + G.last_rounds / 4 + 2;
            rc = capture(G, out);
            if (rc != GG_OK) status = rc;
        }
        if (hipEventRecord(G.done, G.stream) != hipSuccess) return GG_EHIP;
    }
    // replays that stopped short of the end continue eagerly
    for (size_t i = 0; i < b->groups.size(); ++i) {
        if (!replayed[i]) continue;
        Group& G = b->groups[i];
        if (hipEventSynchronize(G.done) != hipSuccess) return GG_EHIP;
        if (G.h_ctl[0]) {
            G.last_rounds = G.h_ctl[1];
            continue;
        }
        Plan p;
        int rc = plan_make(G.g, nullptr, G.algo, 0, G.sources, G.nsrc, &G.opts,
                           out_dev + G.out_off, G.stream, &p);
        hipError_t e = hipSuccess;
        const int base = rc == GG_OK ? reserve_stamps(p.ws, G.stream, (long long)G.n + 3, &e) : 0;
        if (rc != GG_OK || e != hipSuccess) return rc != GG_OK ? rc : GG_EHIP;
        p.R.epoch = base;
        long long r_end = 0;
        rc = plan_drive(p, G.r_cap, base, base, &r_end);
        p.ws->epoch = (int)std::min<long long>((long long)base + r_end + 1, 1LL << 30);
        record_last(p, rc, r_end);
        if (rc != GG_OK) status = rc;
        G.last_rounds = (int)r_end;
        G.r_cap = (int)(r_end + r_end / 4 + 2);  // the next run recaptures
        if (G.exec) (void)hipGraphExecDestroy(G.exec);
        G.exec = nullptr;
        if (hipEventRecord(G.done, G.stream) != hipSuccess) return GG_EHIP;
    }
    for (Group& G : b->groups) {
        gg_ws ws = G.g->ws0;
        ws->last_stream = G.stream;
        ws->used = true;
        if (hipEventRecord(ws->finished, G.stream) != hipSuccess ||
            hipStreamWaitEvent(s, G.done, 0) != hipSuccess)
            return GG_EHIP;
    }
    return status;
}

int gg_batch_offsets(gg_batch b, int64_t* v_off) {
    if (!b || !v_off) return GG_EINVAL;
    for (size_t i = 0; i < b->v_off.size(); ++i) v_off[i] = b->v_off[i];
    return GG_OK;
}

int gg_batch_info(gg_batch b, int32_t* groups, int64_t* total_n, int64_t* total_m) {
    if (!b) return GG_EINVAL;
    if (groups) *groups = (int32_t)b->groups.size();
    if (total_n) *total_n = b->total_n;
    if (total_m) *total_m = b->total_m;
    return GG_OK;
}

int gg_batch_group(gg_batch b, int32_t g, int32_t* algo, int32_t* instances, int64_t* n,
                   int64_t* m, int32_t* mode, int32_t* sched, int32_t* mapping,
                   int32_t* captured_rounds, int32_t* last_rounds) {
    if (!b || g < 0 || g >= (int32_t)b->groups.size()) return GG_EINVAL;
    const Group& G = b->groups[g];
    if (algo) *algo = G.algo;
    if (instances) *instances = (int32_t)G.members.size();
    if (n) *n = G.n;
    if (m) *m = G.m;
    if (mode) *mode = G.opts.mode;
    if (sched) *sched = G.opts.sched;
    if (mapping) *mapping = G.opts.mapping;
    if (captured_rounds) *captured_rounds = G.exec ? G.r_cap : 0;
    if (last_rounds) *last_rounds = G.last_rounds;
    return GG_OK;
}

int gg_batch_free(gg_batch b) {
    if (!b) return GG_EINVAL;
    for (Group& G : b->groups) destroy_group(G);
    if (b->start) (void)hipEventDestroy(b->start);
    delete b;
    return GG_OK;
}

}  // extern "C"
