// gg_internal.h -- structures shared by the kernels and the host runtime of
// libgg.  Not part of the public ABI (include/gg.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gg {

constexpr int kInf = 2147483647;
constexpr int kWave = 64;
constexpr int kTile = 64;            // vertices per frontier tile (one wavefront)
constexpr int kMaxStatBlocks = 4096; // per-block statistics slots
// rows longer than the graph's heavy threshold are chunked (balanced
// mapping): 16 on graphs whose largest out-degree is at least 128 times the
// mean, 32 on the others (measured on MI355X: a lower threshold moves more
// edges of a skewed graph into full-wavefront chunks, while on a uniform
// graph it cuts short rows into underfilled chunks)
constexpr int kHeavySkewed = 16;
constexpr int kHeavyUniform = 32;
constexpr int kChunk = 512;          // most edges per heavy-row chunk
constexpr int kKinds = 3;            // statistics kinds: round, heavy chunks, auxiliary
constexpr int kItemTiles = 8;        // most tiles of a frontier work item
constexpr int kFillWaves = 8192;     // wavefronts that fill the device (256 CUs x 32)
// Hooking passes of CC by union-find and, for all but the first, the share of
// the vertices they look from: by the neighbours a vertex has (ms / n, both
// directions).  Trees of a sparse graph touch in few places, so three passes leave
// many apart for the last phase; with more neighbours they join most.  All of CC,
// us, uniform graphs, three passes / five:
//   neighbours      1           1.5          2           2.8         4           7.8
//   2^18       152 / 161   399 / 151    380 / 152   175 / 150   134 / 150   138 / 150
//   2^20       194 / 225   541 / 241   1268 / 259   233 / 259   223 / 266   228 / 264
//   2^22       487 / 649   737 / 757   1442 / 865  1093 / 986   761 / 1129  819 / 1080
// With 8 neighbours and more it is enough to look from one vertex in eight after
// the first pass (16 neighbours, 2^22 vertices: 521 us, from all of them 915).
struct UfPlan {
    int passes, share;
};
inline UfPlan uf_plan(long long n, long long ms) {
    if (ms >= 8 * n) return UfPlan{3, 8};
    return UfPlan{ms >= 3 * n ? 3 : 5, 1};
}
constexpr int kUfLong = 7;
constexpr int kUfSteps = 8;          // steps of a compression's walks but in the last
constexpr int kSmallSteps = 16;      // ... and of a walk in LDS between two barriers
constexpr int kXcd = 8;              // accelerator dies; workgroups go to them round-robin
// Tiles per frontier work item, as a shift: the most (up to kItemTiles) that
// still leave an item for each of kFillWaves wavefronts.  Graphs of 4M
// vertices and more fill the device with 8-tile items, the best size measured
// there; on an R-MAT graph of 2^18 vertices 8-tile items kept 512 wavefronts
// busy and a dense worklist round took 106 us, with one-tile items 25 us.
inline int item_shift_for(long long ntiles) {
    int sh = 0;
    while ((2 << sh) <= kItemTiles && (ntiles >> (sh + 1)) >= kFillWaves) ++sh;
    return sh;
}

// Edges per heavy-row chunk: the least power of two from 128 that cuts the
// graph into at most four chunks for each of kFillWaves wavefronts: 256 above 2^22
// edges, 512 above 2^23.  With 512-edge chunks and 64 chunks a wavefront the dense
// chunk rounds of an R-MAT graph of 2^22 edges took 148 and 97 us (132 blocks); with
// 128-edge chunks, four a wavefront, 84 and 73 us: what is left there is the rate of
// its atomics (27 G/s at most on this device, about 8 G/s on skewed heads, whatever
// the scope; plain loads and stores run at 60-400 G/s).  On larger graphs the size
// matters less, and the list of chunks is shorter with long ones (8 bytes each).  R-MAT,
// us with 128, 256 and 512: SSSP 2^24 edges 608, 636, 645, 2^26 1568, 1574, 1605; BFS
// 2^24 232, 230, 225, 2^26 505, 493, 499.
inline int chunk_for(long long m) {
    int c = 128;
    while (c < kChunk && m / c > 4 * kFillWaves) c *= 2;
    return c;
}

// Whole traversals in one workgroup: the most vertices (4 bytes of LDS each),
// the most edges of an instance of a batch and of a graph traversed alone, and
// threads.  One CU against a launch per round, in us, alone:
//                        SSSP         BFS        CC
//   R-MAT     2^14 edges  57 / 129    42 / 80    30 / 106
//   R-MAT     2^16        87 / 136    59 / 81    58 / 106
//   R-MAT     2^17       156 / 141    84 / 96    96 / 106
//   uniform   2^14        60 / 125    37 / 59    30 / 92
//   uniform   2^16       135 / 175    61 / 60    58 / 95
//   uniform   2^17       227 / 199    81 / 62    94 / 97
//   32 x 32 grid         107 / 331    94 / 133   25 / 127
constexpr int kSmallN = 32768;
constexpr long long kSmallM = 131072;
inline long long small_max_edges(int algo) { return algo == 1 ? 32768 : 65536; }
// ... and where the table does not tell: SSSP and BFS only where the graph is not
// known or likely to be deep, nor skewed and so wide that one CU takes longer than
// the few rounds.  us, one CU / a launch per round:
//   probed (grids, sc: with shortcuts)    edges   levels       SSSP          BFS
//     32 x 32 sc                           4002       31     95 /  152    87 / 109
//     40 x 40                              6240       77    207 /  223   186 / 166
//     64 x 32 sc                           8076       49    146 /  199   119 / 121
//     56 x 56 sc                          12432       47    237 /  242   178 / 153
//     64 x 64                             16128      125    353 /  321   286 / 237
//     126 x 126 sc                        63578      100    919 /  397
//     4 x 500                              6992      502   1919 / 1320  1136 / 963
//     uniform, 8000 vertices              16000       18    107 /  159    98 / 104
//     uniform, 16384 vertices             32768       21    152 /  167   131 / 104
//     uniform, 30000 vertices             40000       41    285 /  240
//   not probed, even degrees:  110 x 110 grid  1448 / 1427   126 x 126       1911 / 1658
//                      16 x 1000 grid         12937 / 7749   90 x 90          910 / 1208
//                      (random graphs of 2 and 4 edges a vertex 138 / 295, 151 / 198)
//   skewed:            star of 16,384            51 / 55     of 32,768         72 / 57
constexpr int kSmallEvenN = 12000;
constexpr int kSmallSkewedN = 20480;
inline bool small_deep(int algo, long long m, int levels) {
    return levels > (algo == 1 ? 20 : 32) && (levels >= 256 || m > (algo == 1 ? 6144 : 12288));
}
inline bool small_even(long long n, long long m, long long max_deg) {
    return n > kSmallEvenN && m >= 2 * n && max_deg * n <= 2 * m;
}
constexpr int kSmallBlock = 1024;
// Edges of a batch's group up to which no edge number of a whole traversal passes
// the int range: a sweep counts in steps of four edges a thread, and looks a step
// ahead of one that may begin as far past the last edge.
constexpr long long kSmallGroupM = (1LL << 31) - 1 - 3 * 4 * kSmallBlock;
// Bytes of LDS: 4 per vertex, 2 bits of frontier, and SSSP and BFS 4 per chunk
// of a long row (rows of more than 64 edges in chunks of 256).
inline size_t small_lds(int algo, int n, long long m) {
    if (algo == 2) return sizeof(int) * (size_t)n;
    return sizeof(int) * ((size_t)n + 2 * (((size_t)n + 31) / 32) + (size_t)(m / 65 + m / 256 + 1));
}

// Vertices from which a pulled BFS round looks its in-neighbours up in a bitmap
// of the frontier (a bit per vertex, resident in every die's L2) instead of in
// the values, on graphs stored in the caller's order.  Values that outgrow the
// L2 are gathered at 62-76 G/s, the bits at ~230; the launch that makes them
// costs ~3 us a round whether it pulls or not.  Uniform graphs: 2^23 vertices and
// 2^26 edges 1.17 -> 0.84 ms, 2^22 and 2^25 0.92 -> 0.58, 2^21 and 2^24 0.44 ->
// 0.34 (values of 8 MB); a renumbered R-MAT graph gathers its hot values at
// 200 G/s as they are.  Graphs with wide levels are shallow: later rounds than
// the first kFrontBitsRounds look the values up, without the launch (a 1500 x 1500
// grid, whose 3000 rounds never pull: 32.9 ms so, 44.5 with it in all of them).
constexpr int kFrontBitsN = 1 << 21;
constexpr int kFrontBitsRounds = 32;

enum Kind { KIND_ROUND = 0, KIND_HEAVY = 1, KIND_AUX = 2 };

enum Algo { SSSP = 0, BFS = 1, CC = 2 };
enum Map { MAP_THREAD = 1, MAP_WAVE = 2, MAP_BALANCED = 3 };

// Loop-control block, one per workspace.  Kernels of one traversal read the
// slots written by earlier kernels of the same stream (kernel boundaries make
// them visible); slot r % 3 belongs to round r.
struct Ctl {
    int done;        // set by the first round kernel that finds nothing left to do
    int iters;       // rounds that ran, set together with done
    int changed[4];  // [r % 3]: round r updated or pushed something
    int bound[4];    // near-far schedule: [r % 3] = distance bound of round r
    int near_[4];    // near-far schedule: [r % 3] = round r pushed below its bound
    int grid[4];     // [r % 3] = grid of round r's round kernel (push counts below)
    int hgrid[4];    // [r % 3] = grid of round r's heavy kernel
    int pull[4];     // [r % 3] = round r took the dense form (BFS pull, CC edge sweep)
    int giant;       // CC by union-find: the root most sampled vertices have
    int hooked[8];   // ... and whether its hooking pass [k] hooked anything; [kUfLong]:
                     // round 3 left long rows to k_uf_long
    int taken;       // batch of whole traversals: instances taken beyond a workgroup's first
    int left[8];     // [k]: the compression before hooking pass [k] left a chain
};

// Per-block counters, summed on the host after a traversal; one array of
// kMaxStatBlocks slots per kernel kind.
struct Stat {
    long long edges, verts, updates, pushes;
    long long swept;  // edges read by the sweeps of a per-round CC schedule
};

// Waits for the loads of x here.  Loads under a lane mask are followed by a
// join where the compiler no longer knows how many are in flight, so each
// later use inside a branch of its own waits for everything outstanding --
// also the gathers, stores and atomics of the branches before it, which then
// run one after another (4096 x 4096 grid, SSSP: 19.95 ms so, 18.96 with the
// waits here; worklist on an R-MAT graph of 2^18 vertices 464 and 432 us).
template <int U>
__device__ __forceinline__ void landed(int (&x)[U]) {
#pragma unroll
    for (int j = 0; j < U; ++j) asm volatile("" : "+v"(x[j]));
}

// Device view of an uploaded graph.  Arrays are owned by the host-side
// handle.  The CSR keeps the input's row order; src is the edge-list form.
struct DevGraph {
    int n, m;
    const int* row;  // [n+1]
    const int* col;  // [m]
    const int* w;    // [m] or null
    const int* src;  // [m] source vertex of each edge
    // both-directions graph for CC (aliases row/col/src when the input is symmetric)
    int ms;
    const int* srow;
    const int* scol;
    const int* ssrc;
    // heavy rows (degree > heavy) as (row, first edge) chunks of `chunk` edges
    int heavy, chunk;
    const int2* hchunks;
    int n_hchunks;
    const int2* shchunks;
    int n_shchunks;
    bool symmetric;  // input already holds both directions of every edge
    // the edge list again, cut into kXcd parts by head vertex (equal edge
    // counts), each padded to a multiple of 4 with self-loops on vertex 0;
    // null when not built
    const int* psrc;
    const int* pcol;
    const int* pw;
    int poff[kXcd + 1];
    // in-edges with their weights (pull rounds of SSSP): row v of trow/tcol
    // lists the tails of v's in-edges, tw their weights; rows longer than
    // `heavy` are also cut into (row, first edge) chunks; null when not built
    const int* trow;
    const int* tcol;
    const int* tw;
    const int2* tchunks;
    int n_tchunks;
};

// Device view of a workspace: frontier flags (one byte per vertex, one per
// 64-vertex tile), two generations; the heavy frontier rows of a round as a
// bit per vertex, two generations; control; stats.
struct DevWs {
    unsigned char* vflag[2];
    unsigned char* tflag[2];
    unsigned* hbits[2];  // [(n + 31) / 32] each: round r marks its heavy rows in hbits[r & 1]
    Ctl* ctl;
    Stat* stat;
    int* pcount;  // [3][2][kMaxStatBlocks]: frontier size pushed per block of round r % 3
                  // (round, heavy): vertices, or with Round::fedges their row lengths
};

// Everything a round kernel needs.  Passed by value.
struct Round {
    DevGraph g;
    DevWs ws;
    int* val;    // dist or label, [n]
    int source;          // single source (when nsrc == 0)
    const int* sources;  // device list of sources of a multi-source traversal
    int nsrc;
    int r;       // round (sweep, level) index
    int epoch;   // tag of this traversal: grows across the traversals of a workspace
    int* host_done; // pinned host word: set to `epoch` by the kernel that finds the end
    unsigned long long* host_round; // pinned: epoch << 32 | rounds reached (null: not reported)
    int mapping; // Map
    int jump;    // CC: apply the label[label[v]] shortcut
    int delta;   // SSSP near-far schedule: bucket width (0 = plain worklist rounds)
    int fedges;  // CC per-round dense/sparse choice: push counts are the row lengths
                 // (both-directions CSR) of the pushed vertices, and edge sweeps push
    int hops;    // worklist rounds (balanced mapping): passes of local expansion (0 = off)
    int far_degree; // near-far: only rows longer than this wait for the bound (0 = all)
    int pullmode;   // per-round schedule: dense rounds pull over in-edges (SSSP: trow;
                    // CC: the both-directions rows) instead of pushing or sweeping
    int direct_lists; // SSSP local expansion: list passes issue their atomics without a
                      // check load of the head value
    const int4* inst; // batch of whole traversals: first vertex, end, source and edges of
                      // each instance, [nsrc] (null otherwise)
    int front_bits; // direction-optimizing BFS: pulled rounds read the frontier as bits
    int item_shift; // log2 of the tiles of a frontier work item
    int* rmin;      // CC on a renumbered graph: per-label minimum of the caller's ids,
                    // filled with INT_MAX by the init kernel (null otherwise)
};

// Launch entry points (gg_kernels.hip).  Each returns the hipError_t of the
// launch.
hipError_t launch_init(const Round& R, int algo, bool async, int grid, int block, hipStream_t s);
hipError_t launch_seed(const Round& R, bool async, int grid, int block, hipStream_t s);
hipError_t launch_vsync(const Round& R, int algo, int grid, int block, hipStream_t s);
hipError_t launch_esync(const Round& R, int algo, int grid, int block, hipStream_t s);
hipError_t launch_vasync(const Round& R, int algo, int grid, int block, hipStream_t s);
hipError_t launch_easync(const Round& R, int algo, int grid, int block, hipStream_t s);
hipError_t launch_heavy(const Round& R, int algo, int grid, int block, hipStream_t s);
hipError_t launch_bfs_diropt(const Round& R, int grid, int block, hipStream_t s);
// ... and the bits of the frontier of round R.r, launched after round R.r - 1
hipError_t launch_front_bits(const Round& R, int grid, int block, hipStream_t s);
hipError_t launch_jump(const Round& R, int grid, int block, hipStream_t s);
hipError_t launch_cc_diropt(const Round& R, int grid, int block, hipStream_t s);
hipError_t launch_sssp_diropt(const Round& R, int grid, int block, hipStream_t s);
// CC by union-find (GG_UNIONFIND), round R.r: join, hook the roots, find the giant
// root, link the rest; the later hooking passes of round 1; the long rows of
// round 3 (graphs with heavy-row chunks); and the compression after each
hipError_t launch_uf(const Round& R, int grid, int block, hipStream_t s);
hipError_t launch_uf_hook(const Round& R, int pass, int share, int grid, int block,
                          hipStream_t s);
hipError_t launch_uf_long(const Round& R, int grid, int block, hipStream_t s);
// pass: the hooking pass before it (-1: none)
hipError_t launch_uf_compress(const Round& R, int pass, int grid, int block, hipStream_t s);
// A whole traversal of a graph of at most kSmallN vertices (or, with R.inst,
// those of a batch) in one launch, with the LDS that the largest needs; a batch
// clears the control block first
hipError_t launch_small(const Round& R, int algo, size_t lds, int grid, hipStream_t s);
hipError_t launch_small_begin(const Round& R, hipStream_t s);
// One thread stores v into the pinned host word *p (system scope) once every
// earlier kernel of the stream has completed.
hipError_t launch_mark(unsigned long long* p, unsigned long long v, hipStream_t s);

// Graph build helpers (gg_kernels.hip).
hipError_t launch_fill_src(const int* row, int n, int m, int* src, int grid, int block,
                           hipStream_t s);
hipError_t launch_count_in(const int* col, int m, int* indeg, int grid, int block, hipStream_t s);
hipError_t launch_sym_fill(const int* row, const int* col, const int* src, int n, int m,
                           const int* srow, int* cursor, int* scol, int grid, int block,
                           hipStream_t s);
hipError_t launch_t_fill(const int* col, const int* w, const int* src, int m, const int* trow,
                         int* cursor, int* tcol, int* tw, int grid, int block, hipStream_t s);
// stats[0..3] = min column, max column, min weight, max weight (initialised
// by the caller to the neutral values); *wsum += the weight sum
hipError_t launch_check(const int* col, const int* w, int m, int* stats,
                        unsigned long long* wsum, int grid, hipStream_t s);
// stable split of the edge list by head part: per-block counts
// (split_blocks(m) x kXcd), then placement from per-block bases
int split_blocks(long long m);
hipError_t launch_split_count(const int* col, int m, const unsigned char* part, int* counts,
                              hipStream_t s);
hipError_t launch_split_place(const int* src, const int* col, const int* w, int m,
                              const unsigned char* part, const long long* base, int* psrc,
                              int* pcol, int* pw, hipStream_t s);
// Renumbering: caller edge e of row u = src[e] goes to place
// nrow[newid[u]] + (e - row[u]) with head newid[col[e]] and weight w[e];
// eorig[place] = e and epos[e] = place.  w and nw may be null.
hipError_t launch_renumber(const int* row, const int* col, const int* w, const int* src, int m,
                           const int* newid, const int* nrow, int* ncol, int* nw, int* eorig,
                           int* epos, int grid, int block, hipStream_t s);
// out[v] = val[newid[v]] for every caller id v; a vertex whose new id is
// >= n_active (no edge) gets 0 if it is the source, else INF
hipError_t launch_unrenumber(int* out, const int* val, const int* newid, int n, int n_active,
                             int source, int grid, int block, hipStream_t s);
// CC: rmin[label[v']] = least oldid[v'] over the vertices v' of each label
hipError_t launch_cc_min_ids(const int* label, const int* oldid, int* rmin, int n, int grid,
                             int block, hipStream_t s);
// CC: out[v] = rmin[label[newid[v]]] for every caller id v (v itself when
// its new id is >= n_active: no edge, a component of its own)
hipError_t launch_cc_min_out(int* out, const int* label, const int* newid, const int* rmin,
                             int n, int n_active, int grid, int block, hipStream_t s);

}  // namespace gg
