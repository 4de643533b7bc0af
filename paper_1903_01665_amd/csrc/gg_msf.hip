// gg_msf.hip -- minimum spanning forest on the device (gg_msf in include/gg.h).
//
// MST is the fourth algorithm of the paper's evaluation (Sec. 4.1, Table 3);
// the DSL's Set type is a union-find structure (Sec. 2).  Every stored edge
// e = (src[e], col[e]) with weight w[e] is an undirected edge with the key
// w[e] * 2^32 + e: keys are distinct, so the forest of least keys is unique
// and every run returns the same edge set.  On a renumbered graph e is the
// caller's index of the edge (eorig of its stored place; epos maps back), so
// keys, ties and the output flags are those of the caller's edge order.
//
// Boruvka rounds, four kernels each:
//   min      every edge whose ends lie in different components offers its key
//            to both components (64-bit atomic minimum, checked first with a
//            plain load); a component is named by its union-find root, and
//            between rounds every vertex points at its root.  Offers to the
//            roots a block meets first collect in its LDS and leave it as one
//            atomic each
//   link     every component with an offer joins the forest with its least
//            edge (cut property) and merges with the other end's component
//            in a lock-free union-find: the larger root is linked under the
//            smaller one by compare-and-swap, so links never form a cycle;
//            two components that chose the same edge mark it once
//   compress, every vertex points at its root again: a pass with path
//   settle   halving shortens the trees, then a pass in which every thread
//            writes only its own vertex (a halving store of the first pass
//            can land after the owner's own store, leaving an ancestor that
//            is not the root; the offers of the next round need the root)
// The rounds come in two phases.  The first takes only the light edges, those
// up to a sampled quantile of the weights (about kLightPerVertex edges per
// vertex): the least crossing light edge of a component is its least crossing
// edge, so every choice stands, and most of the graph is one component before
// the bulk of the edges is looked at.  The second phase takes every edge.  The
// first round of a phase scans all edges and leaves a bit per edge that still
// crosses; the later rounds read only those.  A round with no crossing edge
// ends its phase, the second phase the run; the next round's first kernel
// reports it (same protocol as the traversal rounds).  Each round at least
// halves the number of components that still have a crossing edge, so
// 2 log2(n) + 4 rounds suffice.
//
// Atomics bound the offers: 27 G/s at most on this device, 2-8 G/s on skewed
// addresses, against 60-400 G/s for loads.  With every edge offered in every
// round an R-MAT graph of 2^20 vertices and 2^24 edges took 1.35, 2.22, 0.20
// and 0.07 ms of offers, the whole forest 4.1 ms; now 0.8 ms.

#include <new>

#include "gg_runtime.h"

using namespace gg;

namespace {

constexpr unsigned long long kNoEdge = ~0ull;
constexpr int kMsfMaxRounds = 72;
// A work item is 1 or 4 steps of 256 edges, four per lane: one step while
// that leaves no more than an item for each of kFillWaves wavefronts (a 256 x
// 256 grid's forest: 398 us with four steps, 312 with one).
constexpr int kMsfSteps = 4;
constexpr int kMsfSlots = 1024;  // roots whose offers a block collects
// Light edges per vertex, and the most of the edges that may be light: below
// five edges per vertex one phase is faster (a uniform graph of 2^17 vertices
// and 2^19 edges 0.60 ms in two phases, 0.53 in one; of 2^21 and 2^24 2.15 and
// 2.67; R-MAT, sixteen per vertex, the same within 8% from 0.5 to 3 per vertex).
// Below 2^18 edges as well: each phase's rounds are launches that do little there
// (us, two phases / one: uniform, eight per vertex, 2^13 edges 280 / 217, 2^17
// 375 / 343, 2^18 385 / 416, 2^20 565 / 692; R-MAT 2^13 220 / 154, 2^18 282 / 249,
// 2^20 335 / 289, 2^22 414 / 419; uniform, 32 per vertex, 2^17 312 / 292, 2^18
// 353 / 395, 2^20 463 / 630).
constexpr double kLightPerVertex = 1.0;
constexpr double kLightMost = 0.2;
constexpr long long kLightLeast = 1 << 18;  // edges
constexpr int kMsfSample = 8192;  // weights sampled for the light quantile
constexpr int kMsfBatch = 2;

struct Msf {
    const int* src;
    const int* col;
    const int* w;
    const int* eorig;          // renumbered graph: caller's index of each stored edge
    const int* epos;           // ... and stored place of each caller edge (else null)
    int n, m;
    int max_w;                 // largest weight
    int steps;                 // 256-edge steps of a work item
    int light;                 // samples (of kMsfSample) up to the light weight; 0: one phase
    unsigned long long* mask;  // a bit per edge: crossing when its phase last looked
    int* parent;               // union-find forest
    unsigned long long* best;  // per root: least key of a crossing edge
    unsigned char* in_msf;     // [m] output
    Ctl* ctl;
    Stat* stat;
    int* host_done;
    int tag;
    int r;
};

__device__ __forceinline__ int wsum(int x) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) x += __shfl_xor(x, d, 64);
    return x;
}

// Per-block plain update of a statistics slot (edges, updates, the weight of
// the forest's edges in `swept`) and of the round's flag.
__device__ void msf_finish(const Msf& M, int kind, int edges, int crossing, int links,
                           long long weight) {
    __shared__ int s_v[3][4];
    __shared__ long long s_w[4];
    const int a = wsum(edges), b = wsum(crossing), c = wsum(links);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) weight += __shfl_xor(weight, d, 64);
    const int wid = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s_v[0][wid] = a;
        s_v[1][wid] = b;
        s_v[2][wid] = c;
        s_w[wid] = weight;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        long long E = 0, X = 0, L = 0, W = 0;
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) {
            E += s_v[0][i];
            X += s_v[1][i];
            L += s_v[2][i];
            W += s_w[i];
        }
        if (E | X | L) {
            Stat* st = M.stat + kind * kMaxStatBlocks + blockIdx.x;
            st->edges += E;
            st->verts += X;
            st->updates += L;
            st->swept += W;
        }
        if (X > 0) M.ctl->changed[M.r % 3] = 1;
    }
}

__global__ __launch_bounds__(256) void k_msf_init(Msf M) {
    const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long tt = (long long)gridDim.x * blockDim.x;
    for (long long v = tid; v < M.n; v += tt) {
        M.parent[v] = (int)v;
        M.best[v] = kNoEdge;
    }
    for (long long e = tid; e < M.m; e += tt) M.in_msf[e] = 0;
    for (long long i = tid; i < kKinds * kMaxStatBlocks; i += tt) M.stat[i] = Stat{0, 0, 0, 0, 0};
    if (tid == 0) *M.ctl = Ctl{};
}

// The light weight: the least x with at least M.light of kMsfSample weights,
// spread over the edges by a multiplicative hash, up to x.
__global__ __launch_bounds__(1024) void k_msf_light(Msf M) {
    constexpr int P = kMsfSample / 1024;
    __shared__ int s_c[16];
    int x[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const unsigned h = (unsigned)(i * 1024 + (int)threadIdx.x) * 2654435761u;
        x[i] = M.w[(int)((unsigned long long)h * (unsigned)M.m >> 32)];
    }
    int lo = 0, hi = M.max_w;  // the answer lies in [lo, hi]
    while (lo < hi) {
        const int mid = lo + (hi - lo) / 2;
        int c = 0;
#pragma unroll
        for (int i = 0; i < P; ++i) c += x[i] <= mid;
        c = wsum(c);
        if ((threadIdx.x & 63) == 0) s_c[threadIdx.x >> 6] = c;
        __syncthreads();
        c = 0;
        for (int i = 0; i < 16; ++i) c += s_c[i];
        __syncthreads();
        if (c >= M.light) hi = mid;
        else lo = mid + 1;
    }
    if (threadIdx.x == 0) M.ctl->bound[3] = lo;
}

// Round entry: false once the run has ended (the kernel that sees round r-1
// without a crossing edge in the last phase records the round count and tells
// the host).  Every block derives the phase from round r-1's slots.
__device__ __forceinline__ bool msf_begin(const Msf& M, bool& light, bool& first) {
    Ctl* ctl = M.ctl;
    if (*(volatile int*)&ctl->done) return false;
    light = M.light > 0;
    first = M.r == 0;
    if (M.r > 0) {
        const bool was = *(volatile int*)&ctl->pull[(M.r - 1) % 3] != 0;
        light = was;
        if (*(volatile int*)&ctl->changed[(M.r - 1) % 3] == 0) {
            if (!was) {
                if (blockIdx.x == 0 && threadIdx.x == 0) {
                    ctl->iters = M.r;
                    ctl->done = 1;
                    __hip_atomic_store(M.host_done, M.tag, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_SYSTEM);
                }
                return false;
            }
            light = false;
            first = true;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctl->changed[(M.r + 1) % 3] = 0;
        ctl->pull[M.r % 3] = light;
    }
    return true;
}

struct Offers {
    int* tag;                 // [kMsfSlots] root of each slot, -1 free
    unsigned long long* key;  // its least offer in this block
};

__device__ __forceinline__ void offer_to(const Msf& M, const Offers& o, int root,
                                         unsigned long long key) {
    const int h = (int)((unsigned)root * 2654435761u >> 22);  // kMsfSlots = 2^10
    int tag = o.tag[h];
    if (tag < 0) {
        tag = atomicCAS(&o.tag[h], -1, root);
        if (tag < 0) tag = root;
    }
    if (tag == root) {
        if (key < o.key[h])
            __hip_atomic_fetch_min(&o.key[h], key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    } else if (key < M.best[root]) {
        atomicMin(&M.best[root], key);
    }
}

// A wavefront takes M.steps * 256 consecutive edges, four per lane at a time;
// bit `lane` of mask word 4 * (256-edge step) + j stands for a lane's j-th edge.  The
// parents of a lane's four edges load together (see landed): the forest of an R-MAT
// graph of 2^20 vertices takes 774 us so, edge by edge 810.  Seven wavefronts a
// SIMD leave 72 registers, and 6 of a lane's spill (28 bytes of scratch): with six
// or five and no scratch the same forests take within 4% of this, the uniform one
// of 2^20 vertices and 5.1 edges a vertex 9% more with five.  (The roots' offers
// together too: 96 registers, 745 us, but a uniform graph of 2^17 vertices 640 for
// 550.)
__global__ __launch_bounds__(256, 7) void k_msf_min(Msf M) {
    bool light, first;
    if (!msf_begin(M, light, first)) return;
    __shared__ int s_tag[kMsfSlots];
    __shared__ unsigned long long s_key[kMsfSlots];
    for (int i = threadIdx.x; i < kMsfSlots; i += blockDim.x) {
        s_tag[i] = -1;
        s_key[i] = kNoEdge;
    }
    __syncthreads();
    const Offers o{s_tag, s_key};
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    const long long gw = (long long)blockIdx.x * wpb + (threadIdx.x >> 6);
    const long long tw = (long long)gridDim.x * wpb;
    const int words = 4 * M.steps;
    const long long items = ((long long)M.m + 256 * M.steps - 1) / (256 * M.steps);
    const int top = light ? M.ctl->bound[3] : 2147483647;
    int edges = 0, crossing = 0;
    for (long long it = gw; it < items; it += tw) {
        unsigned long long* mask = M.mask + it * words;
        unsigned long long word = ~0ull;
        if (!first) {
            word = lane < words ? mask[lane] : 0;
            if (__ballot(word != 0) == 0) continue;
        }
        unsigned long long left = 0;  // lane 4c + j keeps word 4c + j
        for (int c = 0; c < M.steps; ++c) {
            const long long e = (it * M.steps + c) * 256 + lane * 4;
            unsigned todo = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                todo |= (unsigned)((__shfl(word, 4 * c + j, 64) >> lane) & 1) << j;
            int u[4] = {0, 0, 0, 0}, v[4] = {0, 0, 0, 0}, w[4] = {0, 0, 0, 0};
            if (todo && e + 4 <= M.m) {
                const int4 w4 = *reinterpret_cast<const int4*>(M.w + e);
                const int4 s4 = *reinterpret_cast<const int4*>(M.src + e);
                const int4 c4 = *reinterpret_cast<const int4*>(M.col + e);
                u[0] = s4.x, u[1] = s4.y, u[2] = s4.z, u[3] = s4.w;
                v[0] = c4.x, v[1] = c4.y, v[2] = c4.z, v[3] = c4.w;
                w[0] = w4.x, w[1] = w4.y, w[2] = w4.z, w[3] = w4.w;
            } else if (todo) {
                for (int j = 0; j < 4; ++j)
                    if (e + j < M.m) {
                        u[j] = M.src[e + j];
                        v[j] = M.col[e + j];
                        w[j] = M.w[e + j];
                    }
            }
            // edges past the end have equal ends
            int ru[4], rv[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool on = ((todo >> j) & 1) && u[j] != v[j] && w[j] <= top;
                edges += on;
                ru[j] = on ? M.parent[u[j]] : 0;
                rv[j] = on ? M.parent[v[j]] : 0;
            }
            landed(ru);
            landed(rv);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool x = ru[j] != rv[j];
                crossing += x;
                const unsigned long long b = __ballot(x);
                if (lane == 4 * c + j) left = b;
                if (x) {
                    const int eo = M.eorig ? M.eorig[e + j] : (int)(e + j);
                    const unsigned long long key =
                        ((unsigned long long)(unsigned)w[j] << 32) | (unsigned)eo;
                    offer_to(M, o, ru[j], key);
                    offer_to(M, o, rv[j], key);
                }
            }
        }
        if (lane < words && (first || left != word)) mask[lane] = left;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kMsfSlots; i += blockDim.x) {
        const int root = s_tag[i];
        if (root >= 0 && s_key[i] < M.best[root]) atomicMin(&M.best[root], s_key[i]);
    }
    msf_finish(M, KIND_ROUND, edges, crossing, 0, 0);
}

// Union-find accesses while links happen: device-scope atomics, so every
// die sees the links of the others.  Path halving only rewrites vertices
// that are no longer roots, which no link touches.
__device__ __forceinline__ int load_parent(int* p, int x) {
    return __hip_atomic_load(p + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int find_linking(int* parent, int x) {
    int p = load_parent(parent, x);
    while (p != x) {
        const int gp = load_parent(parent, p);
        if (gp != p)
            __hip_atomic_store(parent + x, gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x = gp;
        p = load_parent(parent, x);
    }
    return x;
}

__global__ __launch_bounds__(256) void k_msf_link(Msf M) {
    if (*(volatile int*)&M.ctl->done || *(volatile int*)&M.ctl->changed[M.r % 3] == 0) return;
    const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long tt = (long long)gridDim.x * blockDim.x;
    int links = 0;
    long long weight = 0;
    for (long long v = tid; v < M.n; v += tt) {
        const unsigned long long b = M.best[v];
        if (b == kNoEdge) continue;
        M.best[v] = kNoEdge;
        const int e = (int)(b & 0xffffffffu);
        M.in_msf[e] = 1;
        const int ep = M.epos ? M.epos[e] : e;
        int a = M.src[ep], c = M.col[ep];
        for (;;) {
            a = find_linking(M.parent, a);
            c = find_linking(M.parent, c);
            if (a == c) break;
            if (a < c) {
                const int t = a;
                a = c;
                c = t;
            }
            // a > c: hang root a under root c
            int expect = a;
            if (__hip_atomic_compare_exchange_strong(M.parent + a, &expect, c, __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                // every edge of the forest links once: two components that
                // chose the same edge are one after the first link
                ++links;
                weight += (long long)(b >> 32);
                break;
            }
        }
    }
    msf_finish(M, KIND_AUX, 0, 0, links, weight);
}

__global__ __launch_bounds__(256) void k_msf_compress(Msf M) {
    if (*(volatile int*)&M.ctl->done || *(volatile int*)&M.ctl->changed[M.r % 3] == 0) return;
    const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long tt = (long long)gridDim.x * blockDim.x;
    int* parent = M.parent;
    for (long long v = tid; v < M.n; v += tt) {
        int x = (int)v;
        int p = parent[x];
        while (p != x) {
            const int gp = parent[p];
            if (gp != p) parent[x] = gp;
            x = gp;
            p = parent[x];
        }
        parent[v] = x;
    }
}

__global__ __launch_bounds__(256) void k_msf_settle(Msf M) {
    if (*(volatile int*)&M.ctl->done || *(volatile int*)&M.ctl->changed[M.r % 3] == 0) return;
    const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long tt = (long long)gridDim.x * blockDim.x;
    const int* parent = M.parent;
    for (long long v = tid; v < M.n; v += tt) {
        int x = parent[v];
        while (parent[x] != x) x = parent[x];
        M.parent[v] = x;
    }
}

// Weight and edge count of the forest from the links' statistics slots.
__global__ __launch_bounds__(256) void k_msf_sum(const Stat* stat, long long* sum) {
    long long sw = 0, cnt = 0;
    for (int i = threadIdx.x; i < kMaxStatBlocks; i += 256) {
        sw += stat[KIND_AUX * kMaxStatBlocks + i].swept;
        cnt += stat[KIND_AUX * kMaxStatBlocks + i].updates;
    }
    __shared__ long long s_w[4], s_c[4];
    for (int d = 32; d > 0; d >>= 1) {
        sw += __shfl_xor(sw, d, 64);
        cnt += __shfl_xor(cnt, d, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        s_w[threadIdx.x >> 6] = sw;
        s_c[threadIdx.x >> 6] = cnt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        sum[0] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
        sum[1] = s_c[0] + s_c[1] + s_c[2] + s_c[3];
    }
}

// Grid of a launch over `units` items, clamped to the blocks resident at once.
int msf_grid(const void* f, long long units) {
    static int cus = 0;
    if (!cus) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            cus = 256;
    }
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, f, kBlock, 0) != hipSuccess || occ < 1)
        occ = 1;
    const long long cap = std::min<long long>((long long)occ * cus, kMaxStatBlocks);
    return (int)std::max(1LL, std::min<long long>((units + kBlock - 1) / kBlock, cap));
}

}  // namespace

extern "C" {

int gg_msf(gg_graph g, gg_ws ws, uint8_t* in_msf_dev, int64_t* total_weight, int64_t* n_edges,
           void* stream) {
    if (!g) return GG_EINVAL;
    if (g->err != GG_OK) return g->err;
    if (!ws) ws = g->ws0;
    if (ws->owner != g || !g->weighted || (g->m > 0 && !in_msf_dev)) return GG_EINVAL;
    WsClaim claim(ws);
    if (!claim.held()) return GG_EBUSY;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const int n = g->n;
    const int m = (int)g->m;
    // union-find and offers: kept in the workspace after the first call
    if (!ws->msf_parent) HIPCHK(g, dalloc(&ws->msf_parent, (size_t)n));
    if (!ws->msf_best) {
        void* p = nullptr;
        HIPCHK(g, hipMalloc(&p, sizeof(unsigned long long) * (size_t)n));
        ws->msf_best = static_cast<unsigned long long*>(p);
    }
    const int steps = (m + 255LL) / 256 <= kFillWaves ? 1 : kMsfSteps;
    const long long items = ((long long)m + 256 * steps - 1) / (256 * steps);
    if (!ws->msf_mask) HIPCHK(g, dalloc(&ws->msf_mask, (size_t)items * 4 * steps));
    if (ws->used && ws->last_stream != s) HIPCHK(g, hipStreamWaitEvent(s, ws->finished, 0));
    hipError_t e = hipSuccess;
    const int tag = reserve_stamps(ws, s, kMsfMaxRounds + 2, &e);
    HIPCHK(g, e);
    Msf M{};
    M.src = g->src;
    M.col = g->col;
    M.w = g->w;
    M.eorig = g->renumbered ? g->eorig : nullptr;
    M.epos = g->renumbered ? g->epos : nullptr;
    M.n = n;
    M.m = m;
    const double share = m > 0 ? kLightPerVertex * n / m : 1.0;
    M.steps = steps;
    M.light = share < kLightMost && m >= kLightLeast ? std::max(1, (int)(share * kMsfSample)) : 0;
    M.max_w = g->max_w;
    M.mask = ws->msf_mask;
    M.parent = ws->msf_parent;
    M.best = ws->msf_best;
    M.in_msf = in_msf_dev;
    M.ctl = ws->dev.ctl;
    M.stat = ws->dev.stat;
    M.host_done = ws->h_done;
    M.tag = tag;
    const int g_init = msf_grid(reinterpret_cast<const void*>(k_msf_init), std::max(n, m));
    const int g_min = msf_grid(reinterpret_cast<const void*>(k_msf_min), items * 64);
    const int g_vert = msf_grid(reinterpret_cast<const void*>(k_msf_link), n);
    hipLaunchKernelGGL(k_msf_init, dim3(g_init), dim3(kBlock), 0, s, M);
    HIPCHK(g, hipGetLastError());
    if (M.light > 0) {
        hipLaunchKernelGGL(k_msf_light, dim3(1), dim3(1024), 0, s, M);
        HIPCHK(g, hipGetLastError());
    }
    // batches of rounds, two outstanding, as in the traversal driver
    int r = 0, k = 0, status = GG_OK;
    auto enqueue = [&]() -> hipError_t {
        for (int i = 0; i < kMsfBatch && r < kMsfMaxRounds; ++i, ++r) {
            M.r = r;
            hipLaunchKernelGGL(k_msf_min, dim3(g_min), dim3(kBlock), 0, s, M);
            hipLaunchKernelGGL(k_msf_link, dim3(g_vert), dim3(kBlock), 0, s, M);
            hipLaunchKernelGGL(k_msf_compress, dim3(g_vert), dim3(kBlock), 0, s, M);
            hipLaunchKernelGGL(k_msf_settle, dim3(g_vert), dim3(kBlock), 0, s, M);
        }
        hipError_t x = hipGetLastError();
        if (x == hipSuccess) x = hipEventRecord(ws->ev[k & 1], s);
        ++k;
        return x;
    };
    auto reported = [&] { return __atomic_load_n(ws->h_done, __ATOMIC_ACQUIRE) == tag; };
    HIPCHK(g, enqueue());
    HIPCHK(g, enqueue());
    for (;;) {
        HIPCHK(g, hipEventSynchronize(ws->ev[k & 1]));
        if (reported()) break;
        if (r >= kMsfMaxRounds) {
            HIPCHK(g, hipEventSynchronize(ws->ev[(k + 1) & 1]));
            if (!reported()) status = GG_EITER;
            break;
        }
        HIPCHK(g, enqueue());
    }
    // forest weight and size
    long long* sum = reinterpret_cast<long long*>(ws->dev.pcount);
    long long hs[2] = {0, 0};
    hipLaunchKernelGGL(k_msf_sum, dim3(1), dim3(kBlock), 0, s, ws->dev.stat, sum);
    HIPCHK(g, hipGetLastError());
    HIPCHK(g, hipMemcpyAsync(hs, sum, sizeof(hs), hipMemcpyDeviceToHost, s));
    HIPCHK(g, hipEventRecord(ws->finished, s));
    HIPCHK(g, hipEventSynchronize(ws->finished));
    if (total_weight) *total_weight = hs[0];
    if (n_edges) *n_edges = hs[1];
    ws->rounds = r;
    ws->last_stream = s;
    ws->used = true;
    ws->profiled = false;
    ws->small_blocks = 0;
    ws->last = gg_stats{};
    ws->last.algo = GG_ALGO_MSF;
    ws->last.status = status;
    ws->last.grid_blocks = g_min;
    ws->last.block_threads = kBlock;
    return status;
}

}  // extern "C"
