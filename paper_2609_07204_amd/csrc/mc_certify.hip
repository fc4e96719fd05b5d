// Connectivity certificates by edge-disjoint subgraphs: a reduction test that
// contracts the well-connected bulk of a graph in one step, where CAPFOREST
// (Algorithm 1) would take a chain of single pops.
//
// The weight of every edge is split over k subgraphs: with c = ceil(lam / K)
// and k = ceil(lam / c) an edge of weight w has floor(w / c) units of weight
// c, and each subgraph may use one unit of it. Vertices that are connected
// in all k subgraphs are joined by k paths whose units do not overlap, so
// every cut between them weighs at least k c >= lam: they may be contracted,
// as test-1 edges may (the forests of Nagamochi and Ibaraki, which CAPFOREST
// follows, are edge-disjoint in the same sense; here the subgraphs need no
// scan order, only components). How the units are dealt out is free:
//  - an edge belongs to its endpoint of smaller degree (coarse logarithm,
//    then id), so a vertex of small degree spends its own edges on itself
//    and hangs as a leaf below heavier ones;
//  - a vertex deals its units round-robin over the subgraphs, from a hashed
//    first one (from subgraph 0 the last subgraphs would get fewest units:
//    on Erdos-Renyi graphs of mean degree 32 and weights to 100 the weakest
//    subgraph's largest component is then 23 % of the vertices at K = 16, and
//    98 % with hashed starts). The first two rounds, 2 k units, are used.
// The first unit of a vertex in a subgraph points to a heavier vertex, so the
// first round is a forest written without atomics; the second round is
// linked in sweeps over its compressed trees. All k subgraphs are built
// side by side (one row of k n parents), so the test is two dozen launches
// whatever k is.
//
// The vertices connected in every subgraph to a reference (of 64 sampled
// vertices the one with most samples in its class) are joined directly: one
// coalesced comparison of k words a vertex. Others look for a neighbour of
// their own class among their first CERT_NEAR entries.
//
// Solves on MI355X with CAPFOREST alone, with this test's first form before it
// (the label-propagation bound first in both), and now, with the tests before
// that bound: Erdos-Renyi, 300,000 vertices, mean degree 24, weights to 1000:
// 174, 7.6 and 0.97 ms; Chung-Lu 2^20 and 2^22, 10-cores, unit weights: 6.9, 4.7
// and 1.11 ms, 14.0, 11.1 and 2.55 ms.
//
// The kernels are bound by the k n random reads of the two compressions and
// of the linking, not by the rows: one pass over the entries (12 B each, and
// a one-byte gather) deals out the units.
#include "mc_internal.h"

namespace {

constexpr int SUB = 16;          // lanes per row
constexpr int ROWS = 64;         // rows dealt out by one workgroup at a time
constexpr int32_t CERT_ROW = 512;    // entries of a row looked at (a long row is a heavy vertex, which owns little)
constexpr int CERT_NEAR = 8;
constexpr int CERT_SWEEPS = 4;
constexpr int64_t CERT_EASY = 5;
constexpr int CERT_WEDGES = 256;

inline int grid_for(int64_t count, int threads, int cap = 8192) {
    int64_t b = (count + threads - 1) / threads;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (int)b;
}

// subgraph i of a single graph that has no more than i
__device__ __forceinline__ bool unused(const CertArgs& a, int i) { return !a.vinst && i >= a.count[0]; }

__device__ __forceinline__ bool inactive(const CertArgs& a, int64_t v) {
    return a.active && !a.active[a.vinst[v]];
}

// unit weight c and subgraph count k of every graph; no member yet. A single
// graph whose mean degree is CERT_EASY times the bound or more takes half as
// many subgraphs: the weight that wider units lose is not missed there
// (Erdos-Renyi, 300,000 vertices, mean degree 6.5 times the bound: solves of
// 2.1 ms with 16 subgraphs, 2.8 ms with 32).
__global__ void k_cert_plan(CertArgs a) {
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < a.ngraphs; i += gridDim.x * blockDim.x) {
        const int64_t lam = a.lam[i];
        const int32_t kc = !a.vinst && a.kc > CERT_KMAX / 2 && *a.total / CERT_EASY / a.g.n >= lam ? CERT_KMAX / 2 : a.kc;
        const int64_t c = lam > kc ? (lam + kc - 1) / kc : 1;
        a.unit[i] = c;
        a.count[i] = lam > 0 ? (int32_t)((lam + c - 1) / c) : 0;
        if (a.sorted && a.total[1] * 4 >= CERT_WEDGES && a.total[0] / CERT_EASY / a.g.n < lam) a.count[i] = 0;
        a.rep[i] = INT32_MAX;
    }
}

// Whether two neighbours of a vertex are neighbours, for one of CERT_WEDGES
// sampled vertices (sorted rows). Where a quarter of them are, units that go
// round among a vertex's neighbours join patches and not the graph, and a graph
// whose mean degree is below CERT_EASY times the bound is left out before its
// rows are read (k = 0; hyperbolic 2^21, 32-core, 0.5 and more of the wedges
// closed: 0.36 ms of rows and components for the probe to say no; Chung-Lu and
// Erdos-Renyi graphs close fewer than one in ten). One workgroup beside those
// that class the degrees, in their time.
__device__ __forceinline__ bool wedge_closed(const DGraph& g, int i) {
    const int32_t v = (int32_t)(((uint64_t)hash32(i * 2654435761u + 99u) * (uint64_t)g.n) >> 32);
    const int32_t l = g.len[v];
    if (l < 2) return false;
    const uint32_t h = hash32(i * 2246822519u + 7u);
    const int32_t p = (int32_t)(((uint64_t)h * (uint64_t)l) >> 32);
    int32_t q = (int32_t)(((uint64_t)hash32(h) * (uint64_t)(l - 1)) >> 32);
    q += q >= p;
    int32_t x = g.col[g.off[v] + p], y = g.col[g.off[v] + q];
    if (g.len[y] < g.len[x]) { const int32_t t = x; x = y; y = t; }
    const int32_t o = g.off[x];
    int32_t lo = 0, hi = g.len[x];
    while (lo < hi) {
        const int32_t mid = (lo + hi) / 2;
        if (g.col[o + mid] < y) lo = mid + 1; else hi = mid;
    }
    return lo < g.len[x] && g.col[o + lo] == y;
}

// degree class: two bits below the leading one, so degrees within 25 % of
// each other may share a class; the sum of the degrees
__global__ __launch_bounds__(256) void k_cert_level(CertArgs a) {
    static_assert(CERT_WEDGES == 256, "one thread a wedge");
    __shared__ int64_t sum[256 / MC_WAVE];
    int64_t t = 0;
    if (a.sorted && blockIdx.x == gridDim.x - 1) {
        const int closed = __popcll(__ballot(wedge_closed(a.g, threadIdx.x)));
        if (lane_id() == 0) atomicAdd((unsigned long long*)&a.total[1], (unsigned long long)closed);
        return;
    }
    const int64_t step = (int64_t)(gridDim.x - a.sorted) * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < a.g.n; v += step) {
        const uint64_t d = (uint64_t)a.g.deg[v] | 1;
        const int e = 63 - __clzll((long long)d);
        a.level[v] = (uint8_t)((e << 2) | (int)((e >= 2 ? d >> (e - 2) : d << (2 - e)) & 3));
        t += (int64_t)d;
    }
    t = wave_sum_i64(t);
    if (lane_id() == 0) sum[threadIdx.x / MC_WAVE] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < 256 / MC_WAVE; q++) t += sum[q];
        atomicAdd((unsigned long long*)a.total, (unsigned long long)t);
    }
}

// Deals every row's units out: own[r * kc + i][v] = target of v's unit in
// subgraph i, round r. Round 0 is written as a parent (v itself without a
// unit), round 1 as a target or -1. A workgroup stages ROWS rows in LDS and
// writes each subgraph's words of them side by side. It is bound by the
// latency of its loads, each behind the last (row bounds, entries, degree
// classes of the targets), so 16 lanes take PER rows at once: their bounds
// come in one load, and the first entries and classes of all of them are in
// flight together; only the words of the k subgraphs are written, and a row
// is cut at CERT_ROW entries (Chung-Lu 2^22, 10-core, 51 million entries: 0.49
// ms; a row at a time, all words and rows of up to 4096 entries 0.69 ms).
__global__ __launch_bounds__(256) void k_cert_rows(CertArgs a) {
    constexpr int PER = ROWS / (256 / SUB);   // rows of 16 lanes
    constexpr int UN = 2;                     // entries a lane has in flight per row
    __shared__ int32_t tile[ROWS][2 * CERT_KMAX + 1];
    // a single graph writes the words of its own k subgraphs only
    const int km = a.vinst ? a.kc : a.count[0];
    if (km == 0) return;
    const int sl = threadIdx.x % SUB, sub = threadIdx.x / SUB;
    const int32_t n = a.g.n;
    for (int64_t v0 = (int64_t)blockIdx.x * ROWS; v0 < n; v0 += (int64_t)gridDim.x * ROWS) {
        for (int i = threadIdx.x; i < ROWS * 2 * km; i += 256) tile[i % ROWS][i / ROWS] = -1;
        // lane q < PER holds the bounds of the q-th row of the 16 lanes
        const int64_t mv = v0 + sub * PER + sl;
        int32_t m_o = 0, m_l = 0, m_k = 0, m_lv = 0;
        int64_t m_c = 1;
        if (sl < PER && mv < n && !inactive(a, mv)) {
            const int32_t inst = a.vinst ? a.vinst[mv] : 0;
            m_k = a.count[inst];
            m_c = a.unit[inst];
            m_o = a.g.off[mv];
            m_l = a.g.len[mv] < CERT_ROW ? a.g.len[mv] : CERT_ROW;
            m_lv = a.level[mv];
        }
        int32_t x[PER][UN], lx[PER][UN];
        int64_t w[PER][UN];
        auto load = [&](int q, int32_t o, int32_t l, int32_t j0) {
#pragma unroll
            for (int u = 0; u < UN; u++) {
                const int32_t j = j0 + u * SUB + sl;
                x[q][u] = j < l ? a.g.col[o + j] : -1;
                w[q][u] = j < l ? a.g.w[o + j] : 0;
            }
        };
        auto classes = [&](int q, int64_t c) {
#pragma unroll
            for (int u = 0; u < UN; u++) lx[q][u] = w[q][u] >= c && x[q][u] >= 0 ? a.level[x[q][u]] : -1;
        };
#pragma unroll
        for (int q = 0; q < PER; q++) load(q, __shfl(m_o, q, SUB), __shfl(m_l, q, SUB), 0);
#pragma unroll
        for (int q = 0; q < PER; q++) classes(q, __shfl(m_c, q, SUB));
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; q++) {
            const int32_t v = (int32_t)(v0 + sub * PER + q);
            const int32_t o = __shfl(m_o, q, SUB), l = __shfl(m_l, q, SUB), k = __shfl(m_k, q, SUB), lv = __shfl(m_lv, q, SUB);
            const int64_t c = __shfl(m_c, q, SUB);
            const int32_t first = (int32_t)(((uint64_t)hash32((uint32_t)v) * (uint64_t)k) >> 32);
            int32_t base = 0;
            for (int32_t j0 = 0; j0 < l && base < 2 * k;) {
#pragma unroll
                for (int u = 0; u < UN; u++) {
                    int32_t units = 0;
                    if (lx[q][u] > lv || (lx[q][u] == lv && x[q][u] > v)) {
                        int64_t left = w[q][u];
#pragma unroll
                        for (int b = 5; b >= 0; b--)
                            if ((left >> b) >= c) { left -= c << b; units += 1 << b; }
                        if (units > k) units = k;
                    }
                    int32_t incl = units;
#pragma unroll
                    for (int d = 1; d < SUB; d <<= 1) {
                        const int32_t t = __shfl_up(incl, d, SUB);
                        if (sl >= d) incl += t;
                    }
                    const int32_t start = base + incl - units;
                    base += __shfl(incl, SUB - 1, SUB);
                    for (int32_t t = start; t < start + units && t < 2 * k; t++) {
                        const int r = t >= k;
                        int32_t i = t - (r ? k : 0) + first;
                        if (i >= k) i -= k;
                        tile[sub * PER + q][r * km + i] = x[q][u];
                    }
                }
                j0 += UN * SUB;
                if (j0 < l && base < 2 * k) {
                    load(q, o, l, j0);
                    classes(q, c);
                }
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < ROWS * 2 * km; i += 256) {
            const int slot = i / ROWS, q = i % ROWS;
            const int64_t v = v0 + q;
            if (v >= n) continue;
            int32_t t = tile[q][slot];
            if (t < 0 && slot < km) t = (int32_t)v;
            a.own[(int64_t)(slot < km ? slot : slot - km + a.kc) * n + v] = t;
        }
        __syncthreads();
    }
}

// every vertex at its root, in every subgraph (blockIdx.y); after sweep
// `sweep` only in those that it changed
__global__ __launch_bounds__(256) void k_cert_compress(CertArgs a, int sweep) {
    const int32_t n = a.g.n;
    const int i = blockIdx.y;
    if ((sweep > 0 && a.more[i] != sweep) || unused(a, i)) return;
    int32_t* par = a.own + (int64_t)i * n;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        if (inactive(a, v) || i >= a.count[a.vinst ? a.vinst[v] : 0]) continue;
        const int32_t first = ld_old(&par[v]);
        int32_t x = first, p = ld_old(&par[x]);
        while (p != x) { x = p; p = ld_old(&par[x]); }
        if (x != first) st_new(&par[v], x);
    }
}

// The second round's units join the trees of the first: in a sweep a root
// hangs under a heavier root next to one of its tree's vertices (the order of
// the first round, so whichever of the racing stores stays, no cycle
// arises), with a compression after it. The first sweep looks at a quarter of
// the vertices, which a tree of a few dozen can spare; a sweep that finds two
// trees side by side stamps the subgraph, and the next runs only there. What
// CERT_SWEEPS sweeps leave apart stays apart (any subgraph will do). No
// compare-and-swap: linking by union-find, every thread of a tree meets at the
// words of a few roots (300,000 vertices, k = 32: 8.7 ms; sweeps and
// compressions 0.42 ms at k = 16).
__global__ __launch_bounds__(256) void k_cert_sweep(CertArgs a, int sweep) {
    const int32_t n = a.g.n;
    const int i = blockIdx.y;
    if ((sweep > 1 && a.more[i] < sweep - 1) || unused(a, i)) return;   // (this sweep's stamp may be there already)
    int32_t* par = a.own + (int64_t)i * n;
    const int32_t* next = a.own + (int64_t)(a.kc + i) * n;
    bool apart = false;
    // of the quarter, wavefronts of 64 consecutive vertices, others in each subgraph
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;; t += step) {
        const int64_t v = sweep == 1 ? ((t / MC_WAVE) * 4 + (i & 3)) * MC_WAVE + t % MC_WAVE : t;
        if (v >= n) break;
        if (inactive(a, v) || i >= a.count[a.vinst ? a.vinst[v] : 0]) continue;
        const int32_t u = next[v];
        if (u < 0) continue;
        const int32_t x = ld_old(&par[v]), y = ld_old(&par[u]);
        if (x == y) continue;
        apart = true;
        const int hx = a.level[x], hy = a.level[y];
        const bool up = hx > hy || (hx == hy && x > y);   // x is the heavier
        const int32_t from = up ? y : x, to = up ? x : y;
        if (ld_old(&par[from]) == from) st_new(&par[from], to);
    }
    if (apart && a.more[i] != sweep) a.more[i] = sweep;
}

// Whether the test can join much: subgraph 0, built first, is as sparse as
// the others, and a class is no larger than its component there. A graph of
// whose 64 samples fewer than half share their component with another is
// left out (k = 0). On cores of hyperbolic graphs the subgraphs fall apart at
// the smallest degree (2^21, 32-core: 6.2 ms a solve with the probe, 9.3 ms
// without) and hold together, sector by sector, at a quarter of it.
__global__ __launch_bounds__(64) void k_cert_probe(CertArgs a) {
    const int lane = lane_id();
    for (int32_t gi = blockIdx.x; gi < a.ngraphs; gi += gridDim.x) {
        if (a.active && !a.active[gi]) continue;
        const int32_t base = a.voff ? a.voff[gi] : 0;
        const int32_t n = a.voff ? a.voff[gi + 1] - base : a.g.n;
        if (n < 1) continue;
        const int32_t v = base + (int32_t)(((uint64_t)hash32(lane * 2654435761u + 4711u) * (uint64_t)n) >> 32);
        const int32_t root = a.own[v];
        int32_t same = 0;
        for (int q = 0; q < MC_WAVE; q++) same += __shfl(root, q, MC_WAVE) == root;
        const int shared = __popcll(__ballot(same > 1));
        if (lane == 0 && shared * 2 < MC_WAVE) a.count[gi] = 0;
    }
}

// the reference vertex of every graph: of 64 samples the one that shares its
// class (a hash of its components) with most of them, one wavefront a graph.
// Where three quarters of them share it, the others are single weak vertices
// rather than classes of their own, and are not looked at again (near = 0).
__global__ __launch_bounds__(64) void k_cert_ref(CertArgs a) {
    const int lane = lane_id();
    for (int32_t gi = blockIdx.x; gi < a.ngraphs; gi += gridDim.x) {
        if (a.active && !a.active[gi]) continue;
        const int32_t base = a.voff ? a.voff[gi] : 0;
        const int32_t n = a.voff ? a.voff[gi + 1] - base : a.g.n;
        const int32_t k = a.count[gi];
        if (n < 1) continue;
        const int32_t v = base + (int32_t)(((uint64_t)hash32(lane * 2654435761u + 777u) * (uint64_t)n) >> 32);
        uint32_t h = 0;
#pragma unroll 8
        for (int i = 0; i < k; i++) h += hash32((uint32_t)a.own[(int64_t)i * a.g.n + v] + 0x9E3779B9u * (uint32_t)i);
        int64_t same = 0;
        for (int q = 0; q < MC_WAVE; q++) same += __shfl(h, q, MC_WAVE) == h;
        int32_t id = lane, aux = v;
        wave_argmax(same, id, aux);
        if (lane == 0) {
            a.ref[gi] = aux;
            a.near[gi] = same * 4 < 3 * MC_WAVE;
        }
    }
}

__global__ __launch_bounds__(256) void k_cert_member(CertArgs a) {
    const int32_t n = a.g.n;
    if (unused(a, 0)) return;
    for (int64_t v0 = (int64_t)blockIdx.x * blockDim.x; v0 < n; v0 += (int64_t)gridDim.x * blockDim.x) {
        const int64_t v = v0 + threadIdx.x;
        bool in = false;
        int32_t inst = 0;
        if (v < n) {
            inst = a.vinst ? a.vinst[v] : 0;
            if (!a.active || a.active[inst]) {
                const int32_t ref = a.ref[inst], k = a.count[inst];
                int i = 0;
                while (i < k && a.own[(int64_t)i * n + v] == a.own[(int64_t)i * n + ref]) i++;
                in = k > 0 && i == k;
            }
            a.member[v] = in;
        }
        // a graph's first member in the wavefront (a graph's lanes are
        // consecutive) bounds the class's smallest vertex
        const int lane = lane_id();
        const int32_t before = __shfl_up(inst, 1, MC_WAVE);
        const unsigned long long starts = __ballot(lane == 0 || before != inst);
        const int start = 63 - __clzll((long long)(starts & (~0ULL >> (63 - lane))));
        const unsigned long long m = __ballot(in);
        const bool head = in && ((m & ((1ULL << lane) - 1)) >> start) == 0;
        if (head && (int32_t)v < ld_acq(&a.rep[inst])) atomicMin(&a.rep[inst], (int32_t)v);
    }
}

// the workgroup's unions, added to the count once
__device__ void add_marks(int32_t joined, unsigned long long* marks) {
    __shared__ int32_t sum[256 / MC_WAVE];
    joined = wave_sum_i32(joined);
    if (lane_id() == 0) sum[threadIdx.x / MC_WAVE] = joined;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t t = 0;
        for (int q = 0; q < 256 / MC_WAVE; q++) t += sum[q];
        if (t) atomicAdd(marks, (unsigned long long)t);
    }
}

// Members that are roots join the class's smallest vertex by a plain store, and
// nothing else is written by this launch: each store hangs one tree under
// another (the vertex is smaller, and roots are the smallest of their trees),
// so the count is that of the trees joined. Members below other roots follow in
// k_cert_near; unioned here, they hung roots that their own threads hung again
// and counted twice (1402 counted of 1142 trees). 1.6 million members: 22 us, by
// compare-and-swap about 100 us.
__global__ __launch_bounds__(256) void k_cert_join(CertArgs a) {
    const int32_t n = a.g.n;
    if (unused(a, 0)) return;
    int32_t joined = 0;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const int32_t inst = a.vinst ? a.vinst[v] : 0;
        if ((a.active && !a.active[inst]) || !a.member[v]) continue;
        const int32_t rep = a.rep[inst];
        if (v == rep) continue;
        if (ld_old(&a.parent[v]) == (int32_t)v) {
            st_rel(&a.parent[v], rep);
            joined++;
        }
    }
    add_marks(joined, a.marks);
}

// Members below other roots join the class; the others look for their class
// among their first entries (a launch of its own: these unions may move any root)
__global__ __launch_bounds__(256) void k_cert_near(CertArgs a) {
    const int32_t n = a.g.n;
    if (unused(a, 0)) return;
    int32_t joined = 0;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const int32_t inst = a.vinst ? a.vinst[v] : 0;
        if (a.active && !a.active[inst]) continue;
        if (a.member[v]) {
            const int32_t rep = a.rep[inst];
            if (v != rep && ld_old(&a.parent[v]) != rep && uf_union(a.parent, (int32_t)v, rep)) joined++;
            continue;
        }
        const int32_t k = a.count[inst];
        if (k == 0 || !a.near[inst]) continue;
        // targets, memberships and first components of all of them in flight
        const int32_t o = a.g.off[v], l = a.g.len[v] < CERT_NEAR ? a.g.len[v] : CERT_NEAR, mine = a.own[v];
        int32_t u[CERT_NEAR], cu[CERT_NEAR];
#pragma unroll
        for (int j = 0; j < CERT_NEAR; j++) u[j] = j < l ? a.g.col[o + j] : -1;
#pragma unroll
        for (int j = 0; j < CERT_NEAR; j++) cu[j] = u[j] >= 0 && !a.member[u[j]] ? a.own[u[j]] : -1;
        bool found = false;
#pragma unroll
        for (int j = 0; j < CERT_NEAR; j++) {
            if (found || cu[j] != mine) continue;
            int i = 1;
            while (i < k && a.own[(int64_t)i * n + v] == a.own[(int64_t)i * n + u[j]]) i++;
            if (i < k) continue;
            found = true;
            if (uf_union(a.parent, (int32_t)v, u[j])) joined++;
        }
    }
    add_marks(joined, a.marks);
}

}  // namespace

// Carves the test's arrays out of [base, base + bytes): the most subgraphs
// that fit, at most CERT_KMAX. False when fewer than CERT_KMIN fit.
bool cert_carve(CertArgs& a, void* base, size_t bytes) {
    const size_t n = (size_t)a.g.n, k = (size_t)a.ngraphs;
    const size_t fixed = 2 * n + 24 * k + 13 * 256;   // the other arrays and their alignment
    if (bytes < fixed) return false;
    const size_t kc = (bytes - fixed) / (n * 2 * sizeof(int32_t));
    if (kc < (size_t)CERT_KMIN) return false;
    a.kc = (int32_t)(kc < (size_t)CERT_KMAX ? kc : (size_t)CERT_KMAX);
    Arena m;
    m.base = (char*)base;
    m.size = bytes;
    a.total = m.take<int64_t>(2);
    a.unit = m.take<int64_t>(k);
    a.count = m.take<int32_t>(k);
    a.ref = m.take<int32_t>(k);
    a.rep = m.take<int32_t>(k);
    a.near = m.take<int32_t>(k);
    a.more = m.take<int32_t>(CERT_KMAX);
    a.level = m.take<uint8_t>(n);
    a.member = m.take<uint8_t>(n);
    a.own = m.take<int32_t>(2 * (size_t)a.kc * n);
    return m.used <= bytes;
}

// the first ny subgraphs: trees of the first round, joined by the second
static bool components(const CertArgs& a, int ny, hipStream_t s) {
    const dim3 grid(grid_for(a.g.n, 256, 1024), ny), quarter(grid_for(a.g.n / 4 + 1, 256, 1024), ny);
    if (!fill_i32(a.more, 0, a.kc, s)) return false;
    k_cert_compress<<<grid, 256, 0, s>>>(a, 0);
    for (int sweep = 1; sweep <= CERT_SWEEPS; sweep++) {
        k_cert_sweep<<<sweep == 1 ? quarter : grid, 256, 0, s>>>(a, sweep);
        k_cert_compress<<<grid, 256, 0, s>>>(a, sweep);
    }
    MC_LAUNCHED("k_cert_sweep");
    return true;
}

bool certify(const CertArgs& a, hipStream_t s) {
    const int32_t n = a.g.n;
    const int gg = a.ngraphs < 4096 ? a.ngraphs : 4096;
    if (!fill_i64(a.total, 0, 2, s)) return false;
    k_cert_level<<<grid_for(n, 256, 1024) + a.sorted, 256, 0, s>>>(a);
    k_cert_plan<<<grid_for(a.ngraphs, 256), 256, 0, s>>>(a);
    k_cert_rows<<<grid_for(n, ROWS), 256, 0, s>>>(a);
    MC_LAUNCHED("k_cert_rows");
    // The probe's 2 CERT_SWEEPS + 3 launches cost a graph that it lets through
    // about 40 us (Erdos-Renyi, 20,000 vertices: 377 and 416 us a solve), and
    // small ones are bound by their launches. From 32,768 vertices on it is
    // mixed: hyperbolic cores of 79,000 to 116,000 vertices 1.71 to 2.71 ms with
    // it, 1.95 to 2.94 ms without; Erdos-Renyi graphs of 60,000 519 and 483 us;
    // some geometric graphs that it leaves out would be joined (45,000 vertices:
    // 2.5 ms, 0.45 ms without).
    if (n >= CERT_PROBE_N) {
        if (!components(a, 1, s)) return false;
        k_cert_probe<<<gg, 64, 0, s>>>(a);
    }
    if (!components(a, a.kc, s)) return false;
    k_cert_ref<<<gg, 64, 0, s>>>(a);
    k_cert_member<<<grid_for(n, 256), 256, 0, s>>>(a);
    k_cert_join<<<grid_for(n, 256, 1024), 256, 0, s>>>(a);
    k_cert_near<<<grid_for(n, 256, 1024), 256, 0, s>>>(a);
    MC_LAUNCHED("certify");
    return true;
}
