// Device-wide exclusive prefix sums and fill kernels.
//
// Scan: tiles of 2048 int32 (256 threads x 8 consecutive items). Pass 1
// reduces each tile; pass 2 re-reads each tile, scans it in registers (wave
// shuffles + one LDS step across the four waves) and adds the tile's offset.
// Up to SCAN_DIRECT tiles a workgroup of pass 2 adds the sums of the tiles
// before its own itself (at most 16 loads a thread, from L2), so the scan is
// two launches; with more the sums are scanned first. A launch of these
// kernels on vertex arrays takes 2 to 5 us whatever it does, so the scans are
// counted in launches: several arrays of one length go through one scan
// (blockIdx.y), and what is scanned is computed where it is read.
#include "mc_internal.h"

namespace {

constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int64_t SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;
constexpr int64_t SCAN_DIRECT = 4096;

// what is scanned: array blockIdx.y of up to three
struct Arrays {
    const int32_t* in[3];
    __device__ __forceinline__ int32_t operator()(int64_t i) const { return in[blockIdx.y][i]; }
};
// the row lengths of the members in perm order; 0 past the kept ones
struct MemberLen {
    const int32_t* len;
    const int32_t* perm;
    const int32_t* kept;
    __device__ __forceinline__ int32_t operator()(int64_t i) const {
        return !kept || i < *kept ? len[perm ? perm[i] : i] : 0;
    }
};
// the roots of a compressed forest, those of dead graphs left out
struct Roots {
    const int32_t* par;
    const int32_t* vinst;
    const uint8_t* dead;
    __device__ __forceinline__ int32_t operator()(int64_t i) const {
        return par[i] == (int32_t)i && !(dead && dead[vinst[i]]);
    }
};
struct Outs { int32_t* p[3]; };

// the workgroup's total of s, in every thread
__device__ __forceinline__ int32_t block_sum(int32_t s, int32_t* part) {
    s = wave_sum_i32(s);
    if (lane_id() == 0) part[threadIdx.x / MC_WAVE] = s;
    __syncthreads();
    s = 0;
    for (int k = 0; k < SCAN_THREADS / MC_WAVE; k++) s += part[k];
    return s;
}

// the sum of each tile; the items to keep, if they are to be read again from there
template <class LOAD>
__global__ __launch_bounds__(SCAN_THREADS) void k_tile_sums(LOAD load, int64_t count, int32_t* __restrict__ sums,
                                                           int32_t* __restrict__ keep) {
    __shared__ int32_t part[SCAN_THREADS / MC_WAVE];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    int32_t v[SCAN_ITEMS], s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) v[k] = base + k < count ? load(base + k) : 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) s += v[k];
    if (keep) {
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; k++)
            if (base + k < count) keep[base + k] = v[k];
    }
    s = block_sum(s, part);
    if (threadIdx.x == 0) sums[(int64_t)blockIdx.y * (gridDim.x + 1) + blockIdx.x] = s;
}

// Exclusive scan of one tile per block plus the tile's offset: offs[block] of
// scanned tile sums, the sum of the tiles before it of plain ones (raw), 0
// without offs. The last block also writes out[count].
template <class LOAD>
__global__ __launch_bounds__(SCAN_THREADS) void k_tile_scan(LOAD load, Outs outs, int64_t count, const int32_t* offs,
                                                           bool raw) {
    __shared__ int32_t wtot[SCAN_THREADS / MC_WAVE], part[SCAN_THREADS / MC_WAVE];
    int32_t* const out = outs.p[blockIdx.y];
    int32_t off = 0;
    if (offs) {
        const int32_t* o = offs + (int64_t)blockIdx.y * (gridDim.x + 1);
        if (raw) {
            int32_t s = 0;
            for (int i = threadIdx.x; i < (int)blockIdx.x; i += SCAN_THREADS) s += o[i];
            off = block_sum(s, part);
        } else {
            off = o[blockIdx.x];
        }
    }
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    int32_t v[SCAN_ITEMS];
    int32_t tsum = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) v[k] = base + k < count ? load(base + k) : 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) tsum += v[k];
    // inclusive scan of thread sums within the wave
    int lane = lane_id();
    int32_t incl = tsum;
    for (int o = 1; o < MC_WAVE; o <<= 1) {
        int32_t y = __shfl_up(incl, o, MC_WAVE);
        if (lane >= o) incl += y;
    }
    if (lane == MC_WAVE - 1) wtot[threadIdx.x / MC_WAVE] = incl;
    __syncthreads();
    int32_t wpre = 0;
    int wid = threadIdx.x / MC_WAVE;
    for (int k = 0; k < wid; k++) wpre += wtot[k];
    int32_t block_total = 0;
    for (int k = 0; k < SCAN_THREADS / MC_WAVE; k++) block_total += wtot[k];
    int32_t run = off + wpre + incl - tsum;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) {
        int64_t i = base + k;
        if (i < count) out[i] = run;
        run += v[k];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[count] = off + block_total;
}

// Every vertex of the forest at its root, and the roots of each tile counted.
// A thread's vertices climb together, a load of each in flight; a parent read
// late is an ancestor too, so the loads may be cached ones.
constexpr int ROOT_ITEMS = SCAN_TILE / SCAN_THREADS;
template <int ITEMS>
__device__ __forceinline__ void climb(int32_t* par, int64_t first, int step, int64_t n, int32_t (&x)[ITEMS]) {
    int32_t p0[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; k++) {
        const int64_t v = first + (int64_t)k * step;
        p0[k] = x[k] = v < n ? ld_old(&par[v]) : -1;
    }
    for (bool any = true; any;) {
        int32_t p[ITEMS];
        any = false;
#pragma unroll
        for (int k = 0; k < ITEMS; k++) p[k] = x[k] >= 0 ? ld_old(&par[x[k]]) : -1;
#pragma unroll
        for (int k = 0; k < ITEMS; k++) {
            any |= p[k] != x[k];
            x[k] = p[k];
        }
    }
#pragma unroll
    for (int k = 0; k < ITEMS; k++)
        if (x[k] != p0[k]) st_rel(&par[first + (int64_t)k * step], x[k]);
}

__global__ __launch_bounds__(SCAN_THREADS) void k_root_sums(int32_t* par, int32_t n, const int32_t* vinst,
                                                           const uint8_t* dead, int32_t* sums) {
    __shared__ int32_t part[SCAN_THREADS / MC_WAVE];
    const int64_t first = (int64_t)blockIdx.x * SCAN_TILE + threadIdx.x;
    int32_t x[ROOT_ITEMS], s = 0;
    climb(par, first, SCAN_THREADS, n, x);
#pragma unroll
    for (int k = 0; k < ROOT_ITEMS; k++) {
        const int64_t v = first + (int64_t)k * SCAN_THREADS;
        s += v < n && x[k] == (int32_t)v && !(dead && dead[vinst[v]]);
    }
    s = block_sum(s, part);
    if (threadIdx.x == 0) sums[blockIdx.x] = s;
}

// labels of a compressed forest whose roots are ranked; -1 for dead graphs
__global__ void k_label(const int32_t* par, const int32_t* rank, int32_t n, const int32_t* vinst, const uint8_t* dead,
                        int32_t* L, DevScalars* sc) {
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
        L[v] = dead && dead[vinst[v]] ? -1 : rank[par[v]];
    if (blockIdx.x == 0 && threadIdx.x == 0) sc->n2 = rank[n];
}

// The same for forests of at most ROOT_SMALL vertices by one workgroup: roots,
// their ranks and, if asked for, the labels (2000 vertices: one launch of 5 us
// instead of four of 2 to 3 us and their gaps).
constexpr int ROOT_T = 1024;
constexpr int ROOT_PER = 4;
constexpr int ROOT_SMALL = ROOT_T * ROOT_PER;
__global__ __launch_bounds__(ROOT_T) void k_root_small(int32_t* par, int32_t n, const int32_t* vinst, const uint8_t* dead,
                                                      int32_t* rank, int32_t* L, DevScalars* sc) {
    constexpr int WAVES = ROOT_T / MC_WAVE;
    __shared__ int32_t newid[ROOT_SMALL];
    __shared__ int32_t cnt[ROOT_PER * WAVES];
    const int lane = lane_id(), wid = threadIdx.x / MC_WAVE;
    int32_t x[ROOT_PER];
    bool off[ROOT_PER], root[ROOT_PER];
    climb(par, threadIdx.x, ROOT_T, n, x);
#pragma unroll
    for (int k = 0; k < ROOT_PER; k++) {
        const int32_t v = k * ROOT_T + (int)threadIdx.x;
        off[k] = v < n && dead && dead[vinst[v]];
        root[k] = v < n && x[k] == v && !off[k];
        const unsigned long long m = __ballot(root[k]);
        newid[v] = __popcll(m & ((1ULL << lane) - 1));
        if (lane == 0) cnt[k * WAVES + wid] = __popcll(m);
    }
    __syncthreads();
    if (threadIdx.x < MC_WAVE) {
        static_assert(ROOT_PER * WAVES == MC_WAVE, "one lane per count");
        const int32_t c = cnt[lane];
        int32_t incl = c;
        for (int o = 1; o < MC_WAVE; o <<= 1) {
            const int32_t y = __shfl_up(incl, o, MC_WAVE);
            if (lane >= o) incl += y;
        }
        cnt[lane] = incl - c;
        if (lane == MC_WAVE - 1) {
            rank[n] = incl;
            if (L) sc->n2 = incl;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ROOT_PER; k++) {
        const int32_t v = k * ROOT_T + (int)threadIdx.x;
        newid[v] += cnt[k * WAVES + wid];
        if (v < n) rank[v] = newid[v];
    }
    if (!L) return;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ROOT_PER; k++) {
        const int32_t v = k * ROOT_T + (int)threadIdx.x;
        if (v < n) L[v] = off[k] ? -1 : newid[x[k]];
    }
}

__global__ void k_fill_i32(int32_t* p, int32_t v, int64_t count) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
__global__ void k_fill_i64(int64_t* p, int64_t v, int64_t count) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
__global__ void k_fill_u8(uint8_t* p, uint8_t v, int64_t count) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
__global__ void k_iota_i32(int32_t* p, int64_t count) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = (int32_t)i;
}

inline int grid_for(int64_t count, int threads) {
    int64_t b = (count + threads - 1) / threads;
    if (b < 1) b = 1;
    if (b > 8192) b = 8192;
    return (int)b;
}

}  // namespace

size_t scan_tmp_elems(int64_t count) {
    size_t total = 0;
    int64_t c = count;
    while (c > SCAN_TILE) {
        int64_t nt = (c + SCAN_TILE - 1) / SCAN_TILE;
        total += (size_t)nt + 1;
        c = nt;
    }
    return total + 1;
}

// pass 2 over tiles whose sums are in sums
template <class LOAD>
static bool scan_tiles(const LOAD& load, const Outs& outs, int arrays, int64_t count, int32_t* sums, int64_t nt,
                       hipStream_t s) {
    const bool raw = nt <= SCAN_DIRECT;
    if (!raw && (arrays > 1 || !scan_i32(sums, sums, nt, sums + nt + 1, s))) return false;
    k_tile_scan<<<dim3((unsigned)nt, (unsigned)arrays), SCAN_THREADS, 0, s>>>(load, outs, count, sums, raw);
    MC_LAUNCHED("k_tile_scan");
    return true;
}

template <class LOAD>
static bool scan(const LOAD& load, const Outs& outs, int arrays, int64_t count, int32_t* tmp, hipStream_t s) {
    const int64_t nt = (count + SCAN_TILE - 1) / SCAN_TILE;
    if (nt <= 1) {
        k_tile_scan<<<dim3(1, (unsigned)arrays), SCAN_THREADS, 0, s>>>(load, outs, count, nullptr, false);
        MC_LAUNCHED("k_tile_scan");
        return true;
    }
    k_tile_sums<<<dim3((unsigned)nt, (unsigned)arrays), SCAN_THREADS, 0, s>>>(load, count, tmp, nullptr);
    MC_LAUNCHED("k_tile_sums");
    return scan_tiles(load, outs, arrays, count, tmp, nt, s);
}

bool scan_i32(const int32_t* in, int32_t* out, int64_t count, int32_t* tmp, hipStream_t s) {
    return scan(Arrays{{in, nullptr, nullptr}}, Outs{{out, nullptr, nullptr}}, 1, count, tmp, s);
}

bool scan3_i32(int32_t* a, int32_t* b, int32_t* c, int64_t count, int32_t* tmp, hipStream_t s) {
    if ((count + SCAN_TILE - 1) / SCAN_TILE > SCAN_DIRECT)
        return scan_i32(a, a, count, tmp, s) && scan_i32(b, b, count, tmp, s) && scan_i32(c, c, count, tmp, s);
    return scan(Arrays{{a, b, c}}, Outs{{a, b, c}}, 3, count, tmp, s);
}

bool scan_member_len(const int32_t* len, const int32_t* perm, const int32_t* kept, int32_t* out, int64_t count,
                     int32_t* tmp, hipStream_t s) {
    const MemberLen load{len, perm, kept};
    const Outs outs{{out, nullptr, nullptr}};
    const int64_t nt = (count + SCAN_TILE - 1) / SCAN_TILE;
    if (nt <= 1) return scan(load, outs, 1, count, tmp, s);
    // the lengths are gathered once
    k_tile_sums<<<(unsigned)nt, SCAN_THREADS, 0, s>>>(load, count, tmp, out);
    MC_LAUNCHED("k_tile_sums");
    return scan_tiles(Arrays{{out, nullptr, nullptr}}, outs, 1, count, tmp, nt, s);
}

bool root_ranks(int32_t* parent, int32_t n, int32_t* rank, int32_t* tmp, hipStream_t s) {
    return root_labels(parent, n, nullptr, nullptr, rank, nullptr, tmp, nullptr, s);
}

bool root_labels(int32_t* parent, int32_t n, const int32_t* vinst, const uint8_t* dead, int32_t* rank, int32_t* L,
                 int32_t* tmp, DevScalars* sc, hipStream_t s) {
    if (n <= ROOT_SMALL) {
        k_root_small<<<1, ROOT_T, 0, s>>>(parent, n, vinst, dead, rank, L, sc);
        MC_LAUNCHED("k_root_small");
        return true;
    }
    const int64_t nt = ((int64_t)n + SCAN_TILE - 1) / SCAN_TILE;
    k_root_sums<<<(unsigned)nt, SCAN_THREADS, 0, s>>>(parent, n, vinst, dead, tmp);
    MC_LAUNCHED("k_root_sums");
    if (!scan_tiles(Roots{parent, vinst, dead}, Outs{{rank, nullptr, nullptr}}, 1, n, tmp, nt, s)) return false;
    if (!L) return true;
    k_label<<<grid_for(n, 256), 256, 0, s>>>(parent, rank, n, vinst, dead, L, sc);
    MC_LAUNCHED("k_label");
    return true;
}

bool fill_i32(int32_t* p, int32_t v, int64_t count, hipStream_t s) {
    if (count <= 0) return true;
    k_fill_i32<<<grid_for(count, 256), 256, 0, s>>>(p, v, count);
    MC_LAUNCHED("k_fill_i32");
    return true;
}
bool fill_i64(int64_t* p, int64_t v, int64_t count, hipStream_t s) {
    if (count <= 0) return true;
    k_fill_i64<<<grid_for(count, 256), 256, 0, s>>>(p, v, count);
    MC_LAUNCHED("k_fill_i64");
    return true;
}
bool fill_u8(uint8_t* p, uint8_t v, int64_t count, hipStream_t s) {
    if (count <= 0) return true;
    k_fill_u8<<<grid_for(count, 256), 256, 0, s>>>(p, v, count);
    MC_LAUNCHED("k_fill_u8");
    return true;
}
bool iota_i32(int32_t* p, int64_t count, hipStream_t s) {
    if (count <= 0) return true;
    k_iota_i32<<<grid_for(count, 256), 256, 0, s>>>(p, count);
    MC_LAUNCHED("k_iota_i32");
    return true;
}
