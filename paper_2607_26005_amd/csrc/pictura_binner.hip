// HIP kernels for gfx950: uniform-grid scene binner over primitives
// (triangles and triangle pairs: count, exclusive scan, scatter into cell
// order, per-cell bounding boxes) and the kinematic bicycle step of the
// agents.
#include "pictura_device.h"

#pragma clang fp contract(off)

namespace pictura {

// ---------------------------------------------------------------------------
// primitives: triangles and pairs of them
// ---------------------------------------------------------------------------

// Walking each world's triangles in order, triangle t and t + 1 form a pair
// when they have the same class and t + 1 = (a, c, d) for t = (a, b, c) (the
// same a and c, bit for bit); a triangle that starts no pair and is not the
// second half of one is a primitive of its own.  The walk is a scan: a
// triangle is met free or taken (by a pair that starts before it), and maps
// either state to the next triangle's state and the primitives it starts.
// For a run of triangles that map is o0, o1 (the state behind it when it is
// entered free or taken) and n0, n1 (the primitives started); maps compose.
struct PairMap {
    uint32_t n0, n1;   // state in bit 31, primitives below
};

__device__ __forceinline__ PairMap pair_then(PairMap a, PairMap b)   // a, then b
{
    auto go = [&](uint32_t s) {
        const uint32_t t = (s >> 31) ? b.n1 : b.n0;
        return (t & 0x80000000u) | ((s & 0x7FFFFFFFu) + (t & 0x7FFFFFFFu));
    };
    return PairMap{go(a.n0), go(a.n1)};
}

// (entered taken, a triangle starts nothing and leaves the next one free)
__device__ __forceinline__ PairMap pair_map(bool pair) { return PairMap{pair ? 0x80000001u : 1u, 0u}; }

__device__ __forceinline__ PairMap pair_shfl_up(PairMap x, int o)
{
    return PairMap{(uint32_t)__shfl_up((int)x.n0, o), (uint32_t)__shfl_up((int)x.n1, o)};
}

constexpr int kPairItems = 4, kPairTile = kBlock * kPairItems;

// Exclusive composition over the block (identity: both states kept, nothing started); total: the block's.
__device__ __forceinline__ PairMap pair_block_scan(PairMap v, PairMap* s_wave, PairMap& total)
{
    const int lane = lane_id(), wid = threadIdx.x >> 6;
    PairMap x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const PairMap y = pair_shfl_up(x, o);
        if (lane >= o) x = pair_then(y, x);
    }
    if (lane == 63) s_wave[wid] = x;
    PairMap e = pair_shfl_up(x, 1);
    if (lane == 0) e = PairMap{0u, 0x80000000u};
    __syncthreads();
    PairMap off = {0u, 0x80000000u}, tot = off;
#pragma unroll
    for (int k = 0; k < kBlock / 64; ++k) {
        if (k < wid) off = pair_then(off, s_wave[k]);
        tot = pair_then(tot, s_wave[k]);
    }
    __syncthreads();
    total = tot;
    return pair_then(off, e);
}

__device__ __forceinline__ int world_of(const int64_t* offs, int nw, int64_t t);

// Does triangle t (of a world ending at `end`) form a pair with t + 1?
__device__ __forceinline__ bool is_pair(const PairWork& W, int64_t t, int64_t end)
{
    if (t + 1 >= end || W.cls[t] != W.cls[t + 1]) return false;
    const uint32_t* a = (const uint32_t*)W.verts + 9 * t;
    bool eq = true;
#pragma unroll
    for (int k = 0; k < 3; ++k) eq = eq & (a[k] == a[9 + k]) & (a[6 + k] == a[12 + k]);
    return eq;
}

// Apply: false composes each tile's map into tiles[], true writes the
// primitives and the worlds' first ones, entered as tiles[] (scanned) says.
template <bool Apply>
__global__ __launch_bounds__(kBlock) void pair_tiles_kernel(PairWork W)
{
    __shared__ PairMap s_wave[kBlock / 64];
    const int64_t t0 = (int64_t)blockIdx.x * kPairTile + (int64_t)threadIdx.x * kPairItems;
    int w = 0;
    bool pr[kPairItems] = {};
    PairMap v = {0u, 0x80000000u};
    if (t0 < W.T) {
        w = world_of(W.offsets, W.num_worlds, t0);
        int u = w;
        for (int k = 0; k < kPairItems && t0 + k < W.T; ++k) {
            while (W.offsets[u + 1] <= t0 + k) ++u;
            pr[k] = is_pair(W, t0 + k, W.offsets[u + 1]);
            v = pair_then(v, pair_map(pr[k]));
        }
    }
    PairMap total;
    const PairMap before = pair_block_scan(v, s_wave, total);
    if constexpr (!Apply) {
        if (threadIdx.x == 0) W.tiles[blockIdx.x] = make_uint2(total.n0, total.n1);
        return;
    }
    if (t0 >= W.T) return;
    const uint32_t enter = W.tiles[blockIdx.x].x;   // state and primitives before the tile
    const uint32_t mine = (enter >> 31) ? before.n1 : before.n0;
    uint32_t n = (enter & 0x7FFFFFFFu) + (mine & 0x7FFFFFFFu);
    bool taken = (mine >> 31) != 0;
    for (int k = 0; k < kPairItems && t0 + k < W.T; ++k) {
        const int64_t t = t0 + k;
        while (W.offsets[w + 1] <= t) ++w;
        // the first triangle of world w, and of the empty ones before it (it is free: no pair spans worlds)
        if (W.offsets[w] == t)
            for (int u = w; u >= 0 && W.offsets[u] == t; --u) W.prim_offsets[u] = (int64_t)n;
        if (taken) {
            taken = false;
            continue;
        }
        W.prims[n++] = (uint32_t)t | (pr[k] ? kPrimFlagPair : 0u);
        taken = pr[k];
    }
}

// tiles[b] from tile b's map to the state and primitives before it, starting
// free; the total, and the worlds that begin at the end.
__global__ __launch_bounds__(kBlock) void pair_sums_kernel(PairWork W, int64_t ntiles)
{
    __shared__ PairMap s_wave[kBlock / 64];
    uint32_t at = 0;
    for (int64_t b = 0; b < ntiles; b += kBlock) {
        const int64_t i = b + threadIdx.x;
        PairMap v = {0u, 0x80000000u};
        if (i < ntiles) v = PairMap{W.tiles[i].x, W.tiles[i].y};
        PairMap total;
        const PairMap before = pair_block_scan(v, s_wave, total);
        const PairMap here = PairMap{at, at};
        if (i < ntiles) W.tiles[i] = make_uint2(pair_then(here, before).n0, 0u);
        at = pair_then(here, total).n0;
    }
    if (threadIdx.x == 0) {
        const int64_t n = (int64_t)(at & 0x7FFFFFFFu);
        for (int u = W.num_worlds; u >= 0 && W.offsets[u] == W.T; --u) W.prim_offsets[u] = n;
    }
}

int64_t pair_tiles_needed(int64_t T) { return (T + kPairTile - 1) / kPairTile + 1; }

hipError_t launch_pair(const PairWork& W, hipStream_t s)
{
    const int64_t n = (W.T + kPairTile - 1) / kPairTile;
    if (n > 0) hipLaunchKernelGGL(pair_tiles_kernel<false>, dim3((unsigned)n), dim3(kBlock), 0, s, W);
    hipLaunchKernelGGL(pair_sums_kernel, dim3(1), dim3(kBlock), 0, s, W, n);
    if (n > 0) hipLaunchKernelGGL(pair_tiles_kernel<true>, dim3((unsigned)n), dim3(kBlock), 0, s, W);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// binner
// ---------------------------------------------------------------------------

__global__ void bin_init_kernel(uint32_t* count, int64_t cells, uint32_t* margin_bits, int nw)
{
    int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c <= cells) count[c] = 0;
    if (c < nw) margin_bits[c] = 0;
}

__device__ __forceinline__ int world_of(const int64_t* offs, int nw, int64_t t)
{
    int lo = 0, hi = nw - 1;   // largest w with offs[w] <= t
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (offs[mid] <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// The vertices of primitive p: a, b, c of its first triangle and, for a pair,
// d (the third vertex of the second triangle (a, c, d)).  Returns 3 or 4.
__device__ __forceinline__ int prim_verts(const BinWork& W, int64_t p, float* v)
{
    const uint32_t e = W.prims[p];
    const float* a = W.verts + 9 * (int64_t)(e & ~kPrimFlagPair);
#pragma unroll
    for (int k = 0; k < 9; ++k) v[k] = a[k];
    v[9] = v[10] = v[11] = 0.0f;
    if (!(e & kPrimFlagPair)) return 3;
    v[9] = a[15]; v[10] = a[16]; v[11] = a[17];
    return 4;
}

__global__ void bin_count_kernel(BinWork W)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= W.P) return;
    const int w = world_of(W.prim_offsets, W.num_worlds, p);
    const WorldGrid g = W.grids[w];
    float v[12];
    const int nv = prim_verts(W, p, v);
    float lo[3], hi[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        lo[d] = fminf(fminf(v[d], v[3 + d]), v[6 + d]);
        hi[d] = fmaxf(fmaxf(v[d], v[3 + d]), v[6 + d]);
        if (nv == 4) { lo[d] = fminf(lo[d], v[9 + d]); hi[d] = fmaxf(hi[d], v[9 + d]); }
    }
    const float mx = (lo[0] + hi[0]) * 0.5f, my = (lo[1] + hi[1]) * 0.5f;
    const float fx = floorf((mx - g.ox) / W.cell_size);
    const float fy = floorf((my - g.oy) / W.cell_size);
    const int ix = !(fx >= 0.0f) ? 0 : (fx >= (float)(g.nx - 1) ? g.nx - 1 : (int)fx);
    const int iy = !(fy >= 0.0f) ? 0 : (fy >= (float)(g.ny - 1) ? g.ny - 1 : (int)fy);
    const uint32_t c = (uint32_t)(g.cell_base + iy * g.nx + ix);
    W.home[p] = c;
    W.rank[p] = atomicAdd(&W.count[c], 1u);
}

// Three-phase exclusive scan over n = cells + 1 counters (in place).
constexpr int kScanItems = 4;
constexpr int kScanTile = kBlock * kScanItems;

int64_t scan_tmp_needed(int64_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

__global__ __launch_bounds__(kBlock) void scan_tiles_kernel(uint32_t* data, int64_t n, uint32_t* tile_sums)
{
    __shared__ uint32_t s_wave[kBlock / 64];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems], sum = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (base + k < n) ? data[base + k] : 0u;
        sum += v[k];
    }
    uint32_t total;
    uint32_t off = block_excl_scan(sum, s_wave, total);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n) data[base + k] = off;
        off += v[k];
    }
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kBlock) void scan_sums_kernel(uint32_t* sums, int64_t n)
{
    __shared__ uint32_t s_wave[kBlock / 64];
    uint32_t carry = 0;
    for (int64_t b = 0; b < n; b += kBlock) {
        const int64_t i = b + threadIdx.x;
        const uint32_t v = i < n ? sums[i] : 0u;
        uint32_t total;
        const uint32_t off = block_excl_scan(v, s_wave, total);
        if (i < n) sums[i] = carry + off;
        carry += total;
    }
}

__global__ void scan_add_kernel(uint32_t* data, int64_t n, const uint32_t* tile_sums)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) data[i] += tile_sums[i / kScanTile];
}

__global__ void bin_scatter_kernel(BinWork W)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= W.P) return;
    const uint32_t dst = W.count[W.home[p]] + W.rank[p];   // count[] now holds cell starts
    float v[12];
    const int nv = prim_verts(W, p, v);
    const uint32_t e = W.prims[p];
    const uint32_t cw = (uint32_t)W.cls[e & ~kPrimFlagPair] | (nv == 4 ? kPrimPair : 0u);
    W.primA[dst] = make_float4(v[0], v[1], v[2], v[3]);
    W.primB[dst] = make_float4(v[4], v[5], v[6], v[7]);
    W.primC[dst] = make_float4(v[8], __uint_as_float(cw), v[9], v[10]);
    W.primD[dst] = v[11];
    W.perm[dst] = e;
}

__device__ __forceinline__ int world_of_cell(const WorldGrid* g, int nw, int64_t c)
{
    int lo = 0, hi = nw - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if ((int64_t)g[mid].cell_base <= c) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Bounding box of every cell, from its primitives in cell order, and each
// world's margin.  kCellLanes lanes share a cell (about nine primitives on
// average, some hundreds next to roads); minima and maxima are of the
// order-preserving bit patterns.  A wave whose cells lie in one world sends its
// largest margin alone: atomics are what bound this before (six per primitive
// and one per cell: 0.69 ms of the binning of 64 worlds of 45 K triangles, which
// takes 0.35 ms in all this way).
constexpr int kCellLanes = 8;
// Cells of one launch: a grid is limited to 2^32 - 1 threads, a scene to 2^31 - 1 cells.
constexpr int64_t kCellsPerLaunch = 1ll << 28;
__global__ __launch_bounds__(kBlock) void bin_finalize_kernel(BinWork W, int64_t c0)
{
    const int64_t c = c0 + ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kCellLanes;
    const int sub = threadIdx.x % kCellLanes;
    const bool in = c < W.total_cells;
    uint32_t lo[3] = {0xFF800000u, 0xFF800000u, 0xFF800000u};   // ord(+inf)
    uint32_t hi[3] = {0x007FFFFFu, 0x007FFFFFu, 0x007FFFFFu};   // ord(-inf)
    uint32_t p0 = 0, p1 = 0;
    if (in) {
        p0 = W.count[c];
        p1 = W.count[c + 1];
    }
    for (uint32_t p = p0 + sub; p < p1; p += kCellLanes) {
        const float4 A = W.primA[p], B = W.primB[p], C = W.primC[p];
        const float v[12] = {A.x, A.y, A.z, A.w, B.x, B.y, B.z, B.w, C.x, C.z, C.w, W.primD[p]};
        const bool pair = (__float_as_uint(C.y) & kPrimPair) != 0u;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            float l = fminf(fminf(v[d], v[3 + d]), v[6 + d]), h = fmaxf(fmaxf(v[d], v[3 + d]), v[6 + d]);
            if (pair) {
                l = fminf(l, v[9 + d]);
                h = fmaxf(h, v[9 + d]);
            }
            lo[d] = min(lo[d], ord_bits(l));
            hi[d] = max(hi[d], ord_bits(h));
        }
    }
#pragma unroll
    for (int o = 1; o < kCellLanes; o <<= 1)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            lo[d] = min(lo[d], (uint32_t)__shfl_xor((int)lo[d], o));
            hi[d] = max(hi[d], (uint32_t)__shfl_xor((int)hi[d], o));
        }
    int w = -1;
    uint32_t ext = 0;
    if (in && sub == 0) {
        const float4 l = make_float4(ord_float(lo[0]), ord_float(lo[1]), ord_float(lo[2]), 0.0f);
        const float4 h = make_float4(ord_float(hi[0]), ord_float(hi[1]), ord_float(hi[2]), 0.0f);
        W.cell_lo[c] = l;
        W.cell_hi[c] = h;
        if (p1 != p0) {
            w = world_of_cell(W.grids, W.num_worlds, c);
            const WorldGrid g = W.grids[w];
            const int64_t local = c - g.cell_base;
            const int ix = (int)(local % g.nx), iy = (int)(local / g.nx);
            const float x0 = g.ox + (float)ix * W.cell_size, x1 = g.ox + (float)(ix + 1) * W.cell_size;
            const float y0 = g.oy + (float)iy * W.cell_size, y1 = g.oy + (float)(iy + 1) * W.cell_size;
            const float e = fmaxf(fmaxf(x0 - l.x, h.x - x1), fmaxf(y0 - l.y, h.y - y1));
            ext = __float_as_uint(fmaxf(e, 0.0f));
        }
    }
    const uint64_t m = __ballot(w >= 0);
    if (m == 0) return;
    const int w0 = __shfl(w, __ffsll((unsigned long long)m) - 1);
    if (__ballot(w >= 0 && w != w0) != 0) {
        if (w >= 0) atomicMax(&W.margin_bits[w], ext);
        return;
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) ext = max(ext, (uint32_t)__shfl_xor((int)ext, o));
    if (lane_id() == 0) atomicMax(&W.margin_bits[w0], ext);
}

__global__ void bin_margin_kernel(BinWork W)
{
    const int w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= W.num_worlds) return;
    const float m = __uint_as_float(W.margin_bits[w]);
    W.grids[w].margin = m * 1.0009765625f + 0.0009765625f;   // (1 + 2^-10) m + 2^-10
}

hipError_t launch_bin(const BinWork& W, hipStream_t s)
{
    const int64_t cells = W.total_cells;
    const int64_t n = cells + 1;
    auto blocks = [](int64_t m) { return (unsigned)((m + kBlock - 1) / kBlock); };
    const int64_t init_n = (n > W.num_worlds ? n : W.num_worlds);
    hipLaunchKernelGGL(bin_init_kernel, dim3(blocks(init_n)), dim3(kBlock), 0, s,
                       W.count, cells, W.margin_bits, W.num_worlds);
    if (W.P > 0)
        hipLaunchKernelGGL(bin_count_kernel, dim3(blocks(W.P)), dim3(kBlock), 0, s, W);
    const int64_t tiles = (n + kScanTile - 1) / kScanTile;
    hipLaunchKernelGGL(scan_tiles_kernel, dim3((unsigned)tiles), dim3(kBlock), 0, s, W.count, n, W.scan_tmp);
    hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(kBlock), 0, s, W.scan_tmp, tiles);
    hipLaunchKernelGGL(scan_add_kernel, dim3(blocks(n)), dim3(kBlock), 0, s, W.count, n, W.scan_tmp);
    if (W.P > 0)
        hipLaunchKernelGGL(bin_scatter_kernel, dim3(blocks(W.P)), dim3(kBlock), 0, s, W);
    for (int64_t c0 = 0; c0 < cells; c0 += kCellsPerLaunch) {
        const int64_t m = cells - c0 < kCellsPerLaunch ? cells - c0 : kCellsPerLaunch;
        hipLaunchKernelGGL(bin_finalize_kernel, dim3(blocks(m * kCellLanes)), dim3(kBlock), 0, s, W, c0);
    }
    hipLaunchKernelGGL(bin_margin_kernel, dim3(blocks(W.num_worlds)), dim3(kBlock), 0, s, W);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// kinematic bicycle step
// ---------------------------------------------------------------------------

__global__ void agents_step_kernel(const AgentStepParams p)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= p.count) return;
    const float kPi = 3.14159265358979323846f;
    float v = p.speed[i] + p.accel[i] * p.dt;
    v = fminf(fmaxf(v, 0.0f), p.vmax);
    float psi = p.psi[i] + v / (0.6f * p.length[i]) * tanf(p.steer[i]) * p.dt;
    if (psi > kPi) psi -= 2.0f * kPi;
    if (psi <= -kPi) psi += 2.0f * kPi;
    float sn, cs;
    sincosf(psi, &sn, &cs);
    p.x[i] += v * cs * p.dt;
    p.y[i] += v * sn * p.dt;
    p.psi[i] = psi;
    p.speed[i] = v;
    p.cos_h[i] = cs;
    p.sin_h[i] = sn;
}

hipError_t launch_agents_step(const AgentStepParams& p, hipStream_t s)
{
    if (p.count <= 0) return hipSuccess;
    hipLaunchKernelGGL(agents_step_kernel, dim3((unsigned)((p.count + 255) / 256)), dim3(256), 0, s, p);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// streaming-store reference: zeros written with 16-byte non-temporal stores,
// the store pattern of the render's write-out, at whatever rate HBM accepts
// ---------------------------------------------------------------------------

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

__global__ void store_probe_kernel(u32x4_t* dst, uint64_t n16)
{
    const u32x4_t z = {0u, 0u, 0u, 0u};
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
        __builtin_nontemporal_store(z, dst + i);
}

hipError_t launch_store_probe(void* dst, uint64_t bytes, hipStream_t s)
{
    const uint64_t n16 = bytes / 16u;
    if (n16 == 0) return hipSuccess;
    // 8 workgroups of 256 threads per CU slot pair, each thread a strided run of 16-byte stores
    const uint64_t want = (n16 + 255u) / 256u;
    const unsigned blocks = (unsigned)(want < 16384u ? want : 16384u);
    hipLaunchKernelGGL(store_probe_kernel, dim3(blocks), dim3(256), 0, s, (u32x4_t*)dst, n16);
    return hipGetLastError();
}

}  // namespace pictura
