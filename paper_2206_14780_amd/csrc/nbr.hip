// Cell-linked neighbour structure by counting sort, device prefix sums, and
// the canonical neighbour-list export.
#include <algorithm>
#include <cmath>

#include "sph_device.hpp"

namespace sph {

// ---------------------------------------------------------------------------
// Exclusive prefix sum: out[i] = sum_{j<i} in[j], out[n] = total.
// Three passes: per-block scan of 1024 values, scan of the block totals by a
// single block, add-back.
// ---------------------------------------------------------------------------
constexpr int kScanPer = 4;
constexpr int kScanTile = kBlock * kScanPer;

template <typename I>
__device__ inline I block_exclusive_scan(I v, I* lds, I* total) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = threadIdx.x / kWave;
    I inc = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        I t = __shfl_up(inc, off, kWave);
        if (lane >= off) inc += t;
    }
    if (lane == kWave - 1) lds[wid] = inc;
    __syncthreads();
    I wave_off = 0, tot = 0;
    for (int w = 0; w < (int)(blockDim.x / kWave); ++w) {
        if (w < wid) wave_off += lds[w];
        tot += lds[w];
    }
    __syncthreads();
    *total = tot;
    return wave_off + inc - v;
}

template <typename I>
__global__ __launch_bounds__(kBlock) void k_scan_tiles(const I* __restrict__ in, I* __restrict__ out,
                                                       I* __restrict__ tile_sum, int64_t n) {
    __shared__ I lds[kBlock / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
    I v[kScanPer];
    I s = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        v[k] = (base + k < n) ? in[base + k] : I(0);
        s += v[k];
    }
    I total;
    I off = block_exclusive_scan<I>(s, lds, &total);
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        if (base + k < n) out[base + k] = off;
        off += v[k];
    }
    if (threadIdx.x == 0) (gridDim.x == 1 ? out + n : tile_sum + blockIdx.x)[0] = total;
}

template <typename I>
__global__ __launch_bounds__(1024) void k_scan_sums(I* __restrict__ tile_sum, int64_t ntiles,
                                                    I* __restrict__ out_total) {
    __shared__ I lds[1024 / kWave];
    I carry = 0;
    for (int64_t b0 = 0; b0 < ntiles; b0 += blockDim.x) {
        int64_t i = b0 + threadIdx.x;
        I v = i < ntiles ? tile_sum[i] : I(0);
        I total;
        I ex = block_exclusive_scan<I>(v, lds, &total);
        if (i < ntiles) tile_sum[i] = carry + ex;
        carry += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) *out_total = carry;
}

// Adds each tile's offset; OWN: the sum of the tiles before it, by the block
// itself, and the last one's writes the total.
template <typename I, bool OWN>
__global__ __launch_bounds__(kBlock) void k_scan_add(I* __restrict__ out, const I* __restrict__ tile_sum,
                                                     int64_t n) {
    __shared__ I lds[kBlock / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
    I add = 0;
    if constexpr (OWN) {
        I s = 0;
        for (unsigned i = threadIdx.x; i < blockIdx.x; i += blockDim.x) s += tile_sum[i];
        (void)block_exclusive_scan<I>(s, lds, &add);
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = add + tile_sum[blockIdx.x];
    } else {
        add = tile_sum[blockIdx.x];
    }
#pragma unroll
    for (int k = 0; k < kScanPer; ++k)
        if (base + k < n) out[base + k] += add;
}

// Up to this many tiles their offsets are summed by every block, which saves a
// launch (of three, about 5 us each; one tile takes a single launch).
constexpr int64_t kScanOwn = 1024;

template <typename I>
static sph_status scan_impl(sph_ctx* ctx, const I* in, I* out, int64_t n) {
    if (n <= 0) {
        SPH_HIP(hipMemsetAsync(out, 0, sizeof(I), ctx->stream));
        return SPH_OK;
    }
    const int64_t ntiles = ceil_div(n, kScanTile);
    I* tiles = nullptr;
    SPH_TRY(ctx->ensure_t(kScanTmp, (size_t)ntiles, &tiles));
    hipLaunchKernelGGL(k_scan_tiles<I>, dim3((unsigned)ntiles), dim3(kBlock), 0, ctx->stream, in, out,
                       tiles, n);
    if (ntiles > kScanOwn) {
        hipLaunchKernelGGL(k_scan_sums<I>, dim3(1), dim3(1024), 0, ctx->stream, tiles, ntiles, out + n);
        hipLaunchKernelGGL((k_scan_add<I, false>), dim3((unsigned)ntiles), dim3(kBlock), 0, ctx->stream, out, tiles, n);
    } else if (ntiles > 1) {
        hipLaunchKernelGGL((k_scan_add<I, true>), dim3((unsigned)ntiles), dim3(kBlock), 0, ctx->stream, out, tiles, n);
    }
    SPH_LAUNCHED("scan");
    return SPH_OK;
}

sph_status scan_i32(sph_ctx* ctx, const int32_t* in, int32_t* out, int64_t n) {
    return scan_impl<int32_t>(ctx, in, out, n);
}
sph_status scan_i64(sph_ctx* ctx, const int64_t* in, int64_t* out, int64_t n) {
    return scan_impl<int64_t>(ctx, in, out, n);
}

// ---------------------------------------------------------------------------
// Counting sort of particles into cells.
// ---------------------------------------------------------------------------
__device__ inline int32_t cell_axis(double v, double org, double cs, int32_t nc, int32_t per) {
    double u = floor((v - org) / cs);
    int64_t c;
    if (!(u == u)) c = 0;  // NaN position: first cell (the predicate rejects it anyway)
    else if (u < -1e15) c = -1000000000LL;
    else if (u > 1e15) c = 1000000000LL;
    else c = (int64_t)u;
    if (per) {
        c %= nc;
        if (c < 0) c += nc;
    } else {
        if (c < 0) c = 0;
        if (c >= nc) c = nc - 1;
    }
    return (int32_t)c;
}

__global__ __launch_bounds__(kBlock) void k_cell_of(int64_t n, const double* __restrict__ x,
                                                    const double* __restrict__ y,
                                                    const double* __restrict__ z, Grid g,
                                                    int32_t* __restrict__ cell,
                                                    int32_t* __restrict__ place,
                                                    int32_t* __restrict__ count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t cx = cell_axis(x[i], g.org[0], g.cs[0], g.nc[0], g.per[0]);
    const int32_t cy = cell_axis(y[i], g.org[1], g.cs[1], g.nc[1], g.per[1]);
    const int32_t cz = cell_axis(z[i], g.org[2], g.cs[2], g.nc[2], g.per[2]);
    const int32_t c = (cz * g.nc[1] + cy) * g.nc[0] + cx;
    cell[i] = c;
    place[i] = atomicAdd(&count[c], 1);  // its place in the cell, in arrival order
}

// (No atomics here: the counting pass waits for its own instead.  At 33.7M
// particles this 1.27 -> 0.15 ms, k_cell_of 0.80 -> 1.14.)
__global__ __launch_bounds__(kBlock) void k_scatter(int64_t n, const int32_t* __restrict__ cell,
                                                    const int32_t* __restrict__ cell_start,
                                                    const int32_t* __restrict__ place,
                                                    int32_t* __restrict__ perm) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    perm[cell_start[cell[i]] + place[i]] = (int32_t)i;
}

// The scatter above leaves each cell in arrival order; sort every cell by
// original index so the layout is deterministic.  Bounded by the chain of
// dependent accesses: one wave per cell loads up to kSortWave particles at
// once and ranks them against each other in registers (n steps of one readlane
// and a compare per 64 particles).  Against one thread's insertion sort in
// global memory: 57 -> 3.7 us at 5,632 particles, 66 -> 5.7 us at 117,504, and at
// 33.7M, where bandwidth is in reach, 0.66 ms.  A fuller cell, which a smoothing
// length suited to the spacing does not make, is sorted by insertion.  Where
// most cells are empty a wave looks at `per` of them at once (with one each,
// 30M cells around 1000 particles took 1.5 ms).
constexpr int kSortWave = 4 * kWave;

// The cell's n particles at perm[b], by one wave.
__device__ inline void sort_cell(int32_t* __restrict__ perm, int32_t b, int32_t n, int lane) {
    constexpr int E = kSortWave / kWave;
    if (n <= kSortWave) {
        int32_t v[E], rank[E];
#pragma unroll
        for (int j = 0; j < E; ++j) {
            v[j] = j * kWave + lane < n ? perm[b + j * kWave + lane] : INT32_MAX;
            rank[j] = 0;
        }
#pragma unroll
        for (int i = 0; i < E; ++i) {
            const int32_t m = min(n - i * kWave, kWave);
            for (int32_t l = 0; l < m; ++l) {
                const int32_t x = __builtin_amdgcn_readlane(v[i], l);
#pragma unroll
                for (int j = 0; j < E; ++j) rank[j] += x < v[j];
            }
        }
#pragma unroll
        for (int j = 0; j < E; ++j)
            if (j * kWave + lane < n) perm[b + rank[j]] = v[j];
    } else if (lane == 0) {
        for (int32_t i = b + 1; i < b + n; ++i) {
            const int32_t v = perm[i];
            int32_t j = i - 1;
            while (j >= b && perm[j] > v) {
                perm[j + 1] = perm[j];
                --j;
            }
            perm[j + 1] = v;
        }
    }
}

// crowd[k] becomes 1 where a cell of kCrowdLeast particles or more has k
// kCrowdStep of them (k_gather_pos takes it to the host).
__global__ __launch_bounds__(kBlock) void k_sort_cells(int64_t ncell, int32_t per,
                                                       const int32_t* __restrict__ cell_start,
                                                       int32_t* __restrict__ perm, int32_t* __restrict__ crowd) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t c = ((int64_t)blockIdx.x * (kBlock / kWave) + wid) * per + lane;
    int32_t beg = 0, len = 0;
    if (lane < per && c < ncell) {
        beg = cell_start[c];
        len = cell_start[c + 1] - beg;
    }
    if (len >= kCrowdLeast) crowd[min(len / kCrowdStep, kCrowdLevels - 1)] = 1;
    for (uint64_t todo = __ballot(len > 1); todo; todo &= todo - 1) {
        const int l = __builtin_ctzll(todo);
        sort_cell(perm, __builtin_amdgcn_readlane(beg, l), __builtin_amdgcn_readlane(len, l), lane);
    }
}

__global__ __launch_bounds__(kBlock) void k_gather_pos(int64_t n, const int32_t* __restrict__ perm,
                                                       const int32_t* __restrict__ cell,
                                                       const double* __restrict__ x,
                                                       const double* __restrict__ y,
                                                       const double* __restrict__ z,
                                                       Pos4* __restrict__ pos,
                                                       int32_t* __restrict__ scell,
                                                       int32_t* __restrict__ iperm,
                                                       const int32_t* __restrict__ crowd, int32_t* host_crowd) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s < kCrowdLevels) __hip_atomic_store(&host_crowd[s], crowd[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (s >= n) return;
    const int32_t o = perm[s];
    pos[s] = Pos4{x[o], y[o], z[o], 0.0};
    scell[s] = cell[o];
    iperm[o] = (int32_t)s;
}

// ---------------------------------------------------------------------------
// Canonical export: CSR over original indices, columns ascending.
// ---------------------------------------------------------------------------
// Neighbours of every particle, in the caller's order.
__global__ __launch_bounds__(kBlock) void k_count_rows(NbrView nv, const int32_t* __restrict__ iperm,
                                                       int64_t* __restrict__ cnt) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nv.n) return;
    int32_t c = 0;
    for_each_neighbor(nv, iperm[i], [&](int32_t, double) { ++c; });
    cnt[i] = c;
}

// The same from the counts of the scan, and (longest not null) the largest.
__global__ __launch_bounds__(kBlock) void k_count_orig(int64_t n, const int32_t* __restrict__ iperm,
                                                       const int32_t* __restrict__ count, int64_t* __restrict__ cnt,
                                                       int32_t* __restrict__ longest) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int32_t c = 0;
    if (i < n) {
        c = count[iperm[i]];
        cnt[i] = c;
    }
    if (!longest) return;
    __shared__ int32_t most[kBlock / kWave];
    for (int o = kWave / 2; o > 0; o >>= 1) c = max(c, __shfl_xor(c, o, kWave));
    if (threadIdx.x % kWave == 0) most[threadIdx.x / kWave] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < kBlock / kWave; ++k) c = max(c, most[k]);
        atomicMax(longest, c);
    }
}

// Rows with more than `above` neighbours, one thread each.
__global__ __launch_bounds__(kBlock) void k_fill_orig(NbrView nv, const int32_t* __restrict__ iperm,
                                                      const int32_t* __restrict__ perm,
                                                      const int64_t* __restrict__ row_ptr, int32_t above,
                                                      int32_t* __restrict__ cols) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nv.n) return;
    const int64_t b = row_ptr[i];
    if (row_ptr[i + 1] - b <= above) return;
    int64_t k = b;
    for_each_neighbor(nv, iperm[i], [&](int32_t a, double) { cols[k++] = perm[a]; });
    for (int64_t u = b + 1; u < k; ++u) {
        int32_t v = cols[u];
        int64_t j = u - 1;
        while (j >= b && cols[j] > v) {
            cols[j + 1] = cols[j];
            --j;
        }
        cols[j + 1] = v;
    }
}

}  // namespace sph

using namespace sph;

static sph_status make_grid(sph_ctx* ctx, const sph_domain* dom, Grid* g, int64_t* ncell) {
    if (!(dom->h > 0.0) || !std::isfinite(dom->h)) return ctx->fail(SPH_E_ARG, "domain: h must be > 0");
    if (dom->kernel != SPH_KERNEL_WENDLAND && dom->kernel != SPH_KERNEL_GAUSSIAN)
        return ctx->fail(SPH_E_ARG, "domain: kernel");
    g->kernel = dom->kernel;
    // support radius: 2h (Wendland) or k h with k = 3 (truncated Gaussian)
    const double s = (dom->kernel == SPH_KERNEL_GAUSSIAN ? kGaussK : 2.0) * dom->h;
    g->gauss_tail = std::exp(-kGaussK * kGaussK);
    g->gauss_norm = std::pow(kPi, 1.5) * std::erf(kGaussK) -
                    2.0 * kPi / 3.0 * std::exp(-kGaussK * kGaussK) * kGaussK * (3.0 + 2.0 * kGaussK * kGaussK);
    g->h = dom->h;
    g->cut2 = s * s;
    g->inv_h = 1.0 / dom->h;
    g->inv_h3 = g->inv_h * g->inv_h * g->inv_h;
    g->inv_h5 = g->inv_h3 * g->inv_h * g->inv_h;
    int64_t total = 1;
    for (int a = 0; a < 3; ++a) {
        double L = dom->hi[a] - dom->lo[a];
        if (!std::isfinite(L) || !(L >= 0.0)) return ctx->fail(SPH_E_ARG, "domain: hi < lo");
        g->per[a] = dom->periodic[a] ? 1 : 0;
        g->org[a] = dom->lo[a];
        // cells a hair wider than the support, so that rounding in the binning can never
        // separate two neighbours by more than one cell
        double target = s * (1.0 + 1e-9);
        int64_t nc = (int64_t)std::floor(L / target);
        if (g->per[a]) {
            if (!(L > 0.0)) return ctx->fail(SPH_E_ARG, "domain: periodic axis of zero length");
            if (nc < 1) nc = 1;
            g->period[a] = L;
        } else {
            if (nc < 1) nc = 1;
            g->period[a] = 0.0;
        }
        if (nc > (1 << 20)) return ctx->fail(SPH_E_ARG, "domain: too many cells on one axis");
        g->nc[a] = (int32_t)nc;
        g->cs[a] = L > 0.0 ? L / (double)nc : 1.0;
        if (!g->per[a] && nc == 1) g->cs[a] = L > 0.0 ? 2.0 * L : 1.0;
        total *= nc;
    }
    if (total > (int64_t)INT32_MAX / 2) return ctx->fail(SPH_E_ARG, "domain: too many cells");
    *ncell = total;
    return SPH_OK;
}

extern "C" sph_status sph_build_neighbors(sph_ctx* ctx, const sph_particles* p, const sph_domain* dom,
                                          sph_nbr** out) {
    if (!ctx) return SPH_E_ARG;
    if (!p || !dom || !out) return ctx->fail(SPH_E_ARG, "build_neighbors: null argument");
    if (p->n < 1 || p->n >= INT32_MAX) return ctx->fail(SPH_E_ARG, "build_neighbors: n out of range");
    if (!p->x || !p->y || !p->z) return ctx->fail(SPH_E_ARG, "build_neighbors: null position array");
    *out = nullptr;
    Grid g{};
    int64_t ncell = 0;
    SPH_TRY(make_grid(ctx, dom, &g, &ncell));
    const int64_t n = p->n;

    sph_nbr* nb = new sph_nbr();
    nb->device = ctx->device;
    nb->n = n;
    nb->ncell = ncell;
    nb->g = g;
    // temporaries from the context's workspace; the handle's arrays in one
    // allocation (device allocations and frees cost tens of microseconds each)
    int32_t *cell = nullptr, *count = nullptr, *place = nullptr;
    auto fail_oom = [&]() {
        sph_neighbors_free(nb);
        return ctx->fail(SPH_E_OOM, "build_neighbors: device allocation failed");
    };
    {
        const auto up = [](size_t b) { return (b + 255) / 256 * 256; };
        const size_t b_cs = up(sizeof(int32_t) * (size_t)(ncell + 1)), b_i = up(sizeof(int32_t) * (size_t)n);
        const size_t b_pos = up(sizeof(Pos4) * (size_t)n);
        char* base = nullptr;
        if (hipMalloc(&base, b_cs + 3 * b_i + b_pos) != hipSuccess) return fail_oom();
        nb->blob = base;
        nb->cell_start = reinterpret_cast<int32_t*>(base);
        nb->scell = reinterpret_cast<int32_t*>(base + b_cs);
        nb->perm = reinterpret_cast<int32_t*>(base + b_cs + b_i);
        nb->iperm = reinterpret_cast<int32_t*>(base + b_cs + 2 * b_i);
        nb->pos = reinterpret_cast<Pos4*>(base + b_cs + 3 * b_i);
    }
    {
        sph_status st = ctx->ensure_t(kNbrCell, (size_t)n, &cell);
        if (st == SPH_OK) st = ctx->ensure_t(kNbrCount, (size_t)ncell + kCrowdLevels, &count);
        if (st == SPH_OK) st = ctx->ensure_t(kNbrPlace, (size_t)n, &place);
        if (st != SPH_OK) {
            sph_neighbors_free(nb);
            return st;
        }
    }

    hipError_t e = hipSuccess;
    auto hip_err = [&](const char* what) {
        sph_neighbors_free(nb);
        return ctx->hip_fail(e, what);
    };
    if ((e = hipMemsetAsync(count, 0, sizeof(int32_t) * (ncell + kCrowdLevels), ctx->stream)) != hipSuccess) return hip_err("memset");
    const unsigned gp = (unsigned)ceil_div(n, kBlock);
    const int32_t per = (int32_t)std::min<int64_t>(std::max<int64_t>(16 * ncell / n, 1), kWave);
    const unsigned gc = (unsigned)ceil_div(ncell, (int64_t)per * (kBlock / kWave));
    hipLaunchKernelGGL(k_cell_of, dim3(gp), dim3(kBlock), 0, ctx->stream, n, p->x, p->y, p->z, g, cell, place,
                       count);
    if ((e = hipGetLastError()) != hipSuccess) return hip_err("k_cell_of");
    sph_status st = scan_i32(ctx, count, nb->cell_start, ncell);
    if (st != SPH_OK) {
        sph_neighbors_free(nb);
        return st;
    }
    hipLaunchKernelGGL(k_scatter, dim3(gp), dim3(kBlock), 0, ctx->stream, n, cell, nb->cell_start, place, nb->perm);
    hipLaunchKernelGGL(k_sort_cells, dim3(gc), dim3(kBlock), 0, ctx->stream, ncell, per, nb->cell_start,
                       nb->perm, count + ncell);
    hipLaunchKernelGGL(k_gather_pos, dim3(gp), dim3(kBlock), 0, ctx->stream, n, nb->perm, cell, p->x, p->y,
                       p->z, nb->pos, nb->scell, nb->iperm, (const int32_t*)(count + ncell), ctx->mail_dev->crowd);
    if ((e = hipGetLastError()) != hipSuccess) return hip_err("neighbour build kernels");
    if ((e = hipStreamSynchronize(ctx->stream)) != hipSuccess) return hip_err("hipStreamSynchronize");
    for (int32_t k = 0; k < kCrowdLevels; ++k)
        if (__atomic_load_n(&ctx->host_mail->crowd[k], __ATOMIC_RELAXED)) nb->fullest = k * kCrowdStep;
    *out = nb;
    return SPH_OK;
}

// Pairs per particle (caller order) into cnt and the lists behind them (cap
// entries per row, 0: none); *longest: device, the longest row (null without lists).
static sph_status count_pairs(sph_ctx* ctx, const sph_nbr* nb, int32_t cap, int64_t** cnt_out, int32_t** count,
                              int32_t** list, int32_t** longest) {
    int64_t* cnt = nullptr;
    SPH_TRY(ctx->ensure_t(kExportCnt, (size_t)(nb->n + 1), &cnt));
    *cnt_out = cnt;
    *longest = nullptr;
    const dim3 grid((unsigned)ceil_div(nb->n, kBlock));
    if (cap == 0 && count_in_caller_order(nb->occupancy())) {
        hipLaunchKernelGGL(k_count_rows, grid, dim3(kBlock), 0, ctx->stream, nb->view(), nb->iperm, cnt);
        SPH_LAUNCHED("k_count_rows");
        return SPH_OK;
    }
    SPH_TRY(ctx->ensure_t(kCntReal, (size_t)nb->n + 1, count));
    if (cap > 0) {
        *longest = *count + nb->n;
        SPH_HIP(hipMemsetAsync(*longest, 0, sizeof(int32_t), ctx->stream));
    }
    SPH_TRY(neighbour_scan(ctx, nb, cap, *count, list));
    hipLaunchKernelGGL(k_count_orig, grid, dim3(kBlock), 0, ctx->stream, nb->n, nb->iperm, (const int32_t*)*count, cnt,
                       *longest);
    SPH_LAUNCHED("k_count_orig");
    return SPH_OK;
}

extern "C" sph_status sph_neighbors_info(sph_ctx* ctx, const sph_nbr* nb, int64_t* n, int64_t* nnz) {
    if (!ctx) return SPH_E_ARG;
    if (!nb || !n || !nnz) return ctx->fail(SPH_E_ARG, "neighbors_info: null argument");
    if (nb->device != ctx->device) return ctx->fail(SPH_E_ARG, "neighbors_info: handle of another device");
    *n = nb->n;
    if (nb->nnz < 0) {
        int64_t* cnt = nullptr;
        int32_t *count = nullptr, *longest = nullptr;
        SPH_TRY(count_pairs(ctx, nb, 0, &cnt, &count, nullptr, &longest));
        int64_t* rp = nullptr;
        SPH_TRY(ctx->ensure_t(kApplyOut, (size_t)(nb->n + 1), &rp));
        SPH_TRY(scan_i64(ctx, cnt, rp, nb->n));
        int64_t total = 0;
        SPH_HIP(hipMemcpyAsync(&total, rp + nb->n, sizeof(int64_t), hipMemcpyDeviceToHost, ctx->stream));
        SPH_HIP(hipStreamSynchronize(ctx->stream));
        const_cast<sph_nbr*>(nb)->nnz = total;
    }
    *nnz = nb->nnz;
    return SPH_OK;
}

// The export's lists are given back if the context holds more than this for
// their sake (0.7M particles' lists, the Gaussian's of 0.23M): a caller's
// other allocations do not have to live with them.  Smaller ones stay, since an
// allocation and a free cost 0.3 ms (0.8M particles: 1.3 -> 1.6 ms; 8.6M: 12.7 ->
// 13.4).
constexpr size_t kListKeep = size_t(256) << 20;
struct ListLease {
    sph_ctx* ctx;
    size_t held;
    explicit ListLease(sph_ctx* c) : ctx(c), held(c->ws_bytes[kList]) {}
    ~ListLease() {
        if (ctx->ws_bytes[kList] > std::max(held, kListKeep)) ctx->release(kList);
    }
};

extern "C" sph_status sph_neighbors_export(sph_ctx* ctx, const sph_nbr* nb, int64_t* row_ptr, int32_t* cols,
                                           int64_t cap, int64_t* nnz) {
    if (!ctx) return SPH_E_ARG;
    if (!nb || !row_ptr || !nnz) return ctx->fail(SPH_E_ARG, "neighbors_export: null argument");
    if (nb->device != ctx->device) return ctx->fail(SPH_E_ARG, "neighbors_export: handle of another device");
    int64_t* cnt = nullptr;
    int32_t *count = nullptr, *list = nullptr, *longest = nullptr;
    const ListLease lease(ctx);
    // without room for the lists every row is scanned again by the fill
    int32_t lcap = export_cap(nb);
    sph_status st = count_pairs(ctx, nb, lcap, &cnt, &count, &list, &longest);
    if (st == SPH_E_OOM && lcap > 0) {
        (void)hipGetLastError();
        lcap = 0;
        st = count_pairs(ctx, nb, 0, &cnt, &count, nullptr, &longest);
    }
    SPH_TRY(st);
    SPH_TRY(scan_i64(ctx, cnt, row_ptr, nb->n));
    int64_t total = 0;
    int32_t most = INT32_MAX;
    SPH_HIP(hipMemcpyAsync(&total, row_ptr + nb->n, sizeof(int64_t), hipMemcpyDeviceToHost, ctx->stream));
    if (lcap > 0) SPH_HIP(hipMemcpyAsync(&most, longest, sizeof(int32_t), hipMemcpyDeviceToHost, ctx->stream));
    SPH_HIP(hipStreamSynchronize(ctx->stream));
    const_cast<sph_nbr*>(nb)->nnz = total;
    *nnz = total;
    if (total > cap || (!cols && total > 0)) return ctx->fail(SPH_E_OVERFLOW, "neighbors_export: cols too small");
    if (lcap > 0) SPH_TRY(export_rows(ctx, nb, lcap, count, list, row_ptr, cols));
    if (most > lcap && total > 0) {
        hipLaunchKernelGGL(k_fill_orig, dim3((unsigned)ceil_div(nb->n, kBlock)), dim3(kBlock), 0, ctx->stream,
                           nb->view(), nb->iperm, nb->perm, row_ptr, lcap, cols);
        SPH_LAUNCHED("k_fill_orig");
    }
    SPH_HIP(hipStreamSynchronize(ctx->stream));
    return SPH_OK;
}

extern "C" sph_status sph_neighbors_free(sph_nbr* nb) {
    if (!nb) return SPH_OK;
    (void)hipFree(nb->blob);
    delete nb;
    return SPH_OK;
}
