// The viscous operator A(dt): particle data gathers, the cached sliced-ELL
// matrix (coefficients evaluated once per call in FP64), and the operator
// kernels used by sph_visc_apply and the solver.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "operator_kernels.hpp"

namespace sph {

static int32_t env_int(const char* name, int32_t dflt) {
    const char* v = std::getenv(name);
    if (!v || !*v) return dflt;
    long x = std::strtol(v, nullptr, 10);
    return x > 0 ? (int32_t)x : dflt;
}

// ---------------------------------------------------------------------------
// Gathers between the caller's order and cell order.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_gather_props(int64_t n, const int32_t* __restrict__ perm,
                                                         const double* __restrict__ m,
                                                         const double* __restrict__ r,
                                                         const double* __restrict__ mu,
                                                         const uint8_t* __restrict__ t,
                                                         double* __restrict__ om, double* __restrict__ orr,
                                                         double* __restrict__ omu,
                                                         uint8_t* __restrict__ ot, double2* __restrict__ omr,
                                                         double* __restrict__ oir) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const int32_t o = perm[s];
    const double ms = m[o], rs = r[o];
    om[s] = ms;
    orr[s] = rs;
    const double mus = mu[o];
    omu[s] = mus;
    ot[s] = t[o];
    omr[s] = make_double2(mus, ms / rs);
    oir[s] = 1.0 / rs;
}

template <typename S, typename D>
__global__ __launch_bounds__(kBlock) void k_gather_vec3(int64_t n, const int32_t* __restrict__ perm,
                                                        const S* __restrict__ a, const S* __restrict__ b,
                                                        const S* __restrict__ c, D* __restrict__ dst) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const int32_t o = perm[s];
    V3<D> v;
    v.x = (D)a[o];
    v.y = (D)b[o];
    v.z = (D)c[o];
    st3(dst, s, v);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_scatter_vec3(int64_t n, const int32_t* __restrict__ perm,
                                                         const T* __restrict__ src, T* __restrict__ a,
                                                         T* __restrict__ b, T* __restrict__ c) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const int32_t o = perm[s];
    V3<T> v = ld3(src, s);
    a[o] = v.x;
    b[o] = v.y;
    c[o] = v.z;
}

sph_status gather_props_into(sph_ctx* ctx, const sph_nbr* nb, const sph_particles* p, const PropBufs& b,
                             PartView* out) {
    const int64_t n = nb->n;
    hipLaunchKernelGGL(k_gather_props, dim3((unsigned)ceil_div(n, kBlock)), dim3(kBlock), 0, ctx->stream, n,
                       nb->perm, p->mass, p->rho, p->mu, p->type, b.mass, b.rho, b.mu, b.type, b.mu_mr, b.inv_rho);
    SPH_LAUNCHED("k_gather_props");
    out->mass = b.mass;
    out->rho = b.rho;
    out->mu = b.mu;
    out->type = b.type;
    out->mu_mr = b.mu_mr;
    out->inv_rho = b.inv_rho;
    return SPH_OK;
}

sph_status gather_props(sph_ctx* ctx, const sph_nbr* nb, const sph_particles* p, PartView* out) {
    const int64_t n = nb->n;
    PropBufs b;
    SPH_TRY(ctx->ensure_t(kMass, n, &b.mass));
    SPH_TRY(ctx->ensure_t(kRho, n, &b.rho));
    SPH_TRY(ctx->ensure_t(kMu, n, &b.mu));
    SPH_TRY(ctx->ensure_t(kType, n, &b.type));
    SPH_TRY(ctx->ensure_t(kMuMr, n, &b.mu_mr));
    SPH_TRY(ctx->ensure_t(kInvRho, n, &b.inv_rho));
    return gather_props_into(ctx, nb, p, b, out);
}

template <typename S, typename T>
sph_status gather_vec3_cvt(sph_ctx* ctx, const sph_nbr* nb, const void* const src[3], T* dst) {
    hipLaunchKernelGGL((k_gather_vec3<S, T>), dim3((unsigned)ceil_div(nb->n, kBlock)), dim3(kBlock), 0,
                       ctx->stream, nb->n, nb->perm, (const S*)src[0], (const S*)src[1], (const S*)src[2], dst);
    SPH_LAUNCHED("k_gather_vec3");
    return SPH_OK;
}
template sph_status gather_vec3_cvt<double, float>(sph_ctx*, const sph_nbr*, const void* const[3], float*);

template <typename T>
sph_status gather_vec3(sph_ctx* ctx, const sph_nbr* nb, const void* const src[3], T* dst) {
    hipLaunchKernelGGL((k_gather_vec3<T, T>), dim3((unsigned)ceil_div(nb->n, kBlock)), dim3(kBlock), 0, ctx->stream,
                       nb->n, nb->perm, (const T*)src[0], (const T*)src[1], (const T*)src[2], dst);
    SPH_LAUNCHED("k_gather_vec3");
    return SPH_OK;
}

template <typename T>
sph_status scatter_vec3(sph_ctx* ctx, const sph_nbr* nb, const T* src, void* const dst[3]) {
    hipLaunchKernelGGL(k_scatter_vec3<T>, dim3((unsigned)ceil_div(nb->n, kBlock)), dim3(kBlock), 0,
                       ctx->stream, nb->n, nb->perm, src, (T*)dst[0], (T*)dst[1], (T*)dst[2]);
    SPH_LAUNCHED("k_scatter_vec3");
    return SPH_OK;
}

template sph_status gather_vec3<float>(sph_ctx*, const sph_nbr*, const void* const[3], float*);
template sph_status gather_vec3<double>(sph_ctx*, const sph_nbr*, const void* const[3], double*);
template sph_status scatter_vec3<float>(sph_ctx*, const sph_nbr*, const float*, void* const[3]);
template sph_status scatter_vec3<double>(sph_ctx*, const sph_nbr*, const double*, void* const[3]);

// ---------------------------------------------------------------------------
// Delta-coded slots (see Sell): a step outside [0, kEscape) takes an escape
// slot carrying the whole jump.
// ---------------------------------------------------------------------------
__device__ inline bool needs_escape(int64_t step) { return step < 0 || step >= (int64_t)kEscape; }

// Coefficients are evaluated in FP64 and rounded once to T (FP32 also keeps
// the rounding remainder).
__device__ inline void sell_put(float* coef, uint16_t* dcol, float* lo, int64_t i, int32_t step, double c) {
    const float hi = (float)c;
    coef[i] = hi;
    lo[i] = (float)(c - (double)hi);
    dcol[i] = (uint16_t)step;
}
__device__ inline void sell_put(double* coef, uint16_t* dcol, float*, int64_t i, int32_t step, double c) {
    coef[i] = c;
    dcol[i] = (uint16_t)step;
}
__device__ inline void sell_escape(float* coef, uint16_t* dcol, float* lo, int64_t i, int32_t jump) {
    coef[i] = __int_as_float(jump);
    lo[i] = 0.f;
    dcol[i] = kEscape;
}
__device__ inline void sell_escape(double* coef, uint16_t* dcol, float*, int64_t i, int32_t jump) {
    coef[i] = __longlong_as_double((long long)jump);
    dcol[i] = kEscape;
}

// Writes one row's slots in order: put(col, c) per entry (columns as they
// come), then pad() up to the slice width.  c0 receives the first column.
template <typename T>
struct RowWriter {
    T* coef;
    uint16_t* dcol;
    float* lo;
    int64_t base;  // the lane's first slot
    int32_t j = 0;
    int32_t prev = 0;
    __device__ void put(int32_t col, double c) {
        if (j > 0) {
            const int64_t step = (int64_t)col - prev;
            if (needs_escape(step)) {
                sell_escape(coef, dcol, lo, slot_of<T>(base, j), (int32_t)step);
                ++j;
                prev = col;
            }
        } else {
            prev = col;
        }
        sell_put(coef, dcol, lo, slot_of<T>(base, j), col - prev, c);
        ++j;
        prev = col;
    }
    __device__ void pad(int32_t width) {
        for (; j < width; ++j) sell_put(coef, dcol, lo, slot_of<T>(base, j), 0, 0.0);
    }
};

// RowWriter's counterpart for the windowed code: the window index of a column
// comes from the block's ranges, which ascend with the columns of a row, so a
// lane walks them once.  A coefficient that is 0 codes the row itself (as the
// delta-coded row gathers it), so that an Inf or NaN of x which the matrix does
// not see stays out of the sum.
template <typename T>
struct WinWriter {
    T* coef;
    uint16_t* dcol;
    float* lo;
    int64_t base;
    const WinRange* tab;  // the block's ranges
    int32_t own;          // column code of the row itself (padding, zeros)
    int32_t j = 0;
    int32_t q = 0;
    __device__ int32_t code(int32_t col) {
        while (col >= tab[q].beg + tab[q].len) ++q;
        return (col - tab[q].beg + tab[q].base) * kWinStep;
    }
    __device__ void put(int32_t col, double c) {
        sell_put(coef, dcol, lo, slot_of<T>(base, j), (T)c == T(0) ? own : code(col), c);
        ++j;
    }
    __device__ void pad(int32_t width) {
        for (; j < width; ++j) sell_put(coef, dcol, lo, slot_of<T>(base, j), own, 0.0);
    }
};

// Slots of a row with c entries in column order: c plus one escape per step
// outside [0, kEscape).
struct SlotCounter {
    int32_t c = 0, slots = 0, prev = 0;
    __device__ void add(int32_t col) {
        if (c > 0 && needs_escape((int64_t)col - prev)) ++slots;
        ++c;
        ++slots;
        prev = col;
    }
};

// ---------------------------------------------------------------------------
// Matrix build, pass 1: slots and entries per row, FP64 diagonal, dummy-wall
// kernel sum.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_row_count(NbrView nv, PartView pv, OpParams op,
                                                      int32_t* __restrict__ cnt, int32_t* __restrict__ creal,
                                                      double* __restrict__ diag64,
                                                      double* __restrict__ wsum) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nv.n) return;
    const int32_t row = (int32_t)b;
    SlotCounter sc;
    double d = 1.0, sW = 0.0;
    if (pv.type[row] == SPH_FLUID) {
        double sw = 0.0;
        for_each_neighbor(nv, row, [&](int32_t a, double r2) {
            sw += pair_w(pv, nv.g, op.avg, row, a, r2);
            sc.add(a);
        });
        d = 1.0 + op.dt * sw;
    } else if (op.wall == SPH_WALL_DUMMY) {
        for_each_neighbor(nv, row, [&](int32_t a, double r2) {
            if (pv.type[a] != SPH_FLUID) return;
            sW += pair_W(nv.g, r2);
            sc.add(a);
        });
        if (!(sW > 0.0)) sc = SlotCounter{};
    }
    if (cnt) cnt[row] = sc.slots;
    if (creal) creal[row] = sc.c;
    diag64[row] = d;
    if (wsum) wsum[row] = sW;
}

constexpr int kChunk = 16;                    // indices per segment
constexpr int kListCap = 96;                  // listed neighbours per row, Wendland kernel
constexpr int kListCapGauss = 288;            // the same, truncated Gaussian
constexpr size_t kListBudget = size_t(24) << 30;  // bytes of lists and weights at most
constexpr int kBufStride = kChunk + 1;        // LDS words per lane (odd: no bank conflicts)
constexpr int kFillGroup = 8;                 // list entries whose gathers are issued together
static_assert(kListCap % kChunk == 0 && kListCapGauss % kChunk == 0, "whole segments");

__device__ inline int64_t list_base(int64_t r, int32_t cap) {
    return ((r / kWave) * (cap / kChunk) * kWave + (r % kWave)) * kChunk;
}
__device__ inline uint32_t list_off(uint32_t k) {
    return k / kChunk * (kWave * kChunk) + k % kChunk;
}

// Row kinds: fluid rows take every neighbour, dummy-wall rows their fluid
// neighbours, other wall rows none (identity rows).
enum { kRowNone = 0, kRowFluid = 1, kRowDummy = 2 };
__device__ inline int row_kind(const PartView& pv, const OpParams& op, int32_t row) {
    if (pv.type[row] == SPH_FLUID) return kRowFluid;
    return op.wall == SPH_WALL_DUMMY ? kRowDummy : kRowNone;
}

// Slots of a delta-coded row, from its list or, beyond cap, at most: every
// escape takes a step of kEscape or more out of the index range of the row's
// candidates, which is short but where z wraps around in a large system (only
// there the row is scanned again; doing so for every long row took 3.7 ms of
// the 30 of a matrix of 1M scattered particles with the Gaussian kernel, a
// tenth of whose rows are longer than their list).
constexpr int32_t kSpareSlots = 16;
__device__ inline int32_t row_slots(const NbrView& nv, const PartView& pv, const OpParams& op, int32_t row, int32_t c,
                                    const int32_t* __restrict__ list, int32_t cap) {
    SlotCounter sc;
    if (c <= cap) {
        const int32_t* lst = list + list_base(row, cap);
        for (int32_t k = 0; k < c; ++k) sc.add(lst[list_off(k)]);
    } else {
        const int32_t escapes = candidate_span(nv, nv.scell[row]) / kEscape;
        if (escapes <= kSpareSlots) return c + escapes;
        const int kind = row_kind(pv, op, row);
        for_each_neighbor(nv, row, [&](int32_t a, double) {
            if (kind == kRowFluid || pv.type[a] == SPH_FLUID) sc.add(a);
        });
    }
    return sc.slots;
}

// Slice size = 64 x (most slots of a row of the slice); nnz += entries.  Slots
// per row: the entries of windowed columns, which need no escapes (*wmax <=
// wlim), else cnt or (null) those of the delta code, counted here.
__global__ __launch_bounds__(kBlock) void k_slice_size(int64_t n, int64_t nslices, int32_t pack,
                                                       NbrView nv, PartView pv, OpParams op,
                                                       const int32_t* __restrict__ list, int32_t cap,
                                                       const int32_t* __restrict__ wmax, int32_t wlim,
                                                       const int32_t* __restrict__ cnt,
                                                       const int32_t* __restrict__ creal,
                                                       int64_t* __restrict__ size,
                                                       unsigned long long* __restrict__ nnz) {
    // each wave takes slices in turn, lane l reading row 64 s + l; nnz[0]:
    // nonzeros, the low 32 bits of nnz[1]: longest row (nonzeros), one
    // atomic of each kind per block
    __shared__ int64_t bt[kBlock / kWave];
    __shared__ int32_t bl[kBlock / kWave];
    const int lane = threadIdx.x % kWave;
    const int wid = threadIdx.x / kWave;
    const int nw = blockDim.x / kWave;
    int64_t tot = 0;
    int32_t longest = 0;
    const bool windowed = *wmax <= wlim;
    for (int64_t s = (int64_t)blockIdx.x * nw + wid; s < nslices; s += (int64_t)gridDim.x * nw) {
        const int64_t r = s * kWave + lane;
        int32_t w = 0;
        if (r < n) {
            const int32_t c = creal[r];
            w = windowed ? c : cnt ? cnt[r] : row_slots(nv, pv, op, (int32_t)r, c, list, cap);
            tot += c;
            longest = max(longest, c);
        }
        for (int o = kWave / 2; o > 0; o >>= 1) w = max(w, __shfl_xor(w, o, kWave));
        if (lane == 0) size[s] = (int64_t)((w + pack - 1) / pack * pack) * kWave;
    }
    for (int o = kWave / 2; o > 0; o >>= 1) {
        tot += __shfl_xor(tot, o, kWave);
        longest = max(longest, __shfl_xor(longest, o, kWave));
    }
    if (lane == 0) {
        bt[wid] = tot;
        bl[wid] = longest;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < nw; ++k) {
            tot += bt[k];
            longest = max(longest, bl[k]);
        }
        if (tot > 0) {
            atomicAdd(nnz, (unsigned long long)tot);
            atomicMax(reinterpret_cast<int32_t*>(nnz + 1), longest);
        }
    }
}

// Pass 2: write the slots (coefficients evaluated inside the scan).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_row_fill(NbrView nv, PartView pv, OpParams op,
                                                     const double* __restrict__ diag64,
                                                     const double* __restrict__ wsum,
                                                     const int64_t* __restrict__ sl_ptr, T* __restrict__ coef,
                                                     uint16_t* __restrict__ dcol, float* __restrict__ lo,
                                                     int32_t* __restrict__ c0, T* __restrict__ dg,
                                                     double* __restrict__ rs64, int64_t nslices) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nslices * kWave) return;
    const int64_t s = r / kWave;
    const int lane = (int)(r % kWave);
    const int32_t width = (int32_t)((sl_ptr[s + 1] - sl_ptr[s]) / kWave);
    RowWriter<T> wr{coef, dcol, lo, lane_base<T>(sl_ptr[s], lane)};
    if (r < nv.n) {
        const int32_t row = (int32_t)r;
        int32_t first = row;
        const double D = diag64[row];
        if (pv.type[row] == SPH_FLUID) {
            for_each_neighbor(nv, row, [&](int32_t a, double r2) {
                double aba = -op.dt * pair_w(pv, nv.g, op.avg, row, a, r2);
                double c = op.jacobi ? aba / D : aba;
                if (wr.j == 0) first = a;
                wr.put(a, c);
            });
            // row sum: (A 1)_r = 1 (eqs. diag, offdiag), scaled by 1/A_rr with Jacobi
            const double rs = op.jacobi ? 1.0 / D : 1.0;
            dg[row] = (T)rs;
            rs64[row] = rs;
        } else {
            const double sW = wsum[row];
            double rs = 1.0;
            if (op.wall == SPH_WALL_DUMMY && sW > 0.0) {
                for_each_neighbor(nv, row, [&](int32_t a, double r2) {
                    if (pv.type[a] != SPH_FLUID) return;
                    if (wr.j == 0) first = a;
                    wr.put(a, pair_W(nv.g, r2) / sW);
                });
                rs = 2.0;  // 1 + sum_a W_ra / sum_a W_ra (eq. implicit-system-dummy-full)
            }
            dg[row] = (T)rs;
            rs64[row] = rs;
        }
        c0[row] = first;
    }
    wr.pad(width);
}

// ---------------------------------------------------------------------------
// List-based matrix build (the default).
//
// k_row_scan: one wave per cell finds the neighbours of the cell's rows, counts
//   them and writes their indices (k_row_scan_rows: one thread per row does).  List layout, with cap entries per row
//   (cap / kChunk segments): entry k of row r sits at
//   ((r/64 * cap/kChunk + k/kChunk) * 64 + r%64) * kChunk + k%kChunk, so that
//   a lane walking its row reads 16-byte pieces and a slice's lists lie
//   together.
// k_slice_fill: one block per slice evaluates the pair weights in list order
//   (= scan order), which gives the row sum and the FP64 diagonal, scales them
//   and writes the slots.
// k_row_fill_list: the same by one lane per row, for the delta code, the
//   paper's single precision and matrices with a row beyond the list (such a
//   row keeps no list and is rescanned here); the weights are kept in memory
//   between its two walks.
// cap is 96 for the Wendland kernel (~80 neighbours) and 288 for the truncated
// Gaussian (~250), unless the lists of a large system would not fit their
// budget (then 96, and its rows are all rescanned).
// Same pairs, summation order and coefficients as the scan-order build.
// ---------------------------------------------------------------------------
// Largest window (3-vectors) that a block stages at once: 40.1 KB in FP32,
// four blocks (all that the registers allow) in the 160 KB of LDS; 80.2 KB in
// FP64, two blocks.  About a fifth of the blocks then take two windows.
// Operator launch at 33.7M particles, FP32, by limit 1760 / 2250 / 2700 /
// 3340 / 4400 (three blocks) / 4480 (two): 4.23 / 3.79 / 3.58 / 3.44 / 3.54 /
// 4.00 ms; FP64 at 328k by 1760 / 2250 / 2700 / 3340 / 4480 (one block): 91 /
// 80 / 74 / 66 / 81 us.
constexpr int32_t kWinLimit = 3340;
static_assert(kWinLimit <= kWinMax, "window offsets fit 16 bits");

constexpr int kWinRuns = 160;  // runs of cells of a window before merging

// The windows of a block of kWinRows rows, by one wave: the cells of
// the rows taken x-row by x-row of the cell grid, the neighbouring runs of
// cells of each as index ranges, sorted and merged where they touch or nearly
// do.  A block whose window would exceed `limit` takes one per half, or one
// per slice.  wmax receives the largest window (kWinMax + 1 when a slice's
// does not fit either).
__device__ inline void block_windows(const NbrView& nv, int64_t bid, int32_t limit, WinRange* __restrict__ win,
                                     int32_t* __restrict__ wmax, int32_t* lds, int lane) {
    constexpr int kGap = 4;  // particles between two ranges that are rather staged
    constexpr int kRuns = kWinRuns;
    const Grid& g = nv.g;
    const int32_t nx = g.nc[0], ny = g.nc[1];
    int32_t *beg = lds, *end = lds + kRuns, *sb = lds + 2 * kRuns, *se = lds + 3 * kRuns;
    // ranges of rows [r0, r1] into tab; the window's size, or kWinMax + 1
    const auto window = [&](int64_t r0, int64_t r1, WinRange* tab, int32_t parts) -> int32_t {
        const int32_t ca = nv.scell[r0], cb = nv.scell[r1];
        const int32_t l0 = ca / nx, l1 = cb / nx;  // x-rows of cells
        if (l1 - l0 >= kRuns / 9) return kWinMax + 1;
        // tasks: x-row, z and y neighbour, part of the run (middle, wrapped low, wrapped high)
        const int32_t ntask = (l1 - l0 + 1) * 27;
        int32_t cnt = 0;
        for (int32_t t0 = 0; t0 < ntask; t0 += kWave) {
            const int32_t t = t0 + lane;
            int32_t b = 0, e = 0;
            if (t < ntask) {
                const int32_t l = l0 + t / 27, part = t % 3, iy = (t / 3) % 3, iz = (t / 9) % 3;
                int32_t zs[3], ys[3];
                const int nzs = axis_cells(l / ny, g.nc[2], g.per[2], zs);
                const int nys = axis_cells(l % ny, ny, g.per[1], ys);
                const int32_t xa = l == l0 ? ca % nx : 0, xe = l == l1 ? cb % nx : nx - 1;
                int32_t lo = xa > 0 ? xa - 1 : 0, hi = xe < nx - 1 ? xe + 1 : nx - 1;
                if (g.per[0] && nx < 3) {
                    lo = 0;
                    hi = nx - 1;
                }
                bool on = iz < nzs && iy < nys;
                if (part == 1) {
                    on = on && g.per[0] && nx >= 3 && xa == 0;
                    lo = hi = nx - 1;
                } else if (part == 2) {
                    on = on && g.per[0] && nx >= 3 && xe == nx - 1;
                    lo = hi = 0;
                }
                if (on) {
                    const int32_t base = (zs[iz] * ny + ys[iy]) * nx;
                    b = nv.cell_start[base + lo];
                    e = nv.cell_start[base + hi + 1];
                }
            }
            const uint64_t m = __ballot(e > b);
            const int32_t at = cnt + mbcnt64(m);
            cnt += __popcll(m);
            if (cnt > kRuns) return kWinMax + 1;
            if (e > b) {
                beg[at] = b;
                end[at] = e;
            }
        }
        wave_sync();
        for (int32_t k = lane; k < cnt; k += kWave) {
            int32_t rank = 0;
            for (int32_t i = 0; i < cnt; ++i) rank += beg[i] < beg[k] || (beg[i] == beg[k] && i < k);
            sb[rank] = beg[k];
            se[rank] = end[k];
        }
        wave_sync();
        int32_t nr = 0, next = 1;  // window index 0 stays free for the unit before the first range
        if (lane == 0) {
            for (int32_t i = 0; i < cnt;) {
                const int32_t b = sb[i];
                int32_t e = se[i];
                for (++i; i < cnt && sb[i] <= e + kGap; ++i) e = max(e, se[i]);
                // base = b modulo 4; a 16-byte unit may reach one 3-vector over either end
                const int32_t base = next + ((b - next) & 3);
                if (nr == kWinRanges || (int64_t)base + (e - b) + 3 > kWinMax) {
                    next = kWinMax;
                    break;
                }
                tab[nr++] = WinRange{b, e - b, base, 0};
                next = base + (e - b) + 2;
            }
            tab[0].head = nr | parts << 16;  // (at least the rows' own cells)
        }
        wave_sync();
        return __builtin_amdgcn_readfirstlane(next) + 1;
    };
    int32_t largest = kWinMax + 1, parts = 1;
    for (; parts <= kWinParts; parts *= 2) {
        largest = 0;
        const int32_t rows = kWinRows / parts;
        for (int32_t k = 0; k < parts && largest <= limit; ++k) {
            const int64_t r0 = bid * kWinRows + k * rows;
            WinRange* tab = win + (bid * kWinParts + k) * kWinRanges;
            if (r0 < nv.n)
                largest = max(largest, window(r0, min(r0 + rows, nv.n) - 1, tab, parts));
            else if (lane == 0)
                tab[0].head = parts << 16;
        }
        if (largest <= limit) break;
    }
    if (lane == 0) atomicMax(wmax, largest > limit ? kWinMax + 1 : largest);
}

// One wave per cell: the cell's rows share their neighbour candidates, which
// the lanes hold in registers (kScanRounds rounds of 64 at a time, taken from
// the runs of cells around the cell laid end to end); every row is tested
// against each round at once and its neighbours are appended in ascending
// order by their rank in the ballot.  Against one thread per row walking its
// candidates one after the other this loads each candidate once per cell
// instead of once per row, and has no serial chain of loads.  A cell's rows
// are dealt to `split` waves where the grid alone would leave the chip idle.  What
// bounds it is instruction issue: 8 rounds a row of about 31 instructions, 19
// of them vector.  298 -> 22 us at 5,632 particles, 1.08 -> 0.55 ms at 1.16M
// (windows included), 24.1 -> 16.1 ms at 33.7M, 1.28 -> 0.48 ms at 187k with
// the Gaussian kernel.
// all: every row takes every neighbour (the neighbour lists themselves).
// The first blocks of the launch compute the operator's windows instead
// (win_blocks, 0 for none): their latency hides behind the scan.
constexpr int kScanRounds = 8;
constexpr int kScanBatch = kScanRounds * kWave;

__global__ __launch_bounds__(kBlock) void k_row_scan(NbrView nv, PartView pv, OpParams op, int64_t ncell,
                                                     int32_t split, bool all, int32_t* creal,
                                                     int32_t* __restrict__ list, int32_t cap, int32_t win_blocks,
                                                     WinRange* __restrict__ win, int32_t* __restrict__ wmax) {
    constexpr int kW = kBlock / kWave;
    __shared__ int32_t cand_lds[kW][kScanBatch > 4 * kWinRuns ? kScanBatch : 4 * kWinRuns];
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if ((int32_t)blockIdx.x < win_blocks) {
        const int64_t b = (int64_t)blockIdx.x * kW + wid;
        if (b * kWinRows < nv.n) block_windows(nv, b, kWinLimit, win, wmax, cand_lds[wid], lane);
        return;
    }
    const int64_t w64 = (int64_t)xcd_block(blockIdx.x - win_blocks, gridDim.x - win_blocks) * kW + wid;
    if (w64 >= ncell * split) return;
    const int32_t c = (int32_t)(w64 / split), share = (int32_t)(w64 % split);
    const int32_t rb = nv.cell_start[c], re = nv.cell_start[c + 1];
    if (rb >= re) return;
    const Grid& g = nv.g;
    int32_t* cand = cand_lds[wid];
    // the runs of cells around the cell, one per lane, in ascending order, and
    // their places in the sequence of candidates
    int32_t beg, len, total;
    cell_run(nv, c, lane, beg, len);
    const int32_t pre = run_prefix(len, lane, total);
    for (int32_t b0 = 0; b0 < total; b0 += kScanBatch) {
        uint64_t runs = __ballot(len > 0 && pre < b0 + kScanBatch && pre + len > b0);
        while (runs) {
            const int t = __builtin_ctzll(runs);
            runs &= runs - 1;
            const int32_t B = __builtin_amdgcn_readlane(beg, t), L = __builtin_amdgcn_readlane(len, t);
            const int32_t P = __builtin_amdgcn_readlane(pre, t) - b0;
            const int32_t j1 = min(L, kScanBatch - P);
            for (int32_t j = max(0, -P) + lane; j < j1; j += kWave) cand[P + j] = B + j;
        }
        wave_sync();
        const int32_t nc = min(total - b0, kScanBatch);
        int32_t a[kScanRounds];
        double ax[kScanRounds], ay[kScanRounds], az[kScanRounds];
        uint64_t fluid[kScanRounds];  // the fluid candidates of a round
        bool far = false;
        const Pos4 ref = nv.pos[rb];
#pragma unroll
        for (int q = 0; q < kScanRounds; ++q) {
            const bool ok = q * kWave + lane < nc;
            a[q] = ok ? cand[q * kWave + lane] : rb;
            const Pos4* s = nv.pos + a[q];
            // a lane without a candidate never passes the distance test
            ax[q] = ok ? s->x : __builtin_nan("");
            ay[q] = s->y;
            az[q] = s->z;
            fluid[q] = all ? 0 : __ballot(pv.type[a[q]] == SPH_FLUID);
            far = far || (ok && far_image(g, ref, ax[q], ay[q], az[q]));
        }
        wave_sync();
        const bool image = __any(far) || total > kScanBatch;
        for (int32_t g0 = rb; g0 < re; g0 += kWave) {
            // the rows, one per lane
            const int32_t row = g0 + lane;
            const bool on = row < re;
            Pos4 pb{};
            int kind = kRowNone;
            int32_t mine = 0;  // neighbours so far
            if (on) {
                pb = nv.pos[row];
                kind = all ? (int)kRowFluid : row_kind(pv, op, row);
                if (b0 > 0) mine = creal[row];
            }
            const int32_t nrow = min(re - g0, kWave);
            for (int32_t i = share; i < nrow; i += split) {  // (split divides the wave's 64 rows)
                const int kd = __builtin_amdgcn_readlane(kind, i);
                if (kd == kRowNone) continue;
                const double xb = read_lane(pb.x, i), yb = read_lane(pb.y, i), zb = read_lane(pb.z, i);
                const int32_t ri = g0 + i;
                int32_t cnt = __builtin_amdgcn_readlane(mine, i);
                int32_t* out = list + list_base(ri, cap);  // (uniform: a scalar base)
                const auto tests = [&](auto img, auto all) {
#pragma unroll
                    for (int q = 0; q < kScanRounds; ++q) {
                        if (q * kWave >= nc) break;
                        double dx = xb - ax[q], dy = yb - ay[q], dz = zb - az[q];
                        if constexpr (decltype(img)::value) {
                            dx = disp(xb, ax[q], g.period[0]);
                            dy = disp(yb, ay[q], g.period[1]);
                            dz = disp(zb, az[q], g.period[2]);
                        }
                        const double r2 = (dx * dx + dy * dy) + dz * dz;
                        uint64_t m = __ballot(r2 < g.cut2) & __ballot(a[q] != ri);
                        if constexpr (!decltype(all)::value) m &= fluid[q];
                        const uint32_t k = (uint32_t)(cnt + mbcnt64(m));
                        cnt = __builtin_amdgcn_readfirstlane(cnt + __popcll(m));
                        if (cnt > cap) m &= __ballot((int32_t)k < cap);
                        if (__builtin_amdgcn_inverse_ballot_w64(m)) out[list_off(k)] = a[q];
                    }
                };
                if (image) {
                    if (kd == kRowFluid) tests(std::true_type{}, std::true_type{});
                    else tests(std::true_type{}, std::false_type{});
                } else {
                    if (kd == kRowFluid) tests(std::false_type{}, std::true_type{});
                    else tests(std::false_type{}, std::false_type{});
                }
                if (lane == i) mine = cnt;
            }
            if (on && lane % split == share) creal[row] = mine;
        }
    }
}

// The scan by one thread per row, for cells that are mostly empty or too full
// (see scan_by_rows).  The lanes of a wave reach their k-th neighbour at
// different points, so each collects kChunk indices in LDS and writes them as
// one segment.
__global__ __launch_bounds__(kBlock) void k_row_scan_rows(NbrView nv, PartView pv, OpParams op, bool all,
                                                          int32_t* __restrict__ cnt, int32_t* __restrict__ creal,
                                                          int32_t* __restrict__ list, int32_t cap) {
    constexpr int kStride = kChunk + 1;  // LDS words per lane (odd: no bank conflicts)
    __shared__ int32_t buf[kBlock * kStride];
    const int64_t b = (int64_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (b >= nv.n) return;  // (each lane uses only its own LDS words)
    const int32_t row = (int32_t)b;
    int32_t* my = buf + threadIdx.x * kStride;
    int32_t* out = list + list_base(b, cap);
    SlotCounter sc;
    const int32_t& c = sc.c;
    const auto flush = [&](int32_t q) {
        int4* dst = reinterpret_cast<int4*>(out + list_off(q * kChunk));
#pragma unroll
        for (int i = 0; i < kChunk / 4; ++i)
            dst[i] = make_int4(my[4 * i], my[4 * i + 1], my[4 * i + 2], my[4 * i + 3]);
    };
    const int kind = all ? (int)kRowFluid : row_kind(pv, op, row);
    if (kind != kRowNone)
        for_each_neighbor(nv, row, [&](int32_t a, double) {
            if (kind == kRowDummy && pv.type[a] != SPH_FLUID) return;
            const int32_t e = c % kChunk;
            my[e] = a;
            if (e == kChunk - 1 && c < cap) flush(c / kChunk);
            sc.add(a);
        });
    if (c < cap && c % kChunk) flush(c / kChunk);
    creal[row] = c;
    if (cnt) cnt[row] = sc.slots;
}

template <typename T, bool WIN>
__global__ __launch_bounds__(kBlock) void k_row_fill_list(NbrView nv, PartView pv, OpParams op, int64_t nslices,
                                                          const int32_t* __restrict__ creal,
                                                          const int32_t* __restrict__ list,
                                                          double* __restrict__ wlist,
                                                          const int64_t* __restrict__ sl_ptr, T* __restrict__ coef,
                                                          uint16_t* __restrict__ dcol, float* __restrict__ lo,
                                                          int32_t* __restrict__ c0, T* __restrict__ dg,
                                                          double* __restrict__ rs64, double* __restrict__ diag64,
                                                          int32_t cap, Sell<T> A) {
    const int64_t bid = xcd_block(blockIdx.x, gridDim.x);
    const int64_t r = bid * blockDim.x + threadIdx.x;
    __shared__ WinRange tabs[WIN ? kWinParts * kWinRanges : 1];
    const WinRange* tab = tabs;
    if constexpr (WIN) {
        static_assert(kBlock == kWinRows && kWinParts * kWinRanges <= kBlock, "one block's windows");
        if (bid * kWinRows >= nv.n) return;
        if (threadIdx.x < kWinParts * kWinRanges) tabs[threadIdx.x] = A.win[bid * (kWinParts * kWinRanges) + threadIdx.x];
        __syncthreads();
        tab += (threadIdx.x / (kWinRows / (tabs[0].head >> 16))) * kWinRanges;
    }
    if (r >= nslices * kWave) return;
    const Grid& g = nv.g;
    const int64_t s = r / kWave;
    const bool valid = r < nv.n;
    const int32_t row = valid ? (int32_t)r : 0;
    const int kind = valid ? row_kind(pv, op, row) : kRowNone;
    int32_t c = kind != kRowNone ? creal[row] : 0;
    const bool listed = c <= cap;
    const int32_t* lst = list + list_base(r, cap);
    double* wl = wlist + (r / kWave) * ((int64_t)cap * kWave) + r % kWave;  // entry k at wl[k * kWave]
    const Pos4 pb = nv.pos[row];
    const double mu_b = pv.mu[row], ir_b = pv.inv_rho[row];
    const bool f32 = op.f32cell != 0;
    const auto weight = [&](int32_t a, double r2) {
        if (kind != kRowFluid) return pair_W(g, r2);
        const double2 ma = pv.mu_mr[a];
        return pair_w_v(g, op.avg, ma.x, ma.y, mu_b, ir_b, r2);
    };
    // the paper's single precision: FP32 weight from cell-relative positions
    const int32_t cb = nv.scell[row];
    const float mub32 = (float)mu_b, rhob32 = (float)pv.rho[row];
    const auto weight32 = [&](int32_t a) -> double {
        const float r2 = dist2_f32(g, pb, cb, nv.pos[a], nv.scell[a]);
        if (kind != kRowFluid) return (double)wendland_W_f32(g, r2);
        return (double)pair_w_f32(g, op.avg, (float)pv.mu[a], (float)pv.mass[a], (float)pv.rho[a], mub32, rhob32,
                                  r2);
    };
    const auto scan = [&](auto&& f) {  // unlisted rows: the scan again
        for_each_neighbor(nv, row, [&](int32_t a, double r2) {
            if (kind == kRowDummy && pv.type[a] != SPH_FLUID) return;
            f(a, r2);
        });
    };
    double sum = 0.0;
    float sum32 = 0.f, cmp32 = 0.f;  // compensated FP32 sum (f32)
    const auto add = [&](double w) {
        if (f32) kahan_add(sum32, cmp32, (float)w);
        else sum += w;
    };
    if (listed && !f32) {
        // groups of kFillGroup entries: indices, then positions and
        // neighbour data loaded together, then the weights in list order
        for (int32_t k0 = 0; k0 < c; k0 += kFillGroup) {
            int32_t a[kFillGroup];
#pragma unroll
            for (int u = 0; u < kFillGroup; ++u) a[u] = k0 + u < c ? lst[list_off(k0 + u)] : row;
            Pos4 pa[kFillGroup];
            double2 ma[kFillGroup];
#pragma unroll
            for (int u = 0; u < kFillGroup; ++u) pa[u] = nv.pos[a[u]];
            if (kind == kRowFluid) {
#pragma unroll
                for (int u = 0; u < kFillGroup; ++u) ma[u] = pv.mu_mr[a[u]];
            }
#pragma unroll
            for (int u = 0; u < kFillGroup; ++u) {
                if (k0 + u >= c) break;
                // r^2 exactly as the scan computes it
                const double dx = disp(pb.x, pa[u].x, g.period[0]);
                const double dy = disp(pb.y, pa[u].y, g.period[1]);
                const double dz = disp(pb.z, pa[u].z, g.period[2]);
                const double r2 = (dx * dx + dy * dy) + dz * dz;
                const double w = kind != kRowFluid ? pair_W(g, r2)
                                                   : pair_w_v(g, op.avg, ma[u].x, ma[u].y, mu_b, ir_b, r2);
                wl[(k0 + u) * kWave] = w;
                add(w);
            }
        }
    } else if (listed) {
        for (int32_t k = 0; k < c; ++k) {
            const int32_t a = lst[list_off(k)];
            const double w = weight32(a);
            wl[k * kWave] = w;
            add(w);
        }
    } else {
        scan([&](int32_t a, double r2) { add(f32 ? weight32(a) : weight(a, r2)); });
    }
    if (f32) sum = (double)sum32;
    const float D32 = kind == kRowFluid ? 1.0f + (float)op.dt * sum32 : 1.0f;
    const double D = f32 ? (double)D32 : (kind == kRowFluid ? 1.0 + op.dt * sum : 1.0);
    if (kind == kRowDummy && !(sum > 0.0)) c = 0;  // identity row
    const auto coefficient = [&](double w) {
        if (f32) {
            if (kind == kRowFluid) {
                const float aba = -((float)op.dt * (float)w);
                return (double)(op.jacobi ? aba / D32 : aba);
            }
            return (double)((float)w / sum32);
        }
        if (kind == kRowFluid) {
            const double aba = -op.dt * w;
            return op.jacobi ? aba / D : aba;
        }
        return w / sum;
    };
    const int32_t width = (int32_t)((sl_ptr[s + 1] - sl_ptr[s]) / kWave);
    const int64_t lb = lane_base<T>(sl_ptr[s], r % kWave);
    auto wr = [&] {
        if constexpr (WIN) {
            // a padding row beyond the last particle codes its slice's first row
            WinWriter<T> ww{coef, dcol, lo, lb, tab, 0};
            ww.own = ww.code((int32_t)(valid ? r : s * kWave));
            ww.q = 0;
            return ww;
        } else {
            return RowWriter<T>{coef, dcol, lo, lb};
        }
    }();
    int32_t first = row;
    double csum = 0.0;  // f32: FP64 sum of the stored coefficients
    if (listed) {
        for (int32_t k = 0; k < c; ++k) {
            const int32_t a = lst[list_off(k)];
            if (k == 0) first = a;
            const double cv = coefficient(wl[k * kWave]);
            csum += cv;
            wr.put(a, cv);
        }
    } else if (c > 0) {
        scan([&](int32_t a, double r2) {
            if (wr.j == 0) first = a;
            const double cv = coefficient(f32 ? weight32(a) : weight(a, r2));
            csum += cv;
            wr.put(a, cv);
        });
    }
    wr.pad(width);
    if (valid) {
        c0[row] = first;
        if (f32) {
            // the plain diagonal A_rr (1 when scaled, on identity and on
            // dummy rows); the FP64 row sum of the stored FP32 matrix for
            // the difference form of the true residual
            const double dd = kind == kRowFluid && !op.jacobi ? D : 1.0;
            dg[row] = (T)dd;
            rs64[row] = dd + csum;
        } else {
            // row sums: 1/A_rr (Jacobi) or 1 on fluid rows (eqs. diag, offdiag),
            // 2 on dummy rows with fluid neighbours (eq. implicit-system-dummy-full),
            // 1 on identity rows
            const double rs = kind == kRowFluid ? (op.jacobi ? 1.0 / D : 1.0) : (c > 0 ? 2.0 : 1.0);
            dg[row] = (T)rs;
            rs64[row] = rs;
        }
        diag64[row] = D;
    }
}

// The fill of a windowed FP64-evaluated matrix whose rows are all listed: one
// block per slice, lane = row, the four waves sharing the rows' entries in
// blocks of 8 (wave w takes entries 32 t + 8 w + 0..7): weights first, kept in
// registers and laid out in LDS in list order, where every wave adds them up
// one after the other (the same sum as one thread's); then each wave scales
// its own weights and writes their slots, whole packs of the slice at a time.
// Against one lane per row for the whole row this has a quarter of the serial
// work per wave and no weights in memory: 80 -> 26 us at 5,632 particles, 1.33
// -> 0.83 ms at 1.16M, 38.9 -> 25.4 ms at 33.7M, 821 -> 630 us at 187k with the
// Gaussian kernel (whose longer rows take eight waves).  What bounds it is the
// L1 look-ups of its gathers, three 16-byte pieces per entry and lane; three
// waves per SIMD (168 registers, spills) were slower, 29.0 ms.
template <typename T, int CAP, int W>
__global__ __launch_bounds__(W* kWave) __attribute__((amdgpu_waves_per_eu(2))) void k_slice_fill(NbrView nv, PartView pv, OpParams op, int64_t nslices,
                                                       const int32_t* __restrict__ creal,
                                                       const int32_t* __restrict__ list,
                                                       const int64_t* __restrict__ sl_ptr, T* __restrict__ coef,
                                                       uint16_t* __restrict__ dcol, float* __restrict__ lo,
                                                       T* __restrict__ dg, double* __restrict__ rs64,
                                                       double* __restrict__ diag64, const WinRange* __restrict__ win) {
    constexpr int kW = W;
    constexpr int E = 8;                              // entries of a wave per round
    constexpr int R = (CAP + E * kW - 1) / (E * kW);  // rounds
    constexpr int P = pack_of<T>();
    static_assert(CAP % E == 0 && kChunk % E == 0 && E % P == 0, "whole groups");
    __shared__ double buf[2][E * kW][kWave];
    __shared__ WinRange tab[kWinRanges];
    const int64_t s = xcd_block(blockIdx.x, gridDim.x);
    if (s >= nslices) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t r = s * kWave + lane;
    const Grid& g = nv.g;
    {  // the window that serves the slice
        const int64_t blk = s / (kWinRows / kWave);
        const int32_t np = win[blk * kWinParts * kWinRanges].head >> 16;
        const int32_t part = (int32_t)(s % (kWinRows / kWave)) * np / (kWinRows / kWave);
        if (threadIdx.x < kWinRanges) tab[threadIdx.x] = win[(blk * kWinParts + part) * kWinRanges + threadIdx.x];
    }
    const bool valid = r < nv.n;
    const int32_t row = (int32_t)(valid ? r : s * kWave);  // lanes beyond the last row pad with the slice's first
    const int kind = valid ? row_kind(pv, op, row) : kRowNone;
    const int32_t c = kind != kRowNone ? creal[row] : 0;
    const int32_t width = (int32_t)((sl_ptr[s + 1] - sl_ptr[s]) / kWave);
    const int32_t* lst = list + list_base(s * kWave + lane, CAP);
    const Pos4 pb = nv.pos[row];
    const double mu_b = pv.mu[row], ir_b = pv.inv_rho[row];
    double w[R][E];
    int32_t a[R][E];
    double sum = 0.0;
#pragma unroll
    for (int t = 0; t < R; ++t) {
        const int32_t k0 = t * E * kW + wid * E;
#pragma unroll
        for (int u = 0; u < E; ++u) a[t][u] = k0 + u < c ? lst[list_off(k0 + u)] : row;
    }
#pragma unroll
    for (int t = 0; t < R; ++t) {
        if (t * E * kW >= width) break;
        const int32_t k0 = t * E * kW + wid * E;
        Pos4 pa[E];
        double2 ma[E];
#pragma unroll
        for (int u = 0; u < E; ++u) pa[u] = nv.pos[a[t][u]];
#pragma unroll
        for (int u = 0; u < E; ++u) ma[u] = pv.mu_mr[a[t][u]];
#pragma unroll
        for (int u = 0; u < E; ++u) {
            // r^2 exactly as the scan computes it
            const double dx = disp(pb.x, pa[u].x, g.period[0]);
            const double dy = disp(pb.y, pa[u].y, g.period[1]);
            const double dz = disp(pb.z, pa[u].z, g.period[2]);
            const double r2 = (dx * dx + dy * dy) + dz * dz;
            double v = 0.0;  // (adding 0 to the sum of a shorter row changes nothing)
            if (k0 + u < c)
                v = kind != kRowFluid ? pair_W(g, r2) : pair_w_v(g, op.avg, ma[u].x, ma[u].y, mu_b, ir_b, r2);
            w[t][u] = v;
            buf[t & 1][wid * E + u][lane] = v;
        }
        __syncthreads();  // (the other buffer is read in the next round only after its own barrier)
#pragma unroll
        for (int u = 0; u < E * kW; ++u) sum += buf[t & 1][u][lane];
    }
    if (width == 0) __syncthreads();  // (tab)
    const double D = kind == kRowFluid ? 1.0 + op.dt * sum : 1.0;
    const bool identity = kind == kRowNone || (kind == kRowDummy && !(sum > 0.0));
    const int64_t base = lane_base<T>(sl_ptr[s], lane);
    // the range of the last column coded: its end, and base - beg
    int32_t q = -1, q_end = 0, q_off = 0;
    const auto code = [&](int32_t col) {
        while (col >= q_end) {
            const WinRange x = tab[++q];
            q_end = x.beg + x.len;
            q_off = x.base - x.beg;
        }
        return (uint16_t)((col + q_off) * kWinStep);
    };
    const uint16_t own = code(row);
    q = -1;
    q_end = 0;
#pragma unroll
    for (int t = 0; t < R; ++t) {
        if (t * E * kW >= width) break;
        const int32_t k0 = t * E * kW + wid * E;
#pragma unroll
        for (int e = 0; e < E / P; ++e) {
            if (k0 + e * P >= width) break;
            typename Pack<T, P>::v cv;
            typename Pack<uint16_t, P>::v dv;
            typename Pack<float, P>::v lv;
#pragma unroll
            for (int u = 0; u < P; ++u) {
                const int32_t k = k0 + e * P + u;
                const bool on = k < c && !identity;
                double v = 0.0;
                if (on) {
                    if (kind == kRowFluid) {
                        const double aba = -op.dt * w[t][e * P + u];
                        v = op.jacobi ? aba / D : aba;
                    } else {
                        v = w[t][e * P + u] / sum;
                    }
                }
                cv[u] = (T)v;
                dv[u] = cv[u] != T(0) ? code(a[t][e * P + u]) : own;  // (zeros and padding: see WinWriter)
                if constexpr (sizeof(T) == 4) lv[u] = (float)(v - (double)cv[u]);
            }
            const int64_t i = slot_of<T>(base, k0 + e * P);
            *reinterpret_cast<typename Pack<T, P>::v*>(coef + i) = cv;
            *reinterpret_cast<typename Pack<uint16_t, P>::v*>(dcol + i) = dv;
            if constexpr (sizeof(T) == 4) *reinterpret_cast<typename Pack<float, P>::v*>(lo + i) = lv;
        }
    }
    if (valid && wid == 0) {
        // row sums: 1/A_rr (Jacobi) or 1 on fluid rows (eqs. diag, offdiag),
        // 2 on dummy rows with fluid neighbours (eq. implicit-system-dummy-full),
        // 1 on identity rows
        const double rs = kind == kRowFluid ? (op.jacobi ? 1.0 / D : 1.0) : (identity || c == 0 ? 1.0 : 2.0);
        dg[row] = (T)rs;
        rs64[row] = rs;
        diag64[row] = D;
    }
}

sph_status row_diag64(sph_ctx* ctx, const sph_nbr* nb, const PartView& pv, const OpParams& op,
                      const double** diag64) {
    double* d = nullptr;
    SPH_TRY(ctx->ensure_t(kDiag64, nb->n, &d));
    hipLaunchKernelGGL(k_row_count, dim3((unsigned)ceil_div(nb->n, kBlock)), dim3(kBlock), 0, ctx->stream,
                       nb->view(), pv, op, (int32_t*)nullptr, (int32_t*)nullptr, d, (double*)nullptr);
    SPH_LAUNCHED("k_row_count");
    *diag64 = d;
    return SPH_OK;
}

// The scan, and with win the operator's windows (by cells in the same launch);
// cnt: slots of the delta code per row (by rows only, may be null).
static void launch_row_scan(sph_ctx* ctx, const sph_nbr* nb, const PartView& pv, const OpParams& op, bool all,
                            bool by_rows, int32_t* cnt, int32_t* creal, int32_t* list, int32_t cap, WinRange* win,
                            int32_t* wmax) {
    constexpr int64_t kW = kBlock / kWave;
    const int64_t wblk = win ? ceil_div(ceil_div(nb->n, (int64_t)kWinRows), kW) : 0;
    if (by_rows) {
        if (win)
            hipLaunchKernelGGL(k_row_scan, dim3((unsigned)wblk), dim3(kBlock), 0, ctx->stream, nb->view(), pv, op,
                               nb->ncell, 1, all, creal, list, cap, (int32_t)wblk, win, wmax);
        const int64_t blocks = ceil_div(ceil_div(nb->n, (int64_t)kBlock), (int64_t)kNumXcd) * kNumXcd;
        hipLaunchKernelGGL(k_row_scan_rows, dim3((unsigned)blocks), dim3(kBlock), 0, ctx->stream, nb->view(), pv, op,
                           all, cnt, creal, list, cap);
        return;
    }
    // four waves per SIMD (what the scan's registers allow) on every CU
    int32_t split = 1;
    while (split < 8 && nb->ncell * split < 4096) split *= 2;
    const int64_t sblk = ceil_div(ceil_div(nb->ncell * split, kW), (int64_t)kNumXcd) * kNumXcd;
    hipLaunchKernelGGL(k_row_scan, dim3((unsigned)(wblk + sblk)), dim3(kBlock), 0, ctx->stream, nb->view(), pv, op,
                       nb->ncell, split, all, creal, list, cap, (int32_t)wblk, win, wmax);
}

// Lists of every particle's neighbours for the canonical export: caller order,
// columns ascending.  A wave per row reads the row's list, maps it to the
// caller's indices and ranks the entries against each other in registers.
template <int CAP>
__global__ __launch_bounds__(kBlock) void k_export_rows(int64_t n, const int32_t* __restrict__ creal,
                                                        const int32_t* __restrict__ list,
                                                        const int32_t* __restrict__ perm,
                                                        const int64_t* __restrict__ row_ptr,
                                                        int32_t* __restrict__ cols) {
    constexpr int E = (CAP + kWave - 1) / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t r = (int64_t)xcd_block(blockIdx.x, gridDim.x) * (kBlock / kWave) + threadIdx.x / kWave;
    if (r >= n) return;
    const int32_t c = __builtin_amdgcn_readfirstlane(creal[r]);
    if (c > CAP) return;  // no list: k_fill_orig
    const int32_t* lst = list + list_base(r, CAP);
    int32_t* out = cols + row_ptr[perm[r]];
    int32_t v[E], rank[E];
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const int32_t k = j * kWave + lane;
        v[j] = k < c ? perm[lst[list_off(k)]] : INT32_MAX;
        rank[j] = 0;
    }
#pragma unroll
    for (int i = 0; i < E; ++i) {
        const int32_t m = min(c - i * kWave, kWave);
        for (int32_t l = 0; l < m; ++l) {
            const int32_t x = __builtin_amdgcn_readlane(v[i], l);
#pragma unroll
            for (int j = 0; j < E; ++j) rank[j] += x < v[j];
        }
    }
#pragma unroll
    for (int j = 0; j < E; ++j)
        if (j * kWave + lane < c) out[rank[j]] = v[j];
}

int32_t export_cap(const sph_nbr* nb) {
    const int32_t cap = nb->g.kernel == SPH_KERNEL_GAUSSIAN ? kListCapGauss : kListCap;
    if (export_without_lists(nb->occupancy())) return 0;
    return (size_t)ceil_div(nb->n, (int64_t)kWave) * kWave * cap * 4 <= kListBudget ? cap : 0;
}

sph_status neighbour_scan(sph_ctx* ctx, const sph_nbr* nb, int32_t cap, int32_t* count, int32_t** list) {
    int32_t* l = nullptr;
    if (cap > 0) SPH_TRY(ctx->ensure_t(kList, (size_t)ceil_div(nb->n, (int64_t)kWave) * kWave * cap, &l));
    launch_row_scan(ctx, nb, PartView{}, OpParams{}, true, scan_by_rows(nb->occupancy(), cap > 0 ? cap : kListCapGauss),
                    nullptr, count, l, cap, nullptr, nullptr);
    SPH_LAUNCHED("k_row_scan");
    if (list) *list = l;
    return SPH_OK;
}

sph_status export_rows(sph_ctx* ctx, const sph_nbr* nb, int32_t cap, const int32_t* count, const int32_t* list,
                       const int64_t* row_ptr, int32_t* cols) {
    const int64_t blocks = ceil_div(ceil_div(nb->n, (int64_t)(kBlock / kWave)), (int64_t)kNumXcd) * kNumXcd;
    if (cap == kListCap)
        hipLaunchKernelGGL(k_export_rows<kListCap>, dim3((unsigned)blocks), dim3(kBlock), 0, ctx->stream, nb->n, count,
                           list, nb->perm, row_ptr, cols);
    else
        hipLaunchKernelGGL(k_export_rows<kListCapGauss>, dim3((unsigned)blocks), dim3(kBlock), 0, ctx->stream, nb->n,
                           count, list, nb->perm, row_ptr, cols);
    SPH_LAUNCHED("k_export_rows");
    return SPH_OK;
}

template <typename T>
sph_status build_sell(sph_ctx* ctx, const sph_nbr* nb, const PartView& pv, const OpParams& op, Sell<T>* out,
                      const double** diag64, int64_t* nnz_out, int64_t* slots_out, bool once) {
    const int64_t n = nb->n;
    const int64_t nslices = ceil_div(n, kWave);
    // Test hook: the environment variable SPH_BUILD_LEGACY=1 selects the
    // build that evaluates the coefficients inside the neighbour scan, the
    // reference the list-based build is tested against bit for bit.
    if (op.f32cell && nb->g.kernel != SPH_KERNEL_WENDLAND)
        return ctx->fail(SPH_E_ARG, "SPH_OP_PAPER32 is defined for the Wendland kernel");
    const bool legacy = env_int("SPH_BUILD_LEGACY", 0) > 0 && !op.f32cell;
    // list entries per row: room for every neighbour of the kernel's support
    // (int32 index + FP64 weight each) while that fits the budget
    const int32_t cap = nb->g.kernel == SPH_KERNEL_GAUSSIAN &&
                                (size_t)nslices * kWave * kListCapGauss * 12 <= kListBudget
                            ? kListCapGauss
                            : kListCap;
    const Occupancy occ = nb->occupancy();
    const bool by_rows = scan_by_rows(occ, cap);
    const bool windows = !legacy && !delta_coded(occ, cap) && !(once && crowded_scan(occ));
    int32_t *cnt = nullptr, *creal = nullptr, *list = nullptr;
    double *d = nullptr, *ws = nullptr, *wlist = nullptr;
    int64_t *size = nullptr, *ptr = nullptr;
    SPH_TRY(ctx->ensure_t(kCntReal, n, &creal));
    SPH_TRY(ctx->ensure_t(kDiag64, n, &d));
    SPH_TRY(ctx->ensure_t(kSlSize, nslices, &size));
    SPH_TRY(ctx->ensure_t(kSlPtr, nslices + 1, &ptr));
    unsigned long long* nnz_dev = nullptr;  // [0] nonzeros, [1] longest row, [2] largest window
    SPH_TRY(ctx->ensure_t(kNnzCount, 3, &nnz_dev));
    SPH_HIP(hipMemsetAsync(nnz_dev, 0, 3 * sizeof(unsigned long long), ctx->stream));
    // windows of the operator's blocks; [2] of the counters: the largest
    WinRange* win = nullptr;
    if (windows)
        SPH_TRY(ctx->ensure_t(kWin, (size_t)ceil_div(n, (int64_t)kWinRows) * kWinParts * kWinRanges, &win));
    // slice kernels: whole XCD rounds of blocks (xcd_block needs a multiple of 8)
    const dim3 slice_grid((unsigned)(ceil_div(ceil_div(nslices * kWave, kBlock), kNumXcd) * kNumXcd));
    if (legacy || by_rows) SPH_TRY(ctx->ensure_t(kCnt, n, &cnt));
    if (legacy) {
        SPH_TRY(ctx->ensure_t(kWsum, n, &ws));
        hipLaunchKernelGGL(k_row_count, dim3((unsigned)ceil_div(n, kBlock)), dim3(kBlock), 0, ctx->stream,
                           nb->view(), pv, op, cnt, creal, d, ws);
    } else {
        SPH_TRY(ctx->ensure_t(kList, (size_t)nslices * cap * kWave, &list));
        launch_row_scan(ctx, nb, pv, op, false, by_rows, cnt, creal, list, cap, win,
                        reinterpret_cast<int32_t*>(nnz_dev + 2));
    }
    hipLaunchKernelGGL(k_slice_size, dim3((unsigned)std::min<int64_t>(ceil_div(nslices * kWave, kBlock), 1024)),
                       dim3(kBlock), 0, ctx->stream,
                       n, nslices, (int32_t)pack_of<T>(), nb->view(), pv, op, (const int32_t*)list, cap,
                       reinterpret_cast<const int32_t*>(nnz_dev + 2),
                       windows ? kWinLimit : -1, cnt, creal, size, nnz_dev);
    SPH_LAUNCHED("k_row_count/k_slice_size");
    SPH_TRY(scan_i64(ctx, size, ptr, nslices));
    int64_t nnzp = 0;
    unsigned long long hcnt[3] = {0, 0, 0};
    SPH_HIP(hipMemcpyAsync(&nnzp, ptr + nslices, sizeof(int64_t), hipMemcpyDeviceToHost, ctx->stream));
    SPH_HIP(hipMemcpyAsync(hcnt, nnz_dev, sizeof(hcnt), hipMemcpyDeviceToHost, ctx->stream));
    SPH_HIP(hipStreamSynchronize(ctx->stream));
    const int32_t wmax = (int32_t)hcnt[2];
    const bool windowed = windows && wmax <= kWinLimit;
    if (nnz_out) *nnz_out = (int64_t)hcnt[0];
    if (slots_out) *slots_out = nnzp;
    T* coef = nullptr;
    uint16_t* dcol = nullptr;
    float* lo = nullptr;
    int32_t* c0 = nullptr;
    T* dg = nullptr;
    const size_t ns = (size_t)(nnzp > 0 ? nnzp : 1);
    out->win = win;
    out->wmax = windowed ? wmax : 0;
    SPH_TRY(ctx->ensure_t(kCoef, ns, &coef));
    SPH_TRY(ctx->ensure_t(kDcol, ns, &dcol));
    if constexpr (sizeof(T) == 4) SPH_TRY(ctx->ensure_t(kLo, ns, &lo));
    SPH_TRY(ctx->ensure_t(kC0, n, &c0));
    double* rs64 = nullptr;
    SPH_TRY(ctx->ensure_t(kDg, n, &dg));
    SPH_TRY(ctx->ensure_t(kRs64, n, &rs64));
    if (!legacy) {
        const bool listed = (int64_t)(uint32_t)hcnt[1] <= cap;  // (the longest row)
        const bool sliced = windowed && listed && !op.f32cell;
        if (!sliced) SPH_TRY(ctx->ensure_t(kWList, (size_t)nslices * cap * kWave, &wlist));
        // Occupancy limit of k_row_fill_list: the launch reserves LDS it does not use, so that
        // only two blocks share a CU.  The neighbour gathers of the rows in
        // flight on an XCD then fit its L2 (with eight blocks per CU they
        // did not): 8.1 -> 5.8 ms at 4.49M particles.
        constexpr size_t kFillLdsReserve = 60 * 1024;
        const dim3 wave_grid((unsigned)(ceil_div(nslices, kNumXcd) * kNumXcd));
        if (sliced && cap == kListCap)
            hipLaunchKernelGGL((k_slice_fill<T, kListCap, 4>), wave_grid, dim3(4 * kWave), 0, ctx->stream, nb->view(), pv, op,
                               nslices, creal, list, ptr, coef, dcol, lo, dg, rs64, d, win);
        else if (sliced)
            hipLaunchKernelGGL((k_slice_fill<T, kListCapGauss, 8>), wave_grid, dim3(8 * kWave), 0, ctx->stream,
                               nb->view(), pv, op, nslices, creal, list, ptr, coef, dcol, lo, dg, rs64, d, win);
        else if (windowed)
            hipLaunchKernelGGL((k_row_fill_list<T, true>), slice_grid, dim3(kBlock), kFillLdsReserve, ctx->stream,
                               nb->view(), pv, op, nslices, creal, list, wlist, ptr, coef, dcol, lo, c0, dg, rs64, d,
                               cap, *out);
        else
            hipLaunchKernelGGL((k_row_fill_list<T, false>), slice_grid, dim3(kBlock), kFillLdsReserve, ctx->stream,
                               nb->view(), pv, op, nslices, creal, list, wlist, ptr, coef, dcol, lo, c0, dg, rs64, d,
                               cap, *out);
        SPH_LAUNCHED("k_row_fill_list");
    } else {
        hipLaunchKernelGGL(k_row_fill<T>, dim3((unsigned)ceil_div(nslices * kWave, kBlock)), dim3(kBlock), 0,
                           ctx->stream, nb->view(), pv, op, d, ws, ptr, coef, dcol, lo, c0, dg, rs64, nslices);
        SPH_LAUNCHED("k_row_fill");
    }
    out->nslices = nslices;
    out->sl_ptr = ptr;
    out->coef = coef;
    out->dcol = dcol;
    out->lo = lo;
    out->c0 = c0;
    out->dg = dg;
    out->rs64 = rs64;
    if (diag64) *diag64 = d;
    return SPH_OK;
}

template sph_status build_sell<float>(sph_ctx*, const sph_nbr*, const PartView&, const OpParams&, Sell<float>*,
                                      const double**, int64_t*, int64_t*, bool);
template sph_status build_sell<double>(sph_ctx*, const sph_nbr*, const PartView&, const OpParams&,
                                       Sell<double>*, const double**, int64_t*, int64_t*, bool);


// Launch geometry of the row kernels.
Launch make_launch(int64_t n, bool fp64) {
    Launch L;
    L.n = n;
    const int64_t nslices = ceil_div(n, kWave);
    const int32_t ba = kApplyMaxBlock;
    const int64_t wpb = ba / kWave;
    // one 64-row slice per wave: the launch's tail is then one slice long
    // (measured fastest for whole iterations on the 1.16M and 4.49M tanks);
    // the grid is rounded up to a multiple of the XCD count, so that no block
    // gets more slices than it has waves
    int64_t ga = ceil_div(nslices, wpb);
    if (ga >= 64) ga = ceil_div(ga, kNumXcd) * kNumXcd;
    L.grid_apply = (int32_t)std::max<int64_t>(ga, 1);
    L.block_apply = ba;
    // streaming kernels: every block re-reduces the previous kernel's
    // partials, so each thread should stream at least 8 rows of the (at most
    // 256-block) grid: the largest power-of-two block up to 1024 that keeps
    // that (512 at N = 1.16M, 1024 from N = 2.1M; measured 28.8 against
    // 29.3 ms per step on the 1.16M tank, no change at 4.7M).  FP64 vectors,
    // twice the bytes per row, fill blocks of up to 512 threads with two rows
    // each (p update / close-out: 12.7 / 14.3 us with 128 threads at 328k
    // particles, 10.6 / 14.1 with 512).  FP32 vectors would gain less, and
    // their iterates depend on the order of the sums: a flipped rounding of a
    // scalar to FP32 moves a solution by a part of the tolerance.
    const int rows = fp64 ? 2 : 8;
    int32_t bs_def = !fp64 || (int64_t)1024 * 256 * 8 <= n ? 1024 : 512;
    while (bs_def > kWave && (int64_t)bs_def * 256 * rows > n) bs_def /= 2;
    const int32_t bs = bs_def;
    int64_t gs = std::min<int64_t>(ceil_div(n, (int64_t)bs * (fp64 ? 2 : 4)), 256);
    if (gs >= 64) gs = gs / kNumXcd * kNumXcd;
    L.grid_stream = (int32_t)std::max<int64_t>(gs, 1);
    L.block_stream = bs;
    return L;
}

template <typename T>
sph_status apply_plain(sph_ctx* ctx, const sph_nbr* nb, const PartView& pv, const OpParams& op, int mode,
                       const Sell<T>* sell, const T* x, T* y) {
    const Launch L = make_launch(nb->n, sizeof(T) == 8);
    if (mode == SPH_OP_PAPER32) {
        if constexpr (sizeof(T) == 4)
            launch_apply_sell<T, kDotNone, T, true>(ctx->stream, L, nullptr, *sell, x, y, nullptr, nullptr, nullptr);
        else
            return ctx->fail(SPH_E_ARG, "apply: SPH_OP_PAPER32 is single precision");
    } else if (mode == SPH_OP_CACHED) {
        launch_apply_sell<T, kDotNone>(ctx->stream, L, nullptr, *sell, x, y, nullptr, nullptr, nullptr);
    } else {
        launch_apply_otf<T, kDotNone>(ctx->stream, L, nullptr, nb, pv, op, x, y, nullptr, nullptr, nullptr);
    }
    SPH_LAUNCHED("apply");
    return SPH_OK;
}

template sph_status apply_plain<float>(sph_ctx*, const sph_nbr*, const PartView&, const OpParams&, int,
                                       const Sell<float>*, const float*, float*);
template sph_status apply_plain<double>(sph_ctx*, const sph_nbr*, const PartView&, const OpParams&, int,
                                        const Sell<double>*, const double*, double*);

}  // namespace sph

using namespace sph;

sph_status check_particles(sph_ctx* ctx, const sph_nbr* nb, const sph_particles* p) {
    if (!p) return ctx->fail(SPH_E_ARG, "null particles");
    if (p->n != nb->n) return ctx->fail(SPH_E_ARG, "particle count differs from the neighbour handle");
    if (!p->mass || !p->rho || !p->mu || !p->type) return ctx->fail(SPH_E_ARG, "null particle array");
    return SPH_OK;
}

sph_status check_params(sph_ctx* ctx, const sph_visc_params* v, int32_t prec) {
    if (!v) return ctx->fail(SPH_E_ARG, "null params");
    if (!(v->dt >= 0.0) || !std::isfinite(v->dt)) return ctx->fail(SPH_E_ARG, "params: dt must be finite and >= 0");
    if (v->wall != SPH_WALL_DYNAMIC && v->wall != SPH_WALL_DUMMY) return ctx->fail(SPH_E_ARG, "params: wall");
    if (v->avg != SPH_AVG_ARITH && v->avg != SPH_AVG_HARMONIC) return ctx->fail(SPH_E_ARG, "params: avg");
    if (v->op_mode != SPH_OP_CACHED && v->op_mode != SPH_OP_ONTHEFLY && v->op_mode != SPH_OP_PAPER32)
        return ctx->fail(SPH_E_ARG, "params: op_mode");
    if (prec != SPH_F32 && prec != SPH_F64) return ctx->fail(SPH_E_ARG, "prec");
    if (v->op_mode == SPH_OP_PAPER32 && prec != SPH_F32)
        return ctx->fail(SPH_E_ARG, "params: SPH_OP_PAPER32 is single precision (SPH_F32)");
    return SPH_OK;
}

template <typename T>
static sph_status apply_entry(sph_ctx* ctx, const sph_nbr* nb, const sph_particles* p,
                              const sph_visc_params* v, const void* const x[3], void* const y[3]) {
    PartView pv;
    SPH_TRY(gather_props(ctx, nb, p, &pv));
    OpParams op{v->dt, v->wall, v->avg, v->jacobi ? 1 : 0};
    T *xin = nullptr, *yout = nullptr;
    SPH_TRY(ctx->ensure_t(kApplyIn, (size_t)nb->n * 3 + kVecPad, &xin));
    SPH_TRY(ctx->ensure_t(kApplyOut, (size_t)nb->n * 3, &yout));
    SPH_TRY(gather_vec3<T>(ctx, nb, x, xin));
    Sell<T> sell{};
    if (v->op_mode == SPH_OP_PAPER32) op.f32cell = 1;
    if (v->op_mode != SPH_OP_ONTHEFLY) SPH_TRY(build_sell<T>(ctx, nb, pv, op, &sell, nullptr, nullptr, nullptr, true));
    SPH_TRY(apply_plain<T>(ctx, nb, pv, op, v->op_mode, &sell, xin, yout));
    SPH_TRY(scatter_vec3<T>(ctx, nb, yout, y));
    return SPH_OK;
}

extern "C" sph_status sph_visc_apply(sph_ctx* ctx, const sph_nbr* nb, const sph_particles* p,
                                     const sph_visc_params* params, int32_t prec, const void* const x[3],
                                     void* const y[3]) {
    if (!ctx) return SPH_E_ARG;
    if (!nb || !x || !y) return ctx->fail(SPH_E_ARG, "visc_apply: null argument");
    if (nb->device != ctx->device) return ctx->fail(SPH_E_ARG, "visc_apply: handle of another device");
    for (int c = 0; c < 3; ++c)
        if (!x[c] || !y[c]) return ctx->fail(SPH_E_ARG, "visc_apply: null vector");
    SPH_TRY(check_particles(ctx, nb, p));
    SPH_TRY(check_params(ctx, params, prec));
    if (prec == SPH_F64) return apply_entry<double>(ctx, nb, p, params, x, y);
    return apply_entry<float>(ctx, nb, p, params, x, y);
}
