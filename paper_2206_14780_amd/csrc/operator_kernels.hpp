// Operator kernels y = A x, optionally fused with the inner products the
// solver needs from the same pass (the paper's gemv plus dot products,
// appendix "Implementation notes").
#pragma once

#include <cmath>

#include "cell_rows.hpp"

namespace sph {

// Inner products produced per block alongside y = A x:
//   kDotA1     3 partials: w . y            (delta = r0hat . A p)
//   kDotA2     6 partials: x . y, y . y     (r* . A r*,  A r* . A r*)
//   kDotA2Std  9 partials: as kDotA2 plus x . x (textbook half-step check)
//   kDotResid  3 partials: y . y with y = b - A x evaluated in FP64 with the
//              FP64-accurate coefficients (true residual)
//   kDotCG     3 partials: <x, y>_D = sum_i D_i x_i y_i, the CG's p . A p in
//              the Jacobi-weighted inner product (D from the FP64 argument;
//              null: D = 1)
enum DotMode { kDotNone = 0, kDotA1 = 1, kDotA2 = 2, kDotA2Std = 3, kDotResid = 4, kDotCG = 5 };

template <int MODE>
struct DotK {
    static constexpr int K = MODE == kDotA1 ? 3 : MODE == kDotA2 ? 6 : MODE == kDotA2Std ? 9
                             : MODE == kDotResid ? 3 : MODE == kDotCG ? 3 : 1;
};

// KH: the paper's single precision (products rounded to FP32, compensated
// FP32 sums; see kahan_add), else FP64 products and sums.
template <typename T, int MODE, bool KH = false>
__device__ inline void accumulate_dots(double (&acc)[DotK<MODE>::K], float (&cmp)[DotK<MODE>::K], V3<T> xs,
                                       V3<T> yv, V3<T> wv, double dw = 1.0) {
    if constexpr (MODE == kDotCG) {
        dot_add_w<KH>(acc[0], cmp[0], dw, (double)xs.x, (double)yv.x);
        dot_add_w<KH>(acc[1], cmp[1], dw, (double)xs.y, (double)yv.y);
        dot_add_w<KH>(acc[2], cmp[2], dw, (double)xs.z, (double)yv.z);
    } else if constexpr (MODE == kDotA1) {
        dot_add<KH>(acc[0], cmp[0], (double)wv.x, (double)yv.x);
        dot_add<KH>(acc[1], cmp[1], (double)wv.y, (double)yv.y);
        dot_add<KH>(acc[2], cmp[2], (double)wv.z, (double)yv.z);
    } else if constexpr (MODE == kDotA2 || MODE == kDotA2Std) {
        dot_add<KH>(acc[0], cmp[0], (double)xs.x, (double)yv.x);
        dot_add<KH>(acc[1], cmp[1], (double)xs.y, (double)yv.y);
        dot_add<KH>(acc[2], cmp[2], (double)xs.z, (double)yv.z);
        dot_add<KH>(acc[3], cmp[3], (double)yv.x, (double)yv.x);
        dot_add<KH>(acc[4], cmp[4], (double)yv.y, (double)yv.y);
        dot_add<KH>(acc[5], cmp[5], (double)yv.z, (double)yv.z);
        if constexpr (MODE == kDotA2Std) {
            dot_add<KH>(acc[6], cmp[6], (double)xs.x, (double)xs.x);
            dot_add<KH>(acc[7], cmp[7], (double)xs.y, (double)xs.y);
            dot_add<KH>(acc[8], cmp[8], (double)xs.z, (double)xs.z);
        }
    }
}


// Column jump held in the coefficient bits of an escape slot.
__device__ inline int32_t jump_bits(float w) { return __float_as_int(w); }
__device__ inline int32_t jump_bits(double w) { return (int32_t)__double_as_longlong(w); }

// Entries per software-pipelined group: 16 for the FP32 operator (more
// loads in flight), 8 where FP64 values or the FP64-accurate residual would
// not fit the registers.
template <typename T, bool RES>
constexpr int group_of() { return sizeof(T) == 4 && !RES ? 16 : 8; }

// Raw slots of one group (zero beyond the row's width): a lane's kPack
// adjacent slots come in one vector load each for the coefficients, the
// column steps and (residual) the low parts.  Widths and groups are
// multiples of kPack, so a pack is either wholly inside the row or beyond it.
template <typename T, int P>
struct Pack {
    typedef T v __attribute__((ext_vector_type(P)));
};
template <typename T>
struct Pack<T, 1> {
    typedef T v;
};

template <typename T, int P>
__device__ inline T pack_elem(const typename Pack<T, P>::v& v, int e) {
    if constexpr (P == 1) return v;
    else return v[e];
}

template <typename T, bool RES>
__device__ inline void sell_group(const Sell<T>& A, int64_t base, int32_t width, int32_t k0,
                                  T (&w)[group_of<T, RES>()], uint16_t (&d)[group_of<T, RES>()],
                                  double (&l)[group_of<T, RES>()]) {
    constexpr int kGroup = group_of<T, RES>();
    constexpr int P = pack_of<T>();
    static_assert(kGroup % P == 0, "whole packs per group");
#pragma unroll
    for (int q = 0; q < kGroup / P; ++q) {
        const int32_t k = k0 + q * P;
        if (k < width) {
            const int64_t i = slot_of<T>(base, k);
            // read once per launch: non-temporal, so the stream does not
            // evict the x values that the gathers reuse from L2
            const typename Pack<T, P>::v wv =
                __builtin_nontemporal_load(reinterpret_cast<const typename Pack<T, P>::v*>(A.coef + i));
            const typename Pack<uint16_t, P>::v dv =
                __builtin_nontemporal_load(reinterpret_cast<const typename Pack<uint16_t, P>::v*>(A.dcol + i));
#pragma unroll
            for (int e = 0; e < P; ++e) {
                w[q * P + e] = pack_elem<T, P>(wv, e);
                d[q * P + e] = pack_elem<uint16_t, P>(dv, e);
            }
            if constexpr (RES && sizeof(T) == 4) {
                const typename Pack<float, P>::v lv =
                    __builtin_nontemporal_load(reinterpret_cast<const typename Pack<float, P>::v*>(A.lo + i));
#pragma unroll
                for (int e = 0; e < P; ++e) l[q * P + e] = (double)pack_elem<float, P>(lv, e);
            } else {
#pragma unroll
                for (int e = 0; e < P; ++e) l[q * P + e] = 0.0;
            }
        } else {
#pragma unroll
            for (int e = 0; e < P; ++e) {
                w[q * P + e] = T(0);
                d[q * P + e] = 0;
                l[q * P + e] = 0.0;
            }
        }
    }
}

// sum_k coef[r,k] (x[col[r,k]] - x_r) for the row of this lane (the operator's
// difference form: rounding scales with the local variation of x, not with x,
// so smooth fields keep their accuracy in FP32).  `base` is the lane's first
// slot, `width` the slice width (uniform across the wave).  The loop is
// software-pipelined: the gathers of group g are issued before the slot loads
// of group g + 1, so the L2 latency of the gathers and the HBM latency of the
// matrix stream overlap; the column steps of a group are summed before its
// gathers.  RES accumulates in FP64 with the FP64-accurate coefficients; x
// may then be of another precision XT than the matrix (an FP64 solution
// under an FP32 operator).
template <typename T, bool RES, typename ACC, typename XT = T>
__device__ inline void sell_row(const Sell<T>& A, int64_t base, int32_t width, int32_t row,
                                const XT* __restrict__ x, const V3<XT>& xs, ACC& a0, ACC& a1, ACC& a2) {
    constexpr int kGroup = group_of<T, RES>();
    int32_t col = A.c0[row];
    T rw[kGroup];
    uint16_t rd[kGroup];
    double rl[kGroup];
    sell_group<T, RES>(A, base, width, 0, rw, rd, rl);
    for (int32_t k0 = 0; k0 < width; k0 += kGroup) {
        int32_t cc[kGroup];
        T cw[kGroup];
        double cl[kGroup];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            const bool esc = rd[u] == kEscape;
            col += esc ? jump_bits(rw[u]) : (int32_t)rd[u];
            cw[u] = esc ? T(0) : rw[u];
            cl[u] = esc ? 0.0 : rl[u];
            // escape and padding slots (zero weight) gather the lane's own
            // row: the 64 lanes' own rows share a few cache lines, where
            // their last columns would scatter over many
            cc[u] = (cw[u] == T(0) && cl[u] == 0.0) ? row : col;
        }
        V3<XT> xv[kGroup];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) xv[u] = ld3(x, cc[u]);
        sell_group<T, RES>(A, base, width, k0 + kGroup, rw, rd, rl);
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            if constexpr (RES) {
                const double w = (double)cw[u] + cl[u];
                a0 += w * ((double)xv[u].x - (double)xs.x);
                a1 += w * ((double)xv[u].y - (double)xs.y);
                a2 += w * ((double)xv[u].z - (double)xs.z);
            } else {
                a0 = fma_t(cw[u], xv[u].x - xs.x, a0);
                a1 = fma_t(cw[u], xv[u].y - xs.y, a1);
                a2 = fma_t(cw[u], xv[u].z - xs.z, a2);
            }
        }
    }
}

// The paper's single-precision gemv of one row: y_r = A_rr x_r + sum_k
// coef[r,k] x[col[r,k]] with every product rounded to FP32 and the terms
// added in slot order by Kahan's compensated summation (zero-weight escape
// and padding slots add nothing).  d: the plain diagonal A_rr.
__device__ inline void sell_row_kahan(const Sell<float>& A, int64_t base, int32_t width, int32_t row,
                                      const float* __restrict__ x, const V3<float>& xs, float d, V3<float>& y) {
    constexpr int kGroup = group_of<float, false>();
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, c0 = 0.f, c1 = 0.f, c2 = 0.f;
    kahan_add(s0, c0, d * xs.x);
    kahan_add(s1, c1, d * xs.y);
    kahan_add(s2, c2, d * xs.z);
    int32_t col = A.c0[row];
    float rw[kGroup];
    uint16_t rd[kGroup];
    double rl[kGroup];
    sell_group<float, false>(A, base, width, 0, rw, rd, rl);
    for (int32_t k0 = 0; k0 < width; k0 += kGroup) {
        int32_t cc[kGroup];
        float cw[kGroup];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            const bool esc = rd[u] == kEscape;
            col += esc ? jump_bits(rw[u]) : (int32_t)rd[u];
            cw[u] = esc ? 0.f : rw[u];
            cc[u] = cw[u] == 0.f ? row : col;
        }
        V3<float> xv[kGroup];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) xv[u] = ld3(x, cc[u]);
        sell_group<float, false>(A, base, width, k0 + kGroup, rw, rd, rl);
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            if (cw[u] != 0.f) {
                kahan_add(s0, c0, cw[u] * xv[u].x);
                kahan_add(s1, c1, cw[u] * xv[u].y);
                kahan_add(s2, c2, cw[u] * xv[u].z);
            }
        }
    }
    y = V3<float>{s0, s1, s2};
}

// ---------------------------------------------------------------------------
// Windowed rows.
// ---------------------------------------------------------------------------
template <typename XT>
constexpr size_t win_bytes(int32_t wmax) { return (size_t)wmax * 3 * sizeof(XT); }

// Copies a window of nr ranges (lane r holds range r) into LDS: 16-byte units
// by the direct global-to-LDS load (no registers, every unit in flight at
// once), each wave taking whole runs of 64 units.  Ends with a barrier.
template <typename XT>
__device__ inline void win_stage(const WinRange& mine, int32_t nr, const XT* __restrict__ x, unsigned char* lds) {
    constexpr int U = 16 / sizeof(XT);
    typedef const __attribute__((address_space(1))) void* gptr;
    typedef __attribute__((address_space(3))) void* lptr;
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    for (int32_t r = 0; r < nr; ++r) {
        const WinRange t{__builtin_amdgcn_readlane(mine.beg, r), __builtin_amdgcn_readlane(mine.len, r),
                         __builtin_amdgcn_readlane(mine.base, r), 0};
        const int64_t e0 = 3 * (int64_t)t.beg;
        const int32_t pre = (int32_t)(e0 % U);
        const int32_t nv = (pre + 3 * t.len + U - 1) / U;
        const XT* src = x + (e0 - pre);
        XT* dst = reinterpret_cast<XT*>(lds) + (3 * t.base - pre);
        for (int32_t v = wid * kWave; v < nv; v += (int32_t)blockDim.x)
            if (v + lane < nv)
                __builtin_amdgcn_global_load_lds((gptr)(src + (int64_t)(v + lane) * U), (lptr)(dst + v * U), 16, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
}

// Stages the windows of block `bid` in turn and calls f() in the waves whose
// rows the staged window serves.  Called by the whole block.
template <typename T, typename XT, typename F>
__device__ __forceinline__ void win_parts(const Sell<T>& A, int64_t bid, const XT* __restrict__ x, unsigned char* lds, F&& f) {
    if (bid * kWinRows >= A.nslices * kWave) return;
    // one load per lane brings a window's table (a scalar load per range, one
    // after the other, took longer than the copy)
    const WinRange* tab = A.win + bid * kWinParts * kWinRanges + (threadIdx.x & (kWinRanges - 1));
    WinRange r = *tab;
    const int32_t head = __builtin_amdgcn_readfirstlane(r.head);
    const int32_t np = head >> 16;
    win_stage(r, head & 0xFFFF, x, lds);
    if constexpr (sizeof(XT) == 8) {
        // a path of its own for the one-window block: with FP64 windows the
        // LDS, not the registers it costs (160 against 100), bounds the
        // blocks per CU; FP32 takes the shared path and four blocks
        if (np == 1) {
            f();
            return;
        }
    }
    const int32_t own = threadIdx.x / (kWinRows / np);
    for (int32_t k = 0;;) {
        if (own == k) f();
        if (++k == np) break;
        r = tab[k * kWinRanges];
        __syncthreads();
        win_stage(r, __builtin_amdgcn_readfirstlane(r.head) & 0xFFFF, x, lds);
    }
}

// One group of slots in registers: the coefficients, the packed column codes
// and (residual) the coefficients' low parts.
template <typename T, bool RES>
struct WinGroup {
    static constexpr int P = pack_of<T>();
    static constexpr int N = sizeof(T) == 4 ? (RES ? 8 : 16) : 8;  // slots
    typedef uint16_t idv __attribute__((ext_vector_type(P)));
    typename Pack<T, P>::v c[N / P];
    idv d[N / P];
    typename Pack<float, P>::v l[RES && sizeof(T) == 4 ? N / P : 1];
    // slots k0 .. k0 + N - 1 below the slice width (uniform branches)
    __device__ __forceinline__ void load(const Sell<T>& A, int64_t base, int32_t width, int32_t k0) {
#pragma unroll
        for (int q = 0; q < N / P; ++q) {
            if (k0 + q * P < width) {
                const int64_t i = slot_of<T>(base, k0 + q * P);
                // read once per launch: non-temporal, so that the stream does
                // not evict x from L2
                c[q] = __builtin_nontemporal_load(reinterpret_cast<const typename Pack<T, P>::v*>(A.coef + i));
                d[q] = __builtin_nontemporal_load(reinterpret_cast<const idv*>(A.dcol + i));
                if constexpr (RES && sizeof(T) == 4)
                    l[q] = __builtin_nontemporal_load(reinterpret_cast<const typename Pack<float, P>::v*>(A.lo + i));
            }
        }
    }
};

// The slots of a row as a ring of groups in registers: D groups are in flight
// at once, the first of them from before the window is staged.
template <typename T, bool RES, typename XT>
struct WinStream {
    typedef WinGroup<T, RES> G;
    static constexpr int P = G::P;
    static constexpr int D = 3;
    const Sell<T>& A;
    int64_t base;   // the lane's first slot
    int32_t width;  // slice width, uniform across the wave
    G g[D];
    __device__ __forceinline__ WinStream(const Sell<T>& A_, int64_t s, int lane) : A(A_) {
        base = lane_base<T>(A.sl_ptr[s], lane);
        width = (int32_t)((A.sl_ptr[s + 1] - A.sl_ptr[s]) / kWave);
#pragma unroll
        for (int d = 0; d < D; ++d) g[d].load(A, base, width, d * G::N);
    }
    // term(w, lo, x) for every slot in order (lo: 0 but for the residual)
    template <typename F>
    __device__ __forceinline__ void run(const unsigned char* win, F&& term) {
        for (int32_t k0 = 0; k0 < width; k0 += D * G::N) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const G& s = g[d];
#pragma unroll
                for (int q = 0; q < G::N / P; ++q) {
                    if (k0 + d * G::N + q * P >= width) break;
                    V3<XT> xv[P];
#pragma unroll
                    for (int e = 0; e < P; ++e) {
                        const XT* v = reinterpret_cast<const XT*>(win + (uint32_t)s.d[q][e] * (sizeof(XT) / 4));
                        xv[e] = V3<XT>{v[0], v[1], v[2]};
                    }
#pragma unroll
                    for (int e = 0; e < P; ++e) {
                        double lo = 0.0;
                        if constexpr (RES && sizeof(T) == 4) lo = (double)s.l[q][e];
                        term(s.c[q][e], lo, xv[e]);
                    }
                }
                g[d].load(A, base, width, k0 + (d + D) * G::N);
            }
        }
    }
};

// sell_row on the window.
template <typename T, bool RES, typename ACC, typename XT>
__device__ __forceinline__ void win_row(WinStream<T, RES, XT>& st, const unsigned char* win, const V3<XT>& xs, ACC& a0, ACC& a1,
                               ACC& a2) {
    st.run(win, [&](T c, double lo, const V3<XT>& xv) __attribute__((always_inline)) {
        if constexpr (RES) {
            const double w = (double)c + lo;
            a0 += w * ((double)xv.x - (double)xs.x);
            a1 += w * ((double)xv.y - (double)xs.y);
            a2 += w * ((double)xv.z - (double)xs.z);
        } else {
            a0 = fma_t(c, xv.x - xs.x, a0);
            a1 = fma_t(c, xv.y - xs.y, a1);
            a2 = fma_t(c, xv.z - xs.z, a2);
        }
    });
}

// sell_row_kahan on the window.
__device__ __forceinline__ void win_row_kahan(WinStream<float, false, float>& st, const unsigned char* win,
                                     const V3<float>& xs, float d, V3<float>& y) {
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, c0 = 0.f, c1 = 0.f, c2 = 0.f;
    kahan_add(s0, c0, d * xs.x);
    kahan_add(s1, c1, d * xs.y);
    kahan_add(s2, c2, d * xs.z);
    st.run(win, [&](float c, double, const V3<float>& xv) __attribute__((always_inline)) {
        if (c != 0.f) {
            kahan_add(s0, c0, c * xv.x);
            kahan_add(s1, c1, c * xv.y);
            kahan_add(s2, c2, c * xv.z);
        }
    });
    y = V3<float>{s0, s1, s2};
}

template <typename T, bool RES>
struct AccOf {
    typedef T t;
};
template <typename T>
struct AccOf<T, true> {
    typedef double t;
};

// Cached operator: y_r = rs_r x_r + sum_k coef[r,k] (x[col[r,k]] - x_r).
// One wavefront per 64-row slice, a block of consecutive slices (XCD-aware
// order).  With kDotResid
// the kernel writes y = b64 - A x (FP64-accurate, rounded to T) instead, and
// x may be held in another precision XT; with kDotCG, b64 holds the weights
// D of the inner product.
//
// KH (T = float only): the paper's single precision: the row in plain form
// with compensated FP32 sums (sell_row_kahan, A.dg the plain diagonal) and
// the inner products of FP32 products with compensated FP32 sums.
//
// WIN: the windowed column code (see Sell).  The block first copies its
// window of x into LDS (about 130 bytes a row against the matrix's 490); the
// gathers of x, one per slot and lane, are then LDS reads, and the matrix
// stream has the vector memory path to itself.  The wave's first three groups
// of slots are loaded before the window.  A launch (A s with two dots):
// 4.13 -> 3.33 ms at 33.7M particles in FP32 (5.3 TB/s of matrix, vectors and
// windows' own share of HBM), 140 -> 115 us at 1.16M, 85 -> 61 us at 328k in
// FP64; the delta-coded kernel waits for its gathers, this one for HBM and, a
// sixth of its time, for the windows.
template <typename T, int MODE, typename XT = T, bool KH = false, bool WIN = false>
__global__ __launch_bounds__(kApplyMaxBlock) void k_apply_sell(const int32_t* __restrict__ halt, int64_t n, Sell<T> A,
                                                          const XT* __restrict__ x, T* __restrict__ y,
                                                          const T* __restrict__ w, const double* __restrict__ b64,
                                                          double* __restrict__ part) {
    if (halt && *halt) return;
    constexpr int K = DotK<MODE>::K;
    constexpr bool RES = MODE == kDotResid;
    static_assert(!KH || (sizeof(T) == 4 && !RES), "single-precision arithmetic: FP32 operator, not the residual");
    __shared__ double lds[(KH ? 2 : 1) * K * kMaxWaves];
    extern __shared__ __align__(16) unsigned char win_lds[];
    double acc[K];
    float cmp[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        acc[k] = 0.0;
        cmp[k] = 0.f;
    }
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t bid = xcd_block(blockIdx.x, gridDim.x);
    const int64_t s = bid * (kApplyMaxBlock / kWave) + wid;  // the wave's slice
    const int64_t row = s * kWave + lane;
    const bool on = row < n;
    // sums: the row's three sums of c (x_col - x_row), or under KH the whole row
    typedef typename AccOf<T, RES>::t ACC;
    ACC a0 = 0, a1 = 0, a2 = 0;
    V3<T> yv{};
    V3<XT> xs{};
    if constexpr (WIN) {
        static_assert(kApplyMaxBlock == kWinRows, "one block's windows");
        WinStream<T, RES, XT> st(A, min(s, A.nslices - 1), lane);
        if (on) xs = ld3(x, row);
        win_parts(A, bid, x, win_lds, [&]() __attribute__((always_inline)) {
            if (!on) return;
            if constexpr (KH) win_row_kahan(st, win_lds, xs, A.dg[row], yv);
            else win_row<T, RES>(st, win_lds, xs, a0, a1, a2);
        });
    } else if (on) {
        const int64_t base = lane_base<T>(A.sl_ptr[s], lane);
        const int32_t width = (int32_t)((A.sl_ptr[s + 1] - A.sl_ptr[s]) / kWave);
        xs = ld3(x, row);
        if constexpr (KH) sell_row_kahan(A, base, width, (int32_t)row, x, xs, A.dg[row], yv);
        else sell_row<T, RES, ACC, XT>(A, base, width, (int32_t)row, x, xs, a0, a1, a2);
    }
    if (on) {
        if constexpr (RES) {
            const double d = A.rs64[row];
            const V3<double> bb = ld3(b64, row);
            const double r0 = bb.x - (d * (double)xs.x + a0);
            const double r1 = bb.y - (d * (double)xs.y + a1);
            const double r2 = bb.z - (d * (double)xs.z + a2);
            acc[0] += r0 * r0;
            acc[1] += r1 * r1;
            acc[2] += r2 * r2;
            st3(y, row, V3<T>{(T)r0, (T)r1, (T)r2});
        } else {
            if constexpr (!KH) {
                const T d = A.dg[row];
                yv.x = fma_t(d, xs.x, a0);
                yv.y = fma_t(d, xs.y, a1);
                yv.z = fma_t(d, xs.z, a2);
            }
            st3(y, row, yv);
            if constexpr (MODE != kDotNone) {
                V3<T> wv{};
                if constexpr (MODE == kDotA1) wv = ld3(w, row);
                double dw = 1.0;
                if constexpr (MODE == kDotCG) dw = b64 ? b64[row] : 1.0;
                accumulate_dots<T, MODE, KH>(acc, cmp, xs, yv, wv, dw);
            }
        }
    }
    if constexpr (MODE != kDotNone) write_partials_kh<K, KH>(acc, cmp, lds, part);
}

// Row of the operator evaluated from positions in FP64 (the paper's
// matrix-free gemv) for cell_rows: staged per candidate the vector x and the
// pair data (mu, m/rho); sums of the weights and of weight times x; finish
// forms (A x)_b, or (D^-1 A x)_b with Jacobi, and hands it to out(row, y).
template <typename T, class F>
struct OtfBody {
    typedef T X;
    static constexpr int NX = 3 + 16 / sizeof(T);  // x, and (mu, m / rho) in 16 bytes
    static constexpr int NA = 4;  // sum of weights, of weight * x
    PartView pv;
    OpParams op;
    const T* x;
    F out;
    struct Row {
        int take;
        double mu, ir;
        V3<T> x;
    };
    __device__ Row row(int32_t b) const {
        const bool fluid = pv.type[b] == SPH_FLUID;
        const int take = fluid ? kTakeAll : op.wall == SPH_WALL_DUMMY ? kTakeFluid : kTakeNone;
        return Row{take, pv.mu[b], pv.inv_rho[b], ld3(x, b)};
    }
    struct Pair {
        T v[16 / sizeof(T)];
    };
    __device__ void stage(int32_t a, T (&v)[NX]) const {
        const V3<T> xa = ld3(x, a);
        const Pair ma = __builtin_bit_cast(Pair, pv.mu_mr[a]);
        v[0] = xa.x;
        v[1] = xa.y;
        v[2] = xa.z;
        for (int k = 3; k < NX; ++k) v[k] = ma.v[k - 3];
    }
    __device__ bool fluid(int32_t a) const { return pv.type[a] == SPH_FLUID; }
    __device__ void term(const Grid& g, const Row& b, double r2, double, double, double, const T (&v)[NX],
                         double (&acc)[NA]) const {
        Pair p;
        for (int k = 3; k < NX; ++k) p.v[k - 3] = v[k];
        const double2 ma = __builtin_bit_cast(double2, p);
        const double w = b.take == kTakeAll ? pair_w_v(g, op.avg, ma.x, ma.y, b.mu, b.ir, r2) : pair_W(g, r2);
        acc[0] += w;
        acc[1] += w * (double)v[0];
        acc[2] += w * (double)v[1];
        acc[3] += w * (double)v[2];
    }
    __device__ void finish(int32_t b, const Row& r, const double (&acc)[NA]) const {
        double y[3] = {(double)r.x.x, (double)r.x.y, (double)r.x.z};
        if (r.take == kTakeAll) {
            const double diag = 1.0 + op.dt * acc[0];
            for (int c = 0; c < 3; ++c) {
                y[c] = diag * y[c] - op.dt * acc[1 + c];
                if (op.jacobi) y[c] /= diag;
            }
        } else if (r.take == kTakeFluid && acc[0] > 0.0) {
            for (int c = 0; c < 3; ++c) y[c] += acc[1 + c] / acc[0];
        }
        out(b, r.x, y);
    }
};

// On-the-fly operator over the cells, each block a contiguous share of them (W
// waves), or over the rows (W = 0, one thread each); with kDotResid it writes y = b64 - A x instead (FP64 residual rounded to T)
// and its squared norm, x then being of precision XT; with kDotCG, b64 holds
// the weights D.
template <typename T, int MODE, typename XT, int W>
__global__ __launch_bounds__(W ? W * kWave : kApplyMaxBlock) void k_apply_otf(const int32_t* __restrict__ halt, NbrView nv,
                                                                 PartView pv, OpParams op, int64_t ncell, int32_t cap,
                                                                 const XT* __restrict__ x, T* __restrict__ y,
                                                                 const T* __restrict__ w,
                                                                 const double* __restrict__ b64,
                                                                 double* __restrict__ part) {
    if (halt && *halt) return;
    constexpr int K = DotK<MODE>::K;
    __shared__ double lds[K * kMaxWaves];
    extern __shared__ __align__(16) unsigned char cell_lds[];
    double acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = 0.0;
    const int64_t bid = xcd_block(blockIdx.x, gridDim.x);
    const int64_t all = W ? ncell : nv.n;
    const int64_t share = ceil_div(all, (int64_t)gridDim.x);
    const int64_t c0 = bid * share, c1 = min(c0 + share, all);
    const auto out = [&](int32_t r, const V3<XT>& xr, double (&yv)[3]) {
        if constexpr (MODE == kDotResid) {
            const V3<double> bb = ld3(b64, r);
            yv[0] = bb.x - yv[0];
            yv[1] = bb.y - yv[1];
            yv[2] = bb.z - yv[2];
            acc[0] += yv[0] * yv[0];
            acc[1] += yv[1] * yv[1];
            acc[2] += yv[2] * yv[2];
        }
        const V3<T> o{(T)yv[0], (T)yv[1], (T)yv[2]};
        st3(y, r, o);
        if constexpr (MODE != kDotNone && MODE != kDotResid) {
            V3<T> wv{};
            if constexpr (MODE == kDotA1) wv = ld3(w, r);
            double dw = 1.0;
            if constexpr (MODE == kDotCG) dw = b64 ? b64[r] : 1.0;
            float cmp[K];
            accumulate_dots<T, MODE>(acc, cmp, xr, o, wv, dw);
        }
    };
    const OtfBody<XT, decltype(out)> body{pv, op, x, out};
    if constexpr (W > 0) {
        for (int64_t c = c0; c < c1; ++c) cell_rows<W>(nv, (int32_t)c, cap, cell_lds, body);
    } else {
        for (int64_t r = c0 + threadIdx.x; r < c1; r += blockDim.x) row_terms(nv, (int32_t)r, body);
    }
    if constexpr (MODE != kDotNone) write_partials<K>(acc, lds, part);
}

// Launch of the on-the-fly operator: a block per cell, or (dot products, and
// rows) the operator's grid, whose blocks write the partials.
template <typename T, int MODE, typename XT = T>
inline void launch_apply_otf(hipStream_t stream, const Launch& L, const int32_t* halt, const sph_nbr* nb,
                             const PartView& pv, const OpParams& op, const XT* x, T* y, const T* w, const double* b64,
                             double* part) {
    const Occupancy occ = nb->occupancy();
    const int32_t cap = cell_cap(occ);
    const int64_t cells = ceil_div(nb->ncell, (int64_t)kNumXcd) * kNumXcd;
    const auto go = [&](auto waves) {
        constexpr int W = decltype(waves)::value;
        const unsigned grid = MODE == kDotNone && W ? (unsigned)cells : (unsigned)L.grid_apply;
        hipLaunchKernelGGL((k_apply_otf<T, MODE, XT, W>), dim3(grid), dim3(W ? W * kWave : L.block_apply),
                           (cell_bytes<OtfBody<XT, int>, W>(cap)), stream, halt, nb->view(), pv, op, nb->ncell, cap, x,
                           y, w, b64, part);
    };
    if (!sums_by_cells(occ)) go(std::integral_constant<int, 0>{});
    else if (nb->g.kernel == SPH_KERNEL_GAUSSIAN) go(std::integral_constant<int, kCellWavesGauss>{});
    else go(std::integral_constant<int, kCellWaves>{});
}

// Launch of the cached operator in the matrix's column code.
template <typename T, int MODE, typename XT = T, bool KH = false>
inline void launch_apply_sell(hipStream_t stream, const Launch& L, const int32_t* halt, const Sell<T>& A, const XT* x,
                              T* y, const T* w, const double* b64, double* part) {
    const dim3 grid(L.grid_apply), block(L.block_apply);
    if (A.wmax > 0)
        hipLaunchKernelGGL((k_apply_sell<T, MODE, XT, KH, true>), grid, block, win_bytes<XT>(A.wmax), stream, halt,
                           L.n, A, x, y, w, b64, part);
    else
        hipLaunchKernelGGL((k_apply_sell<T, MODE, XT, KH, false>), grid, block, 0, stream, halt, L.n, A, x, y, w, b64,
                           part);
}

}  // namespace sph
