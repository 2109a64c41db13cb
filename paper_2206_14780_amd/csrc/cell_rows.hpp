// Sums over the neighbours of every particle, a cell at a time: the engine of
// the kernels that evaluate pair terms from positions (the on-the-fly operator
// and the viscosity update).
#pragma once

#include <type_traits>

#include "sph_device.hpp"

namespace sph {

// Runs of cells around cell c, one per lane < 27, in ascending order (the
// three z layers, in each the three y rows, in each the wrapped first cell,
// the run around c and the wrapped last cell): first particle and length.
__device__ inline void cell_run(const NbrView& nv, int32_t c, int lane, int32_t& beg, int32_t& len) {
    const Grid& g = nv.g;
    beg = len = 0;
    if (lane >= 27) return;
    const int32_t nx = g.nc[0], ny = g.nc[1];
    const int32_t cx = c % nx, l = c / nx;
    const int32_t part = lane % 3, iy = (lane / 3) % 3, iz = lane / 9;
    int32_t zs[3], ys[3];
    const int nzs = axis_cells(l / ny, g.nc[2], g.per[2], zs);
    const int nys = axis_cells(l % ny, ny, g.per[1], ys);
    const bool wraps = g.per[0] && nx >= 3;
    int32_t lo = cx > 0 ? cx - 1 : 0, hi = cx < nx - 1 ? cx + 1 : nx - 1;
    if (g.per[0] && nx < 3) {
        lo = 0;
        hi = nx - 1;
    }
    bool on = iz < nzs && iy < nys;
    if (part == 0) {  // the first cell, from the last one
        on = on && wraps && cx == nx - 1;
        lo = hi = 0;
    } else if (part == 2) {  // the last cell, from the first one
        on = on && wraps && cx == 0;
        lo = hi = nx - 1;
    }
    if (on) {
        const int32_t base = (zs[iz] * ny + ys[iy]) * nx;
        beg = nv.cell_start[base + lo];
        len = nv.cell_start[base + hi + 1] - beg;
    }
}

// Exclusive prefix of the runs' lengths over the lanes; total: their sum.
__device__ inline int32_t run_prefix(int32_t len, int lane, int32_t& total) {
    int32_t pre = len;
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
        const int32_t v = __shfl_up(pre, o, kWave);
        if (lane >= o) pre += v;
    }
    total = __builtin_amdgcn_readlane(pre, 26);
    return pre - len;
}

// Whether candidate x lies too far from ref (a particle of the cell) for the
// plain difference to be the minimum image of every pair of the cell's rows
// and candidates: beyond a quarter of a period (0.24: clear of rounding) on a
// periodic axis, or not a number.
__device__ inline bool far_image(const Grid& g, const Pos4& ref, double x, double y, double z) {
    return (g.period[0] > 0.0 && !(fabs(ref.x - x) <= 0.24 * g.period[0])) ||
           (g.period[1] > 0.0 && !(fabs(ref.y - y) <= 0.24 * g.period[1])) ||
           (g.period[2] > 0.0 && !(fabs(ref.z - z) <= 0.24 * g.period[2]));
}

// Sum over the 16 lanes of a DPP row, the same in all of them.
__device__ inline double row_sum(double v) {
    v += dpp_move<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v += dpp_move<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    v += dpp_move<0x141>(v);  // row_half_mirror
    v += dpp_move<0x140>(v);  // row_mirror
    return v;
}

// Waves of a block: four with the Wendland kernel's ~500 candidates a cell
// (three or four blocks share a CU); the truncated Gaussian's ~1600 fill the LDS of a
// CU, so one block brings all the waves.
constexpr int kCellWaves = 4, kCellWavesGauss = 16;
constexpr int kCellRows = 4;      // rows of a wave at a time, 16 lanes each
constexpr int kCellList = 192;    // listed neighbours of a row before they are summed
enum { kTakeNone = 0, kTakeAll = 1, kTakeFluid = 2 };  // neighbours of a row

template <class B, int W>
constexpr size_t cell_bytes(int32_t cap) {
    // positions and extras, fluid masks, and the rows' lists, which share their
    // place with the candidates' indices
    return W == 0 ? 0 : (size_t)cap * (24 + sizeof(typename B::X) * B::NX) + 8 * (cap / kWave) +
           (W * kCellRows * kCellList * 2 > cap * 4 ? W * kCellRows * kCellList * 2 : cap * 4);
}

// cell_rows by one thread per row.  Where no row of the wave takes only its
// fluid neighbours the kind of row is a constant of the walk: asking for it at
// every neighbour cost a tenth (896 particles, Gaussian, FP32: 465 -> 410 us).  Mixed
// waves walk once (two walks in turn: 485 -> 635 us at 1M particles, a fifth
// of them walls).
template <class B>
__device__ inline void row_terms(const NbrView& nv, int32_t b, const B& body) {
    const auto r = body.row(b);
    double acc[B::NA] = {};
    const auto walk = [&](auto all) __attribute__((always_inline)) {
        auto mine = r;
        if constexpr (decltype(all)::value) mine.take = kTakeAll;
        const Pos4 pb = nv.pos[b];
        for_each_neighbor(nv, b, [&](int32_t a, double r2) {
            if (mine.take == kTakeFluid && !body.fluid(a)) return;
            typename B::X v[B::NX];
            body.stage(a, v);
            const Pos4 pa = nv.pos[a];
            body.term(nv.g, mine, r2, disp(pb.x, pa.x, nv.g.period[0]), disp(pb.y, pa.y, nv.g.period[1]),
                      disp(pb.z, pa.z, nv.g.period[2]), v, acc);
        });
    };
    if (__any(r.take == kTakeFluid)) {
        if (r.take != kTakeNone) walk(std::false_type{});
    } else if (r.take == kTakeAll) {
        walk(std::true_type{});
    }
    body.finish(b, r, acc);
}

// For every row of cell c: acc = sum of body.term over its neighbours, then
// body.finish.  The block stages the cell's candidates in LDS (positions and
// body.NX values each); a wave takes four rows at a time, tests them against
// 64 candidates at once and lists the hits, and then sums a row's terms over
// 16 lanes, so that the pair arithmetic runs only on neighbours (a sixth of
// the candidates) with every lane busy.  One thread per row walking all its
// candidates, as before, ran the pair arithmetic for every candidate that any
// lane took.  What bounds it is the vector ALU: about 200 instructions a row
// for the tests, 200 for the pair terms, 70 for sums and results.  The
// viscosity update (FP64): 2.08 -> 1.19 ms at 1.03M particles, 487 -> 154 us at
// 118k; the operator (FP32 x): 558 -> 322 us at 227k.  Called by the whole block.
template <int W, class B>
__device__ inline void cell_rows(const NbrView& nv, int32_t c, int32_t cap, unsigned char* lds, const B& body) {
    const Grid& g = nv.g;
    const int32_t rb = nv.cell_start[c], re = nv.cell_start[c + 1];
    if (rb >= re) return;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(tid / kWave);
    double* px = reinterpret_cast<double*>(lds);
    typedef typename B::X X;
    double *py = px + cap, *pz = py + cap;
    uint64_t* fluid = reinterpret_cast<uint64_t*>(pz + cap);
    X* ext = reinterpret_cast<X*>(fluid + cap / kWave);
    int32_t* cand = reinterpret_cast<int32_t*>(ext + (size_t)B::NX * cap);
    uint16_t* list = reinterpret_cast<uint16_t*>(cand) + wid * (kCellRows * kCellList);
    int32_t beg, len, total;
    cell_run(nv, c, lane, beg, len);
    const int32_t pre = run_prefix(len, lane, total);
    const uint64_t own = __ballot(len > 0 && rb >= beg && rb < beg + len);
    const int own_run = __builtin_ctzll(own);
    const int32_t self0 = __builtin_amdgcn_readlane(pre - beg, own_run);  // place of the cell's particles, less their index
    const int32_t nbatch = (total + cap - 1) / cap;
    const int32_t turns = (re - rb + kCellRows * W - 1) / (kCellRows * W);
    bool image = false;
    for (int32_t turn = 0; turn < turns; ++turn) {
        const int32_t g0 = rb + (turn * W + wid) * kCellRows;
        const int32_t nr = min(re - g0, kCellRows);  // may be <= 0: the wave only helps to stage
        const int sub = lane >> 4;
        const int32_t my = g0 + min(sub, max(nr, 1) - 1);  // the row whose terms the lane sums
        const int32_t myrow = min(my, re - 1);
        typename B::Row mine = body.row(myrow);
        const Pos4 pm = nv.pos[myrow];
        int take[kCellRows];
        double rx[kCellRows], ry[kCellRows], rz[kCellRows];
#pragma unroll
        for (int i = 0; i < kCellRows; ++i) {
            const int src = i * 16;
            take[i] = i < nr ? __builtin_amdgcn_readlane(mine.take, src) : kTakeNone;
            rx[i] = read_lane(pm.x, src);
            ry[i] = read_lane(pm.y, src);
            rz[i] = read_lane(pm.z, src);
        }
        double acc[B::NA];
#pragma unroll
        for (int k = 0; k < B::NA; ++k) acc[k] = 0.0;
        for (int32_t b = 0; b < nbatch; ++b) {
            const int32_t b0 = b * cap;
            const int32_t nc = min(total - b0, cap);
            if (turn == 0 || nbatch > 1) {
                __syncthreads();  // the batch before is no longer read
                uint64_t runs = __ballot(len > 0 && pre < b0 + cap && pre + len > b0);
                for (int at = 0; runs; ++at) {
                    const int t = __builtin_ctzll(runs);
                    runs &= runs - 1;
                    if (at % W != wid) continue;
                    const int32_t B0 = __builtin_amdgcn_readlane(beg, t), L = __builtin_amdgcn_readlane(len, t);
                    const int32_t P = __builtin_amdgcn_readlane(pre, t) - b0;
                    const int32_t j1 = min(L, cap - P);
                    for (int32_t j = max(0, -P) + lane; j < j1; j += kWave) cand[P + j] = B0 + j;
                }
                __syncthreads();
                const Pos4 ref = nv.pos[rb];
                bool far = false;
                for (int32_t p = tid; p < (nc + kWave - 1) / kWave * kWave; p += W * kWave) {
                    const bool ok = p < nc;
                    const int32_t a = ok ? cand[p] : rb;
                    const Pos4 s = nv.pos[a];
                    X v[B::NX];
                    body.stage(a, v);
                    // a place without a candidate never passes the distance test
                    px[p] = ok ? s.x : __builtin_nan("");
                    py[p] = s.y;
                    pz[p] = s.z;
#pragma unroll
                    for (int k = 0; k < B::NX; ++k) ext[(size_t)k * cap + p] = v[k];
                    const uint64_t m = __ballot(body.fluid(a));
                    if (lane == 0) fluid[p >> 6] = m;
                    far = far || (ok && far_image(g, ref, s.x, s.y, s.z));
                }
                image = __syncthreads_or(far) || nbatch > 1;
            }
            if (nr <= 0) continue;
            int32_t cnt[kCellRows] = {0, 0, 0, 0};
            const auto flush = [&] {
                wave_sync();
                const int32_t mycnt = sub == 0 ? cnt[0] : sub == 1 ? cnt[1] : sub == 2 ? cnt[2] : cnt[3];
                const uint16_t* ml = list + sub * kCellList;
                for (int32_t e = lane & 15; e < mycnt; e += 16) {
                    const int32_t p = ml[e];
                    double dx = pm.x - px[p], dy = pm.y - py[p], dz = pm.z - pz[p];
                    if (image) {
                        dx = disp(pm.x, px[p], g.period[0]);
                        dy = disp(pm.y, py[p], g.period[1]);
                        dz = disp(pm.z, pz[p], g.period[2]);
                    }
                    X v[B::NX];
#pragma unroll
                    for (int k = 0; k < B::NX; ++k) v[k] = ext[(size_t)k * cap + p];
                    body.term(g, mine, (dx * dx + dy * dy) + dz * dz, dx, dy, dz, v, acc);
                }
                wave_sync();
#pragma unroll
                for (int i = 0; i < kCellRows; ++i) cnt[i] = 0;
            };
            const auto tests = [&](auto img) {
                for (int32_t q = 0; q * kWave < nc; ++q) {
                    const int32_t p = q * kWave + lane;
                    const double x = px[p], y = py[p], z = pz[p];
                    const uint64_t fl = fluid[q];
                    bool full = false;
#pragma unroll
                    for (int i = 0; i < kCellRows; ++i) {
                        if (take[i] == kTakeNone) continue;
                        double dx = rx[i] - x, dy = ry[i] - y, dz = rz[i] - z;
                        if constexpr (decltype(img)::value) {
                            dx = disp(rx[i], x, g.period[0]);
                            dy = disp(ry[i], y, g.period[1]);
                            dz = disp(rz[i], z, g.period[2]);
                        }
                        const double r2 = (dx * dx + dy * dy) + dz * dz;
                        uint64_t m = __ballot(r2 < g.cut2) & __ballot(p != self0 + g0 + i - b0);
                        if (take[i] == kTakeFluid) m &= fl;
                        const int32_t k = cnt[i] + mbcnt64(m);
                        if (__builtin_amdgcn_inverse_ballot_w64(m)) list[i * kCellList + k] = (uint16_t)p;
                        cnt[i] = __builtin_amdgcn_readfirstlane(cnt[i] + __popcll(m));
                        full = full || cnt[i] > kCellList - kWave;
                    }
                    if (full) flush();
                }
            };
            if (image) tests(std::true_type{});
            else tests(std::false_type{});
            flush();
        }
        if (nr > 0) {
#pragma unroll
            for (int k = 0; k < B::NA; ++k) acc[k] = row_sum(acc[k]);
            if ((lane & 15) == 0 && sub < nr) body.finish(g0 + sub, mine, acc);
        }
    }
}

}  // namespace sph
