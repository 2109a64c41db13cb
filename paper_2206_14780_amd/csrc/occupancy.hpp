// Which kernels walk a neighbour structure cell by cell and which row by row:
// rules on how its particles fill its cells (no device code: the host unit
// test compiles it alone).
#pragma once

#include <algorithm>
#include <cstdint>

namespace sph {

// How the particles of a neighbour handle fill its cells.
struct Occupancy {
    int64_t n, ncell;
    bool gauss;       // truncated Gaussian kernel, else Wendland
    int32_t fullest;  // particles of the fullest cell, rounded down to kCrowdStep; 0: below kCrowdLeast
    double support;   // volume of the kernel's support, in cells
    double mean() const { return (double)n / (double)ncell; }
    double row() const { return mean() * support; }  // neighbours of a row, were the cells evenly filled
};

// The neighbour build records the fullest cell in steps, from where it matters
// and up to where any cell is a crowd.
constexpr int32_t kCrowdStep = 32, kCrowdLeast = 96, kCrowdLevels = 32;

// A cell's rows and their tests are one wave's or one block's work, so a cell
// with many times the others' particles outlasts the launch.  One crowded cell
// (or a block of 3x3x3) in an evenly filled box, the operator from positions by
// rows / by cells: 65k particles, 16 in the others, 200: 460 / 376 us, 400: 462
// / 883, 1600: 1.02 / 8.84 ms; 27 of 250: 2.88 / 3.64 ms; 1M: 27 of 120: 2.88 /
// 2.62, of 250: 3.93 / 5.33, 1600: 2.78 / 10.9; Gaussian, whose blocks have
// 16 waves, 65k, 400: 1.52 / 0.93, 800: 1.48 / 2.05, 1M, 800: 6.60 / 6.41, 1600:
// 7.0 / 10.2.  Matrix and one product: 65k, 200: 1.25 / 1.46, 400: 1.59 / 2.39,
// 1600: 3.8 / 12.8, 27 of 120: 5.1 / 6.4; 1M, 400: 4.2 / 5.0, 1600: 6.5 / 16.1;
// Gaussian, 65k, 200: 5.36 / 5.26, 800: 5.47 / 6.13, 1M, 800: 28.3 / 37.2.
// Scanned by rows, the matrix of a solve still gets its windows (a launch of
// their own and a slower fill of the rows beyond their list, 5 to 15 % of the
// build); that of a single product does not.
inline bool crowded_scan(const Occupancy& o) { return o.fullest >= (o.gauss ? 256 : 96); }
inline bool crowded_sums(const Occupancy& o) {
    return o.fullest >= (o.gauss ? 512 : 192) &&
           ((double)o.fullest > 4.0 * o.mean() || o.fullest >= kCrowdStep * (kCrowdLevels - 1));
}

// Candidates that a block stages in LDS for the sums over neighbours (see
// cell_rows): the mean of the 27 cells around a particle and 7 % more (the
// blocks of cells of a lattice hold up to 8^3 where the mean is 7.95^3), in
// whole waves, at most 1088 (1920); a cell with more is done in batches.
constexpr double kStageMost = 1024.0, kStageMostGauss = 1900.0, kStageSpare = 1.07;
inline int32_t cell_cap(const Occupancy& o) {
    const double want = 27.0 * o.mean() * kStageSpare;
    return (int32_t)std::min(want, o.gauss ? kStageMostGauss : kStageMost) / 64 * 64 + 64;
}

// Whether sums over neighbours are taken a cell at a time (cell_rows), or by
// one thread per row (row_terms).  Blocks pay for cells that are empty or hold
// a row or two, as in a box that the particles fill in part: the operator
// (FP64) by cells / by rows at 1M scattered particles with 4, 8, 21 in the mean
// cell: 2.57 / 0.82, 1.77 / 1.23, 1.82 / 2.54 ms; at 65k with 4, 7, 16: 198 /
// 161, 154 / 226, 152 / 400 us; Gaussian, 1M, 21, 64: 3.65 / 2.80, 4.72 / 6.49
// ms; 65k, 7, 16: 446 / 246, 317 / 441 us.  Cells with more candidates than a
// block stages at once still gain while the rows alone are too few for the
// chip: 65k, 65 in a cell, 0.62 / 1.30 ms, but 1M, 64: 7.2 / 5.9; and a few
// blocks do not fill it either (4096 particles in 8 cells: 4.1 / 1.8 ms).
inline bool sums_by_cells(const Occupancy& o) {
    const bool small = o.n < (1 << 18);
    if (o.mean() < (o.gauss ? (small ? 12.0 : 32.0) : (small ? 5.0 : 12.0)) || crowded_sums(o)) return false;
    return o.mean() <= (o.gauss ? kStageMostGauss : kStageMost) / (27.0 * kStageSpare) || (small && o.ncell >= 64);
}

// Whether the matrix keeps the delta code (and is scanned by rows).  A wave
// per cell pays for empty cells too (30M cells around 1000 particles: 4.6 ms),
// the windows of scattered rows are many short ranges, and of rows that are
// mostly longer than their list of cap entries (0: none) the counts of slots
// are wanted.  Matrix and one product, FP64, by cells and windows / by rows and
// delta code: 1M scattered particles with 2, 4, 8, 21 in the mean cell 1.48 /
// 0.75, 1.27 / 1.05, 1.44 / 1.57, 10.4 / 10.6 ms, with 64 29.4 / 27.3; 65k with
// 2, 4, 7: 196 / 180, 188 / 233, 199 / 301 us; Gaussian, 1M with 8, 21: 1.73 /
// 1.61, 2.93 / 3.38 ms.
inline bool delta_coded(const Occupancy& o, int32_t cap) {
    const double least = o.n < (1 << 18) ? 3.0 : o.gauss ? 12.0 : 6.0;
    return o.mean() < least || o.row() > (double)cap;
}

// Whether the neighbours are found by one thread per row (k_row_scan_rows)
// rather than by one wave per cell (k_row_scan).
inline bool scan_by_rows(const Occupancy& o, int32_t cap) { return delta_coded(o, cap) || crowded_scan(o); }

// Whether an export keeps no lists and scans every row twice, to count and to
// write it: rows with next to no neighbours cost less than two launches more.
// Export with lists / without: 4096 particles, 0.1, 0.2, 0.5, 1 in the mean
// cell: 71 / 68, 75 / 74, 79 / 84, 87 / 109 us; 65k, 0.01, 0.2, 0.5, 1: 85 / 76,
// 91 / 76, 98 / 88, 105 / 109 us; 1M, 0.01, 0.2, 0.5, 1: 726 / 232, 707 / 301, 755 /
// 516, 782 / 1074 us; 2 particles: 60 / 33 us.
inline bool export_without_lists(const Occupancy& o) { return o.mean() < 0.6 || o.n <= 16; }
// And then counts them in the caller's order, in one launch, while the
// particles are few enough for the caches (1M, 0.2: 309 us, 93 in cell order).
inline bool count_in_caller_order(const Occupancy& o) { return export_without_lists(o) && o.n < (1 << 17); }

}  // namespace sph
