// Prints what the rules of occupancy.hpp say of the neighbour structures given
// on stdin, one per line (n, cells, Gaussian, particles of the fullest cell,
// volume of the support in cells, entries of a row's list): staged candidates,
// sums by cells, delta coded, scanned by rows, exported without lists, counted
// in the caller's order.
#include <cstdio>

#include "occupancy.hpp"

int main() {
    long long n, ncell;
    int gauss, fullest, cap;
    double support;
    while (std::scanf("%lld %lld %d %d %lf %d", &n, &ncell, &gauss, &fullest, &support, &cap) == 6) {
        // as the neighbour build records it
        const int level = std::min(fullest / sph::kCrowdStep, sph::kCrowdLevels - 1);
        const sph::Occupancy o{n, ncell, gauss != 0, fullest >= sph::kCrowdLeast ? level * sph::kCrowdStep : 0, support};
        std::printf("%d %d %d %d %d %d\n", sph::cell_cap(o), (int)sph::sums_by_cells(o), (int)sph::delta_coded(o, cap),
                    (int)sph::scan_by_rows(o, cap), (int)sph::export_without_lists(o),
                    (int)sph::count_in_caller_order(o));
    }
    return 0;
}
