// Papanastasiou viscosity from the velocity field (Section "Non-Newtonian
// viscosity", eq. papa): per particle the velocity gradient over its
// neighbours, the symmetric shear rate, its second invariant D, and
// mu = tau0 Ybar(D) + mu0 with the regularised yield term Ybar.
#include <cmath>

#include "cell_rows.hpp"

namespace sph {

// Ybar(D) = (1 - exp(-m D))/D for m D >= x0, else m T(m D), T the Maclaurin
// series of (1 - e^-x)/x cut after 8 terms, in Horner form
// 1 - x/2 (1 - x/3 (... (1 - x/7 (1 - x/8)))).  The switch x0 is where the
// first omitted term x^8/9! equals single-precision epsilon (the printed
// switch "D >= m" cannot be meant: the series would then run at m D up to m^2).
__device__ inline double ybar(double D, double m, double x0) {
    const double x = m * D;
    if (x >= x0) return (1.0 - exp(-x)) / D;
    double t = 1.0;
#pragma unroll
    for (int k = 8; k >= 2; --k) t = 1.0 - x / (double)k * t;
    return m * t;
}

// Viscosity update of a row for cell_rows.  G = sum_a (m_a/rho_a) F(r_ab)
// r_ab u_ab^T over the neighbours a (r_ab = r_a - r_b by minimum image,
// u_ab = u_a - u_b; the printed form, minus the usual SPH gradient, which
// the symmetric quadratic invariant does not see), S = (G + G^T)/2,
// D = sqrt(2 S:S) (the shear rate in simple shear).  Only the six sums of S
// are kept, the off-diagonal ones as G_ij + G_ji.  Fluid rows get tau0
// Ybar(D) + mu0, wall rows keep their viscosity; both outputs are written in
// the caller's order.
template <typename T>
struct PapaBody {
    typedef double X;
    static constexpr int NX = 4;  // u, m / rho
    static constexpr int NA = 6;  // xx, yy, zz, xy, xz, yz
    PartView pv;
    const T* u;
    const int32_t* perm;
    double tau0, m, mu0, x0;
    double *mu_out, *d_out;
    struct Row {
        int take;
        double u[3];
    };
    __device__ Row row(int32_t b) const {
        const V3<T> ub = ld3(u, b);
        return Row{kTakeAll, {(double)ub.x, (double)ub.y, (double)ub.z}};
    }
    __device__ void stage(int32_t a, double (&v)[NX]) const {
        const V3<T> ua = ld3(u, a);
        v[0] = (double)ua.x;
        v[1] = (double)ua.y;
        v[2] = (double)ua.z;
        v[3] = pv.mu_mr[a].y;
    }
    __device__ bool fluid(int32_t) const { return true; }
    __device__ void term(const Grid& g, const Row& b, double r2, double dx, double dy, double dz,
                         const double (&v)[NX], double (&acc)[NA]) const {
        const double F = kernel_f(g, sqrt(r2) * g.inv_h) * g.inv_h5;
        const double vf = v[3] * F;
        // r_ab = -(dx, dy, dz)
        const double rx = -dx, ry = -dy, rz = -dz;
        const double ux = v[0] - b.u[0], uy = v[1] - b.u[1], uz = v[2] - b.u[2];
        acc[0] += vf * rx * ux;
        acc[1] += vf * ry * uy;
        acc[2] += vf * rz * uz;
        acc[3] += vf * rx * uy + vf * ry * ux;
        acc[4] += vf * rx * uz + vf * rz * ux;
        acc[5] += vf * ry * uz + vf * rz * uy;
    }
    __device__ void finish(int32_t b, const Row&, const double (&s)[NA]) const {
        // S:S with the off-diagonal pairs (G_ij + G_ji)/2 counted twice
        const double ss = (s[0] * s[0] + s[1] * s[1] + s[2] * s[2]) +
                          0.5 * (s[3] * s[3] + s[4] * s[4] + s[5] * s[5]);
        const double D = sqrt(2.0 * ss);
        const int32_t o = perm[b];
        mu_out[o] = pv.type[b] == SPH_FLUID ? tau0 * ybar(D, m, x0) + mu0 : pv.mu[b];
        if (d_out) d_out[o] = D;
    }
};

// A block of W waves per cell, or (W = 0) a thread per row.
template <typename T, int W>
__global__ __launch_bounds__(W ? W * kWave : kBlock) void k_papa_visc(NbrView nv, int64_t ncell, int32_t cap,
                                                                      PapaBody<T> body) {
    const int64_t c = xcd_block(blockIdx.x, gridDim.x);
    if constexpr (W > 0) {
        extern __shared__ __align__(16) unsigned char cell_lds[];
        if (c < ncell) cell_rows<W>(nv, (int32_t)c, cap, cell_lds, body);
    } else {
        const int64_t b = c * kBlock + threadIdx.x;
        if (b < nv.n) row_terms(nv, (int32_t)b, body);
    }
}

template <typename T>
static sph_status papa_entry(sph_ctx* ctx, const sph_nbr* nb, const sph_particles* p, const void* const u[3],
                             double tau0, double m, double mu0, double* mu_out, double* d_out) {
    PartView pv;
    SPH_TRY(gather_props(ctx, nb, p, &pv));
    T* ucell = nullptr;
    SPH_TRY(ctx->ensure_t(kViscU, (size_t)nb->n * 3, &ucell));
    SPH_TRY(gather_vec3<T>(ctx, nb, u, ucell));
    const double x0 = std::pow(362880.0 * std::ldexp(1.0, -23), 0.125);
    const Occupancy occ = nb->occupancy();
    const int32_t cap = cell_cap(occ);
    const auto go = [&](auto waves) {
        constexpr int W = decltype(waves)::value;
        const int64_t blocks = W ? nb->ncell : ceil_div(nb->n, (int64_t)kBlock);
        const dim3 grid((unsigned)(ceil_div(blocks, (int64_t)kNumXcd) * kNumXcd));
        hipLaunchKernelGGL((k_papa_visc<T, W>), grid, dim3(W ? W * kWave : kBlock), (cell_bytes<PapaBody<T>, W>(cap)), ctx->stream,
                           nb->view(), nb->ncell, cap,
                           (PapaBody<T>{pv, ucell, nb->perm, tau0, m, mu0, x0, mu_out, d_out}));
    };
    if (!sums_by_cells(occ)) go(std::integral_constant<int, 0>{});
    else if (nb->g.kernel == SPH_KERNEL_GAUSSIAN) go(std::integral_constant<int, kCellWavesGauss>{});
    else go(std::integral_constant<int, kCellWaves>{});
    SPH_LAUNCHED("k_papa_visc");
    return SPH_OK;
}

}  // namespace sph

using namespace sph;

extern "C" sph_status sph_visc_papanastasiou(sph_ctx* ctx, const sph_nbr* nb, const sph_particles* p,
                                             int32_t prec, const void* const u[3], double tau0, double m,
                                             double mu0, double* mu_out, double* shear_out) {
    if (!ctx) return SPH_E_ARG;
    if (!nb || !u || !mu_out) return ctx->fail(SPH_E_ARG, "visc_papanastasiou: null argument");
    if (nb->device != ctx->device) return ctx->fail(SPH_E_ARG, "visc_papanastasiou: handle of another device");
    for (int c = 0; c < 3; ++c)
        if (!u[c]) return ctx->fail(SPH_E_ARG, "visc_papanastasiou: null velocity component");
    if (!(tau0 >= 0.0) || !std::isfinite(tau0) || !(m > 0.0) || !std::isfinite(m) || !(mu0 >= 0.0) ||
        !std::isfinite(mu0))
        return ctx->fail(SPH_E_ARG, "visc_papanastasiou: tau0, mu0 must be finite and >= 0, m finite and > 0");
    if (prec != SPH_F64 && prec != SPH_F32) return ctx->fail(SPH_E_ARG, "visc_papanastasiou: prec");
    SPH_TRY(check_particles(ctx, nb, p));
    if (nb->n == 0) return SPH_OK;
    if (prec == SPH_F64) return papa_entry<double>(ctx, nb, p, u, tau0, m, mu0, mu_out, shear_out);
    return papa_entry<float>(ctx, nb, p, u, tau0, m, mu0, mu_out, shear_out);
}
