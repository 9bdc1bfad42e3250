// Types of the time step shared by its linear and quadratic kernels (not part
// of the C-ABI).
#pragma once

#include "mg_internal.h"

namespace nn4mg {

struct Grid {
    int nx, ny, nz;
    double h;
    size_t n;
};

struct Phys {
    double rho_l, rho_g, mu_l, mu_g, g, sigma, dt;
};

struct F3 {
    double *p[3];
};
struct C3 {
    const double *p[3];
};

// Face bits of a boundary rule: bit f set = -mirror on face f
// (xlo, xhi, ylo, yhi, zlo, zhi); clear = +mirror.
constexpr unsigned kEven = 0u;
constexpr unsigned kOddTop = 32u;  // p_nh, its increment, p_hs above
__host__ __device__ constexpr unsigned rule_vel(int d) { return d == 0 ? 3u : (d == 1 ? 12u : 16u); }
__host__ __device__ constexpr unsigned rule_grad(int d) { return 3u << (2 * d); }

// ---- the step's operators with linear filters (mg_step_linear.hip) ----
// rho, mu (Eq. rho), grad C in derivative units, unit normals.
hipError_t step_props(const Grid &g, const Phys &P, const double *C, double *rho, double *mu, F3 Cd, F3 nrm,
                      hipStream_t s);
// Curvature and surface-tension force (Eqs. surface-tension-k, surface-tension-uvw).
hipError_t step_surface(const Grid &g, double sigma, C3 nrm, C3 Cd, F3 st, hipStream_t s);
// Right-hand side of Eq. ph_disc, the affine part of p_hs's bottom halo included.
hipError_t step_rhs_hydrostatic(const Grid &g, double grav, C3 st, const double *rho, double *b, hipStream_t s);
// adv_c = q . grad q_c.
hipError_t step_advection(const Grid &g, C3 q, F3 adv, hipStream_t s);
// Isotropic Petrov-Galerkin diffusivity of each velocity component (Eq. k_Psi-n).
hipError_t step_pg_velocity(const Grid &g, C3 q, C3 adv, const double *rho, const double *mu, F3 kq, hipStream_t s);
// One predictor iteration (Eqs. Petrov, velocity-1): q~ into qt, (q^n + q~) / 2 into qnext.
hipError_t step_momentum(const Grid &g, const Phys &P, C3 qn, const double *p_hs, const double *p_nh,
                         const double *rho, C3 q, C3 kq, C3 st, C3 adv, F3 qt, F3 qnext, hipStream_t s);
// Right-hand side of Eq. ph_disc2 for the pressure increment.
hipError_t step_rhs_nonhydrostatic(const Grid &g, double dt, C3 qt, const double *rho, double *b, hipStream_t s);
// Eq. vel-cor: qout = qin - dt f(dp; w) / (m_l rho); p_nh += dp (qout may be qin).
hipError_t step_correct(const Grid &g, double dt, const double *dp, const double *rho, C3 qin, F3 qout, double *p_nh,
                        hipStream_t s);
// Anisotropic compressive diffusivities of the volume fraction (Sec. 2.3.5); advc = q . grad C.
hipError_t step_pg_volume_fraction(const Grid &g, double dt, const double *C, C3 Cd, C3 q, const double *advc, F3 kd,
                                   hipStream_t s);
// Eqs. Petrov-C, transport-indicator-1.
hipError_t step_volume_fraction(const Grid &g, double dt, const double *C, C3 kd, const double *advc, double *Cnew,
                                hipStream_t s);

}  // namespace nn4mg
