// C entries over the device building blocks of physics.h, built for the CPU
// by tests/test_device_math.py.
#include "physics.h"

using namespace mfc;

extern "C" {

// WENO5 on non-uniform cells from a coefficient row.
int dm_coefs() { return kStretchCoef; }
void dm_weno5_nonuniform(const double *row, const double *s, double eps, double *plus, double *minus)
{
    weno5_nonuniform_pair<double>(row, s[0], s[1], s[2], s[3], s[4], eps, *plus, *minus);
}
void dm_weno5_nonuniform_f(const double *row, const float *s, float eps, float *plus, float *minus)
{
    weno5_nonuniform_pair<float>(row, s[0], s[1], s[2], s[3], s[4], eps, *plus, *minus);
}

// Uniform cells, the epsilon as the host passes it on.
void dm_weno5(const double *s, double eps, double *plus, double *minus)
{
    weno5_pair(s[0], s[1], s[2], s[3], s[4], usable_eps(eps, false, false, false), *plus, *minus);
}
void dm_weno3(const double *s, double eps, double *plus, double *minus)
{
    weno3_pair(s[0], s[1], s[2], usable_eps(eps, true, false, false), *plus, *minus);
}
void dm_weno3_f(const float *s, float eps, float *plus, float *minus)
{
    weno3_pair(s[0], s[1], s[2], (float)usable_eps(eps, true, true, false), *plus, *minus);
}
void dm_weno5_f(const float *s, float eps, float *plus, float *minus)
{
    weno5_pair(s[0], s[1], s[2], s[3], s[4], (float)usable_eps(eps, false, true, false), *plus, *minus);
}

}  // extern "C"

static Grid fluids(const double *gamma, const double *pi_inf)
{
    Grid g{};
    g.g1 = 1.0 / (gamma[0] - 1.0);
    g.g2 = 1.0 / (gamma[1] - 1.0);
    g.h1 = gamma[0] * pi_inf[0] * g.g1;
    g.h2 = gamma[1] * pi_inf[1] * g.g2;
    return g;
}

// One-dimensional HLLC flux (5 rows) and face velocity; whether a side is
// non-physical.
extern "C" int dm_hllc(const double *gamma, const double *pi_inf, const double *wL, const double *wR, double *F, double *uf)
{
    return hllc<1, 0, double>(fluids(gamma, pi_inf), wL, wR, F, *uf);
}
extern "C" int dm_hllc_f(const double *gamma, const double *pi_inf, const float *wL, const float *wR, float *F, float *uf)
{
    return hllc<1, 0, float>(fluids(gamma, pi_inf), wL, wR, F, *uf);
}
