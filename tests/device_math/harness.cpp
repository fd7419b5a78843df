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

}  // extern "C"
