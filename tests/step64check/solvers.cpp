// The FP64 step's small solvers, built for the host: 6x6 (packed upper triangle) and 3x3
// systems in place.  Not a GPU build.
#include <hip/hip_runtime.h>
inline unsigned long long __builtin_amdgcn_ballot_w64(bool p) { return p; }  // named by the step, not called here
#include "mppi_step64.h"

extern "C" void solve_6x6(double* Q, double* r) { mppi::f64::ldl6_solve(Q, r); }

// a: the lower triangle a00, a10, a11, a20, a21, a22; n right sides of three
extern "C" void solve_3x3(const double* a, double* b, int n)
{
    const mppi::f64::Ldl3 f = mppi::f64::ldl3(a[0], a[1], a[2], a[3], a[4], a[5]);
    for (int i = 0; i < n; ++i) mppi::f64::solve3(f, b[3 * i], b[3 * i + 1], b[3 * i + 2]);
}
