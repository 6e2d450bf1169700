// The device arithmetic of csrc/device_math.hpp on arrays, for the CPU tests.
#include "../../paper_2607_19277_amd/csrc/device_math.hpp"

extern "C" void srhd_con2prim(long n, const double *U, double g, double *w, int *ok) {
    for (long q = 0; q < n; ++q) ok[q] = agile::srhd_con2prim_fast(U + 5 * q, g, w + 5 * q);
}
