// The device arithmetic of csrc/device_math.hpp on arrays, for the CPU tests.
#include "../../paper_2607_19277_amd/csrc/device_math.hpp"

extern "C" void srhd_con2prim(long n, const double *U, double g, double *w, int *ok) {
    for (long q = 0; q < n; ++q) ok[q] = agile::srhd_con2prim_fast(U + 5 * q, g, w + 5 * q);
}

// HLL (0), HLLC (1) or local Lax-Friedrichs (2) flux, FP64
extern "C" void euler_flux(int rs, long n, const double *wL, const double *wR, double gamma, double *F) {
    const double igm1 = 1.0 / (gamma - 1.0);
    for (long q = 0; q < n; ++q, wL += 5, wR += 5, F += 5) {
        if (rs == 0) agile::riemann<0, double>(wL, wR, gamma, igm1, F);
        else if (rs == 1) agile::riemann<1, double>(wL, wR, gamma, igm1, F);
        else agile::riemann<2, double>(wL, wR, gamma, igm1, F);
    }
}

extern "C" void mhd_flux(long n, const double *wL, const double *wR, double gamma, double ch, double *F) {
    for (long q = 0; q < n; ++q)
        agile::mhd_hll(wL + 9 * q, wR + 9 * q, gamma, 1.0 / (gamma - 1.0), ch, 0.5 / ch, F + 9 * q);
}

extern "C" void srhd_flux(long n, const double *wL, const double *wR, double g, double *F) {
    for (long q = 0; q < n; ++q)
        agile::riemann<3, double>(wL + 5 * q, wR + 5 * q, g, 1.0 / (g - 1.0), F + 5 * q);
}
