// The GPP off-diagonal self-energy kernel (internal to libgw).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace gw {

// One launch holds ec energies of bc bands; scratch: T of every (band, energy)
// pair at 0, with bc > 1 their products T M^T at off_part, the energies (device
// copy, [ne]) at off_e, total bytes in all.
struct GppLayout {
    int ec = 1, bc = 1;
    size_t off_part = 0, off_e = 0, total = 0;
};
// The layout for nb bands in a workspace of `bytes` (0: the library's scratch).
// Any workspace that holds one band (nb = 1) will do; a larger one takes more
// bands per launch.
GppLayout gpp_layout(int ns, int ng, int nb, int ne, size_t bytes);

// sigma[e] (device [ne][ns][ns], overwritten) = sum_n conj(M_n) P^{n e} M_n^T
// with M device [nb][ns][ng], e_n and occupied host [nb], omega2 device
// [ng][ng], wt device [ng][ng], v device [ng]; the energies are at base +
// L.off_e.
void run_gpp_sigma(const double2* m, int nb, int ns, int ng, const double* e_n,
                   const int32_t* occupied, int ne, const double2* omega2, const double* wt,
                   const double* v, double2* sigma, char* base, const GppLayout& L, hipStream_t s);

}  // namespace gw
