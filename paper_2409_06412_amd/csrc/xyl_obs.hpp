// Scratch sizes and shapes of the observables' launchers, shared by the kernels
// and the host runtime.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>

namespace xyl {

// Axis lengths that go through the transform: no prime factor above 7.
inline bool sf_smooth(int L) {
    for (int p : {2, 3, 5, 7})
        while (L % p == 0) L /= p;
    return L == 1;
}

// Launch shape of the transform: nlb lines per workgroup at a time (at most
// 4096 points), nsub rows of sums per workgroup (short spectra split the lines
// over the threads), and the grid: two workgroups per CU where there are lines
// enough, the rest of the lines in further batches.
struct SfShape {
    int nlb, nsub, grid;
};
inline SfShape sf_shape(int L, int nlines, int kmax) {
    SfShape h;
    h.nlb = std::max(1, 4096 / L);
    // smaller batches while that still leaves CUs without one
    while (h.nlb > 1 && (nlines + h.nlb - 1) / h.nlb < 256) h.nlb = (h.nlb + 1) / 2;
    h.nsub = std::max(1, std::min(h.nlb, 512 / (kmax + 1)));
    h.grid = std::min((nlines + h.nlb - 1) / h.nlb, 512);
    return h;
}

// Doubles of scratch launch_structure_factor needs: the workgroups' sums, or
// for other lengths the lines' rotors (complex) and spectra.
inline size_t structure_factor_scratch(int Lx, int Ly, int axis, int kmax) {
    const int L = axis == 0 ? Lx : Ly, nlines = axis == 0 ? Ly : Lx;
    if (sf_smooth(L)) {
        const SfShape h = sf_shape(L, nlines, kmax);
        return (size_t)h.grid * h.nsub * ((size_t)kmax + 1);
    }
    return 2 * (size_t)Lx * Ly + (size_t)nlines * ((size_t)kmax + 1);
}

// Doubles of scratch launch_correlation needs: the structure factor up to L/2
// and its scratch, or for other lengths one row of pair sums per line.
inline size_t correlation_scratch(int Lx, int Ly, int axis, int rmax) {
    const int L = axis == 0 ? Lx : Ly;
    if (sf_smooth(L)) return structure_factor_scratch(Lx, Ly, axis, L / 2) + (size_t)(L / 2 + 1);
    return (size_t)(axis == 0 ? Ly : Lx) * ((size_t)rmax + 1);
}

// C_delta(r), r = 0..rmax, and S_delta(k), k = 0..kmax, into `out`; tw: the
// axis' twiddle table (launch_sf_twiddles; unused for other lengths).
template <typename R>
void launch_correlation(const R* th, int Lx, int Ly, int sx, int sy, int model, int axis, int rmax, const double* tw,
                        double* scratch, double* out, hipStream_t s);
template <typename R>
void launch_structure_factor(const R* th, int Lx, int Ly, int sx, int sy, int model, int axis, int kmax,
                             const double* tw, double* scratch, double* out, hipStream_t s);
// exp(-2 pi i m / L), m < L, as (re, im)
void launch_sf_twiddles(double* tw, int L, hipStream_t s);

}  // namespace xyl
