// Several steps per launch on tiles held in registers and LDS (xyl_tile.hip).
#pragma once
#include "xyl_internal.hpp"

namespace xyl {

constexpr int kTileMaxSteps = 32;     // steps per launch
constexpr int kTileMaxThreads = 1024;

constexpr int kTileMaxLds = 150 * 1024;

// A lattice cut into ntx x nty tiles of whole quads, T steps per launch, S
// sites per lane (1, 2 or, FP32, 4).
struct TilePlan {
    int ntx = 0, nty = 0;
    int T = 0;                        // most steps per launch
    int S = 0;
    int threads = 0;
};

// The widest and the highest tile, and the sides of the region that a tile of
// w x h sites works on for T steps: no halo along an axis that the tile spans
// whole (the region is periodic there), else T rows, and T columns rounded up
// to whole quads.
inline int tile_max_w(int Lx, int ntx) { return (Lx / kLaneSites + ntx - 1) / ntx * kLaneSites; }
inline int tile_max_h(int Ly, int nty) { return (Ly + nty - 1) / nty; }
inline int tile_region_w(int Lx, int w, int T) { return w == Lx ? w : w + 2 * ((T + 3) / 4 * 4); }
inline int tile_region_h(int Ly, int h, int T) { return h == Ly ? h : h + 2 * T; }
// LDS bytes: two tables of (sin, cos) per site of the region.
template <typename R>
inline size_t tile_lds(int W, int H) { return sizeof(R) * 4 * (size_t)W * (size_t)H; }

// The cheapest way (by the measured cost model in xyl_tile.hip) to take n
// steps, n even, in an even number of launches on `cus` CUs; false if no tile
// fits.  us (nullable) receives the model's time per step.
bool tile_plan(int Lx, int Ly, bool f64, int cus, uint64_t n, TilePlan* plan, double* us);
// Launches (an even number) that n steps take in launches of at most T.
inline uint64_t tile_launches(uint64_t n, int T) { return 2 * ((n + 2 * (uint64_t)T - 1) / (2 * (uint64_t)T)); }

// T steps from step k of the lattice v: angles and velocities read from th_in
// and u_in, written to th_out and u_out (distinct buffers).
template <typename R>
void launch_tile(const Lat<R>& v, const R* th_in, const R* u_in, R* th_out, R* u_out, const TilePlan& p, int T,
                 uint64_t k, hipStream_t s);

}  // namespace xyl
