// Several steps per launch on tiles held in registers and LDS (xyl_tile.hip).
#pragma once
#include <vector>

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

// The cheapest way (by the measured cost model in xyl_tile.hip) to take n
// steps, n even, in an even number of launches on `cus` CUs; false if no tile
// fits.  us (nullable) receives the model's time per step.
bool tile_plan(int Lx, int Ly, bool f64, int cus, uint64_t n, TilePlan* plan, double* us);
// Launches (an even number) that n steps take in launches of at most T.
inline uint64_t tile_launches(uint64_t n, int T) { return 2 * ((n + 2 * (uint64_t)T - 1) / (2 * (uint64_t)T)); }

// The same for lattices of several sizes in one launch: the shape all tiles
// share (T, S, threads), each size's tiles and the largest region's LDS.
struct TileSize {
    int Lx, Ly;
    int ntx = 0, nty = 0;
};
class TileFits {
  public:
    // the fewest tiles of each size at every shape considered for n steps
    TileFits(const std::vector<TileSize>& sizes, bool f64, int cus, uint64_t n);
    // the cheapest shape for count[i] lattices of size i (0: left out): its
    // time per step in us (1e30: none fits), the shape, the tiles of each size
    // and the LDS; the outputs may be NULL
    double best(const std::vector<long>& count, TilePlan* shape, std::vector<TileSize>* tiles, size_t* lds) const;

  private:
    struct Fit {
        int ntx, nty, H;
        size_t lds;
    };
    struct Shape {
        int cost, t, waves;
        uint64_t nl;
        std::vector<Fit> fits;    // by size; ntx = 0: does not fit
    };
    std::vector<TileSize> sizes_;
    std::vector<Shape> shapes_;
    bool f64_;
    int cus_;
    uint64_t n_;
};

// One workgroup of a batched launch: the sites it stores of replica rep.
struct TileTask {
    int32_t rep, x0, y0, w, h, pad;
};
// The tasks of one lattice cut into ntx x nty tiles.
void tile_tasks(int rep, int Lx, int Ly, int ntx, int nty, std::vector<TileTask>* out);
// T steps of every task's replica from step k = k_base + j (+ *kdev), in the
// launch after dk steps of a run that began with the angles in th[(k - dk) & 1]
// and the velocities in u: launch `flip` = 0, 2, .. of the run reads those and
// writes the other angle buffer and u2, launch 1, 3, .. goes back.  u2 is the
// replica's velocities' place in a second array: u2_base + (v.u - u_base).
// FP32 replicas have the factored kick.  lds: the bytes of the largest region.
template <typename R>
void launch_ensemble_tile(const Lat<R>* reps, const TileTask* tasks, int ntasks, const TilePlan& shape, size_t lds,
                          int model, int T, int flip, uint64_t dk, const R* u_base, R* u2_base, const uint64_t* kdev,
                          uint64_t j, hipStream_t s);

// Loads the kernels of xyl_tile.hip on the current device.
void load_tile_kernels();

// T steps from step k of the lattice v: angles and velocities read from th_in
// and u_in, written to th_out and u_out (distinct buffers).
template <typename R>
void launch_tile(const Lat<R>& v, const R* th_in, const R* u_in, R* th_out, R* u_out, const TilePlan& p, int T,
                 uint64_t k, hipStream_t s);

// The same, storing every state (XY): the one after the launch's step j at
// states + 2 j N (angles, then velocities), with `first` also the one it
// starts from, before it.
template <typename R>
void launch_tile_states(const Lat<R>& v, const R* th_in, const R* u_in, bool first, R* states, const TilePlan& p,
                        int T, uint64_t k, hipStream_t s);
// The same as launch_tile, also summing the staggered order parameter of every
// state that a step starts from (XY): order[j] has tile_order_parts(p) partial
// sums of the launch's step j.  launch_tile_order_sum adds those of `steps`
// steps up: out[6 j + 2] = sum / N.
inline int tile_order_parts(const TilePlan& p) { return p.ntx * p.nty * (p.threads / kWave); }
template <typename R>
void launch_tile_order(const Lat<R>& v, const R* th_in, const R* u_in, R* th_out, R* u_out, double* order,
                       const TilePlan& p, int T, uint64_t k, hipStream_t s);
void launch_tile_order_sum(const double* order, int n, double N, double* out, int steps, hipStream_t s);

// Checks a plan against what the kernels assume; the LDS of T steps with
// `tables` numbers per site.
size_t tile_check(int Lx, int Ly, bool f64, const TilePlan& p, int T, int tables);
// Reverse steps k + T - 1 .. k (xyl_adjoint.hip): states as
// launch_tile_states stores them (step k + j at states + 2 j N), (lt_in,
// lu_in) the adjoint at k + T, (lt_out, lu_out) at k, gacc 4 per tile.
template <typename R>
void launch_adjoint_tile(const Lat<R>& v, const R* states, const R* lt_in, const R* lu_in, R* lt_out, R* lu_out,
                         const double* cm, uint64_t cm_base, double* gacc, const TilePlan& p, int T, uint64_t k,
                         hipStream_t s);
// tile_plan for the reverse steps of the adjoint (any number of launches).
bool tile_plan_reverse(int Lx, int Ly, bool f64, int cus, uint64_t n, TilePlan* plan, double* us);

}  // namespace xyl
