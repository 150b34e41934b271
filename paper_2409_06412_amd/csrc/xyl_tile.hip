// Several BBK steps per launch on 2-D tiles, for lattices too small to keep
// the chip busy with one or two steps per launch.
//
// What bounded those: a launch that steps 512^2 sites once or twice takes 5 to
// 7 us, most of it dispatch, one round trip to memory and the latency of one
// wave's chain of instructions, whatever the lattice's size.  Here a workgroup
// loads a region (its tile and a halo of T sites on each side), keeps angles,
// velocities and own rotors in registers and all rotors in LDS, and takes T
// steps, each of them valid on a region one site smaller; only the tile is
// stored.  The halo is recomputed by the neighbouring tiles with the same
// arithmetic (the shared rotor / site_force / site_update / noise4), so the
// states equal single steps bit for bit.  An axis that a tile spans whole has
// no halo: the region is periodic there.
//
// One barrier per step (the rotor tables are double-buffered).  The draws of a
// step do not depend on the state and are computed before the barrier.  Left
// and right rotors come from the adjacent lanes by DPP, except at a wave's
// ends and at a periodic region's, upper and lower ones from the table.
//
// Sites per lane S: a lane of S = 4 owns a Philox block; with S = 2 (and 1)
// the 2 (4) lanes of a block each compute it for one of 2 (4) successive steps
// and exchange the draws, which shortens a step's chain where there is about
// one wave per SIMD (256^2, FP32, T = 8: 1.03 -> 0.90 us per step; 64^2, FP64:
// 2.37 -> 1.82 with S = 1) and costs throughput where there are many.  In FP64
// with S = 2 each lane draws its own Box-Muller pair from a block of its own
// (the FP64 logarithm, root and sine are what a step waits for; 512^2: 4.4 us
// per step against 4.9 with the exchange).
//
// Measured, us per step before (one or two steps per launch) and with tiles:
// 64^2 FP64 7.4 -> 1.8; 96^2 FP32 5.3 -> 0.9; 512^2 FP32 3.04 -> 1.30 and FP64
// 8.1 -> 4.5; 772 x 501 FP32 4.3 -> 1.54; 1024^2 FP32 4.6 -> 2.9; 1448^2 10.8
// -> 5.4.  With one wave per SIMD a step costs 0.45 to 0.7 us of latency, from
// about three waves per SIMD on it is bound by VALU issue (0.317 us per wave
// and SIMD, 190 issue slots), of which the halo takes about half (512^2: 95
// lane-instructions per site-update, 41 where whole rows step); a launch's
// dispatch, first loads and stores take another 2.75 us.
#include <cmath>
#include <mutex>
#include <set>
#include <type_traits>

#include "xyl_tile_device.hpp"

namespace xyl {

// What a tile launch does beyond storing the last state:
enum : int {
    kTilePlain = 0,
    kTileStates = 1,   // stores every state, step j of the run at out + 2 j N (angles, then velocities)
    kTileOrder = 2     // sums the staggered order parameter's component of every state it steps from (XY)
};
template <typename R>
struct TileIO {
    const R* th_in;
    const R* u_in;
    R* th_out;
    R* u_out;
    R* states = nullptr;         // kTileStates: where the state after the launch's first step goes
    int first = 0;               //   1: the state it starts from goes before it
    double* order = nullptr;     // kTileOrder: [step of the launch][workgroup][wave]
};

template <typename R, int M, bool F, int S, int KIND>
__device__ __forceinline__ void tile_run(const Lat<R>& v, const TileIO<R>& io, const TileBox& b, int T, uint64_t k,
                                         R* lds, R* coef) {
    constexpr bool kPair = tile_own_pair<R, S>();
    constexpr int P = tile_share<R, S>();
    const TileLane<S> L(v.Lx, v.Ly, b, T);
    const int WH = L.W * L.H;
    const size_t N = (size_t)v.Lx * v.Ly;
    R th[S], u[S], s[S], c[S];
    tile_load<R, S>(io.th_in + L.off, th);
    tile_load<R, S>(io.u_in + L.off, u);
    // the steps' noise amplitudes, while the loads are under way
    for (int j = threadIdx.x; j < T; j += (int)blockDim.x) coef[j] = noise_coeff<R, F>(v, k + (uint64_t)j);
    if constexpr (KIND == kTileStates) {
        if (io.first && L.own) {
            tile_store<R, S>(io.states - 2 * N + L.off, th);
            tile_store<R, S>(io.states - N + L.off, u);
        }
    }
    const int tab = 2 * WH;
#pragma unroll
    for (int e = 0; e < S; ++e) rotor<R, M>(th[e], s[e], c[e]);
    if (L.in) {
        tile_store<R, S>(lds + L.i0, s);
        tile_store<R, S>(lds + WH + L.i0, c);
    }
    __syncthreads();
    R d[4];
    auto draw = [&](int t) {
        const uint64_t kt = k + (uint64_t)(t + (P > 1 ? L.part : 0));
        if constexpr (kPair) {
            const U32x4 r = philox4x32_10(L.q, v.replica, (uint32_t)kt, (uint32_t)(kt >> 32), v.seed_lo, v.seed_hi);
            const bool hi = (L.off & 2) != 0;
            Prec<R>::box_muller(hi ? r.v[2] : r.v[0], hi ? r.v[3] : r.v[1], d[0], d[1]);
        } else if constexpr (sizeof(R) == 4) {
            const R hs = coef[min(t + (P > 1 ? L.part : 0), T - 1)];
            noise4_kick<R>(L.q, v.replica, kt, v.seed_lo, v.seed_hi, hs, d, noise_u2<R, F>(v));
        } else {
            noise4<R>(L.q, v.replica, kt, v.seed_lo, v.seed_hi, d);
        }
    };
    auto step = [&](auto sub, int t) {
        constexpr int J = decltype(sub)::value;
        const uint64_t kt = k + (uint64_t)t;
        const bool act = t < L.dist;
        if constexpr (J == 0) {
            if (P > 1 || act) draw(t);
        }
        if constexpr (KIND == kTileOrder) {
            // signs: the group starts at a multiple of S on the lattice
            double m = 0.0;
            if (L.own) {
#pragma unroll
                for (int e = 0; e < S; ++e) {
                    const bool neg = ((((L.gx + e) * v.stag_x) + (L.gy * v.stag_y)) & 1) != 0;
                    m += neg ? -(double)c[e] : (double)c[e];
                }
            }
            m = wave_sum1(m);
            if ((threadIdx.x & (kWave - 1)) == 0)
                io.order[((size_t)t * gridDim.x + blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave] = m;
        }
        if (t) __syncthreads();
        const R* St = lds + (t & 1) * tab;
        const R* Ct = St + WH;
        // (the DPP moves run with every lane of the wave enabled)
        R sL = from_lane_below(s[S - 1]), cL = from_lane_below(c[S - 1]);
        R sR = from_lane_above(s[0]), cR = from_lane_above(c[0]);
        R su[S], cu[S], sd[S], cd[S];
        tile_load<R, S>(St + L.iu, su);
        tile_load<R, S>(Ct + L.iu, cu);
        tile_load<R, S>(St + L.id, sd);
        tile_load<R, S>(Ct + L.id, cd);
        if (L.edge_l) {
            sL = St[L.il];
            cL = Ct[L.il];
        }
        if (L.edge_r) {
            sR = St[L.ir];
            cR = Ct[L.ir];
        }
        R n[S];
        tile_draws<S, P, J>(d, L.part, n);
        if (act) {
            const bool fresh = kt == v.fresh_k;
            const R hs = coef[t];
#pragma unroll
            for (int e = 0; e < S; ++e) {
                const R sxm = e == 0 ? sL : s[e - 1], cxm = e == 0 ? cL : c[e - 1];
                const R sxp = e == S - 1 ? sR : s[e + 1], cxp = e == S - 1 ? cR : c[e + 1];
                const R f = site_force<R, M, F>(v, s[e], c[e], sxm, cxm, sxp, cxp, su[e], cu[e], sd[e], cd[e], th[e],
                                                n[e]);
                R w;
                site_update<R, M, F>(v, f, u[e], th[e], n[e], hs, fresh, w, u[e], th[e]);
            }
            if constexpr (KIND == kTileStates) {
                if (L.own) {
                    tile_store<R, S>(io.states + 2 * N * (size_t)t + L.off, th);
                    tile_store<R, S>(io.states + 2 * N * (size_t)t + N + L.off, u);
                }
            }
            if (t + 1 < T) {
                R* Sn = lds + ((t + 1) & 1) * tab;
#pragma unroll
                for (int e = 0; e < S; ++e) rotor<R, M>(th[e], s[e], c[e]);
                tile_store<R, S>(Sn + L.i0, s);
                tile_store<R, S>(Sn + WH + L.i0, c);
            }
        }
    };
    for (int t = 0; t < T; t += P) {
        step(std::integral_constant<int, 0>{}, t);
        if constexpr (P >= 2) {
            if (t + 1 < T) step(std::integral_constant<int, 1>{}, t + 1);
        }
        if constexpr (P == 4) {
            if (t + 2 < T) step(std::integral_constant<int, 2>{}, t + 2);
            if (t + 3 < T) step(std::integral_constant<int, 3>{}, t + 3);
        }
    }
    if constexpr (KIND != kTileStates) {
        if (L.own) {
            tile_store<R, S>(io.th_out + L.off, th);
            tile_store<R, S>(io.u_out + L.off, u);
        }
    }
}

template <typename R, int M, bool F, int S, int KIND, int NT>
__global__ __launch_bounds__(NT) void k_tile(Lat<R> v, TileIO<R> io, int ntx, int nty, int T, uint64_t k) {
    extern __shared__ double2 tile_lds_mem[];
    __shared__ R coef[kTileMaxSteps];
    const int b = xcd_contiguous_block(blockIdx.x, gridDim.x);
    const int ty = b / ntx, tx = b - ty * ntx;
    tile_run<R, M, F, S, KIND>(v, io, tile_box(tx, ty, ntx, nty, v.Lx, v.Ly), T, k, reinterpret_cast<R*>(tile_lds_mem),
                               coef);
}

template <typename R, int M, bool F, int S, int NT>
__global__ __launch_bounds__(NT) void k_ensemble_tile(const Lat<R>* __restrict__ reps,
                                                      const TileTask* __restrict__ tasks, int T, int flip,
                                                      uint64_t dk, const R* u_base, R* u2_base, const uint64_t* kdev,
                                                      uint64_t j0) {
    extern __shared__ double2 tile_lds_mem[];
    __shared__ R coef[kTileMaxSteps];
    const TileTask t = tasks[xcd_contiguous_block(blockIdx.x, gridDim.x)];
    const Lat<R>& v = reps[t.rep];
    const uint64_t k = v.k_base + j0 + (kdev ? *kdev : 0);
    const int a = (int)((k - dk + (uint64_t)v.cur) & 1) ^ flip;
    R* u = v.u;
    R* u2 = u2_base + (u - u_base);
    const TileIO<R> io{v.th[a], flip ? u2 : u, v.th[a ^ 1], flip ? u : u2};
    tile_run<R, M, F, S, kTilePlain>(v, io, TileBox{t.x0, t.y0, t.w, t.h}, T, k, reinterpret_cast<R*>(tile_lds_mem), coef);
}

// Cost model of one launch of T steps, in us: a fixed part (dispatch, the
// first loads, the stores), a part per wave of the busiest CU (its prologue),
// and per step the larger of the latency of one wave's step and the issue
// time of the busiest CU's resident waves, combined as
// sqrt(lat^2 + (issue x)^2) with x the waves per SIMD; workgroups beyond what
// a CU holds at once run in further rounds.  Rows of the region whose last
// valid step has passed drop out wave by wave, so x counts them about half.
struct TileCost {
    int S;
    double fixed, prologue, lat, issue;
    int max_waves;            // waves per CU by registers
};

static const TileCost kCost32[] = {{4, 2.75, 0.25, 0.60, 0.317, 32}, {2, 2.75, 0.15, 0.45, 0.22, 32}};
static const TileCost kCost64[] = {{2, 3.0, 0.5, 1.20, 0.90, 16}, {1, 3.0, 0.3, 0.73, 0.56, 16}};

// Time per step (us) of n steps in nl launches of up to t: `wgs` workgroups of
// `waves` waves and `lds` bytes on the busiest CU, a region's rows alive for
// the fraction `alive` of the steps.
static double tile_cost(const TileCost& c, uint64_t n, uint64_t nl, int waves, size_t lds, int wgs, double alive) {
    const int fit = std::max(1, std::min((int)(160 * 1024 / lds), c.max_waves / waves));
    auto round = [&](int held) {
        const double x = 0.25 * waves * held * alive;
        return std::sqrt(c.lat * c.lat + c.issue * c.issue * x * x);
    };
    const double step = (wgs / fit) * round(fit) + (wgs % fit ? round(wgs % fit) : 0.0);
    return ((double)nl * (c.fixed + c.prologue * 0.25 * waves * wgs) + (double)n * step) / (double)n;
}
static double tile_alive(int H, int Ly, int t) {
    return H == Ly ? 1.0 : 0.5 + 0.5 * (double)std::max(0, H - t - 1) / H;
}

// The cheapest plan for n >= 2 steps, two or more per launch, with `tables` LDS
// numbers per site, in an even number of launches or (pairs = false) in any.
static bool tile_search(const TileCost* costs, int tables, bool pairs, int max_lanes, int Lx, int Ly, bool f64, int cus, uint64_t n,
                        TilePlan* plan, double* us) {
    const size_t es = f64 ? 8 : 4;
    const int quads = Lx / kLaneSites;
    double best = 1e30;
    for (int i = 0; i < 2; ++i) {
        const TileCost& c = costs[i];
        for (int T = 2; T <= 12; ++T) {
            const uint64_t nl = pairs ? tile_launches(n, T) : (n + T - 1) / T;
            const int t = (int)((n + nl - 1) / nl);      // the longest launch's steps
            if (t < T && T > 2) continue;                // as a smaller T
            if (t > Lx || t > Ly) continue;
            int last_w = 0;
            for (int ntx = 1; ntx <= quads && ntx <= 256; ntx += std::max(1, ntx / 8)) {
                const int w = tile_max_w(Lx, ntx);
                if (w == last_w) continue;               // more tiles of the same width
                last_w = w;
                const int W = tile_region_w(Lx, w, t);
                if (W != Lx && (W - w) / 2 > Lx) continue;
                // the tallest region that fits, hence the fewest tiles; more
                // than about twice as many only add halo
                const long rows = std::min<long>((long)max_lanes * c.S / W, (long)(kTileMaxLds / (tables * es * (size_t)W)));
                const long h_most = rows >= Ly ? Ly : rows - 2 * t;
                if (h_most < 1) continue;
                const int per0 = (int)std::max<long>(1, ((Ly + h_most - 1) / h_most) * ntx / cus);
                for (int per = per0; per <= 2 * per0 + 2; per += std::max(1, per / 6)) {
                    const int nty = std::min(Ly, std::max(1, per * cus / ntx));
                    const int h = tile_max_h(Ly, nty), H = tile_region_h(Ly, h, t);
                    const long lanes = (long)(W / c.S) * H;
                    if (lanes > max_lanes) continue;
                    const size_t lds = tables * es * (size_t)W * H;
                    if (lds > (size_t)kTileMaxLds) continue;
                    const int waves = (int)((lanes + kWave - 1) / kWave);
                    const int wgs = (ntx * nty + cus - 1) / cus;
                    const double total = tile_cost(c, n, nl, waves, lds, wgs, tile_alive(H, Ly, t));
                    if (total < best) {
                        best = total;
                        plan->ntx = ntx;
                        plan->nty = nty;
                        plan->T = t;
                        plan->S = c.S;
                        plan->threads = waves * kWave;
                    }
                }
            }
        }
    }
    if (us) *us = best;
    return best < 1e30;
}

bool tile_plan(int Lx, int Ly, bool f64, int cus, uint64_t n, TilePlan* plan, double* us) {
    if (Lx % kLaneSites != 0 || n < 2) return false;
    return tile_search(f64 ? kCost64 : kCost32, 4, true, kTileMaxThreads, Lx, Ly, f64, cus, n, plan, us);
}

bool tile_plan_reverse(int Lx, int Ly, bool f64, int cus, uint64_t n, TilePlan* plan, double* us) {
    // (FP64 regions of more than 512 lanes would spill)
    static const TileCost rev32[] = {{4, 4.0, 0.35, 0.80, 0.62, 16}, {2, 4.0, 0.2, 0.50, 0.36, 16}};
    static const TileCost rev64[] = {{2, 4.0, 0.5, 1.50, 1.25, 8}, {1, 4.0, 0.3, 0.90, 0.88, 12}};
    if (Lx % kLaneSites != 0 || n < 2) return false;
    return tile_search(f64 ? rev64 : rev32, 6, false, f64 ? 512 : kTileMaxThreads, Lx, Ly, f64, cus, n, plan, us);
}

// The fewest tiles of a lattice whose regions fit `lanes` lanes of S sites;
// false if none fit.
static bool tile_fit(int Lx, int Ly, int S, int T, int lanes, size_t es, int* ntx_o, int* nty_o, int* H_o,
                     size_t* lds_o) {
    if (T > Lx || T > Ly) return false;
    long best = 0;
    int last_w = 0;
    // (a region has at least min(Ly, 2 T + 1) rows: wider tiles cannot fit)
    const int w_max = std::max(kLaneSites, lanes * S / std::min(Ly, 2 * T + 1));
    for (int ntx = std::max(1, Lx / w_max); ntx <= Lx / kLaneSites; ++ntx) {
        const int w = tile_max_w(Lx, ntx);
        if (w == last_w) continue;
        last_w = w;
        if (best && ntx >= best) break;
        const int W = tile_region_w(Lx, w, T);
        if (W != Lx && (W - w) / 2 > Lx) continue;
        const int rows = (int)std::min<long>(lanes / (W / S), (long)(kTileMaxLds / (4 * es * (size_t)W)));
        const int h = rows >= Ly ? Ly : rows - 2 * T;
        if (h < 1) continue;
        const int nty = (Ly + h - 1) / h;
        if (best && (long)ntx * nty >= best) continue;
        best = (long)ntx * nty;
        *ntx_o = ntx;
        *nty_o = nty;
        *H_o = tile_region_h(Ly, tile_max_h(Ly, nty), T);
        *lds_o = 4 * es * (size_t)W * (size_t)*H_o;
    }
    return best != 0;
}

TileFits::TileFits(const std::vector<TileSize>& sizes, bool f64, int cus, uint64_t n)
    : sizes_(sizes), f64_(f64), cus_(cus), n_(n) {
    if (n < 2) return;
    for (int c = 0; c < 2; ++c) {
        const int S = (f64 ? kCost64 : kCost32)[c].S;
        for (int T : {2, 4, 6, 8, 10}) {
            Shape sh;
            sh.cost = c;
            sh.nl = tile_launches(n, T);
            sh.t = (int)((n + sh.nl - 1) / sh.nl);
            bool seen = false;
            for (const Shape& o : shapes_) seen = seen || (o.cost == c && o.t == sh.t);
            if (seen) continue;
            for (int waves : {4, 6, 8, 10, 12, 14, 15, 16}) {
                sh.waves = waves;
                sh.fits.clear();
                for (const TileSize& z : sizes) {
                    Fit f{0, 0, 0, 0};
                    if (!tile_fit(z.Lx, z.Ly, S, sh.t, waves * kWave, f64 ? 8 : 4, &f.ntx, &f.nty, &f.H, &f.lds))
                        f.ntx = 0;
                    sh.fits.push_back(f);
                }
                shapes_.push_back(sh);
            }
        }
    }
}

double TileFits::best(const std::vector<long>& count, TilePlan* shape, std::vector<TileSize>* tiles,
                      size_t* lds_o) const {
    double best = 1e30;
    const Shape* pick = nullptr;
    size_t pick_lds = 0;
    for (const Shape& sh : shapes_) {
        long wgs = 0;
        size_t lds = 0;
        double alive = 0.0;
        bool ok = true;
        for (size_t i = 0; i < sizes_.size(); ++i) {
            if (count[i] == 0) continue;
            const Fit& f = sh.fits[i];
            if (f.ntx == 0) {
                ok = false;
                break;
            }
            wgs += (long)f.ntx * f.nty * count[i];
            lds = std::max(lds, f.lds);
            alive = std::max(alive, tile_alive(f.H, sizes_[i].Ly, sh.t));
        }
        if (!ok || wgs == 0 || wgs > (1L << 30)) continue;
        const double us = tile_cost((f64_ ? kCost64 : kCost32)[sh.cost], n_, sh.nl, sh.waves, lds,
                                    (int)((wgs + cus_ - 1) / cus_), alive);
        if (us < best) {
            best = us;
            pick = &sh;
            pick_lds = lds;
        }
    }
    if (!pick) return best;
    if (shape) {
        *shape = TilePlan();
        shape->T = pick->t;
        shape->S = (f64_ ? kCost64 : kCost32)[pick->cost].S;
        shape->threads = pick->waves * kWave;
    }
    if (tiles) {
        *tiles = sizes_;
        for (size_t i = 0; i < sizes_.size(); ++i) {
            (*tiles)[i].ntx = count[i] ? pick->fits[i].ntx : 0;
            (*tiles)[i].nty = count[i] ? pick->fits[i].nty : 0;
        }
    }
    if (lds_o) *lds_o = pick_lds;
    return best;
}

template <typename K>
static void allow_tile_lds(K* kernel) {
    static std::mutex mu;
    static std::set<std::pair<int, const void*>> allowed;
    int dev = 0;
    check_hip(hipGetDevice(&dev), "hipGetDevice");
    std::lock_guard<std::mutex> lk(mu);
    const auto key = std::make_pair(dev, reinterpret_cast<const void*>(kernel));
    if (allowed.count(key)) return;
    check_hip(hipFuncSetAttribute(key.second, hipFuncAttributeMaxDynamicSharedMemorySize, kTileMaxLds),
              "hipFuncSetAttribute");
    allowed.insert(key);
}

template <typename R, int M, bool F, int S, int KIND, int NT>
static void launch_tile_nt(const Lat<R>& v, const TileIO<R>& io, const TilePlan& p, int T, size_t lds, uint64_t k,
                           hipStream_t s) {
    allow_tile_lds(k_tile<R, M, F, S, KIND, NT>);
    k_tile<R, M, F, S, KIND, NT><<<p.ntx * p.nty, p.threads, lds, s>>>(v, io, p.ntx, p.nty, T, k);
    check_hip(hipGetLastError(), "tile kernel launch");
}

template <typename R, int M, bool F, int S, int KIND>
static void launch_tile_s(const Lat<R>& v, const TileIO<R>& io, const TilePlan& p, int T, size_t lds, uint64_t k,
                          hipStream_t s) {
    if (p.threads <= 512) launch_tile_nt<R, M, F, S, KIND, 512>(v, io, p, T, lds, k, s);
    else launch_tile_nt<R, M, F, S, KIND, 1024>(v, io, p, T, lds, k, s);
}

template <typename R, int M, bool F, int KIND>
static void launch_tile_m(const Lat<R>& v, const TileIO<R>& io, const TilePlan& p, int T, size_t lds, uint64_t k,
                          hipStream_t s) {
    if constexpr (sizeof(R) == 4) {
        if (p.S == 4) {
            launch_tile_s<R, M, F, 4, KIND>(v, io, p, T, lds, k, s);
            return;
        }
    }
    if constexpr (sizeof(R) == 4) {
        launch_tile_s<R, M, F, 2, KIND>(v, io, p, T, lds, k, s);
    } else {
        if (p.S == 2) launch_tile_s<R, M, F, 2, KIND>(v, io, p, T, lds, k, s);
        else launch_tile_s<R, M, F, 1, KIND>(v, io, p, T, lds, k, s);
    }
}

static bool sites_per_lane_ok(int S, bool f64) { return S == 2 || S == (f64 ? 1 : 4); }

void tile_tasks(int rep, int Lx, int Ly, int ntx, int nty, std::vector<TileTask>* out) {
    for (int ty = 0; ty < nty; ++ty)
        for (int tx = 0; tx < ntx; ++tx) {
            const TileBox b = tile_box(tx, ty, ntx, nty, Lx, Ly);
            out->push_back(TileTask{rep, b.x0, b.y0, b.w, b.h, 0});
        }
}

template <typename R, int M, bool F, int S, int NT>
static void launch_ensemble_tile_nt(const Lat<R>* reps, const TileTask* tasks, int ntasks, const TilePlan& p,
                                    size_t lds, int T, int flip, uint64_t dk, const R* ub, R* u2b,
                                    const uint64_t* kdev, uint64_t j, hipStream_t s) {
    allow_tile_lds(k_ensemble_tile<R, M, F, S, NT>);
    k_ensemble_tile<R, M, F, S, NT>
        <<<ntasks, p.threads, lds, s>>>(reps, tasks, T, flip, dk, ub, u2b, kdev, j);
    check_hip(hipGetLastError(), "ensemble tile kernel launch");
}

template <typename R, int M>
static void launch_ensemble_tile_m(const Lat<R>* reps, const TileTask* tasks, int ntasks, const TilePlan& p,
                                   size_t lds, int T, int flip, uint64_t dk, const R* ub, R* u2b,
                                   const uint64_t* kdev, uint64_t j, hipStream_t s) {
    constexpr bool F = sizeof(R) == 4;
    if constexpr (sizeof(R) == 4) {
        if (p.S == 4) {
            launch_ensemble_tile_nt<R, M, F, 4, 1024>(reps, tasks, ntasks, p, lds, T, flip, dk, ub, u2b, kdev, j, s);
            return;
        }
    }
    if constexpr (sizeof(R) == 8) {
        if (p.S == 1) {
            launch_ensemble_tile_nt<R, M, F, 1, 1024>(reps, tasks, ntasks, p, lds, T, flip, dk, ub, u2b, kdev, j, s);
            return;
        }
    }
    launch_ensemble_tile_nt<R, M, F, 2, 1024>(reps, tasks, ntasks, p, lds, T, flip, dk, ub, u2b, kdev, j, s);
}

template <typename R>
void launch_ensemble_tile(const Lat<R>* reps, const TileTask* tasks, int ntasks, const TilePlan& p, size_t lds,
                          int model, int T, int flip, uint64_t dk, const R* u_base, R* u2_base, const uint64_t* kdev,
                          uint64_t j, hipStream_t s) {
    if (ntasks < 1 || T < 1 || T > p.T || p.T > kTileMaxSteps || p.threads > kTileMaxThreads ||
        p.threads % kWave != 0 || lds > kTileMaxLds || !sites_per_lane_ok(p.S, sizeof(R) == 8))
        throw Error(-5, "ensemble tile launch: shape not supported");
    if (model == kModelSI)
        launch_ensemble_tile_m<R, kModelSI>(reps, tasks, ntasks, p, lds, T, flip, dk, u_base, u2_base, kdev, j, s);
    else
        launch_ensemble_tile_m<R, kModelXY>(reps, tasks, ntasks, p, lds, T, flip, dk, u_base, u2_base, kdev, j, s);
}

// The LDS of the plan's launches of T steps with `tables` rotor tables; checks
// what the kernels assume.
size_t tile_check(int Lx, int Ly, bool f64, const TilePlan& p, int T, int tables) {
    const int wmax = tile_max_w(Lx, p.ntx), hmax = tile_max_h(Ly, p.nty);
    const int W = tile_region_w(Lx, wmax, T), H = tile_region_h(Ly, hmax, T);
    const size_t lds = (f64 ? 8 : 4) * (size_t)tables * (size_t)W * H;
    if (T < 1 || T > p.T || p.T > kTileMaxSteps || p.ntx < 1 || p.nty < 1 || p.ntx > Lx / kLaneSites || p.nty > Ly ||
        !sites_per_lane_ok(p.S, f64) || (W / p.S) * H > p.threads || p.threads > kTileMaxThreads ||
        p.threads % kWave != 0 || lds > kTileMaxLds || (W != Lx && (W - wmax) / 2 > Lx) || (H != Ly && T > Ly))
        throw Error(-5, "tile launch: shape not supported");
    return lds;
}

template <typename R>
void launch_tile(const Lat<R>& v, const R* th_in, const R* u_in, R* th_out, R* u_out, const TilePlan& p, int T,
                 uint64_t k, hipStream_t s) {
    const size_t lds = tile_check(v.Lx, v.Ly, sizeof(R) == 8, p, T, 4);
    const TileIO<R> io{th_in, u_in, th_out, u_out};
    if constexpr (sizeof(R) == 4) {
        if (v.model == kModelSI) {
            if (v.fact) launch_tile_m<R, kModelSI, true, kTilePlain>(v, io, p, T, lds, k, s);
            else launch_tile_m<R, kModelSI, false, kTilePlain>(v, io, p, T, lds, k, s);
        } else {
            if (v.fact) launch_tile_m<R, kModelXY, true, kTilePlain>(v, io, p, T, lds, k, s);
            else launch_tile_m<R, kModelXY, false, kTilePlain>(v, io, p, T, lds, k, s);
        }
    } else {
        if (v.model == kModelSI) launch_tile_m<R, kModelSI, false, kTilePlain>(v, io, p, T, lds, k, s);
        else launch_tile_m<R, kModelXY, false, kTilePlain>(v, io, p, T, lds, k, s);
    }
}

template <typename R, int KIND>
static void launch_tile_xy(const Lat<R>& v, const TileIO<R>& io, const TilePlan& p, int T, uint64_t k, hipStream_t s) {
    const size_t lds = tile_check(v.Lx, v.Ly, sizeof(R) == 8, p, T, 4);
    if (v.model != kModelXY) throw Error(-5, "tile launch: XY lattices only");
    if constexpr (sizeof(R) == 4) {
        if (v.fact) launch_tile_m<R, kModelXY, true, KIND>(v, io, p, T, lds, k, s);
        else launch_tile_m<R, kModelXY, false, KIND>(v, io, p, T, lds, k, s);
    } else {
        launch_tile_m<R, kModelXY, false, KIND>(v, io, p, T, lds, k, s);
    }
}

template <typename R>
void launch_tile_states(const Lat<R>& v, const R* th_in, const R* u_in, bool first, R* states, const TilePlan& p,
                        int T, uint64_t k, hipStream_t s) {
    TileIO<R> io{th_in, u_in, nullptr, nullptr};
    io.states = states;
    io.first = first ? 1 : 0;
    launch_tile_xy<R, kTileStates>(v, io, p, T, k, s);
}

template <typename R>
void launch_tile_order(const Lat<R>& v, const R* th_in, const R* u_in, R* th_out, R* u_out, double* order,
                       const TilePlan& p, int T, uint64_t k, hipStream_t s) {
    TileIO<R> io{th_in, u_in, th_out, u_out};
    io.order = order;
    launch_tile_xy<R, kTileOrder>(v, io, p, T, k, s);
}

// One workgroup per step: the sum of its n partials (strided per thread, then
// a fixed tree) over N into out[6 step + 2].
__global__ __launch_bounds__(256) void k_tile_order_sum(const double* __restrict__ order, int n, double N,
                                                        double* __restrict__ out) {
    __shared__ double red[4];
    const double* p = order + (size_t)blockIdx.x * n;
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) acc += p[i];
    acc = wave_sum1(acc);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[6 * (size_t)blockIdx.x + 2] = ((red[0] + red[1]) + (red[2] + red[3])) / N;
}

void load_tile_kernels() {
    hipFuncAttributes a;
    check_hip(hipFuncGetAttributes(&a, reinterpret_cast<const void*>(k_tile_order_sum)), "hipFuncGetAttributes");
}

void launch_tile_order_sum(const double* order, int n, double N, double* out, int steps, hipStream_t s) {
    if (steps <= 0) return;
    k_tile_order_sum<<<steps, 256, 0, s>>>(order, n, N, out);
    check_hip(hipGetLastError(), "order-parameter sum launch");
}

template void launch_tile_states<float>(const Lat<float>&, const float*, const float*, bool, float*, const TilePlan&,
                                        int, uint64_t, hipStream_t);
template void launch_tile_states<double>(const Lat<double>&, const double*, const double*, bool, double*,
                                         const TilePlan&, int, uint64_t, hipStream_t);
template void launch_tile_order<float>(const Lat<float>&, const float*, const float*, float*, float*, double*,
                                       const TilePlan&, int, uint64_t, hipStream_t);
template void launch_tile_order<double>(const Lat<double>&, const double*, const double*, double*, double*, double*,
                                        const TilePlan&, int, uint64_t, hipStream_t);
template void launch_tile<float>(const Lat<float>&, const float*, const float*, float*, float*, const TilePlan&, int,
                                 uint64_t, hipStream_t);
template void launch_tile<double>(const Lat<double>&, const double*, const double*, double*, double*, const TilePlan&,
                                  int, uint64_t, hipStream_t);

template void launch_ensemble_tile<float>(const Lat<float>*, const TileTask*, int, const TilePlan&, size_t, int, int,
                                          int, uint64_t, const float*, float*, const uint64_t*, uint64_t,
                                          hipStream_t);
template void launch_ensemble_tile<double>(const Lat<double>*, const TileTask*, int, const TilePlan&, size_t, int,
                                           int, int, uint64_t, const double*, double*, const uint64_t*, uint64_t,
                                           hipStream_t);

}  // namespace xyl
