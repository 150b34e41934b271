// Three BBK steps per pass for large FP32 lattices: single waves march down
// column tiles with all state in registers.
//
// What bounded the two-step pass there: 16 bytes a site for two steps, a
// barrier per row, and rows that fill a workgroup's waves badly (3000 sites: 12
// waves of a CU's 16).  Here a wave owns up to 62 quads of columns and a strip
// of rows, and nothing outside the wave is shared: left and right rotors come
// from the adjacent lanes by DPP, upper and lower ones are the lane's own of
// the rows before, and a quad on each side (the outer lanes, not stored) covers
// the three sites per side that go stale.  No LDS, no barrier.  Stage j of an
// iteration takes the step k + j of the row j behind the newest one, so a pass
// reads and writes every row once for three steps.  The per-site arithmetic is
// the shared rotor / noise4_kick / site_force / site_update: states equal
// single steps bit for bit.
//
// Two waves per SIMD (200 registers): independent stages keep the VALU busy
// even with one.  Three waves (168 registers) spill, four stages need 242 and
// gain nothing (a wave's two ends recompute D - 1 rows each on average).
// Bound by VALU issue (83% of the slots at 4096^2), 0.295 us per wave of a
// SIMD, row and step, two halo rows included; the halo takes 10 to 20%.
// Measured, us per step, with two steps per pass and with this pass (tiles
// where those were the next best): 2048^2 9.4 and 8.3, 2564 x 2503 14.3 and
// 10.8, 3000^2 17.3 and 14.1, 3584 x 3000 17.7 and 15.4, 4096^2 24.6 and 22.5,
// 5000 x 2001 20.4 and 14.6, 6144^2 70.8 and 52.7, 8192^2 114.9 and 88.6.
#include "xyl_march.hpp"

#include <algorithm>
#include <type_traits>

#include "xyl_device.hpp"

namespace xyl {

// Rows [y0, y1) of the columns [c0, c0 + w) (multiples of 4, w up to 248),
// downwards (d = 1) or upwards (the force is symmetric in the y-neighbours),
// three steps from step k.
template <int M>
__device__ __forceinline__ void march_strip(const Lat<float>& v, const MarchBuffers& B, int c0, int w, int y0, int y1,
                                            int d, uint64_t k) {
    using R = float;
    constexpr int D = kMarchSteps;
    static_assert(D == 3, "the iterations below are written out for three stages");
    const int Lx = v.Lx, Ly = v.Ly;
    const int lane = threadIdx.x & (kWave - 1);
    const int last = w / kLaneSites + 1;                       // the tile's quads and one on each side
    const int xl = c0 + kLaneSites * (min(lane, last) - 1);
    const int gx = xl < 0 ? xl + Lx : (xl >= Lx ? xl - Lx : xl);
    const bool own = lane >= 1 && lane < last;
    const uint32_t qx = (uint32_t)gx >> 2, qrow = (uint32_t)Lx >> 2, gxb = (uint32_t)gx * 4u;
    R hs[D];
    bool fresh[D];
#pragma unroll
    for (int j = 0; j < D; ++j) {
        hs[j] = noise_coeff<R, true>(v, k + (uint64_t)j);
        fresh[j] = k + (uint64_t)j == v.fresh_k;
    }
    const int n = y1 - y0, nit = n + 2 * D;
    const int ys = d > 0 ? y0 - D : y1 - 1 + D;
    auto rowof = [&](int i) {
        int y = ys + d * i;
        y += y < 0 ? Ly : 0;
        return y >= Ly ? y - Ly : y;
    };
    R s[D][3][4], c[D][3][4], t[D][2][4], u[D][2][4];
    auto load = [&](int i, int b) {
        const int y = rowof(i);
        load4(at_byte(row_start(B.th_in, y, Lx), gxb), t[0][b]);
        load4(at_byte(row_start(B.u_in, y, Lx), gxb), u[0][b]);
    };
    // Iteration `it` (PH = it mod 6) with the first NS stages: row it comes in,
    // stage j works on row it - 1 - j.  s, c[j][i mod 3] hold the rotors of row
    // i at step k + j, t, u[j][i mod 2] its angles and velocities.
    auto iterate = [&](auto ph, auto ns, int it) {
        constexpr int PH = decltype(ph)::value, NS = decltype(ns)::value;
        constexpr int n3 = PH % 3, c3 = (PH + 2) % 3, p3 = (PH + 1) % 3, nb = PH % 2, cb = nb ^ 1;
#pragma unroll
        for (int e = 0; e < 4; ++e) rotor<R, M>(t[0][nb][e], s[0][n3][e], c[0][n3][e]);
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const int y = rowof(it - 1 - j);
            R z[4];
            noise4_kick<R>((uint32_t)y * qrow + qx, v.replica, k + (uint64_t)j, v.seed_lo, v.seed_hi, hs[j], z,
                           noise_u2<R, true>(v));
            const R (&sc)[4] = s[j][c3];
            const R (&cc)[4] = c[j][c3];
            const R sL = from_lane_below(sc[3]), cL = from_lane_below(cc[3]);
            const R sR = from_lane_above(sc[0]), cR = from_lane_above(cc[0]);
            R to[4], uo[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const R sxm = e == 0 ? sL : sc[e - 1], cxm = e == 0 ? cL : cc[e - 1];
                const R sxp = e == 3 ? sR : sc[e + 1], cxp = e == 3 ? cR : cc[e + 1];
                const R f = site_force<R, M, true>(v, sc[e], cc[e], sxm, cxm, sxp, cxp, s[j][p3][e], c[j][p3][e],
                                                   s[j][n3][e], c[j][n3][e], t[j][cb][e], z[e]);
                R w2;
                site_update<R, M, true>(v, f, u[j][cb][e], t[j][cb][e], z[e], hs[j], fresh[j], w2, uo[e], to[e]);
            }
            if (j == 0) load(min(it + 1, nit - 1), cb);      // the row of the next iteration
            if (j + 1 < D) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    t[j + 1][nb][e] = to[e];
                    u[j + 1][nb][e] = uo[e];
                    rotor<R, M>(to[e], s[j + 1][n3][e], c[j + 1][n3][e]);
                }
            } else if (own) {
                store4(at_byte(row_start(B.th_out, y, Lx), gxb), to);
                store4(at_byte(row_start(B.u_out, y, Lx), gxb), uo);
            }
        }
        if constexpr (NS == 0) load(it + 1, cb);
    };
    using std::integral_constant;
#define XYL_IT(PH, NS, IT) iterate(integral_constant<int, PH>{}, integral_constant<int, NS>{}, IT)
    load(0, 0);
    // (rows here count from the first one loaded, D before the strip's first
    // one; stage j has its three rows from iteration 2 j + 2 on and row it - 1 -
    // j is one of the strip's or of its halo from then on)
    XYL_IT(0, 0, 0);
    XYL_IT(1, 0, 1);
    XYL_IT(2, 1, 2);
    XYL_IT(3, 1, 3);
    XYL_IT(4, 2, 4);
    XYL_IT(5, 2, 5);
    for (int it = 6;;) {
        XYL_IT(0, D, it);
        if (++it == nit) break;
        XYL_IT(1, D, it);
        if (++it == nit) break;
        XYL_IT(2, D, it);
        if (++it == nit) break;
        XYL_IT(3, D, it);
        if (++it == nit) break;
        XYL_IT(4, D, it);
        if (++it == nit) break;
        XYL_IT(5, D, it);
        if (++it == nit) break;
    }
#undef XYL_IT
}

// Wave b of the launch takes column tile b % ntx of strip b / ntx; strips run
// down and up in turn, so that two neighbours read their common halo rows at
// the same end of their passes.
template <int M>
__global__ __launch_bounds__(256, 2) void k_march(Lat<float> v, MarchBuffers B, int ntx, int nstrips, uint64_t k) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int task = xcd_contiguous_block(blockIdx.x, gridDim.x) * (256 / kWave) + wave;
    if (task >= ntx * nstrips) return;
    const int strip = task / ntx, tx = task - strip * ntx;
    const int nq = v.Lx / kLaneSites;
    const int xa = (int)((long)tx * nq / ntx), xb = (int)((long)(tx + 1) * nq / ntx);
    const int y0 = (int)((long)strip * v.Ly / nstrips), y1 = (int)((long)(strip + 1) * v.Ly / nstrips);
    march_strip<M>(v, B, xa * kLaneSites, (xb - xa) * kLaneSites, y0, y1, (strip & 1) ? -1 : 1, k);
}

// Two waves per SIMD in one round, or four in two where strips stay taller than
// 40 rows (us per step in one round and in two: 16384 x 4096 90.1 and 88.8,
// 8192^2 89.1 and 88.6; 4096^2, with strips of 18 rows, 22.5 and 23.8).
// The time is a fit to passes from 1100^2 (5.2 us per step) over 1604^2 (6.6),
// 2048^2 (8.3), 3000^2 (14.1) and 4096^2 (22.5) to 8192^2 (88.6), within 10%.
MarchPlan march_plan(int Lx, int Ly, int cus) {
    MarchPlan p;
    const int nq = Lx / kLaneSites, most = kWave - 2;
    p.ntx = (nq + most - 1) / most;
    p.strips = std::max(1, 8 * cus / p.ntx);
    if (Ly / (2 * p.strips) >= 40) p.strips *= 2;
    p.strips = std::min(p.strips, std::max(1, Ly / 4));
    const int rows = (Ly + p.strips - 1) / p.strips;
    const int per_simd = (int)(((long)p.ntx * p.strips + 4 * cus - 1) / (4 * cus));
    p.us = 1.7 + 0.295 * per_simd * (rows + kMarchSteps - 1);
    return p;
}

void load_march_kernels() {
    hipFuncAttributes a;
    check_hip(hipFuncGetAttributes(&a, reinterpret_cast<const void*>(k_march<kModelXY>)), "hipFuncGetAttributes");
}

void launch_march(const Lat<float>& v, const MarchBuffers& b, const MarchPlan& p, uint64_t k, hipStream_t s) {
    if (v.Lx % kLaneSites != 0 || v.Ly < kMarchSteps || p.ntx < 1 || p.strips < 1 || p.strips > v.Ly ||
        (v.Lx / kLaneSites + p.ntx - 1) / p.ntx > kWave - 2 || !v.fact)
        throw Error(-5, "march plan does not fit the lattice");
    const long waves = (long)p.ntx * p.strips;
    const unsigned blocks = (unsigned)((waves + 3) / 4);
    if (v.model == kModelSI) k_march<kModelSI><<<blocks, 256, 0, s>>>(v, b, p.ntx, p.strips, v.k_base + k);
    else k_march<kModelXY><<<blocks, 256, 0, s>>>(v, b, p.ntx, p.strips, v.k_base + k);
    check_hip(hipGetLastError(), "march kernel launch");
}

}  // namespace xyl
