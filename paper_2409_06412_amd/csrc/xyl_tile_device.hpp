// Device side of the tile kernels: a workgroup's region and a lane's place in
// it (xyl_tile.hip, xyl_adjoint.hip).
#pragma once
#include "xyl_device.hpp"
#include "xyl_tile.hpp"

namespace xyl {

struct TileBox {
    int x0, y0, w, h;     // the sites a workgroup stores
};

template <typename R, int S>
__device__ __forceinline__ void tile_load(const R* p, R* o) {
    if constexpr (S == 4) {
        load4(p, o);
    } else if constexpr (S == 2) {
        typedef R V2 __attribute__((ext_vector_type(2)));
        const V2 d = *reinterpret_cast<const V2*>(p);
        o[0] = d.x;
        o[1] = d.y;
    } else {
        o[0] = *p;
    }
}
template <typename R, int S>
__device__ __forceinline__ void tile_store(R* p, const R* o) {
    if constexpr (S == 4) {
        store4(p, o);
    } else if constexpr (S == 2) {
        typedef R V2 __attribute__((ext_vector_type(2)));
        V2 d;
        d.x = o[0];
        d.y = o[1];
        *reinterpret_cast<V2*>(p) = d;
    } else {
        *p = o[0];
    }
}

// The value of lane J of the lane's group of P lanes (P = 2 or 4, a Philox
// block's lanes), by DPP.
template <int P, int J, typename R>
__device__ __forceinline__ R group_lane(R x) {
    constexpr int ctrl = P == 4 ? J * 0x55 : (J | (J << 2) | ((2 + J) << 4) | ((2 + J) << 6));
    if constexpr (sizeof(R) == 4)
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, 0xF, 0xF, false));
    else
        return dpp_f64<ctrl>(x);
}

// Tile (tx, ty) of ntx x nty about equal ones, whole quads wide.
__host__ __device__ __forceinline__ TileBox tile_box(int tx, int ty, int ntx, int nty, int Lx, int Ly) {
    constexpr int S = kLaneSites;
    const int nqx = Lx / S;
    TileBox b;
    const int xa = (int)((long)tx * nqx / ntx), xb = (int)((long)(tx + 1) * nqx / ntx);
    const int ya = (int)((long)ty * Ly / nty), yb = (int)((long)(ty + 1) * Ly / nty);
    b.x0 = xa * S;
    b.w = (xb - xa) * S;
    b.y0 = ya;
    b.h = yb - ya;
    return b;
}

// A lane's group of S sites in the region of box b for T steps (W x H sites,
// row-major; no halo along an axis the box spans whole): lane tid has group
// tid.  Lanes past the region's end repeat its last Philox block and never
// store or become valid.
template <int S>
struct TileLane {
    bool px, py;               // the region is periodic along the axis
    int W, H;
    bool in, own;              // in the region; in the box
    int y, xq;                 // row, group in the row
    int gx, gy;                // the first site on the lattice
    uint32_t off, q;           // its index, its Philox block
    int part;                  // the lane's place in the block (S < 4)
    // table slots of the group and of its neighbours (the region's outer ring
    // of a non-periodic axis has none: its values are never used)
    int i0, iu, id, il, ir;
    bool edge_l, edge_r;       // the left / right neighbour is not in the adjacent lane
    int dist;                  // steps the group's sites stay valid for: the
                               // distance of its innermost site from the edge

    __device__ __forceinline__ TileLane(int Lx, int Ly, const TileBox& b, int T) {
        constexpr int P = 4 / S;
        px = b.w == Lx;
        py = b.h == Ly;
        const int hx = px ? 0 : (T + 3) / 4 * 4, hy = py ? 0 : T;
        W = b.w + 2 * hx;
        H = b.h + 2 * hy;
        const int Wq = W / S, nq = Wq * H;
        const int tid = threadIdx.x, lane = tid & (kWave - 1);
        in = tid < nq;
        const int g = in ? tid : nq - P + (tid & (P - 1));
        y = g / Wq;
        xq = g - y * Wq;
        gy = b.y0 - hy + y;
        gx = b.x0 - hx + S * xq;
        gy = gy < 0 ? gy + Ly : (gy >= Ly ? gy - Ly : gy);
        gx = gx < 0 ? gx + Lx : (gx >= Lx ? gx - Lx : gx);
        off = (uint32_t)gy * (uint32_t)Lx + (uint32_t)gx;
        q = off >> 2;
        part = tid & (P - 1);
        i0 = S * g;
        iu = y == 0 ? (py ? i0 + (H - 1) * W : i0) : i0 - W;
        id = y == H - 1 ? (py ? i0 - (H - 1) * W : i0) : i0 + W;
        il = xq == 0 ? (px ? i0 + W - 1 : i0) : i0 - 1;
        ir = xq == Wq - 1 ? (px ? i0 + S - W : i0) : i0 + S;
        edge_l = lane == 0 || (xq == 0 && px);
        edge_r = lane == kWave - 1 || (xq == Wq - 1 && px);
        dist = T;
        if (!py) dist = min(dist, min(y, H - 1 - y));
        if (!px) dist = min(dist, min(S * xq + S - 1, W - 1 - S * xq));
        if (!in) dist = 0;
        own = in && y >= hy && y < hy + b.h && S * xq >= hx && S * xq < hx + b.w;
    }
};

// The draws a lane takes per block's turn: where the lanes of a block share
// it, those of one step for the whole block (d[4]), else its own pair.
template <typename R, int S>
constexpr bool tile_own_pair() { return sizeof(R) == 8 && S == 2; }
template <typename R, int S>
constexpr int tile_share() { return tile_own_pair<R, S>() ? 1 : 4 / S; }

// The lane's S draws of sub-step J of its block's turn.
template <int S, int P, int J, typename R>
__device__ __forceinline__ void tile_draws(const R d[4], int part, R n[S]) {
#pragma unroll
    for (int e = 0; e < S; ++e) {
        if constexpr (P == 1) {
            n[e] = d[e];
        } else {
            n[e] = group_lane<P, J>(d[e]);
#pragma unroll
            for (int l = 1; l < P; ++l) {
                const R o = group_lane<P, J>(d[l * S + e]);
                n[e] = part == l ? o : n[e];
            }
        }
    }
}

// Sum of an FP64 value over the 64 lanes of a wave, in a fixed pattern.
__device__ __forceinline__ double wave_sum1(double x) {
    x += dpp_f64<kDppQuadXor1>(x);
    x += dpp_f64<kDppQuadXor2>(x);
    x += dpp_f64<kDppRowHalfMirror>(x);
    x += dpp_f64<kDppRowRor8>(x);
    double y = x;
    swap16_f64(x, y);
    x += y;
    y = x;
    swap32_f64(x, y);
    return x + y;
}

}  // namespace xyl
