// Measurements outside the step: the staggered rotor correlation function and
// the frozen-domain labelling.
#include <algorithm>

#include "xyl_device.hpp"
#include "xyl_domains.hpp"
#include "xyl_obs.hpp"
#include "xyl_sincos.hpp"

namespace xyl {

// --------------------------------------------------------- correlation
// C(r) = (1/N) sum_i eps_i eps_j cos(q (th_i - th_j)), j = i + r along one
// axis (App. C, two-point function of the rotors averaged over the lattice;
// q = 1 for XY, 2 for the Si mapping).  One workgroup per line (row for axis
// 0, column for axis 1) stages the line's staggered rotors (eps cos q th,
// eps sin q th) in LDS in FP64; thread r sums the line's products in index
// order.  A second pass sums the lines in order.
template <typename R>
__global__ __launch_bounds__(256) void k_corr_lines(const R* __restrict__ th, int Lx, int Ly, int sx, int sy,
                                                    double q, int axis, int rmax, double* __restrict__ part) {
    extern __shared__ double lds[];
    const int line = blockIdx.x;
    const int L = axis == 0 ? Lx : Ly;
    double* cs = lds;
    double* sn = lds + L;
    for (int p = threadIdx.x; p < L; p += blockDim.x) {
        const int x = axis == 0 ? p : line;
        const int y = axis == 0 ? line : p;
        const double t = (double)th[(size_t)y * Lx + x];
        const double e = (((x * sx) + (y * sy)) & 1) ? -1.0 : 1.0;
        double s, c;
        sincos(q * t, &s, &c);
        cs[p] = e * c;
        sn[p] = e * s;
    }
    __syncthreads();
    for (int r = threadIdx.x; r <= rmax; r += blockDim.x) {
        double acc = 0.0;
        for (int p = 0; p < L; ++p) {
            int q = p + r;
            if (q >= L) q -= L;
            acc += cs[p] * cs[q] + sn[p] * sn[q];
        }
        part[(size_t)line * (rmax + 1) + r] = acc;
    }
}

// Sum of the rows part[l][0..rmax], l < nrows, over l, divided by N: a
// workgroup takes 16 columns and its 16 thread rows every 16th row (128-B
// reads), then a fixed tree adds the 16 partial sums of a column.  One launch
// of 4 us for 512 rows of 1025 (before: chunk sums and their sum, two of 5).
__global__ __launch_bounds__(256) void k_row_sum(const double* __restrict__ part, int nrows, int rmax, double N,
                                                 double* __restrict__ out) {
    __shared__ double red[16][17];
    const int c = threadIdx.x & 15, g = threadIdx.x >> 4;
    const int r = blockIdx.x * 16 + c;
    double acc = 0.0;
    if (r <= rmax) {
#pragma unroll 8
        for (int l = g; l < nrows; l += 16) acc += part[(size_t)l * (rmax + 1) + r];
    }
    red[g][c] = acc;
    __syncthreads();
    for (int w = 8; w >= 1; w >>= 1) {
        if (g < w) red[g][c] += red[g + w][c];
        __syncthreads();
    }
    if (g == 0 && r <= rmax) out[r] = red[0][c] / N;
}

static void launch_row_sum(const double* part, int nrows, int rmax, double N, double* out, hipStream_t s) {
    k_row_sum<<<rmax / 16 + 1, 256, 0, s>>>(part, nrows, rmax, N, out);
    check_hip(hipGetLastError(), "row sum launch");
}

// Sums carried as an FP64 number and what its roundings left out.
__device__ __forceinline__ void two_add(double2& a, double b) {
    const double s = a.x + b, t = s - a.x;
    a.y += (a.x - (s - t)) + (b - t);
    a.x = s;
}

// C(r) from the structure factor of an axis that goes through the transform
// (App. C: C and S are a Fourier pair along the axis): C(r) = (1/L) sum_{k<L}
// S(k) cos(2 pi k r / L) with S(L - k) = S(k), i.e. (1/L) [S(0) + (even L)
// (-1)^r S(L/2) + 2 sum_{0<k<L/2} S(k) cos(2 pi k r / L)].  One workgroup per r
// sums in a fixed order (strided partial sums, then a fixed tree); cos from the
// twiddle table tw.  Products and sums keep their roundings (the errors of the
// S(k) average out, those of a plain sum left C(0) an ulp beside 1).
__global__ __launch_bounds__(256) void k_corr_from_sf(const double* __restrict__ S, const double2* __restrict__ tw,
                                                      int L, double* __restrict__ out) {
    __shared__ double2 red[256];
    const int r = blockIdx.x;
    const int h = (L + 1) / 2;
    double2 acc = make_double2(0.0, 0.0);
    for (int k = 1 + (int)threadIdx.x; k < h; k += blockDim.x) {
        const double c = tw[(unsigned)(k * r) % (unsigned)L].x, p = S[k] * c;
        two_add(acc, p);
        acc.y += fma(S[k], c, -p);
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            double2 a = red[threadIdx.x];
            const double2 b = red[threadIdx.x + w];
            two_add(a, b.x);
            a.y += b.y;
            red[threadIdx.x] = a;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        double2 a = make_double2(2.0 * red[0].x, 2.0 * red[0].y);
        two_add(a, S[0]);
        if (L % 2 == 0) two_add(a, (r & 1) ? -S[h] : S[h]);
        out[r] = (a.x + a.y) / (double)L;
    }
}

template <typename R>
void launch_correlation(const R* th, int Lx, int Ly, int sx, int sy, int model, int axis, int rmax, const double* tw,
                        double* scratch, double* out, hipStream_t s) {
    const int nlines = axis == 0 ? Ly : Lx;
    const int L = axis == 0 ? Lx : Ly;
    if (sf_smooth(L)) {
        double* S = scratch + structure_factor_scratch(Lx, Ly, axis, L / 2);
        launch_structure_factor<R>(th, Lx, Ly, sx, sy, model, axis, L / 2, tw, scratch, S, s);
        k_corr_from_sf<<<rmax + 1, 256, 0, s>>>(S, reinterpret_cast<const double2*>(tw), L, out);
        check_hip(hipGetLastError(), "correlation kernel launch");
        return;
    }
    const size_t lds = 2 * sizeof(double) * (size_t)L;
    k_corr_lines<R><<<nlines, 256, lds, s>>>(th, Lx, Ly, sx, sy, model == kModelSI ? 2.0 : 1.0, axis, rmax, scratch);
    check_hip(hipGetLastError(), "correlation kernel launch");
    launch_row_sum(scratch, nlines, rmax, (double)Lx * (double)Ly, out, s);
}

// ------------------------------------------------- structure factor
// S_delta(k) = (1/N) sum over lines along delta of sum_kappa |s~^kappa_k|^2,
// s~^kappa_k = sum_r s^kappa_r exp(-2 pi i k r / L) (App. C, Eq.
// S-as-lattice-FT: the transform of C_delta(r), Eq. FT-Corr-delta).  Each
// line's two real rotor components are packed as one complex sequence
// z = eps (cos q th + i sin q th), whose transform Z gives
// sum_kappa |s~^kappa_k|^2 = (|Z_k|^2 + |Z_{L-k}|^2) / 2.
// Lengths with no prime factor above 7 go through k_sf_lines (below), others
// through the direct sum k_sf_direct on the rotors z, written line-major first
// (rows as they are; columns through a 32 x 32 LDS transpose).  Either way the
// lines' spectra are added by launch_row_sum.
template <typename R>
__global__ __launch_bounds__(256) void k_rotor_rows(const R* __restrict__ th, int Lx, int Ly, int sx, int sy,
                                                    double q, double2* __restrict__ z) {
    const size_t N = (size_t)Lx * Ly;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (size_t)gridDim.x * blockDim.x) {
        const int y = (int)(i / (size_t)Lx), x = (int)(i - (size_t)y * Lx);
        const double e = (((x * sx) + (y * sy)) & 1) ? -1.0 : 1.0;
        double sn, cs;
        sincos(q * (double)th[i], &sn, &cs);
        z[i] = make_double2(e * cs, e * sn);
    }
}

template <typename R>
__global__ __launch_bounds__(256) void k_rotor_cols(const R* __restrict__ th, int Lx, int Ly, int sx, int sy,
                                                    double q, double2* __restrict__ z) {
    __shared__ double2 tile[32][33];
    const int x0 = blockIdx.x * 32, y0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int x = x0 + tx, y = y0 + ty + 8 * j;
        if (x < Lx && y < Ly) {
            const double e = (((x * sx) + (y * sy)) & 1) ? -1.0 : 1.0;
            double sn, cs;
            sincos(q * (double)th[(size_t)y * Lx + x], &sn, &cs);
            tile[ty + 8 * j][tx] = make_double2(e * cs, e * sn);
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int x = x0 + ty + 8 * j, y = y0 + tx;
        if (x < Lx && y < Ly) z[(size_t)x * Ly + y] = tile[tx][ty + 8 * j];
    }
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// tw[m] = exp(-2 pi i m / L), m < L: the twiddle table of one transform length
__global__ void k_sf_twiddles(double2* __restrict__ tw, int L) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m < L) {
        double sn, cs;
        sincospi(2.0 * (double)m / (double)L, &sn, &cs);
        tw[m] = make_double2(cs, -sn);
    }
}

// LDS slot of point i of a line: one 16-B pad after every 16 points, so that
// the strided stores of the early passes spread over the banks.
__host__ __device__ __forceinline__ int sf_slot(int i) { return i + (i >> 4); }
__host__ __device__ __forceinline__ int sf_pitch(int L) { return sf_slot(L) + 1; }
constexpr int kSfPoints = 4096;    // points of the lines that a workgroup transforms at a time
constexpr int kSfThreads = 512;

constexpr int bit_reverse_c(int q, int bits) {
    int r = 0;
    for (int b = 0; b < bits; ++b) r |= ((q >> b) & 1) << (bits - 1 - b);
    return r;
}
constexpr int log2_c(int n) { return n <= 1 ? 0 : 1 + log2_c(n / 2); }

// v exp(-2 pi i m / 8), m < 4
__device__ __forceinline__ double2 turn8(double2 v, int m) {
    constexpr double h = 0.70710678118654752440;
    if (m == 1) return make_double2(h * (v.x + v.y), h * (v.y - v.x));
    if (m == 2) return make_double2(v.y, -v.x);
    if (m == 3) return make_double2(h * (v.y - v.x), -h * (v.x + v.y));
    return v;
}

// R-point DFT in registers, natural order in and out: R = 3, 5, 7 by the
// definition (w_R^m = tw[m L / R]); 2, 4, 8 by radix-2 decimation in
// frequency (its result comes out bit-reversed and is read back through the
// bit reversal).
template <int R>
__device__ __forceinline__ void dft_regs(double2 v[R], const double2* __restrict__ tw, int L) {
    double2 t[R];
    if constexpr (R == 3 || R == 5 || R == 7) {
        // V_q and V_{R-q} = A +- i B with A = v_0 + sum_r (v_r + v_{R-r}) Re w^(q r),
        // B = sum_r (v_r - v_{R-r}) Im w^(q r), r = 1 .. (R-1)/2
        constexpr int H = (R - 1) / 2;
        t[0] = v[0];
#pragma unroll
        for (int r = 1; r <= H; ++r) {
            const double2 a = cadd(v[r], v[R - r]), b = csub(v[r], v[R - r]);
            t[0] = cadd(t[0], a);
            v[r] = a;
            v[R - r] = b;
        }
#pragma unroll
        for (int q = 1; q <= H; ++q) {
            double2 A = v[0], B = make_double2(0.0, 0.0);
#pragma unroll
            for (int r = 1; r <= H; ++r) {
                const double2 w = tw[(q * r) % R * (L / R)];
                A.x += v[r].x * w.x;
                A.y += v[r].y * w.x;
                B.x += v[R - r].x * w.y;
                B.y += v[R - r].y * w.y;
            }
            t[q] = make_double2(A.x - B.y, A.y + B.x);
            t[R - q] = make_double2(A.x + B.y, A.y - B.x);
        }
    } else {
#pragma unroll
        for (int span = R / 2; span >= 1; span >>= 1) {
#pragma unroll
            for (int i0 = 0; i0 < R; i0 += 2 * span) {
#pragma unroll
                for (int j = 0; j < span; ++j) {
                    const double2 a = v[i0 + j], b = v[i0 + j + span];
                    v[i0 + j] = cadd(a, b);
                    v[i0 + j + span] = turn8(csub(a, b), j * (4 / span));
                }
            }
        }
#pragma unroll
        for (int q = 0; q < R; ++q) t[q] = v[bit_reverse_c(q, log2_c(R))];
    }
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = t[q];
}

// t / d for t < 2^20 with inv = 1 / d good to a few ulp: (t + 1/2) / d is half
// of 1 / d or more away from a whole number, its error below 2^-21 of itself.
__device__ __forceinline__ int small_div(int t, float inv) { return (int)(((float)t + 0.5f) * inv); }

// One Stockham pass of radix R over nl lines of L points held in LDS, with Ns
// the product of the radices of the passes before it: group j (of G = L / R)
// of a line takes the points j + r G, multiplies point r by w^(r (j mod Ns))
// with w = exp(-2 pi i / (Ns R)), takes their R-point DFT and stores output q
// at (j - j mod Ns) R + j mod Ns + q Ns.  After the last pass a line holds its
// transform in natural order.  Every group of the pass is loaded before any is
// stored, so the pass runs in place; a thread has up to K groups.
template <int R>
__device__ __forceinline__ void sf_pass(double2* buf, const double2* __restrict__ tw, int L, int nl, int Ns) {
    constexpr int K = (kSfPoints / R + kSfThreads - 1) / kSfThreads;
    const int G = L / R, total = nl * G, pitch = sf_pitch(L);
    const float inv_G = 1.0f / (float)G, inv_Ns = 1.0f / (float)Ns;
    double2 v[K][R];
    int base[K], out[K];
#pragma unroll
    for (int g = 0; g < K; ++g) {
        const int t = (int)threadIdx.x + g * kSfThreads;
        if (t < total) {
            const int line = small_div(t, inv_G), j = t - line * G, k = j - small_div(j, inv_Ns) * Ns;
            out[g] = (j - k) * R + k;
            double2* b = buf + line * pitch;
            base[g] = line * pitch;
#pragma unroll
            for (int r = 0; r < R; ++r) v[g][r] = b[sf_slot(j + r * G)];
            if (Ns > 1) {
                // w^r from the table, for eight points w and w^2 (the others are
                // products of up to four of them).  Powers multiplied up from w
                // made the spectrum of 384 points 2.3e-16 wrong, so 1.2e-16;
                // 1.5e-16 by the direct sum.  w^4 from the table too gains
                // nothing and takes 2% longer at 4096^2.
                const int step = k * (L / (Ns * R));
                if constexpr (R == 8) {
                    const double2 w1 = tw[step], w2 = tw[2 * step];
                    v[g][1] = cmul(v[g][1], w1);
                    v[g][2] = cmul(v[g][2], w2);
                    const double2 w4 = cmul(w2, w2);
                    v[g][5] = cmul(v[g][5], cmul(w4, w1));
                    v[g][6] = cmul(v[g][6], cmul(w4, w2));
                    const double2 w3 = cmul(w1, w2);
                    v[g][3] = cmul(v[g][3], w3);
                    v[g][4] = cmul(v[g][4], w4);
                    v[g][7] = cmul(v[g][7], cmul(w4, w3));
                } else {
#pragma unroll
                    for (int r = 1; r < R; ++r) v[g][r] = cmul(v[g][r], tw[r * step]);
                }
            }
            dft_regs<R>(v[g], tw, L);
        }
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < K; ++g) {
        const int t = (int)threadIdx.x + g * kSfThreads;
        if (t < total) {
#pragma unroll
            for (int q = 0; q < R; ++q) buf[base[g] + sf_slot(out[g] + q * Ns)] = v[g][q];
        }
    }
    __syncthreads();
}

// The spectra of lines of L points (at most 4096, no prime factor above 7),
// straight from the angles: a workgroup takes nlb lines at a time, as many as
// kSfPoints points hold, transforms them in LDS (Stockham passes of radix 8
// and what is left of L), and adds their |.|^2 over all its batches in
// registers, thread t those of k = t mod (kmax + 1), .. and the lines of
// sub-row t / (kmax + 1); one row of sums per workgroup and sub-row.
// Bound by the FP64 sine, cosine and butterflies (some 120 operations a site)
// and the LDS passes, not by the 4 bytes a site it reads.  2048^2, one axis,
// all k: 38 us rows, 41 us columns, then 5 us for the sum (before: a line per
// workgroup with the general sincos, 61 us, columns through a transposed field
// of rotors, 18 + 32 us, and every line's spectrum written and summed, 10 us;
// 384 x 360, which then took the direct sum: 10 us against 32).
template <typename R, int AXIS, bool SEVEN>
__global__ __launch_bounds__(kSfThreads, SEVEN ? 2 : 4)
void k_sf_lines(const R* __restrict__ th, int Lx, int sx, int sy, double q, const double2* __restrict__ tw, int L,
                int nlines, int nlb, int kmax, int nsub, double* __restrict__ part) {
    extern __shared__ double2 sm[];
    constexpr int kAcc = (kSfPoints / 2 + 1 + kSfThreads - 1) / kSfThreads;
    double acc[kAcc];
#pragma unroll
    for (int a = 0; a < kAcc; ++a) acc[a] = 0.0;
    const int pitch = sf_pitch(L);
    const int nk = kmax + 1;
    const int sub = nsub > 1 ? (int)threadIdx.x / nk : 0;
    const int k0 = nsub > 1 ? (int)threadIdx.x - sub * nk : (int)threadIdx.x;
    // columns: the workgroups of an XCD (every eighth) take neighbouring lines,
    // which share cache lines
    const int lb = AXIS == 1 && gridDim.x % 8 == 0 ? (int)((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3))
                                                   : (int)blockIdx.x;
    for (int l0 = lb * nlb; l0 < nlines; l0 += (int)gridDim.x * nlb) {
        const int nl = min(nlb, nlines - l0);
        // the staggered rotors, all of a thread's angles in flight at once;
        // columns take the lines fastest across the threads, so that a row's
        // angles are read together
        constexpr int kPer = kSfPoints / kSfThreads;
        const int npt = nl * L;
        int d = AXIS == 0 ? L : nl;
        asm volatile("" : "+s"(d));   // opaque, as in the passes below
        const float inv_d = 1.0f / (float)d;
        R ang[kPer];
#pragma unroll
        for (int g = 0; g < kPer; ++g) {
            const int t = (int)threadIdx.x + g * kSfThreads;
            const int a = small_div(t, inv_d), b = t - a * d;
            if (t < npt) ang[g] = AXIS == 0 ? th[(size_t)l0 * Lx + t] : th[(size_t)a * Lx + l0 + b];
        }
        bool wild = false;
#pragma unroll
        for (int g = 0; g < kPer; ++g) {
            const int t = (int)threadIdx.x + g * kSfThreads;
            const int a = small_div(t, inv_d), b = t - a * d;
            if (t < npt) {
                const double x = q * (double)ang[g];
                double sn, cs;
                sincos_reduced(x, sn, cs);
                wild |= !sincos_reducible(x);
                const bool odd = AXIS == 0 ? (b * sx + (l0 + a) * sy) & 1 : ((l0 + b) * sx + a * sy) & 1;
                const int slot = AXIS == 0 ? a * pitch + sf_slot(b) : b * pitch + sf_slot(a);
                sm[slot] = odd ? make_double2(-cs, -sn) : make_double2(cs, sn);
            }
            if (g & 1) __builtin_amdgcn_sched_barrier(0);   // two at a time: more would spill
        }
        if (wild) {
            // angles that no stepping leaves (a caller's own state)
            for (int t = (int)threadIdx.x; t < npt; t += kSfThreads) {
                const int a = small_div(t, inv_d), b = t - a * d;
                const double x = q * (double)(AXIS == 0 ? th[(size_t)l0 * Lx + t] : th[(size_t)a * Lx + l0 + b]);
                if (sincos_reducible(x)) continue;
                const bool odd = AXIS == 0 ? (b * sx + (l0 + a) * sy) & 1 : ((l0 + b) * sx + a * sy) & 1;
                const int slot = AXIS == 0 ? a * pitch + sf_slot(b) : b * pitch + sf_slot(a);
                const double2 z = sincos_general(x);
                sm[slot] = odd ? make_double2(-z.x, -z.y) : z;
            }
        }
        __syncthreads();
        for (int Ns = 1; Ns < L;) {
            // opaque here: the index arithmetic of all the passes, hoisted out
            // of the loops, would spill
            int Lv = L;
            asm volatile("" : "+s"(Lv));
            const int left = Lv / Ns;
            if (left % 8 == 0) {
                sf_pass<8>(sm, tw, Lv, nl, Ns);
                Ns *= 8;
            } else if (left % 4 == 0) {
                sf_pass<4>(sm, tw, Lv, nl, Ns);
                Ns *= 4;
            } else if (left % 2 == 0) {
                sf_pass<2>(sm, tw, Lv, nl, Ns);
                Ns *= 2;
            } else if (left % 3 == 0) {
                sf_pass<3>(sm, tw, Lv, nl, Ns);
                Ns *= 3;
            } else if (left % 5 == 0) {
                sf_pass<5>(sm, tw, Lv, nl, Ns);
                Ns *= 5;
            } else if constexpr (SEVEN) {
                sf_pass<7>(sm, tw, Lv, nl, Ns);
                Ns *= 7;
            } else {
                break;   // not reached
            }
        }
        // sum_kappa |s~^kappa_k|^2 = (|Z_k|^2 + |Z_{L-k}|^2) / 2
        if (sub < nsub) {
#pragma unroll
            for (int a = 0; a < kAcc; ++a) {
                const int k = k0 + a * kSfThreads;
                if (k > kmax || (a && nsub > 1)) break;
                const int i = sf_slot(k), m = sf_slot(k ? L - k : 0);
                for (int l = sub; l < nl; l += nsub) {
                    const double2 x = sm[l * pitch + i], y = sm[l * pitch + m];
                    acc[a] += 0.5 * (x.x * x.x + x.y * x.y + y.x * y.x + y.y * y.y);
                }
            }
        }
        __syncthreads();
    }
    if (sub < nsub) {
        double* o = part + ((size_t)blockIdx.x * nsub + sub) * nk;
#pragma unroll
        for (int a = 0; a < kAcc; ++a) {
            const int k = k0 + a * kSfThreads;
            if (k > kmax || (a && nsub > 1)) break;
            o[k] = acc[a];
        }
    }
}

// Other lengths: the direct sum, one line per workgroup, with the full-circle
// twiddle table in LDS.
__global__ __launch_bounds__(256) void k_sf_direct(const double2* __restrict__ z, int L, int kmax,
                                                   double* __restrict__ part) {
    extern __shared__ double2 sm[];
    double2* buf = sm;
    double2* tw = sm + L;   // tw[m] = exp(-2 pi i m / L)
    const double2* zl = z + (size_t)blockIdx.x * L;
    for (int m = threadIdx.x; m < L; m += blockDim.x) {
        double sn, cs;
        sincospi(2.0 * (double)m / (double)L, &sn, &cs);
        tw[m] = make_double2(cs, -sn);
    }
    double* out = part + (size_t)blockIdx.x * (kmax + 1);
    for (int i = threadIdx.x; i < L; i += blockDim.x) buf[i] = zl[i];
    __syncthreads();
    for (int k = threadIdx.x; k <= kmax; k += blockDim.x) {
        // A = Z_k = sum z_x w^(k x), B = Z_{L-k} = sum z_x conj(w)^(k x)
        double ar = 0.0, ai = 0.0, br = 0.0, bi = 0.0;
        int m = 0;
        for (int x = 0; x < L; ++x) {
            const double2 w = tw[m], v = buf[x];
            ar += v.x * w.x - v.y * w.y;
            ai += v.x * w.y + v.y * w.x;
            br += v.x * w.x + v.y * w.y;
            bi += v.y * w.x - v.x * w.y;
            m += k;
            if (m >= L) m -= L;
        }
        out[k] = 0.5 * (ar * ar + ai * ai + br * br + bi * bi);
    }
}

void launch_sf_twiddles(double* tw, int L, hipStream_t s) {
    k_sf_twiddles<<<(L + 255) / 256, 256, 0, s>>>(reinterpret_cast<double2*>(tw), L);
    check_hip(hipGetLastError(), "twiddle kernel launch");
}

template <typename R>
void launch_structure_factor(const R* th, int Lx, int Ly, int sx, int sy, int model, int axis, int kmax,
                             const double* tw, double* scratch, double* out, hipStream_t s) {
    const double q = model == kModelSI ? 2.0 : 1.0;
    const int L = axis == 0 ? Lx : Ly;
    const int nlines = axis == 0 ? Ly : Lx;
    const double N = (double)Lx * (double)Ly;
    if (sf_smooth(L)) {
        const SfShape h = sf_shape(L, nlines, kmax);
        const size_t lds = sizeof(double2) * (size_t)h.nlb * (size_t)sf_pitch(L);
        const double2* t = reinterpret_cast<const double2*>(tw);
        // the radix-7 pass alone needs more than 128 registers (two workgroups
        // per CU): a kernel of its own for the lengths that have it
        const auto kf = L % 7 == 0 ? (axis == 0 ? k_sf_lines<R, 0, true> : k_sf_lines<R, 1, true>)
                                   : (axis == 0 ? k_sf_lines<R, 0, false> : k_sf_lines<R, 1, false>);
        check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kf), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)lds),
                  "hipFuncSetAttribute");
        kf<<<h.grid, kSfThreads, lds, s>>>(th, Lx, sx, sy, q, t, L, nlines, h.nlb, kmax, h.nsub, scratch);
        check_hip(hipGetLastError(), "structure factor kernel launch");
        launch_row_sum(scratch, h.grid * h.nsub, kmax, N, out, s);
        return;
    }
    double2* z = reinterpret_cast<double2*>(scratch);
    double* part = scratch + 2 * (size_t)Lx * Ly;
    if (axis == 0) {
        const size_t n = (size_t)Lx * Ly;
        const unsigned nb = (unsigned)std::min<size_t>((n + 255) / 256, 65536);
        k_rotor_rows<R><<<nb, 256, 0, s>>>(th, Lx, Ly, sx, sy, q, z);
    } else {
        const dim3 grid((Lx + 31) / 32, (Ly + 31) / 32);
        k_rotor_cols<R><<<grid, 256, 0, s>>>(th, Lx, Ly, sx, sy, q, z);
    }
    check_hip(hipGetLastError(), "rotor kernel launch");
    const size_t lds = sizeof(double2) * (size_t)(2 * L);
    check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(k_sf_direct),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds),
              "hipFuncSetAttribute");
    k_sf_direct<<<nlines, 256, lds, s>>>(z, L, kmax, part);
    check_hip(hipGetLastError(), "structure factor kernel launch");
    launch_row_sum(part, nlines, kmax, N, out, s);
}

// -------------------------------------------------------------- domains
// Spin of site (x, y), decided in the state precision: eps * (|th| <= pi_p/2
// ? +1 : -1) (the sign of cos th, XY) or eps * (th >= 0 ? +1 : -1) (the sign
// of sin 2th on the half circle, SI).
template <typename R>
__device__ __forceinline__ int spin_of(const R* th, int Lx, int x, int y, int sx, int sy, int model) {
    const R t = th[(size_t)y * Lx + x];
    const bool up = model == kModelSI ? t >= R(0) : (t <= Prec<R>::kHalfPi && t >= -Prec<R>::kHalfPi);
    const int s = up ? 1 : -1;
    return (((x * sx) + (y * sy)) & 1) ? -s : s;
}

__device__ __forceinline__ int32_t uf_load(const int32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int32_t uf_find(const int32_t* parent, int32_t a) {
    int32_t p = uf_load(parent + a);
    while (p != a) {
        a = p;
        p = uf_load(parent + a);
    }
    return a;
}

// Union with monotone links (the larger root is hooked under the smaller by
// atomicMin; parent[i] <= i always, so every find terminates).  If the hook
// finds that another thread re-parented that root first (to `old`), atomicMin
// may have replaced the link to `old` by the link to the other root, so the
// loop goes on uniting `old` with the other root: no connection is lost
// (Playne and Hawick, IEEE TPDS 2018).  The surviving root of a cluster is its
// smallest index.
__device__ __forceinline__ void uf_union(int32_t* parent, int32_t a, int32_t b) {
    while (true) {
        a = uf_find(parent, a);
        b = uf_find(parent, b);
        if (a == b) return;
        if (a < b) {
            const int32_t t = a;
            a = b;
            b = t;
        }
        // a > b: hook root a under b
        const int32_t old = atomicMin(parent + a, b);
        if (old == a) return;
        a = old;
    }
}

// The same find and union on a workgroup's LDS labels.
__device__ __forceinline__ int32_t uf_lds_load(const int32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ int32_t uf_lds_find(const int32_t* lab, int32_t a) {
    int32_t p = uf_lds_load(lab + a);
    while (p != a) {
        a = p;
        p = uf_lds_load(lab + a);
    }
    return a;
}
__device__ __forceinline__ void uf_lds_union(int32_t* lab, int32_t a, int32_t b) {
    while (true) {
        a = uf_lds_find(lab, a);
        b = uf_lds_find(lab, b);
        if (a == b) return;
        if (a < b) {
            const int32_t t = a;
            a = b;
            b = t;
        }
        const int32_t old = atomicMin(lab + a, b);
        if (old == a) return;
        a = old;
    }
}

// Labelling in two levels.  First every kUfTile x kUfTile tile is labelled in
// LDS with the bonds that lie inside it: a tile's sites in row-major order are
// in the lattice's index order, so the smallest local index of a piece is also
// its smallest lattice index, and parent[i] = that index keeps parent[i] <= i.
// Then only the bonds across a tile's right and bottom edges (the periodic
// wrap among them) are united in global memory, a few percent of all bonds
// (every bond on the global atomics before).
constexpr int kUfTile = 32;

// The tile's rows as 32-bit words of spins (a wave's ballot covers two rows):
// a site starts at the first site of its run in the row, and a run is united
// with the row below once per stretch of equal columns, at its first one; the
// other bonds join sites that are joined already.  At 2048^2 after a quench
// 25 us a launch where every bond was united in LDS (49); also clears what the
// later launches add to (size, hist, the count of sizes).
template <typename R>
__global__ __launch_bounds__(256) void k_uf_local(const R* __restrict__ th, int Lx, int Ly, int sx, int sy,
                                                  int model, int ntx, int32_t* parent, uint32_t* size,
                                                  uint32_t* hist, uint32_t* stats) {
    static_assert(kUfTile == 32, "a row per 32-bit word");
    constexpr int kPer = kUfTile * kUfTile / 256;
    __shared__ int32_t lab[kUfTile * kUfTile];
    __shared__ uint32_t up[kUfTile];
    const int tx = (int)(blockIdx.x % (unsigned)ntx), ty = (int)(blockIdx.x / (unsigned)ntx);
    const int x0 = tx * kUfTile, y0 = ty * kUfTile;
    const int w = min(kUfTile, Lx - x0), h = min(kUfTile, Ly - y0);
    const int lx = (int)threadIdx.x % kUfTile, r0 = (int)threadIdx.x / kUfTile;   // row r0 + 8 k of site k
    if (blockIdx.x == 0 && threadIdx.x < kDomainPairs) stats[threadIdx.x] = 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) hist[0] = 0u;
    int8_t sp[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int ly = r0 + 8 * k;
        sp[k] = (lx < w && ly < h) ? (int8_t)spin_of(th, Lx, x0 + lx, y0 + ly, sx, sy, model) : (int8_t)0;
    }
    uint32_t same[kPer];   // bit i: site i of the row has the spin of site i - 1
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int ly = r0 + 8 * k;
        const uint32_t m = (uint32_t)(__ballot(sp[k] > 0) >> ((threadIdx.x & 32) ? 32 : 0));
        same[k] = ~(m ^ (m << 1)) & ~1u;
        const uint32_t breaks = ~same[k] & (0xFFFFFFFFu >> (31 - lx));   // bit 0 is always one
        lab[ly * kUfTile + lx] = ly * kUfTile + 31 - __clz((int)breaks);
        if (lx == 0) up[ly] = m;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int ly = r0 + 8 * k;
        if (lx >= w || ly + 1 >= h) continue;
        const uint32_t v = ~(up[ly] ^ up[ly + 1]);          // bit i: equal to the site below
        const uint32_t first = v & ~((v << 1) & same[k]);   // where the bond to the left does not say it too
        if ((first >> lx) & 1u) uf_lds_union(lab, ly * kUfTile + lx, (ly + 1) * kUfTile + lx);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int ly = r0 + 8 * k;
        if (lx >= w || ly >= h) continue;
        const int32_t r = uf_lds_find(lab, ly * kUfTile + lx);
        const size_t gi = (size_t)(y0 + ly) * Lx + (size_t)(x0 + lx);
        parent[gi] = (int32_t)((size_t)(y0 + r / kUfTile) * Lx + (size_t)(x0 + r % kUfTile));
        size[gi] = 0u;
        hist[gi + 1] = 0u;
    }
}

// Bonds across tile edges: thread t < ntx Ly takes the right edge of tile
// column t / Ly in row t % Ly (the last column's bond wraps to x = 0); the
// next nty Lx threads take the bottom edges of the tile rows (the last row's
// bond wraps to y = 0).  A bond whose four sites with the bond before it (in
// the same pair of tiles) are alike joins what that one joins.
template <typename R>
__global__ void k_uf_boundary(const R* __restrict__ th, int Lx, int Ly, int sx, int sy, int model, int ntx, int nty,
                              int32_t* parent) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t nr = (size_t)ntx * Ly;
    int x, y, xn, yn, dx = 0, dy = 0;
    if (t < nr) {
        const int tx = (int)(t / (size_t)Ly);
        y = (int)(t % (size_t)Ly);
        x = min((tx + 1) * kUfTile, Lx) - 1;
        xn = x + 1 == Lx ? 0 : x + 1;
        yn = y;
        dy = y % kUfTile ? 1 : 0;
    } else if (t < nr + (size_t)nty * Lx) {
        const size_t u = t - nr;
        const int ty = (int)(u / (size_t)Lx);
        x = (int)(u % (size_t)Lx);
        y = min((ty + 1) * kUfTile, Ly) - 1;
        xn = x;
        yn = y + 1 == Ly ? 0 : y + 1;
        dx = x % kUfTile ? 1 : 0;
    } else {
        return;
    }
    const int a = spin_of(th, Lx, x, y, sx, sy, model), b = spin_of(th, Lx, xn, yn, sx, sy, model);
    const int ap = spin_of(th, Lx, x - dx, y - dy, sx, sy, model);
    const int bp = spin_of(th, Lx, xn - dx, yn - dy, sx, sy, model);
    if (a != b || (dx + dy && ap == a && bp == a)) return;
    uf_union(parent, (int32_t)((size_t)y * Lx + x), (int32_t)((size_t)yn * Lx + xn));
}

// Labels and sizes per tile, after the edge merge.  Only roots had their
// parent changed by the merge, so a site's parent is its tile-local root or,
// for a local root, itself or the root it was hooked under.  In LDS each site
// points at its parent where that lies in the tile (an index no larger than
// its own); a chain ends at a root of the whole lattice or at a site whose
// parent lies outside the tile, which takes one find in global memory.  Every
// site's label is its chain end's, and each chain end adds its count of
// sites to its root's size once.  Concurrent finds from other tiles see a
// site's old parent or its root, both ancestors, so they still end at the
// root.
// Launched with 256 threads per tile (each thread keeps the chain ends of its
// TILE^2 / 256 sites in registers).
template <int TILE>
__global__ __launch_bounds__(256) void k_uf_flatten_tiles(int32_t* parent, uint32_t* size, int Lx, int Ly, int ntx) {
    static_assert(TILE * TILE % 256 == 0, "whole sites per thread");
    __shared__ int32_t nxt[TILE * TILE];
    __shared__ int32_t fin[TILE * TILE];
    __shared__ uint32_t cnt[TILE * TILE];
    const int tx = (int)(blockIdx.x % (unsigned)ntx), ty = (int)(blockIdx.x / (unsigned)ntx);
    const int x0 = tx * TILE, y0 = ty * TILE;
    const int w = min(TILE, Lx - x0), h = min(TILE, Ly - y0);
    for (int l = threadIdx.x; l < TILE * TILE; l += blockDim.x) {
        const int ly = l / TILE, lx = l % TILE;
        cnt[l] = 0u;
        nxt[l] = l;
        if (lx >= w || ly >= h) continue;
        const size_t gi = (size_t)(y0 + ly) * Lx + (size_t)(x0 + lx);
        const int32_t p = uf_load(parent + gi);
        const int py = (int)((size_t)p / (size_t)Lx), px = (int)((size_t)p % (size_t)Lx);
        if ((size_t)p == gi) {
            fin[l] = p;                                        // a root of the lattice
        } else if (py >= y0 && py < y0 + h && px >= x0 && px < x0 + w) {
            nxt[l] = (py - y0) * TILE + (px - x0);             // in the tile: at most l
        } else {
            nxt[l] = -1;                                       // leaves the tile
            fin[l] = uf_find(parent, p);
        }
    }
    __syncthreads();
    // the chain ends of the thread's sites (nxt is not written in this phase)
    constexpr int kPer = TILE * TILE / 256;
    int ends[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int l = (int)threadIdx.x + 256 * k;
        const int ly = l / TILE, lx = l % TILE;
        ends[k] = -1;
        if (lx >= w || ly >= h) continue;
        int e = l;
        while (nxt[e] >= 0 && nxt[e] != e) e = nxt[e];
        atomicAdd(&cnt[e], 1u);
        ends[k] = e;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int l = (int)threadIdx.x + 256 * k;
        if (ends[k] < 0) continue;
        const int ly = l / TILE, lx = l % TILE;
        const size_t gi = (size_t)(y0 + ly) * Lx + (size_t)(x0 + lx);
        __hip_atomic_store(parent + gi, fin[ends[k]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cnt[l]) atomicAdd(size + fin[l], cnt[l]);
    }
}

// After the flatten pass the sites with a size are the roots: histogram the
// cluster sizes.  Each workgroup takes a contiguous chunk of sites and counts
// sizes below kHistLds in LDS, flushing each nonzero bin with one atomic;
// larger sizes (few, and spread over many bins) go to the histogram directly.
// This keeps the many small domains from queueing on a few global addresses.
constexpr int kHistLds = 1024;
__global__ __launch_bounds__(1024) void k_uf_finish(const uint32_t* __restrict__ size, uint32_t* hist, size_t N) {
    __shared__ uint32_t h[kHistLds];
    for (int b = threadIdx.x; b < kHistLds; b += blockDim.x) h[b] = 0u;
    __syncthreads();
    // four sites per load (N is a multiple of 4)
    const size_t nq = N / 4, chunk = (nq + gridDim.x - 1) / gridDim.x;
    const size_t i0 = (size_t)blockIdx.x * chunk;
    const size_t i1 = i0 + chunk < nq ? i0 + chunk : nq;
#pragma unroll 4
    for (size_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
        const uint4 v = reinterpret_cast<const uint4*>(size)[i];
        const uint32_t sz[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (!sz[j]) continue;
            if (sz[j] < (uint32_t)kHistLds) atomicAdd(&h[sz[j]], 1u);
            else atomicAdd(hist + sz[j], 1u);
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kHistLds; b += blockDim.x)
        if (h[b]) atomicAdd(hist + b, h[b]);
}

// The size distribution as (size, count) pairs: every nonzero histogram entry
// hist[sz], sz = 1..N, appends one pair from stats[kDomainPairs] on (stats[0]
// counts them; the order is arbitrary).  Distinct sizes sum to at most N, so
// there are at most `cap` >= sqrt(2 N) of them.
__global__ void k_uf_sizes(const uint32_t* __restrict__ hist, uint32_t* stats, size_t N, uint32_t cap) {
    const size_t sz = (size_t)blockIdx.x * blockDim.x + threadIdx.x + 1;
    if (sz > N) return;
    const uint32_t c = hist[sz];
    if (c == 0u) return;
    const uint32_t j = atomicAdd(stats, 1u);
    if (j < cap) {
        stats[kDomainPairs + 2 * (size_t)j] = (uint32_t)sz;
        stats[kDomainPairs + 2 * (size_t)j + 1] = c;
    }
}

template <typename R>
void launch_domains(const R* th, int Lx, int Ly, int sx, int sy, int model, int32_t* parent, uint32_t* size,
                    uint32_t* hist,
                    uint32_t* stats, hipStream_t s) {
    const size_t N = (size_t)Lx * Ly;
    const unsigned nb = (unsigned)((N + 255) / 256);
    const int ntx = (Lx + kUfTile - 1) / kUfTile, nty = (Ly + kUfTile - 1) / kUfTile;
    k_uf_local<R><<<(unsigned)((size_t)ntx * nty), 256, 0, s>>>(th, Lx, Ly, sx, sy, model, ntx, parent, size,
                                                                hist, stats);
    check_hip(hipGetLastError(), "uf local labelling launch");
    const size_t nbond = (size_t)ntx * Ly + (size_t)nty * Lx;
    k_uf_boundary<R><<<(unsigned)((nbond + 255) / 256), 256, 0, s>>>(th, Lx, Ly, sx, sy, model, ntx, nty, parent);
    check_hip(hipGetLastError(), "uf boundary merge launch");
    k_uf_flatten_tiles<kUfTile><<<(unsigned)((size_t)ntx * nty), 256, 0, s>>>(parent, size, Lx, Ly, ntx);
    check_hip(hipGetLastError(), "uf flatten launch");
    // few workgroups: the flushes of one bin queue on its address (2048^2 after
    // a quench: 256 of 1024 threads 8.6 us, 1024 of 256 threads 21 us)
    k_uf_finish<<<(unsigned)std::min<size_t>((N + 16383) / 16384, 256), 1024, 0, s>>>(size, hist, N);
    check_hip(hipGetLastError(), "uf finish launch");
    k_uf_sizes<<<nb, 256, 0, s>>>(hist, stats, N, domain_size_cap(N));
    check_hip(hipGetLastError(), "uf sizes launch");
}

template void launch_correlation<float>(const float*, int, int, int, int, int, int, int, const double*, double*,
                                        double*, hipStream_t);
template void launch_correlation<double>(const double*, int, int, int, int, int, int, int, const double*, double*,
                                         double*, hipStream_t);
template void launch_structure_factor<float>(const float*, int, int, int, int, int, int, int, const double*, double*,
                                             double*, hipStream_t);
template void launch_structure_factor<double>(const double*, int, int, int, int, int, int, int, const double*, double*,
                                              double*, hipStream_t);
template void launch_domains<float>(const float*, int, int, int, int, int, int32_t*, uint32_t*, uint32_t*, uint32_t*,
                                    hipStream_t);
template void launch_domains<double>(const double*, int, int, int, int, int, int32_t*, uint32_t*, uint32_t*, uint32_t*,
                                     hipStream_t);

}  // namespace xyl
