// Host runtime behind the C-ABI of include/xyl.h.  Its sections, in order:
//   * devices, buffers (device memory and pinned host memory), parameters and
//     their validation, the launch rules;
//   * the lattice: creation (with its measurement phase tables), stepping
//     through captured graphs and two-step passes, sampled runs, observables,
//     correlation, structure factor, domains (and the allocation-free call),
//     the autotuner;
//   * the ensemble: replica tables, two-step classes on their own streams
//     (issued pass by pass), whole-in-LDS replicas on a side stream, chunk
//     graphs, samples through a finalize-job arena, its autotuner;
//   * the adjoint: the checkpointed forward run and the reverse sweep with
//     its recompute on a side stream.
// The host-only estimators (Binder cumulant, errors, fits) are in
// xyl_host.cpp.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <set>
#include <string>
#include <tuple>
#include <type_traits>
#include <vector>

#include "../../include/xyl.h"
#include "xyl_device.hpp"
#include "xyl_domains.hpp"
#include "xyl_internal.hpp"
#include "xyl_march.hpp"
#include "xyl_obs.hpp"
#include "xyl_tile.hpp"

namespace xyl {

void launch_finalize_jobs(const void* jobs, int njobs, hipStream_t s);

struct FinalizeJobHost {
    const double* part;
    int nrp;
    double N;
    double* out;
};

void check_hip(hipError_t e, const char* what) {
    if (e != hipSuccess) throw Error(XYL_EDEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

static void check_alloc(hipError_t e, const char* what) {
    if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation)
        throw Error(XYL_ENOMEM, std::string(what) + ": out of device memory");
    check_hip(e, what);
}

// ------------------------------------------------------------- devices
static bool is_gfx950(int dev) {
    hipDeviceProp_t p;
    if (hipGetDeviceProperties(&p, dev) != hipSuccess) return false;
    return std::strncmp(p.gcnArchName, "gfx950", 6) == 0;
}

static void select_device(int dev) {
    int n = 0;
    check_hip(hipGetDeviceCount(&n), "hipGetDeviceCount");
    require(dev >= 0 && dev < n, XYL_EINVAL, "device index out of range");
    require(is_gfx950(dev), XYL_EDEVICE, "device is not gfx950 (MI355X)");
    check_hip(hipSetDevice(dev), "hipSetDevice");
}

// Loads the kernels that the stepping rules may choose, on the current device:
// once per process, when a handle is created, not in a caller's step (2.5 ms for
// the tiles, 0.5 for the three-step pass).
static void load_stepping_kernels(int dev) {
    static std::mutex mu;
    static std::set<int> loaded;
    std::lock_guard<std::mutex> lk(mu);
    if (loaded.count(dev)) return;
    load_tile_kernels();
    load_march_kernels();
    loaded.insert(dev);
}

struct DeviceGuard {
    int prev = -1;
    explicit DeviceGuard(int dev) {
        (void)hipGetDevice(&prev);
        check_hip(hipSetDevice(dev), "hipSetDevice");
    }
    ~DeviceGuard() {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
};

template <typename T>
struct DevBuf {
    T* p = nullptr;
    size_t n = 0;
    // owns its allocation: movable, not copyable
    DevBuf() = default;
    DevBuf(const DevBuf&) = delete;
    DevBuf& operator=(const DevBuf&) = delete;
    DevBuf(DevBuf&& o) noexcept : p(o.p), n(o.n) {
        o.p = nullptr;
        o.n = 0;
    }
    DevBuf& operator=(DevBuf&& o) noexcept {
        if (this != &o) {
            release();
            p = o.p;
            n = o.n;
            o.p = nullptr;
            o.n = 0;
        }
        return *this;
    }
    void reserve(size_t count) {
        if (count <= n && p) return;
        if (p) (void)hipFree(p);
        p = nullptr;
        n = 0;
        check_alloc(hipMalloc(reinterpret_cast<void**>(&p), sizeof(T) * std::max<size_t>(count, 1)), "hipMalloc");
        n = count;
    }
    void release() {
        if (p) (void)hipFree(p);
        p = nullptr;
        n = 0;
    }
    ~DevBuf() { release(); }
};

// Page-locked host memory (hipHostMalloc): device-to-host copies of samples
// land here directly instead of through the runtime's staging of pageable
// memory, then go to the caller's array with a plain memcpy.
template <typename T>
struct PinnedBuf {
    T* p = nullptr;
    size_t n = 0;
    PinnedBuf() = default;
    PinnedBuf(const PinnedBuf&) = delete;
    PinnedBuf& operator=(const PinnedBuf&) = delete;
    void reserve(size_t count) {
        if (count <= n && p) return;
        release();
        check_alloc(hipHostMalloc(reinterpret_cast<void**>(&p), sizeof(T) * std::max<size_t>(count, 1),
                                  hipHostMallocDefault),
                    "hipHostMalloc");
        n = count;
    }
    void release() {
        if (p) (void)hipHostFree(p);
        p = nullptr;
        n = 0;
    }
    ~PinnedBuf() { release(); }
};

// What a handle keeps for its structure factors and correlations: scratch, the
// twiddle table of each axis length it has transformed (at most 64 KB each)
// and the results' landing place.
struct SpectrumBufs {
    DevBuf<double> scratch;
    std::map<int, DevBuf<double>> twiddles;
    PinnedBuf<double> host;
    // made, and waited for, by the first call of a length: a later call finds
    // it complete on any stream
    const double* table(int L, hipStream_t s) {
        if (!sf_smooth(L)) return nullptr;
        DevBuf<double>& t = twiddles[L];
        if (!t.p) {
            t.reserve(2 * (size_t)L);
            try {
                launch_sf_twiddles(t.p, L, s);
                check_hip(hipStreamSynchronize(s), "hipStreamSynchronize");
            } catch (...) {
                t.release();
                throw;
            }
        }
        return t.p;
    }
};

// Large results to pageable host memory: the runtime's own path copies such
// data to its staging memory and on, one after the other (16.8 MB of labels:
// 950 us); here the device writes one slot of a pinned ring while the host
// empties another (600 us).  The ring is made by the second copy of at least
// kMin bytes: pinning and first touching it takes as long as it saves once.
// Memory that the runtime knows (pinned by the caller) takes the copy directly:
// 2048^2 with labels 425 us, through the ring 750.
struct HostRing {
    static constexpr size_t kSlot = size_t(1) << 20, kMin = size_t(2) << 20;
    static constexpr int kSlots = 2;
    PinnedBuf<char> buf;
    hipEvent_t ev[kSlots] = {};
    bool asked = false;
    HostRing() = default;
    HostRing(const HostRing&) = delete;
    HostRing& operator=(const HostRing&) = delete;
    ~HostRing() {
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
    }
    // no ring where it cannot be had: the plain copy serves
    bool ready() {
        if (buf.p && ev[kSlots - 1]) return true;
        if (!asked) {
            asked = true;
            return false;
        }
        for (hipEvent_t& e : ev)
            if (!e && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
                (void)hipGetLastError();
                e = nullptr;
                return false;
            }
        try {
            buf.reserve(kSlot * kSlots);
        } catch (const Error&) {
            return false;
        }
        return true;
    }
    static bool pageable(const void* p) {
        hipPointerAttribute_t a{};
        if (hipPointerGetAttributes(&a, p) != hipSuccess) {
            (void)hipGetLastError();
            return true;
        }
        return a.type == hipMemoryTypeUnregistered;
    }
    // dst = src after what the stream holds; returns when dst is complete
    void copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
        if (bytes < kMin || !pageable(dst) || !ready()) {
            check_hip(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s), "D2H");
            check_hip(hipStreamSynchronize(s), "hipStreamSynchronize");
            return;
        }
        const size_t n = (bytes + kSlot - 1) / kSlot;
        auto size_of = [&](size_t c) { return std::min(kSlot, bytes - c * kSlot); };
        auto send = [&](size_t c) {
            const size_t b = c % kSlots;
            check_hip(hipMemcpyAsync(buf.p + b * kSlot, static_cast<const char*>(src) + c * kSlot, size_of(c),
                                     hipMemcpyDeviceToHost, s),
                      "D2H");
            check_hip(hipEventRecord(ev[b], s), "hipEventRecord");
        };
        for (size_t c = 0; c < std::min<size_t>(n, kSlots); ++c) send(c);
        for (size_t c = 0; c < n; ++c) {
            check_hip(hipEventSynchronize(ev[c % kSlots]), "hipEventSynchronize");
            std::memcpy(static_cast<char*>(dst) + c * kSlot, buf.p + c % kSlots * kSlot, size_of(c));
            if (c + kSlots < n) send(c + kSlots);
        }
    }
};

// What a handle keeps for its domain labellings.
struct DomainBufs {
    DevBuf<int32_t> parent;
    DevBuf<uint32_t> size, hist, stats;
    PinnedBuf<uint32_t> stats_host;
    HostRing labels;
};

// ------------------------------------------------------------ parameters
struct Params {
    double Jx = 1.0, Jy = -0.1, h = 0.5, gamma = 1.0, dt = 0.01;
    int model = kModelXY;   // XYL_MODEL_XY / XYL_MODEL_SI
    double p = 2.0;         // field order
};

static void validate_model(int model, double p) {
    require(model == XYL_MODEL_XY || model == XYL_MODEL_SI, XYL_EINVAL, "model must be XYL_MODEL_XY or XYL_MODEL_SI");
    if (model == XYL_MODEL_XY) require(p == 2.0, XYL_EINVAL, "the XY model has p = 2");
    else require(std::isfinite(p) && p > 0.0 && p <= 16.0, XYL_EINVAL, "p must be in (0, 16]");
}

static void validate_params(const Params& p) {
    require(std::isfinite(p.Jx) && std::isfinite(p.Jy) && std::isfinite(p.h) && std::isfinite(p.gamma) &&
                std::isfinite(p.dt),
            XYL_EINVAL, "parameters must be finite");
    require(p.dt > 0.0, XYL_EINVAL, "dt must be > 0");
    require(p.gamma >= 0.0, XYL_EINVAL, "gamma must be >= 0");
}

static Schedule make_schedule(const uint64_t* ks, const double* Ts, int32_t n, const int32_t* gs = nullptr) {
    require(n >= 1 && n <= kMaxKnots, XYL_EINVAL, "schedule needs 1..16 knots");
    require(ks != nullptr && Ts != nullptr, XYL_EINVAL, "schedule arrays are NULL");
    Schedule s{};
    s.n = n;
    for (int j = 0; j < n; ++j) {
        require(std::isfinite(Ts[j]) && Ts[j] >= 0.0, XYL_EINVAL, "schedule temperatures must be finite and >= 0");
        if (j > 0) require(ks[j] > ks[j - 1], XYL_EINVAL, "schedule steps must be strictly increasing");
        s.step[j] = ks[j];
        s.T[j] = Ts[j];
        const int g = gs ? gs[j] : 1;
        require(g >= -16 && g <= 16, XYL_EINVAL, "schedule shape exponents must lie in [-16, 16]");
        s.g[j] = g == 0 ? 1 : g;
    }
    return s;
}

// Whether the FP32 kick may be factored by the x coupling: it divides by
// hdt q Jx, so that and the ratios it creates must stay well inside binary32's
// range.  The two-step passes need it (their kernels are compiled for that
// form only); other lattices keep the unfactored kick in every kernel.
static bool kick_factored(const Params& p) {
    if (p.Jx == 0.0) return false;
    const double q = p.model == kModelSI ? 2.0 : 1.0;
    const double kjx = 0.5 * p.dt * q * p.Jx, big = 1048576.0;
    return std::fabs(p.Jy / p.Jx) <= big && std::fabs(4.0 * p.h / (q * p.Jx)) <= big &&
           std::fabs(p.p * p.h / (q * p.Jx)) <= big && std::fabs(kjx) >= 1e-12 && std::fabs(kjx) <= big;
}

template <typename R>
static void fill_lat(Lat<R>& v, int Lx, int Ly, const Params& p, const Schedule& s, uint64_t seed, uint32_t replica) {
    v.Lx = Lx;
    v.Ly = Ly;
    v.nxw = (Lx + kWaveSites - 1) / kWaveSites;
    v.stag_x = p.Jx > 0.0 ? 1 : 0;
    v.stag_y = p.Jy > 0.0 ? 1 : 0;
    v.model = p.model;
    const double q = p.model == kModelSI ? 2.0 : 1.0;
    v.Jx = (R)(q * p.Jx);
    v.Jy = (R)(q * p.Jy);
    v.h4 = (R)(4.0 * p.h);
    v.ph = (R)(p.p * p.h);
    // FP32 native sine takes revolutions: sin(p t) = sin_rev(t * p / 2pi)
    v.pf = sizeof(R) == 4 ? (R)(p.p / (2.0 * M_PI)) : (R)p.p;
    v.pd = p.p;
    v.a = (R)(1.0 - 0.5 * p.gamma * p.dt);
    v.c = (R)(1.0 / (1.0 + 0.5 * p.gamma * p.dt));
    const double acd = (1.0 - 0.5 * p.gamma * p.dt) / (1.0 + 0.5 * p.gamma * p.dt);
    v.ac = (R)acd;
    // the FP32 kick factored by the x coupling (site_force)
    v.fact = (sizeof(R) == 4 && kick_factored(p)) ? 1 : 0;
    const double kjx = 0.5 * p.dt * q * p.Jx;
    v.fr = v.fact ? (R)(p.Jy / p.Jx) : R(0);
    v.fh = v.fact ? (R)(4.0 * p.h / (q * p.Jx)) : R(0);
    v.fph = v.fact ? (R)(p.p * p.h / (q * p.Jx)) : R(0);
    v.fc1 = (R)(kjx * (1.0 + acd));
    v.fnoise = v.fact ? 1.0 / (kjx * kjx) : 1.0;
    // the draws divided by hdt q Jx: their scale goes through the Box-Muller
    // square root, so a negative divisor flips the angle by half a turn
    v.fu2 = (R)(v.fact && kjx < 0.0 ? 0.5 - 0x1p-24 : 1.0 - 0x1p-24);
    v.hdt = (R)(0.5 * p.dt);
    v.dt = (R)p.dt;
    v.kJx = (R)(0.5 * p.dt * q * p.Jx);
    v.kJy = (R)(0.5 * p.dt * q * p.Jy);
    v.kh4 = (R)(0.5 * p.dt * 4.0 * p.h);
    v.kph = (R)(0.5 * p.dt * p.p * p.h);
    v.Jxd = p.Jx;
    v.Jyd = p.Jy;
    v.hd = p.h;
    v.gamma = p.gamma;
    v.dtd = p.dt;
    v.sched = s;
    v.seed_lo = (uint32_t)seed;
    v.seed_hi = (uint32_t)(seed >> 32);
    v.replica = replica;
}

static void validate_shape(int Lx, int Ly) {
    require(Lx >= 2 && Ly >= 2, XYL_EINVAL, "Lx and Ly must be >= 2");
    require((double)Lx * (double)Ly < 17179869184.0, XYL_EINVAL, "Lx*Ly must be < 2^34");
    require(Lx % 4 == 0, XYL_EUNSUPPORTED, "Lx must be a multiple of 4 (one Philox block per 4 sites of a row)");
    require((double)Lx * (double)Ly < 2147483647.0, XYL_EUNSUPPORTED, "Lx*Ly must fit int32 labels");
}

static size_t elem_size(int dtype) { return dtype == XYL_F64 ? sizeof(double) : sizeof(float); }

// -------------------------------------------------------- launch tuning
static std::mutex g_tune_mu;
static std::map<std::tuple<int, int, int>, Launch> g_tuned;
// How runs of steps go, as xyl_autotune measured it: the steps per pass, the
// rows per strip and the waves per column tile of the two-step pass, and
// whether tiles or the three-step pass were the fastest (the rules' choice
// where nothing was measured).
enum : int { kByRule = 0, kChosen = 1, kSlower = 2 };
struct Tuned2 {
    int fusion = 2, rows = 0, tile_waves = 0;
    int tiles = kByRule, march = kByRule;
};
// by Lx, Ly, precision, model and form of the FP32 kick
static std::map<std::tuple<int, int, int, int, int>, Tuned2> g_tuned2;
// launch shape of measurements without a step, chosen by xyl_autotune
static std::map<std::tuple<int, int, int>, Launch> g_tunedm;

// Launch shape before any autotuning: enough waves to occupy every SIMD of
// the 256 CUs (strips of up to 16 rows while there are >= 4096 wave-rows,
// down to single-row strips and one-wave workgroups for small lattices).
static Launch default_launch(int Lx, int Ly) {
    const long wave_rows = (long)Ly * ((Lx + kWaveSites - 1) / kWaveSites);
    Launch l;
    l.rows = (int)std::max<long>(1, std::min<long>(16, wave_rows / 4096));
    const long waves = wave_rows / l.rows;
    l.wpb = waves >= 8192 ? 4 : (waves >= 2048 ? 2 : 1);
    return l;
}

static void validate_launch(const Launch& l) {
    require(l.rows >= 1, XYL_EINVAL, "rows per strip must be >= 1");
    require(l.wpb == 1 || l.wpb == 2 || l.wpb == 4 || l.wpb == 8, XYL_EINVAL, "waves per block must be 1, 2, 4 or 8");
}


}  // namespace xyl

using namespace xyl;

// ===================================================================== lattice
struct xyl_lattice {
    int dtype = XYL_F32;
    int device = 0;
    int Lx = 0, Ly = 0;
    size_t N = 0;
    bool owns = true;
    void* th[2] = {nullptr, nullptr};
    void* u = nullptr;
    int cur = 0;                  // th^k lives in th[(k + cur) & 1]
    hipStream_t stream = nullptr;
    hipStream_t cap_stream = nullptr;
    Params p;
    Schedule sched{};
    uint64_t seed = 0;
    uint32_t replica = 0;
    uint64_t k = 0;
    uint64_t fresh_k = 0;
    bool initialized = false;
    Launch launch;
    // launch shape of measurements without a step (xyl_autotune's choice;
    // otherwise the stepping shape)
    Launch mlaunch;
    bool mlaunch_tuned = false;
    int graph_steps = 32;
    // captured step sequences, keyed by what their kernel arguments bake in
    struct GraphEntry {
        int mode = 0, S = 0, cur = 0;
        double* part = nullptr;
        uint64_t part_k0 = 0, part_stride = 0;
        uint64_t version = 0;
        hipGraphExec_t exec = nullptr;
    };
    std::vector<GraphEntry> graphs;
    uint64_t version = 0;
    bool counter_valid = false;
    int fusion = 2;                // steps per pass of plain FP32 stepping where the shape allows (1 or 2)
    int cus = 256;                 // compute units of the device
    int march = kByRule;           // three steps per pass (xyl_march.hip)
    int step2_rows_tuned = 0;      // rows per strip of the two-step pass from xyl_autotune (0: the size rule)
    int step2_tw_tuned = 0;        // most waves per column tile (widths above 4096) from xyl_autotune (0: the rule)
    int tiles = kByRule;           // several steps per launch on tiles
    bool shaped = false;           // the caller shaped the two-step pass
    bool own_path = false;         // the caller set or tuned the path: the process's record is not looked up again
    // by the steps to take and the form of the kick (T = 0: none)
    std::map<std::pair<uint64_t, bool>, TilePlan> tile_plans;
    int adj2_rows = 0;             // rows per strip of the two-step reverse pass (0: the rule)
    int adj_fusion = 2;            // reverse steps per pass of the adjoint sweep (1 or 2)
    DevBuf<char> u2;               // second velocity buffer of the paths with several steps per launch
    bool second_u = true;          // false: it did not fit
    // device scratch
    DevBuf<uint64_t> kdev;
    DevBuf<double> part;
    DevBuf<double> samples;       // partial sums of the samples of a call, reduced together
    DevBuf<double> obs;
    PinnedBuf<double> obs_host;   // host landing place of the samples' copy
    DevBuf<double> dscratch;
    SpectrumBufs spectrum;
    DevBuf<char> omega_buf;
    DomainBufs domains;
    DevBuf<uint32_t> flag;        // validation result of xyl_set_state_device
    DevBuf<double> phases;        // measurement phases: the x table (2 Lx), then the y table (2 Ly)
    // adjoint state (see xyl_adjoint.hip)
    void* adj = nullptr;

    template <typename R>
    Lat<R> view() {
        Lat<R> v{};
        v.th[0] = static_cast<R*>(th[0]);
        v.th[1] = static_cast<R*>(th[1]);
        v.u = static_cast<R*>(u);
        v.cur = cur;
        fill_lat(v, Lx, Ly, p, sched, seed, replica);
        v.k_base = 0;
        v.fresh_k = fresh_k;
        v.k_end = ~(uint64_t)0;
        v.part = part.p;
        v.xph = phases.p;
        v.yph = phases.p + 2 * (size_t)Lx;
        v.omega_out = reinterpret_cast<R*>(omega_buf.p);
        v.pingpong = 1;
        v.u_out = nullptr;
        v.part_k0 = 0;
        v.part_stride = 0;
        return v;
    }
    void* cur_theta() { return th[(int)((k + (uint64_t)cur) & 1)]; }
    int nrowparts() const { return Ly * ((Lx + kWaveSites - 1) / kWaveSites); }
    void touch() { ++version; }
};

// State of a pathwise-gradient run between xyl_adjoint_forward and
// xyl_adjoint_backward: checkpoints every K steps, the loss samples and the
// device buffers of the reverse sweep.
struct AdjState {
    bool valid = false;          // a forward run completed and may be differentiated
    uint64_t run = 0;            // identifier of that run (process-wide, never reused)
    uint64_t version = 0;        // the lattice's configuration version when it ended
    uint64_t k0 = 0, N = 0, K = 0, W = 0;
    double loss = 0.0;
    std::vector<double> m;       // m_s at steps k0+N-W+1 .. k0+N
    DevBuf<char> ckpt, seg, lam;
    DevBuf<double> cm, gacc, obs, win;
    DevBuf<uint64_t> kseg;                 // step counters: [0] reverse (main stream), [1] recompute (side)
    // Backward sweep: segment buffers b = 0, 1 (K + 1 states each); the
    // recomputation of the next segment runs on a second stream into one
    // buffer while the reverse steps of the current one read the other.
    hipStream_t side = nullptr;
    hipEvent_t ev_rec[2] = {nullptr, nullptr}, ev_rev[2] = {nullptr, nullptr}, ev_start = nullptr;
    hipGraphExec_t rec_graph[2] = {nullptr, nullptr};        // K recompute steps into buffer b
    hipGraphExec_t rev_graph[2][2] = {{nullptr, nullptr}, {nullptr, nullptr}};   // [b][adjoint parity]
    // tile plans of the recompute and of the reverse steps for segments of
    // tile_K steps (64 and more share one; T = 0: none fits)
    uint64_t tile_K = 0;
    TilePlan rec, rev;
    double rec_us = 0.0, rev_us = 0.0;   // their modelled times per step
    // what the captured graphs bake in; they are rebuilt when it changes
    std::vector<uint64_t> graph_key;
    void drop_graphs() {
        for (auto& g : rec_graph) {
            if (g) (void)hipGraphExecDestroy(g);
            g = nullptr;
        }
        for (auto& r : rev_graph)
            for (auto& g : r) {
                if (g) (void)hipGraphExecDestroy(g);
                g = nullptr;
            }
    }
    ~AdjState() {
        drop_graphs();
        for (int b = 0; b < 2; ++b) {
            if (ev_rec[b]) (void)hipEventDestroy(ev_rec[b]);
            if (ev_rev[b]) (void)hipEventDestroy(ev_rev[b]);
        }
        if (ev_start) (void)hipEventDestroy(ev_start);
        if (side) (void)hipStreamDestroy(side);
    }
};

// Identifiers of adjoint forward runs: a backward call names the run it
// differentiates, and a later forward on the same lattice (which replaces the
// checkpoints) makes earlier identifiers stale.
static std::atomic<uint64_t> g_adj_runs{0};

static void adjoint_release(xyl_lattice* h) {
    delete static_cast<AdjState*>(h->adj);
    h->adj = nullptr;
}

static void destroy_graph(xyl_lattice* h) {
    for (auto& g : h->graphs)
        if (g.exec) (void)hipGraphExecDestroy(g.exec);
    h->graphs.clear();
}

template <typename R>
static void lattice_launch_one(xyl_lattice* h, int mode, double* part = nullptr) {
    Lat<R> v = h->view<R>();
    if (part) v.part = part;
    const Launch& l = (mode == kMeasure && h->mlaunch_tuned) ? h->mlaunch : h->launch;
    launch_step<R>(v, mode, l, nullptr, h->k, h->stream);
}

// Captures S consecutive steps whose step index comes from the device counter
// (node j runs step *kdev + j), followed by a node that advances the counter.
template <typename R>
static hipGraphExec_t capture_steps(xyl_lattice* h, const Lat<R>& v, int mode, int S) {
    hipGraph_t g = nullptr;
    check_hip(hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
    try {
        for (int j = 0; j < S; ++j) launch_step<R>(v, mode, h->launch, h->kdev.p, (uint64_t)j, h->cap_stream);
        launch_bump(h->kdev.p, (uint64_t)S, h->cap_stream);
    } catch (...) {
        (void)hipStreamEndCapture(h->cap_stream, &g);
        if (g) (void)hipGraphDestroy(g);
        throw;
    }
    check_hip(hipStreamEndCapture(h->cap_stream, &g), "hipStreamEndCapture");
    hipGraphExec_t ex = nullptr;
    hipError_t e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    check_hip(e, "hipGraphInstantiate");
    return ex;
}

// Two steps per pass (FP32 plain stepping, width a multiple of 256 up to 4096).
static bool step2_shape(int Lx, int Ly) { return step2_width_ok(Lx) && Ly >= 4; }
// single lattices also take widths above 4096, as column tiles
static bool step2_lattice_shape(int Lx, int Ly) {
    Step2Tiles t;
    return Ly >= 4 && (step2_width_ok(Lx) || step2_tiles(Lx, &t));
}
static bool step2_eligible(const xyl_lattice* h) {
    return h->dtype == XYL_F32 && h->fusion == 2 && kick_factored(h->p) && step2_lattice_shape(h->Lx, h->Ly);
}
// The caller shaped the two-step pass, and the lattice can take it: it does, in
// place of tiles and of three steps per pass.
static bool step2_shaped(const xyl_lattice* h) { return h->shaped && step2_eligible(h); }

// Waves per column tile of the two-step pass when not tuned: rows up to 4096
// sites wide run whole (one workgroup per strip); wider ones as tiles of at
// most 4 waves, four workgroups per CU (8192^2: 9 tiles, 119 against 143 us
// per step with the fewest tiles, 3 of 11 waves; 6144^2, 12288 x 4096 and
// 16384 x 2048 gain 14-18% the same way), where such a tiling exists.
static int step2_tile_waves(int Lx) {
    Step2Tiles t;
    return Lx > 16 * kWaveSites && step2_tiles(Lx, &t, 4) ? 4 : 16;
}
static int step2_tile_waves(const xyl_lattice* h) {
    return h->step2_tw_tuned ? h->step2_tw_tuned : step2_tile_waves(h->Lx);
}

// Time per step (us) of whole-row two-step passes with strips of `rows` rows,
// as a rule for choosing: a pass takes 3 us and, for every round of strips
// that the CUs hold at once, rows + 2 iterations (two halo rows) of
// sqrt(1 + (0.6 x)^2) us each, x the waves per SIMD (a row of 256 sites per
// wave; min(16 / waves, 160 KiB / LDS) workgroups per CU).  Within 15% of the
// passes measured at 512^2 .. 4096^2, 4096 x 1024, 1024 x 4096, 256 x 8192
// and 2900^2 (29.2 us per step with 11-row strips, 264 of them on 256 CUs).
static double step2_us(int Lx, int Ly, int cus, int rows) {
    const int waves = (Lx + kWaveSites - 1) / kWaveSites;
    const int fit = std::max(1, std::min(16 / waves, (160 * 1024) / (32 * Lx)));
    const int strips = (Ly + rows - 1) / rows;
    int left = (strips + cus - 1) / cus;
    double us = 3.0;
    for (; left > 0; left -= fit) {
        const double x = 0.6 * 0.25 * waves * std::min(left, fit);
        us += (std::min(rows, Ly) + 2) * std::sqrt(1.0 + x * x);
    }
    return 0.5 * us;
}

// Rows per strip of the two-step kernel: whole rows, the cheapest by the rule
// above (strip counts just above a multiple of what the CUs hold leave a last
// round of a few workgroups); column tiles as below.
static int step2_rows(int Lx, int Ly, int cus, int tile_waves) {
    Step2Tiles t;
    if (step2_tiles(Lx, &t, tile_waves) || step2_tiles(Lx, &t)) {
        // column tiles.  Several workgroups per CU (tiles of at most 8 waves:
        // as many as 16 waves of 128 VGPRs and the 160 KiB of LDS allow):
        // 16-row strips, measured best at 8192^2, 6144^2 and 16384 x 2048
        // with 2- to 4-wave tiles (8-row strips 6-7% slower, 32-row 0-10%).
        const int W = t.w + 2 * kLaneSites;
        const int waves = (W + kWaveSites - 1) / kWaveSites;
        const int per_cu =
            waves > 8 ? 1 : std::max(1, std::min(16 / waves, (160 * 1024) / (int)(sizeof(float) * 2 * kStep2Slots * W)));
        if (per_cu >= 2) return 16;
        // One workgroup per CU: the last round of workgroups matters.  Score =
        // rows / (rows + 1) (the halo rows' share of the work) times the
        // fraction of the last round that is filled; strips of up to 32 rows.
        int best = 32;
        double best_score = -1.0;
        for (int rows = 32; rows >= 2; rows /= 2) {
            const long wgs = (long)((Ly + rows - 1) / rows) * t.ntx;
            const long rounds = (wgs + cus - 1) / cus;
            const double score = (double)rows / (rows + 1) * (double)wgs / (double)(rounds * cus);
            if (score > best_score + 1e-9) {
                best_score = score;
                best = rows;
            }
        }
        return best;
    }
    int best = 2;
    double best_us = 1e30;
    for (int rows = 32; rows >= 2; --rows) {
        const double us = step2_us(Lx, Ly, cus, rows);
        if (us < 0.98 * best_us) {   // taller strips where two are about equal
            best_us = us;
            best = rows;
        }
    }
    return best;
}
static int step2_rows(const xyl_lattice* h) {
    return h->step2_rows_tuned ? h->step2_rows_tuned : step2_rows(h->Lx, h->Ly, h->cus, step2_tile_waves(h));
}

// Launches for 4m steps from the current step: pairs of two-step passes,
// (A, u) -> (B, u2) -> (A, u), A the buffer holding the angles at step k, so
// that the state ends where it started.  With kdev the step index comes from
// the device counter (graph capture), else from j.
static void step2_launches(xyl_lattice* h, const Lat<float>& v, uint64_t nsteps, const uint64_t* kdev, uint64_t j,
                           int parity, hipStream_t s) {
    float* A = static_cast<float*>(h->th[parity]);
    float* Bb = static_cast<float*>(h->th[parity ^ 1]);
    float* u = static_cast<float*>(h->u);
    float* u2 = reinterpret_cast<float*>(h->u2.p);
    const int rows = step2_rows(h), tw = step2_tile_waves(h);
    for (uint64_t i = 0; i < nsteps; i += 4) {
        launch_step2(v, A, u, Bb, u2, rows, kdev, j + i, s, tw);
        launch_step2(v, Bb, u2, A, u, rows, kdev, j + i + 2, s, tw);
    }
}

// Captures S (a multiple of 4) steps as two-step passes, then the counter bump.
static hipGraphExec_t capture_steps2(xyl_lattice* h, const Lat<float>& v, int S, int parity) {
    hipGraph_t g = nullptr;
    check_hip(hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
    try {
        step2_launches(h, v, (uint64_t)S, h->kdev.p, 0, parity, h->cap_stream);
        launch_bump(h->kdev.p, (uint64_t)S, h->cap_stream);
    } catch (...) {
        (void)hipStreamEndCapture(h->cap_stream, &g);
        if (g) (void)hipGraphDestroy(g);
        throw;
    }
    check_hip(hipStreamEndCapture(h->cap_stream, &g), "hipStreamEndCapture");
    hipGraphExec_t ex = nullptr;
    hipError_t e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    check_hip(e, "hipGraphInstantiate");
    return ex;
}

// Time per step (us) of the path that a lattice takes without tiles: two-step
// passes of whole rows, or single steps.  Single steps were measured at 7.0,
// 15.1 and 28.2 us for 1028^2, 2052^2 and 3076 x 3000 (FP32) and 8.1, 19.4 and
// 48.5 us for 512^2, 1024^2 and 2048^2 (FP64).
// Wider than 4096 the two-step pass runs on column tiles, about 5.8e5 sites per
// us (8192^2 114 us per step).
static double lattice_step2_us(const xyl_lattice* h) {
    return h->Lx > 16 * kWaveSites ? (double)h->N / 5.8e5 : step2_us(h->Lx, h->Ly, h->cus, step2_rows(h));
}
// Three steps per pass where that is faster than the two-step pass or, for
// widths that pass does not take, than single steps, by the rules' times (never
// for a lattice whose caller shaped the two-step pass).
static double lattice_single_us(const xyl_lattice* h) {
    return h->dtype == XYL_F64 ? 6.5 + (double)h->N / 1.15e5 : 3.3 + (double)h->N / 3.7e5;
}
static bool march_shape_ok(int dtype, int Ly) { return dtype == XYL_F32 && Ly >= 4; }
static bool lattice_march_plan(const xyl_lattice* h, MarchPlan* p) {
    if (h->march == kSlower || step2_shaped(h) || h->fusion != 2) return false;
    if (!march_shape_ok(h->dtype, h->Ly) || !kick_factored(h->p)) return false;
    *p = march_plan(h->Lx, h->Ly, h->cus);
    return h->march == kChosen || p->us < (step2_eligible(h) ? lattice_step2_us(h) : lattice_single_us(h));
}
// Steps of a run of n that go three per pass: pairs of passes, 6m steps.  The
// last two or three of a run would be single steps; where six, two of them
// single, take longer than eight on two-step passes, eight are left to those
// (4096^2: a call of 8 steps 238 us so against 260, of 20 steps 512 against 538).
static uint64_t lattice_march_steps(const xyl_lattice* h, uint64_t n, MarchPlan* p) {
    if (n < 2 * kMarchSteps || !lattice_march_plan(h, p)) return 0;
    const uint64_t r = n % (2 * kMarchSteps), m = n - r;
    const bool eight = (r == 2 || r == 3) && step2_eligible(h) &&
                       2 * kMarchSteps * p->us + 2 * lattice_single_us(h) > 8 * lattice_step2_us(h);
    return eight ? m - 2 * kMarchSteps : m;
}
static double lattice_untiled_us(const xyl_lattice* h) {
    MarchPlan p;
    if (lattice_march_plan(h, &p)) return p.us;
    if (step2_eligible(h)) return lattice_step2_us(h);
    return lattice_single_us(h);
}

// Whether the caller captures the lattice's stream (or it cannot be told):
// nothing is allocated and no graph of the library's is launched then.
static bool stream_captured(const xyl_lattice* h) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(h->stream, &st) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return st != hipStreamCaptureStatusNone;
}

// The second velocity buffer, which every path but single steps needs: where it
// does not fit, and in a caller's capture before it exists, the steps go one by
// one.
static bool lattice_second_u(xyl_lattice* h) {
    const size_t bytes = elem_size(h->dtype) * h->N;
    if (!h->second_u) return false;
    if (h->u2.p && h->u2.n >= bytes) return true;
    if (stream_captured(h)) return false;
    try {
        h->u2.reserve(bytes);
    } catch (const Error& e) {
        if (e.code != XYL_ENOMEM) throw;
        (void)hipGetLastError();
        h->second_u = false;
    }
    return h->second_u;
}

// Widths above 4096 and lattices beyond 2^24 sites never gain by tiles (their
// passes are bound by issue already, and tiles recompute more halo).
static bool tile_shape_ok(int Lx, int Ly) {
    return Lx <= 16 * kWaveSites && (size_t)Lx * Ly <= (size_t(1) << 24);
}
// Several steps per launch on tiles (xyl_tile.hip): the plan for a run of n
// steps (n >= 2), or NULL where another path is faster by the rules' times.
// Plans are kept per run length (64 steps and more share one) and form of the
// kick (the three-step pass that tiles are weighed against has one only).
static const TilePlan* lattice_tile_choice(xyl_lattice* h, uint64_t n) {
    if (h->tiles == kSlower || step2_shaped(h) || h->fusion != 2) return nullptr;
    if (n < 2 || !tile_shape_ok(h->Lx, h->Ly)) return nullptr;
    n = std::min<uint64_t>(n, 64);
    const auto key = std::make_pair(n, kick_factored(h->p));
    auto it = h->tile_plans.find(key);
    if (it == h->tile_plans.end()) {
        TilePlan p;
        MarchPlan mp;
        double us = 0.0;
        // Against three steps per pass the tiles' time counts 8% more: at the
        // sizes where the two meet it comes out so much short (measured, tiles
        // and march: 1500^2 5.8 and 6.5 us per step, 1604^2 8.0 and 6.7, 1800^2
        // 7.8 and 7.5, 2048 x 1024 5.3 and 5.9, 3000 x 1000 6.9 and 7.1).
        // (tiles reach 4.7e5 sites per us at best)
        const bool rule = h->tiles == kByRule;
        const bool hopeless = rule && (double)h->N > 4.8e5 * lattice_untiled_us(h);
        if (hopeless || !tile_plan(h->Lx, h->Ly, h->dtype == XYL_F64, h->cus, n, &p, &us) ||
            (rule && (us > lattice_untiled_us(h) || (lattice_march_plan(h, &mp) && 1.08 * us > mp.us))))
            p = TilePlan();
        it = h->tile_plans.emplace(key, p).first;
    }
    return it->second.T ? &it->second : nullptr;
}
// The same with the second velocity buffer that the tiles need.
static const TilePlan* lattice_tile_plan(xyl_lattice* h, uint64_t n) {
    const TilePlan* p = lattice_tile_choice(h, n);
    return p && lattice_second_u(h) ? p : nullptr;
}

// n steps through an even number of launches, (A, u) -> (B, u2) -> (A, u), A
// the buffer holding the angles at step k: the state ends where it started
// (after an odd number of steps the angle buffers so trade parities).  With
// `order` the launches also leave the partial sums of every step's order
// parameter there (launch_tile_order).
template <typename R>
static void lattice_tile_steps(xyl_lattice* h, const TilePlan& p, uint64_t n, double* order = nullptr) {
    const Lat<R> v = h->view<R>();
    const int parity = (int)((h->k + (uint64_t)h->cur) & 1);
    R* th[2] = {static_cast<R*>(h->th[parity]), static_cast<R*>(h->th[parity ^ 1])};
    R* u[2] = {static_cast<R*>(h->u), reinterpret_cast<R*>(h->u2.p)};
    const uint64_t nl = tile_launches(n, p.T);
    for (uint64_t i = 0; i < nl; ++i) {
        const int t = (int)(n / nl + (i < n % nl ? 1 : 0));
        const int a = (int)(i & 1);
        if (order) {
            launch_tile_order<R>(v, th[a], u[a], th[a ^ 1], u[a ^ 1], order, p, t, h->k, h->stream);
            order += (size_t)t * tile_order_parts(p);
        } else {
            launch_tile<R>(v, th[a], u[a], th[a ^ 1], u[a ^ 1], p, t, h->k, h->stream);
        }
        h->k += (uint64_t)t;
    }
    h->cur ^= (int)(n & 1);
    h->counter_valid = false;
}

// Advances n steps in the given mode.  With part_stride > 0 every step writes
// its measurement partials to part + (k - part_k0) * part_stride.
template <typename R>
static void lattice_steps_mode(xyl_lattice* h, uint64_t n, int mode, double* part, uint64_t part_k0,
                               uint64_t part_stride) {
    if (mode == kStore && part_stride == 0) {
        if (const TilePlan* p = lattice_tile_plan(h, n)) {
            lattice_tile_steps<R>(h, *p, n);
            return;
        }
    }
    if constexpr (sizeof(R) == 4) {
        MarchPlan mp;
        uint64_t m = mode == kStore && part_stride == 0 ? lattice_march_steps(h, n, &mp) : 0;
        if (m && lattice_second_u(h)) {
            // pairs of passes, (A, u) -> (B, u2) -> (A, u): six steps later A
            // again holds the angles of its parity
            Lat<float> v3 = h->view<float>();
            v3.k_base = 0;
            const int parity = (int)((h->k + (uint64_t)h->cur) & 1);
            float* A = static_cast<float*>(h->th[parity]);
            float* B = static_cast<float*>(h->th[parity ^ 1]);
            float* u = static_cast<float*>(h->u);
            float* u2 = reinterpret_cast<float*>(h->u2.p);
            for (n -= m; m > 0; m -= 2 * kMarchSteps) {
                launch_march(v3, MarchBuffers{A, u, B, u2}, mp, h->k, h->stream);
                launch_march(v3, MarchBuffers{B, u2, A, u}, mp, h->k + kMarchSteps, h->stream);
                h->k += 2 * kMarchSteps;
            }
            h->counter_valid = false;
            if (n == 0) return;
        }
        if (mode == kStore && part_stride == 0 && step2_eligible(h) && n >= 4 && lattice_second_u(h)) {
            Lat<float> v2 = h->view<float>();
            v2.k_base = 0;
            const uint64_t n4 = n - n % 4;
            uint64_t done = 0;
            int S = h->graph_steps - h->graph_steps % 4;
            if (S >= 4 && n4 >= (uint64_t)S && stream_captured(h)) S = 0;
            while (done < n4) {
                const int parity = (int)((h->k + (uint64_t)h->cur) & 1);
                if (S >= 4 && n4 - done >= (uint64_t)S) {
                    const int key = kStore | (2 << 8) | (parity << 10);
                    xyl_lattice::GraphEntry* ge = nullptr;
                    for (auto& g : h->graphs)
                        if (g.mode == key && g.S == S) ge = &g;
                    if (ge && ge->version != h->version) {
                        (void)hipGraphExecDestroy(ge->exec);
                        ge->exec = nullptr;
                    }
                    if (!ge) {
                        if (h->graphs.size() >= 8) destroy_graph(h);
                        h->graphs.push_back(xyl_lattice::GraphEntry());
                        ge = &h->graphs.back();
                        ge->mode = key;
                        ge->S = S;
                    }
                    if (!ge->exec) {
                        ge->exec = capture_steps2(h, v2, S, parity);
                        ge->version = h->version;
                    }
                    if (!h->counter_valid) {
                        launch_set_counter(h->kdev.p, h->k, h->stream);
                        h->counter_valid = true;
                    }
                    check_hip(hipGraphLaunch(ge->exec, h->stream), "hipGraphLaunch");
                    h->k += (uint64_t)S;
                    done += (uint64_t)S;
                } else {
                    const uint64_t m = std::min<uint64_t>(n4 - done, 4);
                    step2_launches(h, v2, m, nullptr, h->k, parity, h->stream);
                    h->k += m;
                    done += m;
                    h->counter_valid = false;
                }
            }
            n -= n4;
        }
    }
    Lat<R> v = h->view<R>();
    if (part_stride) {
        v.part = part;
        v.part_k0 = part_k0;
        v.part_stride = part_stride;
    }
    int S = h->graph_steps;
    if (S > 1 && n >= (uint64_t)S && stream_captured(h)) S = 0;
    while (n > 0) {
        if (S > 1 && n >= (uint64_t)S) {
            xyl_lattice::GraphEntry* ge = nullptr;
            for (auto& g : h->graphs)
                if (g.mode == mode && g.S == S && g.cur == h->cur && g.part == v.part && g.part_k0 == v.part_k0 &&
                    g.part_stride == v.part_stride)
                    ge = &g;
            if (ge && ge->version != h->version) {
                (void)hipGraphExecDestroy(ge->exec);
                ge->exec = nullptr;
            }
            if (!ge) {
                if (h->graphs.size() >= 8) destroy_graph(h);   // bound the cache
                h->graphs.push_back(xyl_lattice::GraphEntry());
                ge = &h->graphs.back();
                ge->mode = mode;
                ge->S = S;
                ge->cur = h->cur;
                ge->part = v.part;
                ge->part_k0 = v.part_k0;
                ge->part_stride = v.part_stride;
            }
            if (!ge->exec) {
                ge->exec = capture_steps<R>(h, v, mode, S);
                ge->version = h->version;
            }
            if (!h->counter_valid) {
                launch_set_counter(h->kdev.p, h->k, h->stream);
                h->counter_valid = true;
            }
            check_hip(hipGraphLaunch(ge->exec, h->stream), "hipGraphLaunch");
            h->k += (uint64_t)S;
            n -= (uint64_t)S;
        } else {
            launch_step<R>(v, mode, h->launch, nullptr, h->k, h->stream);
            h->k += 1;
            h->counter_valid = false;
            n -= 1;
        }
    }
}

template <typename R>
static void lattice_steps(xyl_lattice* h, uint64_t n) {
    lattice_steps_mode<R>(h, n, kStore, nullptr, 0, 0);
}

// Observables of the current step into obs_dev; with `part` only their partial
// sums there.
template <typename R>
static void lattice_measure_into(xyl_lattice* h, bool advance, double* obs_dev, double* part = nullptr) {
    lattice_launch_one<R>(h, advance ? (kStore | kMeasure) : kMeasure, part);
    if (!part) launch_finalize_obs(h->part.p, h->nrowparts(), (double)h->N, obs_dev, h->stream);
    if (advance) {
        h->k += 1;
        h->counter_valid = false;
    }
}

// Observables of the current step into obs_dev, then `span` >= 1 steps.
// Where two steps per pass apply and the span holds at least one pair of
// passes, or tiles do and it holds three steps, the sample is a measurement
// without a step (the same partial sums as a measured step) and every step of
// the span goes through the passes or tiles; otherwise the measured step
// advances one step and the rest follow (two steps on tiles are two launches
// beside the sample's: 48 steps of 64 x 6 sampled every 2 took 316 us so, 245
// with a measured step and a single one each).
template <typename R>
static void lattice_sample_and_advance(xyl_lattice* h, uint64_t span, double* obs_dev, double* part) {
    if ((span >= 4 && step2_eligible(h)) || (span >= 3 && lattice_tile_plan(h, span))) {
        lattice_measure_into<R>(h, false, obs_dev, part);
        lattice_steps<R>(h, span);
        return;
    }
    lattice_measure_into<R>(h, true, obs_dev, part);
    lattice_steps<R>(h, span - 1);
}

// A blown-up integration (dt far too large, say) shows up as non-finite
// values; calls that bring results to the host report it as XYL_ENUMERIC
// (the copied values are still written).
static void require_finite(const double* x, size_t n, const char* what) {
    for (size_t i = 0; i < n; ++i)
        if (!std::isfinite(x[i])) throw Error(XYL_ENUMERIC, std::string("non-finite ") + what + " (numeric fault)");
}

static void require_init(xyl_lattice* h) {
    require(h != nullptr, XYL_EINVAL, "NULL handle");
    require(h->initialized, XYL_ESTATE, "lattice state not initialised (call an init or set_state first)");
}

template <typename R>
static void to_host(const void* dev, double* host, size_t n, hipStream_t s) {
    std::vector<R> tmp(n);
    check_hip(hipMemcpyAsync(tmp.data(), dev, sizeof(R) * n, hipMemcpyDeviceToHost, s), "hipMemcpyAsync D2H");
    check_hip(hipStreamSynchronize(s), "hipStreamSynchronize");
    for (size_t i = 0; i < n; ++i) host[i] = (double)tmp[i];
}

template <typename R>
static void to_device(void* dev, const double* host, size_t n, hipStream_t s) {
    std::vector<R> tmp(n);
    for (size_t i = 0; i < n; ++i) tmp[i] = (R)host[i];
    check_hip(hipMemcpyAsync(dev, tmp.data(), sizeof(R) * n, hipMemcpyHostToDevice, s), "hipMemcpyAsync H2D");
    check_hip(hipStreamSynchronize(s), "hipStreamSynchronize");
}

template <typename R>
static void lattice_omega(xyl_lattice* h, double* omega) {
    if (h->k == h->fresh_k) {
        to_host<R>(h->u, omega, h->N, h->stream);
        return;
    }
    h->omega_buf.reserve(sizeof(R) * h->N);
    lattice_launch_one<R>(h, kOmega);
    to_host<R>(h->omega_buf.p, omega, h->N, h->stream);
}

template <typename R>
static void run_domains(const R* th, int Lx, int Ly, int sx, int sy, int model, DomainBufs& w, hipStream_t s,
                        int32_t* labels, uint64_t* sizes, uint64_t* counts, uint64_t cap, uint64_t* n_sizes,
                        uint64_t* n_domains, uint64_t* max_size) {
    const size_t N = (size_t)Lx * Ly;
    const uint32_t pcap = domain_size_cap(N);
    const size_t nst = kDomainPairs + 2 * (size_t)pcap;
    w.parent.reserve(N);
    w.size.reserve(N);
    w.hist.reserve(N + 1);
    w.stats.reserve(nst);
    w.stats_host.reserve(nst);
    launch_domains<R>(th, Lx, Ly, sx, sy, model, w.parent.p, w.size.p, w.hist.p, w.stats.p, s);
    // the (size, count) pairs were compacted on the device: only they come back
    const uint32_t* st = w.stats_host.p;
    check_hip(hipMemcpyAsync(w.stats_host.p, w.stats.p, sizeof(uint32_t) * nst, hipMemcpyDeviceToHost, s), "D2H");
    if (labels) w.labels.copy(labels, w.parent.p, sizeof(int32_t) * N, s);
    else check_hip(hipStreamSynchronize(s), "hipStreamSynchronize");
    const uint64_t ns = st[0];
    require(ns >= 1 && ns <= pcap, XYL_EDEVICE, "domain size distribution overflowed its bound");
    std::vector<std::pair<uint32_t, uint32_t>> pairs(ns);
    for (uint64_t j = 0; j < ns; ++j) pairs[j] = {st[kDomainPairs + 2 * j], st[kDomainPairs + 2 * j + 1]};
    std::sort(pairs.begin(), pairs.end());
    if (sizes || counts) require(cap >= ns, XYL_EINVAL, "size-distribution capacity too small");
    uint64_t nd = 0, covered = 0;
    for (uint64_t j = 0; j < ns; ++j) {
        if (sizes) sizes[j] = pairs[j].first;
        if (counts) counts[j] = pairs[j].second;
        nd += pairs[j].second;
        covered += (uint64_t)pairs[j].first * pairs[j].second;
    }
    require(covered == N, XYL_EDEVICE, "domain sizes do not cover the lattice");
    if (n_sizes) *n_sizes = ns;
    if (n_domains) *n_domains = nd;
    if (max_size) *max_size = pairs[ns - 1].first;
}


#define DISPATCH(dt, FN, ...) ((dt) == XYL_F64 ? FN<double>(__VA_ARGS__) : FN<float>(__VA_ARGS__))

extern "C" {

int xyl_device_count(void) {
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess) return 0;
    int m = 0;
    for (int d = 0; d < n; ++d)
        if (is_gfx950(d)) ++m;
    return m;
}

// The path that xyl_autotune chose in this process for such a lattice, else the
// rules'.
static void apply_tuned_path(xyl_lattice* h) {
    if (h->own_path) return;
    Tuned2 t;
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        auto it = g_tuned2.find({h->Lx, h->Ly, h->dtype, h->p.model, (int)kick_factored(h->p)});
        if (it != g_tuned2.end()) t = it->second;
    }
    h->fusion = t.fusion;
    h->step2_rows_tuned = t.rows;
    h->step2_tw_tuned = t.tile_waves;
    if (h->tiles != t.tiles || h->march != t.march) h->tile_plans.clear();
    h->tiles = t.tiles;
    h->march = t.march;
}

static int create_impl(xyl_lattice** out, int32_t Lx, int32_t Ly, int32_t dtype, int32_t device, void* ta, void* tb,
                       void* vel) {
    return guarded([&] {
        require(out != nullptr, XYL_EINVAL, "out is NULL");
        *out = nullptr;
        require(dtype == XYL_F32 || dtype == XYL_F64, XYL_EINVAL, "dtype must be XYL_F32 or XYL_F64");
        validate_shape(Lx, Ly);
        select_device(device);
        std::unique_ptr<xyl_lattice> h(new xyl_lattice());
        h->dtype = dtype;
        h->device = device;
        check_hip(hipDeviceGetAttribute(&h->cus, hipDeviceAttributeMultiprocessorCount, device), "hipDeviceGetAttribute");
        h->Lx = Lx;
        h->Ly = Ly;
        h->N = (size_t)Lx * Ly;
        load_stepping_kernels(device);
        const uint64_t k0[1] = {0};
        const double T0[1] = {0.0};
        h->sched = make_schedule(k0, T0, 1);
        if (ta) {
            require(tb && vel && ta != tb && ta != vel && tb != vel, XYL_EINVAL, "wrapped buffers must be distinct");
            h->owns = false;
            h->th[0] = ta;
            h->th[1] = tb;
            h->u = vel;
        } else {
            const size_t bytes = elem_size(dtype) * h->N;
            for (int b = 0; b < 2; ++b) check_alloc(hipMalloc(&h->th[b], bytes), "hipMalloc theta");
            check_alloc(hipMalloc(&h->u, bytes), "hipMalloc velocity");
        }
        check_hip(hipStreamCreateWithFlags(&h->cap_stream, hipStreamNonBlocking), "hipStreamCreate");
        h->kdev.reserve(1);
        h->part.reserve(part_elems(h->nrowparts()));
        h->phases.reserve(2 * ((size_t)Lx + Ly));
        launch_phase_table(h->phases.p, Lx, nullptr);
        launch_phase_table(h->phases.p + 2 * (size_t)Lx, Ly, nullptr);
        check_hip(hipStreamSynchronize(nullptr), "hipStreamSynchronize");
        h->obs.reserve(16 * 6);
        h->launch = default_launch(Lx, Ly);
        {
            std::lock_guard<std::mutex> lk(g_tune_mu);
            auto it = g_tuned.find({Lx, Ly, dtype});
            if (it != g_tuned.end()) h->launch = it->second;
            auto itm = g_tunedm.find({Lx, Ly, dtype});
            if (itm != g_tunedm.end()) {
                h->mlaunch = itm->second;
                h->mlaunch_tuned = true;
            }
        }
        apply_tuned_path(h.get());
        *out = h.release();
    });
}

int xyl_create(xyl_lattice** out, int32_t Lx, int32_t Ly, int32_t dtype, int32_t device) {
    return create_impl(out, Lx, Ly, dtype, device, nullptr, nullptr, nullptr);
}

int xyl_create_wrapped(xyl_lattice** out, int32_t Lx, int32_t Ly, int32_t dtype, int32_t device, void* theta_a,
                       void* theta_b, void* vel) {
    if (!theta_a || !theta_b || !vel) {
        g_err = "wrapped buffers must be non-NULL";
        return XYL_EINVAL;
    }
    return create_impl(out, Lx, Ly, dtype, device, theta_a, theta_b, vel);
}

int xyl_destroy(xyl_lattice* h) {
    if (!h) return XYL_OK;
    return guarded([&] {
        DeviceGuard g(h->device);
        (void)hipStreamSynchronize(h->stream);
        destroy_graph(h);
        adjoint_release(h);
        if (h->owns) {
            for (int b = 0; b < 2; ++b)
                if (h->th[b]) (void)hipFree(h->th[b]);
            if (h->u) (void)hipFree(h->u);
        }
        if (h->cap_stream) (void)hipStreamDestroy(h->cap_stream);
        delete h;
    });
}

int xyl_set_stream(xyl_lattice* h, void* stream) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        h->stream = static_cast<hipStream_t>(stream);
    });
}

int xyl_set_params(xyl_lattice* h, double Jx, double Jy, double hf, double gamma, double dt) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        Params p = h->p;
        p.Jx = Jx;
        p.Jy = Jy;
        p.h = hf;
        p.gamma = gamma;
        p.dt = dt;
        validate_params(p);
        h->p = p;
        apply_tuned_path(h);
        h->touch();
    });
}

int xyl_set_model(xyl_lattice* h, int32_t model, double pfield) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        validate_model(model, pfield);
        if (model != h->p.model) h->initialized = false;   // the angle ranges differ
        h->p.model = model;
        h->p.p = pfield;
        apply_tuned_path(h);
        h->touch();
    });
}

int xyl_set_schedule(xyl_lattice* h, const uint64_t* ks, const double* Ts, int32_t n) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        h->sched = make_schedule(ks, Ts, n);
        h->touch();
    });
}

int xyl_set_schedule_shaped(xyl_lattice* h, const uint64_t* ks, const double* Ts, const int32_t* gs, int32_t n) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        require(gs != nullptr, XYL_EINVAL, "shape array is NULL");
        h->sched = make_schedule(ks, Ts, n, gs);
        h->touch();
    });
}

int xyl_set_seed(xyl_lattice* h, uint64_t seed, uint32_t replica) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        h->seed = seed;
        h->replica = replica;
        h->touch();
    });
}

int xyl_init_random(xyl_lattice* h) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        DeviceGuard g(h->device);
        h->k = 0;
        h->fresh_k = 0;
        h->cur = 0;
        h->counter_valid = false;
        h->touch();
        if (h->dtype == XYL_F64) launch_init_random<double>(h->view<double>(), h->stream);
        else launch_init_random<float>(h->view<float>(), h->stream);
        h->initialized = true;
    });
}

// Host values for the state precision: finite, |th| <= 3 pi, and for the half
// circle inside [-pi_p/2, pi_p/2) after rounding to the state precision.
static void validate_host_state(const xyl_lattice* h, const double* theta, const double* vel, const char* vname) {
    const bool si = h->p.model == kModelSI;
    const double wp = h->dtype == XYL_F64 ? Prec<double>::kHalfPi : (double)Prec<float>::kHalfPi;
    for (size_t i = 0; i < h->N; ++i) {
        require(std::isfinite(theta[i]) && std::fabs(theta[i]) <= 3.0 * M_PI, XYL_EINVAL,
                "theta entries must be finite with |theta| <= 3 pi");
        if (si) {
            const double t = h->dtype == XYL_F64 ? theta[i] : (double)(float)theta[i];
            require(t >= -wp && t < wp, XYL_EINVAL, "theta entries must lie in [-pi/2, pi/2) for the SI model");
        }
        require(std::isfinite(vel[i]), XYL_EINVAL, std::string(vname) + " entries must be finite");
    }
}

int xyl_set_state(xyl_lattice* h, const double* theta, const double* omega, uint64_t step) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        require(theta != nullptr && omega != nullptr, XYL_EINVAL, "theta/omega are NULL");
        // SI: the field is evaluated on the raw angle, so the state must already
        // lie in the half circle [-pi_p/2, pi_p/2) of the state precision
        validate_host_state(h, theta, omega, "omega");
        DeviceGuard g(h->device);
        h->k = step;
        h->fresh_k = step;
        h->counter_valid = false;
        h->touch();
        if (h->dtype == XYL_F64) {
            to_device<double>(h->cur_theta(), theta, h->N, h->stream);
            to_device<double>(h->u, omega, h->N, h->stream);
        } else {
            to_device<float>(h->cur_theta(), theta, h->N, h->stream);
            to_device<float>(h->u, omega, h->N, h->stream);
        }
        h->initialized = true;
    });
}

int xyl_get_raw_state(xyl_lattice* h, double* theta, double* u, uint64_t* step, int32_t* fresh) {
    return guarded([&] {
        require_init(h);
        DeviceGuard g(h->device);
        if (theta) {
            if (h->dtype == XYL_F64) to_host<double>(h->cur_theta(), theta, h->N, h->stream);
            else to_host<float>(h->cur_theta(), theta, h->N, h->stream);
        }
        if (u) {
            if (h->dtype == XYL_F64) to_host<double>(h->u, u, h->N, h->stream);
            else to_host<float>(h->u, u, h->N, h->stream);
        }
        if (step) *step = h->k;
        if (fresh) *fresh = h->k == h->fresh_k ? 1 : 0;
        if (theta) require_finite(theta, h->N, "angles");
        if (u) require_finite(u, h->N, "velocities");
    });
}

int xyl_set_raw_state(xyl_lattice* h, const double* theta, const double* u, uint64_t step, int32_t fresh) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        require(theta != nullptr && u != nullptr, XYL_EINVAL, "theta/u are NULL");
        require(fresh == 0 || fresh == 1, XYL_EINVAL, "fresh must be 0 or 1");
        validate_host_state(h, theta, u, "u");
        DeviceGuard g(h->device);
        h->k = step;
        // a stored half-step velocity is never the synchronized one again
        h->fresh_k = fresh ? step : ~(uint64_t)0;
        h->counter_valid = false;
        h->touch();
        if (h->dtype == XYL_F64) {
            to_device<double>(h->cur_theta(), theta, h->N, h->stream);
            to_device<double>(h->u, u, h->N, h->stream);
        } else {
            to_device<float>(h->cur_theta(), theta, h->N, h->stream);
            to_device<float>(h->u, u, h->N, h->stream);
        }
        h->initialized = true;
    });
}

int xyl_set_state_device(xyl_lattice* h, const void* theta, const void* omega, int32_t dtype, uint64_t step) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        require(theta != nullptr && omega != nullptr, XYL_EINVAL, "theta/omega are NULL");
        require(dtype == XYL_F32 || dtype == XYL_F64, XYL_EINVAL, "dtype must be XYL_F32 or XYL_F64");
        DeviceGuard g(h->device);
        const int src64 = dtype == XYL_F64 ? 1 : 0, st64 = h->dtype == XYL_F64 ? 1 : 0;
        // validate where the state lies; only the verdict comes back
        h->flag.reserve(1);
        launch_fill_u32(h->flag.p, 1, 0u, h->stream);
        launch_check_state(theta, omega, src64, h->N, h->p.model == kModelSI ? 1 : 0, st64, h->flag.p, h->stream);
        uint32_t bad = 0;
        check_hip(hipMemcpyAsync(&bad, h->flag.p, sizeof(bad), hipMemcpyDeviceToHost, h->stream), "D2H");
        check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
        require(!(bad & kStateBadTheta), XYL_EINVAL, "theta entries must be finite with |theta| <= 3 pi");
        require(!(bad & kStateBadOmega), XYL_EINVAL, "omega entries must be finite");
        require(!(bad & kStateBadHalfCircle), XYL_EINVAL, "theta entries must lie in [-pi/2, pi/2) for the SI model");
        h->k = step;
        h->fresh_k = step;
        h->counter_valid = false;
        h->touch();
        launch_convert(theta, src64, h->cur_theta(), st64, h->N, 1.0, false, h->stream);
        launch_convert(omega, src64, h->u, st64, h->N, 1.0, false, h->stream);
        // the caller may release or rewrite its buffers once this returns
        check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
        h->initialized = true;
    });
}

int xyl_init_ordered(xyl_lattice* h, int32_t sign) {
    if (!h) {
        g_err = "NULL handle";
        return XYL_EINVAL;
    }
    std::vector<double> th(h->N), om(h->N, 0.0);
    const double pi_p = h->dtype == XYL_F64 ? Prec<double>::kPi : (double)Prec<float>::kPi;
    // SI: the field -h cos(p th) with h < 0 is lowest at th = +-pi/p
    const double th0 = (h->p.h < 0.0 && h->p.p > 2.0) ? M_PI / h->p.p : 0.0;
    const int sx = h->p.Jx > 0.0, sy = h->p.Jy > 0.0;
    for (int y = 0; y < h->Ly; ++y)
        for (int x = 0; x < h->Lx; ++x) {
            int e = ((x * sx + y * sy) & 1) ? -1 : 1;
            if (sign < 0) e = -e;
            if (h->p.model == kModelSI) th[(size_t)y * h->Lx + x] = e > 0 ? th0 : -th0;
            else th[(size_t)y * h->Lx + x] = e > 0 ? 0.0 : -pi_p;
        }
    return xyl_set_state(h, th.data(), om.data(), 0);
}

int xyl_get_state(xyl_lattice* h, double* theta, double* omega, uint64_t* step) {
    return guarded([&] {
        require_init(h);
        DeviceGuard g(h->device);
        if (theta) {
            if (h->dtype == XYL_F64) to_host<double>(h->cur_theta(), theta, h->N, h->stream);
            else to_host<float>(h->cur_theta(), theta, h->N, h->stream);
        }
        if (omega) {
            if (h->dtype == XYL_F64) lattice_omega<double>(h, omega);
            else lattice_omega<float>(h, omega);
        }
        if (step) *step = h->k;
        if (theta) require_finite(theta, h->N, "angles");
        if (omega) require_finite(omega, h->N, "velocities");
    });
}

int xyl_state_buffers(xyl_lattice* h, void** theta, void** vel, int32_t* fresh) {
    return guarded([&] {
        require_init(h);
        if (theta) *theta = h->cur_theta();
        if (vel) *vel = h->u;
        if (fresh) *fresh = h->k == h->fresh_k ? 1 : 0;
    });
}

int xyl_step(xyl_lattice* h, uint64_t nsteps) {
    return guarded([&] {
        require_init(h);
        DeviceGuard g(h->device);
        if (h->dtype == XYL_F64) lattice_steps<double>(h, nsteps);
        else lattice_steps<float>(h, nsteps);
    });
}

int xyl_step_measured(xyl_lattice* h, uint64_t nsteps, uint64_t every, xyl_obs* out, uint64_t cap, uint64_t* nout) {
    return guarded([&] {
        require_init(h);
        require(every >= 1, XYL_EINVAL, "every must be >= 1");
        require(out != nullptr, XYL_EINVAL, "out is NULL");
        const uint64_t ns = nsteps / every + 1;
        require(cap >= ns, XYL_EINVAL, "sample capacity too small");
        DeviceGuard g(h->device);
        h->obs.reserve(6 * ns);
        h->obs_host.reserve(6 * ns);
        // Where one workgroup reduces a sample (a 3.6 us launch each), the
        // partial sums of up to kSampleBatch samples wait for one launch that
        // reduces them all, one workgroup each (the same sums).
        constexpr uint64_t kSampleBatch = 64;
        const size_t stride = (size_t)h->nrowparts() * kNPart;
        const uint64_t batch = h->nrowparts() <= kFinalizeSplit && ns > 1 ? std::min<uint64_t>(ns, kSampleBatch) : 0;
        if (batch) h->samples.reserve(batch * stride);
        for (uint64_t j = 0; j < ns; ++j) {
            double* o = h->obs.p + 6 * j;
            double* part = batch ? h->samples.p + (j % batch) * stride : nullptr;
            if (batch && j && j % batch == 0)
                launch_finalize_many(h->samples.p, h->nrowparts(), stride, (double)h->N, o - 6 * batch, (int)batch,
                                     h->stream);
            if (j * every == nsteps) {
                // a sample at the last step: measured without stepping
                if (h->dtype == XYL_F64) lattice_measure_into<double>(h, false, o, part);
                else lattice_measure_into<float>(h, false, o, part);
            } else {
                // up to the next sample, or to the end (nsteps not a multiple of every)
                const uint64_t span = std::min<uint64_t>(every, nsteps - j * every);
                if (h->dtype == XYL_F64) lattice_sample_and_advance<double>(h, span, o, part);
                else lattice_sample_and_advance<float>(h, span, o, part);
            }
        }
        if (batch) {
            const uint64_t last = (ns - 1) % batch + 1;
            launch_finalize_many(h->samples.p, h->nrowparts(), stride, (double)h->N, h->obs.p + 6 * (ns - last),
                                 (int)last, h->stream);
        }
        check_hip(hipMemcpyAsync(h->obs_host.p, h->obs.p, sizeof(double) * 6 * ns, hipMemcpyDeviceToHost, h->stream),
                  "D2H");
        check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
        std::memcpy(out, h->obs_host.p, sizeof(double) * 6 * ns);
        if (nout) *nout = ns;
        require_finite(reinterpret_cast<const double*>(out), 6 * ns, "observables");
    });
}

int xyl_step_adaptive(xyl_lattice* h, uint64_t nsteps, uint64_t ds0, uint64_t ds_min, uint64_t ds_max, int32_t which,
                      uint64_t block, xyl_obs* out, uint64_t* steps, uint64_t cap, uint64_t* nout) {
    return guarded([&] {
        require_init(h);
        require(out != nullptr && steps != nullptr, XYL_EINVAL, "out/steps are NULL");
        require(ds_min >= 1 && ds_min <= ds0 && ds0 <= ds_max, XYL_EINVAL, "need 1 <= ds_min <= ds0 <= ds_max");
        require(which >= 0 && which < 6, XYL_EINVAL, "which must index an observable (0..5)");
        require(block >= 4, XYL_EINVAL, "block must be >= 4 samples");
        require(cap >= nsteps / ds_min + 2, XYL_EINVAL, "cap must be >= nsteps / ds_min + 2");
        DeviceGuard g(h->device);
        h->obs.reserve(6 * block);
        const uint64_t kend = h->k + nsteps;
        uint64_t ds = ds0, n = 0;
        std::vector<double> vals;
        vals.reserve(block);
        // samples are measured into a device block and copied out when it is
        // full (the spacing decision needs them) or at the end
        uint64_t in_dev = 0;
        auto flush = [&]() {
            if (!in_dev) return;
            check_hip(hipMemcpyAsync(out + (n - in_dev), h->obs.p, sizeof(double) * 6 * in_dev,
                                     hipMemcpyDeviceToHost, h->stream),
                      "D2H");
            check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
            in_dev = 0;
        };
        auto sample = [&](bool advance) {
            if (in_dev == block) flush();
            steps[n] = h->k;
            if (h->dtype == XYL_F64) lattice_measure_into<double>(h, advance, h->obs.p + 6 * in_dev);
            else lattice_measure_into<float>(h, advance, h->obs.p + 6 * in_dev);
            ++in_dev;
            ++n;
        };
        uint64_t blk = 0;   // samples in the current block (equal spacing)
        while (true) {
            const bool last = h->k == kend;
            sample(!last);   // measures at k and, unless last, advances one step
            ++blk;
            if (last) break;
            if (blk == block) {
                // the block's series of the chosen observable decides the
                // spacing from here on: ds' = ds tau / 10 with tau in samples
                // (App. B: ds ~ tau_C / 10)
                flush();
                vals.assign(block, 0.0);
                const xyl_obs* o = out + (n - block);
                for (uint64_t i = 0; i < block; ++i) vals[i] = reinterpret_cast<const double*>(o + i)[which];
                const double tau = tau_int(vals.data(), block);
                const double want = std::floor((double)ds * tau / 10.0 + 0.5);
                ds = (uint64_t)std::min<double>(std::max<double>(want, (double)ds_min), (double)ds_max);
                blk = 0;
            }
            const uint64_t adv = std::min<uint64_t>(ds, kend - (h->k - 1));
            if (adv > 1) {
                if (h->dtype == XYL_F64) lattice_steps<double>(h, adv - 1);
                else lattice_steps<float>(h, adv - 1);
            }
        }
        flush();
        if (nout) *nout = n;
        require_finite(reinterpret_cast<const double*>(out), 6 * n, "observables");
    });
}

int xyl_measure(xyl_lattice* h, xyl_obs* out) {
    return guarded([&] {
        require_init(h);
        require(out != nullptr, XYL_EINVAL, "out is NULL");
        DeviceGuard g(h->device);
        h->obs.reserve(6);
        h->obs_host.reserve(6);
        if (h->dtype == XYL_F64) lattice_measure_into<double>(h, false, h->obs.p);
        else lattice_measure_into<float>(h, false, h->obs.p);
        check_hip(hipMemcpyAsync(h->obs_host.p, h->obs.p, sizeof(double) * 6, hipMemcpyDeviceToHost, h->stream), "D2H");
        check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
        std::memcpy(out, h->obs_host.p, sizeof(double) * 6);
        require_finite(reinterpret_cast<const double*>(out), 6, "observables");
    });
}

int xyl_correlation(xyl_lattice* h, int32_t axis, int32_t rmax, double* C) {
    return guarded([&] {
        require_init(h);
        require(axis == 0 || axis == 1, XYL_EINVAL, "axis must be 0 or 1");
        const int L = axis == 0 ? h->Lx : h->Ly;
        require(rmax >= 0 && rmax <= L / 2, XYL_EINVAL, "rmax must be in [0, L/2]");
        require(L <= 4096, XYL_EUNSUPPORTED, "correlation needs the axis length <= 4096");
        require(C != nullptr, XYL_EINVAL, "C is NULL");
        DeviceGuard g(h->device);
        const size_t nscr = correlation_scratch(h->Lx, h->Ly, axis, rmax);
        SpectrumBufs& w = h->spectrum;
        w.scratch.reserve(nscr + (rmax + 1));
        w.host.reserve(rmax + 1);
        const double* tw = w.table(L, h->stream);
        double* outd = w.scratch.p + nscr;
        const int sx = h->p.Jx > 0.0, sy = h->p.Jy > 0.0;
        if (h->dtype == XYL_F64)
            launch_correlation<double>(static_cast<const double*>(h->cur_theta()), h->Lx, h->Ly, sx, sy, h->p.model,
                                       axis, rmax, tw, w.scratch.p, outd, h->stream);
        else
            launch_correlation<float>(static_cast<const float*>(h->cur_theta()), h->Lx, h->Ly, sx, sy, h->p.model,
                                      axis, rmax, tw, w.scratch.p, outd, h->stream);
        check_hip(hipMemcpyAsync(w.host.p, outd, sizeof(double) * (rmax + 1), hipMemcpyDeviceToHost, h->stream), "D2H");
        check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
        std::memcpy(C, w.host.p, sizeof(double) * (rmax + 1));
    });
}

}  // extern "C"

// S_delta(k) of one lattice's current angles into host S[0..kmax].
template <typename R>
static void structure_factor_into(const void* th, int Lx, int Ly, int sx, int sy, int model, int axis, int kmax,
                                  SpectrumBufs& w, hipStream_t s, double* S) {
    const size_t nscr = structure_factor_scratch(Lx, Ly, axis, kmax);
    w.scratch.reserve(nscr + (kmax + 1));
    w.host.reserve(kmax + 1);
    const double* tw = w.table(axis == 0 ? Lx : Ly, s);
    double* outd = w.scratch.p + nscr;
    launch_structure_factor<R>(static_cast<const R*>(th), Lx, Ly, sx, sy, model, axis, kmax, tw, w.scratch.p, outd, s);
    check_hip(hipMemcpyAsync(w.host.p, outd, sizeof(double) * (kmax + 1), hipMemcpyDeviceToHost, s), "D2H");
    check_hip(hipStreamSynchronize(s), "hipStreamSynchronize");
    std::memcpy(S, w.host.p, sizeof(double) * (kmax + 1));
    require_finite(S, (size_t)kmax + 1, "structure factor");
}

static void validate_sf(int Lx, int Ly, int axis, int kmax, const double* S) {
    require(axis == 0 || axis == 1, XYL_EINVAL, "axis must be 0 or 1");
    const int L = axis == 0 ? Lx : Ly;
    require(kmax >= 0 && kmax <= L / 2, XYL_EINVAL, "kmax must be in [0, L/2]");
    require(L <= 4096, XYL_EUNSUPPORTED, "the structure factor needs the axis length <= 4096");
    require(S != nullptr, XYL_EINVAL, "S is NULL");
}


extern "C" {

int xyl_structure_factor(xyl_lattice* h, int32_t axis, int32_t kmax, double* S) {
    return guarded([&] {
        require_init(h);
        validate_sf(h->Lx, h->Ly, axis, kmax, S);
        DeviceGuard g(h->device);
        const int sx = h->p.Jx > 0.0, sy = h->p.Jy > 0.0;
        if (h->dtype == XYL_F64)
            structure_factor_into<double>(h->cur_theta(), h->Lx, h->Ly, sx, sy, h->p.model, axis, kmax, h->spectrum,
                                          h->stream, S);
        else
            structure_factor_into<float>(h->cur_theta(), h->Lx, h->Ly, sx, sy, h->p.model, axis, kmax, h->spectrum,
                                         h->stream, S);
    });
}


int xyl_domains(xyl_lattice* h, int32_t* labels, uint64_t* sizes, uint64_t* counts, uint64_t cap, uint64_t* n_sizes,
                uint64_t* n_domains, uint64_t* max_size) {
    return guarded([&] {
        require_init(h);
        DeviceGuard g(h->device);
        const int sx = h->p.Jx > 0.0, sy = h->p.Jy > 0.0;
        if (h->dtype == XYL_F64)
            run_domains<double>(static_cast<const double*>(h->cur_theta()), h->Lx, h->Ly, sx, sy, h->p.model,
                                h->domains, h->stream, labels, sizes, counts, cap, n_sizes, n_domains, max_size);
        else
            run_domains<float>(static_cast<const float*>(h->cur_theta()), h->Lx, h->Ly, sx, sy, h->p.model,
                               h->domains, h->stream, labels, sizes, counts, cap, n_sizes, n_domains, max_size);
    });
}

}  // extern "C"

// ----------------------------------------------- allocation-free domains
// Scratch of xyl_domains_noalloc, the domain labelling for callers that cannot
// allocate device memory: the union-find's parent, cluster-size and histogram
// arrays and its (size, count) pair list for lattices of up to
// kNoAllocMaxSites sites, 3 * 4 * 2^22 + 4 * (5 + 2 * 4096) bytes (about
// 48 MiB).  Each device the library runs on holds one copy until the process
// ends.  Host code never names the array itself (there it is a host-side
// stand-in): it uses the device address hipGetSymbolAddress returns, looked up
// once per device with that device current.
constexpr size_t kNoAllocMaxSites = size_t(1) << 22;
constexpr size_t kNoAllocMaxPairs = 4096;
constexpr size_t kNoAllocWords = 3 * kNoAllocMaxSites + 1 + kDomainPairs + 2 * kNoAllocMaxPairs;
static __device__ __align__(256) uint32_t scratch[kNoAllocWords];

constexpr int kNoAllocMaxDevices = 64;
static std::mutex g_scratch_mu;                         // one call at a time in this process
static uint32_t* g_scratch_dev[kNoAllocMaxDevices] = {};

// Device address of `scratch` on device dev (current); g_scratch_mu held.
static uint32_t* scratch_address(int dev) {
    require(dev >= 0 && dev < kNoAllocMaxDevices, XYL_EUNSUPPORTED, "device index beyond the scratch table");
    if (!g_scratch_dev[dev]) {
        uint32_t* ptr = nullptr;
        check_hip(hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
        require(ptr != nullptr, XYL_EDEVICE, "hipGetSymbolAddress returned no address for the scratch array");
        g_scratch_dev[dev] = ptr;
    }
    return g_scratch_dev[dev];
}

// xyl_domains on the static scratch: cleared by the kernels (no memset), results
// read back into the caller's arrays and a fixed stack buffer (no heap).
template <typename R>
static void domains_noalloc(xyl_lattice* h, int32_t* labels, uint64_t* sizes, uint64_t* counts, uint64_t cap,
                            uint64_t* n_sizes, uint64_t* n_domains, uint64_t* max_size) {
    const size_t N = h->N;
    const uint32_t pcap = domain_size_cap(N);
    require(pcap <= kNoAllocMaxPairs, XYL_EDEVICE, "size-distribution bound exceeds the scratch");
    hipStream_t s = h->stream;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    uint32_t* base = scratch_address(h->device);
    int32_t* parent = reinterpret_cast<int32_t*>(base);
    uint32_t* usz = base + N;
    uint32_t* hist = base + 2 * N;
    uint32_t* stats = base + 3 * N + 1;
    const int sx = h->p.Jx > 0.0, sy = h->p.Jy > 0.0;
    launch_domains<R>(static_cast<const R*>(h->cur_theta()), h->Lx, h->Ly, sx, sy, h->p.model, parent, usz, hist,
                      stats, s);
    uint32_t head[kDomainPairs];
    check_hip(hipMemcpyAsync(head, stats, sizeof(head), hipMemcpyDeviceToHost, s), "D2H");
    if (labels) check_hip(hipMemcpyAsync(labels, parent, sizeof(int32_t) * N, hipMemcpyDeviceToHost, s), "D2H");
    check_hip(hipStreamSynchronize(s), "hipStreamSynchronize");
    const uint64_t ns = head[0];
    require(ns >= 1 && ns <= pcap, XYL_EDEVICE, "domain size distribution overflowed its bound");
    if (sizes || counts) require(cap >= ns, XYL_EINVAL, "size-distribution capacity too small");
    // (size, count) pairs as two 32-bit words each; sorted by size as 64-bit
    // keys size << 32 | count (sizes are distinct)
    uint64_t pairs[kNoAllocMaxPairs];
    check_hip(hipMemcpyAsync(pairs, stats + kDomainPairs, sizeof(uint32_t) * 2 * ns, hipMemcpyDeviceToHost, s),
              "D2H");
    check_hip(hipStreamSynchronize(s), "hipStreamSynchronize");
    for (uint64_t j = 0; j < ns; ++j) {
        uint32_t w[2];
        std::memcpy(w, &pairs[j], sizeof(w));
        pairs[j] = ((uint64_t)w[0] << 32) | (uint64_t)w[1];
    }
    std::sort(pairs, pairs + ns);
    uint64_t nd = 0, covered = 0;
    for (uint64_t j = 0; j < ns; ++j) {
        const uint64_t sz = pairs[j] >> 32, ct = pairs[j] & 0xFFFFFFFFull;
        if (sizes) sizes[j] = sz;
        if (counts) counts[j] = ct;
        nd += ct;
        covered += sz * ct;
    }
    require(covered == N, XYL_EDEVICE, "domain sizes do not cover the lattice");
    if (n_sizes) *n_sizes = ns;
    if (n_domains) *n_domains = nd;
    if (max_size) *max_size = pairs[ns - 1] >> 32;
}

extern "C" {

int xyl_domains_noalloc(xyl_lattice* h, int32_t* labels, uint64_t* sizes, uint64_t* counts, uint64_t cap,
                        uint64_t* n_sizes, uint64_t* n_domains, uint64_t* max_size) {
    return guarded([&] {
        require_init(h);
        require(h->N <= kNoAllocMaxSites, XYL_EINVAL,
                "xyl_domains_noalloc takes lattices of at most 2^22 sites (its static scratch)");
        DeviceGuard g(h->device);
        if (h->dtype == XYL_F64) domains_noalloc<double>(h, labels, sizes, counts, cap, n_sizes, n_domains, max_size);
        else domains_noalloc<float>(h, labels, sizes, counts, cap, n_sizes, n_domains, max_size);
    });
}

int xyl_sync(xyl_lattice* h) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        DeviceGuard g(h->device);
        check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
    });
}

int xyl_set_launch(xyl_lattice* h, int32_t rows, int32_t wpb) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        Launch l = h->launch;
        if (rows) l.rows = rows;
        if (wpb) l.wpb = wpb;
        validate_launch(l);
        h->launch = l;
        h->touch();
    });
}

int xyl_get_launch(xyl_lattice* h, int32_t* rows, int32_t* wpb) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        if (rows) *rows = h->launch.rows;
        if (wpb) *wpb = h->launch.wpb;
    });
}

}  // extern "C"

// Times the single-step launch shapes, for FP32 lattices of a shape the
// two-step pass takes that pass at several strip heights, the three-step pass
// and tiles; returns the best single-step shape and sets *t to the fastest path
// (fusion 1: single steps) with the best two-step shape (rows 0 if none).
template <typename R>
static Launch autotune_impl(xyl_lattice* h, Tuned2* t, Launch* mlaunch) {
    int *fusion = &t->fusion, *rows2 = &t->rows, *tw2 = &t->tile_waves;
    // time candidates on scratch copies so the lattice state is untouched;
    // each candidate runs as a captured graph of back-to-back steps, so the
    // host's launch overhead does not mask kernel time on small lattices
    const size_t bytes = sizeof(R) * h->N;
    DevBuf<char> tmp;
    tmp.reserve(4 * bytes);
    DevBuf<uint64_t> kc;
    kc.reserve(1);
    Lat<R> v = h->view<R>();
    v.th[0] = reinterpret_cast<R*>(tmp.p);
    v.th[1] = reinterpret_cast<R*>(tmp.p + bytes);
    v.u = reinterpret_cast<R*>(tmp.p + 2 * bytes);
    check_hip(hipMemcpyAsync(v.th[0], h->cur_theta(), bytes, hipMemcpyDeviceToDevice, h->stream), "D2D");
    check_hip(hipMemcpyAsync(v.th[1], h->cur_theta(), bytes, hipMemcpyDeviceToDevice, h->stream), "D2D");
    check_hip(hipMemcpyAsync(v.u, h->u, bytes, hipMemcpyDeviceToDevice, h->stream), "D2D");
    v.fresh_k = ~(uint64_t)0;
    launch_set_counter(kc.p, 0, h->stream);
    check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
    hipEvent_t e0, e1;
    check_hip(hipEventCreate(&e0), "hipEventCreate");
    check_hip(hipEventCreate(&e1), "hipEventCreate");
    const int rows_c[] = {1, 2, 4, 8, 16, 32, 64};
    const int wpb_c[] = {1, 2, 4, 8};
    // about 2 ms of work per timing (at least 16 steps)
    const int reps = (int)std::max<double>(16.0, std::min<double>(512.0, 2.0e11 * 2e-3 / (double)h->N));
    auto time_graph = [&](const Launch& l, int repeats, int mode = kStore) {
        hipGraph_t g = nullptr;
        hipGraphExec_t ex = nullptr;
        check_hip(hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
        for (int i = 0; i < reps; ++i) launch_step<R>(v, mode, l, kc.p, (uint64_t)i, h->cap_stream);
        check_hip(hipStreamEndCapture(h->cap_stream, &g), "hipStreamEndCapture");
        hipError_t err = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        check_hip(err, "hipGraphInstantiate");
        check_hip(hipGraphLaunch(ex, h->stream), "hipGraphLaunch");   // warm-up
        float best_t = 1e30f;
        for (int rep = 0; rep < repeats; ++rep) {
            check_hip(hipEventRecord(e0, h->stream), "hipEventRecord");
            check_hip(hipGraphLaunch(ex, h->stream), "hipGraphLaunch");
            check_hip(hipEventRecord(e1, h->stream), "hipEventRecord");
            check_hip(hipEventSynchronize(e1), "hipEventSynchronize");
            float ms = 0.f;
            check_hip(hipEventElapsedTime(&ms, e0, e1), "hipEventElapsedTime");
            best_t = std::min(best_t, ms);
        }
        (void)hipGraphExecDestroy(ex);
        return best_t;
    };
    std::vector<std::pair<float, Launch>> scores;
    for (int r : rows_c) {
        if (r > h->Ly) continue;
        for (int w : wpb_c) {
            Launch l;
            l.rows = r;
            l.wpb = w;
            scores.push_back({time_graph(l, 1), l});
        }
    }
    // re-time the three fastest with repeats and keep the best minimum
    std::sort(scores.begin(), scores.end(), [](const auto& a, const auto& b) { return a.first < b.first; });
    Launch best = scores.front().second;
    float best_ms = 1e30f;
    for (size_t i = 0; i < std::min<size_t>(3, scores.size()); ++i) {
        const float t = time_graph(scores[i].second, 3);
        if (t < best_ms) {
            best_ms = t;
            best = scores[i].second;
        }
    }
    // measurements without a step (the samples of a run): the same timing
    // over the shapes, the partial sums written to the lattice's own buffer
    {
        std::vector<std::pair<float, Launch>> ms;
        for (int r : rows_c) {
            if (r > h->Ly) continue;
            for (int w : wpb_c) {
                Launch l;
                l.rows = r;
                l.wpb = w;
                ms.push_back({time_graph(l, 1, kMeasure), l});
            }
        }
        std::sort(ms.begin(), ms.end(), [](const auto& a, const auto& b) { return a.first < b.first; });
        *mlaunch = ms.front().second;
        float mbest = 1e30f;
        for (size_t i = 0; i < std::min<size_t>(3, ms.size()); ++i) {
            const float t = time_graph(ms[i].second, 3, kMeasure);
            if (t < mbest) {
                mbest = t;
                *mlaunch = ms[i].second;
            }
        }
    }
    float best_step = best_ms / (float)reps;
    // two steps per pass: the same timing over a multiple of 4 steps, per step
    *fusion = sizeof(R) == 4 ? 1 : 2;
    *rows2 = 0;
    *tw2 = 0;
    if constexpr (std::is_same<R, float>::value) {
        if (step2_lattice_shape(h->Lx, h->Ly) && kick_factored(h->p)) {
            const int reps4 = (reps + 3) / 4 * 4;
            float* A = v.th[0];
            float* B = v.th[1];
            float* u = v.u;
            float* u2 = reinterpret_cast<float*>(tmp.p + 3 * bytes);
            check_hip(hipMemcpyAsync(u2, v.u, bytes, hipMemcpyDeviceToDevice, h->stream), "D2D");
            auto time_step2 = [&](int rows, int tw, int repeats) {
                hipGraph_t g = nullptr;
                hipGraphExec_t ex = nullptr;
                check_hip(hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeThreadLocal),
                          "hipStreamBeginCapture");
                for (int i = 0; i < reps4; i += 4) {
                    launch_step2(v, A, u, B, u2, rows, kc.p, (uint64_t)i, h->cap_stream, tw);
                    launch_step2(v, B, u2, A, u, rows, kc.p, (uint64_t)i + 2, h->cap_stream, tw);
                }
                check_hip(hipStreamEndCapture(h->cap_stream, &g), "hipStreamEndCapture");
                hipError_t err = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
                (void)hipGraphDestroy(g);
                check_hip(err, "hipGraphInstantiate");
                check_hip(hipGraphLaunch(ex, h->stream), "hipGraphLaunch");   // warm-up
                float best_t = 1e30f;
                for (int rep = 0; rep < repeats; ++rep) {
                    check_hip(hipEventRecord(e0, h->stream), "hipEventRecord");
                    check_hip(hipGraphLaunch(ex, h->stream), "hipGraphLaunch");
                    check_hip(hipEventRecord(e1, h->stream), "hipEventRecord");
                    check_hip(hipEventSynchronize(e1), "hipEventSynchronize");
                    float ms = 0.f;
                    check_hip(hipEventElapsedTime(&ms, e0, e1), "hipEventElapsedTime");
                    best_t = std::min(best_t, ms);
                }
                (void)hipGraphExecDestroy(ex);
                return best_t / (float)reps4;
            };
            // the tile width first (whole rows or the fewest tiles, and
            // narrower tiles; each at the rule's strip height for it), then
            // the strip height at the best width
            int tw = 16;
            {
                std::vector<std::pair<float, int>> st;
                std::vector<std::pair<int, int>> seen;   // (tiles, width) of the candidates timed
                for (int c : {16, 11, 8, 4, 3, 2}) {
                    Step2Tiles t;
                    if (!step2_tiles(h->Lx, &t, c)) {
                        if (c != 16) continue;
                        t.ntx = 1;             // whole rows
                        t.w = h->Lx;
                    }
                    if (std::find(seen.begin(), seen.end(), std::make_pair(t.ntx, t.w)) != seen.end()) continue;
                    seen.push_back({t.ntx, t.w});
                    st.push_back({time_step2(step2_rows(h->Lx, h->Ly, h->cus, c), c, 2), c});
                }
                std::sort(st.begin(), st.end());
                tw = st.front().second;
            }
            Step2Tiles t0;
            const bool tiled = step2_tiles(h->Lx, &t0, tw);
            std::vector<int> rows_c2 = {2, 4, 8, 16, step2_rows(h->Lx, h->Ly, h->cus, tw)};
            if (tiled) rows_c2.push_back(32);
            std::sort(rows_c2.begin(), rows_c2.end());
            rows_c2.erase(std::unique(rows_c2.begin(), rows_c2.end()), rows_c2.end());
            std::vector<std::pair<float, int>> s2;
            for (int r : rows_c2)
                if (r <= h->Ly) s2.push_back({time_step2(r, tw, 1), r});
            std::sort(s2.begin(), s2.end());
            float best2 = 1e30f;
            for (size_t i = 0; i < std::min<size_t>(2, s2.size()); ++i) {
                const float t = time_step2(s2[i].second, tw, 3);
                if (t < best2) {
                    best2 = t;
                    *rows2 = s2[i].second;
                }
            }
            *tw2 = tw;
            if (best2 < best_step) *fusion = 2;
            best_step = std::min(best_step, best2);
        }
    }
    // the paths with more steps per launch: 60 or 64 steps issued as the
    // stepping issues them
    t->tiles = t->march = kSlower;
    R* th[2] = {v.th[0], v.th[1]};
    R* u[2] = {v.u, reinterpret_cast<R*>(tmp.p + 3 * bytes)};
    auto time_direct = [&](int nsteps, auto&& issue) {
        float best_t = 1e30f;
        for (int rep = 0; rep < 4; ++rep) {
            check_hip(hipEventRecord(e0, h->stream), "hipEventRecord");
            issue();
            check_hip(hipEventRecord(e1, h->stream), "hipEventRecord");
            check_hip(hipEventSynchronize(e1), "hipEventSynchronize");
            float ms = 0.f;
            check_hip(hipEventElapsedTime(&ms, e0, e1), "hipEventElapsedTime");
            if (rep) best_t = std::min(best_t, ms / (float)nsteps);
        }
        return best_t;
    };
    if constexpr (std::is_same<R, float>::value) {
        if (march_shape_ok(h->dtype, h->Ly) && kick_factored(h->p)) {
            const MarchPlan p = march_plan(h->Lx, h->Ly, h->cus);
            const float ms = time_direct(60, [&] {
                for (int i = 0; i < 60; i += kMarchSteps) {
                    const int a = (i / kMarchSteps) & 1;
                    launch_march(v, MarchBuffers{th[a], u[a], th[a ^ 1], u[a ^ 1]}, p, (uint64_t)i, h->stream);
                }
            });
            if (ms < best_step) {
                best_step = ms;
                t->march = kChosen;
                *fusion = 2;
            }
        }
    }
    TilePlan p;
    if (tile_shape_ok(h->Lx, h->Ly) && tile_plan(h->Lx, h->Ly, h->dtype == XYL_F64, h->cus, 64, &p, nullptr)) {
        const float ms = time_direct(64, [&] {
            const uint64_t nl = tile_launches(64, p.T);
            uint64_t k = 0;
            for (uint64_t i = 0; i < nl; ++i) {
                const int n = (int)(64 / nl + (i < 64 % nl ? 1 : 0)), a = (int)(i & 1);
                launch_tile<R>(v, th[a], u[a], th[a ^ 1], u[a ^ 1], p, n, k, h->stream);
                k += (uint64_t)n;
            }
        });
        if (ms < best_step) {
            t->tiles = kChosen;
            t->march = kSlower;
            *fusion = 2;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return best;
}

extern "C" {

int xyl_autotune(xyl_lattice* h) {
    return guarded([&] {
        require_init(h);
        DeviceGuard g(h->device);
        Tuned2 t;
        Launch lm;
        const Launch l = h->dtype == XYL_F64 ? autotune_impl<double>(h, &t, &lm) : autotune_impl<float>(h, &t, &lm);
        h->launch = l;
        h->mlaunch = lm;
        h->mlaunch_tuned = true;
        {
            std::lock_guard<std::mutex> lk(g_tune_mu);
            g_tuned[{h->Lx, h->Ly, h->dtype}] = l;
            g_tunedm[{h->Lx, h->Ly, h->dtype}] = lm;
            g_tuned2[{h->Lx, h->Ly, h->dtype, h->p.model, (int)kick_factored(h->p)}] = t;
        }
        h->own_path = h->shaped = false;
        h->tile_plans.clear();
        apply_tuned_path(h);
        h->own_path = true;
        h->touch();
    });
}

int xyl_set_fusion(xyl_lattice* h, int32_t steps_per_pass) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        require(steps_per_pass == 1 || steps_per_pass == 2, XYL_EINVAL, "steps_per_pass must be 1 or 2");
        h->fusion = steps_per_pass;
        h->own_path = true;
    });
}

int xyl_get_fusion(const xyl_lattice* h, int32_t* steps_per_pass, int32_t* rows) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        if (steps_per_pass) *steps_per_pass = h->fusion;
        if (rows) *rows = step2_eligible(h) ? step2_rows(h) : 0;
    });
}

int xyl_stepping_path(xyl_lattice* h, uint64_t nsteps, int32_t* path, int32_t* steps_per_launch) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        int p = XYL_PATH_SINGLE, t = 1;
        MarchPlan mp;
        if (!h->second_u) {
        } else if (const TilePlan* tp = lattice_tile_choice(h, nsteps)) {
            const uint64_t nl = tile_launches(nsteps, tp->T);
            p = XYL_PATH_TILES;
            t = (int)((nsteps + nl - 1) / nl);
        } else if (lattice_march_steps(h, nsteps, &mp)) {
            p = XYL_PATH_MARCH;
            t = kMarchSteps;
        } else if (nsteps >= 4 && step2_eligible(h)) {
            p = XYL_PATH_TWO_STEP;
            t = 2;
        }
        if (path) *path = p;
        if (steps_per_launch) *steps_per_launch = t;
    });
}

int xyl_set_step2_shape(xyl_lattice* h, int32_t rows, int32_t tile_waves) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        require(rows == 0 || (rows >= 2 && rows <= 64), XYL_EINVAL, "rows per strip must be 0 or in [2, 64]");
        require(tile_waves == 0 || (tile_waves >= 2 && tile_waves <= 16), XYL_EINVAL,
                "waves per tile must be 0 or in [2, 16]");
        if (rows) h->step2_rows_tuned = rows;
        if (tile_waves) h->step2_tw_tuned = tile_waves;
        if (rows || tile_waves) h->shaped = h->own_path = true;
        h->touch();
    });
}

int xyl_get_step2_shape(const xyl_lattice* h, int32_t* rows, int32_t* tile_waves, int32_t* tiles) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        const bool on = step2_eligible(h);
        int tw = 0, ntx = 0;
        if (on) {
            Step2Tiles t;
            const int want = step2_tile_waves(h);
            if (step2_tiles(h->Lx, &t, want) || step2_tiles(h->Lx, &t)) {
                tw = want;
                ntx = t.ntx;
            } else {
                tw = (h->Lx + kWaveSites - 1) / kWaveSites;   // whole rows
                ntx = 1;
            }
        }
        if (rows) *rows = on ? step2_rows(h) : 0;
        if (tile_waves) *tile_waves = tw;
        if (tiles) *tiles = ntx;
    });
}

int xyl_set_graph_steps(xyl_lattice* h, int32_t steps) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        require(steps >= 0 && steps <= 4096, XYL_EINVAL, "graph steps must be in [0, 4096]");
        h->graph_steps = steps;
        h->touch();
    });
}

int xyl_choose_path(xyl_lattice* h, int32_t path) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        require(path >= XYL_PATH_SINGLE && path <= XYL_PATH_TILES, XYL_EINVAL, "not a path of a lattice");
        h->fusion = path == XYL_PATH_SINGLE ? 1 : 2;
        h->march = path == XYL_PATH_MARCH ? kChosen : kSlower;
        h->tiles = path == XYL_PATH_TILES ? kChosen : kSlower;
        h->shaped = false;
        h->own_path = true;
        h->tile_plans.clear();
        h->touch();
    });
}

int xyl_deny_second_buffer(xyl_lattice* h) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        h->second_u = false;
    });
}

int xyl_philox_blocks(int32_t device, uint64_t seed, const uint32_t* ctr, uint32_t* out, uint64_t n) {
    return guarded([&] {
        require(ctr != nullptr && out != nullptr, XYL_EINVAL, "NULL array");
        require(n >= 1 && n <= (1ull << 26), XYL_EINVAL, "n out of range");
        select_device(device);
        DevBuf<uint32_t> dc, dout;
        dc.reserve(4 * n);
        dout.reserve(4 * n);
        check_hip(hipMemcpy(dc.p, ctr, sizeof(uint32_t) * 4 * n, hipMemcpyHostToDevice), "H2D");
        launch_philox_blocks(seed, dc.p, dout.p, n, nullptr);
        check_hip(hipMemcpy(out, dout.p, sizeof(uint32_t) * 4 * n, hipMemcpyDeviceToHost), "D2H");
    });
}

int xyl_stream_ceiling(int32_t device, uint64_t n, int32_t reps, double* gbs) {
    return guarded([&] {
        require(gbs != nullptr, XYL_EINVAL, "gbs is NULL");
        require(n >= 4 && n % 4 == 0, XYL_EINVAL, "n must be a positive multiple of 4");
        require(reps >= 2, XYL_EINVAL, "reps must be >= 2");
        select_device(device);
        DevBuf<float> buf;
        buf.reserve(4 * n);
        check_hip(hipMemset(buf.p, 0, sizeof(float) * 4 * n), "hipMemset");
        float* A = buf.p;
        float* B = buf.p + n;
        float* C = buf.p + 2 * n;
        float* D = buf.p + 3 * n;
        hipEvent_t e0, e1;
        check_hip(hipEventCreate(&e0), "hipEventCreate");
        check_hip(hipEventCreate(&e1), "hipEventCreate");
        double best = 0.0;
        for (int grid : {1024, 2048, 4096, 8192, 16384, 65536}) {
            for (int w = 0; w < 4; ++w) launch_stream_probe(A, B, C, D, n / 4, grid, nullptr);
            check_hip(hipEventRecord(e0, nullptr), "hipEventRecord");
            for (int r = 0; r < reps; ++r) {
                // ping-pong between the two pairs, like a lattice's state
                if (r & 1) launch_stream_probe(C, D, A, B, n / 4, grid, nullptr);
                else launch_stream_probe(A, B, C, D, n / 4, grid, nullptr);
            }
            check_hip(hipEventRecord(e1, nullptr), "hipEventRecord");
            check_hip(hipEventSynchronize(e1), "hipEventSynchronize");
            float ms = 0.f;
            check_hip(hipEventElapsedTime(&ms, e0, e1), "hipEventElapsedTime");
            best = std::max(best, 16.0 * (double)n * reps / ((double)ms * 1e-3) / 1e9);
        }
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        *gbs = best;
    });
}

int xyl_noise(xyl_lattice* h, uint64_t k, double* out) {
    return guarded([&] {
        require(h != nullptr && out != nullptr, XYL_EINVAL, "NULL argument");
        DeviceGuard g(h->device);
        h->dscratch.reserve(h->N);
        if (h->dtype == XYL_F64) launch_noise<double>(h->view<double>(), k, h->dscratch.p, h->stream);
        else launch_noise<float>(h->view<float>(), k, h->dscratch.p, h->stream);
        check_hip(hipMemcpyAsync(out, h->dscratch.p, sizeof(double) * h->N, hipMemcpyDeviceToHost, h->stream), "D2H");
        check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
    });
}


}  // extern "C"

// ==================================================================== ensemble
struct xyl_ensemble {
    int dtype = XYL_F32;
    int device = 0;
    int n = 0;
    int mode = 0;
    hipStream_t stream = nullptr;
    std::vector<xyl_replica_desc> desc;
    std::vector<size_t> off;        // element offset of each replica
    std::vector<size_t> poff;       // partial-sum offset of each replica
    size_t total = 0, ptotal = 0;
    void* th[2] = {nullptr, nullptr};
    void* u = nullptr;
    std::vector<uint64_t> k;        // current step of each replica
    std::vector<uint64_t> fresh_k;
    std::vector<uint64_t> last_sample;  // step of the last recorded sample (+1), 0 = none
    uint64_t j = 0;                 // batched launches issued
    Launch launch;
    DevBuf<char> reps;              // Lat<R>[n]
    bool reps_ok = false;           // reps holds every active replica's view
    // two steps per pass for FP32 replicas on the tile path: one batched launch
    // per class of replicas spanning the same number of waves, per pass; the
    // other tile-path replicas keep one tile launch per step (tasks_rest)
    struct Step2Class {
        int waves = 0;
        bool partial = false;
        int max_lx = 0;
        int rows = 0;
        DevBuf<Task2> tasks;
        int ntasks = 0;
    };
    // How the replicas step in chunks of one class, and the launches' tables.
    // They are kept per class, so that a first short chunk decides nothing for
    // long ones, and alternating lengths rebuild nothing.
    struct Tables {
        bool built = false;
        uint64_t n = 0;                 // the chunk length that the plan was made for
        std::vector<int> planned_for;   // the active replicas that the plan was made for
        std::vector<int> strips;        // those of them in the tables: all but the LDS path's own
        std::vector<int> meas;          // those that the strip kernels measure: not the LDS path's
        // tasks: [0, ntasks_flat) stepped by two-step classes or tile-table
        // steps, [ntasks_flat, ntasks) on tiles; [0, ntasks_meas) those of meas
        DevBuf<Task> tasks;
        int ntasks = 0, ntasks_flat = 0, ntasks_meas = 0;
        // replicas that take several steps per launch on tiles (xyl_tile.hip)
        TilePlan tile_shape;            // T = 0: none
        size_t tile_lds = 0;
        std::map<std::pair<int, int>, std::pair<int, int>> boxes;   // tiles of each distinct size
        DevBuf<TileTask> tiles;
        int ntiles = 0;
        std::vector<char> tiled;        // per replica: on tiles (one of the LDS path then only measures in LDS)
        std::vector<Step2Class> s2cls;
        DevBuf<Task> tasks_rest;
        int ntasks_rest = 0;
        // groups of replicas stepped in parallel: the two-step classes, the tiles
        size_t groups() const { return s2cls.size() + (ntiles ? 1 : 0); }
        // the tile fits of the sizes met so far
        std::unique_ptr<TileFits> fits;
        std::vector<TileSize> fit_sizes;
    };
    // Classes 0 to 3: fewer than 4, 8, 16 steps, and longer, each planned for the
    // first length of it that was met.  Below 16 steps also: 4, chunks at whose
    // end a replica ends (on tiles that replica's end would make new tables after
    // a few steps: 48 LDS replicas of 32^2 to 64^2 ending 7 steps apart took 2.8
    // ms with some of them on tiles, 2.4 without), and 5 and 6, chunks that start
    // with samples of LDS replicas.
    static constexpr int kClasses = 7;
    Tables tables[kClasses];
    Tables* tab = &tables[0];       // of the last chunk
    static int chunk_class(uint64_t n, bool ending, bool lds_sampled) {
        if (n < 4 || n >= 16) return n < 4 ? 0 : 3;
        return ending ? 4 : (n < 8 ? 1 : 2) + (lds_sampled ? 4 : 0);
    }
    bool tiles_ok = true;           // false: no memory for the second velocity buffer
    // the tables serve neither steps nor measurements any more
    void drop_tables() {
        reps_ok = false;
        for (Tables& t : tables) {
            t.built = false;
            t.planned_for.clear();
            t.meas.clear();
            t.n = 0;
        }
    }
    DevBuf<double> part;
    DevBuf<double> phases;                  // measurement phase tables, one per side length
    std::map<int, size_t> phase_off;        // side length -> offset of its table in phases
    DevBuf<double> obs;
    DevBuf<FinalizeJobHost> jobs;
    PinnedBuf<FinalizeJobHost> jobs_host;   // the source of each flush's copy into `jobs`
    SpectrumBufs spectrum;
    DevBuf<char> omega_buf;
    DomainBufs domains;
    // small FP32 replicas stepped whole-in-LDS on a second stream
    std::vector<char> lds;          // per replica: 1 = LDS path
    int lds_max_sites = 0, lds_threads = 0;
    hipStream_t side = nullptr;
    hipEvent_t ev_main = nullptr, ev_side = nullptr;
    // the LDS launches' tables, double-buffered: a chunk writes table b while
    // the previous chunk's launch may still read table b ^ 1; ev_lds[b] marks
    // the end of the last launch that read table b (and of the copies into it)
    DevBuf<char> lds_reps[2];
    DevBuf<LdsJobHost> lds_jobs[2];
    // host sides of those tables in pinned memory: an asynchronous copy from
    // pageable memory waits for its stream to drain, which left the GPU idle
    // at every chunk boundary while the host waited
    PinnedBuf<LdsJobHost> lds_jobs_host[2];
    PinnedBuf<Lat<float>> lds_tab_host[2];
    hipEvent_t ev_lds[2] = {nullptr, nullptr};
    bool ev_lds_used[2] = {false, false};
    int lds_buf = 0;
    int fusion = 2;
    int cus = 256;
    int tables_fusion = 0;          // fusion setting the task tables were built for
    DevBuf<char> u2;                // second velocity buffer, allocated on first use
    // the classes hold different replicas: all but the first run on streams of
    // their own (default priority), forked from and joined to the ensemble's
    std::vector<hipStream_t> cls_streams;
    std::vector<hipEvent_t> cls_events;   // [0] fork, [1 + i] join of class i + 1
    // Chunks of steps captured as graphs (step index from the device counter
    // kc): keyed by (tables, first step within the chunk, steps), captured the second
    // time a key is met and replayed after; all dropped when a table, the
    // launch shape or the steps per pass change (graph_version).
    // 0: no graphs; 1: graphs for chunks with at most one class of two-step
    // passes; 2: graphs for every repeated chunk.  A replayed graph dispatches
    // the parallel branches of several classes one after the other (one
    // class's whole chain before the next class's first pass), so the classes
    // barely overlap; issued directly, pass by pass across the classes, they
    // run together.
    int use_graphs = 1;
    hipStream_t cap_stream = nullptr;
    DevBuf<uint64_t> kc;
    uint64_t graph_version = 0, graphs_built_for = ~(uint64_t)0;
    struct ChunkGraph {
        int seen = 0;
        hipGraphExec_t exec = nullptr;
    };
    std::map<std::tuple<const Tables*, uint64_t, uint64_t>, ChunkGraph> graphs;
    void drop_graphs() {
        for (auto& g : graphs)
            if (g.second.exec) (void)hipGraphExecDestroy(g.second.exec);
        graphs.clear();
    }
    void class_streams(size_t ncls) {
        while (cls_streams.size() + 1 < ncls) {
            hipStream_t st = nullptr;
            check_hip(hipStreamCreateWithFlags(&st, hipStreamNonBlocking), "hipStreamCreate");
            cls_streams.push_back(st);
        }
        // [0] fork, [1 + i] join of class i + 1, [ncls] end of a chunk's sample
        while (cls_events.size() < ncls + 1) {
            hipEvent_t ev = nullptr;
            check_hip(hipEventCreateWithFlags(&ev, hipEventDisableTiming), "hipEventCreate");
            cls_events.push_back(ev);
        }
    }

    template <typename R>
    Lat<R> view(int r, uint64_t jbase) {
        const xyl_replica_desc& d = desc[r];
        Lat<R> v{};
        R* t0 = static_cast<R*>(th[0]) + off[r];
        R* t1 = static_cast<R*>(th[1]) + off[r];
        v.th[0] = t0;
        v.th[1] = t1;
        v.u = static_cast<R*>(u) + off[r];
        v.cur = 0;
        Params p{d.Jx, d.Jy, d.h, d.gamma, d.dt, d.model, d.p};
        Schedule s{};
        s.n = d.nknots;
        for (int q = 0; q < d.nknots; ++q) {
            s.step[q] = d.knot_step[q];
            s.T[q] = d.knot_T[q];
            s.g[q] = d.knot_gamma[q] == 0 ? 1 : d.knot_gamma[q];
        }
        fill_lat(v, d.Lx, d.Ly, p, s, d.seed, d.replica);
        v.k_base = k[r] - jbase;   // k = k_base + j for the launches numbered from jbase
        v.fresh_k = fresh_k[r];
        v.k_end = d.nsteps;
        v.part = part.p + poff[r];
        v.xph = phases.p + phase_off.at(d.Lx);
        v.yph = phases.p + phase_off.at(d.Ly);
        v.omega_out = reinterpret_cast<R*>(omega_buf.p);
        v.pingpong = 1;
        v.u_out = nullptr;
        v.part_k0 = 0;
        v.part_stride = 0;
        return v;
    }
    void* cur_theta(int r) {
        const size_t es = elem_size(dtype);
        return static_cast<char*>(th[(int)(k[r] & 1)]) + es * off[r];
    }
    int nrp(int r) const { return desc[r].Ly * ((desc[r].Lx + kWaveSites - 1) / kWaveSites); }
    int model() const { return desc[0].model; }
};

static bool replica_factored(const xyl_replica_desc& d) {
    return kick_factored(Params{d.Jx, d.Jy, d.h, d.gamma, d.dt, d.model, d.p});
}

// Strips of a two-step class as tall as keep at least two waves per SIMD busy
// (2 to 32 rows; 32 for the 60 x 2048^2 quench batch: 5.83 -> 5.98e11
// site-updates/s against 16, 5.86e11 with 64).  Rows of more than 8 waves hold
// one workgroup per CU and go to 64 (eight 4096^2 replicas: 6.05 -> 6.19e11).
static int class_rows(const xyl_ensemble* e, int waves, const std::vector<int>& reps, long* strips_o) {
    for (int rows = waves > 8 ? 64 : 32; rows >= 2; rows /= 2) {
        long strips = 0;
        for (int r : reps) strips += (e->desc[r].Ly + rows - 1) / rows;
        *strips_o = strips;
        if (strips * waves >= 8L * e->cus || rows == 2) return rows;
    }
    return 2;
}

// How the active replicas step with two steps per pass on: which go on tiles,
// by the paths' times per step.
//   * Two-step classes: step2_us's form over the class's strips, times 1.15
//     (1-wave class of 192^2 and 256^2 replicas, 32 each: 10.3 us per step
//     measured; 2-wave class of 384^2 and 512^2: 25.5); parallel groups
//     together 0.9 of their sum.
//   * Whole in LDS: the largest replica's step on its one CU, 4.5 us for 128^2
//     (5.6 Si), beside the other replicas on a stream of its own, whose issue
//     it shares.  128 Si replicas of 32^2 to 144^2: the LDS launches took 5.6
//     us per step and the 144^2 ones 16 in single tile-table steps; on tiles
//     all of them take about 3.
//   * Other widths: single tile-table steps, lattice_untiled_us's form.
//   * Tiles: TileFits::best.
// For chunks of tab.n steps; another split than none is taken only where it
// gains 5%.  With `ending` the LDS replicas stay whole in LDS; with `lds_sampled`
// they are measured at the chunk's start, which is part of their launch whole in
// LDS and a launch and two waits of its own beside tiles, some 10 us (20 replicas
// of up to 5000 sites sampled every 4 steps: 51 us a chunk on tiles, 37 in LDS).
struct EnsTilePlan {
    TilePlan shape;                 // T = 0: no tiles
    size_t lds = 0;
    std::map<std::pair<int, int>, std::pair<int, int>> boxes;
    std::vector<char> tiled;
};
static EnsTilePlan ens_plan_tiles(xyl_ensemble* e, xyl_ensemble::Tables& tab, const std::vector<int>& active,
                                  bool ending, bool lds_sampled) {
    EnsTilePlan out;
    const uint64_t n = tab.n;
    out.tiled.assign(e->n, 0);
    if (e->fusion != 2 || n < 4 || !e->tiles_ok) return out;
    const bool f64 = e->dtype == XYL_F64;
    // units that step on tiles or not: 0 the LDS replicas, 1..16 the two-step
    // classes, 17 the others
    constexpr int kUnits = 18;
    std::vector<std::vector<int>> unit(kUnits);
    double lds_fixed_sites = 0.0;
    for (int r : active) {
        const xyl_replica_desc& d = e->desc[r];
        const bool fact = f64 || replica_factored(d);
        const bool fits = fact && tile_shape_ok(d.Lx, d.Ly);
        const bool stays = !fits || (ending && e->lds[r]);
        if (stays && e->lds[r]) lds_fixed_sites += (double)d.Lx * d.Ly;
        if (stays) continue;
        if (e->lds[r]) unit[0].push_back(r);
        else if (!f64 && step2_shape(d.Lx, d.Ly)) unit[(d.Lx + kWaveSites - 1) / kWaveSites].push_back(r);
        else unit[17].push_back(r);
    }
    std::vector<int> used;
    std::vector<double> flat_us(kUnits, 0.0);
    double lds_sites = lds_fixed_sites, full_us = 0.0;
    int full = 0;              // classes that fill the chip
    for (int q = 0; q < kUnits; ++q) {
        if (unit[q].empty()) continue;
        if (q == 0) {
            int nmax = 0;
            for (int r : unit[0]) {
                const int N = e->desc[r].Lx * e->desc[r].Ly;
                lds_sites += N;
                nmax = std::max(nmax, N);
            }
            const int fit = std::max(1, std::min(32 / (e->lds_threads / kWave), 160 * 1024 / (8 * e->lds_max_sites)));
            int left = (int)((unit[0].size() + e->cus - 1) / e->cus);
            for (; left > 0; left -= fit) {
                const double x = 0.3 * (nmax / 1024.0) * std::min(left, fit);
                flat_us[0] += std::sqrt(1.44 + x * x);
            }
        } else if (q <= 16) {
            long strips = 0;
            int max_lx = 0;
            for (int r : unit[q]) max_lx = std::max(max_lx, e->desc[r].Lx);
            const int rows = class_rows(e, q, unit[q], &strips);
            const int fit = std::max(1, std::min(16 / q, (160 * 1024) / (32 * max_lx)));
            double us = 3.0;
            for (long left = (strips + e->cus - 1) / e->cus; left > 0; left -= fit) {
                const double x = 0.6 * 0.25 * q * (double)std::min<long>(left, fit);
                us += (rows + 2) * std::sqrt(1.0 + x * x);
            }
            flat_us[q] = 1.15 * 0.5 * us;
            // tiles reach 4.6e5 sites per us at best: a class that fills the
            // chip stays as it is
            double N = 0.0;
            for (int r : unit[q]) N += (double)e->desc[r].Lx * e->desc[r].Ly;
            if (N / flat_us[q] > 4.8e5) {
                full_us += flat_us[q];
                ++full;
                continue;
            }
        } else {
            double N = 0.0;
            for (int r : unit[q]) N += (double)e->desc[r].Lx * e->desc[r].Ly;
            flat_us[q] = f64 ? 6.5 + N / 1.15e5 : 3.3 + N / 3.7e5;
        }
        used.push_back(q);
    }
    if (used.empty()) return out;
    // the sizes' fits are kept: a replica that ends changes the counts only
    std::vector<TileSize>& sizes = tab.fit_sizes;
    std::vector<int> size_of(e->n, -1);
    const size_t known = sizes.size();
    for (int q : used)
        for (int r : unit[q]) {
            const int Lx = e->desc[r].Lx, Ly = e->desc[r].Ly;
            size_t i = 0;
            while (i < sizes.size() && (sizes[i].Lx != Lx || sizes[i].Ly != Ly)) ++i;
            if (i == sizes.size()) {
                TileSize z;
                z.Lx = Lx;
                z.Ly = Ly;
                sizes.push_back(z);
            }
            size_of[r] = (int)i;
        }
    if (!tab.fits || sizes.size() != known) tab.fits.reset(new TileFits(sizes, f64, e->cus, n));
    const TileFits& fits = *tab.fits;
    // (more than 6 units never occur in practice; the first ones are split then)
    const int nu = std::min<int>((int)used.size(), 6);
    double best = 1e30;
    unsigned pick = 0;
    std::vector<long> pick_count;
    for (unsigned m = 0; m < (1u << nu); ++m) {
        std::vector<long> count(sizes.size(), 0);
        double main_us = full_us, lds_us = 0.0, lds_share = lds_fixed_sites / 6.3e5, single_us = 0.0;
        int groups = full;
        for (size_t b = 0; b < used.size(); ++b) {
            const int q = used[b];
            if (b < (size_t)nu && (m >> b & 1u)) {
                for (int r : unit[q]) count[size_of[r]] += 1;
            } else if (q == 0) {
                lds_us = flat_us[0];
                lds_share = lds_sites / 6.3e5;
            } else if (q <= 16) {
                main_us += flat_us[q];
                ++groups;
            } else {
                single_us += flat_us[q];
            }
        }
        // (what is left to the other paths may cost more already)
        if (std::max(lds_us, 0.9 * main_us + single_us + lds_share) >= 0.95 * best) continue;
        if (m) {
            const double t = fits.best(count, nullptr, nullptr, nullptr);
            if (t >= 1e30) continue;
            main_us += t;
            ++groups;
        }
        if (groups > 1) main_us *= 0.9;
        main_us += single_us;
        if (lds_sampled && used[0] == 0 && (m & 1u)) main_us += 10.0 / (double)n;
        const double us = main_us > 0.0 ? std::max(lds_us, main_us + lds_share) : lds_us;
        if (us < best * (m ? 0.95 : 1.0)) {
            best = us;
            pick = m;
            pick_count = count;
        }
    }
    if (!pick) return out;
    std::vector<TileSize> tiles;
    fits.best(pick_count, &out.shape, &tiles, &out.lds);
    for (int b = 0; b < nu; ++b)
        if (pick >> b & 1u)
            for (int r : unit[used[b]]) out.tiled[r] = 1;
    for (const TileSize& z : tiles)
        if (z.ntx) out.boxes[{z.Lx, z.Ly}] = {z.ntx, z.nty};
    return out;
}

// What the ensemble's stream and the LDS path's each hold so far is done before
// either goes on: a replica may change between them.
static void ens_join_streams(xyl_ensemble* e) {
    if (!e->side) return;
    check_hip(hipEventRecord(e->ev_main, e->stream), "hipEventRecord");
    check_hip(hipEventRecord(e->ev_side, e->side), "hipEventRecord");
    check_hip(hipStreamWaitEvent(e->side, e->ev_main, 0), "hipStreamWaitEvent");
    check_hip(hipStreamWaitEvent(e->stream, e->ev_side, 0), "hipStreamWaitEvent");
}

// Makes e->tab the tables for a chunk of n steps of the `active` replicas (LDS
// replicas among them), one of which ends with it if `ending`.  A chunk too
// short for tiles and passes goes with the last chunk's tables where those are
// the same replicas'.  What the tables hold of the replicas that step on
// strips and tiles stays while those and their plan do: an LDS replica that
// ends changes nothing, and an ensemble that only the LDS path steps uploads
// nothing.
template <typename R>
static void ens_upload_table(xyl_ensemble* e, uint64_t jbase, const std::vector<int>& active, uint64_t n,
                             bool ending, bool lds_sampled) {
    if (e->tables_fusion != e->fusion) e->drop_tables();
    e->tables_fusion = e->fusion;
    const int cls = xyl_ensemble::chunk_class(n, ending, lds_sampled);
    xyl_ensemble::Tables* before = e->tab;
    if (cls == 0 && before->built && before->planned_for == active) return;
    xyl_ensemble::Tables& t = e->tables[cls];
    e->tab = &t;
    // (the replicas on tiles before: a replica that ended since changes between
    // the streams too, as a sample of its last step is taken by the other)
    const std::vector<char> tiled_before = before->tiled;
    auto join = [&] {
        if (t.tiled != tiled_before) ens_join_streams(e);
    };
    if (t.built && t.planned_for == active) {
        join();
        return;
    }
    if (!t.n) {
        t.n = n;
        t.fits.reset();
        t.fit_sizes.clear();
    }
    EnsTilePlan plan = ens_plan_tiles(e, t, active, cls == 4, cls > 4);
    if (plan.shape.T) {
        // where the second velocity buffer does not fit, the other paths do
        // (the classes, which need it too, report that)
        try {
            e->u2.reserve(sizeof(R) * e->total);
        } catch (const Error& err) {
            if (err.code != XYL_ENOMEM) throw;
            (void)hipGetLastError();
            e->tiles_ok = false;
            e->drop_tables();
            t.n = n;
            plan = ens_plan_tiles(e, t, active, cls == 4, cls > 4);
        }
    }
    std::vector<int> strips, meas;
    for (int r : active) {
        if (!e->lds[r]) meas.push_back(r);
        if (!e->lds[r] || plan.tiled[r]) strips.push_back(r);
    }
    const bool same = t.built && t.strips == strips && t.tiled == plan.tiled && t.boxes == plan.boxes &&
                      t.tile_shape.T == plan.shape.T && t.tile_shape.S == plan.shape.S &&
                      t.tile_shape.threads == plan.shape.threads;
    t.planned_for = active;
    t.tiled = plan.tiled;
    join();
    if (same) return;
    t.built = false;
    t.strips = strips;
    t.meas = meas;
    t.boxes = plan.boxes;
    t.tile_shape = plan.shape;
    t.tile_lds = plan.lds;
    t.ntasks = t.ntasks_flat = t.ntasks_meas = t.ntiles = t.ntasks_rest = 0;
    t.s2cls.clear();
    e->graph_version += 1;
    if (strips.empty()) {
        t.built = true;
        return;
    }
    std::vector<Lat<R>> views;
    if (!e->reps_ok) {
        views.resize(e->n);
        for (int r = 0; r < e->n; ++r) views[r] = e->view<R>(r, jbase);
        e->reps.reserve(sizeof(Lat<R>) * e->n);
        check_hip(hipMemcpyAsync(e->reps.p, views.data(), sizeof(Lat<R>) * e->n, hipMemcpyHostToDevice, e->stream),
                  "H2D");
    }
    std::vector<TileTask> tt;
    std::vector<Task> tk;
    auto tile_rows = [&](int r) {
        const int nxw = (e->desc[r].Lx + kWaveSites - 1) / kWaveSites;
        const int nstrips = (e->desc[r].Ly + e->launch.rows - 1) / e->launch.rows;
        for (int s = 0; s < nstrips; ++s)
            for (int x = 0; x < nxw; ++x) tk.push_back(Task{r, x, s, 0});
    };
    for (int r : active)
        if (!e->lds[r] && !t.tiled[r]) tile_rows(r);
    t.ntasks_flat = (int)tk.size();
    for (int r : active)
        if (!e->lds[r] && t.tiled[r]) tile_rows(r);
    t.ntasks_meas = (int)tk.size();
    for (int r : active)
        if (e->lds[r] && t.tiled[r]) tile_rows(r);
    for (int r : active)
        if (t.tiled[r]) {
            const auto& b = t.boxes.at({e->desc[r].Lx, e->desc[r].Ly});
            tile_tasks(r, e->desc[r].Lx, e->desc[r].Ly, b.first, b.second, &tt);
        }
    t.ntiles = (int)tt.size();
    t.tiles.reserve(std::max<size_t>(tt.size(), 1));
    if (!tt.empty())
        check_hip(hipMemcpyAsync(t.tiles.p, tt.data(), sizeof(TileTask) * tt.size(), hipMemcpyHostToDevice, e->stream),
                  "H2D");
    t.ntasks = (int)tk.size();
    t.tasks.reserve(std::max<size_t>(tk.size(), 1));
    if (!tk.empty())
        check_hip(hipMemcpyAsync(t.tasks.p, tk.data(), sizeof(Task) * tk.size(), hipMemcpyHostToDevice, e->stream),
                  "H2D");
    // two-step classes (FP32, chunks of four steps and more): replicas whose
    // width the two-step pass takes, grouped by waves per row; the rest of the
    // tile-path replicas
    std::vector<std::vector<Task2>> t2(17);
    std::vector<Task> rest;
    if (e->dtype == XYL_F32 && e->fusion == 2 && cls > 0) {
        std::vector<std::vector<int>> byw(17);
        for (int r : active) {
            if (e->lds[r] || t.tiled[r]) continue;
            const xyl_replica_desc& d = e->desc[r];
            if (step2_shape(d.Lx, d.Ly) && replica_factored(d))
                byw[(d.Lx + kWaveSites - 1) / kWaveSites].push_back(r);
            else
                for (const Task& t : tk)
                    if (t.rep == r) rest.push_back(t);
        }
        for (int w = 1; w <= 16; ++w) {
            if (byw[w].empty()) continue;
            xyl_ensemble::Step2Class cl;
            cl.waves = w;
            long strips = 0;
            cl.rows = class_rows(e, w, byw[w], &strips);
            for (int r : byw[w]) {
                const xyl_replica_desc& d = e->desc[r];
                cl.partial = cl.partial || d.Lx % kWaveSites != 0;
                cl.max_lx = std::max(cl.max_lx, d.Lx);
                for (int s = 0; s * cl.rows < d.Ly; ++s)
                    t2[w].push_back(Task2{r, s * cl.rows, std::min(d.Ly, (s + 1) * cl.rows), (s & 1) ? -1 : 1});
            }
            cl.ntasks = (int)t2[w].size();
            cl.tasks.reserve(t2[w].size());
            check_hip(hipMemcpyAsync(cl.tasks.p, t2[w].data(), sizeof(Task2) * t2[w].size(), hipMemcpyHostToDevice,
                                     e->stream),
                      "H2D");
            t.s2cls.push_back(std::move(cl));
        }
        t.ntasks_rest = (int)rest.size();
        t.tasks_rest.reserve(std::max<size_t>(rest.size(), 1));
        if (!rest.empty())
            check_hip(hipMemcpyAsync(t.tasks_rest.p, rest.data(), sizeof(Task) * rest.size(), hipMemcpyHostToDevice,
                                     e->stream),
                      "H2D");
    }
    // the second velocity buffer and the group streams now, not in the first
    // chunk that steps through the groups
    if (t.groups()) {
        e->u2.reserve(sizeof(R) * e->total);
        e->class_streams(t.groups());
    }
    // the host vectors must outlive the copies
    check_hip(hipStreamSynchronize(e->stream), "hipStreamSynchronize");
    e->reps_ok = true;
    t.built = true;
}

// Sample bookkeeping of one xyl_ensemble_step call: observables gathered in
// device memory (slots), copied out at the end.
struct EnsSamples {
    xyl_ensemble* e;
    uint64_t every, cap;
    std::vector<uint64_t> cnt;
    size_t nsamp = 0;
    std::vector<std::pair<size_t, size_t>> copies;   // (device slot, host index)
    // finalize jobs of this call: each flush takes the next slots of the
    // device arena, copied from the same slots of its pinned host mirror
    size_t njobs = 0;
    EnsSamples(xyl_ensemble* e_, uint64_t every_, uint64_t cap_, const uint64_t* nout)
        : e(e_), every(every_), cap(cap_), cnt(e_->n, 0) {
        if (every && nout)
            for (int r = 0; r < e->n; ++r) cnt[r] = nout[r];
    }
    EnsSamples(const EnsSamples&) = delete;
    EnsSamples& operator=(const EnsSamples&) = delete;
    // the pinned job slots are the sources of copies that may still be
    // queued; the next call writes them again
    ~EnsSamples() {
        if (njobs) (void)hipStreamSynchronize(e->stream);
    }
    bool wants(int r) const {
        return every && e->k[r] <= e->desc[r].nsteps && e->k[r] % every == 0 && e->last_sample[r] != e->k[r] + 1;
    }
    void reserve(size_t extra) {
        const size_t need = nsamp + extra;
        if (need * 6 <= e->obs.n) return;
        // the side stream may still be writing samples into the old buffer
        if (e->side) check_hip(hipStreamSynchronize(e->side), "hipStreamSynchronize");
        DevBuf<double> nb;
        nb.reserve(std::max(need * 6, e->obs.n * 2));
        if (e->obs.p && nsamp)
            check_hip(hipMemcpyAsync(nb.p, e->obs.p, sizeof(double) * 6 * nsamp, hipMemcpyDeviceToDevice, e->stream),
                      "D2D");
        check_hip(hipStreamSynchronize(e->stream), "hipStreamSynchronize");
        std::swap(e->obs.p, nb.p);
        std::swap(e->obs.n, nb.n);
    }
    double* take(int r) {   // device slot of replica r's next sample
        require(cnt[r] < cap, XYL_EINVAL, "ensemble sample capacity too small");
        const size_t slot = nsamp++;
        copies.push_back({slot, (size_t)r * cap + cnt[r]});
        cnt[r] += 1;
        e->last_sample[r] = e->k[r] + 1;
        return e->obs.p + 6 * slot;
    }
    void finish(xyl_obs* out, uint64_t* nout) {
        if (!every) return;
        std::vector<double> host(6 * nsamp);
        if (nsamp)
            check_hip(hipMemcpyAsync(host.data(), e->obs.p, sizeof(double) * 6 * nsamp, hipMemcpyDeviceToHost,
                                     e->stream),
                      "D2H");
        check_hip(hipStreamSynchronize(e->stream), "hipStreamSynchronize");
        for (auto& c : copies) std::memcpy(&out[c.second], &host[6 * c.first], sizeof(double) * 6);
        if (nout)
            for (int r = 0; r < e->n; ++r) nout[r] = cnt[r];
    }
};

// Reduces the measurement partials of `jobs` into their sample slots, on the
// ensemble's stream, without waiting for it: the job list moves into the
// call's store and takes the next slots of the device arena (a full arena is
// replaced, after the stream has drained, by one twice as large).
static void flush_finalize(xyl_ensemble* e, EnsSamples& smp, std::vector<FinalizeJobHost>& jobs) {
    if (jobs.empty()) return;
    if (smp.njobs + jobs.size() > e->jobs.n || !e->jobs.p || e->jobs_host.n < e->jobs.n) {
        check_hip(hipStreamSynchronize(e->stream), "hipStreamSynchronize");
        const size_t cap = std::max<size_t>(2 * e->jobs.n, std::max<size_t>(jobs.size(), 256));
        e->jobs.reserve(cap);
        e->jobs_host.reserve(e->jobs.n);
        smp.njobs = 0;
    }
    FinalizeJobHost* src = e->jobs_host.p + smp.njobs;
    std::memcpy(src, jobs.data(), sizeof(FinalizeJobHost) * jobs.size());
    FinalizeJobHost* dst = e->jobs.p + smp.njobs;
    check_hip(hipMemcpyAsync(dst, src, sizeof(FinalizeJobHost) * jobs.size(), hipMemcpyHostToDevice, e->stream),
              "H2D");
    launch_finalize_jobs(dst, (int)jobs.size(), e->stream);
    smp.njobs += jobs.size();
    jobs.clear();
}

// Reference loop: every replica launched on its own, one step at a time.
template <typename R>
static void ens_step_per_replica(xyl_ensemble* e, uint64_t nsteps, EnsSamples& smp) {
    std::vector<FinalizeJobHost> jobs;
    for (uint64_t it = 0; it <= nsteps; ++it) {
        std::vector<int> active, measuring;
        for (int r = 0; r < e->n; ++r) {
            if (smp.wants(r)) measuring.push_back(r);
            if (it < nsteps && e->k[r] < e->desc[r].nsteps) active.push_back(r);
        }
        if (active.empty() && measuring.empty()) break;
        smp.reserve(measuring.size());
        for (int r = 0; r < e->n; ++r) {
            const bool adv = std::find(active.begin(), active.end(), r) != active.end();
            const bool m = std::find(measuring.begin(), measuring.end(), r) != measuring.end();
            if (!adv && !m) continue;
            Lat<R> v = e->view<R>(r, e->j);
            launch_step<R>(v, (adv ? kStore : 0) | (m ? kMeasure : 0), e->launch, nullptr, e->j, e->stream);
            if (m)
                jobs.push_back(FinalizeJobHost{e->part.p + e->poff[r], e->nrp(r),
                                               (double)e->desc[r].Lx * (double)e->desc[r].Ly, smp.take(r)});
        }
        flush_finalize(e, smp, jobs);
        for (int r : active) e->k[r] += 1;
        if (!active.empty()) e->j += 1;
    }
}

// Batched loop: the steps every active replica takes before the next sample
// or end of any of them form a chunk; large replicas advance through one
// tile-table launch per step (after the chunk's first step, runs of 4m steps
// as batched two-step passes for the FP32 replicas whose width that pass
// takes, or several steps per launch on tiles where ens_plan_tiles finds that
// faster), small FP32 replicas through one whole-in-LDS launch per chunk on a
// second stream, or on tiles too; those are still measured in LDS, so a
// sample's sums do not depend on the path.
template <typename R>
static void ens_step_batched(xyl_ensemble* e, uint64_t nsteps, EnsSamples& smp) {
    std::vector<FinalizeJobHost> jobs;
    const bool have_lds = std::any_of(e->lds.begin(), e->lds.end(), [](char c) { return c != 0; });
    if (have_lds) {
        check_hip(hipEventRecord(e->ev_main, e->stream), "hipEventRecord");
        check_hip(hipStreamWaitEvent(e->side, e->ev_main, 0), "hipStreamWaitEvent");
    }
    uint64_t it = 0;
    while (true) {
        std::vector<int> active, meas_g, only_meas_g, lds_set;
        std::vector<char> meas(e->n, 0), act(e->n, 0);
        bool any = false;
        for (int r = 0; r < e->n; ++r) {
            meas[r] = smp.wants(r);
            act[r] = it < nsteps && e->k[r] < e->desc[r].nsteps;
            any = any || meas[r] || act[r];
            if (act[r]) active.push_back(r);
        }
        if (!any) break;
        uint64_t chunk = 0;
        bool any_active = false;
        for (int r = 0; r < e->n; ++r) {
            if (!act[r]) continue;
            uint64_t c = std::min<uint64_t>(nsteps - it, e->desc[r].nsteps - e->k[r]);
            if (smp.every) c = std::min<uint64_t>(c, smp.every - e->k[r] % smp.every);
            chunk = any_active ? std::min(chunk, c) : c;
            any_active = true;
        }
        bool ending = false, lds_sampled = false;
        for (int r : active) {
            ending = ending || e->k[r] + chunk == e->desc[r].nsteps;
            lds_sampled = lds_sampled || (meas[r] && e->lds[r]);
        }
        if (!active.empty()) ens_upload_table<R>(e, e->j, active, chunk, ending, lds_sampled);
        xyl_ensemble::Tables& t = *e->tab;
        bool step_g = false;   // replicas that step on the ensemble's stream and its class streams
        for (int r : active) step_g = step_g || !e->lds[r] || t.tiled[r];
        for (int r = 0; r < e->n; ++r) {
            if (!e->lds[r]) {
                if (meas[r]) (act[r] ? meas_g : only_meas_g).push_back(r);
            } else if (meas[r] || (act[r] && !t.tiled[r])) {
                lds_set.push_back(r);
            }
        }
        size_t nmeas = 0;
        for (int r = 0; r < e->n; ++r) nmeas += meas[r];
        smp.reserve(nmeas);
        // replicas on tiles that are measured in LDS: the sample reads the
        // state the tiles have stepped to, and their next launch that writes
        // over it waits for the sample
        hipEvent_t lds_sample = nullptr;
        bool lds_from_tiles = false;
        for (int r : lds_set) lds_from_tiles = lds_from_tiles || (meas[r] && !t.tiled.empty() && t.tiled[r]);
        if (lds_from_tiles) {
            check_hip(hipEventRecord(e->ev_main, e->stream), "hipEventRecord");
            check_hip(hipStreamWaitEvent(e->side, e->ev_main, 0), "hipStreamWaitEvent");
        }
        // small replicas: one launch for the whole chunk
        if (!lds_set.empty()) {
            // replicas with the factored FP32 kick first, then the others: one
            // launch per form of the kick
            const int b = e->lds_buf;
            e->lds_buf ^= 1;
            // table b was last read by the launch two chunks ago
            if (e->ev_lds_used[b]) check_hip(hipEventSynchronize(e->ev_lds[b]), "hipEventSynchronize");
            std::vector<LdsJobHost> jh;
            jh.reserve(lds_set.size());
            int nfact = 0;
            for (int pass = 0; pass < 2; ++pass)
                for (int r : lds_set) {
                    const xyl_replica_desc& d = e->desc[r];
                    const bool f = kick_factored(Params{d.Jx, d.Jy, d.h, d.gamma, d.dt, d.model, d.p});
                    if (f != (pass == 0)) continue;
                    nfact += f ? 1 : 0;
                    jh.push_back(LdsJobHost{r, meas[r] ? 1 : 0, act[r] && !t.tiled[r] ? (int32_t)chunk : 0, 0,
                                            meas[r] ? smp.take(r) : nullptr});
                }
            // (pinned table b's last copy went with that launch, so it is free)
            e->lds_jobs[b].reserve(jh.size());
            e->lds_jobs_host[b].reserve(jh.size());
            std::memcpy(e->lds_jobs_host[b].p, jh.data(), sizeof(LdsJobHost) * jh.size());
            check_hip(hipMemcpyAsync(e->lds_jobs[b].p, e->lds_jobs_host[b].p, sizeof(LdsJobHost) * jh.size(),
                                     hipMemcpyHostToDevice, e->side),
                      "H2D");
            e->lds_tab_host[b].reserve(e->n);
            Lat<float>* tab = e->lds_tab_host[b].p;
            for (int r = 0; r < e->n; ++r) tab[r] = e->view<float>(r, e->j);
            e->lds_reps[b].reserve(sizeof(Lat<float>) * e->n);
            check_hip(hipMemcpyAsync(e->lds_reps[b].p, tab, sizeof(Lat<float>) * e->n, hipMemcpyHostToDevice, e->side),
                      "H2D");
            const Lat<float>* lreps = reinterpret_cast<const Lat<float>*>(e->lds_reps[b].p);
            if (nfact)
                launch_ensemble_lds(lreps, e->lds_jobs[b].p, nfact, e->lds_threads, e->lds_max_sites, e->model(), true,
                                    e->j, e->side);
            if ((int)lds_set.size() > nfact)
                launch_ensemble_lds(lreps, e->lds_jobs[b].p + nfact, (int)lds_set.size() - nfact, e->lds_threads,
                                    e->lds_max_sites, e->model(), false, e->j, e->side);
            check_hip(hipEventRecord(e->ev_lds[b], e->side), "hipEventRecord");
            e->ev_lds_used[b] = true;
            if (lds_from_tiles) lds_sample = e->ev_lds[b];
        }
        // the replicas on the ensemble's stream
        if (step_g) {
            const Lat<R>* reps = reinterpret_cast<const Lat<R>*>(e->reps.p);
            const size_t ncls = t.s2cls.size(), groups = t.groups();
            const R* ub = static_cast<const R*>(e->u);
            R* u2b = reinterpret_cast<R*>(e->u2.p);
            // group g (a class, or the tiles last) runs on the ensemble's
            // stream (g = 0) or on a stream of its own
            auto stream_of = [&](size_t g, hipStream_t main) { return g == 0 ? main : e->cls_streams[g - 1]; };
            // launch i of nl of the tiles' n steps from step offset jb
            auto tile_launch = [&](uint64_t i, uint64_t nl, uint64_t n, const uint64_t* kdev, uint64_t jb,
                                   hipStream_t st) {
                const uint64_t q = n / nl, m = n % nl, off = i * q + std::min(i, m);
                launch_ensemble_tile<R>(reps, t.tiles.p, t.ntiles, t.tile_shape, t.tile_lds, e->model(),
                                        (int)(q + (i < m ? 1 : 0)), (int)(i & 1), off, ub, u2b, kdev, jb + off, st);
            };
            // With groups the sample is a measurement without a step, and the
            // whole chunk runs in passes and tile launches; otherwise (and in
            // chunks too short for them) the chunk's first step carries it.
            const bool passes = groups > 0 && chunk >= 4;
            uint64_t c = 0;
            bool preforked = false;   // the later groups' first launch already issued (below)
            if (!meas_g.empty()) {
                // several groups issued directly: the groups after the first
                // start their first launch beside the measurement (it reads
                // the sampled state and writes the other buffers); their
                // second, which overwrites that state, waits for the
                // measurement's end
                if (passes && groups > 1 && e->use_graphs != 2) {
                    check_hip(hipEventRecord(e->cls_events[0], e->stream), "hipEventRecord");
                    for (size_t g = 1; g < groups; ++g) {
                        hipStream_t st = stream_of(g, e->stream);
                        check_hip(hipStreamWaitEvent(st, e->cls_events[0], 0), "hipStreamWaitEvent");
                        if (g < ncls) {
                            if constexpr (std::is_same<R, float>::value) {
                                const auto& cl = t.s2cls[g];
                                launch_ensemble_step2(reps, cl.tasks.p, cl.ntasks, cl.waves, cl.partial, cl.max_lx,
                                                      e->model(), 0, ub, u2b, nullptr, e->j, st);
                            }
                        } else {
                            const uint64_t n2 = chunk / 2 * 2;
                            tile_launch(0, tile_launches(n2, t.tile_shape.T), n2, nullptr, e->j, st);
                        }
                    }
                    preforked = true;
                }
                launch_ensemble_step<R>(reps, t.tasks.p, t.ntasks_meas, passes ? kMeasure : (kStore | kMeasure),
                                        e->model(), e->launch.rows, e->launch.wpb, nullptr, e->j, e->stream);
                if (preforked) check_hip(hipEventRecord(e->cls_events[groups], e->stream), "hipEventRecord");
                for (int r : meas_g)
                    jobs.push_back(FinalizeJobHost{e->part.p + e->poff[r], e->nrp(r),
                                                   (double)e->desc[r].Lx * (double)e->desc[r].Ly, smp.take(r)});
                flush_finalize(e, smp, jobs);
            }
            if (!passes) {
                if (lds_sample) check_hip(hipStreamWaitEvent(e->stream, lds_sample, 0), "hipStreamWaitEvent");
                lds_sample = nullptr;
                // (the tiles' replicas measured in LDS take that step here)
                if (!meas_g.empty()) {
                    if (t.ntasks > t.ntasks_meas)
                        launch_ensemble_step<R>(reps, t.tasks.p + t.ntasks_meas, t.ntasks - t.ntasks_meas, kStore,
                                                e->model(), e->launch.rows, e->launch.wpb, nullptr, e->j, e->stream);
                    c = 1;
                }
            }
            // steps c0 .. c0 + n - 1 of the chunk, step offsets jb + c (with
            // kdev, jb = 0 and the device counter holds e->j)
            auto issue = [&](uint64_t c0, uint64_t n, const uint64_t* kdev, uint64_t jb, hipStream_t main) {
                // classes: 4m steps; tiles: an even number; the rest of the
                // chunk in single tile-table steps
                const uint64_t n4 = passes && ncls ? n / 4 * 4 : 0;
                const uint64_t n2 = passes && t.ntiles ? n / 2 * 2 : 0;
                if (n4 || n2) {
                    // with `preforked` (a direct chunk of several groups, from
                    // its start), the later groups are forked and their first
                    // launch issued; their second waits for the sample
                    const bool pre = preforked && c0 == 0 && kdev == nullptr;
                    if (groups > 1 && !pre) {
                        check_hip(hipEventRecord(e->cls_events[0], main), "hipEventRecord");
                        for (size_t g = 1; g < groups; ++g)
                            check_hip(hipStreamWaitEvent(stream_of(g, main), e->cls_events[0], 0), "hipStreamWaitEvent");
                    }
                    // launch by launch across the groups: issued group by
                    // group, a group's first launch would wait for every
                    // launch of the groups before it to be issued (in a
                    // replayed graph, dispatched), and the groups would hardly
                    // overlap
                    const uint64_t np = n4 / 2, nl = n2 ? tile_launches(n2, t.tile_shape.T) : 0;
                    const uint64_t rounds = std::max(np, nl);
                    uint64_t p = 0, l = 0;
                    for (uint64_t r = 0; r < rounds; ++r) {
                        for (; p * rounds < (r + 1) * np && p < np; ++p)
                            for (size_t g = 0; g < ncls; ++g) {
                                hipStream_t st = stream_of(g, main);
                                if (pre && g > 0 && p <= 1) {
                                    if (p == 0) continue;   // issued before the sample
                                    check_hip(hipStreamWaitEvent(st, e->cls_events[groups], 0), "hipStreamWaitEvent");
                                }
                                if constexpr (std::is_same<R, float>::value) {
                                    const auto& cl = t.s2cls[g];
                                    launch_ensemble_step2(reps, cl.tasks.p, cl.ntasks, cl.waves, cl.partial,
                                                          cl.max_lx, e->model(), (int)(p & 1), ub, u2b, kdev,
                                                          jb + c0 + 2 * p, st);
                                }
                            }
                        for (; l * rounds < (r + 1) * nl && l < nl; ++l) {
                            hipStream_t st = stream_of(groups - 1, main);
                            if (pre && groups > 1 && l <= 1) {
                                if (l == 0) continue;
                                check_hip(hipStreamWaitEvent(st, e->cls_events[groups], 0), "hipStreamWaitEvent");
                            }
                            if (l == 1 && lds_sample && kdev == nullptr)
                                check_hip(hipStreamWaitEvent(st, lds_sample, 0), "hipStreamWaitEvent");
                            tile_launch(l, nl, n2, kdev, jb + c0, st);
                        }
                    }
                    for (size_t g = 1; g < groups; ++g) {
                        check_hip(hipEventRecord(e->cls_events[g], e->cls_streams[g - 1]), "hipEventRecord");
                        check_hip(hipStreamWaitEvent(main, e->cls_events[g], 0), "hipStreamWaitEvent");
                    }
                    if (n4 && t.ntasks_rest)
                        for (uint64_t i = 0; i < n4; ++i)
                            launch_ensemble_step<R>(reps, t.tasks_rest.p, t.ntasks_rest, kStore, e->model(),
                                                    e->launch.rows, e->launch.wpb, kdev, jb + c0 + i, main);
                }
                // single steps: tasks [a, b), both sets where both have them left
                for (uint64_t i = std::min(n4, n2); i < n; ++i) {
                    const int a = i >= n4 ? 0 : t.ntasks_flat, b = i >= n2 ? t.ntasks : t.ntasks_flat;
                    if (b > a)
                        launch_ensemble_step<R>(reps, t.tasks.p + a, b - a, kStore, e->model(), e->launch.rows,
                                                e->launch.wpb, kdev, jb + c0 + i, main);
                }
            };
            const uint64_t n = chunk - c;
            // launches the chunk's stepping takes
            uint64_t nl = n;
            if (passes && ncls) nl = n / 4 * 2 * ncls + n % 4 + (t.ntasks_rest ? n / 4 * 4 : 0);
            xyl_ensemble::ChunkGraph* cg = nullptr;
            // (tile launches are few and long enough to be issued directly)
            const bool graphs = e->use_graphs == 2 || (e->use_graphs == 1 && groups <= 1 && t.ntiles == 0);
            if (graphs && nl >= 8) {
                if (e->graphs_built_for != e->graph_version) {
                    e->drop_graphs();
                    e->graphs_built_for = e->graph_version;
                }
                // at most kMaxChunkGraphs chunk shapes hold a graph at a time
                // (adaptive sampling can meet many)
                constexpr size_t kMaxChunkGraphs = 32;
                if (!e->graphs.count({&t, c, n}) && e->graphs.size() >= 4 * kMaxChunkGraphs) e->drop_graphs();
                cg = &e->graphs[{&t, c, n}];
                if (!cg->exec && cg->seen + 1 >= 2) {
                    size_t held = 0;
                    for (auto& g : e->graphs) held += g.second.exec != nullptr;
                    if (held >= kMaxChunkGraphs) {
                        e->drop_graphs();
                        cg = &e->graphs[{&t, c, n}];
                        cg->seen = 1;
                    }
                }
                if (!cg->exec && ++cg->seen >= 2) {
                    // everything that allocates or creates happens before the capture
                    if (!e->cap_stream)
                        check_hip(hipStreamCreateWithFlags(&e->cap_stream, hipStreamNonBlocking), "hipStreamCreate");
                    e->kc.reserve(1);
                    hipGraph_t gr = nullptr;
                    check_hip(hipStreamBeginCapture(e->cap_stream, hipStreamCaptureModeThreadLocal),
                              "hipStreamBeginCapture");
                    try {
                        issue(c, n, e->kc.p, 0, e->cap_stream);
                    } catch (...) {
                        (void)hipStreamEndCapture(e->cap_stream, &gr);
                        if (gr) (void)hipGraphDestroy(gr);
                        throw;
                    }
                    check_hip(hipStreamEndCapture(e->cap_stream, &gr), "hipStreamEndCapture");
                    hipError_t err = hipGraphInstantiate(&cg->exec, gr, nullptr, nullptr, 0);
                    (void)hipGraphDestroy(gr);
                    check_hip(err, "hipGraphInstantiate");
                }
            }
            if (cg && cg->exec) {
                if (lds_sample) check_hip(hipStreamWaitEvent(e->stream, lds_sample, 0), "hipStreamWaitEvent");
                launch_set_counter(e->kc.p, e->j, e->stream);
                check_hip(hipGraphLaunch(cg->exec, e->stream), "hipGraphLaunch");
            } else {
                issue(c, n, nullptr, e->j, e->stream);
            }
        }
        // replicas that only take a sample (a call ending on a sample step):
        // one batched measurement over the task table when they are the
        // replicas it was built for (the same strips and sums as one launch
        // per replica, which took about 1 ms for the 288-replica ensemble)
        const bool batched_only = !only_meas_g.empty() && only_meas_g == t.meas && t.ntasks_meas > 0;
        if (batched_only)
            launch_ensemble_step<R>(reinterpret_cast<const Lat<R>*>(e->reps.p), t.tasks.p, t.ntasks_meas, kMeasure,
                                    e->model(), e->launch.rows, e->launch.wpb, nullptr, e->j, e->stream);
        for (int r : only_meas_g) {
            if (!batched_only) {
                Lat<R> v = e->view<R>(r, e->j);
                launch_step<R>(v, kMeasure, e->launch, nullptr, e->j, e->stream);
            }
            jobs.push_back(FinalizeJobHost{e->part.p + e->poff[r], e->nrp(r),
                                           (double)e->desc[r].Lx * (double)e->desc[r].Ly, smp.take(r)});
        }
        flush_finalize(e, smp, jobs);
        if (!any_active) break;
        for (int r = 0; r < e->n; ++r)
            if (act[r]) e->k[r] += chunk;
        e->j += chunk;
        it += chunk;
    }
    if (have_lds) {
        check_hip(hipEventRecord(e->ev_side, e->side), "hipEventRecord");
        check_hip(hipStreamWaitEvent(e->stream, e->ev_side, 0), "hipStreamWaitEvent");
    }
}

// Launch shape of the tile launches, timed on scratch copies of the state of
// the replicas that use the tile path (graph-captured steps, as for lattices).
template <typename R>
static Launch ensemble_autotune_impl(xyl_ensemble* e) {
    std::vector<int> reps;
    for (int r = 0; r < e->n; ++r)
        if (!e->lds[r]) reps.push_back(r);
    if (reps.empty()) return e->launch;
    const size_t bytes = sizeof(R) * e->total;
    DevBuf<char> tmp;
    tmp.reserve(4 * bytes);   // angles (2), velocities, second velocities of the two-step passes
    for (int b = 0; b < 2; ++b)
        check_hip(hipMemcpyAsync(tmp.p + b * bytes, e->th[b], bytes, hipMemcpyDeviceToDevice, e->stream), "D2D");
    check_hip(hipMemcpyAsync(tmp.p + 2 * bytes, e->u, bytes, hipMemcpyDeviceToDevice, e->stream), "D2D");
    check_hip(hipMemcpyAsync(tmp.p + 3 * bytes, e->u, bytes, hipMemcpyDeviceToDevice, e->stream), "D2D");
    std::vector<Lat<R>> tab(e->n);
    for (int r = 0; r < e->n; ++r) {
        tab[r] = e->view<R>(r, 0);
        tab[r].th[0] = reinterpret_cast<R*>(tmp.p) + e->off[r];
        tab[r].th[1] = reinterpret_cast<R*>(tmp.p + bytes) + e->off[r];
        tab[r].u = reinterpret_cast<R*>(tmp.p + 2 * bytes) + e->off[r];
        tab[r].fresh_k = ~(uint64_t)0;
        tab[r].k_end = ~(uint64_t)0;
    }
    DevBuf<char> dtab;
    dtab.reserve(sizeof(Lat<R>) * e->n);
    check_hip(hipMemcpyAsync(dtab.p, tab.data(), sizeof(Lat<R>) * e->n, hipMemcpyHostToDevice, e->stream), "H2D");
    DevBuf<uint64_t> kc;
    kc.reserve(1);
    launch_set_counter(kc.p, 0, e->stream);
    check_hip(hipStreamSynchronize(e->stream), "hipStreamSynchronize");
    size_t sites = 0;
    for (int r : reps) sites += (size_t)e->desc[r].Lx * e->desc[r].Ly;
    const int steps = (int)std::max<double>(4.0, std::min<double>(256.0, 2.0e11 * 2e-3 / (double)sites));
    hipStream_t cap = nullptr;
    check_hip(hipStreamCreateWithFlags(&cap, hipStreamNonBlocking), "hipStreamCreate");
    hipEvent_t e0, e1;
    check_hip(hipEventCreate(&e0), "hipEventCreate");
    check_hip(hipEventCreate(&e1), "hipEventCreate");
    DevBuf<Task> dtasks;
    Launch best = e->launch;
    float best_ms = 1e30f;
    const int rows_c[] = {1, 2, 4, 8, 16, 32};
    const int wpb_c[] = {1, 2, 4, 8};
    for (int rows : rows_c) {
        std::vector<Task> tk;
        for (int r : reps) {
            const int nxw = (e->desc[r].Lx + kWaveSites - 1) / kWaveSites;
            const int nstrips = (e->desc[r].Ly + rows - 1) / rows;
            for (int st = 0; st < nstrips; ++st)
                for (int x = 0; x < nxw; ++x) tk.push_back(Task{r, x, st, 0});
        }
        dtasks.reserve(tk.size());
        check_hip(hipMemcpy(dtasks.p, tk.data(), sizeof(Task) * tk.size(), hipMemcpyHostToDevice), "H2D");
        for (int w : wpb_c) {
            hipGraph_t g = nullptr;
            hipGraphExec_t ex = nullptr;
            check_hip(hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
            for (int i = 0; i < steps; ++i)
                launch_ensemble_step<R>(reinterpret_cast<const Lat<R>*>(dtab.p), dtasks.p, (int)tk.size(), kStore,
                                        e->model(), rows, w, kc.p, (uint64_t)i, cap);
            check_hip(hipStreamEndCapture(cap, &g), "hipStreamEndCapture");
            hipError_t err = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
            (void)hipGraphDestroy(g);
            check_hip(err, "hipGraphInstantiate");
            check_hip(hipGraphLaunch(ex, e->stream), "hipGraphLaunch");
            float t = 1e30f;
            for (int rep = 0; rep < 2; ++rep) {
                check_hip(hipEventRecord(e0, e->stream), "hipEventRecord");
                check_hip(hipGraphLaunch(ex, e->stream), "hipGraphLaunch");
                check_hip(hipEventRecord(e1, e->stream), "hipEventRecord");
                check_hip(hipEventSynchronize(e1), "hipEventSynchronize");
                float ms = 0.f;
                check_hip(hipEventElapsedTime(&ms, e0, e1), "hipEventElapsedTime");
                t = std::min(t, ms);
            }
            (void)hipGraphExecDestroy(ex);
            if (t < best_ms) {
                best_ms = t;
                best.rows = rows;
                best.wpb = w;
            }
        }
    }
    // Steps per pass (FP32): the two-step classes' passes plus the tile steps
    // of the replicas outside them, against the best tile launch for every
    // step, over the same steps.
    if constexpr (std::is_same<R, float>::value) {
        std::vector<int> active;
        for (int r : reps)
            if (e->k[r] < e->desc[r].nsteps) active.push_back(r);
        const int fusion0 = e->fusion;
        const Launch launch0 = e->launch;
        e->launch = best;
        e->fusion = 2;
        const int steps4 = (steps + 3) / 4 * 4;
        if (!active.empty()) ens_upload_table<R>(e, e->j, active, (uint64_t)steps4, false, false);
        const xyl_ensemble::Tables& tab = *e->tab;
        if (!active.empty() && tab.groups()) {
            const Lat<float>* dreps = reinterpret_cast<const Lat<float>*>(dtab.p);
            const float* ub = reinterpret_cast<const float*>(tmp.p + 2 * bytes);
            float* u2b = reinterpret_cast<float*>(tmp.p + 3 * bytes);
            auto time_graph = [&](auto&& body, int nsteps) {
                hipGraph_t g = nullptr;
                hipGraphExec_t ex = nullptr;
                check_hip(hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
                body();
                check_hip(hipStreamEndCapture(cap, &g), "hipStreamEndCapture");
                hipError_t err = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
                (void)hipGraphDestroy(g);
                check_hip(err, "hipGraphInstantiate");
                check_hip(hipGraphLaunch(ex, e->stream), "hipGraphLaunch");
                float t = 1e30f;
                for (int rep = 0; rep < 2; ++rep) {
                    check_hip(hipEventRecord(e0, e->stream), "hipEventRecord");
                    check_hip(hipGraphLaunch(ex, e->stream), "hipGraphLaunch");
                    check_hip(hipEventRecord(e1, e->stream), "hipEventRecord");
                    check_hip(hipEventSynchronize(e1), "hipEventSynchronize");
                    float ms = 0.f;
                    check_hip(hipEventElapsedTime(&ms, e0, e1), "hipEventElapsedTime");
                    t = std::min(t, ms);
                }
                (void)hipGraphExecDestroy(ex);
                return t / (float)nsteps;
            };
            // the classes' passes as the stepping issues them: on their own
            // streams, pass by pass across the classes, where a chunk with
            // several classes runs direct; one after the other in a graph
            // otherwise
            const size_t ncls = tab.s2cls.size();
            auto classes = [&](hipStream_t main, bool fork) {
                if (fork) {
                    e->class_streams(ncls);
                    check_hip(hipEventRecord(e->cls_events[0], main), "hipEventRecord");
                    for (size_t c2 = 1; c2 < ncls; ++c2)
                        check_hip(hipStreamWaitEvent(e->cls_streams[c2 - 1], e->cls_events[0], 0),
                                  "hipStreamWaitEvent");
                }
                for (int i = 0; i < steps4; i += 4)
                    for (int ph = 0; ph < 2; ++ph)
                        for (size_t c2 = 0; c2 < ncls; ++c2) {
                            const auto& cl = tab.s2cls[c2];
                            launch_ensemble_step2(dreps, cl.tasks.p, cl.ntasks, cl.waves, cl.partial, cl.max_lx,
                                                  e->model(), ph, ub, u2b, kc.p, (uint64_t)(i + 2 * ph),
                                                  fork && c2 > 0 ? e->cls_streams[c2 - 1] : main);
                        }
                if (fork)
                    for (size_t c2 = 1; c2 < ncls; ++c2) {
                        check_hip(hipEventRecord(e->cls_events[c2], e->cls_streams[c2 - 1]), "hipEventRecord");
                        check_hip(hipStreamWaitEvent(main, e->cls_events[c2], 0), "hipStreamWaitEvent");
                    }
                if (tab.ntiles) {
                    const uint64_t nl = tile_launches((uint64_t)steps4, tab.tile_shape.T);
                    const uint64_t q = (uint64_t)steps4 / nl, m = (uint64_t)steps4 % nl;
                    for (uint64_t i = 0, off = 0; i < nl; ++i) {
                        const uint64_t t = q + (i < m ? 1 : 0);
                        launch_ensemble_tile<R>(dreps, tab.tiles.p, tab.ntiles, tab.tile_shape, tab.tile_lds,
                                                e->model(), (int)t, (int)(i & 1), off, ub, u2b, kc.p, off, main);
                        off += t;
                    }
                }
                const Task* single = ncls ? tab.tasks_rest.p : tab.tasks.p;
                const int nsingle = ncls ? tab.ntasks_rest : tab.ntasks_flat;
                if (nsingle)
                    for (int i = 0; i < steps4; ++i)
                        launch_ensemble_step<R>(dreps, single, nsingle, kStore, e->model(), best.rows, best.wpb, kc.p,
                                                (uint64_t)i, main);
            };
            const bool direct = e->use_graphs == 0 || (ncls > 1 && e->use_graphs == 1);
            float t2 = 1e30f;
            if (direct) {
                classes(e->stream, ncls > 1);
                for (int rep = 0; rep < 2; ++rep) {
                    check_hip(hipEventRecord(e0, e->stream), "hipEventRecord");
                    classes(e->stream, ncls > 1);
                    check_hip(hipEventRecord(e1, e->stream), "hipEventRecord");
                    check_hip(hipEventSynchronize(e1), "hipEventSynchronize");
                    float ms = 0.f;
                    check_hip(hipEventElapsedTime(&ms, e0, e1), "hipEventElapsedTime");
                    t2 = std::min(t2, ms / (float)steps4);
                }
            } else {
                t2 = time_graph([&] { classes(cap, false); }, steps4);
            }
            const float t1 = time_graph(
                [&] {
                    for (int i = 0; i < steps4; ++i)
                        launch_ensemble_step<R>(reinterpret_cast<const Lat<R>*>(dtab.p), tab.tasks.p, tab.ntasks,
                                                kStore, e->model(), best.rows, best.wpb, kc.p, (uint64_t)i, cap);
                },
                steps4);
            e->fusion = t2 < t1 ? 2 : 1;
        } else {
            e->fusion = fusion0;
        }
        e->launch = launch0;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    (void)hipStreamDestroy(cap);
    return best;
}

extern "C" {

int xyl_ensemble_autotune(xyl_ensemble* e) {
    return guarded([&] {
        require(e != nullptr, XYL_EINVAL, "NULL handle");
        DeviceGuard g(e->device);
        e->launch = e->dtype == XYL_F64 ? ensemble_autotune_impl<double>(e) : ensemble_autotune_impl<float>(e);
        e->drop_tables();   // the strips have a new height
    });
}

int xyl_ensemble_get_launch(xyl_ensemble* e, int32_t* rows, int32_t* wpb) {
    return guarded([&] {
        require(e != nullptr, XYL_EINVAL, "NULL handle");
        if (rows) *rows = e->launch.rows;
        if (wpb) *wpb = e->launch.wpb;
    });
}

int xyl_ensemble_create(xyl_ensemble** out, const xyl_replica_desc* desc, int32_t n, int32_t dtype, int32_t device) {
    return guarded([&] {
        require(out != nullptr && desc != nullptr, XYL_EINVAL, "NULL argument");
        *out = nullptr;
        require(n >= 1, XYL_EINVAL, "need at least one replica");
        require(dtype == XYL_F32 || dtype == XYL_F64, XYL_EINVAL, "dtype must be XYL_F32 or XYL_F64");
        select_device(device);
        std::unique_ptr<xyl_ensemble> e(new xyl_ensemble());
        e->dtype = dtype;
        e->device = device;
        check_hip(hipDeviceGetAttribute(&e->cus, hipDeviceAttributeMultiprocessorCount, device), "hipDeviceGetAttribute");
        e->n = n;
        e->desc.assign(desc, desc + n);
        for (int r = 0; r < n; ++r) {
            const xyl_replica_desc& d = desc[r];
            validate_shape(d.Lx, d.Ly);
            validate_params(Params{d.Jx, d.Jy, d.h, d.gamma, d.dt, d.model, d.p});
            validate_model(d.model, d.p);
            require(d.model == desc[0].model, XYL_EINVAL, "all replicas of an ensemble must use the same model");
            (void)make_schedule(d.knot_step, d.knot_T, d.nknots, d.knot_gamma);
            e->off.push_back(e->total);
            // keep every replica's base 256-byte aligned
            const size_t N = (size_t)d.Lx * d.Ly;
            e->total += (N + 63) / 64 * 64;
            e->poff.push_back(e->ptotal);
            e->ptotal += part_elems(e->nrp(r));
        }
        load_stepping_kernels(device);
        const size_t bytes = elem_size(dtype) * e->total;
        for (int b = 0; b < 2; ++b) check_alloc(hipMalloc(&e->th[b], bytes), "hipMalloc theta");
        check_alloc(hipMalloc(&e->u, bytes), "hipMalloc velocity");
        e->part.reserve(e->ptotal);
        {
            size_t nph = 0;
            for (int r = 0; r < n; ++r)
                for (int L : {desc[r].Lx, desc[r].Ly})
                    if (e->phase_off.emplace(L, nph).second) nph += 2 * (size_t)L;
            e->phases.reserve(nph);
            for (const auto& t : e->phase_off) launch_phase_table(e->phases.p + t.second, t.first, nullptr);
            check_hip(hipStreamSynchronize(nullptr), "hipStreamSynchronize");
        }
        e->lds.assign(n, 0);
        for (auto& t : e->tables) t.tiled.assign(n, 0);
        for (int r = 0; r < n; ++r) {
            const int N = desc[r].Lx * desc[r].Ly;
            if (dtype == XYL_F32 && N <= kLdsMaxSites) {
                e->lds[r] = 1;
                e->lds_max_sites = std::max(e->lds_max_sites, N);
            }
        }
        if (e->lds_max_sites) {
            e->lds_threads = lds_threads(e->lds_max_sites);
            check_hip(hipStreamCreateWithFlags(&e->side, hipStreamNonBlocking), "hipStreamCreate");
            check_hip(hipEventCreateWithFlags(&e->ev_main, hipEventDisableTiming), "hipEventCreate");
            check_hip(hipEventCreateWithFlags(&e->ev_side, hipEventDisableTiming), "hipEventCreate");
            for (int b = 0; b < 2; ++b)
                check_hip(hipEventCreateWithFlags(&e->ev_lds[b], hipEventDisableTiming), "hipEventCreate");
        }
        e->k.assign(n, 0);
        e->fresh_k.assign(n, 0);
        e->last_sample.assign(n, 0);
        for (int r = 0; r < n; ++r) {
            if (dtype == XYL_F64) launch_init_random<double>(e->view<double>(r, 0), e->stream);
            else launch_init_random<float>(e->view<float>(r, 0), e->stream);
        }
        check_hip(hipStreamSynchronize(e->stream), "hipStreamSynchronize");
        *out = e.release();
    });
}

int xyl_ensemble_destroy(xyl_ensemble* e) {
    if (!e) return XYL_OK;
    return guarded([&] {
        DeviceGuard g(e->device);
        (void)hipStreamSynchronize(e->stream);
        if (e->side) (void)hipStreamSynchronize(e->side);
        for (int b = 0; b < 2; ++b)
            if (e->th[b]) (void)hipFree(e->th[b]);
        if (e->u) (void)hipFree(e->u);
        for (hipStream_t st : e->cls_streams) (void)hipStreamSynchronize(st);
        if (e->side) (void)hipStreamDestroy(e->side);
        if (e->ev_main) (void)hipEventDestroy(e->ev_main);
        if (e->ev_side) (void)hipEventDestroy(e->ev_side);
        for (int b = 0; b < 2; ++b)
            if (e->ev_lds[b]) (void)hipEventDestroy(e->ev_lds[b]);
        for (hipStream_t st : e->cls_streams) (void)hipStreamDestroy(st);
        for (hipEvent_t ev : e->cls_events) (void)hipEventDestroy(ev);
        e->drop_graphs();
        if (e->cap_stream) (void)hipStreamDestroy(e->cap_stream);
        delete e;
    });
}

int xyl_ensemble_set_stream(xyl_ensemble* e, void* stream) {
    return guarded([&] {
        require(e != nullptr, XYL_EINVAL, "NULL handle");
        e->stream = static_cast<hipStream_t>(stream);
    });
}

int xyl_ensemble_set_graphs(xyl_ensemble* e, int32_t enable) {
    return guarded([&] {
        require(e != nullptr, XYL_EINVAL, "NULL handle");
        require(enable >= 0 && enable <= 2, XYL_EINVAL, "enable must be 0, 1 or 2");
        e->use_graphs = enable;
    });
}

int xyl_ensemble_get_fusion(const xyl_ensemble* e, int32_t* steps_per_pass) {
    return guarded([&] {
        require(e != nullptr && steps_per_pass != nullptr, XYL_EINVAL, "NULL argument");
        *steps_per_pass = e->fusion;
    });
}

int xyl_ensemble_set_fusion(xyl_ensemble* e, int32_t steps_per_pass) {
    return guarded([&] {
        require(e != nullptr, XYL_EINVAL, "NULL handle");
        require(steps_per_pass == 1 || steps_per_pass == 2, XYL_EINVAL, "steps_per_pass must be 1 or 2");
        e->fusion = steps_per_pass;
    });
}

int xyl_ensemble_set_mode(xyl_ensemble* e, int32_t mode) {
    return guarded([&] {
        require(e != nullptr, XYL_EINVAL, "NULL handle");
        require(mode == 0 || mode == 1, XYL_EINVAL, "mode must be 0 or 1");
        e->mode = mode;
    });
}

int xyl_ensemble_step(xyl_ensemble* e, uint64_t nsteps, uint64_t every, xyl_obs* out, uint64_t cap, uint64_t* nout) {
    return guarded([&] {
        require(e != nullptr, XYL_EINVAL, "NULL handle");
        if (every) require(out != nullptr && nout != nullptr, XYL_EINVAL, "out/nout are NULL");
        DeviceGuard g(e->device);
        EnsSamples smp(e, every, cap, nout);
        if (e->mode == 1) {
            if (e->dtype == XYL_F64) ens_step_per_replica<double>(e, nsteps, smp);
            else ens_step_per_replica<float>(e, nsteps, smp);
        } else {
            if (e->dtype == XYL_F64) ens_step_batched<double>(e, nsteps, smp);
            else ens_step_batched<float>(e, nsteps, smp);
        }
        smp.finish(out, nout);
    });
}

int xyl_ensemble_get_state(xyl_ensemble* e, int32_t r, double* theta, double* omega, uint64_t* step) {
    return guarded([&] {
        require(e != nullptr && r >= 0 && r < e->n, XYL_EINVAL, "bad handle or replica");
        DeviceGuard g(e->device);
        const size_t N = (size_t)e->desc[r].Lx * e->desc[r].Ly;
        if (theta) {
            if (e->dtype == XYL_F64) to_host<double>(e->cur_theta(r), theta, N, e->stream);
            else to_host<float>(e->cur_theta(r), theta, N, e->stream);
        }
        if (omega) {
            const size_t es = elem_size(e->dtype);
            if (e->k[r] == e->fresh_k[r]) {
                void* up = static_cast<char*>(e->u) + es * e->off[r];
                if (e->dtype == XYL_F64) to_host<double>(up, omega, N, e->stream);
                else to_host<float>(up, omega, N, e->stream);
            } else {
                e->omega_buf.reserve(es * N);
                if (e->dtype == XYL_F64) {
                    Lat<double> v = e->view<double>(r, 0);
                    v.k_end = ~(uint64_t)0;
                    launch_step<double>(v, kOmega, e->launch, nullptr, e->k[r] - v.k_base, e->stream);
                    to_host<double>(e->omega_buf.p, omega, N, e->stream);
                } else {
                    Lat<float> v = e->view<float>(r, 0);
                    v.k_end = ~(uint64_t)0;
                    launch_step<float>(v, kOmega, e->launch, nullptr, e->k[r] - v.k_base, e->stream);
                    to_host<float>(e->omega_buf.p, omega, N, e->stream);
                }
            }
        }
        if (step) *step = e->k[r];
    });
}

int xyl_ensemble_set_state(xyl_ensemble* e, int32_t r, const double* theta, const double* omega, uint64_t step) {
    return guarded([&] {
        require(e != nullptr && r >= 0 && r < e->n, XYL_EINVAL, "bad handle or replica");
        require(theta != nullptr && omega != nullptr, XYL_EINVAL, "theta/omega are NULL");
        const size_t N = (size_t)e->desc[r].Lx * e->desc[r].Ly;
        const bool si = e->model() == kModelSI;
        const double wp = e->dtype == XYL_F64 ? Prec<double>::kHalfPi : (double)Prec<float>::kHalfPi;
        for (size_t i = 0; i < N; ++i) {
            require(std::isfinite(theta[i]) && std::fabs(theta[i]) <= 3.0 * M_PI && std::isfinite(omega[i]), XYL_EINVAL,
                    "state entries must be finite with |theta| <= 3 pi");
            if (si) {
                const double t = e->dtype == XYL_F64 ? theta[i] : (double)(float)theta[i];
                require(t >= -wp && t < wp, XYL_EINVAL, "theta entries must lie in [-pi/2, pi/2) for the SI model");
            }
        }
        DeviceGuard g(e->device);
        e->k[r] = step;
        e->fresh_k[r] = step;
        e->last_sample[r] = 0;
        e->drop_tables();   // they hold the replica's former step
        const size_t es = elem_size(e->dtype);
        void* up = static_cast<char*>(e->u) + es * e->off[r];
        if (e->dtype == XYL_F64) {
            to_device<double>(e->cur_theta(r), theta, N, e->stream);
            to_device<double>(up, omega, N, e->stream);
        } else {
            to_device<float>(e->cur_theta(r), theta, N, e->stream);
            to_device<float>(up, omega, N, e->stream);
        }
    });
}

int xyl_ensemble_domains(xyl_ensemble* e, int32_t r, int32_t* labels, uint64_t* sizes, uint64_t* counts, uint64_t cap,
                         uint64_t* n_sizes, uint64_t* n_domains, uint64_t* max_size) {
    return guarded([&] {
        require(e != nullptr && r >= 0 && r < e->n, XYL_EINVAL, "bad handle or replica");
        DeviceGuard g(e->device);
        const xyl_replica_desc& d = e->desc[r];
        const int sx = d.Jx > 0.0, sy = d.Jy > 0.0;
        if (e->dtype == XYL_F64)
            run_domains<double>(static_cast<const double*>(e->cur_theta(r)), d.Lx, d.Ly, sx, sy, d.model, e->domains,
                                e->stream, labels, sizes, counts, cap, n_sizes, n_domains, max_size);
        else
            run_domains<float>(static_cast<const float*>(e->cur_theta(r)), d.Lx, d.Ly, sx, sy, d.model, e->domains,
                               e->stream, labels, sizes, counts, cap, n_sizes, n_domains, max_size);
    });
}

int xyl_ensemble_structure_factor(xyl_ensemble* e, int32_t r, int32_t axis, int32_t kmax, double* S) {
    return guarded([&] {
        require(e != nullptr && r >= 0 && r < e->n, XYL_EINVAL, "bad handle or replica");
        const xyl_replica_desc& d = e->desc[r];
        validate_sf(d.Lx, d.Ly, axis, kmax, S);
        DeviceGuard g(e->device);
        check_hip(hipStreamSynchronize(e->side), "hipStreamSynchronize");
        const int sx = d.Jx > 0.0, sy = d.Jy > 0.0;
        if (e->dtype == XYL_F64)
            structure_factor_into<double>(e->cur_theta(r), d.Lx, d.Ly, sx, sy, d.model, axis, kmax, e->spectrum,
                                          e->stream, S);
        else
            structure_factor_into<float>(e->cur_theta(r), d.Lx, d.Ly, sx, sy, d.model, axis, kmax, e->spectrum,
                                         e->stream, S);
    });
}

int xyl_ensemble_paths(xyl_ensemble* e, int32_t* path) {
    return guarded([&] {
        require(e != nullptr && path != nullptr, XYL_EINVAL, "NULL argument");
        const xyl_ensemble::Tables& t = *e->tab;
        for (int r = 0; r < e->n; ++r) {
            const xyl_replica_desc& d = e->desc[r];
            const bool two = !t.s2cls.empty() && step2_shape(d.Lx, d.Ly) && replica_factored(d);
            path[r] = t.tiled[r] ? XYL_PATH_TILES : e->lds[r] ? XYL_PATH_LDS : two ? XYL_PATH_TWO_STEP : XYL_PATH_SINGLE;
        }
    });
}

int xyl_ensemble_sync(xyl_ensemble* e) {
    return guarded([&] {
        require(e != nullptr, XYL_EINVAL, "NULL handle");
        DeviceGuard g(e->device);
        check_hip(hipStreamSynchronize(e->stream), "hipStreamSynchronize");
    });
}

}  // extern "C"

// ===================================================================== adjoint
template <typename R>
static void adjoint_forward_impl(xyl_lattice* h, uint64_t N, uint64_t K, uint64_t W, double* loss, uint64_t* run) {
    // the state (buffers, streams, captured backward graphs) is kept from one
    // forward run to the next, so repeated gradient evaluations reuse it
    if (!h->adj) h->adj = new AdjState();
    AdjState* a = static_cast<AdjState*>(h->adj);
    a->valid = false;
    const size_t bytes = sizeof(R) * h->N;
    a->k0 = h->k;
    a->N = N;
    a->K = K;
    a->W = W;
    const uint64_t S = (N + K - 1) / K;
    a->ckpt.reserve(S * 2 * bytes);
    a->obs.reserve(6 * W);
    const uint64_t kw = a->k0 + N - W + 1;   // first step of the loss window
    // the window's measurement partials, one block per step, reduced together
    // at the end (falls back to one reduction per step for huge lattices)
    const uint64_t stride = (uint64_t)h->nrowparts() * kNPart;
    // (on tiles in pieces whose partials take 64 MB at most)
    constexpr uint64_t kMaxWindowBytes = uint64_t(64) << 20;
    const bool tiles = lattice_tile_plan(h, std::min<uint64_t>(K, W)) != nullptr;
    const bool batched = !tiles && (double)W * (double)stride * 8.0 <= 1.0e9;
    if (batched) a->win.reserve(W * stride);
    for (uint64_t s = 0; s < S; ++s) {
        char* slot = a->ckpt.p + s * 2 * bytes;
        check_hip(hipMemcpyAsync(slot, h->cur_theta(), bytes, hipMemcpyDeviceToDevice, h->stream), "D2D");
        check_hip(hipMemcpyAsync(slot + bytes, h->u, bytes, hipMemcpyDeviceToDevice, h->stream), "D2D");
        const uint64_t kend = a->k0 + std::min<uint64_t>((s + 1) * K, N);
        while (h->k < kend) {
            if (h->k >= kw) {
                // the loss needs the order parameter only: on tiles each step
                // sums it beside the stepping
                // (single steps where a piece of the window is too short)
                const TilePlan* tp = tiles ? lattice_tile_plan(h, kend - h->k) : nullptr;
                if (tp) {
                    const size_t parts = (size_t)tile_order_parts(*tp);
                    const uint64_t most = std::max<uint64_t>(kMaxWindowBytes / (parts * sizeof(double)), 64);
                    const uint64_t n = std::min(kend - h->k, most), i = h->k - kw;
                    a->win.reserve(n * parts);
                    lattice_tile_steps<R>(h, *tp, n, a->win.p);
                    launch_tile_order_sum(a->win.p, (int)parts, (double)h->N, a->obs.p + 6 * i, (int)n, h->stream);
                } else if (batched) {
                    lattice_steps_mode<R>(h, kend - h->k, kStore | kMeasure, a->win.p, kw, stride);
                } else {
                    lattice_measure_into<R>(h, true, a->obs.p + 6 * (h->k - kw));
                }
            } else {
                lattice_steps<R>(h, std::min(kend, kw) - h->k);
            }
        }
    }
    if (batched) {
        // the last sample (step k0 + N) is a measurement without a step
        Lat<R> v = h->view<R>();
        v.part = a->win.p;
        v.part_k0 = kw;
        v.part_stride = stride;
        launch_step<R>(v, kMeasure, h->launch, nullptr, h->k, h->stream);
        launch_finalize_many(a->win.p, h->nrowparts(), stride, (double)h->N, a->obs.p, (int)W, h->stream);
    } else {
        lattice_measure_into<R>(h, false, a->obs.p + 6 * (W - 1));
    }
    std::vector<double> o(6 * W);
    check_hip(hipMemcpyAsync(o.data(), a->obs.p, sizeof(double) * 6 * W, hipMemcpyDeviceToHost, h->stream), "D2H");
    check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
    a->m.resize(W);
    double L = 0.0;
    for (uint64_t i = 0; i < W; ++i) {
        a->m[i] = o[6 * i + 2];
        L += a->m[i] * a->m[i];
    }
    a->loss = L / (double)W;
    if (loss) *loss = a->loss;
    a->run = ++g_adj_runs;
    a->version = h->version;
    a->valid = true;
    if (run) *run = a->run;
}

// Gradients of the lattice's adjoint run into grad[4] (host, times `scale`) and dL/dth^{k0},
// dL/dw^{k0}: host float64 arrays (dth0, dom0) or, with dev_out, caller
// device buffers of precision out_f64 (written on the lattice's stream, times
// `scale`).
// Rows per strip of the two-step reverse pass (1, 2 or 4): 2, where its LDS
// fits (512^2: 4.9 us per step, against 5.1 with 1-row strips and 7.8 with
// single reverse steps; 768^2 and 1024^2 within 2% of single reverse steps);
// where it does not (FP64 rows above 568 sites), single reverse steps.
static int adjoint2_rows(const xyl_lattice* h) { return h->adj2_rows ? h->adj2_rows : 2; }

// Times per step (us) of the sweep without tiles, for choosing.  The reverse
// steps go on tiles, but for single ones in FP64 (rows too long for two per pass)
// where those are faster.  Sweeps measured, us per step, tiles for both and
// neither: FP32 512^2 3.8 and 6.3, 1024^2 9.9 and 15.2, 2048^2 32.4 and 43.2,
// 4096^2 124 and 154 (121 with the recompute two steps per pass); FP64 1024^2
// 35.6 and 51.9, 1448^2 69.8 and 79.5, but 2048 x 1024 86 and 73, 2048^2 134 and
// 121, 4096 x 2048 276 and 212.  Reverse on tiles and two steps per pass, the
// recompute on tiles both times, over 60 shapes of up to 2^20 sites in FP64 and 2^24
// in FP32, 4 to 200 steps a segment: FP64 512^2 10.3 and 10.9, 68 x 2400 8.3 and
// 10.8, 200 x 1400 11.1 and 14.4, 512 x 1400 25.6 and 28.0; 128 x 1400 alone 9.7
// and 9.4.
static double adjoint_single_us(const xyl_lattice* h) {
    return h->dtype == XYL_F64 ? 18.0 + (double)h->N / 7.6e4 : 1e30;
}
// (without tiles a segment of K steps, K - 1 of them recomputed, also starts
// with two copies of the checkpoint)
static double adjoint_recompute_us(const xyl_lattice* h, bool two_step, uint64_t K) {
    const double elem = h->dtype == XYL_F64 ? 8.0 : 4.0;
    return (two_step ? 1.15 * step2_us(h->Lx, h->Ly, h->cus, step2_rows(h)) : lattice_single_us(h)) +
           (6.0 + 4.0 * elem * (double)h->N / 4.5e6) / (double)(K - 1);
}

template <typename R>
static void adjoint_backward_impl(xyl_lattice* h, double* grad, void* dth0, void* dom0, bool dev_out, int out_f64,
                                  double scale) {
    AdjState* a = static_cast<AdjState*>(h->adj);
    const size_t bytes = sizeof(R) * h->N;
    const uint64_t N = a->N, K = a->K, W = a->W, k0 = a->k0;
    const uint64_t S = (N + K - 1) / K;
    // direct loss coefficients dL/dm_k * dm_k/d(eps cos th) = (2 m_k / W) / Nsites
    std::vector<double> cmh(N + 1, 0.0);
    for (uint64_t i = 0; i < W; ++i) cmh[N - W + 1 + i] = 2.0 * a->m[i] / (double)W / (double)h->N;
    a->cm.reserve(N + 1);
    check_hip(hipMemcpyAsync(a->cm.p, cmh.data(), sizeof(double) * (N + 1), hipMemcpyHostToDevice, h->stream), "H2D");
    Launch l = h->launch;
    l.wpb = std::min(l.wpb, 4);
    Lat<R> v = h->view<R>();
    // two reverse steps per pass where the rows fit one workgroup's LDS rings
    const int rows2 = adjoint2_rows(h);
    const bool fuse = h->adj_fusion == 2 && adjoint2_fits<R>(v, rows2);
    // two recompute steps per pass (storing the state after each) where the
    // forward's two-step pass takes the lattice whole-row: the same states
    bool rec2 = false;
    if constexpr (std::is_same<R, float>::value)
        rec2 = h->adj_fusion == 2 && v.fact == 1 && v.model == kModelXY && step2_shape(h->Lx, h->Ly);
    // several reverse and several recompute steps per launch on tiles where
    // those are faster by the rules' times, unless the caller shaped the
    // two-step pass
    const bool may_tile = h->adj_fusion == 2 && h->adj2_rows == 0 && K >= 2 && tile_shape_ok(h->Lx, h->Ly);
    if (may_tile && a->tile_K != std::min<uint64_t>(K, 64)) {
        a->tile_K = std::min<uint64_t>(K, 64);
        const bool f64 = h->dtype == XYL_F64;
        if (!tile_plan(h->Lx, h->Ly, f64, h->cus, a->tile_K, &a->rec, &a->rec_us)) a->rec = TilePlan();
        if (!tile_plan_reverse(h->Lx, h->Ly, f64, h->cus, a->tile_K, &a->rev, &a->rev_us)) a->rev = TilePlan();
    }
    const TilePlan &rev = a->rev, &rec = a->rec;
    const bool rev_tiles = may_tile && rev.T > 0 && (fuse || a->rev_us < adjoint_single_us(h));
    const bool rec_tiles = may_tile && rec.T > 0 && a->rec_us < adjoint_recompute_us(h, rec2, K);
    const int ntasks = rev_tiles ? rev.ntx * rev.nty : adjoint_tasks<R>(v, l.rows, fuse ? rows2 : 0);
    a->gacc.reserve((size_t)ntasks * 4);
    check_hip(hipMemsetAsync(a->gacc.p, 0, sizeof(double) * ntasks * 4, h->stream), "hipMemsetAsync");
    a->lam.reserve(4 * bytes);
    R* lt[2] = {reinterpret_cast<R*>(a->lam.p), reinterpret_cast<R*>(a->lam.p + bytes)};
    R* lu[2] = {reinterpret_cast<R*>(a->lam.p + 2 * bytes), reinterpret_cast<R*>(a->lam.p + 3 * bytes)};
    launch_adjoint_seed<R>(v, static_cast<const R*>(h->cur_theta()), lt[0], lu[0], cmh[N], h->stream);
    int li = 0;
    const size_t seg_bytes = (K + 1) * 2 * bytes;
    a->seg.reserve(2 * seg_bytes);
    auto slot_th = [&](int b, uint64_t j) { return reinterpret_cast<R*>(a->seg.p + b * seg_bytes + j * 2 * bytes); };
    auto slot_u = [&](int b, uint64_t j) {
        return reinterpret_cast<R*>(a->seg.p + b * seg_bytes + j * 2 * bytes + bytes);
    };
    a->kseg.reserve(2);
    if (!a->side) {
        check_hip(hipStreamCreateWithFlags(&a->side, hipStreamNonBlocking), "hipStreamCreate");
        for (int b = 0; b < 2; ++b) {
            check_hip(hipEventCreateWithFlags(&a->ev_rec[b], hipEventDisableTiming), "hipEventCreate");
            check_hip(hipEventCreateWithFlags(&a->ev_rev[b], hipEventDisableTiming), "hipEventCreate");
        }
        check_hip(hipEventCreateWithFlags(&a->ev_start, hipEventDisableTiming), "hipEventCreate");
    }
    auto recompute_node = [&](int b, uint64_t j, const uint64_t* kdev, uint64_t kj, hipStream_t st) {
        Lat<R> w = v;
        w.pingpong = 0;
        w.th[0] = slot_th(b, j);
        w.th[1] = slot_th(b, j + 1);
        w.u = slot_u(b, j);
        w.u_out = slot_u(b, j + 1);
        launch_step<R>(w, kStore, h->launch, kdev, kj, st);
    };
    const int rows_rec2 = rec2 ? step2_rows(h) : 0;
    auto recompute_run = [&](int b, uint64_t len, const uint64_t* kdev, uint64_t kbase, hipStream_t st) {
        uint64_t j = 0;
        if constexpr (std::is_same<R, float>::value) {
            if (rec2)
                for (; j + 2 <= len; j += 2)
                    launch_step2_mid(v, slot_th(b, j), slot_u(b, j), slot_th(b, j + 1), slot_u(b, j + 1),
                                     slot_th(b, j + 2), slot_u(b, j + 2), rows_rec2, kdev, kbase + j, st);
        }
        for (; j < len; ++j) recompute_node(b, j, kdev, kbase + j, st);
    };
    auto reverse_node = [&](int b, uint64_t j, int parity, const uint64_t* kdev, uint64_t kj, hipStream_t st) {
        launch_adjoint_step<R>(v, slot_th(b, j), slot_u(b, j), lt[parity], lu[parity], lt[parity ^ 1],
                               lu[parity ^ 1], a->cm.p, k0, a->gacc.p, kdev, kj, l, st);
    };
    // reverse steps j+1 and j of the segment in one pass
    auto reverse2_node = [&](int b, uint64_t j, int parity, const uint64_t* kdev, uint64_t kj, hipStream_t st) {
        launch_adjoint_step2<R>(v, slot_th(b, j), slot_u(b, j), slot_th(b, j + 1), slot_u(b, j + 1), lt[parity],
                                lu[parity], lt[parity ^ 1], lu[parity ^ 1], a->cm.p, k0, a->gacc.p, kdev, kj, rows2,
                                st);
    };
    // the reverse steps len-1 .. 0 of a segment from adjoint buffer `parity`
    // (an odd one first, then pairs); returns the buffer they end in
    auto reverse_segment = [&](int b, uint64_t len, int parity, const uint64_t* kdev, uint64_t kbase,
                               hipStream_t st) {
        uint64_t j = len;
        if (fuse) {
            if (j % 2 == 1) {
                --j;
                reverse_node(b, j, parity, kdev, kbase + j, st);
                parity ^= 1;
            }
            while (j >= 2) {
                j -= 2;
                reverse2_node(b, j, parity, kdev, kbase + j, st);
                parity ^= 1;
            }
        } else {
            while (j-- > 0) {
                reverse_node(b, j, parity, kdev, kbase + j, st);
                parity ^= 1;
            }
        }
        return parity;
    };
    // Full segments of even length replay captured graphs whose step indices
    // come from device counters set to the segment's first step: one graph
    // per buffer for the K recompute steps, one per (buffer, adjoint parity)
    // for the K reverse steps.
    const bool use_graph = h->graph_steps > 1 && K % 2 == 0 && K <= 4096;
    // key: every kernel argument the graphs capture (the lattice view by value,
    // the buffers, the step base and the launch shapes)
    std::vector<uint64_t> key = {K, (uint64_t)(uintptr_t)a->seg.p, (uint64_t)(uintptr_t)a->lam.p,
                                 (uint64_t)(uintptr_t)a->cm.p, (uint64_t)(uintptr_t)a->gacc.p,
                                 (uint64_t)(uintptr_t)a->kseg.p, (uint64_t)l.rows, (uint64_t)l.wpb, (uint64_t)rows2,
                                 (uint64_t)fuse, (uint64_t)rec2, (uint64_t)rows_rec2,
                                 (uint64_t)h->launch.rows, (uint64_t)h->launch.wpb, (uint64_t)ntasks, k0};
    {
        Lat<R> vz{};
        std::memcpy(&vz, &v, sizeof(vz));
        const size_t nw = (sizeof(vz) + 7) / 8;
        std::vector<uint64_t> words(nw, 0);
        std::memcpy(words.data(), &vz, sizeof(vz));
        key.insert(key.end(), words.begin(), words.end());
    }
    if (key != a->graph_key) {
        a->drop_graphs();
        a->graph_key = key;
    }
    auto capture = [&](auto&& body) {
        hipGraph_t gr = nullptr;
        hipGraphExec_t ex = nullptr;
        check_hip(hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
        try {
            body();
        } catch (...) {
            (void)hipStreamEndCapture(h->cap_stream, &gr);
            if (gr) (void)hipGraphDestroy(gr);
            throw;
        }
        check_hip(hipStreamEndCapture(h->cap_stream, &gr), "hipStreamEndCapture");
        hipError_t e = hipGraphInstantiate(&ex, gr, nullptr, nullptr, 0);
        (void)hipGraphDestroy(gr);
        check_hip(e, "hipGraphInstantiate");
        return ex;
    };
    // segment s occupies buffer (S - 1 - s) & 1
    auto recompute_segment = [&](uint64_t s) {
        const int b = (int)((S - 1 - s) & 1);
        const uint64_t ks = k0 + s * K;
        const uint64_t len = std::min<uint64_t>(K, k0 + N - ks);
        const char* ck = a->ckpt.p + s * 2 * bytes;
        if (rec_tiles && len >= 2) {
            // states 1 .. len - 1 (the reverse steps need no more), the
            // checkpoint itself into slot 0 on the way
            const uint64_t n = len - 1, nl = (n + rec.T - 1) / rec.T;
            const R* th_in = reinterpret_cast<const R*>(ck);
            const R* u_in = reinterpret_cast<const R*>(ck + bytes);
            uint64_t j = 0;
            for (uint64_t i = 0; i < nl; ++i) {
                const int t = (int)(n / nl + (i < n % nl ? 1 : 0));
                launch_tile_states<R>(v, th_in, u_in, i == 0, slot_th(b, j + 1), rec, t, ks + j, a->side);
                j += (uint64_t)t;
                th_in = slot_th(b, j);
                u_in = slot_u(b, j);
            }
            check_hip(hipEventRecord(a->ev_rec[b], a->side), "hipEventRecord");
            return;
        }
        check_hip(hipMemcpyAsync(slot_th(b, 0), ck, bytes, hipMemcpyDeviceToDevice, a->side), "D2D");
        check_hip(hipMemcpyAsync(slot_u(b, 0), ck + bytes, bytes, hipMemcpyDeviceToDevice, a->side), "D2D");
        if (len == 1) {
            // a single step: its state is the checkpoint
        } else if (use_graph && len == K) {
            if (!a->rec_graph[b])
                a->rec_graph[b] = capture([&] {
                    recompute_run(b, K, a->kseg.p + 1, 0, h->cap_stream);
                });
            launch_set_counter(a->kseg.p + 1, ks, a->side);
            check_hip(hipGraphLaunch(a->rec_graph[b], a->side), "hipGraphLaunch");
        } else {
            recompute_run(b, len, nullptr, ks, a->side);
        }
        check_hip(hipEventRecord(a->ev_rec[b], a->side), "hipEventRecord");
    };
    // the side stream starts after everything issued so far (checkpoints, seed)
    check_hip(hipEventRecord(a->ev_start, h->stream), "hipEventRecord");
    check_hip(hipStreamWaitEvent(a->side, a->ev_start, 0), "hipStreamWaitEvent");
    recompute_segment(S - 1);
    for (uint64_t s = S; s-- > 0;) {
        const int b = (int)((S - 1 - s) & 1);
        if (s > 0) {
            // the next segment's buffer is free once the reverse that used it ended
            if (S - 1 - s >= 1) check_hip(hipStreamWaitEvent(a->side, a->ev_rev[b ^ 1], 0), "hipStreamWaitEvent");
            recompute_segment(s - 1);
        }
        check_hip(hipStreamWaitEvent(h->stream, a->ev_rec[b], 0), "hipStreamWaitEvent");
        const uint64_t ks = k0 + s * K;
        const uint64_t len = std::min<uint64_t>(K, k0 + N - ks);
        if (rev_tiles) {
            const uint64_t nl = (len + rev.T - 1) / rev.T;
            uint64_t j = len;
            for (uint64_t i = 0; i < nl; ++i) {
                const int t = (int)(len / nl + (i < len % nl ? 1 : 0));
                j -= (uint64_t)t;
                launch_adjoint_tile<R>(v, slot_th(b, j), lt[li], lu[li], lt[li ^ 1], lu[li ^ 1], a->cm.p, k0,
                                       a->gacc.p, rev, t, ks + j, h->stream);
                li ^= 1;
            }
        } else if (use_graph && len == K) {
            int end = li;
            if (!a->rev_graph[b][li])
                a->rev_graph[b][li] = capture([&] { end = reverse_segment(b, K, li, a->kseg.p, 0, h->cap_stream); });
            else
                end = fuse ? li ^ (int)((K / 2) & 1) : li;   // K even
            launch_set_counter(a->kseg.p, ks, h->stream);
            check_hip(hipGraphLaunch(a->rev_graph[b][li], h->stream), "hipGraphLaunch");
            li = end;
        } else {
            li = reverse_segment(b, len, li, nullptr, ks, h->stream);
        }
        check_hip(hipEventRecord(a->ev_rev[b], h->stream), "hipEventRecord");
    }
    constexpr int kR64 = sizeof(R) == 8 ? 1 : 0;
    if (dev_out) {
        // the state adjoints stay on the device: converted (and scaled) into
        // the caller's buffers on the lattice's stream
        if (dth0) launch_convert(lt[li], kR64, dth0, out_f64, h->N, scale, true, h->stream);
        if (dom0) launch_convert(lu[li], kR64, dom0, out_f64, h->N, scale, true, h->stream);
    }
    std::vector<double> g((size_t)ntasks * 4);
    check_hip(hipMemcpyAsync(g.data(), a->gacc.p, sizeof(double) * ntasks * 4, hipMemcpyDeviceToHost, h->stream),
              "D2H");
    if (!dev_out && dth0) {
        std::vector<R> t(h->N);
        check_hip(hipMemcpyAsync(t.data(), lt[li], bytes, hipMemcpyDeviceToHost, h->stream), "D2H");
        check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
        double* o = static_cast<double*>(dth0);
        for (size_t i = 0; i < h->N; ++i) o[i] = (double)t[i];
    }
    if (!dev_out && dom0) {
        std::vector<R> t(h->N);
        check_hip(hipMemcpyAsync(t.data(), lu[li], bytes, hipMemcpyDeviceToHost, h->stream), "D2H");
        check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
        double* o = static_cast<double*>(dom0);
        for (size_t i = 0; i < h->N; ++i) o[i] = (double)t[i];
    }
    check_hip(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
    if (grad) {
        for (int p = 0; p < 4; ++p) grad[p] = 0.0;
        for (int t = 0; t < ntasks; ++t)
            for (int p = 0; p < 4; ++p) grad[p] += g[(size_t)t * 4 + p];
        if (dev_out)
            for (int p = 0; p < 4; ++p) grad[p] *= scale;
    }
}

extern "C" {

int xyl_adjoint_forward(xyl_lattice* h, uint64_t nsteps, uint64_t ckpt_every, uint64_t window, double* loss,
                        uint64_t* run) {
    return guarded([&] {
        require_init(h);
        require(nsteps >= 1, XYL_EINVAL, "nsteps must be >= 1");
        require(window >= 1 && window <= nsteps, XYL_EINVAL, "window must be in [1, nsteps]");
        require(ckpt_every >= 1, XYL_EINVAL, "ckpt_every must be >= 1");
        require(h->p.model == kModelXY, XYL_EUNSUPPORTED,
                "the adjoint needs a smooth force: the SI model's field jumps at the wrap point");
        DeviceGuard g(h->device);
        if (h->dtype == XYL_F64) adjoint_forward_impl<double>(h, nsteps, ckpt_every, window, loss, run);
        else adjoint_forward_impl<float>(h, nsteps, ckpt_every, window, loss, run);
    });
}

// The forward run `run` may be differentiated: it is the lattice's latest,
// and neither the state nor any parameter changed since.
static void require_adjoint_run(xyl_lattice* h, uint64_t run) {
    require_init(h);
    AdjState* a = static_cast<AdjState*>(h->adj);
    require(a != nullptr && a->valid, XYL_ESTATE, "no adjoint forward run to differentiate");
    require(run == a->run, XYL_ESTATE,
            "stale adjoint run: another xyl_adjoint_forward replaced its checkpoints on this lattice");
    require(h->k == a->k0 + a->N && h->version == a->version, XYL_ESTATE,
            "lattice was stepped, reset or reconfigured after xyl_adjoint_forward");
    require(h->p.model == kModelXY, XYL_EUNSUPPORTED, "the adjoint supports the XY model only");
}

int xyl_set_adjoint_fusion(xyl_lattice* h, int32_t steps_per_pass, int32_t rows) {
    return guarded([&] {
        require(h != nullptr, XYL_EINVAL, "NULL handle");
        require(steps_per_pass == 1 || steps_per_pass == 2, XYL_EINVAL, "steps_per_pass must be 1 or 2");
        require(rows == 0 || rows == 1 || rows == 2 || rows == 4, XYL_EINVAL, "rows per strip must be 0, 1, 2 or 4");
        h->adj_fusion = steps_per_pass;
        if (rows) h->adj2_rows = rows;
    });
}

int xyl_adjoint_backward(xyl_lattice* h, uint64_t run, double* grad, double* dtheta0, double* domega0) {
    return guarded([&] {
        require_adjoint_run(h, run);
        DeviceGuard g(h->device);
        if (h->dtype == XYL_F64) adjoint_backward_impl<double>(h, grad, dtheta0, domega0, false, 1, 1.0);
        else adjoint_backward_impl<float>(h, grad, dtheta0, domega0, false, 1, 1.0);
    });
}

int xyl_adjoint_backward_device(xyl_lattice* h, uint64_t run, double scale, double* grad, void* dtheta0,
                                void* domega0, int32_t dtype) {
    return guarded([&] {
        require_adjoint_run(h, run);
        require(dtype == XYL_F32 || dtype == XYL_F64, XYL_EINVAL, "dtype must be XYL_F32 or XYL_F64");
        require(std::isfinite(scale), XYL_EINVAL, "scale must be finite");
        DeviceGuard g(h->device);
        const int of64 = dtype == XYL_F64 ? 1 : 0;
        if (h->dtype == XYL_F64) adjoint_backward_impl<double>(h, grad, dtheta0, domega0, true, of64, scale);
        else adjoint_backward_impl<float>(h, grad, dtheta0, domega0, true, of64, scale);
    });
}

}  // extern "C"
