// lbfv.hip -- host side of liblbfv: contexts, mesh metrics, boundary descriptors,
// launch shapes, HIP graphs, checks, observables, the autotuner and the batched form.
// The public ABI is include/lbfv.h.
#include "lbfv.h"
#include "aux_kernels.hpp"
#include "batch_kernels.hpp"
#include "patch_kernels.hpp"
#include "schedule.hpp"

#include <algorithm>
#include <type_traits>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <map>
#include <mutex>
#include <new>
#include <sstream>
#include <string>
#include <thread>
#include <vector>

using namespace lbfv;

namespace {

thread_local std::string g_last_error;

enum Variant { V_F64 = 0, V_F32 = 1, V_BF16 = 2, V_F16 = 3 };

struct HostCase {
    int nx = 0, ny = 0;
    std::vector<double> xf, yf;
    double rt = 1.0 / 3.0, c = 1.0, tau = 1.0, dt = 1.0;
    int bc[4] = {-1, -1, -1, -1};
    double bcval[4][3] = {};
    int wfrom[4] = {-1, -1, -1, -1};   // south / north wall segment: first cell, or -1
    double wsv[4][2] = {};             // the segment's wall velocity
    int variant = V_F64;
    double rho0 = 0.0;        // 0 for native storage
    double u0[2] = {0.0, 0.0};   // reference velocity of the deviation storage (physical units)
    int strip = STRIP1;       // output columns per 64-slot block of the current state
    int tblock = 1;           // time steps per launch of the single-case step (1 to 4)
    int64_t pitch = 0, plane = 0;
    size_t esize = 8;
    void *buf[2] = {nullptr, nullptr};
    bool own = true;
    bool joint = false;       // both buffers lie in one allocation, buf[0]'s
    int cur = 0;              // buffer holding the current state
    void *d_xm = nullptr, *d_ym = nullptr;   // metrics in the compute type (d_xm owns the block of all four)
    double *d_dx = nullptr, *d_dy = nullptr; // cell sizes (FP64) for volumes
    bool metrics_dirty = true;
    double ext[4] = {0, 0, 0, 0};   // ghost extrapolation factors, of the uploaded metrics

    // buffers fit the state in every strip layout (the narrowest strip pads most)
    size_t buffer_bytes() const { return (size_t)padded_pitch(nx, STRIP4) * ny * 9 * esize; }
    void set_strip(int w) {
        strip = w;
        pitch = padded_pitch(nx, w);
        plane = pitch * ny;
    }
    bool sides_set() const { return bc[0] >= 0 && bc[1] >= 0 && bc[2] >= 0 && bc[3] >= 0; }
    bool periodic_x() const { return bc[SIDE_W] == BC_PERIODIC; }
    bool periodic_y() const { return bc[SIDE_S] == BC_PERIODIC; }
    // the reference state in the kernels' units: rho0 and m0 = rho0 U0 / c
    RefState ref() const { return RefState{rho0, rho0 * u0[0] / c, rho0 * u0[1] / c}; }
};

// Which kernels advance a context: the forms that plan_advance picks by the size of the mesh, until
// the caller sets a march shape (FORM_MARCH) or the autotuner picks one of the two.
enum Form { FORM_AUTO = 0, FORM_MARCH = 1, FORM_PATCH = 2 };

// Patches of a mesh and the waves of a workgroup; cost: what the cost model gives them, us per
// step.  halo = 0: not planned yet; waves = 0: the mesh takes none.  per_wave and max_waves
// are the limits it was made for (at most 64 / per_wave columns, max_waves waves).
struct PatchPlan {
    PatchGrid g = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    int waves = 0;
    int per_wave = 0, max_waves = 0;
    double cost = 0.0;
};

#define HIPCHK(expr)                                                                            \
    do {                                                                                        \
        hipError_t e_ = (expr);                                                                 \
        if (e_ != hipSuccess) {                                                                 \
            return c->fail(LBFV_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_));       \
        }                                                                                       \
    } while (0)

// Fields between caller-owned (pageable) host arrays and the state.  The conversion kernels read
// and write pinned host memory directly, in chunks of cells; a chunk is copied between the
// caller's arrays and its slot of the buffer while other chunks are with the GPU.  Large fields
// take several threads, each with two slots and its own chunks: one thread copies 5 to 10 GB/s
// (the arrays' pages are often touched for the first time), the GPU's link 50.  The buffer and
// its events belong to one context or batch and are kept until it is destroyed; calls from several
// threads (fields of one batch, say) take turns with them.
// No allocation here can throw: the entry points pass no exception on.
struct FieldArrays {   // arrays of one value per cell each
    double *a[12];
    int count = 0;
    // `n` component arrays of one [n][ny][nx] array
    void add(const double *f, int n, int64_t cells) {
        for (int k = 0; k < n; ++k) a[count++] = const_cast<double *>(f) + k * cells;
    }
};
class Transfer {
public:
    // f(range, slot): enqueue the conversion kernel of `range` on the stream
    template <typename F>
    hipError_t run(bool up, int64_t cells, const FieldArrays &arrays, hipStream_t stream, F f) {
        const int64_t width = 8 * (int64_t)arrays.count, total = cells * width;
        // chunks of about 1 MiB; a thread per 2 MiB, at most 8 and half the CPUs
        int threads = (int)std::min<int64_t>({total >> 21, kThreads, (int64_t)std::thread::hardware_concurrency() / 2});
        threads = std::max(threads, 1);
        const std::lock_guard<std::mutex> turn_of(mutex_);
        const int64_t chunk = threads == 1 && total <= kBuffer / 2 ? cells : std::max<int64_t>(1, (1 << 20) / width);
        if (chunk == cells) {
            // one chunk: the stream itself is waited for
            hipError_t e = reserve((size_t)std::max(total, (int64_t)4096), 0);
            if (e != hipSuccess) return e;
            if (up) copy(true, arrays, 0, cells, slot(0, total));
            f(CellRange{0, cells}, slot(0, total));
            e = hipGetLastError();
            const hipError_t done = hipStreamSynchronize(stream);
            if (e == hipSuccess) e = done;
            if (e == hipSuccess && !up) copy(false, arrays, 0, cells, slot(0, total));
            return e;
        }
        hipError_t e = reserve((size_t)std::min<int64_t>(2 * threads * chunk * width, total), 2 * threads + 1);
        if (e != hipSuccess) return e;
        int dev = 0;
        if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
        // The handle hipStreamPerThread means another stream in each thread: what the other threads
        // enqueue has to wait for what is queued on the caller's.
        const bool own_streams = stream == hipStreamPerThread && threads > 1;
        const hipEvent_t queued = events_[2 * threads];
        if (own_streams && (e = hipEventRecord(queued, stream)) != hipSuccess) return e;
        hipError_t result[kThreads] = {};   // (hipSuccess)
        // thread t: chunks t, t + threads, ..., alternating between its two slots
        auto work = [&](int t, int stride) {
            hipError_t &r = result[t];
            if (t && (r = hipSetDevice(dev)) != hipSuccess) return;
            if (t && own_streams && (r = hipStreamWaitEvent(stream, queued, 0)) != hipSuccess) return;
            int64_t from[2] = {0, 0}, count[2] = {0, 0};
            int turn = 0;
            auto finish = [&](int k) {
                if (!count[k] || r != hipSuccess) return;
                if ((r = hipEventSynchronize(events_[2 * t + k])) != hipSuccess) return;
                if (!up) copy(false, arrays, from[k], count[k], slot(2 * t + k, chunk * width));
                count[k] = 0;
            };
            for (int64_t k0 = t * chunk; k0 < cells && r == hipSuccess; k0 += stride * chunk, turn ^= 1) {
                finish(turn);
                if (r != hipSuccess) break;
                double *buf = slot(2 * t + turn, chunk * width);
                from[turn] = k0;
                count[turn] = std::min(chunk, cells - k0);
                if (up) copy(true, arrays, k0, count[turn], buf);
                f(CellRange{k0, count[turn]}, buf);
                if ((r = hipGetLastError()) == hipSuccess) r = hipEventRecord(events_[2 * t + turn], stream);
            }
            finish(turn);
            finish(turn ^ 1);
            // an error leaves kernels that may still use the buffer
            if (r != hipSuccess) (void)hipStreamSynchronize(stream);
        };
        std::thread pool[kThreads];
        int started = 1;
        try {
            for (; started < threads; ++started) pool[started] = std::thread(work, started, threads);
        } catch (...) {
        }
        work(0, threads);
        for (int t = 1; t < started; ++t) pool[t].join();
        // chunks of threads that could not be started
        for (int t = started; t < threads; ++t) work(t, threads);
        const hipError_t done = hipStreamSynchronize(stream);
        for (hipError_t r : result)
            if (r != hipSuccess) return r;
        return done;
    }
    void release() {
        if (pinned_) (void)hipHostFree(pinned_);
        for (; nevents_ > 0; --nevents_) (void)hipEventDestroy(events_[nevents_ - 1]);
        pinned_ = nullptr;
        size_ = 0;
    }

private:
    static constexpr int64_t kBuffer = 16 << 20;   // most bytes kept
    static constexpr int kThreads = 8;
    std::mutex mutex_;
    char *pinned_ = nullptr;
    size_t size_ = 0;
    hipEvent_t events_[2 * kThreads + 1];
    int nevents_ = 0;

    double *slot(int k, int64_t bytes) const {
        return (double *)(pinned_ + std::min<int64_t>(k * bytes, (int64_t)size_ - bytes));
    }
    hipError_t reserve(size_t bytes, int events) {
        hipError_t e;
        if (bytes > size_) {
            if (pinned_) (void)hipHostFree(pinned_);
            pinned_ = nullptr;
            size_ = 0;
            if ((e = hipHostMalloc((void **)&pinned_, bytes, hipHostMallocDefault)) != hipSuccess) {
                (void)hipGetLastError();
                pinned_ = nullptr;
                return e;
            }
            size_ = bytes;
        }
        for (; nevents_ < events; ++nevents_)
            if ((e = hipEventCreateWithFlags(&events_[nevents_], hipEventDisableTiming)) != hipSuccess) return e;
        return hipSuccess;
    }
    static void copy(bool up, const FieldArrays &arrays, int64_t k0, int64_t n, double *buf) {
        for (int a = 0; a < arrays.count; ++a) {
            if (up) memcpy(buf + a * n, arrays.a[a] + k0, n * 8);
            else memcpy(arrays.a[a] + k0, buf + a * n, n * 8);
        }
    }
};

}  // namespace

struct lbfv_ctx {
    HostCase hc;
    int check_every = 1000;
    hipStream_t stream = nullptr;
    int device = -1;                 // the device current at lbfv_create
    bool has_state = false;
    bool unstable = false;
    int64_t steps = 0, steps_at_check = 0;
    int rows = 0, wpb = 4;           // rows 0: not set, default_rows decides
    int pairs = 0;                   // two steps per launch, periodic mesh: a pair of waves per item
    int cus = 0;                     // compute units of the device (0: not asked yet)
    int rows_of[2][5][2] = {};       // default_rows of the BKG / other kernels, time block and pairs (0: not asked yet)
    bool pinned = false;             // a program may hold captured work on the state's layout, or owns the
                                     // buffers: keep it
    int64_t singles = 0;             // one-step launches in a row in the layout of several (no shape set)
    // graphs of `gsteps` launches, per scheme (+4 per further step per launch) and starting buffer
    int gsteps = 32;
    // (16 + scheme: the patch form)
    hipGraphExec_t gexec[20][2] = {};
    int form = FORM_AUTO;
    PatchPlan plan[2];               // patches of the current sides, for the DUGKS and the BKG kernels
    // reductions
    double *d_partial = nullptr, *d_out = nullptr, *h_out = nullptr, *d_uprev = nullptr;
    int red_blocks = 0;
    bool check_pending = false;
    hipEvent_t check_event = nullptr;
    bool uprev_valid = false;
    // parameters of the kernels that take them through a pointer, one slot per scheme:
    // device copy, pinned staging copy, the bytes last uploaded and the event of that upload
    void *d_p2b = nullptr, *h_p2b = nullptr;
    hipEvent_t p2b_event[4] = {};
    bool p2b_pending[4] = {};
    std::vector<char> p2b_last[4];
    Transfer transfer;
    std::string last_error;

    int fail(int status, const std::string &msg) {
        last_error = msg;
        g_last_error = msg;
        return status;
    }
};

struct lbfv_batch {
    std::vector<HostCase> cases;
    int variant = V_F32;
    double rho0 = 1.0;
    hipStream_t stream = nullptr;
    void *d_params = nullptr;        // StepParams<T>[n]
    BatchItem *d_items = nullptr;
    int nitems = 0, rows = 8, gsteps = 100;      // rows: from a sweep on the 96-case batch
    int parity = 0;                  // all cases share the step parity
    int tblock = 1;                  // time steps per launch (1 or 2; 2: 60-column strips)
    bool wave_per_item = false;      // grid of one wave per work item instead of the resident waves
    bool pairs = false;              // two steps per launch: a pair of waves per work item
    bool bnd = false;                // some case has a non-periodic side
    int slots[3][2] = {{0, 0}, {0, 0}, {0, 0}};   // resident work items of the batch kernels: one step, two
                                                   // steps, two steps with pairs of waves; per scheme
    hipGraphExec_t gexec[4][2] = {};              // per scheme (+2: the patch form) and starting buffer
    int form = FORM_AUTO;
    bool captured = false;           // a program may hold captured work on the buffers
    // the patch form, per scheme: halo and waves of all patches (halo 0: not planned yet; waves
    // 0: the batch takes none), their count and what the cost model gives them, us per step
    struct Patches {
        int halo = 0, waves = 0, count = 0;
        double cost = 0.0;
        PatchGrid *d_grids = nullptr;
        PatchItem *d_items = nullptr;
    } patches[2];
    bool has_state = false;
    Transfer transfer;
    std::string last_error;
    int fail(int status, const std::string &msg) {
        last_error = msg;
        g_last_error = msg;
        return status;
    }
};

namespace {

// ------------------------------------------------------------------ metrics
// Cell centres with one ghost on each side: mirrored for walls / inflow / outflow,
// wrapped for a periodic axis (the ghost takes the size of the wrapped cell).
void axis_metrics(const std::vector<double> &f, bool periodic, double dt, double c, std::vector<double> &m,
                  double &ext_lo, double &ext_hi, std::vector<double> &sizes) {
    const int n = (int)f.size() - 1;
    std::vector<double> xc(n + 2);   // xc[i + 1], i = -1..n
    sizes.resize(n);
    for (int i = 0; i < n; ++i) {
        sizes[i] = f[i + 1] - f[i];
        xc[i + 1] = 0.5 * (f[i] + f[i + 1]);
    }
    if (periodic) {
        xc[0] = f[0] - 0.5 * sizes[n - 1];
        xc[n + 1] = f[n] + 0.5 * sizes[0];
    } else {
        xc[0] = f[0] - 0.5 * sizes[0];
        xc[n + 1] = f[n] + 0.5 * sizes[n - 1];
    }
    auto X = [&](int i) { return xc[i + 1]; };
    m.assign(4 * n + 2, 0.0);
    for (int g = 0; g <= n; ++g) {
        const double d = X(g) - X(g - 1);
        m[g] = (f[g] - X(g - 1)) / d;
        m[n + 1 + g] = 1.0 / d;
    }
    if (periodic) {
        // faces 0 and n are the same face of a periodic axis: one set of values, so
        // that every march evaluates it identically whichever end it reaches it from
        m[n] = m[0];
        m[n + 1 + n] = m[n + 1];
    }
    for (int i = 0; i < n; ++i) {
        m[2 * n + 2 + i] = 1.0 / (X(i + 1) - X(i - 1));
        m[3 * n + 2 + i] = dt * c / sizes[i];
    }
    ext_lo = (X(0) - X(-1)) / (X(1) - X(0));
    ext_hi = (X(n) - X(n - 1)) / (X(n - 1) - X(n - 2));
}

template <typename T>
void copy_as(const std::vector<double> &in, std::vector<T> &out) {
    out.resize(in.size());
    for (size_t i = 0; i < in.size(); ++i) out[i] = (T)in[i];
}

template <typename T>
StepParams<T> make_params(const HostCase &h, double ext[4], int scheme = SCHEME_DUGKS) {
    StepParams<T> P;
    memset(&P, 0, sizeof(P));
    const RefState R = h.ref();
    P.buf[0] = h.buf[0];
    P.buf[1] = h.buf[1];
    P.nx = h.nx;
    P.ny = h.ny;
    P.pitch = h.pitch;
    P.plane = h.plane;
    P.strip = h.strip;
    P.xm = (const T *)h.d_xm;
    P.ym = (const T *)h.d_ym;
    for (int s = 0; s < 4; ++s) {
        P.bc[s] = h.bc[s];
        P.ext[s] = (T)ext[s];
        // walls: the bounce-back's momentum term relative to the reference momentum
        // (F_a - F_rev(a) = 6 w_a e_a.m0 cancels from it)
        if (h.bc[s] == BC_WALL) {
            P.bcv[s][0] = (T)(6.0 * (h.bcval[s][0] / h.c - R.m0x));
            P.bcv[s][1] = (T)(6.0 * (h.bcval[s][1] / h.c - R.m0y));
        } else if (h.bc[s] == BC_INFLOW) {
            P.bcv[s][0] = (T)h.bcval[s][0];
            P.bcv[s][1] = (T)(h.bcval[s][1] / h.c);
            P.bcv[s][2] = (T)(h.bcval[s][2] / h.c);
        } else if (h.bc[s] == BC_OUTFLOW) {
            P.bcv[s][0] = (T)h.bcval[s][0];
        }
        P.wfrom[s] = h.wfrom[s];
        P.wsv[s][0] = (T)(6.0 * (h.wsv[s][0] / h.c - R.m0x));
        P.wsv[s][1] = (T)(6.0 * (h.wsv[s][1] / h.c - R.m0y));
    }
    const double tau = h.tau, dt = h.dt, hh = 0.5 * dt;
    P.rho0 = (T)h.rho0;
    P.m0x = (T)R.m0x;
    P.m0y = (T)R.m0y;
    if (h.rho0 > 0) {
        const double ux = h.u0[0] / h.c, uy = h.u0[1] / h.c;
        for (int a = 0; a < 9; ++a) {
            const double eu = EX[a] * ux + EY[a] * uy;
            P.q0[a] = (T)(h.rho0 * (4.5 * eu * eu - 1.5 * (ux * ux + uy * uy)));
        }
    }
    for (int s = 0; s < 4; ++s) {
        P.gext[s] = (h.bc[s] == BC_OUTFLOW && h.bcval[s][0] < 0.5) ? (T)0 : P.ext[s];
        if (h.bc[s] == BC_INFLOW) {
            // the inflow ghost state: the kernels' equilibrium of (rho, u), formed once here
            const T rho = P.bcv[s][0], ux = P.bcv[s][1], uy = P.bcv[s][2];
            const T mx = kRefVel<T> ? fmaT(rho, ux, -P.m0x) : rho * ux;
            const T my = kRefVel<T> ? fmaT(rho, uy, -P.m0y) : rho * uy;
            for (int a = 0; a < 9; ++a)
                P.gin[s][a] = dfeq<T>(a, rho - P.rho0, rho, mx, my, ux, uy, usq_term<T>(ux, uy),
                                      kRefVel<T> ? P.q0[a] : (T)0);
        }
    }
    P.hc = (T)(hh * h.c);
    P.cb = (T)(3.0 * hh / (2.0 * tau + dt));
    P.cd = (T)(2.0 * dt / (2.0 * tau + dt));
    P.m2 = (T)(hh / (2.0 * tau + hh));
    if (scheme == SCHEME_CENTRAL || scheme == SCHEME_UPWIND) {
        // Sec. 2.4, Eqs. cfd1 / cfd2: the face value is built from f itself,
        // f = x + dt/(2 tau + dt) (feq - x), and is used as it is (collision ignored);
        // the central form takes no characteristic trace.
        P.cb = (T)(dt / (2.0 * tau + dt));
        P.m2 = (T)0;
        if (scheme == SCHEME_CENTRAL) P.hc = (T)0;
    }
    return P;
}

bool is_f64(int v) { return v == V_F64; }

// (Re)build and upload the per-axis metric arrays of a case.  Returns a HIP error.
hipError_t upload_metrics(HostCase &h, double ext[4], hipStream_t s) {
    std::vector<double> mx, my, sx, sy;
    axis_metrics(h.xf, h.periodic_x(), h.dt, h.c, mx, ext[SIDE_W], ext[SIDE_E], sx);
    axis_metrics(h.yf, h.periodic_y(), h.dt, h.c, my, ext[SIDE_S], ext[SIDE_N], sy);
    // one block on the device, x and y metrics, then cell sizes, and one copy into it
    const size_t tsz = is_f64(h.variant) ? 8 : 4;
    const size_t nmx = mx.size() * tsz, nmy = my.size() * tsz, at_dx = (nmx + nmy + 7) / 8 * 8;
    std::vector<char> block(at_dx + (sx.size() + sy.size()) * 8);
    if (tsz == 8) {
        memcpy(block.data(), mx.data(), nmx);
        memcpy(block.data() + nmx, my.data(), nmy);
    } else {
        std::vector<float> fx, fy;
        copy_as(mx, fx);
        copy_as(my, fy);
        memcpy(block.data(), fx.data(), nmx);
        memcpy(block.data() + nmx, fy.data(), nmy);
    }
    memcpy(block.data() + at_dx, sx.data(), sx.size() * 8);
    memcpy(block.data() + at_dx + sx.size() * 8, sy.data(), sy.size() * 8);
    hipError_t e;
    if (!h.d_xm) {
        if ((e = hipMalloc(&h.d_xm, block.size())) != hipSuccess) return e;
        h.d_ym = (char *)h.d_xm + nmx;
        h.d_dx = (double *)((char *)h.d_xm + at_dx);
        h.d_dy = h.d_dx + sx.size();
    }
    if ((e = hipMemcpyAsync(h.d_xm, block.data(), block.size(), hipMemcpyHostToDevice, s)) != hipSuccess) return e;
    // the host block dies here: wait for the copy
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    h.metrics_dirty = false;
    memcpy(h.ext, ext, sizeof(h.ext));
    return hipSuccess;
}

// The two state buffers of a case, zeroed (the pad slots are never read by the step, but are kept
// defined); small ones in one allocation.
hipError_t allocate_buffers(HostCase &h, hipStream_t s) {
    const size_t bytes = (h.buffer_bytes() + 255) / 256 * 256;
    h.joint = bytes <= (16 << 20);
    hipError_t e = hipMalloc(&h.buf[0], h.joint ? 2 * bytes : bytes);
    if (e == hipSuccess && h.joint) h.buf[1] = (char *)h.buf[0] + bytes;
    if (e == hipSuccess && !h.joint) e = hipMalloc(&h.buf[1], bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        if (h.buf[0]) (void)hipFree(h.buf[0]);
        h.buf[0] = h.buf[1] = nullptr;
        return e;
    }
    h.own = true;
    e = hipMemsetAsync(h.buf[0], 0, h.joint ? 2 * bytes : bytes, s);
    if (e == hipSuccess && !h.joint) e = hipMemsetAsync(h.buf[1], 0, bytes, s);
    return e;
}
void free_buffers(HostCase &h) {
    if (h.own) {
        if (h.buf[0]) (void)hipFree(h.buf[0]);
        if (h.buf[1] && !h.joint) (void)hipFree(h.buf[1]);
    }
    h.buf[0] = h.buf[1] = nullptr;
    h.joint = false;
}

void free_case(HostCase &h) {
    free_buffers(h);
    if (h.d_xm) (void)hipFree(h.d_xm);
    h.d_xm = h.d_ym = nullptr;
    h.d_dx = h.d_dy = nullptr;
}

// ------------------------------------------------------------------ kernel dispatch
struct StepShape {
    int rows, wpb, nstrips, nwork, nblocks;
    int side_rows = 0;        // pairs with x sides: rows of the row blocks of the strips at the sides,
    uint32_t side_step = 0;   // and their share of the items in 2^-32, rounded up (0: as the others)
};
StepShape step_shape(const HostCase &h, int rows, int wpb) {
    StepShape s;
    s.rows = rows;
    s.wpb = wpb;
    s.nstrips = (h.nx + h.strip - 1) / h.strip;
    s.nwork = s.nstrips * ((h.ny + rows - 1) / rows);
    s.nblocks = (s.nwork + wpb - 1) / wpb;
    return s;
}

// Shorter row blocks for the strips at the x sides of a mesh that a pair of waves per item
// advances.  A row takes longer there (ghost cells, wall faces), and where all items run at once
// those strips set the time of the launch.  With blocks of 1 / 1.3 of the rows, those that fill and
// drain the levels included, they end with the others; us per step with blocks of 1, 1 / 1.15,
// 1 / 1.3 and 1 / 1.6: 1024^2 cavity, 19 rows, FP64 DUGKS 25.0, 23.7, 23.2, 23.2, BKG 23.4, 22.4,
// 21.9, 21.9, FP32 20.4, 18.8, 18.1, 18.1; 1200^2, 26 rows, FP64 DUGKS 31.4, 28.9, 28.2, 28.3.
int side_block_rows(int rows) { return std::max(1, (rows + 4) * 10 / 13 - 4); }
// work items with the sides' row blocks of `side_rows`
int64_t items_with_sides(const HostCase &h, int nstrips, int rows, int side_rows) {
    return (int64_t)(nstrips - 2) * ((h.ny + rows - 1) / rows) + 2 * (int64_t)((h.ny + side_rows - 1) / side_rows);
}
bool has_side_strips(const HostCase &h, int nstrips) { return !h.periodic_x() && nstrips >= 3; }
// They go only as far as the additional items leave the items per SIMD what they were (a pair puts
// a wave on two of a CU's four SIMDs).
void balance_sides(const HostCase &h, int cus, StepShape &s) {
    if (!has_side_strips(h, s.nstrips) || cus <= 0) return;
    const int64_t quantum = 2 * cus, loads = (s.nwork + quantum - 1) / quantum;
    for (int rows = side_block_rows(s.rows); rows < s.rows; ++rows) {
        const int64_t n = items_with_sides(h, s.nstrips, s.rows, rows);
        if ((n + quantum - 1) / quantum > loads) continue;
        s.side_rows = rows;
        s.side_step = (uint32_t)((2ull * (uint64_t)((h.ny + rows - 1) / rows) * (1ull << 32) + n - 1) / n);
        s.nwork = (int)n;
        return;
    }
}

// Kernels of a mesh with a non-periodic side read their parameters through a device copy
// (passed by value, the parameters of the longer march with sides spill from the scalar
// registers); doubly periodic meshes pass them by value.
bool params_by_pointer(bool bnd) { return bnd; }

// one step per launch
template <typename T, typename S, bool REF>
void *step_fn(int scheme, bool bnd) {
    if (bnd) {
        return scheme == SCHEME_BKG ? (void *)step_ptr_kernel<T, S, SCHEME_BKG, REF>
                                    : (void *)step_ptr_kernel<T, S, SCHEME_DUGKS, REF>;
    }
    return scheme == SCHEME_BKG ? (void *)step_kernel<T, S, SCHEME_BKG, false, REF>
                                : (void *)step_kernel<T, S, SCHEME_DUGKS, false, REF>;
}
template <typename T, typename S, bool REF>
void *step2_fn(int scheme, bool bnd) {
    if (bnd) {
        return scheme == SCHEME_BKG ? (void *)step2b_ptr_kernel<T, S, SCHEME_BKG, REF>
                                    : (void *)step2b_ptr_kernel<T, S, SCHEME_DUGKS, REF>;
    }
    return scheme == SCHEME_BKG ? (void *)step2_kernel<T, S, SCHEME_BKG, REF>
                                : (void *)step2_kernel<T, S, SCHEME_DUGKS, REF>;
}
// two steps per launch, a pair of waves per work item (bnd: some side is not periodic;
// that form reads its parameters through the device copy)
template <typename T, typename S, bool REF>
void *step2p_fn(int scheme, bool bnd) {
    if (bnd)
        return scheme == SCHEME_BKG ? (void *)step2bp_kernel<T, S, SCHEME_BKG, REF>
                                    : (void *)step2bp_kernel<T, S, SCHEME_DUGKS, REF>;
    return scheme == SCHEME_BKG ? (void *)step2p_kernel<T, S, SCHEME_BKG, REF>
                                : (void *)step2p_kernel<T, S, SCHEME_DUGKS, REF>;
}
// K steps per launch on a doubly periodic mesh, a chain of K waves per work item (K = 3, 4)
template <typename T, typename S, bool REF>
void *stepc_fn(int scheme, int K) {
    if (K == 3)
        return scheme == SCHEME_BKG ? (void *)stepc_kernel<T, S, SCHEME_BKG, REF, 3>
                                    : (void *)stepc_kernel<T, S, SCHEME_DUGKS, REF, 3>;
    return scheme == SCHEME_BKG ? (void *)stepc_kernel<T, S, SCHEME_BKG, REF, 4>
                                : (void *)stepc_kernel<T, S, SCHEME_DUGKS, REF, 4>;
}
// The kernel of a variant; ref: the FP32 forms with the reference-velocity terms (a
// reference velocity is set), else without them.  FP64 has none.
#define LBFV_PICK(FN, variant, ref, ...)                                                        \
    switch (variant) {                                                                        \
    case V_F64: return FN<double, double, false>(__VA_ARGS__);                                \
    case V_F32: return ref ? FN<float, float, true>(__VA_ARGS__) : FN<float, float, false>(__VA_ARGS__); \
    case V_BF16: return ref ? FN<float, __bf16, true>(__VA_ARGS__) : FN<float, __bf16, false>(__VA_ARGS__); \
    default: return ref ? FN<float, _Float16, true>(__VA_ARGS__) : FN<float, _Float16, false>(__VA_ARGS__); \
    }
void *step2p_fn_variant(int variant, int scheme, bool bnd, bool ref) { LBFV_PICK(step2p_fn, variant, ref, scheme, bnd) }
// two steps per launch; bnd: some side is not periodic
void *step2_fn_variant(int variant, int scheme, bool bnd, bool ref) { LBFV_PICK(step2_fn, variant, ref, scheme, bnd) }
// bnd: some side is not periodic (ghost cells / walls present)
void *step_fn_variant(int variant, int scheme, bool bnd, bool ref) { LBFV_PICK(step_fn, variant, ref, scheme, bnd) }
// K = 3, 4 steps per launch (doubly periodic meshes only)
void *stepc_fn_variant(int variant, int scheme, int K, bool ref) { LBFV_PICK(stepc_fn, variant, ref, scheme, K) }
// the patch form; bnd: some side is not periodic
template <typename T, typename S, bool REF>
void *patch_fn(int scheme, bool bnd) {
    if (bnd)
        return scheme == SCHEME_BKG ? (void *)patch_ptr_kernel<T, S, SCHEME_BKG, REF>
                                    : (void *)patch_ptr_kernel<T, S, SCHEME_DUGKS, REF>;
    return scheme == SCHEME_BKG ? (void *)patch_kernel<T, S, SCHEME_BKG, REF>
                                : (void *)patch_kernel<T, S, SCHEME_DUGKS, REF>;
}
void *patch_fn_variant(int variant, int scheme, bool bnd, bool ref) { LBFV_PICK(patch_fn, variant, ref, scheme, bnd) }
#undef LBFV_PICK
template <typename T, typename S, bool BND>
void *batch_fn_b(int scheme, bool two, bool pairs) {
    if (two && pairs)
        return scheme == SCHEME_DUGKS ? (void *)batch2p_kernel<T, S, SCHEME_DUGKS, BND>
                                      : (void *)batch2p_kernel<T, S, SCHEME_BKG, BND>;
    if (two)
        return scheme == SCHEME_DUGKS ? (void *)batch2_kernel<T, S, SCHEME_DUGKS, BND>
                                      : (void *)batch2_kernel<T, S, SCHEME_BKG, BND>;
    return scheme == SCHEME_DUGKS ? (void *)batch_kernel<T, S, SCHEME_DUGKS, BND>
                                  : (void *)batch_kernel<T, S, SCHEME_BKG, BND>;
}
template <typename T, typename S>
void *batch_fn(int scheme, bool bnd, bool two, bool pairs) {
    return bnd ? batch_fn_b<T, S, true>(scheme, two, pairs) : batch_fn_b<T, S, false>(scheme, two, pairs);
}
template <typename T, typename S>
void *batch_patch_fn(int scheme, bool bnd) {
    if (bnd)
        return scheme == SCHEME_DUGKS ? (void *)batch_patch_kernel<T, S, SCHEME_DUGKS, true>
                                      : (void *)batch_patch_kernel<T, S, SCHEME_BKG, true>;
    return scheme == SCHEME_DUGKS ? (void *)batch_patch_kernel<T, S, SCHEME_DUGKS, false>
                                  : (void *)batch_patch_kernel<T, S, SCHEME_BKG, false>;
}
void *batch_patch_fn_variant(int variant, int scheme, bool bnd) {
    switch (variant) {
    case V_F64: return batch_patch_fn<double, double>(scheme, bnd);
    case V_F32: return batch_patch_fn<float, float>(scheme, bnd);
    case V_BF16: return batch_patch_fn<float, __bf16>(scheme, bnd);
    default: return batch_patch_fn<float, _Float16>(scheme, bnd);
    }
}
// two: two time steps per launch (the cases in the 60-column strip layout); pairs: with a
// pair of waves per work item
void *batch_fn_variant(int variant, int scheme, bool bnd, bool two, bool pairs = false) {
    switch (variant) {
    case V_F64: return batch_fn<double, double>(scheme, bnd, two, pairs);
    case V_F32: return batch_fn<float, float>(scheme, bnd, two, pairs);
    case V_BF16: return batch_fn<float, __bf16>(scheme, bnd, two, pairs);
    default: return batch_fn<float, _Float16>(scheme, bnd, two, pairs);
    }
}

bool has_boundary(const HostCase &h) { return !(h.periodic_x() && h.periodic_y()); }
// the FP32 step kernels with the reference-velocity terms: only while a reference velocity is set
bool ref_terms(const HostCase &h) { return !is_f64(h.variant) && (h.u0[0] != 0.0 || h.u0[1] != 0.0); }

// A wall segment on a mesh that is periodic in x ends at the seam, and the two cells that meet there
// see each other's ghost row differently: to cell 0 the column west of it lies ahead of the segment,
// to cell nx - 1 the column east of it lies in the segment, while each takes its own rule for itself.
// A launch of one step evaluates the seam once for each of them, in the outer lanes of two strips.
// One of several steps would need both values of either cell at every level, so such a mesh
// advances one step per launch, whatever shape is set.
bool one_step_only(const HostCase &h) { return h.periodic_x() && (h.wfrom[SIDE_S] >= 0 || h.wfrom[SIDE_N] >= 0); }

// ------------------------------------------------------------------ patches
// Widest extent, ghost and halo cells included, of `parts` patches along an axis of n cells.
// Patches within a halo of a non-periodic side are cut off by it (at most 9 of them per end),
// the others differ in length only (patch r is the first short one).
int patch_extent(int n, bool periodic, int parts, int halo) {
    const int q = n / parts, r = n % parts;
    auto extent = [&](int p) {
        const int o0 = p * q + std::min(p, r), o1 = o0 + q + (p < r ? 1 : 0);
        const int lo = periodic ? o0 - halo : std::max(o0 - halo, -1);
        const int hi = periodic ? o1 + halo : std::min(o1 + halo, n + 1);
        return hi - lo;
    };
    int w = std::max(extent(r), extent(std::max(r - 1, 0)));
    for (int p = 0; p < std::min(parts, 10); ++p) w = std::max(w, std::max(extent(p), extent(parts - 1 - p)));
    return w;
}
// Fewest patches along an axis whose extent fits `cap` cells (0: none does).
int patch_parts(int n, bool periodic, int halo, int cap) {
    if (!periodic && n + 2 <= cap) return 1;
    // an end patch holds a ghost cell and one halo, the others two halos
    const int edge = cap - halo - (periodic ? halo : 1), inner = cap - 2 * halo;
    if (edge < 1) return 0;
    const int last = inner < 1 ? std::min(n, 2) : std::min(n, (n + inner - 1) / inner);
    for (int parts = std::max(1, (n + edge - 1) / edge); parts <= last; ++parts)
        if (patch_extent(n, periodic, parts, halo) <= cap) return parts;
    return 0;
}
constexpr int PATCH_HALO = 8;   // most steps per launch of the patch form
// Largest mesh that takes the patch form at all where no launch shape was set: in 16-bit storage, and
// in FP64 and FP32 in short calls (patch_cells is the line of calls of any length).  Against one-step
// marches of the default shape, us per step (DUGKS and BKG in FP64, then in FP32): 64^2 vortex
// 1.7 / 1.3 / 1.4 / 1.2 against 11.6 / 8.9 / 10.6 / 8.4, 512^2 cavity 13 / 8 / 7 / 5 against 32 / 28
// / 28 / 24, 1024^2 vortex 30 / 23 / 20 / 15 against 50 / 49 / 30 / 28, 1024^2 cavity 39 / 26 / 24 /
// 16 against 63 / 54 / 37 / 34.
constexpr int64_t PATCH_CELLS = 1 << 20;
// Largest mesh of a batch that takes it where no launch shape was set.  Against one-step marches
// of the default shape, us per step (DUGKS and BKG in FP64, then in FP32): 100 cavities of 64^2
// 19 / 14 / 12 / 9 against 41 / 32 / 22 / 20, 6 of 512^2 59 / 41 / 36 / 25 against 75 / 65 / 56 / 38;
// 96 uneven cases of 64^2 to 512^2 in FP32 210 / 154 against 213 / 208.
constexpr int64_t BATCH_PATCH_CELLS = 1 << 18;
// The autotuner tries it on meshes up to PATCH_CELLS too.  Its marches of several steps pass the patch
// form from about 410^2 cells (FP64) and 610^2 (FP32) on doubly periodic meshes, with sides from
// 510^2 and 740^2 (the lines of patch_cells); in 16-bit storage they round less often, but on larger
// meshes patches still beat those of one step.

// Largest mesh on which a launch of one step takes patches; above, a march of one step (in the same
// layout, with the same bits) comes cheaper than a halo made for several.  us a call of one step,
// patches and marches: FP64 DUGKS periodic 640^2 21.7 and 25.6, 680^2 29.6 and 25.3, BKG 570^2 19.3
// and 22.8, 600^2 25.3 and 22.9; FP32 DUGKS 720^2 17.9 and 21.3, 1000^2 37.9 and 30.7, cavity 800^2
// 28.7 and 29.1, 1000^2 48.0 and 37.2; BKG 640^2 14.9 and 16.1, 680^2 19.5 and 16.3, cavity 680^2
// 20.0 and 24.8, 800^2 29.7 and 25.1.
int64_t patch_single_cells(bool f64, int scheme) { return f64 ? 340000 : (scheme == SCHEME_BKG ? 440000 : 640000); }
// And the cells of all cases of a batch.  FP64 224 x 32^2 18.3 (cavities, DUGKS) and 23.5, 512^2 24.9
// and 19.4; FP32 512^2 14.2 and 16.8, 8 x 256^2 26.7 and 21.4, 24 of 64^2 to 512^2 105 and 56.
int64_t batch_single_cells(bool f64) { return f64 ? 240000 : 350000; }

// Patches of at most 64 / per_wave columns and waves x per_wave rows with the given halo.
bool plan_patch(const HostCase &h, int per_wave, int waves, int halo, PatchPlan &p) {
    PatchGrid &g = p.g;
    g.halo = halo;
    p.waves = 0;
    p.per_wave = per_wave;
    p.max_waves = waves;
    if (h.plane * (int64_t)h.esize >= (1ll << 31)) return false;   // 32-bit offsets within a plane
    if (one_step_only(h)) return false;
    if ((h.periodic_x() && h.nx <= halo) || (h.periodic_y() && h.ny <= halo)) return false;   // the halo wraps once
    g.npx = patch_parts(h.nx, h.periodic_x(), halo, 64 / per_wave);
    g.npy = g.npx ? patch_parts(h.ny, h.periodic_y(), halo, waves * per_wave) : 0;
    if (!g.npy) return false;
    g.tw = patch_extent(h.nx, h.periodic_x(), g.npx, halo);
    g.fit = 64 / g.tw;
    g.qx = h.nx / g.npx;
    g.rx = h.nx % g.npx;
    g.qy = h.ny / g.npy;
    g.ry = h.ny % g.npy;
    p.waves = (patch_extent(h.ny, h.periodic_y(), g.npy, halo) + g.fit - 1) / g.fit;
    return true;
}

// What the cost model needs of the device: CUs, and the workgroups of a patch kernel that fit
// on a CU with at most 4 and at most 8 waves each.  A workgroup's waves go round the four SIMDs
// from the first one on, so that its share of a SIMD is 1 or 2 waves whatever the others hold.
struct PatchDevice {
    int cus = 256;
    int fit[2] = {1, 1};
};
PatchDevice patch_device(bool f64, void *fn) {
    PatchDevice d;
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
        d.cus = n;
    for (int k = 0; k < 2; ++k) {
        const int lanes = 256 * (k + 1);
        const size_t lds = (size_t)PATCH_LDS * lanes * (f64 ? 8 : 4);
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, lanes, lds) == hipSuccess && n > 0) d.fit[k] = n;
        else (void)hipGetLastError();
    }
    return d;
}

// us per step of `groups` workgroups of at most 4 or 8 waves, `halo` steps per launch, from
// timings on gfx950 (meshes of 32^2 to 1024^2 alone and in batches, both schemes and precisions,
// every halo and workgroup size).  A launch costs 1.4 us.  Where all workgroups are resident at
// once, or a CU takes one at a time, latency counts, per round: 1.6 us and 0.4 us per resident
// wave of a SIMD for addresses, loads and stores, and per step a part that one wave alone cannot
// hide (barriers, dependent arithmetic; 0.6 us more where patches hold ghost cells) and a part
// per resident wave.  Otherwise the workgroups hide each other's waits and their throughput counts,
// per wave of a SIMD: loads and stores and the steps' arithmetic, but at least the time of its
// memory traffic.  Of 640 plans of single meshes 75 % lie within 15 % of their timings and 97 % within
// 30 %, of 600 of batches 50 and 83 %; the halo that the model picks is the fastest or equal in half of
// the cases, 22 % slower at worst (profiles/patch_form_timings.txt has them all).
double patch_cost(bool f64, bool bkg, bool bnd, const PatchDevice &d, int64_t groups, int waves, int halo) {
    const int per_cu = (int)((groups + d.cus - 1) / d.cus), fit = d.fit[waves > 4];
    const int share = std::min(per_cu, fit) * (waves > 4 ? 2 : 1);   // resident waves of a SIMD
    if (per_cu <= fit || fit == 1) {
        const int rounds = (per_cu + fit - 1) / fit;
        const double alone = (f64 ? (bkg ? 0.55 : 0.3) : 0.35) + (bnd ? 0.6 : 0.0);
        const double each = f64 ? (bkg ? 0.33 : 0.75) : (bkg ? 0.2 : 0.5);
        return (1.4 + rounds * (1.6 + 0.4 * share + halo * (alone + each * share))) / halo;
    }
    const double least = f64 ? (bkg ? 2.0 : 2.6) : (bkg ? 1.6 : 2.05);
    const double load = f64 ? (bkg ? 1.4 : 1.7) : (bkg ? 0.85 : 0.7);
    const double step = f64 ? (bkg ? 0.33 : 0.57) : (bkg ? 0.2 : 0.45);
    return (1.4 + ((double)per_cu / fit + 0.3) * share * std::max(least, load + halo * step)) / halo;
}

// The cheapest plan of the cost model with a halo in [lo, hi] (waves = 0: the mesh takes none).
PatchPlan best_patch_plan(const HostCase &h, const PatchDevice &d, int scheme, int lo = 1, int hi = PATCH_HALO) {
    PatchPlan best, p;
    best.g.halo = lo;
    for (int halo = lo; halo <= hi; ++halo)
        for (int per_wave = 1; per_wave <= 6; ++per_wave)
            for (int waves : {2, 4, 8}) {
                if (!plan_patch(h, per_wave, waves, halo, p)) continue;
                p.cost = patch_cost(is_f64(h.variant), scheme == SCHEME_BKG, has_boundary(h), d,
                                    (int64_t)p.g.npx * p.g.npy, p.waves, halo);
                if (!best.waves || p.cost < best.cost) best = p;
            }
    return best;
}

// Kernel arguments of one step launch, in a form usable by hipLaunchKernel and by
// graph kernel nodes.
struct StepArgs {
    StepParams<double> pd;
    StepParams<float> pf;
    const void *pptr = nullptr;   // device copy of the parameters, for kernels that take a pointer
    int parity, rows, nstrips, nwork;
    int side_rows;
    uint32_t side_step;
    int steps;                    // patch form: steps of the launch and the patches
    PatchGrid grid;
    void *args[7];
    void bind(bool f64) {
        args[0] = f64 ? (void *)&pd : (void *)&pf;
        args[1] = &parity;
        args[2] = &rows;
        args[3] = &nstrips;
        args[4] = &nwork;
        args[5] = &side_rows;
        args[6] = &side_step;
    }
    void bind_patch(const PatchGrid &g, int n) {
        grid = g;
        steps = n;
        args[2] = &steps;
        args[3] = &grid;
    }
};

void fill_args(const HostCase &h, const double ext[4], const StepShape &sh, int parity, int scheme, StepArgs &a) {
    double e[4] = {ext[0], ext[1], ext[2], ext[3]};
    if (is_f64(h.variant)) a.pd = make_params<double>(h, e, scheme);
    else a.pf = make_params<float>(h, e, scheme);
    a.parity = parity;
    a.rows = sh.rows;
    a.nstrips = sh.nstrips;
    a.nwork = sh.nwork;
    a.side_rows = sh.side_rows;
    a.side_step = sh.side_step;
    a.bind(is_f64(h.variant));
}

// compute units of the current device (0: unknown)
int device_cus() {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess)
        return n;
    (void)hipGetLastError();
    return 0;
}

// Wave slots the step kernel can keep resident on the whole device (CUs x waves per CU).
int resident_waves(void *fn, int wpb) {
    int dev = 0, blocks = 0;
    hipDeviceProp_t p;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&p, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, (const void *)fn, 64 * wpb, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return blocks * wpb * p.multiProcessorCount;
}

// Row-block heights whose wave count fills the resident slots in k whole rounds:
// few prologue rows re-read and no partial last round (strip: output columns per wave).
// sides: room for the row blocks that balance_sides makes.
std::vector<int> balanced_rows(const HostCase &h, int slots, int strip, int kmax = 4, bool sides = false) {
    std::vector<int> out;
    if (slots <= 0) return out;
    const int nstrips = (h.nx + strip - 1) / strip;
    for (int k = 1; k <= kmax; ++k) {
        const int blocks = (k * slots) / nstrips;   // row blocks per strip
        if (blocks < 1) continue;
        int r = (h.ny + blocks - 1) / blocks;
        if (sides && has_side_strips(h, nstrips))
            while (r < h.ny && items_with_sides(h, nstrips, r, side_block_rows(r)) > (int64_t)k * slots) ++r;
        if (r >= 4 && r <= h.ny) out.push_back(r);
    }
    return out;
}

// Rows of the row blocks of chains of tb waves where none were set.  With `load` chains on a CU, as
// many as all its items need, a launch takes (rows + 3 tb)(1 + x waves) units: an item's own rows and
// those that fill and drain its levels, each longer by x for every wave on the fullest SIMD (300^2
// and 450^2, 2 to 17 rows; more chains than are resident take turns).  One chain per CU on
// small meshes is then better than all that fit: 300^2 FP64 DUGKS 8 rows (228 items) 5.25 us a step,
// 6 (300) 6.27, 4 (450) 5.59.  In FP32 arithmetic blocks of more than 100 rows lose to more rounds:
// 4096^2 FP32 DUGKS 316, 122 and 64 rows 173, 159 and 163 us, FP16 173, 157 and 161.
int chain_rows(const HostCase &h, int scheme, int tb, int resident, int cus) {
    const int strip = SLOTS - 2 * tb, nstrips = (h.nx + strip - 1) / strip;
    const int fit = std::max(1, resident / cus);   // chains of a CU
    const bool f64 = is_f64(h.variant), bkg = scheme == SCHEME_BKG;
    const double x = f64 ? (bkg ? 0.32 : 0.49) : (bkg ? 0.17 : 0.21);
    int best = 0;
    double least = 0;
    for (int load = 1; load <= 8 * fit; ++load) {
        const int blocks = (int)std::min<int64_t>((int64_t)load * cus / nstrips, h.ny);
        if (blocks < 1) continue;
        const int rows = (h.ny + blocks - 1) / blocks, rest = load % fit;
        if (!f64 && rows > 100 && load < 8 * fit) continue;
        auto share = [&](int chains) { return (tb * chains + 3) / 4; };   // waves on the fullest SIMD
        const double cost = (rows + 3 * tb) * (load / fit * (1 + x * share(fit)) + (rest ? 1 + x * share(rest) : 0));
        if (!best || cost < least) {
            best = rows;
            least = cost;
        }
    }
    return best;
}

// Row-block height of a march whose height was not set.  One step per launch: 8 or 16 rows, and
// on large meshes one round of resident waves.  Two steps per launch: k whole rounds of resident
// work items (waves or pairs), k such that the rows a slot marches are fewest, each item's own and
// the 6 that fill and drain its levels (1024^2 FP64 DUGKS: 40 rows; 512^2: 11).
int default_rows(const HostCase &h, int scheme, int wpb, int tb = 1, bool pairs = false) {
    const int64_t cells = (int64_t)h.nx * h.ny;
    const bool bnd = !(h.periodic_x() && h.periodic_y()), ref = ref_terms(h);
    if (tb >= 3) {
        const int waves = resident_waves(stepc_fn_variant(h.variant, scheme, tb, ref), tb), cus = device_cus();
        const int rows = waves > 0 && cus > 0 ? chain_rows(h, scheme, tb, waves / tb, cus) : 0;
        if (rows) return rows;
    } else if (tb == 2) {
        const int slots = pairs ? resident_waves(step2p_fn_variant(h.variant, scheme, bnd, ref), 2) / 2
                                : resident_waves(step2_fn_variant(h.variant, scheme, bnd, ref), wpb);
        const int strip = SLOTS - 2 * tb, nstrips = (h.nx + strip - 1) / strip;
        int best = 0, least = 0;
        for (int k = 1; k <= 8; ++k) {
            const int blocks = std::min(k * slots / nstrips, h.ny);
            if (blocks < 1) continue;
            int rows = (h.ny + blocks - 1) / blocks;
            if (pairs && has_side_strips(h, nstrips))   // room for balance_sides
                while (rows < h.ny && items_with_sides(h, nstrips, rows, side_block_rows(rows)) > (int64_t)k * slots) ++rows;
            const int cost = k * (rows + 3 * tb);
            if (!best || cost < least) {
                best = rows;
                least = cost;
            }
        }
        if (best) return best;
    }
    if (cells >= (1 << 22)) {
        // large meshes: one round of resident waves, of the strips that the state is laid out in now
        // (heights made for 62 columns overflow the round in 56: 4096^2 FP64 DUGKS, one step a call
        // after a long one, 652 us, and 565 with heights made for 56)
        auto r = balanced_rows(h, resident_waves(step_fn_variant(h.variant, scheme, bnd, ref), wpb), h.strip);
        if (!r.empty()) return r[0];
        return std::min(64, h.ny);
    }
    return std::min(cells >= (1 << 18) ? 16 : 8, h.ny);
}

}  // namespace

// ====================================================================== context
extern "C" {

const char *lbfv_strerror(int status) {
    switch (status) {
    case LBFV_OK: return "ok";
    case LBFV_EINVAL: return "invalid argument";
    case LBFV_ESTATE: return "invalid state for this call";
    case LBFV_ENOMEM: return "out of memory";
    case LBFV_EHIP: return "HIP runtime error";
    case LBFV_EUNSTABLE: return "non-finite value found (unstable run)";
    case LBFV_EUNSUPPORTED: return "unsupported";
    default: return "unknown status";
    }
}

const char *lbfv_last_error(const lbfv_ctx *ctx) {
    return ctx ? ctx->last_error.c_str() : g_last_error.c_str();
}

const char *lbfv_batch_last_error(const lbfv_batch *b) {
    return b ? b->last_error.c_str() : g_last_error.c_str();
}

int lbfv_dt_from_cfl(const lbfv_mesh *mesh, double rt, double cfl, double *dt) {
    if (!mesh || !dt || !mesh->xf || !mesh->yf || mesh->nx < 1 || mesh->ny < 1 || !(rt > 0) || !(cfl > 0)) {
        g_last_error = "lbfv_dt_from_cfl: bad argument";
        return LBFV_EINVAL;
    }
    double dmin = INFINITY;
    for (int i = 0; i < mesh->nx; ++i) dmin = std::min(dmin, mesh->xf[i + 1] - mesh->xf[i]);
    for (int j = 0; j < mesh->ny; ++j) dmin = std::min(dmin, mesh->yf[j + 1] - mesh->yf[j]);
    if (!(dmin > 0)) {
        g_last_error = "lbfv_dt_from_cfl: faces not strictly increasing";
        return LBFV_EINVAL;
    }
    *dt = cfl * dmin / std::sqrt(6.0 * rt);
    return LBFV_OK;
}

}  // extern "C"

namespace {

int validate_case(const lbfv_mesh *mesh, const lbfv_velset *vel, double tau, double dt, int compute, int storage,
                  std::string &msg) {
    if (!mesh || !vel) { msg = "NULL mesh or velocity set"; return LBFV_EINVAL; }
    if (mesh->nx < 2 || mesh->ny < 2) { msg = "nx and ny must be >= 2"; return LBFV_EINVAL; }
    if (!mesh->xf || !mesh->yf) { msg = "NULL face coordinates"; return LBFV_EINVAL; }
    for (int i = 0; i < mesh->nx; ++i)
        if (!(mesh->xf[i + 1] > mesh->xf[i])) { msg = "x faces not strictly increasing"; return LBFV_EINVAL; }
    for (int j = 0; j < mesh->ny; ++j)
        if (!(mesh->yf[j + 1] > mesh->yf[j])) { msg = "y faces not strictly increasing"; return LBFV_EINVAL; }
    if (vel->q != 9) { msg = "only D2Q9 (q = 9) is provided"; return LBFV_EINVAL; }
    if (!(vel->rt > 0) || !std::isfinite(vel->rt)) { msg = "rt must be > 0"; return LBFV_EINVAL; }
    if (!(tau > 0) || !(dt > 0) || !std::isfinite(dt)) { msg = "tau and dt must be > 0"; return LBFV_EINVAL; }
    if (compute != LBFV_FP64 && compute != LBFV_FP32) { msg = "compute must be LBFV_FP64 or LBFV_FP32"; return LBFV_EINVAL; }
    if (storage < LBFV_STORE_NATIVE || storage > LBFV_STORE_DEV_FP16) { msg = "unknown storage"; return LBFV_EINVAL; }
    if (compute == LBFV_FP64 && storage != LBFV_STORE_NATIVE) {
        msg = "deviation / 16-bit storage needs FP32 compute";
        return LBFV_EINVAL;
    }
    return LBFV_OK;
}

void init_host_case(HostCase &h, const lbfv_mesh *mesh, const lbfv_velset *vel, double tau, double dt, int compute,
                    int storage, double rho0) {
    h.nx = mesh->nx;
    h.ny = mesh->ny;
    h.xf.assign(mesh->xf, mesh->xf + mesh->nx + 1);
    h.yf.assign(mesh->yf, mesh->yf + mesh->ny + 1);
    h.rt = vel->rt;
    h.c = std::sqrt(3.0 * vel->rt);
    h.tau = tau;
    h.dt = dt;
    if (compute == LBFV_FP64) h.variant = V_F64;
    else if (storage == LBFV_STORE_DEV_BF16) h.variant = V_BF16;
    else if (storage == LBFV_STORE_DEV_FP16) h.variant = V_F16;
    else h.variant = V_F32;
    h.rho0 = storage == LBFV_STORE_NATIVE ? 0.0 : rho0;
    h.esize = h.variant == V_F64 ? 8 : (h.variant == V_F32 ? 4 : 2);
    h.set_strip(STRIP1);   // strip-padded rows (see kernels.hpp)
}

int set_side(HostCase &h, int side, int kind, double a, double b, double c) {
    if (side < 0 || side > 3) return LBFV_EINVAL;
    // a periodic axis is set as a whole: replacing one side of it clears the other
    const int other = side ^ 1;
    if (h.bc[side] == BC_PERIODIC && kind != BC_PERIODIC && h.bc[other] == BC_PERIODIC) h.bc[other] = -1;
    h.bc[side] = kind;
    h.wfrom[side] = -1;       // a new kind replaces the whole side
    h.bcval[side][0] = a;
    h.bcval[side][1] = b;
    h.bcval[side][2] = c;
    h.metrics_dirty = true;
    return LBFV_OK;
}

}  // namespace

// internal helpers operating on a context
namespace {

void drop_graphs(lbfv_ctx *c) {
    for (auto &row : c->gexec)
        for (auto &g : row)
            if (g) {
                (void)hipGraphExecDestroy(g);
                g = nullptr;
            }
}

int ensure_buffers(lbfv_ctx *c) {
    HostCase &h = c->hc;
    if (h.buf[0]) return LBFV_OK;
    const hipError_t e = allocate_buffers(h, c->stream);
    if (!h.buf[0]) return c->fail(LBFV_ENOMEM, "cannot allocate the two state buffers");
    HIPCHK(e);
    drop_graphs(c);
    return LBFV_OK;
}

int ensure_metrics(lbfv_ctx *c, double ext[4]) {
    HostCase &h = c->hc;
    if (h.metrics_dirty) {
        if (!h.sides_set()) return c->fail(LBFV_ESTATE, "all four sides must be set");
        HIPCHK(upload_metrics(h, ext, c->stream));
        drop_graphs(c);
        c->plan[0] = c->plan[1] = PatchPlan();   // (the patches depend on the kinds of sides)
        memset(c->rows_of, 0, sizeof(c->rows_of));
    }
    return LBFV_OK;
}

// current extrapolation factors (of the uploaded metrics, or formed on the host)
void current_ext(const HostCase &h, double ext[4]) {
    if (!h.metrics_dirty) {
        memcpy(ext, h.ext, sizeof(h.ext));
        return;
    }
    std::vector<double> m, s;
    axis_metrics(h.xf, h.periodic_x(), h.dt, h.c, m, ext[SIDE_W], ext[SIDE_E], s);
    axis_metrics(h.yf, h.periodic_y(), h.dt, h.c, m, ext[SIDE_S], ext[SIDE_N], s);
}

void *patch_kernel_of(const lbfv_ctx *c, int scheme) {
    return patch_fn_variant(c->hc.variant, scheme, has_boundary(c->hc), ref_terms(c->hc));
}
// the patches of a scheme's kernels, planned on first use
PatchPlan &patch_plan(lbfv_ctx *c, int scheme) {
    PatchPlan &p = c->plan[scheme == SCHEME_BKG];
    if (!p.g.halo) p = best_patch_plan(c->hc, patch_device(is_f64(c->hc.variant), patch_kernel_of(c, scheme)), scheme);
    return p;
}
// grid, workgroup and LDS of a patch launch
void patch_dims(const lbfv_ctx *c, const PatchPlan &p, dim3 &grid, dim3 &block, unsigned &lds) {
    grid = dim3(p.g.npx * p.g.npy);
    block = dim3(64 * p.waves);
    lds = (unsigned)(PATCH_LDS * 64 * p.waves * (is_f64(c->hc.variant) ? 8 : 4));
}

// a launch of two steps with the pair-of-waves form (also where no shape was set)
bool paired(const lbfv_ctx *c, int tb) { return tb == 2 && (c->pairs || c->form == FORM_AUTO); }
// rows of the row blocks of a launch of tb steps
int march_rows(lbfv_ctx *c, int scheme, int tb) {
    if (c->rows > 0) return c->rows;
    int &rows = c->rows_of[scheme == SCHEME_BKG][tb][paired(c, tb)];
    if (!rows) rows = default_rows(c->hc, scheme, c->wpb, tb, paired(c, tb));
    return rows;
}

int device_cus(lbfv_ctx *c) {
    if (!c->cus) c->cus = device_cus();
    return c->cus;
}
// the shape of a march of tb steps per launch
StepShape march_shape(lbfv_ctx *c, int scheme, int tb) {
    StepShape sh = step_shape(c->hc, march_rows(c, scheme, tb), c->wpb);
    if (paired(c, tb) && !c->hc.periodic_x()) balance_sides(c->hc, device_cus(c), sh);
    return sh;
}

// the step kernel of a launch of tb steps: a chain of tb waves per work item (tb = 3, 4;
// doubly periodic meshes), two steps (in a strip layout of 60 columns or fewer; with or
// without non-periodic sides; one wave or a pair of waves per work item), or one
void *launch_fn(const lbfv_ctx *c, int scheme, int tb) {
    const HostCase &h = c->hc;
    const bool bnd = has_boundary(h), ref = ref_terms(h);
    if (tb >= 3) return stepc_fn_variant(h.variant, scheme, tb, ref);
    if (paired(c, tb)) return step2p_fn_variant(h.variant, scheme, bnd, ref);
    return tb == 2 ? step2_fn_variant(h.variant, scheme, bnd, ref) : step_fn_variant(h.variant, scheme, bnd, ref);
}
// grid and workgroup of a launch: wpb items of one wave per workgroup, or one item of a
// pair (a chain) of waves per workgroup
void launch_dims(const lbfv_ctx *c, int tb, const StepShape &sh, dim3 &grid, dim3 &block) {
    if (tb >= 3 || paired(c, tb)) {
        grid = dim3(sh.nwork);
        block = dim3(64 * tb);
    } else {
        grid = dim3(sh.nblocks);
        block = dim3(64 * sh.wpb);
    }
}

// Device copy of the launch parameters for the kernels that take them through a pointer
// (params_by_pointer), one slot per scheme.
// A changed set is staged in pinned memory and copied on the context's stream, so launches
// queued before the copy still read the previous set; the staging slot is rewritten only
// after its previous copy has run.
constexpr size_t P2B_SLOT = (sizeof(StepParams<double>) + 255) / 256 * 256;
static_assert(sizeof(StepParams<float>) <= P2B_SLOT, "parameter slot too small");

int p2b_upload(lbfv_ctx *c, int scheme, const void *p, size_t bytes, const void **dptr) {
    if (!c->d_p2b) {
        void *d = nullptr, *hs = nullptr;
        if (hipMalloc(&d, 4 * P2B_SLOT) != hipSuccess || hipHostMalloc(&hs, 4 * P2B_SLOT, hipHostMallocDefault) != hipSuccess) {
            if (d) (void)hipFree(d);
            (void)hipGetLastError();
            return c->fail(LBFV_ENOMEM, "cannot allocate the launch parameter copy");
        }
        for (auto &e : c->p2b_event)
            if (!e && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
                (void)hipFree(d);
                (void)hipHostFree(hs);
                return c->fail(LBFV_EHIP, "hipEventCreate failed");
            }
        c->d_p2b = d;
        c->h_p2b = hs;
    }
    char *d = (char *)c->d_p2b + scheme * P2B_SLOT, *hs = (char *)c->h_p2b + scheme * P2B_SLOT;
    std::vector<char> &last = c->p2b_last[scheme];
    if (last.size() != bytes || memcmp(last.data(), p, bytes) != 0) {
        if (c->p2b_pending[scheme]) HIPCHK(hipEventSynchronize(c->p2b_event[scheme]));
        memcpy(hs, p, bytes);
        last.assign((const char *)p, (const char *)p + bytes);
        HIPCHK(hipMemcpyAsync(d, hs, bytes, hipMemcpyHostToDevice, c->stream));
        HIPCHK(hipEventRecord(c->p2b_event[scheme], c->stream));
        c->p2b_pending[scheme] = true;
    }
    *dptr = d;
    return LBFV_OK;
}

// the arguments of a launch; the kernels that read their parameters through a pointer get
// the device copy
int launch_args(lbfv_ctx *c, int scheme, int parity, const double ext[4], const StepShape &sh, StepArgs &a) {
    HostCase &h = c->hc;
    fill_args(h, ext, sh, parity, scheme, a);
    if (params_by_pointer(has_boundary(h))) {
        const bool f64 = is_f64(h.variant);
        int st = p2b_upload(c, scheme, f64 ? (const void *)&a.pd : (const void *)&a.pf, f64 ? sizeof(a.pd) : sizeof(a.pf),
                            &a.pptr);
        if (st) {
            // a failed upload must not leave a stale record of what the device holds
            c->p2b_last[scheme].clear();
            return st;
        }
        a.args[0] = &a.pptr;
    }
    return LBFV_OK;
}

// one launch of `steps` time steps of the patch form
int launch_patch(lbfv_ctx *c, int scheme, int parity, const double ext[4], int steps) {
    HostCase &h = c->hc;
    const PatchPlan &p = patch_plan(c, scheme);
    StepShape sh = step_shape(h, 1, 1);
    StepArgs a;
    int st = launch_args(c, scheme, parity, ext, sh, a);
    if (st) return st;
    a.bind_patch(p.g, steps);
    dim3 grid, block;
    unsigned lds;
    patch_dims(c, p, grid, block, lds);
    HIPCHK(hipLaunchKernel(patch_kernel_of(c, scheme), grid, block, a.args, lds,
                           c->stream));
    return LBFV_OK;
}

int launch_one(lbfv_ctx *c, int scheme, int parity, const double ext[4], int tb = 1) {
    StepShape sh = march_shape(c, scheme, tb);
    StepArgs a;
    int st = launch_args(c, scheme, parity, ext, sh, a);
    if (st) return st;
    dim3 grid, block;
    launch_dims(c, tb, sh, grid, block);
    HIPCHK(hipLaunchKernel(launch_fn(c, scheme, tb), grid, block, a.args, 0, c->stream));
    return LBFV_OK;
}

// a graph of gsteps launches of tb steps each, in the patch form or as marches
int build_graph(lbfv_ctx *c, int scheme, int parity0, const double ext[4], int tb, bool patch) {
    HostCase &h = c->hc;
    const StepShape sh = patch ? step_shape(h, 1, 1) : march_shape(c, scheme, tb);
    hipGraph_t g;
    HIPCHK(hipGraphCreate(&g, 0));
    hipGraphNode_t prev = nullptr;
    for (int s = 0; s < c->gsteps; ++s) {
        StepArgs a;
        int st = launch_args(c, scheme, (parity0 + s) & 1, ext, sh, a);
        if (st) {
            (void)hipGraphDestroy(g);
            return st;
        }
        hipKernelNodeParams kp;
        memset(&kp, 0, sizeof(kp));
        if (patch) {
            const PatchPlan &p = patch_plan(c, scheme);
            a.bind_patch(p.g, tb);
            kp.func = patch_kernel_of(c, scheme);
            patch_dims(c, p, kp.gridDim, kp.blockDim, kp.sharedMemBytes);
        } else {
            kp.func = launch_fn(c, scheme, tb);
            launch_dims(c, tb, sh, kp.gridDim, kp.blockDim);
        }
        kp.kernelParams = a.args;
        kp.extra = nullptr;
        hipGraphNode_t node;
        hipError_t e = hipGraphAddKernelNode(&node, g, prev ? &prev : nullptr, prev ? 1 : 0, &kp);
        if (e != hipSuccess) {
            (void)hipGraphDestroy(g);
            return c->fail(LBFV_EHIP, std::string("hipGraphAddKernelNode: ") + hipGetErrorString(e));
        }
        prev = node;
    }
    hipError_t e = hipGraphInstantiate(&c->gexec[patch ? 16 + scheme : scheme + 4 * (tb - 1)][parity0], g, nullptr,
                                       nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) return c->fail(LBFV_EHIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(e));
    return LBFV_OK;
}

int ensure_reduction(lbfv_ctx *c) {
    if (c->d_partial) return LBFV_OK;
    c->red_blocks = RED_GRID;
    HIPCHK(hipMalloc((void **)&c->d_partial, sizeof(double) * RED_N * c->red_blocks));
    HIPCHK(hipMalloc((void **)&c->d_out, sizeof(double) * RED_N));
    HIPCHK(hipHostMalloc((void **)&c->h_out, sizeof(double) * RED_N, hipHostMallocDefault));
    HIPCHK(hipEventCreateWithFlags(&c->check_event, hipEventDisableTiming));
    return LBFV_OK;
}

template <typename T, typename S>
void launch_reduce_t(lbfv_ctx *c, const double ext[4], int mode) {
    HostCase &h = c->hc;
    double e[4] = {ext[0], ext[1], ext[2], ext[3]};
    StepParams<T> P = make_params<T>(h, e);
    hipLaunchKernelGGL((reduce_kernel<T, S>), dim3(c->red_blocks), dim3(RED_BLOCK), 0, c->stream, P, h.cur, h.d_dx,
                       h.d_dy, c->d_uprev, mode, h.ref(), h.c, c->d_partial);
    hipLaunchKernelGGL(reduce_final_kernel, dim3(1), dim3(RED_BLOCK), 0, c->stream, c->d_partial, c->red_blocks,
                       c->d_out, 0);
}

int launch_reduce(lbfv_ctx *c, int mode) {
    int st = ensure_reduction(c);
    if (st) return st;
    double ext[4];
    current_ext(c->hc, ext);
    switch (c->hc.variant) {
    case V_F64: launch_reduce_t<double, double>(c, ext, mode); break;
    case V_F32: launch_reduce_t<float, float>(c, ext, mode); break;
    case V_BF16: launch_reduce_t<float, __bf16>(c, ext, mode); break;
    default: launch_reduce_t<float, _Float16>(c, ext, mode); break;
    }
    HIPCHK(hipGetLastError());
    HIPCHK(hipMemcpyAsync(c->h_out, c->d_out, sizeof(double) * RED_N, hipMemcpyDeviceToHost, c->stream));
    return LBFV_OK;
}

// Examine a finished asynchronous check (wait for it when `wait`).
int poll_check(lbfv_ctx *c, bool wait) {
    if (!c->check_pending) return LBFV_OK;
    if (wait) {
        HIPCHK(hipEventSynchronize(c->check_event));
    } else {
        hipError_t q = hipEventQuery(c->check_event);
        if (q == hipErrorNotReady) return LBFV_OK;
        if (q != hipSuccess) return c->fail(LBFV_EHIP, std::string("hipEventQuery: ") + hipGetErrorString(q));
    }
    c->check_pending = false;
    if (c->h_out[5] > 0) c->unstable = true;
    return LBFV_OK;
}

// the check of the stepping loop: the rest-direction plane only (check_rest_kernel)
int launch_check(lbfv_ctx *c) {
    int st = ensure_reduction(c);
    if (st) return st;
    const HostCase &h = c->hc;
    const dim3 grid(c->red_blocks), block(RED_BLOCK);
    switch (h.variant) {
    case V_F64:
        hipLaunchKernelGGL(check_rest_kernel<double>, grid, block, 0, c->stream, (const double *)h.buf[h.cur],
                           h.nx, h.ny, h.pitch, h.strip, c->d_partial);
        break;
    case V_F32:
        hipLaunchKernelGGL(check_rest_kernel<float>, grid, block, 0, c->stream, (const float *)h.buf[h.cur], h.nx,
                           h.ny, h.pitch, h.strip, c->d_partial);
        break;
    case V_BF16:
        hipLaunchKernelGGL(check_rest_kernel<__bf16>, grid, block, 0, c->stream, (const __bf16 *)h.buf[h.cur],
                           h.nx, h.ny, h.pitch, h.strip, c->d_partial);
        break;
    default:
        hipLaunchKernelGGL(check_rest_kernel<_Float16>, grid, block, 0, c->stream,
                           (const _Float16 *)h.buf[h.cur], h.nx, h.ny, h.pitch, h.strip, c->d_partial);
        break;
    }
    hipLaunchKernelGGL(reduce_final_kernel, dim3(1), dim3(RED_BLOCK), 0, c->stream, c->d_partial, c->red_blocks,
                       c->d_out, 0);
    HIPCHK(hipGetLastError());
    HIPCHK(hipMemcpyAsync(c->h_out, c->d_out, sizeof(double) * RED_N, hipMemcpyDeviceToHost, c->stream));
    return LBFV_OK;
}

int start_check(lbfv_ctx *c) {
    int st = poll_check(c, true);
    if (st) return st;
    st = launch_check(c);
    if (st) return st;
    HIPCHK(hipEventRecord(c->check_event, c->stream));
    c->check_pending = true;
    c->steps_at_check = c->steps;
    return LBFV_OK;
}

// Copy the state in buf[from] into buf[from ^ 1] in the layout of strip width w (the
// case's own strip and pitch still describe the source).
hipError_t relayout(const HostCase &h, int from, int w, hipStream_t stream) {
    const int64_t n = (int64_t)h.nx * h.ny;
    const int blocks = (int)std::min<int64_t>((n + 255) / 256, 8192);
    const int64_t pitch_d = padded_pitch(h.nx, w);
    const void *src = h.buf[from];
    void *dst = h.buf[from ^ 1];
    if (h.esize == 8)
        hipLaunchKernelGGL(relayout_kernel<uint64_t>, dim3(blocks), dim3(256), 0, stream, (const uint64_t *)src,
                           (uint64_t *)dst, h.nx, h.ny, h.pitch, h.strip, pitch_d, w);
    else if (h.esize == 4)
        hipLaunchKernelGGL(relayout_kernel<uint32_t>, dim3(blocks), dim3(256), 0, stream, (const uint32_t *)src,
                           (uint32_t *)dst, h.nx, h.ny, h.pitch, h.strip, pitch_d, w);
    else
        hipLaunchKernelGGL(relayout_kernel<uint16_t>, dim3(blocks), dim3(256), 0, stream, (const uint16_t *)src,
                           (uint16_t *)dst, h.nx, h.ny, h.pitch, h.strip, pitch_d, w);
    return hipGetLastError();
}

// a symmetry side (or the symmetry part of a side ending in a wall segment) needs the
// reference velocity to have no normal component there: F must be mirror-symmetric
const char *reference_conflict(const HostCase &h) {
    for (int s = 0; s < 4; ++s) {
        if (h.bc[s] != BC_SYMMETRY) continue;
        if (h.u0[s < 2 ? 0 : 1] != 0.0) return "the reference velocity has a component normal to a symmetry side";
    }
    return nullptr;
}

// Move the current state to the strip layout of w output columns (into the other buffer).
int set_layout(lbfv_ctx *c, int w) {
    HostCase &h = c->hc;
    if (w == h.strip) return LBFV_OK;
    if (c->has_state) {
        int st = poll_check(c, true);
        if (st) return st;
        HIPCHK(relayout(h, h.cur, w, c->stream));
        h.cur ^= 1;
    }
    h.set_strip(w);
    drop_graphs(c);
    memset(c->rows_of, 0, sizeof(c->rows_of));
    return LBFV_OK;
}

// How a call of n steps advances the context.  per: most steps of a launch.  exact: the call behaves
// as one-step launches do, since no shape was asked for: checks fall due at their step, and the
// state ends in the buffer that n launches would leave it in (a program may replay captured work
// that names that buffer).
struct Advance {
    bool patch = false, exact = false;
    bool single_marches = false;   // patches, but marches for the launches of one step
    int per = 1;
};
// The steps per launch of marches where no shape was set: a chain of four waves on a doubly
// periodic mesh, a pair of waves with sides.
int unasked_time_block(const HostCase &h) { return !has_boundary(h) && std::min(h.nx, h.ny) >= 8 ? 4 : 2; }
// Where no shape was set, meshes up to this size take patches in calls of any length, larger ones
// in long calls the marches above.  us a step, patches and marches: periodic, DUGKS FP64 384^2 5.6
// and 6.4, 448^2 8.4 and 7.1; FP32 512^2 5.6 and 7.2, 640^2 10.7 and 8.6; BKG crosses where DUGKS does
// to within a patch more or less, FP64 420^2 5.0 and 5.4, 448^2 5.6 and 5.6, 512^2 7.2 and 6.6, FP32
// 576^2 4.9 and 6.2, 608^2 7.0 and 6.3.  With sides the pairs
// gain more on DUGKS than on BKG: cavity FP64 DUGKS 384^2 6.8 and 7.6, 416^2 8.0 and 7.8, 512^2
// 12.9 and 9.8, BKG 448^2 6.7 and 7.2, 512^2 8.1 and 8.3; FP32 DUGKS 576^2 8.4 and 9.1, 608^2 9.5
// and 9.0, BKG 672^2 7.8 and 8.8, 736^2 9.1 and 9.1.
int64_t patch_cells(const HostCase &h, int scheme) {
    const bool f64 = is_f64(h.variant);
    if (has_boundary(h) && scheme == SCHEME_BKG) return f64 ? 1 << 18 : 1 << 19;
    return f64 ? 170000 : (has_boundary(h) ? 360000 : 350000);
}
constexpr int LONG_CALL = 16;   // steps from which moving the state to another layout pays
// One-step launches in a row after which moving it back to 62 columns pays: a launch takes 5 to 10 %
// longer in 56 or 60 on large meshes, and the move about as long as a launch.
constexpr int SINGLES_BACK = 8;
int plan_advance(lbfv_ctx *c, int scheme, int n, Advance &a) {
    HostCase &h = c->hc;
    const int64_t cells = (int64_t)h.nx * h.ny;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &capture) != hipSuccess) (void)hipGetLastError();
    if (!one_step_only(h)) a.per = h.tblock;
    const bool capturing = capture != hipStreamCaptureStatusNone;
    if (capturing) c->pinned = true;
    if (c->form == FORM_MARCH) {
        // (a shape that was set after a call had moved the state to another layout; one-step
        // marches run in every layout)
        return c->pinned ? (int)LBFV_OK : set_layout(c, SLOTS - 2 * h.tblock);
    }
    // The autotuner may pick launches of several steps in any form: their calls take the fewest
    // launches, as those of marches do, unless a program holds captured work (calls of two steps of a
    // tuned 256^2 FP64 BKG vortex: 14.1 us in two launches, 10.0 in one of a march).
    a.exact = c->form == FORM_AUTO || c->pinned;
    // a stream under capture gets one-step launches
    if (capturing) return LBFV_OK;
    // 16-bit storage is rounded after every step unless several per launch were asked for
    const bool wide = h.variant == V_F64 || h.variant == V_F32;
    if (c->form == FORM_AUTO && wide && cells > patch_cells(h, scheme) && !one_step_only(h)) {
        const int tb = unasked_time_block(h), strip = SLOTS - 2 * tb;
        // calls, or intervals between checks, so short that their parity leaves single steps only
        // (2 of a chain's, 3 of a pair's)
        const bool singles = (c->check_every > 0 ? std::min(n, c->check_every) : n) <= (tb == 2 ? 3 : 2);
        if (!singles && (h.strip == strip || (n >= LONG_CALL && !c->pinned))) {
            a.per = tb;
            c->singles = 0;
            return set_layout(c, strip);
        }
        if (!singles) c->singles = 0;
        else if (h.strip != STRIP1 && !c->pinned && (c->singles += n) > SINGLES_BACK) {
            int st = set_layout(c, STRIP1);
            if (st) return st;
        }
    }
    // (short calls on larger meshes: patches too, but for FP64 with sides, whose few resident
    // waves gain nothing there: 1024^2 cavity, three steps of DUGKS, 70 us a step against 68)
    const int64_t most = has_boundary(h) && h.variant == V_F64 ? 1 << 18 : PATCH_CELLS;
    if (c->form == FORM_PATCH || cells <= most) {
        const PatchPlan &p = patch_plan(c, scheme);
        a.patch = p.waves > 0;
        if (a.patch) a.per = p.g.halo;
        a.single_marches = a.patch && cells > patch_single_cells(is_f64(h.variant), scheme);
    }
    return LBFV_OK;
}
// lbfv_set_time_block, the form of the launches left as it is
int set_time_block(lbfv_ctx *c, int32_t steps) {
    HostCase &h = c->hc;
    if (steps < 1 || steps > 4) return c->fail(LBFV_EINVAL, "lbfv_set_time_block: steps must be 1 to 4");
    if (steps >= 2 && !h.sides_set())
        return c->fail(LBFV_EINVAL, "lbfv_set_time_block: set all four sides first");
    if (steps >= 3 && has_boundary(h))
        return c->fail(LBFV_EINVAL, "lbfv_set_time_block: 3 or 4 steps per launch need a doubly periodic mesh");
    if (steps >= 3 && (h.nx < 2 * steps || h.ny < 2 * steps))
        return c->fail(LBFV_EINVAL, "lbfv_set_time_block: 3 or 4 steps per launch need at least 2 x steps cells per side");
    int st = set_layout(c, SLOTS - 2 * steps);   // 62, 60, 58 or 56 output columns per strip
    if (st) return st;
    h.tblock = steps;
    return LBFV_OK;
}

// A march control was set: marches from here on (the next call moves the state to their layout).
// Graphs built without a shape may hold other kernels and row heights for the same time block.
int take_marches(lbfv_ctx *c) {
    c->form = FORM_MARCH;
    drop_graphs(c);
    return LBFV_OK;
}

int do_steps(lbfv_ctx *c, int scheme, int32_t n) {
    if (!c) return LBFV_EINVAL;
    if (n < 0) return c->fail(LBFV_EINVAL, "nsteps must be >= 0");
    HostCase &h = c->hc;
    if (!h.sides_set()) return c->fail(LBFV_ESTATE, "all four sides must be set before stepping");
    if (const char *why = reference_conflict(h)) return c->fail(LBFV_ESTATE, why);
    if (!c->has_state) return c->fail(LBFV_ESTATE, "no initial state (init_equilibrium or set_f first)");
    int st = poll_check(c, false);
    if (st) return st;
    if (c->unstable) return c->fail(LBFV_EUNSTABLE, "a non-finite value was found at a check");
    double ext[4];
    st = ensure_metrics(c, ext);
    if (st) return st;
    if (h.tblock >= 3 && has_boundary(h)) {
        // a side stopped being periodic: the chains of waves have no ghost cells, so the
        // mesh continues with two steps per launch
        if ((st = set_time_block(c, 2))) return st;
    }
    if (n == 0) return LBFV_OK;   // (nor does it move the state to another layout)
    current_ext(h, ext);
    Advance adv;
    if ((st = plan_advance(c, scheme, n, adv))) return st;
    const bool patch = adv.patch;
    const int per = adv.per;
    auto launch = [&](int steps) {
        const bool as_patch = patch && !(steps == 1 && adv.single_marches);
        int ls = as_patch ? launch_patch(c, scheme, h.cur, ext, steps) : launch_one(c, scheme, h.cur, ext, steps);
        if (!ls) h.cur ^= 1;
        return ls;
    };
    while (n > 0) {
        int seg = n;
        if (c->check_every > 0) {
            // the check comes at the first launch boundary at or after check_every steps, so
            // that a check never splits a launch of `per` steps that was asked for
            int64_t to_check = std::max<int64_t>(c->check_every - (c->steps - c->steps_at_check), 1);
            if (!adv.exact) to_check = (to_check + per - 1) / per * per;
            seg = (int)std::min<int64_t>(seg, to_check);
        }
        int left = seg;
        while (left >= per * c->gsteps) {
            hipGraphExec_t &g = c->gexec[patch ? 16 + scheme : scheme + 4 * (per - 1)][h.cur];
            if (!g) {
                st = build_graph(c, scheme, h.cur, ext, per, patch);
                if (st) return st;
            }
            HIPCHK(hipGraphLaunch(g, c->stream));
            h.cur ^= (c->gsteps & 1);
            left -= per * c->gsteps;
        }
        // the steps left over, in the same strip layout (every narrower march fits a wider halo's
        // strip)
        Cut cut(left, per, adv.exact, patch && adv.single_marches);
        while (const int k = cut.next())
            if ((st = launch(k))) return st;
        c->steps += seg;
        n -= seg;
        if (c->check_every > 0 && c->steps - c->steps_at_check >= c->check_every) {
            st = start_check(c);
            if (st) return st;
        }
    }
    return LBFV_OK;
}

// ------------------------------------------------------------------ fields to and from the host
enum Field { F_INIT_EQ, F_INIT_CE, F_SET_F, F_GET_F, F_MOMENTS };

template <typename T, typename S>
void launch_field(const HostCase &h, const StepParams<T> &P, int parity, Field which, CellRange C, double *buf,
                  hipStream_t stream) {
    const dim3 grid((unsigned)std::min<int64_t>((C.n + 255) / 256, 8192)), block(256);
    const RefState R = h.ref();
    switch (which) {
    case F_INIT_EQ: hipLaunchKernelGGL((init_eq_kernel<T, S>), grid, block, 0, stream, P, parity, C, buf, 1.0 / h.c, R); break;
    case F_INIT_CE: hipLaunchKernelGGL((init_ce_kernel<T, S>), grid, block, 0, stream, P, parity, C, buf, h.c, h.tau, h.dt, R); break;
    case F_SET_F: hipLaunchKernelGGL((set_f_kernel<T, S>), grid, block, 0, stream, P, parity, C, buf, R); break;
    case F_GET_F: hipLaunchKernelGGL((get_f_kernel<T, S>), grid, block, 0, stream, P, parity, C, buf, R); break;
    default: hipLaunchKernelGGL((moments_kernel<T, S>), grid, block, 0, stream, P, parity, C, buf, R, h.c); break;
    }
}

// Move fields between the caller's arrays (one value per cell each) and the state in
// buf[parity]; the stream is synchronised.
hipError_t move_fields(const HostCase &h, int parity, Transfer &t, hipStream_t stream, Field which,
                       const FieldArrays &arrays) {
    double ext[4];
    current_ext(h, ext);
    StepParams<double> pd;
    StepParams<float> pf;
    if (is_f64(h.variant)) pd = make_params<double>(h, ext);
    else pf = make_params<float>(h, ext);
    return t.run(which < F_GET_F, (int64_t)h.nx * h.ny, arrays, stream, [&](CellRange C, double *buf) {
        switch (h.variant) {
        case V_F64: launch_field<double, double>(h, pd, parity, which, C, buf, stream); break;
        case V_F32: launch_field<float, float>(h, pf, parity, which, C, buf, stream); break;
        case V_BF16: launch_field<float, __bf16>(h, pf, parity, which, C, buf, stream); break;
        default: launch_field<float, _Float16>(h, pf, parity, which, C, buf, stream); break;
        }
    });
}
// single arrays `one`, then arrays `three` of three components each
FieldArrays field_arrays(const HostCase &h, std::initializer_list<const double *> one,
                         std::initializer_list<const double *> three = {}) {
    const int64_t n = (int64_t)h.nx * h.ny;
    FieldArrays a;
    for (const double *f : one) a.add(f, 1, n);
    for (const double *f : three) a.add(f, 3, n);
    return a;
}
FieldArrays state_arrays(const HostCase &h, const double *f) {
    FieldArrays a;
    a.add(f, 9, (int64_t)h.nx * h.ny);
    return a;
}
template <typename Owner>
int moved(Owner *o, hipError_t e, const char *what) {
    if (e == hipSuccess) return LBFV_OK;
    if (e == hipErrorOutOfMemory) return o->fail(LBFV_ENOMEM, std::string(what) + ": cannot allocate the transfer buffer");
    return o->fail(LBFV_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

template <typename T, typename S>
void reref_t(lbfv_ctx *c, const RefState &from, const RefState &to) {
    HostCase &h = c->hc;
    double ext[4] = {0, 0, 0, 0};
    StepParams<T> P = make_params<T>(h, ext);
    const int64_t n = (int64_t)h.nx * h.ny;
    const int blocks = (int)std::min<int64_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL((reref_kernel<T, S>), dim3(blocks), dim3(256), 0, c->stream, P, h.cur, from, to);
}

// a new state given by the caller's arrays
int new_state(lbfv_ctx *c, Field which, const FieldArrays &arrays, const char *what) {
    int st = ensure_buffers(c);
    if (!st) st = moved(c, move_fields(c->hc, c->hc.cur, c->transfer, c->stream, which, arrays), what);
    if (st) return st;
    c->has_state = true;
    c->unstable = false;
    c->uprev_valid = false;
    return LBFV_OK;
}

}  // namespace

// ------------------------------------------------------------------ allocation-free totals
// Scratch of lbfv_totals_device: the per-block partial sums of the check reduction (the
// grid and kernels of lbfv_totals, so both give the same bits).  Its need is fixed
// (RED_GRID blocks x RED_N sums) whatever the mesh size.  Each GPU holds its own copy
// until the process ends; calls that overlap on one GPU race on it.  Host code never
// passes this name to a kernel: it takes the device address found by
// hipGetSymbolAddress, per device.
constexpr int SCRATCH_DOUBLES = RED_GRID * RED_N;   // 48 KiB
static __device__ __align__(256) double scratch[SCRATCH_DOUBLES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch_ptr[kMaxDevices] = {};

// the address of `scratch` on the current device, looked up once per device
int scratch_address(lbfv_ctx *c, int dev, double **p) {
    if (dev < 0 || dev >= kMaxDevices) return c->fail(LBFV_EUNSUPPORTED, "lbfv_totals_device: device index too large");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return c->fail(LBFV_EHIP, std::string("lbfv_totals_device: hipGetSymbolAddress(scratch): ") +
                                          hipGetErrorString(e));
        }
        g_scratch_ptr[dev] = (double *)ptr;
    }
    *p = g_scratch_ptr[dev];
    return LBFV_OK;
}

template <typename T, typename S>
void launch_reduce_into(lbfv_ctx *c, const double ext[4], double *partial, double *out) {
    HostCase &h = c->hc;
    double e[4] = {ext[0], ext[1], ext[2], ext[3]};
    StepParams<T> P = make_params<T>(h, e);
    hipLaunchKernelGGL((reduce_kernel<T, S>), dim3(RED_GRID), dim3(RED_BLOCK), 0, c->stream, P, h.cur, h.d_dx,
                       h.d_dy, (double *)nullptr, 0, h.ref(), h.c, partial);
    hipLaunchKernelGGL(reduce_final_kernel, dim3(1), dim3(RED_BLOCK), 0, c->stream, partial, RED_GRID, out, 1);
}
}  // namespace

extern "C" {

int lbfv_create(const lbfv_mesh *mesh, const lbfv_velset *vel, double tau, double dt, const lbfv_opts *opts,
                lbfv_ctx **ctx) {
    if (!ctx) {
        g_last_error = "NULL ctx pointer";
        return LBFV_EINVAL;
    }
    *ctx = nullptr;
    lbfv_opts o = {LBFV_FP64, LBFV_STORE_NATIVE, 1.0, 1000, nullptr};
    if (opts) o = *opts;
    std::string msg;
    int st = validate_case(mesh, vel, tau, dt, o.compute, o.storage, msg);
    if (st) {
        g_last_error = "lbfv_create: " + msg;
        return st;
    }
    if (!(o.rho0 > 0) && o.storage != LBFV_STORE_NATIVE) {
        g_last_error = "lbfv_create: rho0 must be > 0 for deviation storage";
        return LBFV_EINVAL;
    }
    if (o.check_every < 0) {
        g_last_error = "lbfv_create: check_every must be >= 0";
        return LBFV_EINVAL;
    }
    lbfv_ctx *c = new (std::nothrow) lbfv_ctx();
    if (!c) return LBFV_ENOMEM;
    init_host_case(c->hc, mesh, vel, tau, dt, o.compute, o.storage, o.rho0);
    c->check_every = o.check_every;
    c->stream = (hipStream_t)o.hip_stream;
    if (hipGetDevice(&c->device) != hipSuccess) {
        (void)hipGetLastError();
        c->device = -1;
    }
    *ctx = c;
    return LBFV_OK;
}

int lbfv_destroy(lbfv_ctx *c) {
    if (!c) return LBFV_EINVAL;
    (void)hipStreamSynchronize(c->stream);
    drop_graphs(c);
    free_case(c->hc);
    if (c->d_partial) (void)hipFree(c->d_partial);
    if (c->d_out) (void)hipFree(c->d_out);
    if (c->h_out) (void)hipHostFree(c->h_out);
    if (c->d_uprev) (void)hipFree(c->d_uprev);
    if (c->check_event) (void)hipEventDestroy(c->check_event);
    c->transfer.release();
    if (c->d_p2b) (void)hipFree(c->d_p2b);
    if (c->h_p2b) (void)hipHostFree(c->h_p2b);
    for (auto e : c->p2b_event)
        if (e) (void)hipEventDestroy(e);
    delete c;
    return LBFV_OK;
}

int lbfv_set_periodic(lbfv_ctx *c, int axis) {
    if (!c) return LBFV_EINVAL;
    if (axis != LBFV_X && axis != LBFV_Y) return c->fail(LBFV_EINVAL, "axis must be LBFV_X or LBFV_Y");
    const int s0 = axis == LBFV_X ? SIDE_W : SIDE_S;
    set_side(c->hc, s0, BC_PERIODIC, 0, 0, 0);
    set_side(c->hc, s0 + 1, BC_PERIODIC, 0, 0, 0);
    return LBFV_OK;
}

int lbfv_set_wall(lbfv_ctx *c, int side, double uwx, double uwy) {
    if (!c) return LBFV_EINVAL;
    if (side < 0 || side > 3 || !std::isfinite(uwx) || !std::isfinite(uwy))
        return c->fail(LBFV_EINVAL, "lbfv_set_wall: bad side or velocity");
    return set_side(c->hc, side, BC_WALL, uwx, uwy, 0);
}

int lbfv_set_inflow_eq(lbfv_ctx *c, int side, double rho, double ux, double uy) {
    if (!c) return LBFV_EINVAL;
    if (side < 0 || side > 3 || !(rho > 0) || !std::isfinite(ux) || !std::isfinite(uy))
        return c->fail(LBFV_EINVAL, "lbfv_set_inflow_eq: bad side or state");
    return set_side(c->hc, side, BC_INFLOW, rho, ux, uy);
}

int lbfv_set_symmetry(lbfv_ctx *c, int side) {
    if (!c) return LBFV_EINVAL;
    if (side < 0 || side > 3) return c->fail(LBFV_EINVAL, "lbfv_set_symmetry: bad side");
    return set_side(c->hc, side, BC_SYMMETRY, 0, 0, 0);
}

int lbfv_set_wall_from(lbfv_ctx *c, int side, int32_t first_cell, double uwx, double uwy) {
    if (!c) return LBFV_EINVAL;
    HostCase &h = c->hc;
    if (side != LBFV_SOUTH && side != LBFV_NORTH)
        return c->fail(LBFV_EINVAL, "lbfv_set_wall_from: only the south and north sides take a wall segment");
    if (first_cell < 0 || first_cell >= h.nx || !std::isfinite(uwx) || !std::isfinite(uwy))
        return c->fail(LBFV_EINVAL, "lbfv_set_wall_from: bad first cell or velocity");
    if (h.bc[side] < 0 || h.bc[side] == BC_PERIODIC)
        return c->fail(LBFV_EINVAL, "lbfv_set_wall_from: set a non-periodic kind on the side first");
    h.wfrom[side] = first_cell;
    h.wsv[side][0] = uwx;
    h.wsv[side][1] = uwy;
    h.metrics_dirty = true;
    return LBFV_OK;
}

int lbfv_set_outflow_extrap(lbfv_ctx *c, int side, int order) {
    if (!c) return LBFV_EINVAL;
    if (side < 0 || side > 3 || (order != 0 && order != 1))
        return c->fail(LBFV_EINVAL, "lbfv_set_outflow_extrap: bad side or order");
    return set_side(c->hc, side, BC_OUTFLOW, (double)order, 0, 0);
}

int lbfv_required_bytes(const lbfv_ctx *c, size_t *bytes) {
    if (!c || !bytes) return LBFV_EINVAL;
    *bytes = c->hc.buffer_bytes();
    return LBFV_OK;
}

int lbfv_bind_buffers(lbfv_ctx *c, void *a, void *b, size_t bytes) {
    if (!c) return LBFV_EINVAL;
    if (!a || !b || a == b) return c->fail(LBFV_EINVAL, "lbfv_bind_buffers: two distinct buffers needed");
    if (bytes < c->hc.buffer_bytes()) return c->fail(LBFV_EINVAL, "lbfv_bind_buffers: buffers too small");
    HIPCHK(hipStreamSynchronize(c->stream));
    HostCase &h = c->hc;
    free_buffers(h);
    h.buf[0] = a;
    h.buf[1] = b;
    h.own = false;
    h.cur = 0;
    // the layout of the time block, for good: the program may save and restore what the buffers hold
    h.set_strip(SLOTS - 2 * h.tblock);
    c->pinned = true;
    c->has_state = false;
    drop_graphs(c);
    HIPCHK(hipMemsetAsync(a, 0, h.buffer_bytes(), c->stream));
    HIPCHK(hipMemsetAsync(b, 0, h.buffer_bytes(), c->stream));
    return LBFV_OK;
}

int lbfv_init_equilibrium(lbfv_ctx *c, const double *rho, const double *ux, const double *uy) {
    if (!c) return LBFV_EINVAL;
    if (!rho || !ux || !uy) return c->fail(LBFV_EINVAL, "lbfv_init_equilibrium: NULL field");
    return new_state(c, F_INIT_EQ, field_arrays(c->hc, {rho, ux, uy}), "init_equilibrium");
}

int lbfv_init_chapman_enskog(lbfv_ctx *c, const double *rho, const double *ux, const double *uy,
                             const double *drho, const double *dux, const double *duy) {
    if (!c) return LBFV_EINVAL;
    if (!rho || !ux || !uy || !drho || !dux || !duy)
        return c->fail(LBFV_EINVAL, "lbfv_init_chapman_enskog: NULL field");
    return new_state(c, F_INIT_CE, field_arrays(c->hc, {rho, ux, uy}, {drho, dux, duy}), "init_chapman_enskog");
}

int lbfv_set_f(lbfv_ctx *c, const double *f) {
    if (!c) return LBFV_EINVAL;
    if (!f) return c->fail(LBFV_EINVAL, "lbfv_set_f: NULL array");
    return new_state(c, F_SET_F, state_arrays(c->hc, f), "set_f");
}

int lbfv_get_f(lbfv_ctx *c, double *f) {
    if (!c) return LBFV_EINVAL;
    if (!f) return c->fail(LBFV_EINVAL, "lbfv_get_f: NULL array");
    if (!c->has_state) return c->fail(LBFV_ESTATE, "no state");
    return moved(c, move_fields(c->hc, c->hc.cur, c->transfer, c->stream, F_GET_F, state_arrays(c->hc, f)), "get_f");
}

int dugks_step(lbfv_ctx *c, int32_t n) { return do_steps(c, SCHEME_DUGKS, n); }
int bkg_step(lbfv_ctx *c, int32_t n) { return do_steps(c, SCHEME_BKG, n); }
int lbfv_step(lbfv_ctx *c, int scheme, int32_t n) {
    if (!c) return LBFV_EINVAL;
    if (scheme < LBFV_DUGKS || scheme > LBFV_UPWIND) return c->fail(LBFV_EINVAL, "unknown scheme");
    return do_steps(c, scheme, n);
}

int lbfv_moments(lbfv_ctx *c, double *rho, double *ux, double *uy) {
    if (!c) return LBFV_EINVAL;
    if (!rho || !ux || !uy) return c->fail(LBFV_EINVAL, "lbfv_moments: NULL output");
    if (!c->has_state) return c->fail(LBFV_ESTATE, "no state");
    const FieldArrays a = field_arrays(c->hc, {rho, ux, uy});
    return moved(c, move_fields(c->hc, c->hc.cur, c->transfer, c->stream, F_MOMENTS, a), "moments");
}

int lbfv_totals(lbfv_ctx *c, double out[3]) {
    if (!c) return LBFV_EINVAL;
    if (!out) return c->fail(LBFV_EINVAL, "lbfv_totals: NULL output");
    if (!c->has_state) return c->fail(LBFV_ESTATE, "no state");
    int st = poll_check(c, true);
    if (st) return st;
    double ext[4];
    st = ensure_metrics(c, ext);   // volumes come with the metric upload
    if (st) return st;
    st = launch_reduce(c, 0);
    if (st) return st;
    HIPCHK(hipStreamSynchronize(c->stream));
    out[0] = c->h_out[0];
    out[1] = c->h_out[1];
    out[2] = c->h_out[2];
    if (c->h_out[5] > 0) c->unstable = true;
    if (c->unstable) return c->fail(LBFV_EUNSTABLE, "a non-finite value was found");
    return LBFV_OK;
}

int lbfv_totals_device(lbfv_ctx *c, double *dev_out) {
    if (!c) return LBFV_EINVAL;
    if (!dev_out) return c->fail(LBFV_EINVAL, "lbfv_totals_device: NULL output");
    if (!c->has_state) return c->fail(LBFV_ESTATE, "no state");
    if (c->hc.metrics_dirty)
        return c->fail(LBFV_ESTATE, "lbfv_totals_device: the mesh metrics are not on the device yet (step the "
                                    "context or call lbfv_totals once; their upload allocates)");
    static_assert(RED_GRID * RED_N <= SCRATCH_DOUBLES, "scratch too small for the reduction grid");
    c->pinned = true;   // (it may be captured: its launches name the state's buffer and layout)
    int dev = -1;
    HIPCHK(hipGetDevice(&dev));
    if (dev != c->device) return c->fail(LBFV_EINVAL, "lbfv_totals_device: the context's device must be current");
    double *partial = nullptr;
    int st = scratch_address(c, dev, &partial);
    if (st) return st;
    double ext[4];
    current_ext(c->hc, ext);
    switch (c->hc.variant) {
    case V_F64: launch_reduce_into<double, double>(c, ext, partial, dev_out); break;
    case V_F32: launch_reduce_into<float, float>(c, ext, partial, dev_out); break;
    case V_BF16: launch_reduce_into<float, __bf16>(c, ext, partial, dev_out); break;
    default: launch_reduce_into<float, _Float16>(c, ext, partial, dev_out); break;
    }
    HIPCHK(hipGetLastError());
    return LBFV_OK;
}

int lbfv_residual(lbfv_ctx *c, double *r) {
    if (!c) return LBFV_EINVAL;
    if (!r) return c->fail(LBFV_EINVAL, "lbfv_residual: NULL output");
    if (!c->has_state) return c->fail(LBFV_ESTATE, "no state");
    double ext[4];
    int st = ensure_metrics(c, ext);
    if (st) return st;
    st = poll_check(c, true);
    if (st) return st;
    const int64_t n = (int64_t)c->hc.nx * c->hc.ny;
    if (!c->d_uprev) {
        if (hipMalloc((void **)&c->d_uprev, sizeof(double) * 2 * n) != hipSuccess) {
            (void)hipGetLastError();
            return c->fail(LBFV_ENOMEM, "cannot allocate the residual buffer");
        }
        c->uprev_valid = false;
    }
    st = launch_reduce(c, 1);
    if (st) return st;
    HIPCHK(hipStreamSynchronize(c->stream));
    if (c->h_out[5] > 0) {
        c->unstable = true;
        return c->fail(LBFV_EUNSTABLE, "a non-finite value was found");
    }
    *r = c->uprev_valid ? std::sqrt(c->h_out[3] / c->h_out[4]) : 1.0;
    c->uprev_valid = true;
    return LBFV_OK;
}

int lbfv_set_time_block(lbfv_ctx *c, int32_t steps) {
    if (!c) return LBFV_EINVAL;
    int st = set_time_block(c, steps);
    return st ? st : take_marches(c);
}

int lbfv_get_time_block(const lbfv_ctx *c, int32_t *steps) {
    if (!c || !steps) return LBFV_EINVAL;
    *steps = c->hc.tblock;
    return LBFV_OK;
}

int lbfv_set_reference_velocity(lbfv_ctx *c, double ux, double uy) {
    if (!c) return LBFV_EINVAL;
    HostCase &h = c->hc;
    if (!std::isfinite(ux) || !std::isfinite(uy))
        return c->fail(LBFV_EINVAL, "lbfv_set_reference_velocity: velocity must be finite");
    if (!(h.rho0 > 0))
        return c->fail(LBFV_EINVAL, "lbfv_set_reference_velocity: needs deviation storage (FP32 compute)");
    if (ux == h.u0[0] && uy == h.u0[1]) return LBFV_OK;
    const RefState from = h.ref();
    const double old[2] = {h.u0[0], h.u0[1]};
    h.u0[0] = ux;
    h.u0[1] = uy;
    if (c->has_state) {
        int st = poll_check(c, true);
        if (st) {
            h.u0[0] = old[0];
            h.u0[1] = old[1];
            return st;
        }
        const RefState to = h.ref();
        switch (h.variant) {
        case V_F32: reref_t<float, float>(c, from, to); break;
        case V_BF16: reref_t<float, __bf16>(c, from, to); break;
        default: reref_t<float, _Float16>(c, from, to); break;
        }
        HIPCHK(hipGetLastError());
    }
    drop_graphs(c);
    c->plan[0] = c->plan[1] = PatchPlan();   // (another form of the kernels)
    memset(c->rows_of, 0, sizeof(c->rows_of));
    return LBFV_OK;
}

int lbfv_get_reference_velocity(const lbfv_ctx *c, double *ux, double *uy) {
    if (!c || !ux || !uy) return LBFV_EINVAL;
    *ux = c->hc.u0[0];
    *uy = c->hc.u0[1];
    return LBFV_OK;
}

int lbfv_set_tile(lbfv_ctx *c, int32_t rows, int32_t wpb) {
    if (!c) return LBFV_EINVAL;
    if (rows < 0 || (wpb != 0 && wpb != 1 && wpb != 2 && wpb != 4))
        return c->fail(LBFV_EINVAL, "lbfv_set_tile: rows >= 1, waves per block 1, 2 or 4");
    if (rows > 0) c->rows = rows;
    if (wpb > 0) c->wpb = wpb;
    memset(c->rows_of, 0, sizeof(c->rows_of));
    return rows > 0 || wpb > 0 ? take_marches(c) : (int)LBFV_OK;
}

int lbfv_get_tile(const lbfv_ctx *c, int32_t *rows, int32_t *wpb) {
    if (!c || !rows || !wpb) return LBFV_EINVAL;
    const HostCase &h = c->hc;
    *rows = c->rows > 0 ? c->rows : default_rows(h, SCHEME_DUGKS, c->wpb, h.sides_set() ? h.tblock : 1, c->pairs);
    *wpb = c->wpb;
    return LBFV_OK;
}

int lbfv_set_wave_pairs(lbfv_ctx *c, int32_t on) {
    if (!c) return LBFV_EINVAL;
    if (on != 0 && on != 1) return c->fail(LBFV_EINVAL, "lbfv_set_wave_pairs: 0 or 1");
    c->pairs = on;
    return take_marches(c);
}

int lbfv_get_wave_pairs(const lbfv_ctx *c, int32_t *on) {
    if (!c || !on) return LBFV_EINVAL;
    *on = c->pairs;
    return LBFV_OK;
}

}  // extern "C"

// ====================================================================== autotuner
namespace {

std::string arch_name() {
    int dev = 0;
    hipDeviceProp_t p;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&p, dev) != hipSuccess) return "unknown";
    std::string a = p.gcnArchName;
    return a.substr(0, a.find(':'));
}

int size_class(int n) {
    int k = 0;
    while ((1 << (k + 1)) <= n) ++k;
    return k;
}

std::string tune_key(const HostCase &h, int scheme) {
    std::ostringstream s;
    static const char *names[4] = {"dugks", "bkg", "central", "upwind"};
    s << arch_name() << " " << names[scheme] << " v" << h.variant << (has_boundary(h) ? " b" : " p") << " x"
      << size_class(h.nx) << " y" << size_class(h.ny);
    return s.str();
}

// patch: halo, per_wave and max_waves of a plan of the patch form (halo 0: marches)
bool cache_lookup(const char *path, const std::string &key, int &rows, int &wpb, double &ms, int &tb, int &pairs,
                  std::array<int, 3> &patch) {
    if (!path) return false;
    std::ifstream in(path);
    std::string line;
    bool found = false;
    while (std::getline(in, line)) {
        if (line.compare(0, key.size(), key) == 0 && line.size() > key.size() && line[key.size()] == '|') {
            std::istringstream t(line.substr(key.size() + 1));
            int r, w, k = 1, pr = 0;
            double m;
            if (t >> r >> w >> m) {
                if (!(t >> k) || k < 1 || k > 4) k = 1;
                if (!(t >> pr) || (pr != 0 && pr != 1)) pr = 0;
                patch = {0, 0, 0};
                if (!(t >> patch[0] >> patch[1] >> patch[2]) || patch[0] < 1 || patch[0] > PATCH_HALO || patch[1] < 1 ||
                    patch[1] > 64 || patch[2] < 1 || patch[2] > PATCH_WAVES)
                    patch = {0, 0, 0};
                rows = r;
                wpb = w;
                ms = m;
                tb = k;
                pairs = pr;
                found = true;   // last entry wins
            }
        }
    }
    return found;
}

void cache_store(const char *path, const std::string &key, int rows, int wpb, double ms, int tb, int pairs,
                 const std::array<int, 3> &patch) {
    if (!path) return;
    std::ofstream out(path, std::ios::app);
    out << key << "|" << rows << " " << wpb << " " << ms << " " << tb << " " << pairs;
    if (patch[0]) out << " " << patch[0] << " " << patch[1] << " " << patch[2];
    out << "\n";
}

}  // namespace

extern "C" int lbfv_autotune(lbfv_ctx *c, int scheme, int32_t trial_steps, const char *cache_path,
                             double *best_ms) {
    if (!c) return LBFV_EINVAL;
    if (scheme < LBFV_DUGKS || scheme > LBFV_UPWIND) return c->fail(LBFV_EINVAL, "unknown scheme");
    if (trial_steps < 1) return c->fail(LBFV_EINVAL, "trial_steps must be >= 1");
    if (!c->has_state) return c->fail(LBFV_ESTATE, "autotune needs a state to step");
    if (!c->hc.sides_set()) return c->fail(LBFV_ESTATE, "all four sides must be set");
    const char *path = cache_path ? cache_path : getenv("LBFV_TUNE_CACHE");
    HostCase &h = c->hc;
    const std::string key = tune_key(h, scheme);
    int rows, wpb, tb, pairs;
    std::array<int, 3> patch;
    double ms;
    // (an entry of the same size class whose time block or patches this mesh cannot take is ignored)
    if (cache_lookup(path, key, rows, wpb, ms, tb, pairs, patch) &&
        (tb < 3 || (!has_boundary(h) && std::min(h.nx, h.ny) >= 2 * tb))) {
        PatchPlan plan;
        if (!patch[0] || plan_patch(h, patch[1], patch[2], patch[0], plan)) {
            double ext[4];
            int st = ensure_metrics(c, ext);   // (it drops the plans of other sides)
            if (!st) st = set_time_block(c, tb);
            if (st) return st;
            c->rows = std::min(rows, h.ny);
            c->wpb = wpb;
            c->pairs = pairs;
            c->form = patch[0] ? FORM_PATCH : FORM_MARCH;
            if (patch[0]) c->plan[scheme == SCHEME_BKG] = plan;
            drop_graphs(c);
            if (best_ms) *best_ms = ms;
            return LBFV_OK;
        }
    }
    // save the state; trials step it (and may move it between strip layouts)
    void *save = nullptr;
    if (hipMalloc(&save, h.buffer_bytes()) != hipSuccess) {
        (void)hipGetLastError();
        return c->fail(LBFV_ENOMEM, "autotune: cannot allocate the save buffer");
    }
    const int saved_cur = h.cur, saved_strip = h.strip, saved_tb = h.tblock;
    const int64_t saved_steps = c->steps, saved_at = c->steps_at_check;
    const int saved_check = c->check_every;
    HIPCHK(hipMemcpyAsync(save, h.buf[h.cur], h.buffer_bytes(), hipMemcpyDeviceToDevice, c->stream));
    hipEvent_t e0, e1;
    HIPCHK(hipEventCreate(&e0));
    HIPCHK(hipEventCreate(&e1));
    c->check_every = 0;
    int best_r = 0, best_w = 0, best_t = 1, best_p = 0;
    int one_r = 0, one_w = 0;                 // the fastest march of one step per launch
    double best = INFINITY, best_one = INFINITY;
    const int saved_pairs = c->pairs, saved_form = c->form;
    int st = LBFV_OK;
    // candidate shapes: (time block, pair of waves per item, rows, waves per block)
    std::vector<std::array<int, 4>> cands;
    for (int t : {1, 2}) {
        for (int w : {1, 2, 4}) {
            // (1 and 2 rows: more waves for small, latency-bound meshes)
            for (int r : {1, 2, 4, 8, 16, 32, 64, 128, 256})
                if (r <= h.ny || r == 1) cands.push_back({t, 0, std::min(r, h.ny), w});
            // balanced heights; the two-step kernel holds more registers (fewer resident
            // waves), so its heights of up to 8 rounds are tried
            void *fn = t == 1 ? step_fn_variant(h.variant, scheme, has_boundary(h), ref_terms(h))
                              : step2_fn_variant(h.variant, scheme, has_boundary(h), ref_terms(h));
            for (int r : balanced_rows(h, resident_waves(fn, w), t == 1 ? STRIP1 : STRIP2, t == 1 ? 4 : 8))
                cands.push_back({t, 0, r, w});
        }
    }
    // two steps per launch with a pair of waves per item (one workgroup each); the balanced
    // heights count resident pairs
    for (int r : {1, 2, 4, 8, 16, 32, 64, 128, 256})
        if (r <= h.ny || r == 1) cands.push_back({2, 1, std::min(r, h.ny), 1});
    for (int r : balanced_rows(h, resident_waves(step2p_fn_variant(h.variant, scheme, has_boundary(h), ref_terms(h)), 2) / 2,
                               STRIP2, 8))
        cands.push_back({2, 1, r, 1});
    // with x sides: whole rounds of the SIMDs, whose loads the shorter row blocks there even out
    if (const int cus = has_side_strips(h, (h.nx + STRIP2 - 1) / STRIP2) ? device_cus(c) : 0)
        for (int r : balanced_rows(h, 2 * cus, STRIP2, 8, true)) cands.push_back({2, 1, r, 1});
    // three and four steps per launch on doubly periodic meshes: a chain of waves per item
    // (one workgroup each); the balanced heights count resident chains
    if (!has_boundary(h))
        for (int t : {3, 4}) {
            if (std::min(h.nx, h.ny) < 2 * t) continue;
            for (int r : {1, 2, 4, 8, 16, 32, 64, 128, 256})
                if (r <= h.ny || r == 1) cands.push_back({t, 0, std::min(r, h.ny), 1});
            void *fn = stepc_fn_variant(h.variant, scheme, t, ref_terms(h));
            for (int r : balanced_rows(h, resident_waves(fn, t) / t, SLOTS - 2 * t, 8)) cands.push_back({t, 0, r, 1});
        }
    if (one_step_only(h))
        cands.erase(std::remove_if(cands.begin(), cands.end(), [](const std::array<int, 4> &k) { return k[0] > 1; }),
                    cands.end());
    std::sort(cands.begin(), cands.end());
    cands.erase(std::unique(cands.begin(), cands.end()), cands.end());
    // one trial of the shape set on the context, `steps` of them timed: ms per step
    auto trial = [&](int steps, double &per, int warm = 2) {
        drop_graphs(c);
        int ts = do_steps(c, scheme, warm);
        if (ts) return ts;
        hipError_t he = hipEventRecord(e0, c->stream);
        if (he == hipSuccess && (ts = do_steps(c, scheme, steps))) return ts;
        float t = 0;
        if (he == hipSuccess) he = hipEventRecord(e1, c->stream);
        if (he == hipSuccess) he = hipEventSynchronize(e1);
        if (he == hipSuccess) he = hipEventElapsedTime(&t, e0, e1);
        if (he != hipSuccess) return c->fail(LBFV_EHIP, std::string("autotune timing: ") + hipGetErrorString(he));
        per = t / steps;
        return (int)LBFV_OK;
    };
    c->form = FORM_MARCH;
    for (const auto &cand : cands) {
        if ((st = set_time_block(c, cand[0]))) break;
        c->pairs = cand[1];
        c->rows = cand[2];
        c->wpb = cand[3];
        double per;
        if ((st = trial(trial_steps, per))) break;
        if (per < best) {
            best = per;
            best_t = cand[0];
            best_p = cand[1];
            best_r = cand[2];
            best_w = cand[3];
        }
        if (cand[0] == 1 && per < best_one) {
            best_one = per;
            one_r = cand[2];
            one_w = cand[3];
        }
    }
    // the patch form on small meshes: the cost model's best plan at each halo width, unless the
    // model puts it far behind its best one
    PatchPlan best_plan;
    double best_patch = INFINITY;
    if (!st && (int64_t)h.nx * h.ny <= PATCH_CELLS && !(st = set_time_block(c, 1))) {
        const PatchDevice dev = patch_device(is_f64(h.variant), patch_kernel_of(c, scheme));
        const double limit = 1.4 * best_patch_plan(h, dev, scheme).cost;
        c->form = FORM_PATCH;
        for (int halo = 1; halo <= PATCH_HALO && !st; ++halo) {
            const PatchPlan p = best_patch_plan(h, dev, scheme, halo, halo);
            if (!p.waves || p.cost > limit) continue;
            c->plan[scheme == SCHEME_BKG] = p;
            double per;
            if ((st = trial(trial_length(halo, trial_steps), per))) break;
            if (per < best_patch) {
                best_patch = per;
                best_plan = p;
            }
        }
        // A trial's first launches weigh on both forms differently (700^2 FP32 DUGKS: patches 9.6 and
        // chains 10.0 us a step in trials, 9.5 and 9.0 in long calls): where the two come near, graph
        // replays decide.
        if (!st && best_plan.waves && std::max(best, best_patch) < 1.15 * std::min(best, best_patch)) {
            const int halo = best_plan.g.halo, rounds = 2 * c->gsteps;
            c->plan[scheme == SCHEME_BKG] = best_plan;
            st = trial(rounds * halo, best_patch, c->gsteps * halo);
            c->form = FORM_MARCH;
            c->pairs = best_p;
            c->rows = best_r;
            c->wpb = best_w;
            if (!st) st = set_time_block(c, best_t);
            if (!st) st = trial(rounds * best_t, best, c->gsteps * best_t);
        }
        if (best_patch < best) best = best_patch;
        else best_plan = PatchPlan();
    }
    if (best_plan.waves) {
        // the march controls then hold the fastest march of the same (one-step) layout
        best_t = 1;
        best_p = 0;
        best_r = one_r;
        best_w = one_w;
    }
    // restore the saved state in its own layout, then move it to the chosen one
    h.set_strip(saved_strip);
    h.tblock = saved_tb;
    h.cur = saved_cur;
    hipError_t re = hipMemcpyAsync(h.buf[h.cur], save, h.buffer_bytes(), hipMemcpyDeviceToDevice, c->stream);
    if (re == hipSuccess) re = hipStreamSynchronize(c->stream);
    (void)hipFree(save);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (re != hipSuccess && !st) st = c->fail(LBFV_EHIP, std::string("autotune restore: ") + hipGetErrorString(re));
    c->steps = saved_steps;
    c->steps_at_check = saved_at;
    c->check_every = saved_check;
    c->pairs = saved_pairs;
    c->form = saved_form;
    c->plan[scheme == SCHEME_BKG] = best_plan;   // (none: planned again on use)
    drop_graphs(c);
    if (st) return st;
    if ((st = set_time_block(c, best_t))) return st;
    c->rows = best_r;
    c->wpb = best_w;
    c->pairs = best_p;
    c->form = best_plan.waves ? FORM_PATCH : FORM_MARCH;
    drop_graphs(c);
    cache_store(path, key, best_r, best_w, best, best_t, best_p,
                {best_plan.waves ? best_plan.g.halo : 0, best_plan.per_wave, best_plan.max_waves});
    if (best_ms) *best_ms = best;
    return LBFV_OK;
}

// ====================================================================== batch
namespace {

template <typename T>
int batch_upload_params(lbfv_batch *b) {
    std::vector<StepParams<T>> ps;
    for (auto &h : b->cases) {
        double ext[4];
        current_ext(h, ext);
        ps.push_back(make_params<T>(h, ext));
    }
    if (!b->d_params && hipMalloc(&b->d_params, ps.size() * sizeof(StepParams<T>)) != hipSuccess) {
        (void)hipGetLastError();
        return b->fail(LBFV_ENOMEM, "batch: cannot allocate the case table");
    }
    if (hipMemcpy(b->d_params, ps.data(), ps.size() * sizeof(StepParams<T>), hipMemcpyHostToDevice) != hipSuccess)
        return b->fail(LBFV_EHIP, "batch: case table upload failed");
    return LBFV_OK;
}

void batch_drop_graphs(lbfv_batch *b) {
    for (auto &row : b->gexec)
        for (auto &g : row)
            if (g) {
                (void)hipGraphExecDestroy(g);
                g = nullptr;
            }
}

int batch_build_items(lbfv_batch *b) {
    std::vector<BatchItem> items;
    // largest cases first so that the grid-stride walk ends on small items
    std::vector<int> order(b->cases.size());
    for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
    std::stable_sort(order.begin(), order.end(), [&](int a, int c) {
        return (int64_t)b->cases[a].nx * b->cases[a].ny > (int64_t)b->cases[c].nx * b->cases[c].ny;
    });
    for (int ci : order) {
        const HostCase &h = b->cases[ci];
        const int rows = std::min(b->rows, h.ny);
        for (int j0 = 0; j0 < h.ny; j0 += rows)
            for (int x0 = 0; x0 < h.nx; x0 += h.strip) items.push_back({ci, x0, j0, std::min(h.ny, j0 + rows)});
    }
    if (b->d_items) (void)hipFree(b->d_items);
    b->d_items = nullptr;
    if (hipMalloc((void **)&b->d_items, items.size() * sizeof(BatchItem)) != hipSuccess) {
        (void)hipGetLastError();
        return b->fail(LBFV_ENOMEM, "batch: cannot allocate the work list");
    }
    if (hipMemcpy(b->d_items, items.data(), items.size() * sizeof(BatchItem), hipMemcpyHostToDevice) != hipSuccess)
        return b->fail(LBFV_EHIP, "batch: work list upload failed");
    b->nitems = (int)items.size();
    batch_drop_graphs(b);
    return LBFV_OK;
}

// ------------------------------------------------------------------ patches of a batch
// Patches of at most 4 or 8 waves with one halo width for every case: of each kind of mesh the
// fewest.  grids: one per case.  false if some case takes none.
bool plan_batch_patches(const lbfv_batch *b, int max_waves, int halo, std::vector<PatchGrid> &grids, int &waves,
                        int64_t &count) {
    std::map<std::array<int, 4>, PatchPlan> kinds;
    grids.clear();
    waves = 0;
    count = 0;
    for (const auto &h : b->cases) {
        PatchPlan &best = kinds[{h.nx, h.ny, h.periodic_x(), h.periodic_y()}];
        for (int per_wave = best.waves ? 7 : 1; per_wave <= 6; ++per_wave) {
            PatchPlan p;
            if (!plan_patch(h, per_wave, max_waves, halo, p)) continue;
            if (!best.waves || (int64_t)p.g.npx * p.g.npy < (int64_t)best.g.npx * best.g.npy) best = p;
        }
        if (!best.waves) return false;
        grids.push_back(best.g);
        waves = std::max(waves, best.waves);
        count += (int64_t)best.g.npx * best.g.npy;
    }
    return count < (1 << 24);
}
// (with the graphs whose launches name their tables)
void drop_patches(lbfv_batch *b, int scheme) {
    for (auto &g : b->gexec[2 + scheme])
        if (g) {
            (void)hipGraphExecDestroy(g);
            g = nullptr;
        }
    lbfv_batch::Patches &p = b->patches[scheme];
    if (p.d_grids) (void)hipFree(p.d_grids);
    if (p.d_items) (void)hipFree(p.d_items);
    p = lbfv_batch::Patches();
}
// Put the patches of a halo width (0: the cost model's choice of it) and workgroup size in place;
// without any that every case takes, waves stays 0.  So it does where there is no memory for
// their tables: the batch marches then, which needs none.
int make_patches_or_throw(lbfv_batch *b, int scheme, int halo, int max_waves) {
    lbfv_batch::Patches &out = b->patches[scheme];
    drop_patches(b, scheme);
    out.halo = std::max(halo, 1);
    const bool f64 = is_f64(b->variant);
    const PatchDevice dev = patch_device(f64, batch_patch_fn_variant(b->variant, scheme, b->bnd));
    std::vector<PatchGrid> grids, best;
    for (int hw = halo ? halo : 1; hw <= (halo ? halo : PATCH_HALO); ++hw)
        for (int mw : {4, 8}) {
            if (max_waves && mw != max_waves) continue;
            int waves;
            int64_t count;
            if (!plan_batch_patches(b, mw, hw, grids, waves, count)) continue;
            const double cost = patch_cost(f64, scheme == SCHEME_BKG, b->bnd, dev, count, waves, hw);
            if (out.waves && cost >= out.cost) continue;
            out.halo = hw;
            out.waves = waves;
            out.count = (int)count;
            out.cost = cost;
            best.swap(grids);
        }
    if (!out.waves) return LBFV_OK;
    std::vector<PatchItem> items;
    items.reserve(out.count);
    for (int c = 0; c < (int)best.size(); ++c)
        for (int py = 0; py < best[c].npy; ++py)
            for (int px = 0; px < best[c].npx; ++px) items.push_back({c, px, py});
    if (hipMalloc((void **)&out.d_grids, best.size() * sizeof(PatchGrid)) != hipSuccess ||
        hipMalloc((void **)&out.d_items, items.size() * sizeof(PatchItem)) != hipSuccess) {
        (void)hipGetLastError();
        drop_patches(b, scheme);
        out.halo = std::max(halo, 1);
        return LBFV_OK;
    }
    if (hipMemcpyAsync(out.d_grids, best.data(), best.size() * sizeof(PatchGrid), hipMemcpyHostToDevice, b->stream) != hipSuccess ||
        hipMemcpyAsync(out.d_items, items.data(), items.size() * sizeof(PatchItem), hipMemcpyHostToDevice, b->stream) != hipSuccess ||
        hipStreamSynchronize(b->stream) != hipSuccess) {
        drop_patches(b, scheme);
        return b->fail(LBFV_EHIP, "batch: patch list upload failed");
    }
    return LBFV_OK;
}
// The first steps of a batch come here: the thread may be capturing work on another stream, which
// an allocation would break off but for the relaxed mode.
int make_patches(lbfv_batch *b, int scheme, int halo, int max_waves) {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    int st = LBFV_OK;
    try {
        st = make_patches_or_throw(b, scheme, halo, max_waves);
    } catch (const std::bad_alloc &) {
        drop_patches(b, scheme);
        b->patches[scheme].halo = std::max(halo, 1);
    }
    if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
    return st;
}

// Whether the patch form advances the batch: asked for by the autotuner, or by the sizes of the
// meshes where no shape was set.  As for one case, a stream under capture gets marches.
int batch_use_patches(lbfv_batch *b, int scheme, bool &yes) {
    yes = false;
    if (b->form == FORM_MARCH) return LBFV_OK;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(b->stream, &capture) != hipSuccess) (void)hipGetLastError();
    else if (capture != hipStreamCaptureStatusNone) {
        b->captured = true;
        return LBFV_OK;
    }
    if (b->form == FORM_AUTO)
        for (const auto &h : b->cases)
            if ((int64_t)h.nx * h.ny > BATCH_PATCH_CELLS) return LBFV_OK;
    if (!b->patches[scheme].halo) {
        int st = make_patches(b, scheme, 0, 0);
        if (st) return st;
    }
    yes = b->patches[scheme].waves > 0;
    return LBFV_OK;
}

struct PatchArgs {
    const void *params;
    const PatchGrid *grids;
    const PatchItem *items;
    int parity, steps;
    void *args[5];
    PatchArgs(const lbfv_batch *b, int scheme, int parity_, int steps_)
        : params(b->d_params), grids(b->patches[scheme].d_grids), items(b->patches[scheme].d_items), parity(parity_),
          steps(steps_), args{&params, &grids, &items, &parity, &steps} {}
    PatchArgs(const PatchArgs &) = delete;
};
unsigned patch_lds_bytes(const lbfv_batch *b, int scheme) {
    return (unsigned)(PATCH_LDS * 64 * b->patches[scheme].waves * (is_f64(b->variant) ? 8 : 4));
}

struct BatchArgs {
    const void *params;
    const BatchItem *items;
    int nitems, parity;
    void *args[4];
    void bind() {
        args[0] = &params;
        args[1] = &items;
        args[2] = &nitems;
        args[3] = &parity;
    }
};

bool batch_paired(const lbfv_batch *b, bool two) { return two && b->pairs; }

// work items the batch kernel keeps resident on the device (from its occupancy): one per
// wave, or one per pair of waves
int batch_slots(lbfv_batch *b, int scheme, bool two) {
    const bool pr = batch_paired(b, two);
    int &slots = b->slots[pr ? 2 : (two ? 1 : 0)][scheme];
    if (slots <= 0) {
        slots = pr ? resident_waves(batch_fn_variant(b->variant, scheme, b->bnd, two, true), 2) / 2
                   : resident_waves(batch_fn_variant(b->variant, scheme, b->bnd, two), 4);
        if (slots <= 0) slots = 256 * 4;
    }
    return slots;
}

// Persistent grid: exactly the workgroups that fit on the device at once (4 waves, or one
// pair of waves), capped by the work list; or one item per wave (per pair), so that the
// hardware hands a freed slot the next workgroup (items of uneven cost then balance
// themselves).
int batch_grid(lbfv_batch *b, int scheme, bool two) {
    if (batch_paired(b, two)) {
        const int all = std::max(1, b->nitems);
        return b->wave_per_item ? all : std::min(all, batch_slots(b, scheme, two));
    }
    const int all = std::max(1, (b->nitems + 3) / 4);
    if (b->wave_per_item) return all;
    return std::min(all, batch_slots(b, scheme, two) / 4);
}
int batch_block(const lbfv_batch *b, bool two) { return batch_paired(b, two) ? 128 : 256; }

// Row-block heights in 2 ... 64 that a cost model ranks best for the batch: whole rounds
// of the resident waves times the rows each item marches (its rows plus the rows the
// stencil reads around them at each step level); returns up to `count` heights.
std::vector<int> batch_balanced_rows(const lbfv_batch *b, int slots, int count) {
    std::vector<std::pair<double, int>> cost;
    for (int r = 2; r <= 64; ++r) {
        int64_t n = 0;
        for (const auto &h : b->cases) n += (int64_t)((h.nx + h.strip - 1) / h.strip) * ((h.ny + r - 1) / r);
        const int64_t rounds = (n + slots - 1) / slots;
        cost.push_back({(double)rounds * (r + 2 * b->tblock), r});
    }
    std::stable_sort(cost.begin(), cost.end());
    std::vector<int> out;
    for (int i = 0; i < count && i < (int)cost.size(); ++i) out.push_back(cost[i].second);
    return out;
}

// one launch: one time step, or two when two is set (the cases then hold 60-column strips)
int batch_launch_one(lbfv_batch *b, int scheme, int parity, bool two = false) {
    BatchArgs a{b->d_params, b->d_items, b->nitems, parity};
    a.bind();
    hipError_t e = hipLaunchKernel(batch_fn_variant(b->variant, scheme, b->bnd, two, batch_paired(b, two)),
                                   dim3(batch_grid(b, scheme, two)), dim3(batch_block(b, two)), a.args, 0, b->stream);
    if (e != hipSuccess) return b->fail(LBFV_EHIP, std::string("batch launch: ") + hipGetErrorString(e));
    return LBFV_OK;
}

int batch_launch_patches(lbfv_batch *b, int scheme, int parity, int steps) {
    PatchArgs a(b, scheme, parity, steps);
    hipError_t e = hipLaunchKernel(batch_patch_fn_variant(b->variant, scheme, b->bnd), dim3(b->patches[scheme].count),
                                   dim3(64 * b->patches[scheme].waves), a.args, patch_lds_bytes(b, scheme), b->stream);
    if (e != hipSuccess) return b->fail(LBFV_EHIP, std::string("batch launch: ") + hipGetErrorString(e));
    return LBFV_OK;
}

// Launches of a graph.  In the patch form an even number, whatever length was set: the state then
// comes back to the buffer it was in, as after the even number of steps that one-step launches
// would have taken (a program may replay captured work that names that buffer).
int64_t graph_launches(const lbfv_batch *b, bool patch) {
    return patch ? (int64_t)b->gsteps + (b->gsteps & 1) : b->gsteps;
}

// a graph of launches of the current time block, or of the patch form
int batch_build_graph(lbfv_batch *b, int scheme, int parity0, bool patch) {
    const bool two = b->tblock == 2;
    hipGraph_t g;
    if (hipGraphCreate(&g, 0) != hipSuccess) return b->fail(LBFV_EHIP, "hipGraphCreate failed");
    hipGraphNode_t prev = nullptr;
    for (int64_t s = 0; s < graph_launches(b, patch); ++s) {
        BatchArgs a{b->d_params, b->d_items, b->nitems, (int)((parity0 + s) & 1)};
        a.bind();
        hipKernelNodeParams kp;
        memset(&kp, 0, sizeof(kp));
        PatchArgs pa(b, scheme, (int)((parity0 + s) & 1), b->patches[scheme].halo);
        if (patch) {
            kp.func = batch_patch_fn_variant(b->variant, scheme, b->bnd);
            kp.gridDim = dim3(b->patches[scheme].count);
            kp.blockDim = dim3(64 * b->patches[scheme].waves);
            kp.sharedMemBytes = patch_lds_bytes(b, scheme);
            kp.kernelParams = pa.args;
        } else {
            kp.func = batch_fn_variant(b->variant, scheme, b->bnd, two, batch_paired(b, two));
            kp.gridDim = dim3(batch_grid(b, scheme, two));
            kp.blockDim = dim3(batch_block(b, two));
            kp.kernelParams = a.args;
        }
        hipGraphNode_t node;
        hipError_t e = hipGraphAddKernelNode(&node, g, prev ? &prev : nullptr, prev ? 1 : 0, &kp);
        if (e != hipSuccess) {
            (void)hipGraphDestroy(g);
            return b->fail(LBFV_EHIP, std::string("hipGraphAddKernelNode: ") + hipGetErrorString(e));
        }
        prev = node;
    }
    hipError_t e = hipGraphInstantiate(&b->gexec[scheme + (patch ? 2 : 0)][parity0], g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) return b->fail(LBFV_EHIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(e));
    return LBFV_OK;
}

// lbfv_batch_set_time_block, the form of the launches left as it is
int batch_set_time_block(lbfv_batch *b, int32_t steps) {
    if (steps == b->tblock) return LBFV_OK;
    // launches in flight read the case table that is rewritten below
    hipError_t es = hipStreamSynchronize(b->stream);
    if (es != hipSuccess) return b->fail(LBFV_EHIP, std::string("batch: ") + hipGetErrorString(es));
    // every case moves its current state into the other buffer in the new strip layout
    const int w = steps == 2 ? STRIP2 : STRIP1;
    for (auto &h : b->cases) {
        hipError_t e = relayout(h, b->parity, w, b->stream);
        if (e != hipSuccess) return b->fail(LBFV_EHIP, std::string("batch relayout: ") + hipGetErrorString(e));
        h.set_strip(w);
    }
    b->parity ^= 1;
    b->tblock = steps;
    int st = is_f64(b->variant) ? batch_upload_params<double>(b) : batch_upload_params<float>(b);
    if (!st) st = batch_build_items(b);
    return st;
}

}  // namespace

extern "C" {

int lbfv_batch_create(int32_t n, const lbfv_case *cs, const lbfv_velset *vel, const lbfv_opts *opts,
                      lbfv_batch **out) {
    if (!out) {
        g_last_error = "NULL batch pointer";
        return LBFV_EINVAL;
    }
    *out = nullptr;
    if (n < 1 || !cs) {
        g_last_error = "lbfv_batch_create: need n >= 1 cases";
        return LBFV_EINVAL;
    }
    lbfv_opts o = {LBFV_FP32, LBFV_STORE_DEV_FP32, 1.0, 0, nullptr};
    if (opts) o = *opts;
    std::string msg;
    for (int i = 0; i < n; ++i) {
        int st = validate_case(&cs[i].mesh, vel, cs[i].tau, cs[i].dt, o.compute, o.storage, msg);
        if (st) {
            g_last_error = "lbfv_batch_create: case " + std::to_string(i) + ": " + msg;
            return st;
        }
        for (int s = 0; s < 4; ++s)
            if (cs[i].bc_kind[s] < 0 || cs[i].bc_kind[s] > BC_SYMMETRY) {
                g_last_error = "lbfv_batch_create: bad boundary kind";
                return LBFV_EINVAL;
            }
        if ((cs[i].bc_kind[0] == BC_PERIODIC) != (cs[i].bc_kind[1] == BC_PERIODIC) ||
            (cs[i].bc_kind[2] == BC_PERIODIC) != (cs[i].bc_kind[3] == BC_PERIODIC)) {
            g_last_error = "lbfv_batch_create: a periodic axis needs both sides periodic";
            return LBFV_EINVAL;
        }
    }
    lbfv_batch *b = new (std::nothrow) lbfv_batch();
    if (!b) return LBFV_ENOMEM;
    b->stream = (hipStream_t)o.hip_stream;
    b->cases.resize(n);
    int st = LBFV_OK;
    for (int i = 0; i < n && !st; ++i) {
        HostCase &h = b->cases[i];
        init_host_case(h, &cs[i].mesh, vel, cs[i].tau, cs[i].dt, o.compute, o.storage, o.rho0);
        for (int s = 0; s < 4; ++s) {
            h.bc[s] = cs[i].bc_kind[s];
            for (int q = 0; q < 3; ++q) h.bcval[s][q] = cs[i].bc_val[s][q];
        }
        b->variant = h.variant;
        double ext[4];
        const hipError_t e = allocate_buffers(h, b->stream);
        if (e != hipSuccess) {
            st = h.buf[0] ? b->fail(LBFV_EHIP, std::string("batch: ") + hipGetErrorString(e))
                          : b->fail(LBFV_ENOMEM, "batch: cannot allocate case buffers");
            break;
        }
        if (upload_metrics(h, ext, b->stream) != hipSuccess) st = b->fail(LBFV_EHIP, "batch: metric upload failed");
    }
    for (auto &h : b->cases) b->bnd = b->bnd || has_boundary(h);
    if (!st) st = is_f64(b->variant) ? batch_upload_params<double>(b) : batch_upload_params<float>(b);
    if (!st) st = batch_build_items(b);
    if (st) {
        lbfv_batch_destroy(b);
        return st;
    }
    *out = b;
    return LBFV_OK;
}

int lbfv_batch_destroy(lbfv_batch *b) {
    if (!b) return LBFV_EINVAL;
    (void)hipStreamSynchronize(b->stream);
    batch_drop_graphs(b);
    for (auto &h : b->cases) free_case(h);
    if (b->d_params) (void)hipFree(b->d_params);
    if (b->d_items) (void)hipFree(b->d_items);
    for (int scheme : {0, 1}) drop_patches(b, scheme);
    b->transfer.release();
    delete b;
    return LBFV_OK;
}

int lbfv_batch_set_shape(lbfv_batch *b, int32_t graph_steps, int32_t rows) {
    if (!b) return LBFV_EINVAL;
    if (graph_steps < 0 || rows < 0) return b->fail(LBFV_EINVAL, "bad shape");
    if (graph_steps > 0) b->gsteps = graph_steps;
    batch_drop_graphs(b);
    if (rows > 0) b->form = FORM_MARCH;
    if (rows > 0 && rows != b->rows) {
        b->rows = rows;
        return batch_build_items(b);
    }
    return LBFV_OK;
}

int lbfv_batch_get_shape(const lbfv_batch *b, int32_t *graph_steps, int32_t *rows) {
    if (!b || !graph_steps || !rows) return LBFV_EINVAL;
    *graph_steps = b->gsteps;
    *rows = b->rows;
    return LBFV_OK;
}

int lbfv_batch_set_grid_form(lbfv_batch *b, int32_t wave_per_item) {
    if (!b) return LBFV_EINVAL;
    if (wave_per_item != 0 && wave_per_item != 1) return b->fail(LBFV_EINVAL, "lbfv_batch_set_grid_form: 0 or 1");
    b->form = FORM_MARCH;
    if ((bool)wave_per_item != b->wave_per_item) {
        b->wave_per_item = wave_per_item;
        batch_drop_graphs(b);
    }
    return LBFV_OK;
}

int lbfv_batch_get_grid_form(const lbfv_batch *b, int32_t *wave_per_item) {
    if (!b || !wave_per_item) return LBFV_EINVAL;
    *wave_per_item = b->wave_per_item ? 1 : 0;
    return LBFV_OK;
}

int lbfv_batch_set_wave_pairs(lbfv_batch *b, int32_t on) {
    if (!b) return LBFV_EINVAL;
    if (on != 0 && on != 1) return b->fail(LBFV_EINVAL, "lbfv_batch_set_wave_pairs: 0 or 1");
    b->form = FORM_MARCH;
    if ((bool)on != b->pairs) {
        b->pairs = on;
        batch_drop_graphs(b);
    }
    return LBFV_OK;
}

int lbfv_batch_get_wave_pairs(const lbfv_batch *b, int32_t *on) {
    if (!b || !on) return LBFV_EINVAL;
    *on = b->pairs ? 1 : 0;
    return LBFV_OK;
}

int lbfv_batch_set_time_block(lbfv_batch *b, int32_t steps) {
    if (!b) return LBFV_EINVAL;
    if (steps != 1 && steps != 2) return b->fail(LBFV_EINVAL, "lbfv_batch_set_time_block: steps must be 1 or 2");
    b->form = FORM_MARCH;
    return batch_set_time_block(b, steps);
}

int lbfv_batch_get_time_block(const lbfv_batch *b, int32_t *steps) {
    if (!b || !steps) return LBFV_EINVAL;
    *steps = b->tblock;
    return LBFV_OK;
}

int lbfv_batch_autotune(lbfv_batch *b, int scheme, int32_t trial_steps, double *best_ms) {
    if (!b) return LBFV_EINVAL;
    if (scheme != LBFV_DUGKS && scheme != LBFV_BKG) return b->fail(LBFV_EINVAL, "unknown scheme");
    if (trial_steps < 1) return b->fail(LBFV_EINVAL, "trial_steps must be >= 1");
    // save the current state of every case in one staging block
    size_t total = 0;
    for (const auto &h : b->cases) total += h.buffer_bytes();
    char *save = nullptr;
    if (hipMalloc((void **)&save, total) != hipSuccess) {
        (void)hipGetLastError();
        return b->fail(LBFV_ENOMEM, "batch autotune: cannot allocate the state copy");
    }
    const int parity0 = b->parity, rows0 = b->rows, gsteps0 = b->gsteps, tb0 = b->tblock, form0 = b->form;
    const bool wpi0 = b->wave_per_item, pairs0 = b->pairs;
    int one_rows = rows0;                    // the fastest marches of one step per launch
    bool one_wpi = wpi0;
    double best_one = INFINITY;
    int patch_halo = 0, patch_waves = 0;     // the patch form, where it is fastest
    hipError_t e = hipSuccess;
    size_t off = 0;
    for (const auto &h : b->cases) {
        if (e == hipSuccess)
            e = hipMemcpyAsync(save + off, h.buf[parity0], h.buffer_bytes(), hipMemcpyDeviceToDevice, b->stream);
        off += h.buffer_bytes();
    }
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (e == hipSuccess) e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    int st = e == hipSuccess ? LBFV_OK : b->fail(LBFV_EHIP, std::string("batch autotune: ") + hipGetErrorString(e));
    // candidates: time blocks 1 and 2, times row-block heights (powers of two and the cost
    // model's best), times the two grid forms; each is timed as one replay of a graph of ts
    // launches after a first replay that builds and warms it (ts even, so both replays use
    // one graph); the trials advance the state, which is put back below
    const int ts = trial_steps + (trial_steps & 1);
    int best_rows = rows0, best_tb = tb0;
    bool best_wpi = wpi0, best_pairs = pairs0;
    double best = INFINITY;
    b->gsteps = ts;
    b->form = FORM_MARCH;
    // one replay of a graph of ts launches of `per` steps after a first that builds and warms it:
    // ms per step
    auto replay = [&](int per, double &ms) {
        int rs = lbfv_batch_step(b, scheme, per * ts);
        if (rs) return rs;
        float t = 0;
        hipError_t he = hipEventRecord(e0, b->stream);
        if (he == hipSuccess && (rs = lbfv_batch_step(b, scheme, per * ts))) return rs;
        if (he == hipSuccess) he = hipEventRecord(e1, b->stream);
        if (he == hipSuccess) he = hipEventSynchronize(e1);
        if (he == hipSuccess) he = hipEventElapsedTime(&t, e0, e1);
        if (he != hipSuccess) return b->fail(LBFV_EHIP, std::string("batch autotune timing: ") + hipGetErrorString(he));
        ms = t / (per * ts);
        return (int)LBFV_OK;
    };
    // (time block, pair of waves per item): one step; two steps with one wave or a pair
    for (auto form : std::vector<std::pair<int, bool>>{{1, false}, {2, false}, {2, true}}) {
        const int tb = form.first;
        b->pairs = form.second;
        if (st || (st = batch_set_time_block(b, tb))) break;
        std::vector<int> heights = {2, 4, 8, 16, 32, 64};
        for (int r : batch_balanced_rows(b, batch_slots(b, scheme, tb == 2), 3))
            if (std::find(heights.begin(), heights.end(), r) == heights.end()) heights.push_back(r);
        for (int trial = 0; trial < 2 * (int)heights.size() && !st; ++trial) {
            const int r = heights[trial >> 1];
            b->wave_per_item = trial & 1;
            b->rows = r;
            if ((st = batch_build_items(b))) break;
            double ms;
            if ((st = replay(tb, ms))) break;
            if (ms < best) {
                best = ms;
                best_rows = r;
                best_tb = tb;
                best_wpi = b->wave_per_item;
                best_pairs = b->pairs;
            }
            if (tb == 1 && ms < best_one) {
                best_one = ms;
                one_rows = r;
                one_wpi = b->wave_per_item;
            }
        }
    }
    // the patch form at each halo width and workgroup size that the cost model does not put far
    // behind the fastest marches
    if (!st && !(st = batch_set_time_block(b, 1))) {
        b->form = FORM_PATCH;
        for (int k = 0; k < 2 * PATCH_HALO && !st; ++k) {
            const int hw = 1 + k / 2, mw = k & 1 ? 8 : 4;
            if ((st = make_patches(b, scheme, hw, mw))) break;
            if (!b->patches[scheme].waves || b->patches[scheme].cost > 1.5e3 * best) continue;
            batch_drop_graphs(b);
            double ms;
            if ((st = replay(hw, ms))) break;
            if (ms < best) {
                best = ms;
                patch_halo = hw;
                patch_waves = mw;
            }
        }
    }
    if (patch_halo) {
        // the march controls then hold the fastest march of the same (one-step) layout
        best_tb = 1;
        best_pairs = false;
        best_rows = one_rows;
        best_wpi = one_wpi;
    }
    // restore the layout, the state, the parity and the graph length (the saved state is
    // in the layout of the entry time block); keep the fastest shape
    (void)hipStreamSynchronize(b->stream);
    b->gsteps = gsteps0;
    b->tblock = tb0;
    b->wave_per_item = st ? wpi0 : best_wpi;
    b->pairs = st ? pairs0 : best_pairs;
    for (auto &h : b->cases) h.set_strip(tb0 == 2 ? STRIP2 : STRIP1);
    b->rows = st ? rows0 : best_rows;
    int st2 = is_f64(b->variant) ? batch_upload_params<double>(b) : batch_upload_params<float>(b);
    if (!st2) st2 = batch_build_items(b);
    off = 0;
    hipError_t re = hipSuccess;
    for (const auto &h : b->cases) {
        if (re == hipSuccess)
            re = hipMemcpyAsync(h.buf[parity0], save + off, h.buffer_bytes(), hipMemcpyDeviceToDevice, b->stream);
        off += h.buffer_bytes();
    }
    if (re == hipSuccess) re = hipStreamSynchronize(b->stream);
    b->parity = parity0;
    (void)hipFree(save);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    drop_patches(b, scheme);
    b->form = st ? form0 : FORM_MARCH;
    if (st) return st;
    if (st2) return st2;
    if (re != hipSuccess) return b->fail(LBFV_EHIP, std::string("batch autotune restore: ") + hipGetErrorString(re));
    if ((st = batch_set_time_block(b, best_tb))) return st;
    if (patch_halo) {
        if ((st = make_patches(b, scheme, patch_halo, patch_waves))) return st;
        if (b->patches[scheme].waves) b->form = FORM_PATCH;
    }
    batch_drop_graphs(b);
    if (best_ms) *best_ms = best;
    return LBFV_OK;
}

int lbfv_batch_info(const lbfv_batch *b, int64_t *cells, int32_t *items) {
    if (!b) return LBFV_EINVAL;
    int64_t t = 0;
    for (auto &h : b->cases) t += (int64_t)h.nx * h.ny;
    if (cells) *cells = t;
    if (items) *items = b->nitems;
    return LBFV_OK;
}

int lbfv_batch_init_equilibrium(lbfv_batch *b, int32_t ci, const double *rho, const double *ux, const double *uy) {
    if (!b) return LBFV_EINVAL;
    if (ci < 0 || ci >= (int)b->cases.size() || !rho || !ux || !uy) return b->fail(LBFV_EINVAL, "bad case or field");
    const HostCase &h = b->cases[ci];
    const FieldArrays a = field_arrays(h, {rho, ux, uy});
    return moved(b, move_fields(h, b->parity, b->transfer, b->stream, F_INIT_EQ, a), "batch init_equilibrium");
}

int lbfv_batch_set_f(lbfv_batch *b, int32_t ci, const double *f) {
    if (!b) return LBFV_EINVAL;
    if (ci < 0 || ci >= (int)b->cases.size() || !f) return b->fail(LBFV_EINVAL, "bad case or array");
    const HostCase &h = b->cases[ci];
    return moved(b, move_fields(h, b->parity, b->transfer, b->stream, F_SET_F, state_arrays(h, f)), "batch set_f");
}

int lbfv_batch_get_f(lbfv_batch *b, int32_t ci, double *f) {
    if (!b) return LBFV_EINVAL;
    if (ci < 0 || ci >= (int)b->cases.size() || !f) return b->fail(LBFV_EINVAL, "bad case or array");
    const HostCase &h = b->cases[ci];
    return moved(b, move_fields(h, b->parity, b->transfer, b->stream, F_GET_F, state_arrays(h, f)), "batch get_f");
}

int lbfv_batch_moments(lbfv_batch *b, int32_t ci, double *rho, double *ux, double *uy) {
    if (!b) return LBFV_EINVAL;
    if (ci < 0 || ci >= (int)b->cases.size() || !rho || !ux || !uy) return b->fail(LBFV_EINVAL, "bad case or output");
    const FieldArrays a = field_arrays(b->cases[ci], {rho, ux, uy});
    return moved(b, move_fields(b->cases[ci], b->parity, b->transfer, b->stream, F_MOMENTS, a), "batch moments");
}

int lbfv_batch_nonfinite(lbfv_batch *b, int32_t *count) {
    if (!b) return LBFV_EINVAL;
    if (!count) return b->fail(LBFV_EINVAL, "NULL count array");
    const int n = (int)b->cases.size();
    int32_t *d;
    if (hipMalloc((void **)&d, n * sizeof(int32_t)) != hipSuccess) {
        (void)hipGetLastError();
        return b->fail(LBFV_ENOMEM, "staging");
    }
    const double c = b->cases[0].c;
    const RefState rho0 = b->cases[0].ref();
    switch (b->variant) {
    case V_F64:
        hipLaunchKernelGGL((batch_nonfinite_kernel<double, double>), dim3(n), dim3(RED_BLOCK), 0, b->stream,
                           (const StepParams<double> *)b->d_params, b->parity, rho0, c, d);
        break;
    case V_F32:
        hipLaunchKernelGGL((batch_nonfinite_kernel<float, float>), dim3(n), dim3(RED_BLOCK), 0, b->stream,
                           (const StepParams<float> *)b->d_params, b->parity, rho0, c, d);
        break;
    case V_BF16:
        hipLaunchKernelGGL((batch_nonfinite_kernel<float, __bf16>), dim3(n), dim3(RED_BLOCK), 0, b->stream,
                           (const StepParams<float> *)b->d_params, b->parity, rho0, c, d);
        break;
    default:
        hipLaunchKernelGGL((batch_nonfinite_kernel<float, _Float16>), dim3(n), dim3(RED_BLOCK), 0, b->stream,
                           (const StepParams<float> *)b->d_params, b->parity, rho0, c, d);
        break;
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(count, d, n * sizeof(int32_t), hipMemcpyDeviceToHost, b->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
    (void)hipFree(d);
    if (e != hipSuccess) return b->fail(LBFV_EHIP, std::string("batch check: ") + hipGetErrorString(e));
    return LBFV_OK;
}

int lbfv_batch_step(lbfv_batch *b, int scheme, int32_t n) {
    if (!b) return LBFV_EINVAL;
    if (scheme != LBFV_DUGKS && scheme != LBFV_BKG) return b->fail(LBFV_EINVAL, "unknown scheme");
    if (n < 0) return b->fail(LBFV_EINVAL, "nsteps must be >= 0");
    bool patch = false;
    int st = batch_use_patches(b, scheme, patch);
    if (st) return st;
    // with a time block of 2 every launch advances two steps; an odd last step is a
    // one-step launch on the same layout.  The patch form takes up to its halo width.
    const bool two = b->tblock == 2;
    const int per = patch ? b->patches[scheme].halo : (two ? 2 : 1);
    const int64_t replay = graph_launches(b, patch);
    while (n >= per * replay) {
        hipGraphExec_t &g = b->gexec[scheme + (patch ? 2 : 0)][b->parity];
        if (!g) {
            st = batch_build_graph(b, scheme, b->parity, patch);
            if (st) return st;
        }
        hipError_t e = hipGraphLaunch(g, b->stream);
        if (e != hipSuccess) return b->fail(LBFV_EHIP, std::string("hipGraphLaunch: ") + hipGetErrorString(e));
        b->parity ^= (int)(replay & 1);
        n -= (int32_t)(per * replay);
    }
    // (patches: an even or odd number of launches as the steps are, like one-step launches, unless
    // the autotuner picked them and no work was captured)
    const bool exact = patch && (b->form == FORM_AUTO || b->captured);
    int64_t cells = 0;
    for (const auto &h : b->cases) cells += (int64_t)h.nx * h.ny;
    const bool single_marches = patch && cells > batch_single_cells(is_f64(b->variant));
    Cut cut(n, per, exact, single_marches);
    while (const int k = cut.next()) {
        st = patch && !(k == 1 && single_marches) ? batch_launch_patches(b, scheme, b->parity, k)
                                                  : batch_launch_one(b, scheme, b->parity, k == 2);
        if (st) return st;
        b->parity ^= 1;
    }
    return LBFV_OK;
}

}  // extern "C"
