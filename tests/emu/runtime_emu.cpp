// The host runtime (mhd_runtime.cpp) on the CPU: the HIP calls work on host memory, with copies that
// happen only when something waits for them, and the kernel launches do nothing. For what the runtime
// promises about its calls: which of them wait, allocate or take a lock, and what is left under way
// after an error.
//
//   runtime_emu SCENARIO     prints "ok" or what went wrong
#include <stdio.h>
#include <stdlib.h>

#include <atomic>
#include <chrono>
#include <functional>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include <hip/hip_runtime.h>

struct emuStream {
    int device = 0;
    bool capturing = false;
    std::vector<std::function<void()>> todo;            // what a wait still has to do
    std::vector<std::pair<const char *, size_t>> host;  // host ranges that those copies use
};
struct emuEvent {
    int device = 0;
    emuStream *on = nullptr;  // recorded on, and not waited for since
    size_t at = 0;
};
struct emuGraph {};

namespace emu {

std::recursive_mutex mu;
thread_local int device = 0;
std::vector<std::string> calls;         // every call since the last clear()
std::string fail_call;                  // this call fails after fail_after more of them
int fail_after = 0;
std::map<char *, size_t> pinned;
std::string complaint;
extern const size_t sizeof_ctrl;
std::atomic<int> resident_launches{0}, sweep_launches{0};
std::function<void(hipStream_t)> on_graph_launch;
bool gpu_busy = false;  // roll calls are given up
int prepared_on = -1;  // GPU that was current when the resident kernels were prepared

void complain(const std::string &s) {
    if (complaint.empty()) complaint = s;
}
// Notes the call; true if it is to fail.
bool note(const char *name) {
    calls.push_back(name);
    return fail_call == name && fail_after-- == 0;
}
int count(const std::set<std::string> &names) {
    int n = 0;
    for (const auto &c : calls) n += names.count(c) ? 1 : 0;
    return n;
}
void clear() { calls.clear(); }
void drain(emuStream *s, size_t n) {
    for (size_t i = 0; i < n; ++i) s->todo[i]();
    s->todo.erase(s->todo.begin(), s->todo.begin() + (long)n);
    if (s->todo.empty()) s->host.clear();
}
emuStream null_stream;
emuStream *of(hipStream_t s) { return s ? s : &null_stream; }

}  // namespace emu
using namespace emu;

#define CALL(name)                                    \
    std::lock_guard<std::recursive_mutex> lock_(mu);  \
    if (note(name)) return hipErrorUnknown

hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "emulated error"; }
hipError_t hipGetDevice(int *d) { return *d = device, hipSuccess; }
hipError_t hipSetDevice(int d) { return device = d, hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { CALL("hipFuncSetAttribute"); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    CALL("hipHostMalloc");
    *p = aligned_alloc(4096, (n + 4095) / 4096 * 4096);
    pinned[(char *)*p] = n;
    return hipSuccess;
}
std::vector<emuStream *> streams{&null_stream};
hipError_t hipHostFree(void *p) {
    CALL("hipHostFree");
    const size_t n = pinned[(char *)p];
    for (emuStream *s : streams)
        for (auto &r : s->host)
            if (r.first < (char *)p + n && (char *)p < r.first + r.second) complain("pinned memory freed under a copy");
    pinned.erase((char *)p);
    free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { return *d = h, hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st) {
    CALL("hipMemcpyAsync");
    if (k == hipMemcpyDeviceToHost && n == sizeof_ctrl && (uintptr_t)d % 8) complain("control block read to a misaligned address");
    const char *host = k == hipMemcpyDeviceToHost ? (const char *)d : k == hipMemcpyHostToDevice ? (const char *)s : nullptr;
    bool deferred = false;  // a copy from or to pageable memory waits for itself
    for (auto &r : pinned) deferred = deferred || (host >= r.first && host < r.first + r.second);
    if (!deferred && k != hipMemcpyDeviceToDevice) {
        drain(of(st), of(st)->todo.size());
        memcpy(d, s, n);
        return hipSuccess;
    }
    if (host) of(st)->host.push_back({host, n});
    of(st)->todo.push_back([=] { memcpy(d, s, n); });
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st) {
    CALL("hipMemsetAsync");
    of(st)->todo.push_back([=] { memset(d, v, n); });
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    CALL("hipStreamSynchronize");
    drain(of(s), of(s)->todo.size());
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { CALL("hipStreamWaitEvent"); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c) {
    CALL("hipStreamIsCapturing");
    *c = of(s)->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) { CALL("hipStreamBeginCapture"); s->capturing = true; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) {
    CALL("hipStreamEndCapture");
    s->capturing = false;
    *g = new emuGraph;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    CALL("hipGraphInstantiate");
    *e = new emuGraph;
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { delete e; return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) {
    {
        CALL("hipGraphLaunch");
    }
    if (on_graph_launch) on_graph_launch(s);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { CALL("hipEventCreate"); *e = new emuEvent; (*e)->device = device; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { CALL("hipEventDestroy"); delete e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    CALL("hipEventRecord");
    if (e->device != of(s)->device) return hipErrorInvalidHandle;  // as HIP has it
    e->on = of(s);
    e->at = of(s)->todo.size();
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) { CALL("hipEventQuery"); return e->on && !e->on->todo.empty() ? hipErrorNotReady : hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) {
    CALL("hipEventSynchronize");
    if (e->on) drain(e->on, e->on->todo.size());  // later copies as well: they may have happened
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }

#include "../../paper_2211_09370_amd/csrc/mhd_runtime.cpp"

const size_t emu::sizeof_ctrl = sizeof(mhd::DevCtrl);

namespace mhd {  // launches: counted, nothing else
SweepArgs make_sweep_args(const void *, const void *, void *, const float *, StepConst, SweepLaunch) {
    SweepArgs a{};
    a.nblocks = 1;
    return a;
}
hipError_t launch_ctrl_begin(hipStream_t, DevCtrl *, StepConst, int *, int) { return hipSuccess; }
hipError_t launch_step_end(hipStream_t, DevCtrl *, const double *, StepConst, double) { return hipSuccess; }
hipError_t launch_mag_sweep(hipStream_t, int, const SweepArgs &, SweepLaunch, hipEvent_t, hipEvent_t) { return ++sweep_launches, hipSuccess; }
hipError_t launch_mag_resident(hipStream_t, const ResArgs &a, const ResPlan &, bool) {
    if (gpu_busy) ++a.host[0];  // as the stand-in of a roll call given up counts it
    return ++resident_launches, hipSuccess;
}
hipError_t prepare_mag_resident(const ResPlan &) { return prepared_on = device, hipSuccess; }
hipError_t launch_ib(hipStream_t, int, void *, float, float, const IbArgs &) { return hipSuccess; }
hipError_t launch_lorentz(hipStream_t, int, const void *, const void *, const float *, const float *, const DevCtrl *, float *, StepConst) { return hipSuccess; }
hipError_t launch_fluid(hipStream_t, int, const void *, const void *, const float *, void *, void *, void *, StepConst) { return hipSuccess; }
hipError_t launch_flow_partial(hipStream_t, int, const void *, double *, StepConst) { return hipSuccess; }
hipError_t launch_lorentz_fluid(hipStream_t, const LfArgs &) { return hipSuccess; }
hipError_t launch_budget(hipStream_t, int, const void *, const void *, const void *, const void *, const float *, const float *, DevCtrl *, double *, mhd_budget *, StepConst) { return hipSuccess; }
hipError_t launch_ctrl_begin_batch(hipStream_t, const PipeStep *, int) { return hipSuccess; }
hipError_t launch_step_end_batch(hipStream_t, const PipeStep *, int) { return hipSuccess; }
hipError_t launch_mag_sweep_batch(hipStream_t, int, SweepLaunch, const PipeStep *, const BlockMap *, int, int, hipEvent_t, hipEvent_t) { return ++sweep_launches, hipSuccess; }
hipError_t launch_ib_interp_batch(hipStream_t, int, const PipeStep *, const BlockMap *, int, int) { return hipSuccess; }
hipError_t launch_ib_spread_batch(hipStream_t, int, const PipeStep *, const BlockMap *, int, int) { return hipSuccess; }
hipError_t launch_lorentz_batch(hipStream_t, int, const PipeStep *, const BlockMap *, int, bool) { return hipSuccess; }
hipError_t launch_fluid_batch(hipStream_t, int, const PipeStep *, const BlockMap *, int, bool) { return hipSuccess; }
hipError_t launch_flow_partial_batch(hipStream_t, int, const PipeStep *, int) { return hipSuccess; }
hipError_t launch_store_kind(hipStream_t, int, const float *, void *, int64_t) { return hipSuccess; }
hipError_t launch_load_kind(hipStream_t, int, const void *, float *, int64_t) { return hipSuccess; }
hipError_t launch_store_split(hipStream_t, const float *, void *, void *, int64_t) { return hipSuccess; }
hipError_t launch_reset_records(hipStream_t, DevCtrl *) { return hipSuccess; }
hipError_t launch_residual_final(hipStream_t, const double *, double *) { return hipSuccess; }
}  // namespace mhd

void mark_stalled(DevCtrl *c) { c->stalled = 1; }

// A box of 8 x 32 x 32 with a ring wall (it has a resident plan) on a stream of a device.
struct Box {
    emuStream stream;
    std::vector<char> ws;
    mhd_sim *sim = nullptr;
    mhd_grid_desc g{};
    explicit Box(int dev = 0, int nx = 8, int ny = 32, int nz = 32) {
        stream.device = dev;
        {
            std::lock_guard<std::recursive_mutex> l(mu);
            streams.push_back(&stream);
        }
        g.nx = nx;
        g.ny = ny;
        g.nz = nz;
        const int lines = 60;
        size_t bytes = 0;
        check(mhd_workspace_size(&g, (int64_t)lines * nx, &bytes));
        ws.resize(bytes + 256);
        const int before = device;
        device = dev;
        check(mhd_create(&g, (int64_t)lines * nx, (void *)(((uintptr_t)ws.data() + 255) & ~(uintptr_t)255), bytes, &stream, &sim));
        device = before;
    }
    static void check(mhd_status st) {
        if (st != MHD_OK) {
            printf("status %d: %s\n", st, mhd_last_error());
            fflush(stdout);
            _Exit(0);
        }
    }
    void wall(double R = 9.0) {
        const int lines = 60, M = lines * g.nx;
        std::vector<double> x(3 * (size_t)M);
        for (int l = 0; l < lines; ++l)
            for (int i = 0; i < g.nx; ++i) {
                x[(size_t)(l * g.nx + i)] = i;
                x[(size_t)(M + l * g.nx + i)] = g.ny / 2 + R * std::cos(2 * M_PI * l / lines);
                x[(size_t)(2 * M + l * g.nx + i)] = g.nz / 2 + R * std::sin(2 * M_PI * l / lines);
            }
        check(mhd_set_markers(sim, x.data(), M, nullptr, nullptr));
    }
    void params(int n_mag = 12) {
        mhd_params p{};
        p.nu = 0.05;
        p.eta = 3.0;
        p.n_mag = n_mag;
        check(mhd_set_params(sim, &p));
    }
    ~Box() { check(mhd_destroy(sim)); }
};
const std::set<std::string> kWaits{"hipStreamSynchronize", "hipEventSynchronize", "hipMemcpyAsync", "hipMemsetAsync"};
const std::set<std::string> kAllocs{"hipHostMalloc", "hipHostFree", "hipEventCreate", "hipEventDestroy"};

const char *first_call(const std::set<std::string> &names) {
    for (const auto &c : calls)
        if (names.count(c)) return c.c_str();
    return "";
}

// The first step after new markers or parameters only launches.
std::string step_only_launches(bool noalloc) {
    std::vector<char> scratch(64 << 20);
    for (int order = 0; order < 2; ++order) {
        Box b;
        if (order) b.params();
        b.wall();
        if (!order) b.params();
        for (int k = 0; k < 3; ++k) {
            clear();
            const int before = resident_launches;
            Box::check(noalloc ? step_in_scratch(b.sim, 2, 0, scratch.data()) : mhd_step(b.sim, 2, 0));
            if (count(kWaits)) return std::string("a step called ") + first_call(kWaits);
            if (count(kAllocs)) return std::string("a step called ") + first_call(kAllocs);
            if (resident_launches == before && (noalloc || k == 0)) return "the step was not a resident one";
            if (k == 0) b.wall(8.0);
            if (k == 1) b.params(13);
        }
    }
    return "ok";
}

// While a box is held up in the middle of a long call (its launches block, as they do when the stream is
// full), a box on another GPU steps all the same.
std::string other_gpu_steps() {
    Box a(0), b(1);
    for (Box *x : {&a, &b}) device = x->stream.device, x->wall(), x->params();
    std::atomic<bool> held{false}, go{false}, done{false};
    on_graph_launch = [&](hipStream_t s) {
        if (s != &a.stream) return;
        held = true;
        while (!go) std::this_thread::yield();
    };
    std::thread ta([&] { Box::check(mhd_step(a.sim, 4, 0)); });
    while (!held) std::this_thread::yield();
    std::thread tb([&] {
        device = 1;
        Box::check(mhd_step(b.sim, 2, 0));
        done = true;
    });
    for (int i = 0; i < 2000 && !done; ++i) std::this_thread::sleep_for(std::chrono::milliseconds(1));
    const bool free_to_go = done;
    go = true;
    ta.join();
    tb.join();
    device = 0;
    on_graph_launch = nullptr;
    return free_to_go ? "ok" : "a step on another GPU waited for this call";
}

// On one GPU, a short call waits for a bounded part of a long one at most.
std::string long_call_lets_others_in() {
    Box a, b;
    for (Box *x : {&a, &b}) x->wall(), x->params(), Box::check(mhd_step(x->sim, 2, 0));
    std::atomic<int> launched{0};
    on_graph_launch = [&](hipStream_t s) {
        if (s == &a.stream) ++launched, std::this_thread::sleep_for(std::chrono::milliseconds(1));
    };
    const int steps = 2000;
    std::thread ta([&] { Box::check(mhd_step(a.sim, steps, 0)); });
    while (launched < 10) std::this_thread::yield();
    Box::check(mhd_step(b.sim, 1, 0));
    const int at = launched;
    ta.join();
    on_graph_launch = nullptr;
    return at < steps / 2 ? "ok" : "a step waited for " + std::to_string(at) + " steps of another box";
}

// Calls made while another GPU is the thread's current one: what they create belongs to the machine's GPU.
std::string other_device_current() {
    Box b(1);
    device = 0;
    const size_t n = 3 * (size_t)b.g.nx * b.g.ny * b.g.nz;
    std::vector<double> f(n, 0.25), g(n);
    b.wall();
    b.params();
    Box::check(mhd_set_field(b.sim, MHD_FIELD_U, f.data()));
    Box::check(mhd_step(b.sim, 2, 0));
    Box::check(mhd_get_field(b.sim, MHD_FIELD_RHO, g.data()));
    if (prepared_on != 1) return "the kernels were prepared on another GPU";
    return device == 0 ? "ok" : "the current GPU was changed";
}

// Fields of boxes of odd cell counts, alone, read and written back.
std::string odd_counts() {
    for (int nx : {1, 5, 7}) {
        Box b(0, nx, 9, 11);
        b.params();
        const size_t n = (size_t)nx * 9 * 11;
        std::vector<double> f(3 * n, 0.25), g(3 * n);
        Box::check(mhd_set_field(b.sim, MHD_FIELD_U, f.data()));
        Box::check(mhd_get_field(b.sim, MHD_FIELD_U, g.data()));
        if (f != g) return "read back differs";
        Box::check(mhd_get_field(b.sim, MHD_FIELD_RHO, g.data()));
    }
    return "ok";
}

// A HIP call that fails in the middle of a field copy: the call returns with no copy of the pinned chunks
// under way, and the next calls work.
std::string error_in_a_copy() {
    for (const char *call : {"hipMemcpyAsync", "hipEventRecord", "hipEventSynchronize", "hipHostMalloc", "hipEventCreate"})
        for (int after = 0; after < 6; ++after)
            for (int write = 0; write < 2; ++write) {
                Box b(0, 96, 80, 80);  // several chunks
                b.params();
                const size_t n = 3 * (size_t)b.g.nx * b.g.ny * b.g.nz;
                std::vector<double> f(n, 0.25), g(n);
                auto copy = [&] { return write ? mhd_set_field(b.sim, MHD_FIELD_U, f.data()) : mhd_get_field(b.sim, MHD_FIELD_U, g.data()); };
                fail_call = call;
                fail_after = after;
                const mhd_status st = copy();
                const bool failed = fail_after < 0;
                fail_call = "";
                if (failed != (st != MHD_OK)) return std::string("an error of ") + call + " was not reported";
                if (failed && !b.stream.host.empty()) return std::string("copies under way after an error of ") + call;
                Box::check(mhd_set_field(b.sim, MHD_FIELD_U, f.data()));
                Box::check(mhd_get_field(b.sim, MHD_FIELD_U, g.data()));
                if (f != g) return std::string("read back differs after an error of ") + call;
            }
    return "ok";
}

// A step that stalled is reported as such, also where the state it left is an unstable one.
std::string stall_report() {
    Box b;
    b.params();
    std::vector<double> g(3 * (size_t)b.g.nx * b.g.ny * b.g.nz);
    DevCtrl *c = b.sim->ctrl();
    mark_stalled(c);
    c->status = 1;  // as the fluid update and the budget pass store it
    const mhd_status st = mhd_get_field(b.sim, MHD_FIELD_U, g.data());
    if (st != MHD_ERR_HIP) return "the stall of a step was reported as " + std::to_string(st);
    int64_t n = 0;
    if (mhd_get_budgets(b.sim, nullptr, 0, &n) != MHD_ERR_HIP) return "the stall was not reported with the budgets";
    return "ok";
}

// After a roll call was given up, steps launch their sweeps one by one for a while: 64, then twice as
// many each time it happens again, and 64 again once the GPU has long been free.
std::string given_up() {
    Box b;
    b.wall();
    b.params(1);
    Box::check(mhd_set_graph(b.sim, 0));
    auto resident_steps = [&](int n) {
        const int before = resident_launches;
        for (int i = 0; i < n; ++i) Box::check(mhd_step(b.sim, 1, 0));
        return resident_launches - before;
    };
    if (resident_steps(5) != 5) return "not resident on a free GPU";
    for (int wait = 64; wait <= 256; wait *= 2) {
        gpu_busy = true;
        if (resident_steps(1) != 1) return "the step before the roll call is given up";
        gpu_busy = false;
        if (resident_steps(wait) != 0) return "resident right after a roll call was given up (" + std::to_string(wait) + ")";
        if (resident_steps(3) != 3) return "not resident again after " + std::to_string(wait) + " steps";
    }
    if (resident_steps(16 * 256) != 16 * 256) return "not resident on a GPU that is free again";
    gpu_busy = true;
    resident_steps(1);
    gpu_busy = false;
    if (resident_steps(66) != 2) return "the number of steps was not set back";
    // a long call looks between its steps
    gpu_busy = true;
    const int before = resident_launches;
    Box::check(mhd_step(b.sim, 1000, 0));
    const int tried = resident_launches - before;
    gpu_busy = false;
    return tried > 0 && tried < 1000 / 4 ? "ok" : "a long call made " + std::to_string(tried) + " resident steps of 1000 on a busy GPU";
}

// Sweep launches of a round of a batch of n boxes of each of the given lengths (32 x 32 cross-section).
int batch_launches(int n, std::vector<int> lengths) {
    std::vector<mhd_pipe_desc> d;
    for (int i = 0; i < n; ++i)
        for (int nx : lengths) {
            mhd_pipe_desc p{};
            p.grid.nx = nx;
            p.grid.ny = p.grid.nz = 32;
            d.push_back(p);
        }
    size_t bytes = 0;
    Box::check(mhd_batch_workspace_size(d.data(), (int)d.size(), &bytes));
    char *ws = (char *)aligned_alloc(256, (bytes + 255) / 256 * 256);
    emuStream st;
    mhd_batch *b = nullptr;
    Box::check(mhd_batch_create(d.data(), (int)d.size(), ws, bytes, &st, &b));
    for (int i = 0; i < (int)d.size(); ++i) {
        mhd_sim *s = nullptr;
        Box::check(mhd_batch_pipe(b, i, &s));
        mhd_params p{};
        p.nu = 0.05;
        p.eta = 3.0;
        p.n_mag = 2;
        Box::check(mhd_set_params(s, &p));
    }
    Box::check(mhd_batch_set_graph(b, 0));
    const int before = sweep_launches;
    Box::check(mhd_batch_step(b, 1, 0));
    const int launches = (sweep_launches - before) / 2;
    Box::check(mhd_batch_destroy(b));
    free(ws);
    return launches;
}

// Boxes of different tile forms share a sweep launch where that saves more than it costs: 2000 workgroups
// of single cells a launch saved (4, 8 and 16 of a box of 8, 16 and 32 here).
std::string batch_forms() {
    struct {
        int n;
        std::vector<int> lengths;
        int launches;
    } cases[] = {{2, {16, 32}, 1}, {32, {16, 32}, 1}, {128, {16, 32}, 2}, {128, {8, 16, 32}, 1}, {160, {8, 16, 32}, 3}, {64, {32}, 1},
                 {300, {32}, 1}, {8, {8, 64, 128}, 1}, {40, {64, 128}, 1}, {64, {64, 128}, 2}};
    for (const auto &c : cases) {
        const int got = batch_launches(c.n, c.lengths);
        if (got != c.launches)
            return std::to_string(c.n) + " boxes of " + std::to_string(c.lengths.size()) + " lengths from " + std::to_string(c.lengths[0]) +
                   ": " + std::to_string(got) + " launches";
    }
    return "ok";
}

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    std::string r = "unknown scenario";
    if (what == "step") r = step_only_launches(false);
    if (what == "step_noalloc") r = step_only_launches(true);
    if (what == "other_gpu") r = other_gpu_steps();
    if (what == "device") r = other_device_current();
    if (what == "odd_counts") r = odd_counts();
    if (what == "copy_error") r = error_in_a_copy();
    if (what == "stall") r = stall_report();
    if (what == "given_up") r = given_up();
    if (what == "batch_forms") r = batch_forms();
    if (what == "long_call") r = long_call_lets_others_in();
    puts((complaint.empty() ? r : complaint).c_str());
    fflush(stdout);
    return 0;
}
