// The resident magnetic iteration (mhd_resident.hip) on the CPU: launched through its own launcher on
// emulated workgroups and compared, bit for bit, with the same sweeps and wall corrections written as
// plain loops over the box. The emulation checks that all work-items of a workgroup come to the same
// barrier, and runs them in turn forwards and backwards between barriers, so that an unordered
// access to LDS shows as a difference.
//
//   resident_emu nx ny nz radius n_mag lattice alpha magnets max_wg mode workers
//
// radius 0: no wall; max_wg: compute units the plan is made for; mode: 1 resident, 2 the stand-in, 3 the
// stand-in after a roll call given up, 4 resident and a neighbour never comes, 5 the stand-in of a later
// step; workers: workgroups on the chip at once (the others start when one ends). Prints one line: the
// plan, then "ok" or what went wrong.
#include <sched.h>
#include <stdio.h>
#include <stdlib.h>
#include <time.h>
#include <ucontext.h>

#include <atomic>
#include <functional>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include <hip/hip_runtime.h>

namespace emu {

thread_local Lane lane;

struct Group {  // a workgroup in flight
    ucontext_t main;
    std::vector<ucontext_t> ctx;
    std::vector<char> stacks;
    std::vector<int> at;  // line of the barrier a work-item waits at; 0 under way, -1 ended
    int cur = 0;
    std::function<void()> body;
};
thread_local Group *group = nullptr;
std::mutex error_mu;

[[noreturn]] void report(const std::string &what) {  // ends the process: other workgroups would wait for this one
    std::lock_guard<std::mutex> l(error_mu);
    puts(what.c_str());
    fflush(stdout);
    _Exit(0);
}
void leave(int at) {
    Group &g = *group;
    g.at[(size_t)g.cur] = at;
    swapcontext(&g.ctx[(size_t)g.cur], &g.main);
}
void barrier(int line) { leave(line); }
void pause() { leave(0); }
bool fast_clock = false;
long long clock() {  // a slow clock: the emulation is slow as well
    static std::atomic<long long> fast{0};
    if (fast_clock) return fast += 10000000;
    timespec t;
    clock_gettime(CLOCK_MONOTONIC, &t);
    return t.tv_sec * 1000000ll + t.tv_nsec / 1000;
}
void entry() {
    group->body();
    leave(-1);
}

constexpr size_t kStack = 48 * 1024;
void run_group(unsigned block, unsigned blocks, unsigned threads, const std::function<void()> &body) {
    Group g;
    g.ctx.resize(threads);
    g.stacks.resize(threads * kStack);
    g.at.assign(threads, 0);
    g.body = body;
    group = &g;
    for (unsigned t = 0; t < threads; ++t) {
        getcontext(&g.ctx[t]);
        g.ctx[t].uc_stack.ss_sp = g.stacks.data() + t * kStack;
        g.ctx[t].uc_stack.ss_size = kStack;
        g.ctx[t].uc_link = nullptr;
        makecontext(&g.ctx[t], entry, 0);
    }
    for (int phase = 0;; ++phase) {
        std::fill(g.at.begin(), g.at.end(), 0);
        for (bool again = true; again;) {
            again = false;
            for (unsigned k = 0; k < threads; ++k) {
                const unsigned t = phase & 1 ? threads - 1 - k : k;
                if (g.at[t] != 0) continue;
                g.cur = (int)t;
                lane = {t, block, threads, blocks};
                swapcontext(&g.main, &g.ctx[t]);
                again = again || g.at[t] == 0;
            }
            if (again) sched_yield();
        }
        for (unsigned t = 1; t < threads; ++t)
            if (g.at[t] != g.at[0])
                report("workgroup " + std::to_string(block) + ": work-item 0 is at line " + std::to_string(g.at[0]) +
                       " and work-item " + std::to_string(t) + " at line " + std::to_string(g.at[t]));
        if (g.at[0] < 0) return;
    }
}

int workers = 1;

}  // namespace emu

namespace mhd {
thread_local __attribute__((aligned(16))) float lds[160 * 1024 / 4];
}

// the kernel's asm statements are empty ones that hide a value from the optimiser
#define asm
#define volatile(...)
#include "../../paper_2211_09370_amd/csrc/mhd_resident.hip"
#undef asm
#undef volatile

hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t bytes, hipStream_t) {
    if (bytes > sizeof mhd::lds) return hipErrorUnknown;
    std::atomic<unsigned> next{0};
    std::vector<std::thread> pool;
    for (int w = 0; w < emu::workers; ++w)
        pool.emplace_back([&] {
            for (unsigned b; (b = next.fetch_add(1)) < grid.x;) {
                memset(mhd::lds, 0xff, sizeof mhd::lds);  // NaN: what is read before it is written shows
                emu::run_group(b, grid.x, block.x, [&] {
                    reinterpret_cast<void (*)(mhd::ResArgs)>(const_cast<void *>(f))(*static_cast<mhd::ResArgs *>(args[0]));
                });
            }
        });
    for (auto &t : pool) t.join();
    return hipSuccess;
}

using namespace mhd;

// Wall of a straight pipe around the box's middle as mhd_set_markers stores it: lines at unit spacing on
// a circle, the nonzero ones of their 3 x 3 Lagrange taps (padded with the first, weight 0).
ResWall ring_wall(int ny, int nz, double R) {
    ResWall w;
    if (R <= 0) return w;
    const int n = (int)(2 * M_PI * R + 0.5);
    auto lagrange = [](double X, double (&v)[3]) {
        const int n0 = (int)floor(X + 0.5);
        const double s = X - n0;
        v[0] = -0.5 * s * (1 - s);
        v[1] = 1 - s * s;
        v[2] = 0.5 * s * (1 + s);
        return n0 - 1;
    };
    using Taps = std::vector<std::pair<int, float>>;  // (row or line, weight)
    std::vector<Taps> lines((size_t)n), rows((size_t)ny * nz);
    for (int l = 0; l < n; ++l) {
        double wy[3], wz[3];
        const int y = lagrange(ny / 2 + R * cos(2 * M_PI * l / n), wy), z = lagrange(nz / 2 + R * sin(2 * M_PI * l / n), wz);
        for (int c = 0; c < 9; ++c) {
            const int row = ((y + c % 3) % ny + ny) % ny + ny * (((z + c / 3) % nz + nz) % nz);
            const double wt = wy[c % 3] * wz[c / 3];
            if (wt == 0.0) continue;
            lines[(size_t)l].push_back({row, (float)wt});
            rows[(size_t)row].push_back({l, (float)wt});
        }
    }
    auto put = [](const Taps &t, int len, std::vector<int> &at, std::vector<float> &wt) {
        for (int q = 0; q < len; ++q) {
            at.push_back(q < (int)t.size() ? t[(size_t)q].first : t[0].first);
            wt.push_back(q < (int)t.size() ? t[(size_t)q].second : 0.0f);
        }
    };
    for (const Taps &t : lines) w.tm = std::max(w.tm, (int)t.size());
    for (const Taps &t : rows) w.km = std::max(w.km, (int)t.size());
    for (const Taps &t : lines) put(t, w.tm, w.tap_row, w.tap_w);
    for (size_t r = 0; r < rows.size(); ++r) {
        if (rows[r].empty()) continue;
        w.band_row.push_back((int)r);
        put(rows[r], w.km, w.band_line, w.band_w);
    }
    return w;
}

// What the tables have to hold for every wait to end and every read to find its value. Empty: all right.
std::string check_plan(const ResPlan &p, int nx, int ny, int nz, const ResWall &w, int max_wg) {
    auto bad = [](const char *what) { return std::string(what); };
    const int PY = p.ty + 2, GR = PY * (p.tz + 2), nyz = p.gy * p.gz;
    if (p.nwg != p.gx * nyz || p.nwg > max_wg || p.nwg > kResMaxTiles) return bad("more tiles than compute units");
    if (p.tx * p.gx < nx || p.tx * (p.gx - 1) >= nx || p.ty * p.gy < ny || p.tz * p.gz < nz) return bad("tiles do not cover the box");
    if (p.lw != (p.gx > 1 ? p.tx + 2 : nx)) return bad("local columns");
    if (p.threads > kResMaxThreads || p.threads % 64 || p.lw > p.threads) return bad("work-items");
    const int RS = p.threads / p.lw;
    if (RS * p.ns < GR) return bad("staged rows beyond the work-items");
    if (RS < p.ty * ((p.tz + p.cz - 1) / p.cz)) return bad("columns beyond the work-items");
    if (p.lds_bytes > kResMaxLds) return bad("LDS");
    if (p.tab.size() + p.tab_off.size() > resident_tab_ints(ny, nz)) return bad("table space");
    std::vector<std::vector<int>> nb((size_t)nyz);
    std::vector<char> exported((size_t)(ny * nz), 0);
    for (int t = 0; t < nyz; ++t) {
        const int *v = p.tab.data() + p.tab_off[(size_t)t];
        for (int y = 0; y < p.ty && (t % p.gy) * p.ty + y < ny; ++y)
            for (int z = 0; z < p.tz && (t / p.gy) * p.tz + z < nz; ++z)
                exported[(size_t)((t % p.gy) * p.ty + y + ny * ((t / p.gy) * p.tz + z))] = (char)v[v[kResOExp] + y + p.ty * z];
        nb[(size_t)t].assign(v + v[kResONb], v + v[kResONb] + v[kResNNb]);
        if ((p.gx > 1 ? 3 : 1) * v[kResNNb] > p.threads) return bad("more neighbours than work-items");
    }
    auto has = [](const std::vector<int> &l, int x) { return std::find(l.begin(), l.end(), x) != l.end(); };
    for (int t = 0; t < nyz; ++t) {
        const int *v = p.tab.data() + p.tab_off[(size_t)t];
        const int y0 = (t % p.gy) * p.ty, z0 = (t / p.gy) * p.tz;
        const int th = std::min(p.ty, ny - y0), tw = std::min(p.tz, nz - z0);
        for (int n : nb[(size_t)t])
            if (!has(nb[(size_t)n], t)) return bad("neighbour lists are not symmetric");
        std::vector<int> row_at((size_t)p.slots, -1);  // row of the box in every row of LDS
        for (int y = 0; y < th; ++y)
            for (int z = 0; z < tw; ++z) row_at[(size_t)(y + 1 + PY * (z + 1))] = y0 + y + ny * (z0 + z);
        for (int k = 0; k < v[kResNLoad]; ++k) {
            const int *e = v + v[kResOLoad] + 2 * k, slot = e[0] / (3 * p.lw), row = e[1] / nx;
            if (e[0] % (3 * p.lw) || slot < 0 || slot >= p.slots || e[1] % nx || row < 0 || row >= ny * nz) return bad("row read");
            if (row_at[(size_t)slot] >= 0) return bad("two rows in one place");
            row_at[(size_t)slot] = row;
            if (!exported[(size_t)row]) return bad("a row read is not written");
            const int own = (row % ny) / p.ty + p.gy * ((row / ny) / p.tz);
            if (!has(nb[(size_t)t], own)) return bad("a row is read without a wait for its tile");
        }
        for (int hz = 0; hz < tw + 2; ++hz)
            for (int hy = 0; hy < th + 2; ++hy)
                if (row_at[(size_t)(hy + PY * hz)] != (y0 - 1 + hy + ny) % ny + ny * ((z0 - 1 + hz + nz) % nz)) return bad("halo row");
        if (v[kResNMk] > p.mk_max) return bad("markers beyond their space");
        std::vector<int> line((size_t)std::max(v[kResNMk], 1), -1);
        for (int m = 0; m < v[kResNMk]; ++m) {
            const int *e = v + v[kResOMk] + m * kResMkInts, l = e[kResTaps];
            line[(size_t)m] = l;
            for (int i = 0; i < w.tm; ++i)
                if (row_at[(size_t)(e[i] / (3 * p.lw))] != w.tap_row[(size_t)(l * w.tm + i)]) return bad("tap row not in LDS");
        }
        int corrected = 0;
        for (int r : w.band_row)
            for (int hz = 0; hz < tw + 2; ++hz)
                for (int hy = 0; hy < th + 2; ++hy) corrected += row_at[(size_t)(hy + PY * hz)] == r;
        if (corrected != v[kResNCor]) return bad("corrected rows");
        for (int k = 0; k < v[kResNCor]; ++k) {
            const int *e = v + v[kResOCor] + k * (2 * p.km4 + 4);
            const int row = row_at[(size_t)(e[2 * p.km4] / (3 * p.lw))];
            const auto at = std::find(w.band_row.begin(), w.band_row.end(), row);
            if (at == w.band_row.end()) return bad("corrected row");
            const size_t r = (size_t)(at - w.band_row.begin());
            for (int q = 0; q < w.km; ++q)
                if (line[(size_t)(e[q] / (3 * p.lw))] != w.band_line[r * w.km + q]) return bad("line of a correction");
        }
    }
    return "";
}

template <bool Q27>
void reference(const ResArgs &a, const ResWall &w, std::vector<float> &b) {
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const size_t N = (size_t)nx * ny * nz;
    const SweepWeights W = sweep_weights<Q27>(a.kappa, a.omega);
    std::vector<float> f(3 * N), out(3 * N);
    for (int it = 0; it < a.n_mag; ++it) {
        for (size_t k = 0; k < N; ++k) {
            const size_t row = k / nx, yz = (size_t)ny * nz;
            float e[3];
            for (int c = 0; c < 3; ++c) {
                e[c] = a.bext[c * nx + k % nx];
                if (a.bext_yz) e[c] += a.bext_yz[c * yz + row];
            }
            sweep_flux(b[k] + e[0], b[N + k] + e[1], b[2 * N + k] + e[2], a.u[k], a.u[N + k], a.u[2 * N + k], f[k], f[N + k], f[2 * N + k]);
        }
        for (int z = 0; z < nz; ++z)
            for (int y = 0; y < ny; ++y)
                for (int x = 0; x < nx; ++x) {
                    March<1> march;
                    float o[1][3];
                    for (int p = -1; p <= 1; ++p) {
                        auto rows = [&](int k, float (&v)[3][3]) {
                            for (int r = 0; r < 3; ++r)
                                for (int j = 0; j < 3; ++j) {
                                    const size_t q = (size_t)((x + j - 1 + nx) % nx) +
                                                     (size_t)nx * ((y + r - 1 + ny) % ny + (size_t)ny * ((z + p + nz) % nz));
                                    v[r][j] = k < 3 ? b[k * N + q] : f[(k - 3) * N + q];
                                }
                        };
                        float S[1][3], B[1][3], P[1][2], cen[1][3];
                        plane_terms<1, Q27>(columns_rows<1>(rows), W, S, B, P, cen);
                        march.take(W, S, B, P, cen, o);
                    }
                    for (int c = 0; c < 3; ++c) out[c * N + x + (size_t)nx * (y + (size_t)ny * z)] = o[0][c];
                }
        b = out;
        const size_t lines = w.tap_row.size() / (size_t)w.tm;
        for (int c = 0; c < 3; ++c)
            for (int x = 0; x < nx; ++x) {
                std::vector<float> d(lines);
                for (size_t l = 0; l < lines; ++l) {
                    float I = 0.0f;
                    for (int t = 0; t < w.tm; ++t) I = fmaf(w.tap_w[l * w.tm + t], b[c * N + x + (size_t)nx * w.tap_row[l * w.tm + t]], I);
                    d[l] = a.sj[l * nx + x] * (a.wall[c * a.M + l * nx + x] - I);
                }
                for (size_t r = 0; r < w.band_row.size(); ++r) {
                    float s = 0.0f;
                    for (int q = 0; q < w.km; ++q) s = fmaf(w.band_w[r * w.km + q], d[(size_t)w.band_line[r * w.km + q]], s);
                    float &v = b[c * N + x + (size_t)nx * w.band_row[r]];
                    v = v + s;
                }
            }
    }
}

int main(int argc, char **argv) {
    if (argc == 2) {  // a file of boxes, one a line: nx ny nz radius max_wg; checks their plans only
        FILE *f = fopen(argv[1], "r");
        int nx, ny, nz, wg;
        double R;
        while (f && fscanf(f, "%d %d %d %lf %d", &nx, &ny, &nz, &R, &wg) == 5) {
            const ResWall w = ring_wall(ny, nz, R);
            const ResPlan p = make_resident_plan(nx, ny, nz, w, wg);
            const std::string e = p.ok ? check_plan(p, nx, ny, nz, w, wg) : "";
            printf("%d %d %d %g planned %d lw %d short %d sweeps %d %s\n", nx, ny, nz, R, p.ok, p.lw, p.gx > 1 && nx % p.tx != 0,
                   p.ok ? resident_min_sweeps(p, nx, ny, nz, R > 0) : 0, e.empty() ? "ok" : e.c_str());
        }
        return 0;
    }
    if (argc != 12) return 2;
    const int nx = atoi(argv[1]), ny = atoi(argv[2]), nz = atoi(argv[3]);
    const double R = atof(argv[4]);
    const int n_mag = atoi(argv[5]);
    const bool q27 = atoi(argv[6]) == 27;
    const float omega = (float)(1.0 / atof(argv[7]));
    const bool magnets = atoi(argv[8]) != 0;
    const int max_wg = atoi(argv[9]), mode = atoi(argv[10]);
    emu::workers = atoi(argv[11]);
    const ResWall w = ring_wall(ny, nz, R);
    ResPlan p = make_resident_plan(nx, ny, nz, w, max_wg);
    printf("planned %d tiles %d x %d x %d of %d x %d x %d lw %d short %d threads %d ns %d cz %d ", p.ok, p.gx, p.gy, p.gz, p.tx, p.ty, p.tz,
           p.lw, p.gx > 1 && nx % p.tx != 0, p.threads, p.ns, p.cz);
    if (!p.ok) return puts("no plan"), 0;
    const std::string e = check_plan(p, nx, ny, nz, w, max_wg);
    if (!e.empty()) return puts(e.c_str()), 0;

    const size_t N = (size_t)nx * ny * nz, lines = w.tap_row.size() / (size_t)w.tm;
    unsigned state = 12345;
    auto rnd = [&] {
        state = state * 1664525u + 1013904223u;
        return (float)(state >> 8) / (1 << 24) - 0.5f;
    };
    std::vector<float> u(3 * N), b0(3 * N), b1(3 * N), bext(3 * (size_t)nx), byz(3 * (size_t)ny * nz), sj(lines * nx), wall(3 * lines * nx);
    for (auto *v : {&u, &b0, &b1, &bext, &byz, &sj, &wall})
        for (float &x : *v) x = 0.1f * rnd();
    std::vector<int> sync(kResSyncInts, 0);
    int32_t stalled = 0;
    ResArgs a{};
    a.u = u.data();
    a.b[0] = b0.data();
    a.b[1] = b1.data();
    a.bext = bext.data();
    a.bext_yz = magnets ? byz.data() : nullptr;
    a.sj = sj.data();
    a.wall = wall.data();
    a.M = (int64_t)lines * nx;
    a.km4 = p.km4;
    a.nx = nx;
    a.ny = ny;
    a.nz = nz;
    a.tx = p.tx;
    a.ty = p.ty;
    a.tz = p.tz;
    a.gx = p.gx;
    a.gy = p.gy;
    a.nwg = p.nwg;
    a.lw = p.lw;
    a.slots = p.slots;
    a.mk_max = p.mk_max;
    a.n_mag = n_mag;
    a.kappa = 0.4f;
    a.omega = omega;
    a.tab = p.tab.data();
    a.tab_off = p.tab_off.data();
    a.sync = sync.data();
    a.stalled = &stalled;
    a.roll_ticks = mode == 2 || mode == 3 ? -1 : 1000000000ll;
    int host[2] = {0, 0};
    a.record = mode != 2;
    a.host = host;
    if (mode == 5) sync[kResState] = kResHeld, sync[kResHold] = 7;
    if (mode == 4) {  // as after a roll call that all but one workgroup left: its waits end all the same
        sync[kResState] = kResGo;
        emu::workers = 1;
        emu::fast_clock = true;
    }
    std::vector<float> want = b0;
    if (q27)
        reference<true>(a, w, want);
    else
        reference<false>(a, w, want);
    if (launch_mag_resident(nullptr, a, p, q27) != hipSuccess) return puts("launch"), 0;
    const std::vector<float> &got = n_mag & 1 ? b0 : b1;
    size_t differ = 0;
    for (size_t i = 0; i < 3 * N; ++i) differ += memcmp(&want[i], &got[i], 4) != 0;
    if (stalled) return puts("stalled"), 0;
    if (differ) return printf("%zu values differ\n", differ), 0;
    const int given_up = mode == 3, stood_in = mode == 2 || mode == 3 || mode == 5, hold = mode == 3 ? kResHoldSteps : mode == 5 ? 7 : 0;
    if (sync[kResGiveUps] != given_up || host[0] != given_up || sync[kResStandIns] != stood_in || host[1] != stood_in ||
        sync[kResHold] != hold)
        return printf("given up %d %d stood in %d %d hold %d\n", sync[kResGiveUps], host[0], sync[kResStandIns], host[1], sync[kResHold]), 0;
    return puts("ok"), 0;
}
