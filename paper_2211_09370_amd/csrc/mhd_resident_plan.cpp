// Host side of the resident magnetic iteration: tiles of the cross-section, the rows, markers and
// neighbours of each tile, and the launch shape (mhd_resident.hip describes the kernel).
#include <algorithm>
#include <climits>
#include <cstring>
#include <set>

#include "mhd_resident.h"

namespace mhd {

namespace {

int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Launch shape for tiles of ty x tz rows: the column height (CZ planes; each column also takes the two
// planes around it) that costs least. A plane of a column measured about 660 ns of latency and 23 ns
// for every wave of the workgroup's columns. The workgroup is as large as the rows read and staged
// can use.
bool launch_shape(int lw, int ty, int tz, ResPlan &p, long &cost) {
    const int gr = (ty + 2) * (tz + 2);
    const int forms[5][2] = {{1, 1}, {2, 1}, {6, 2}, {6, 4}, {6, 6}};
    long best = -1;
    for (const auto &f : forms) {
        const int ns = f[0], cz = f[1], cols = lw * ty * ceil_div(tz, cz);
        int nt = std::max({lw * ceil_div(gr, ns), cols, 64});
        nt = ceil_div(nt, 64) * 64;
        if (nt > kResMaxThreads) continue;
        const long t = (long)(cz + 2) * (660 + 23L * ceil_div(cols, 64));
        if (best < 0 || t < best) {
            best = t;
            p.ns = ns;
            p.cz = cz;
            // a round of rows read from memory costs more than the barriers of a larger workgroup
            p.threads = std::max(nt, std::min(kResMaxThreads, ceil_div(lw * ceil_div(gr, 2), 64) * 64));
        }
    }
    cost = best;
    return best >= 0;
}

bool build(int nx, int ny, int nz, const ResWall &w, ResPlan &p) {
    const int ty = p.ty, tz = p.tz, lw = p.lw, PY = ty + 2, GR = PY * (tz + 2), nrows = ny * nz;
    const int nyz = p.gy * p.gz;
    auto owner = [&](int row) { return (row % ny) / ty + p.gy * ((row / ny) / tz); };
    std::vector<int> band((size_t)nrows, -1);
    for (size_t r = 0; r < w.band_row.size(); ++r) band[(size_t)w.band_row[r]] = (int)r;
    std::vector<char> exported((size_t)nrows, 0);
    std::vector<std::set<int>> nb((size_t)nyz);
    struct Tile {
        std::vector<int> load, mk, cor;
        int n_mk = 0, n_cor = 0;
    };
    std::vector<Tile> tiles((size_t)nyz);
    std::vector<int> slot_of((size_t)nrows), mk_of(w.tap_row.size() / (size_t)w.tm);
    p.slots = GR;
    p.mk_max = 0;
    p.km4 = (w.km + 3) & ~3;
    if (w.tm > kResTaps) return false;
    for (int t = 0; t < nyz; ++t) {
        Tile &T = tiles[(size_t)t];
        const int y0 = (t % p.gy) * ty, z0 = (t / p.gy) * tz;
        const int th = std::min(ty, ny - y0), tw = std::min(tz, nz - z0);
        std::fill(slot_of.begin(), slot_of.end(), -1);
        std::fill(mk_of.begin(), mk_of.end(), -1);
        auto row_at = [&](int hy, int hz) {
            return (y0 - 1 + hy + ny) % ny + ny * ((z0 - 1 + hz + nz) % nz);
        };
        for (int hz = 1; hz <= tw; ++hz)  // the tile's own rows first: their b* is in LDS
            for (int hy = 1; hy <= th; ++hy) slot_of[(size_t)row_at(hy, hz)] = hy + PY * hz;
        std::vector<std::pair<int, int>> load;  // (slot, row)
        for (int hz = 0; hz < tw + 2; ++hz)
            for (int hy = 0; hy < th + 2; ++hy) {
                if (hy >= 1 && hy <= th && hz >= 1 && hz <= tw) continue;
                const int row = row_at(hy, hz);
                load.push_back({hy + PY * hz, row});
                if (slot_of[(size_t)row] < 0) slot_of[(size_t)row] = hy + PY * hz;
            }
        int extra = GR;
        for (int hz = 0; hz < tw + 2; ++hz)
            for (int hy = 0; hy < th + 2; ++hy) {
                const int r = band[(size_t)row_at(hy, hz)];
                if (r < 0) continue;
                std::vector<int> line((size_t)p.km4), wt((size_t)p.km4, 0);
                for (int q = 0; q < p.km4; ++q) {  // padding: the first line with weight 0
                    const int k = q < w.km ? q : 0, l = w.band_line[(size_t)r * w.km + k];
                    if (mk_of[(size_t)l] < 0) {
                        mk_of[(size_t)l] = T.n_mk++;
                        std::vector<int> e((size_t)kResMkInts, 0);
                        for (int i = 0; i < kResTaps; ++i) {
                            const int row = w.tap_row[(size_t)l * w.tm + (i < w.tm ? i : 0)];
                            if (slot_of[(size_t)row] < 0) {
                                slot_of[(size_t)row] = extra;
                                load.push_back({extra++, row});
                            }
                            e[(size_t)i] = 3 * lw * slot_of[(size_t)row];
                            if (i < w.tm) std::memcpy(&e[(size_t)(kResTaps + 1 + i)], &w.tap_w[(size_t)l * w.tm + i], 4);
                        }
                        e[kResTaps] = l;
                        T.mk.insert(T.mk.end(), e.begin(), e.end());
                    }
                    line[(size_t)q] = 3 * lw * mk_of[(size_t)l];
                    if (q < w.km) std::memcpy(&wt[(size_t)q], &w.band_w[(size_t)r * w.km + q], 4);
                }
                T.n_cor += 1;
                T.cor.insert(T.cor.end(), line.begin(), line.end());
                T.cor.insert(T.cor.end(), wt.begin(), wt.end());
                T.cor.insert(T.cor.end(), {3 * lw * (hy + PY * hz), 0, 0, 0});
            }
        nb[(size_t)t].insert(t);
        for (const auto &l : load) {
            T.load.push_back(3 * lw * l.first);
            T.load.push_back(nx * l.second);
            exported[(size_t)l.second] = 1;
            nb[(size_t)t].insert(owner(l.second));  // a reader and its source wait for each other
            nb[(size_t)owner(l.second)].insert(t);
        }
        p.slots = std::max(p.slots, extra);
        p.mk_max = std::max(p.mk_max, T.n_mk);
    }
    p.tab.clear();
    p.tab_off.assign(1, 0);
    size_t longest = 0, most_nb = 0;
    for (int t = 0; t < nyz; ++t) {
        const Tile &T = tiles[(size_t)t];
        const int y0 = (t % p.gy) * ty, z0 = (t / p.gy) * tz;
        std::vector<int> v(kResHeader, 0);
        auto put = [&](int at, const std::vector<int> &x) {
            v.resize((v.size() + 3) & ~size_t(3));  // 16-byte aligned lists
            v[(size_t)at] = (int)v.size();
            v.insert(v.end(), x.begin(), x.end());
        };
        v[kResNLoad] = (int)T.load.size() / 2;
        put(kResOLoad, T.load);
        v[kResNMk] = T.n_mk;
        put(kResOMk, T.mk);
        v[kResNCor] = T.n_cor;
        put(kResOCor, T.cor);
        v[kResNNb] = (int)nb[(size_t)t].size();
        put(kResONb, std::vector<int>(nb[(size_t)t].begin(), nb[(size_t)t].end()));
        std::vector<int> e((size_t)ty * tz, 0);
        for (int z = 0; z < std::min(tz, nz - z0); ++z)
            for (int y = 0; y < std::min(ty, ny - y0); ++y)
                e[(size_t)(y + ty * z)] = exported[(size_t)(y0 + y + ny * (z0 + z))];
        put(kResOExp, e);
        p.tab.insert(p.tab.end(), v.begin(), v.end());
        p.tab_off.push_back((int)p.tab.size());
        longest = std::max(longest, v.size());
        most_nb = std::max(most_nb, nb[(size_t)t].size());
    }
    p.lds_bytes = 4 * (3 * (size_t)(p.slots + std::max(GR, p.mk_max)) * lw + 3 * (size_t)GR + 3 + longest);
    return p.lds_bytes <= kResMaxLds && p.tab.size() + p.tab_off.size() <= resident_tab_ints(ny, nz) && 3 * (int)most_nb <= p.threads;
}

}  // namespace

ResPlan make_resident_plan(int nx, int ny, int nz, const ResWall &wall, int max_wg) {
    struct Cand {
        long cost;
        ResPlan p;
    };
    std::vector<Cand> cand;
    max_wg = std::min(max_wg, kResMaxTiles);
    // Tiles of at least 4 x 4 rows and 8 columns (or the whole box): smaller ones read more than they own.
    // The cost is an iteration's time in ns beyond what all forms share (1.4 us): the columns' time
    // (launch_shape), 1 ns for every staged cell and, cut along x, 700 ns (three times the neighbours)
    // and 9 ns for every row's end cells, which are written and read by themselves. It reproduced 36
    // measured forms of nine boxes (5 to 18.5 us an iteration, 1 to 28 tiles along x) within 4% rms.
    for (int gx = 1; gx <= std::max(1, nx / 8); ++gx)
        for (int ty = std::min(4, ny); ty <= std::min(ny, 24); ++ty)
            for (int tz = std::min(4, nz); tz <= std::min(nz, 24); ++tz) {
                Cand c;
                ResPlan &p = c.p;
                p.tx = ceil_div(nx, gx);
                p.gx = ceil_div(nx, p.tx);
                if (p.gx != gx) continue;
                p.lw = gx == 1 ? nx : p.tx + 2;
                p.ty = ty;
                p.tz = tz;
                p.gy = ceil_div(ny, ty);
                p.gz = ceil_div(nz, tz);
                const long nwg = (long)gx * p.gy * p.gz, staged = (long)(ty + 2) * (tz + 2) * p.lw;
                if (nwg > max_wg || 24 * staged > (long)kResMaxLds || staged > kResMaxStaged) continue;
                p.nwg = (int)nwg;
                if (!launch_shape(p.lw, ty, tz, p, c.cost)) continue;
                c.cost += staged + (gx > 1 ? 700 + 9L * (ty + 2) * (tz + 2) : 0);
                p.iter_ns = 1400 + c.cost;
                p.start_ns = 9500 + 22 * staged / 10;
                cand.push_back(c);
            }
    std::stable_sort(cand.begin(), cand.end(), [](const Cand &a, const Cand &b) {
        return a.cost != b.cost ? a.cost < b.cost : a.p.nwg < b.p.nwg;
    });
    for (size_t i = 0; i < cand.size() && i < 6; ++i) {
        ResPlan &p = cand[i].p;
        if (!build(nx, ny, nz, wall, p)) continue;
        p.ok = true;
        return p;
    }
    return ResPlan{};
}

// A step takes start_ns + n iter_ns here (without a wall, iter_ns less 1.7 us), beyond a step without
// sweeps, and otherwise n times the launches of a sweep and of a correction: a sweep 10.4 us on small
// boxes and 5 us more per million cells beyond 0.3 million, counting the tiles' empty places, the paired
// sweep 11.5 us on rows of 128 cells and 14.2 us on longer ones; a correction 4.6 us and 3.2 us more per
// million cells. D3Q27 adds about as much to both. Measured on 42 boxes of 4 k to 0.94 M cells, both
// lattices, with a wall and without: with a wall 192 x 70 x 70 breaks even at 3.8 sweeps (2 sweeps: 125 us
// a step here, 111 there), 100 x 75 x 75 at 1.9, 32^3 at 1; without one 32^3 at 1.6, 100 x 75 x 75 at
// 4.6, and 128 x 80 x 80 never (12.6 us a sweep against 11.8).
int resident_min_sweeps(const ResPlan &p, int nx, int ny, int nz, bool wall) {
    const double cells = (double)nx * ny * nz;
    const int tx = nx > 32 ? 64 : nx > 16 ? 32 : nx > 8 ? 16 : 8;  // tiles of the single-cell sweep
    const double places = (double)ceil_div(nx, tx) * tx * ny * nz;
    double seq = nx % 128 ? 10400 + 5e-3 * std::max(0.0, places - 3e5) : nx == 128 ? 11500 : 14200;
    if (wall) seq += 4600 + 3.2e-3 * cells;
    const double gain = seq - (double)(p.iter_ns - (wall ? 0 : 1700));
    return gain * 1e6 > (double)p.start_ns ? (int)((double)p.start_ns / gain) + 1 : INT_MAX;
}

}  // namespace mhd
