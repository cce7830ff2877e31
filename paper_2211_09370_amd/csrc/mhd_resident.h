// Resident magnetic iteration (mhd_resident.hip): plan, tile tables and launch arguments.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

namespace mhd {

constexpr int kResMaxThreads = 1024;
constexpr int kResMaxStaged = 6 * kResMaxThreads;  // staged cells (tile and halo) of a workgroup
constexpr int kResNoRow = 1 << 20;               // first row of a work-item that takes none
constexpr size_t kResMaxLds = 160 * 1024 - 256;  // LDS of a CU less the kernel's own words
constexpr int kResMaxTiles = 256;                // flags reserved in the workspace
// table words reserved in the workspace (a box whose tables need more has no resident iteration)
constexpr size_t resident_tab_ints(int ny, int nz) {
    const size_t rows = (size_t)ny * nz;
    return (rows < 9000 ? 40 * rows : 360000) + 4096;
}

// Words of the synchronisation area. Those below kResKept and the flags (64 bytes apart) are set anew by
// every step's first launch; the others last: steps left that take the stand-in without a roll call,
// roll calls given up, steps done by the stand-in.
enum { kResCount = 0, kResState = 1, kResStalled = 2, kResTicket = 3, kResKept = 8, kResHold = 8, kResGiveUps = 9, kResStandIns = 10 };
enum { kResFlags = 16, kResFlagStride = 16 };
enum { kResCounting = 0, kResGo = 1, kResGivenUp = 2, kResHeld = 3 };
constexpr int kResHoldSteps = 64;                // steps without a roll call after one was given up
constexpr size_t kResSyncInts = kResFlags + (size_t)kResFlagStride * kResMaxTiles;
constexpr long long kResRollTicks = 2000000;     // roll call: 20 ms of the 100 MHz clock
constexpr long long kResStallTicks = 1000000000; // a wait after it: 10 s

// The tables are per place in the cross-section: those of all x tiles there are the same.
// Header: counts and offsets (in words from the table's start). Places in LDS are
// given in words, ready to use: 3 lw times the local row or the marker's index.
enum {
    kResNLoad, kResOLoad,  // rows read each iteration: (place, first cell n_x (y + n_y z))
    kResNMk, kResOMk,      // markers' lines: places of 9 taps, line, 9 weights, padding
    kResNCor, kResOCor,    // corrected rows: places of km4 corrections, km4 weights, place of the row, padding
    kResNNb, kResONb,      // places in the cross-section (y tile + gy z tile) exchanged with, itself among them
    kResOExp,              // ty x tz words: 1 if another tile reads the row
    kResHeader = 12
};
constexpr int kResTaps = 9, kResMkInts = 20;  // taps of a line's marker, words of its entry

struct ResArgs {
    const float *u;
    float *b[2];           // b before the iteration, and the other buffer
    const float *bext, *bext_yz;
    const float *sj, *wall;
    int64_t M;
    int km4;
    int nx, ny, nz;
    int tx, ty, tz, gx, gy, nwg;  // tile, tiles in x and y, tiles
    int lw;                // local columns: n_x if gx = 1, else tx + 2
    int slots, mk_max;     // rows of b in LDS (tile, halo, extra), markers' lines of a tile at most
    int n_mag;
    float kappa, omega;
    const int *tab, *tab_off;
    int *sync;
    int32_t *stalled;      // DevCtrl::stalled
    long long roll_ticks;  // limit of the roll call; < 0: given up at once
    int record;            // 1: a roll call given up is remembered (kResHold, and host for the next calls)
    int *host;             // pinned: roll calls given up, steps done by the stand-in
};

// Tiles are tx columns of ty x tz rows: whole rows (gx = 1, periodic in the tile) or, where the box is
// longer than a workgroup can hold or more workgroups shorten the work, a part of them between two
// halo columns. Tile index = x tile + gx (y tile + gy z tile).
struct ResPlan {
    bool ok = false;
    int tx = 0, ty = 0, tz = 0, gx = 0, gy = 0, gz = 0, nwg = 0, lw = 0;
    int ns = 0, cz = 0, threads = 0;
    int slots = 0, mk_max = 0, km4 = 0;
    size_t lds_bytes = 0;
    long iter_ns = 0, start_ns = 0;  // estimates: an iteration; what a launch takes beyond its iterations
    std::vector<int> tab, tab_off;  // until uploaded
};

// A wall made of lines along x: each line's taps (rows y + ny z, weights; tm a line) and each band
// row's entries (km lines and weights, padding repeats the first line with weight 0).
struct ResWall {
    int tm = 1, km = 1;
    std::vector<int> tap_row, band_row, band_line;
    std::vector<float> tap_w, band_w;
};

// Tiles, tables and launch shape of a box for at most max_wg workgroups; ok = false if it does not fit.
ResPlan make_resident_plan(int nx, int ny, int nz, const ResWall &wall, int max_wg);

// Smallest number of sweeps a step for which plan p is faster than a launch a sweep and two a wall
// correction (INT_MAX: none).
int resident_min_sweeps(const ResPlan &p, int nx, int ny, int nz, bool wall);

// Readies the kernels of plan p on the current GPU (once, before launches).
hipError_t prepare_mag_resident(const ResPlan &p);
// The launches of one step's iteration; a.sync set by the step's first launch (launch_ctrl_begin).
hipError_t launch_mag_resident(hipStream_t s, const ResArgs &a, const ResPlan &p, bool q27);

}  // namespace mhd
