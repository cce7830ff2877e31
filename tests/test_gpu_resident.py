"""The resident magnetic iteration (all sweeps of a step and their wall corrections in one launch)
against the launch sequence of a sweep, an interpolation and a spreading per iteration: the same
fields bit for bit. MHD_RESIDENT at mhd_set_params selects the form: 0 = launch sequence, 1 = resident
where the box fits, 2 = its stand-in, which a launch whose workgroups do not all
become resident leaves the work to (roll call given up by the first workgroup)."""
import threading

import numpy as np
import pytest

import workloads as W
from tests.test_gpu_parity import TOL, compare, oracle_run, random_box

pytestmark = pytest.mark.gpu


def box(case):
    """(workload, parameter overrides, use the wall)"""
    if case == "pipe_walls":  # nonzero wall values, odd count
        return W.small_pipe(rho_amp=1e-3, b_amp=1e-3, n_mag=5), {}, True
    if case == "cube_even":
        return random_box(32, 32, 32, key=400, n_mag=4, R=13.0), {}, True
    if case == "ragged_tiles":  # tiles that do not divide the cross-section, a box shorter than a wave
        return random_box(5, 47, 53, key=401, n_mag=3, R=20.0), {}, True
    if case == "one_sweep":
        return random_box(37, 21, 13, key=402, n_mag=1, R=5.0), {}, True
    if case == "no_wall":
        return random_box(9, 14, 30, key=403, n_mag=4), {}, False
    if case == "one_cell_wide":  # every halo row wraps onto the tile itself
        return random_box(1, 24, 1, key=404, n_mag=3), {}, False
    if case == "six_magnets":
        return W.pipe_workload("six", 405, 16, 33, 33, 14.0, 50.0, 10.0, 1e-2, bext_kind=W.BEXT_SIX_MAGNETS, n_mag=4,
                               b_amp=1e-3, noise=1e-2), {}, True
    if case == "q27_accelerated":
        return random_box(20, 26, 22, key=406, n_mag=4, R=8.0), dict(lattice=27, alpha=0.5), True
    if case == "long_rows":  # several staged rows and a tall column per work-item
        return random_box(100, 40, 44, key=407, n_mag=3, R=15.0), {}, True
    if case == "x_tiles":  # rows cut into tiles with halo columns, the last one shorter
        return random_box(203, 26, 30, key=410, n_mag=4, R=9.0), {}, True
    if case == "x_tiles_magnets_q27":
        return W.pipe_workload("six_x", 411, 150, 29, 29, 12.0, 50.0, 10.0, 1e-2, bext_kind=W.BEXT_SIX_MAGNETS, n_mag=3,
                               b_amp=1e-3, noise=1e-2), dict(lattice=27), True
    if case == "two_x_tiles_no_wall":  # the same tile on both sides in x
        return random_box(64, 53, 53, key=412, n_mag=3), {}, False
    if case == "tall_columns":  # six planes a work-item
        return random_box(40, 157, 157, key=414, n_mag=2), {}, False
    if case == "largest":  # close to what a workgroup's LDS holds
        return random_box(192, 70, 70, key=413, n_mag=2, R=33.0), {}, True
    if case == "pair_width":  # n_x = 128: the launch sequence is the paired sweep
        return random_box(128, 20, 22, key=408, n_mag=3, R=7.0), {}, True
    if case == "wall_through_the_faces":  # markers whose taps wrap around the box
        w = random_box(12, 24, 24, key=409, n_mag=3, R=11.9)
        return w, {}, True
    raise KeyError(case)


CASES = ("pipe_walls", "cube_even", "ragged_tiles", "one_sweep", "no_wall", "one_cell_wide", "six_magnets",
         "q27_accelerated", "long_rows", "pair_width", "wall_through_the_faces", "x_tiles", "x_tiles_magnets_q27",
         "two_x_tiles_no_wall", "tall_columns", "largest")


def make(w, over, wall, mode, monkeypatch):
    from paper_2211_09370_amd import Sim

    monkeypatch.setenv("MHD_RESIDENT", mode)
    M = w.markers.shape[1] if wall else 0
    sim = Sim(w.nx, w.ny, w.nz, M)
    if M:
        g = np.random.default_rng(77)
        sim.set_markers(w.markers, u_wall=g.uniform(-1e-4, 1e-4, (3, M)), b_wall=g.uniform(-1e-4, 1e-4, (3, M)))
    sim.set_params(w.params, **over)
    for f in ("rho", "u", "b"):
        sim.set_field(f, getattr(w, f))
    return sim


@pytest.mark.parametrize("case", CASES)
def test_resident_equals_the_launch_sequence_bitwise(case, monkeypatch):
    print("case resident", case, flush=True)
    w, over, wall = box(case)
    out = {}
    for mode in ("0", "1", "2"):
        sim = make(w, over, wall, mode, monkeypatch)
        sim.step(3)  # captured and replayed
        sim.set_graph(False)
        sim.step(1)
        sim.step_noalloc(1)
        out[mode] = [sim.get_field(f) for f in ("rho", "u", "b")]
        sim.close()
    for mode in ("1", "2"):
        for f, x, y in zip(("rho", "u", "b"), out["0"], out[mode]):
            assert np.array_equal(x, y), (case, mode, f, float(np.abs(x - y).max()))


def test_resident_matches_the_oracle(monkeypatch):
    print("case resident oracle", flush=True)
    w = W.quarter_fringe_pipe(n_mag=24)
    from paper_2211_09370_amd import Sim

    sim = Sim(w.nx, w.ny, w.nz, w.markers.shape[1])
    sim.set_markers(w.markers)
    sim.set_params(w.params)
    for f in ("rho", "u", "b"):
        sim.set_field(f, getattr(w, f))
    sim.step(4)
    compare(sim, oracle_run(w, 4), tol=TOL, label="resident")
    sim.close()


def test_resident_boxes_on_several_streams_and_threads(monkeypatch):
    """Four boxes whose workgroups would not fit the chip together, each stepped by a thread of its
    own on its own stream, then all from one thread in turn: the fields of each equal those of a
    box stepped alone."""
    print("case resident threads", flush=True)
    w, over, wall = box("ragged_tiles")
    ref = make(w, over, wall, "0", monkeypatch)
    ref.step(44)
    want = [ref.get_field(f) for f in ("rho", "u", "b")]
    ref.close()
    sims = [make(w, over, wall, "1", monkeypatch) for _ in range(4)]
    threads = [threading.Thread(target=lambda s=s: [s.step(4) for _ in range(10)]) for s in sims]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for s in sims:
        s.step(4)
    for s in sims:
        assert all(np.array_equal(s.get_field(f), x) for f, x in zip(("rho", "u", "b"), want))
        s.close()


def test_new_markers_and_parameters_between_steps(monkeypatch):
    """The plan follows the wall: markers replaced, then removed, between steps."""
    print("case resident replan", flush=True)
    w, over, wall = box("cube_even")
    other = W.pipe_markers(32, 9.0, 16.0, 16.0)
    out = []
    for mode in ("0", "1"):
        sim = make(w, over, wall, mode, monkeypatch)
        sim.step(2)
        sim.set_markers(other)
        sim.step(1)
        sim.set_params(w.params, n_mag=7)
        sim.step(1)
        sim.set_markers(np.zeros((3, 0)))
        sim.step(1)
        out.append([sim.get_field(f) for f in ("rho", "u", "b")])
        sim.close()
    assert all(np.array_equal(x, y) for x, y in zip(*out))


def test_few_sweeps_are_launched_one_by_one(monkeypatch):
    """n_mag below what makes the resident launch the faster form, at it, and changed between steps."""
    print("case resident few sweeps", flush=True)
    w = random_box(192, 70, 70, key=413, n_mag=1, R=33.0)
    out = []
    for mode in ("0", "1"):
        sim = make(w, {}, True, mode, monkeypatch)
        for n_mag in (1, 3, 5, 2):
            sim.set_params(w.params, n_mag=n_mag)
            sim.step(1)
            assert sim.iteration_info()["planned"] == (mode == "1" and n_mag == 5), (mode, n_mag)
        assert sim.iteration_info()["steps"] == (1 if mode == "1" else 0)
        out.append([sim.get_field(f) for f in ("rho", "u", "b")])
        sim.close()
    assert all(np.array_equal(x, y) for x, y in zip(*out))


@pytest.mark.parametrize("case", ["131x57x57", "400x42x42", "163x53x53", "497x31x31", "131x43x43 six magnets q27"])
def test_wide_x_tiles_with_a_shorter_last_one(case, monkeypatch):
    """Tiles of more columns than a wave, the last one shorter, so that waves with and without idle
    columns share a workgroup (the CPU tests check that these boxes are cut so): the same fields in
    every form."""
    print("case resident wide", case, flush=True)
    shape, *rest = case.split(" ")
    nx, ny, nz = (int(v) for v in shape.split("x"))
    R = {57: 25.0, 42: 18.0, 53: 24.0, 31: 13.0, 43: 18.0}[ny]
    if rest:
        w = W.pipe_workload("six_wide", 416, nx, ny, nz, R, 50.0, 10.0, 1e-2, bext_kind=W.BEXT_SIX_MAGNETS, n_mag=3, b_amp=1e-3,
                            noise=1e-2)
        over = dict(lattice=27)
    else:
        w, over = random_box(nx, ny, nz, key=415, n_mag=3, R=R), {}
    out = {}
    for mode in ("0", "4", "2"):
        sim = make(w, over, True, mode, monkeypatch)
        sim.step(2)
        out[mode] = [sim.get_field(f) for f in ("rho", "u", "b")]
        info = sim.iteration_info()
        assert info["steps"] == (0 if mode == "0" else 2) and (mode == "0" or 62 < info["tile"][0] and nx % info["tile"][0]), info
        sim.close()
    for mode in ("4", "2"):
        for f, x, y in zip(("rho", "u", "b"), out["0"], out[mode]):
            assert np.array_equal(x, y), (case, mode, f, float(np.abs(x - y).max()))


def test_roll_calls_given_up(monkeypatch):
    """Every resident launch finds the GPU busy: the stand-in takes over, the steps already launched go to
    it as well, later calls launch their sweeps one by one and then try again. The same fields."""
    print("case resident given up", flush=True)
    w, over, wall = box("x_tiles")
    out = []
    for mode in ("0", "3"):
        sim = make(w, over, wall, mode, monkeypatch)
        for n in (3, 40, 1, 64, 2):
            sim.step(n)
        sim.step_noalloc(2)
        out.append([sim.get_field(f) for f in ("rho", "u", "b")])
        sim.close()
    assert all(np.array_equal(x, y) for x, y in zip(*out))


@pytest.mark.parametrize("case", CASES)
def test_the_forms_compared_are_the_forms_that_ran(case, monkeypatch):
    """mode 0 has no plan; in mode 4 every step is resident, whatever the number of sweeps, and its roll
    call ends in "go"; in mode 2 every step is done by the stand-in. The same fields."""
    print("case resident forms", case, flush=True)
    w, over, wall = box(case)
    ref = None
    for mode in ("0", "4", "2"):
        sim = make(w, over, wall, mode, monkeypatch)
        sim.step(3)
        sim.set_graph(False)
        sim.step(1)
        sim.step_noalloc(1)
        got = [sim.get_field(f) for f in ("rho", "u", "b")]
        ref = ref or got
        assert all(np.array_equal(x, y) for x, y in zip(ref, got)), (case, mode)
        info = sim.iteration_info()
        want = {"0": (False, 0, 0, 0), "4": (True, 5, 0, 0), "2": (True, 5, 0, 5)}[mode]
        assert (info["planned"], info["steps"], info["given_up"], info["stand_in"]) == want, (case, mode, info)
        if mode != "0" and case.startswith("x_tiles"):
            assert info["tile"][0] < w.nx, info
        sim.close()


def test_steps_keep_away_from_a_busy_gpu_for_a_while(monkeypatch):
    """A roll call given up: the other steps of its call are done by the stand-in without one, the next
    calls launch their sweeps one by one, and then the resident launch is tried again."""
    print("case resident keeps away", flush=True)
    w, over, wall = box("cube_even")
    sim = make(w, over, wall, "3", monkeypatch)
    def after(n):
        sim.step(n)
        sim.get_field("b")
        info = sim.iteration_info()
        return info["steps"], info["given_up"], info["stand_in"]
    assert after(3) == (3, 1, 3)
    assert after(10) == (3, 1, 3)
    assert after(54) == (3, 1, 3)
    assert after(1) == (4, 2, 4)
    assert after(128) == (4, 2, 4)
    assert after(1) == (5, 3, 5)
    sim.close()
    from paper_2211_09370_amd import Sim
    sim = Sim(128, 128, 128, 0)  # beyond the LDS
    sim.set_params(w.params)
    sim.step(1)
    assert not sim.iteration_info()["planned"] and sim.iteration_info()["steps"] == 0
    sim.close()
