"""The tests of sweep tiles, wall tables and graphs whose boxes are small enough for the resident
iteration, with MHD_RESIDENT=0: the kernels that they name are then the ones that run (the paired and
8-row sweeps, the line and the general wall tables, a graph's new tiles)."""
import inspect


import pytest

import tests.test_gpu_graph as G
import tests.test_gpu_parity as P
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def launch_sequence(monkeypatch):
    monkeypatch.setenv("MHD_RESIDENT", "0")


@pytest.mark.parametrize("bext", [W.BEXT_TANH_FRINGE_Y, W.BEXT_SIX_MAGNETS])
@pytest.mark.parametrize("test", [P.test_paired_tiles_agree_bitwise_on_a_128_wide_box, P.test_paired_tiles_agree_bitwise_on_a_256_wide_box])
def test_paired_tiles(test, bext):
    test(bext)


@pytest.mark.parametrize("case", P.LINE_CASES)
def test_line_wall_tables(case, monkeypatch):
    P.test_line_wall_tables_equal_the_general_tables_bitwise(case, monkeypatch)


@pytest.mark.parametrize("shape,markers", [((37, 21, 13), False), ((128, 13, 9), False), ((8, 32, 32), True)])
def test_d3q27(shape, markers):
    P.test_d3q27_one_step(shape, markers)


@pytest.mark.parametrize("shape", [(37, 21, 13), (8, 32, 32), (16, 16, 9), (32, 11, 17), (64, 8, 5), (100, 12, 10), (1, 24, 1),
                                   (130, 5, 3), (128, 13, 9), (256, 6, 5), (128, 1, 3), (1, 1, 1), (2, 3, 1)])
def test_one_step_ragged_shapes(shape):
    P.test_one_step_no_wall_ragged_shapes(shape)


@pytest.mark.parametrize("nx,steps,n_mag", [(8, 1, 4), (128, 1, 4), (8, 10, 20)])
def test_six_magnets(nx, steps, n_mag):
    P.test_six_magnet_field(nx, steps, n_mag)


@pytest.mark.parametrize("test", [P.test_small_pipe_10_steps_full_sweeps, P.test_quarter_fringe_pipe_20_steps, P.test_dense_marker_cloud,
                                  P.test_markers_across_box_faces])
def test_pipes_and_walls(test):
    assert not inspect.signature(test).parameters
    test()


def test_graph_replay():
    G.test_graph_replay_equals_direct_launches({})


def test_the_8_row_sweep_agrees_with_the_other_tiles_on_ragged_rows():
    """128- and 256-wide boxes of odd cross-sections, D3Q27 among them: 8-row tiles (k_sweep_rows), 4-row
    tiles and single-cell tiles, with chunks shorter and longer than n_z: the same bits."""
    from paper_2211_09370_amd import Sim
    import numpy as np

    for nx, ny, nz, lattice in ((128, 11, 7, 19), (128, 17, 9, 27), (256, 9, 19, 19), (256, 13, 5, 27)):
        w = P.random_box(nx, ny, nz, key=430 + ny, n_mag=3)
        ref = None
        for tiles in ((64, 8, 1, 8), (64, 128, 1, 8), (64, 2, 1, 8), (64, 1, 1, 8), (64, 8, 1, 4), (64, 4, 0, 4), (16, 8, 0, 4)):
            print("case rows", nx, ny, nz, lattice, tiles, flush=True)
            s = Sim(nx, ny, nz, w.markers.shape[1])
            s.set_markers(w.markers)
            s.set_params(w.params, lattice=lattice)
            for f in ("rho", "u", "b"):
                s.set_field(f, getattr(w, f))
            s.tiles = tiles
            s.step(2)
            assert not s.iteration_info()["planned"]
            got = [s.get_field(f) for f in ("rho", "u", "b")]
            s.close()
            if ref is None:
                ref = got
            assert all(np.array_equal(x, y) for x, y in zip(got, ref)), (nx, ny, nz, lattice, tiles)


@pytest.mark.parametrize("lattice", [19, 27])
@pytest.mark.parametrize("magnets", [False, True])
@pytest.mark.parametrize("nx,ny,nz,tiles", [
    (70, 30, 50, ((64, 8, 0, 4), (64, 1, 0, 4))),           # 112 and 800 workgroups: the forms for few and for many
    (30, 40, 160, ((32, 8, 0, 4), (32, 1, 0, 4))),          # 100 and 800
    (14, 33, 270, ((16, 8, 0, 4), (16, 1, 0, 4))),          # 102 and 810
    (7, 33, 400, ((8, 8, 0, 4), (8, 1, 0, 4))),             # 100 and 800
    (256, 21, 72, ((64, 8, 1, 4), (64, 1, 1, 4), (64, 2, 1, 4), (64, 72, 1, 4))),  # pairs: 108, 864, 432 and 12
    (256, 21, 55, ((64, 1, 1, 4), (64, 8, 1, 4), (64, 8, 0, 4))),                   # 660
])
def test_forms_for_few_and_for_many_workgroups_agree(nx, ny, nz, tiles, magnets, lattice):
    from paper_2211_09370_amd import Sim
    import numpy as np

    print("case few and many", nx, ny, nz, magnets, lattice, flush=True)
    if magnets:
        w = W.pipe_workload("few", 440, nx, ny, nz, 8.0, 50.0, 10.0, 1e-2, bext_kind=W.BEXT_SIX_MAGNETS, n_mag=3, b_amp=1e-3, noise=1e-2)
    else:
        w = P.random_box(nx, ny, nz, key=441, n_mag=3)
    ref = None
    for t in tiles:
        s = Sim(nx, ny, nz, w.markers.shape[1])
        s.set_markers(w.markers)
        s.set_params(w.params, lattice=lattice)
        for f in ("rho", "u", "b"):
            s.set_field(f, getattr(w, f))
        s.tiles = t
        s.step(2)
        got = [s.get_field(f) for f in ("rho", "u", "b")]
        s.close()
        ref = ref or got
        assert all(np.array_equal(x, y) for x, y in zip(got, ref)), t
