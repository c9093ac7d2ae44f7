"""The streaming passes of the predictor-corrector against the oracle, by their number: one
pass runs the last pass alone (populations), more put the passes that only sum the
moments of the next gauge before it.  Lattices ragged against the tiles and narrower than
the stencil, with a flow fast enough that the stencils of a workgroup do not agree.

Tolerances: FP64 repeats the oracle's sums in another order (1e-12, the parity bound of
the other FP64 tests), the FP32 forms have the bounds of their box tests: 1e-6 where only
the stored deviations are rounded, 1e-4 where the window arithmetic is too."""
import dataclasses
import functools

import numpy as np
import pytest

from paper_2002_09217_amd import pond, workloads as W
from tests.common import compare, pond_config, run_gpu, run_oracle, run_oracle3

pytestmark = pytest.mark.gpu

TOL = {pond.FP64: 1e-12, pond.FP32_STORE: 1e-4, pond.FP32_STORE_FP64_MATH: 1e-6}


def check(ref, got, fields, tol, name):
    errs = compare(got, ref, fields)
    print(name, {k: f"{v:.2e}" for k, v in errs.items()}, flush=True)
    assert all(v <= tol for v in errs.values()), f"{name}: {errs}"


@pytest.mark.parametrize("precision", list(TOL))
@pytest.mark.parametrize("n", [(17, 9, 5), (33, 8, 3), (3, 25, 2), (16, 8, 1)])
@pytest.mark.parametrize("n_pass", [1, 2, 3])
def test_passes_in_three_dimensions(n, n_pass, precision):
    print(f"3d {n} n_pass {n_pass} precision {precision}", flush=True)
    case = W.perturbed3(*n, seed=5, u0=(0.3, -0.47, 0.2), kappa=0.0176, n_pass=n_pass)
    check(run_oracle3(case, 4), run_gpu(case, 4, precision), ("rho", "ux", "uy", "uz", "E", "T", "p"), TOL[precision],
          case.name)


@functools.lru_cache(maxsize=None)
def cell(kappa):
    case = W.perturbed3(30, 11, 37, seed=8, u0=(0.2, -0.1, 0.3), kappa=kappa)
    return case, run_oracle3(case, 2)


@pytest.mark.parametrize("kappa", [0.0, 0.0176])
@pytest.mark.parametrize("copies", [(1, 1), (9, 15), (18, 20)])
def test_closure_in_chunks_of_planes(copies, kappa):
    """The closure of a box in blocks of 32 x 8 columns and chunks of 4, 6 and 16 planes (the
    larger the box the more), ragged in all three, against the oracle on the periodic cell that
    the box repeats."""
    kx, ky = copies
    print(f"closure of {kx} x {ky} cells, kappa {kappa}", flush=True)
    case, ref = cell(kappa)
    nx, ny, nz = case.n

    def tiled(f):
        return np.tile(np.asarray(f).reshape(nz, ny, nx), (1, ky, kx)).ravel()

    box = dataclasses.replace(case, n=(nx * kx, ny * ky, nz), rho=tiled(case.rho), T=tiled(case.T),
                              u=np.stack([tiled(c) for c in case.u]))
    got = run_gpu(box, 2, pond.FP64)
    keys = ("rho", "ux", "uy", "uz", "E", "T", "p")
    check({k: tiled(ref[k]) for k in keys}, got, keys, TOL[pond.FP64], case.name)


@functools.lru_cache(maxsize=None)
def shear(n_pass):
    """A sheared flow, subsonic in some rows and supersonic in others, with an inflow and an
    outflow face: 288 tiles of 16 x 16 or 32 x 8, more than one a compute unit (the kernels
    with one lane a receiver), ragged on both sides.  With the oracle's fields after 3 steps."""
    nx, ny = 275, 250
    case = W.perturbed(nx, ny, seed=21, rho0=1.0, t_over_tcr=1.4, kappa=0.0176, n_pass=n_pass, dt=0.2)
    case.u[0] = 0.4 + 0.8 * np.sin(2.0 * np.pi * np.arange(ny) / ny).repeat(nx)
    case.bc = ((W.INFLOW, W.OUTFLOW), (W.PERIODIC, W.PERIODIC))
    case.inflow = ((0, 0, (1.0, 0.4, 0.0, 1.4 * W.T_CR)),)
    return case, run_oracle(case, 3)


@pytest.mark.parametrize("precision", list(TOL))
@pytest.mark.parametrize("two_kernel", [0, 1])
@pytest.mark.parametrize("tile", [0, 5])
@pytest.mark.parametrize("n_pass", [1, 2, 3])
def test_passes_with_one_lane_a_receiver(n_pass, tile, two_kernel, precision):
    print(f"2d n_pass {n_pass} tile {tile} two_kernel {two_kernel} precision {precision}", flush=True)
    case, ref = shear(n_pass)
    got = run_gpu(case, 3, precision, tile=tile, two_kernel=two_kernel)
    check(ref, got, ("rho", "ux", "uy", "E", "T", "p"), TOL[precision], case.name)


@pytest.mark.parametrize("precision", [pond.FP64, pond.FP32_STORE])
def test_batch_mixes_lanes_a_receiver(precision):
    """Members of one tile shape, one above and one below a tile a compute unit: each runs the
    kernel that it runs alone, so the results are the same bits."""
    cases = [shear(2)[0], W.perturbed(70, 33, seed=2, kappa=0.0176)]
    print(f"batch precision {precision}", flush=True)
    alone = [run_gpu(c, 7, precision, tile=5) for c in cases]
    lats = [pond.Lattice(pond_config(c, precision, tile=5)).init_fields(c.rho, c.u, c.T) for c in cases]
    with pond.Batch() as batch:
        for lat in lats:
            batch.add(lat)
        assert batch.step(7) == []
        for lat, ref in zip(lats, alone):
            got = lat.moments()
            assert all(np.array_equal(got[k], ref[k]) for k in ref)
    for lat in lats:
        lat.close()


@pytest.mark.parametrize("two_kernel", [0, 1])
@pytest.mark.parametrize("groups", [1, 2, 3, 5])
def test_batch_runs_its_groups_side_by_side(groups, two_kernel):
    """Long runs take the groups in up to three branches, on few and on more groups than that;
    the members' results are the bits of the same steps alone."""
    tiles, steps = [2, 5, 2, 5, 0][:groups], 94
    prec = [pond.FP64, pond.FP64, pond.FP32_STORE, pond.FP32_STORE, pond.FP64][:groups]
    cases = [W.perturbed(40 + 9 * k, 33, seed=k, kappa=0.0176) for k in range(groups)]
    print(f"batch of {groups} groups two_kernel {two_kernel}", flush=True)
    alone = [run_gpu(c, steps, p, tile=t, two_kernel=two_kernel) for c, p, t in zip(cases, prec, tiles)]
    lats = [pond.Lattice(pond_config(c, p, tile=t, two_kernel=two_kernel)).init_fields(c.rho, c.u, c.T)
            for c, p, t in zip(cases, prec, tiles)]
    with pond.Batch() as batch:
        for lat in lats:
            batch.add(lat)
        assert batch.step(steps - 1) == [] and batch.step(1) == []
        for lat, ref in zip(lats, alone):
            got = lat.moments()
            assert all(np.array_equal(got[k], ref[k]) for k in ref)
    for lat in lats:
        lat.close()


@pytest.mark.parametrize("precision", list(TOL))
@pytest.mark.parametrize("law", ["isothermal", "double well", "dieterici"])
def test_laws_with_one_lane_a_receiver(law, precision):
    """The equation-of-state variants of the one-lane kernels, on 288 tiles."""
    print(f"law {law} precision {precision}", flush=True)
    kw = {"isothermal": dict(isothermal=1, T0=1.05 * W.T_CR),
          "double well": dict(eos=pond.EOS_DOUBLE_WELL, isothermal=1, T0=0.1, eos_c=(8e-4, 5.0, 0.5, 0.1)),
          "dieterici": dict(eos=pond.EOS_DIETERICI, a=2.0 * W.T_CR / W.RHO_CR, b=0.5 / W.RHO_CR)}[law]
    rho0 = {"isothermal": 1.5, "double well": 5.0, "dieterici": 2.5}[law]
    case = W.perturbed(275, 250, seed=9, rho0=rho0, u0=(0.05, -0.02), kappa=0.0176, dt=0.2, **kw)
    check(run_oracle(case, 2), run_gpu(case, 2, precision, tile=5), ("rho", "ux", "uy", "E", "T", "p"), TOL[precision], law)


def assert_crosses(fields, n, axes, block):
    """In the state that a run ends with, within one block of nodes (so within a tile), some
    node's u_a is above s = sqrt(theta) and some other's not, and within another below -s and
    not, for each a of `axes`: stencils then reach the window's first and its last columns, and
    their neighbours' do not."""
    grid = tuple(reversed(n))
    s = np.sqrt(3.0 * fields["p"] / fields["rho"])
    for a in axes:
        for sign in (1.0, -1.0):
            fast = (sign * fields["u" + "xyz"[a]] > s).reshape(grid)
            blocks = [fast[..., y:y + block[1], x:x + block[0]] for y in range(0, n[1], block[1])
                      for x in range(0, n[0], block[0])]
            assert any(b.any() and not b.all() for b in blocks), f"u_{'xyz'[a]} does not cross {sign} s"


@functools.lru_cache(maxsize=None)
def shear3(axes, n_pass):
    """A box sheared across s and -s in u_x, in u_y or in both, within its tiles of 16 x 8.  The
    flow is that of shear(): its largest speed, temperature and 3 steps, so its tolerances too."""
    nx, ny, nz = n = (35, 25, 6)
    case = W.perturbed3(*n, seed=23, rho0=1.0, t_over_tcr=1.4, kappa=0.0176, n_pass=n_pass, dt=0.2)
    z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    for a in axes:
        wave = y / ny if a == 0 else x / nx
        case.u[a] = (1.2 * np.sin(2.0 * np.pi * wave)).ravel()
    ref = run_oracle3(case, 3)
    assert_crosses(ref, n, axes, (16, 8))
    return case, ref


@pytest.mark.parametrize("precision", list(TOL))
@pytest.mark.parametrize("axes", [(0,), (1,), (0, 1)])
@pytest.mark.parametrize("n_pass", [1, 2, 3])
def test_general_window_in_three_dimensions(n_pass, axes, precision):
    """The window with every tap, which a workgroup takes when one of its stencils reaches
    the outermost columns or rows."""
    print(f"3d shear in axes {axes} n_pass {n_pass} precision {precision}", flush=True)
    case, ref = shear3(axes, n_pass)
    check(ref, run_gpu(case, 3, precision), ("rho", "ux", "uy", "uz", "E", "T", "p"), TOL[precision], case.name)


@functools.lru_cache(maxsize=None)
def cross_shear(n, n_pass):
    """shear() turned by a quarter and periodic: u_y crosses s and -s along x."""
    nx, ny = n
    case = W.perturbed(nx, ny, seed=24, rho0=1.0, t_over_tcr=1.4, kappa=0.0176, n_pass=n_pass, dt=0.2)
    case.u[1] = np.tile(1.2 * np.sin(2.0 * np.pi * np.arange(nx) / nx), ny)
    ref = run_oracle(case, 3)
    assert_crosses(ref, n, (1,), (16, 8))
    return case, ref


@pytest.mark.parametrize("precision", list(TOL))
@pytest.mark.parametrize("two_kernel", [0, 1])
@pytest.mark.parametrize("n,tile", [((250, 275), 0), ((250, 275), 5), ((61, 43), 2), ((61, 43), 5)])
@pytest.mark.parametrize("n_pass", [1, 2, 3])
def test_general_window_across_y(n_pass, n, tile, two_kernel, precision):
    """The outermost rows of the 2D window, whose weights two lanes a receiver split between
    them: on more tiles than compute units (one lane) and on a few (two)."""
    print(f"2d shear in u_y {n} n_pass {n_pass} tile {tile} two_kernel {two_kernel} precision {precision}", flush=True)
    case, ref = cross_shear(n, n_pass)
    got = run_gpu(case, 3, precision, tile=tile, two_kernel=two_kernel)
    check(ref, got, ("rho", "ux", "uy", "E", "T", "p"), TOL[precision], case.name)
