"""Small D2Q9 boxes take several steps per launch: the populations and every
statistics row equal those of single steps bit for bit, whatever the run
length (odd and even chunks, runs of one and two steps) and however the box
divides into tiles.  Needs an MI355X."""
import numpy as np
import pytest

import oracle as O
from paper_2602_16486_amd import Lattice, _lib, rate_vector
from paper_2602_16486_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu_present():
    assert _lib.device_count() > 0, "no HIP device visible: the gpu tests need an MI355X"


# the smallest box, one cell exactly, one site beyond a cell, whole cells,
# ragged cells and tiles, tiles of 4, 8, 12 and 16 rows, the last box of the
# rule and the first beyond it (single steps on both sides), thin boxes
SHAPES = [(8, 8), (16, 16), (17, 9), (64, 32), (37, 29), (130, 70), (130, 210), (200, 200),
          (250, 255), (512, 256), (513, 256), (8, 700), (700, 8)]


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_runs_equal_single_steps(shape, storage):
    n = W.n_sites(shape)
    rho, u = W.random_macro(shape, 5, umax=0.04, dims=2)
    f = O.init_equilibrium(9, n, rho=rho, u=u) + W.perturbation(9, n, 6, 5e-4)
    for rates, runs in (("paper", (3, 7, 4, 2, 41)), ("single", (9,))):
        kw = dict(storage=storage, tau=0.7, kT=1e-4, lam=rate_vector(9, 0.7, rates), seed=(1 << 33) + 3)
        with Lattice(9, shape, **kw) as a, Lattice(9, shape, **kw) as b:
            for lat in (a, b):
                lat.set_populations(f)
                lat.step_index = (1 << 32) - 5
            for k in runs:
                a.step(k)
                for _ in range(k):
                    b.step(1)
                assert np.array_equal(a.get_populations(), b.get_populations()), (rates, k)
            assert a.step_index == b.step_index
            assert np.array_equal(a.stats(), b.stats()), rates


@pytest.mark.parametrize("shape", [(8, 8), (37, 29), (200, 200)])
def test_run_matches_oracle_fp64(shape):
    n, steps = W.n_sites(shape), 20
    rho, u = W.random_macro(shape, 15, umax=0.04, dims=2)
    f = O.init_equilibrium(9, n, rho=rho, u=u)
    with Lattice(9, shape, storage="f64", tau=0.62, kT=1e-4, seed=4) as lat:
        lat.set_populations(f)
        lat.step(steps)
        got, st = lat.get_populations(), lat.stats()
    st_ref = O.run(9, shape, f, 1e-4, O.paper_lambda(9, 1 / 0.62), 4, 0, 0, steps)
    _, w = O.lattice(9)
    assert np.abs(got - f).max() / np.abs(f - w[:, None]).max() < 1e-12
    # N-term FP64 sums of values below 1.1, in another order
    assert np.abs(st - st_ref).max() < 1.1 * n * n * 2.0 ** -53


def test_nonfinite_rows_equal_single_steps():
    kw = dict(storage="f32", kT=50.0, seed=2)
    with Lattice(9, (40, 24), **kw) as a, Lattice(9, (40, 24), **kw) as b:
        a.step(20)
        for _ in range(20):
            b.step(1)
        st, ref = a.stats(raise_nonfinite=False), b.stats(raise_nonfinite=False)
    assert ref[:, 11].any()
    assert np.array_equal(st, ref, equal_nan=True)


@pytest.mark.parametrize("cap", [1, 5, 70])
def test_short_series_and_no_series(cap):
    """Rings shorter than the batch of steps reduced together, and a lattice
    without statistics."""
    kw = dict(storage="f32", kT=1e-4, seed=4)
    with Lattice(9, (50, 40), series_capacity=cap, **kw) as lat, Lattice(9, (50, 40), **kw) as ref, \
            Lattice(9, (50, 40), flags=_lib.FLAG_NO_STATS, **kw) as bare:
        for n in (130, 6):
            for x in (lat, ref, bare):
                x.step(n)
            got, want = lat.stats(), ref.stats()
            assert len(want) == n and np.array_equal(got, want[-cap:])
        assert np.array_equal(lat.get_populations(), bare.get_populations())


def test_launch_shape_asked_for_keeps_single_steps_until_tuned():
    kw = dict(storage="f32", kT=1e-4, seed=4)
    with Lattice(9, (70, 40), **kw) as a, Lattice(9, (70, 40), **kw) as b:
        a.set_launch(64, 33)
        assert a.launch == (64, 33)
        a.step(9)
        b.step(9)
        assert np.array_equal(a.get_populations(), b.get_populations())
        assert np.allclose(a.stats(), b.stats(), rtol=1e-12, atol=1e-12)
        best = min(a.autotune(steps_per_trial=2), key=lambda t: t[2])
        assert a.launch == best[:2]
        a.step(9)
        b.step(9)
        assert np.array_equal(a.get_populations(), b.get_populations())
        assert np.array_equal(a.stats(), b.stats())
