"""3-D boxes whose rows would leave lanes idle take tiles of a plane's sites:
populations equal those of an ensemble of the same box (addresses of its own)
bit for bit, in both streaming forms and every workgroup size, and the
statistics up to the order of their FP64 sums.  The GPU cases need an
MI355X."""
import numpy as np
import pytest

import oracle as O
from paper_2602_16486_amd import Ensemble, Lattice, rate_vector
from paper_2602_16486_amd import workloads as W

# two columns, one row or plane alone, planes below one workgroup, of whole
# tiles and of one site more, rows just beyond a workgroup, rows of whole cache
# lines, more than one round of the tile map (256 tiles) with a remainder
SHAPES = [(2, 9, 5), (2, 130, 3), (17, 1, 6), (40, 7, 1), (9, 6, 5), (16, 16, 3), (33, 31, 4),
          (65, 63, 2), (129, 5, 3), (193, 4, 3), (32, 48, 5), (96, 20, 3), (48, 64, 34)]


def test_row_of_a_lane_by_a_product():
    """t // nx = t (2^32 // nx + 1) >> 32 for every t < nx + 256: the sites on
    both sides of each row's end."""
    for nx in range(2, 8193):
        k = np.arange(1, 256 // nx + 3, dtype=np.uint64)
        t = np.unique(np.concatenate([k * np.uint64(nx), k * np.uint64(nx) - np.uint64(1)]))
        t = np.append(t[t < nx + 256], np.uint64(nx + 255))
        assert np.array_equal(t * np.uint64((1 << 32) // nx + 1) >> np.uint64(32), t // np.uint64(nx))


@pytest.mark.gpu
@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("q", [27, 19])
@pytest.mark.parametrize("shape", SHAPES)
def test_plane_tiles_equal_an_ensemble(shape, q, storage):
    n = W.n_sites(shape)
    rho, u = W.random_macro(shape, 8, umax=0.04)
    f = O.init_equilibrium(q, n, rho=rho, u=u) + W.perturbation(q, n, 9, 5e-4)
    # |v| <= 1.1 of each term; any order of n FP64 additions
    atol = 1.1 * n * n * 2.0 ** -52
    for rates in ("paper", "isotropic"):
        kw = dict(tau=0.7, kT=1e-4, lam=rate_vector(q, 0.7, rates), seed=(1 << 33) + 5, replica=0)
        with Ensemble([dict(q=q, shape=shape, **kw)], storage=storage) as e:
            e.set_populations(0, f)
            e.step(35)
            ref, ref_st = e.get_populations(0), e.stats(0)
        launches = [None] if rates == "isotropic" else [None, (64, 1 << 20), (128, 5), (192, 1 << 20), (256, 1 << 20)]
        for in_place in (False, True):
            for launch in launches:
                with Lattice(q, shape, storage=storage, in_place=in_place, **kw) as lat:
                    if launch:
                        lat.set_launch(*launch)
                    lat.set_populations(f)
                    lat.step(35)
                    assert np.array_equal(lat.get_populations(), ref), (rates, in_place, launch)
                    assert np.allclose(lat.stats(), ref_st, rtol=0, atol=atol), (rates, in_place, launch)


@pytest.mark.gpu
@pytest.mark.parametrize("rates", ["paper", "isotropic"])
def test_plane_tiles_of_a_box_that_draws_late(rates):
    """D3Q27 FP32 beyond 2^22 sites draws its normals when it collides: plane
    tiles there (rows of whole sectors, 200 x 200 x 112) against an ensemble,
    bit for bit."""
    q, shape = 27, (200, 200, 112)
    n = W.n_sites(shape)
    assert n > 1 << 22
    kw = dict(tau=0.7, kT=1e-4, lam=rate_vector(q, 0.7, rates), seed=11, replica=0)
    with Ensemble([dict(q=q, shape=shape, **kw)], storage="f32") as e:
        e.step(5)
        ref, ref_st = e.get_populations(0), e.stats(0)
    with Lattice(q, shape, storage="f32", **kw) as lat:
        # tiles of 256 sites of a plane, one per workgroup; a row would idle 56 lanes
        assert lat.launch == (256, (200 * 200 + 255) // 256 * 112)
        lat.step(5)
        assert np.array_equal(lat.get_populations(), ref)
        assert np.allclose(lat.stats(), ref_st, rtol=0, atol=1.1 * n * n * 2.0 ** -52)
