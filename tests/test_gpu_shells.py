"""Shells of the structure factor where their sort and sums can go wrong: one
shell, more shells than modes per shell, chunks of 64 modes and of more, boxes
transformed as one batch and (beyond 2^22 sites) one field at a time; against
numpy's FFT of the same fields.  Needs an MI355X."""
import numpy as np
import pytest

from oracle import spectra
from paper_2602_16486_amd import Lattice, _lib
from paper_2602_16486_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu_present():
    assert _lib.device_count() > 0, "no HIP device visible: the gpu tests need an MI355X"


@pytest.mark.parametrize("q,shape,nbins", [
    (9, (8, 8), 1024), (9, (200, 96), 1), (27, (70, 66, 48), 1024), (27, (64, 64, 64), 17),
    (9, (2048, 2049), 40), (19, (1, 7, 5), 6)])
def test_shell_averages_match_numpy(q, shape, nbins):
    n = W.n_sites(shape)
    with Lattice(q, shape, storage="f32", kT=1e-4, seed=3) as lat:
        lat.step(3)
        rho, u = lat.macroscopic()
        for bins in (5, nbins):  # the shells can be chosen again
            lat.sk_reset(bins)
            lat.sk_accumulate()
            got, ns = lat.sk_shells()
    sa = spectra.ShellAverager(shape, nbins)
    box = tuple(shape)[::-1] if len(shape) == 3 else (1,) + tuple(shape)[::-1]
    sa.add([a.reshape(box) for a in (rho - 1.0, *u)])
    ref = sa.shells()
    assert ns == 1
    assert np.array_equal(got[:, 1], ref[:, 1])
    assert np.allclose(got[:, 0], ref[:, 0], rtol=1e-12)
    # FP32 fields and transform: 24-bit roundings in log2(n) butterfly stages,
    # relative to the largest shell of the column
    tol = 2.0 ** -24 * 8 * (2 + np.log2(n))
    assert np.all(np.abs(got[:, 2:] - ref[:, 2:]) <= tol * np.abs(ref[:, 2:]).max(axis=0))
