"""Read-outs against the populations they come from: the state reductions where a
row does not fill a block, fills it and passes it, on lattices of one node to more
nodes than the grid covers at once; and S(k) sums of the sizes at which they change
from the polled read-out to a copy."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

fsc = pytest.importorskip("paper_2212_07848_amd")


def _state(lat, shape, seed):
    rng = np.random.default_rng(seed)
    f = lat.get_populations() * (1.0 + 0.05 * rng.uniform(-1, 1, (9 if len(shape) == 2 else 19,) + shape))
    lat.set_populations(f, 3)
    return lat.get_populations()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", [(1, 1), (1, 255), (3, 256), (5, 257), (1100, 255), (1030, 256), (7, 5, 9),
                                   (2, 3, 300)])
def test_stats_of_narrow_and_wide_rows(shape, precision):
    D = len(shape)
    c, _ = O.lattice(D)
    nz, ny, nx = (1,) * (3 - D) + shape
    with fsc.Lattice(fsc.make_params(D=D, nx=nx, ny=ny, nz=nz, stencil=4, precision=precision, T_hat=0.8,
                                     rho0=0.62, kBT=0.0)) as lat:
        lat.init_uniform()
        f = _state(lat, shape, nx)
        for _ in range(2):  # the counter of finished blocks is left at zero
            s = lat.stats()
        n = f.sum(0)
        eps = 1e-12 if precision == "fp64" else 1e-6
        assert s["mass"] == pytest.approx(n.sum(), rel=eps)
        assert s["rho_min"] == pytest.approx(n.min(), rel=eps)
        assert s["rho_max"] == pytest.approx(n.max(), rel=eps)
        for d in range(D):
            j = np.tensordot(np.asarray(c)[:, d], f, 1).sum()
            assert s["mom"][d] == pytest.approx(j, abs=eps * n.sum())


@pytest.mark.parametrize("nx", [508, 510, 512, 514])
def test_structure_factor_readout_at_the_polled_size(nx):
    with fsc.Lattice(fsc.make_params(D=2, nx=nx, ny=4, stencil=4, precision="fp64", T_hat=0.8, rho0=0.62,
                                     kBT=0.0)) as lat:
        lat.init_uniform()
        f = _state(lat, (4, nx), 1)
        for k in range(1, 3):
            lat.measure_sk()
            got, sq, cnt = lat.read_sk(fsc.FSC_SK_AXIS)
            ref = O.sk_sample(O.density(f))["axis"][0]
            assert np.allclose(got[:, : ref.shape[1]], k * ref, rtol=1e-9, atol=1e-9 * ref.max())
