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


def _shells(P):
    n = P.shape[0]
    m = np.minimum(np.arange(n), n - np.arange(n))
    b = O.radial_bins_of((m[:, None] ** 2 + m[None] ** 2).ravel())
    cnt = np.bincount(b).astype(float)
    cnt[0] -= 1.0
    w = P.ravel().copy()
    w[0] = 0.0
    return np.bincount(b, weights=w) / np.maximum(cnt, 1.0)


# sides that are no power of two: chirp transforms of 8 points to 8192 in doubles,
# and beyond 4096 in floats
@pytest.mark.parametrize("n", [3, 5, 33, 48, 90, 100, 150, 301, 487, 750, 1000, 2047, 4095, 4097])
def test_field_spectra_of_odd_sides_lose_no_norm(n):
    """White fields, every |X|^2 / N about 1.  The half spectra are rounded to FP32
    between the axes: 2^-24 / sqrt(3) of a value (rms), 5e-8 of a mode's |X|^2, less
    in a shell of many, and no bias.  A chirp in floats adds 2.4 roundings of 2^-24 per
    axis to a mode."""
    torch = pytest.importorskip("torch")
    batch = 8 if n < 400 else (2 if n < 2000 else 1)
    rng = np.random.default_rng(n)
    f = rng.normal(size=(batch, n, n)).astype(np.float32)
    got, _ = fsc.field_sk(torch.from_numpy(f).cuda(), batch, n)
    e = []
    for b in range(batch):
        ref = _shells(np.abs(np.fft.fft2(f[b].astype(np.float64))) ** 2 / n ** 2)[1:]
        e.append((got[b][1:] - ref) / np.maximum(ref, 1.0))
    e = np.concatenate(e)
    assert abs(e.mean()) < 5e-8
    assert np.sqrt(np.mean(e * e)) < 1e-7


@pytest.mark.parametrize("n", [48, 90, 100, 150, 301])
def test_field_spectra_of_odd_sides_keep_the_tail_of_a_steep_one(n):
    """Spectra that fall by 8 decades.  The rounding between the axes leaves noise of
    power (2^-24)^2 times a column's mean power, s, in every mode P: 2 sqrt(P s) + s,
    and four times that is allowed."""
    torch = pytest.importorskip("torch")
    k = np.hypot(np.fft.fftfreq(n)[:, None], np.fft.fftfreq(n)[None]) * n
    f = np.fft.ifft2(np.fft.fft2(np.random.default_rng(n).normal(size=(n, n))) / (1.0 + (k / 4.0) ** 4)).real
    f = (f / f.std()).astype(np.float32)
    got, _ = fsc.field_sk(torch.from_numpy(f[None]).cuda(), 1, n)
    P = np.abs(np.fft.fft2(f.astype(np.float64))) ** 2 / n ** 2
    ref, s = _shells(P), 2.0 ** -48 * P.mean(0).max()
    assert np.all(np.abs(got[0] - ref)[1:] <= 4.0 * (2.0 * np.sqrt(ref * s) + s)[1:])


@pytest.mark.parametrize("sides", [[(64, 64), (30, 64), (64, 45), (7, 128)],
                                   [(16, 12, 10), (8, 16, 16), (9, 8, 12), (4, 7, 8)]])
def test_samples_of_replicas_with_even_and_odd_sides(sides):
    D = len(sides[0])
    ps = [fsc.make_params(D=D, nx=s[-1], ny=s[-2], nz=s[0] if D == 3 else 1, stencil=4, precision="fp32", T_hat=0.8,
                          rho0=0.62, kBT=1e-5, seed=5, replica=r) for r, s in enumerate(sides)]
    ens = fsc.Ensemble(ps)
    ens.init_uniform()
    ens.run(4, 4)
    for r, s in enumerate(sides):
        P = np.abs(np.fft.fftn(ens.get_populations(r).sum(0) - 0.62)) ** 2 / np.prod(s)
        got = ens.read_sk(r)[0]
        for d in range(D):  # axis d = 0 is x, the last one of the array
            line = np.moveaxis(P, D - 1 - d, 0).reshape(s[D - 1 - d], -1)[:, 0]
            m = line.size
            ref = [line[q] + (line[m - q] if 2 * q != m else 0.0) for q in range(1, m // 2 + 1)]
            assert np.allclose(got[d, 1:m // 2 + 1], ref, rtol=1e-5, atol=1e-6 * np.mean(P))
    ens.close()


@pytest.mark.parametrize("long_x", [True, False])
@pytest.mark.parametrize("precision,n", [("fp64", 4096), ("fp64", 5000), ("fp64", 8192), ("fp32", 4100), ("fp32", 8190),
                                         ("fp32", 8192)])
def test_samples_of_long_lines(precision, n, long_x):
    """Lines that fill a block's LDS, one or two at a time: radix-8 passes to 8192 values,
    an FP32 chirp over 16384, FP64 direct sums.  FP32: the passes leave a few 2^-24 of
    the root mean power in an amplitude, 1e-6 of sqrt(P <P>) in a power."""
    shape = (4, n) if long_x else (n, 4)
    with fsc.Lattice(fsc.make_params(D=2, nx=shape[1], ny=shape[0], stencil=4, precision=precision, T_hat=0.8,
                                     rho0=0.62, kBT=0.0)) as lat:
        lat.init_uniform()
        f = _state(lat, shape, n)
        lat.series_enable(1)
        lat.measure_sk()
        got, L = lat.read_sk(fsc.FSC_SK_AXIS)[0], lat.read_series()["L"][0]
    P = np.abs(np.fft.fft2(f.sum(0) - 0.62)) ** 2 / (4 * n)
    rel, mean = (1e-9, 1e-12) if precision == "fp64" else (1e-5, 1e-6)
    for d, line in enumerate((P[0], P[:, 0])):
        m = line.size
        ref = [line[q] + (line[m - q] if 2 * q != m else 0.0) for q in range(1, m // 2 + 1)]
        assert np.allclose(got[d, 1:m // 2 + 1], ref, rtol=rel, atol=mean * P[0, 1:].mean())
    P[0, 0] = 0.0
    k = 2 * np.pi * np.hypot(np.fft.fftfreq(shape[0])[:, None], np.fft.fftfreq(shape[1])[None])
    assert L == pytest.approx(2 * np.pi * P.sum() / (k * P).sum(), rel=rel)


# one lane per cell: f = 1, and small cells of many narrow rows (10000 and 4097 strips
# of the other kernel; 4096 of them take it)
@pytest.mark.parametrize("shape,f", [((37, 41), 1), ((1, 300), 1), ((20000, 4), 2), ((8194, 2), 2), ((8192, 2), 2),
                                     ((12300, 48), 3), ((16400, 20), 4), ((16400, 24), 4), ((12, 600), 6)])
def test_block_means_of_narrow_and_wide_rows(shape, f):
    torch = pytest.importorskip("torch")
    ny, nx = shape
    with fsc.Lattice(fsc.make_params(D=2, nx=nx, ny=ny, stencil=4, precision="fp32", T_hat=0.8, rho0=0.62,
                                     kBT=0.0)) as lat:
        lat.init_uniform()
        rho = _state(lat, shape, nx + f).sum(0)
        out = torch.full((ny // f, nx // f), -1.0, device="cuda")
        torch.cuda.synchronize()
        lat.coarsen(f, out)
        lat.stats()
    ref = rho.reshape(ny // f, f, nx // f, f).mean((1, 3))
    assert np.allclose(out.cpu().numpy(), ref, rtol=3e-7, atol=0.0)  # FP64 sums, one rounding to FP32


# FP32 densities go to the host formed, as floats (65537 to 6291456 nodes), and formed in
# pieces; against the block means of single nodes, rounded once to FP32
@pytest.mark.parametrize("shape", [(256, 256), (257, 256), (65537, 1), (1, 65537), (2400, 2600), (2600, 2600)])
def test_density_by_the_three_ways_to_the_host(shape):
    torch = pytest.importorskip("torch")
    ny, nx = shape
    with fsc.Lattice(fsc.make_params(D=2, nx=nx, ny=ny, stencil=4, precision="fp32", T_hat=0.8, rho0=0.62,
                                     kBT=1e-4, seed=nx)) as lat:
        lat.init_uniform()
        lat.set_tiling(*fsc.tile_shapes(2, 4, "fp32")[0], 2048)
        lat.step(3)
        out = torch.zeros(ny, nx, device="cuda")
        torch.cuda.synchronize()
        lat.coarsen(1, out)
        rho = lat.density()
        mass = lat.stats()["mass"]
    # nine FP32 additions against FP64 ones, of deviations a tenth of the density
    assert np.allclose(out.cpu().numpy(), rho, rtol=3e-7, atol=0.0)
    assert rho.std() > 1e-3 and rho.sum() == pytest.approx(mass, rel=1e-7)
