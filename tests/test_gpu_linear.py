"""The exact linear S(k) routine (fsc_linear_sk) against the oracle's own
per-k covariance (its Lyapunov doubling, written separately), against the
closed form of Eq. 16 on the axes, against brute force over every mode of
small lattices for the radial shells, and the lattice's measured 3D radial
S(k) against it."""
import math

import numpy as np
import pytest

import oracle as O
from oracle import theory as T

pytestmark = pytest.mark.gpu

fsc = pytest.importorskip("paper_2212_07848_amd")


def _p(D, stencil, T_hat, rho0, kBT, lam=(1, 1, 1), n=16):
    return fsc.make_params(D=D, nx=n, ny=n, nz=n if D == 3 else 1, stencil=stencil, T_hat=T_hat,
                           rho0=rho0, kBT=kBT, lam=lam)


@pytest.mark.parametrize("D,stencil", [(2, 4), (2, 8), (3, 4)])
@pytest.mark.parametrize("lam", [(1.0, 1.0, 1.0), (0.8, 1.3, 1.7)])
def test_random_wave_vectors_match_the_oracle(D, stencil, lam):
    rng = np.random.default_rng(D * 10 + stencil)
    kv = rng.uniform(-math.pi, math.pi, size=(24, D))
    for T_hat, n0 in ((0.9, 0.5), (0.8, 2.2)):
        p = _p(D, stencil, T_hat, n0, 1e-4, lam)
        got = fsc.linear_sk(p, kv)
        ref = np.array([T.sk_linear_stationary(k, D=D, kind=stencil, n0=n0,
                                               G=T.coupling(T_hat), kBT=1e-4, lam=lam) for k in kv])
        assert np.allclose(got, ref, rtol=1e-9, atol=0), np.max(np.abs(got / ref - 1))


@pytest.mark.parametrize("D,stencil", [(2, 4), (2, 8), (3, 4)])
def test_axis_values_are_eq16(D, stencil):
    k = 2 * np.pi * np.arange(1, 33) / 64
    kv = np.zeros((len(k), D))
    kv[:, 0] = k
    for T_hat, n0 in ((0.9, 0.5), (0.8, 0.62), (0.95, 1.6)):
        got = fsc.linear_sk(_p(D, stencil, T_hat, n0, 1e-13), kv)
        ref = T.sk_exact_axis(k, n0, T.coupling(T_hat), 1e-13, D=D, kind=stencil)
        assert np.allclose(got, ref, rtol=1e-9, atol=0)


@pytest.mark.parametrize("D,n", [(2, 20), (3, 8)])
def test_radial_shells_match_brute_force(D, n):
    p = _p(D, 4, 0.85, 0.55, 1e-4, n=n)
    nb = O.radial_bin(D * (n // 2) ** 2) + 1
    mean, cnt = fsc.linear_sk_radial(p, nb)
    # every mode of the lattice, one by one
    m = np.arange(n)
    m = np.where(m > n // 2, m - n, m)
    grids = np.meshgrid(*([m] * D), indexing="ij")
    modes = np.stack([g.ravel() for g in grids], axis=1)
    modes = modes[np.any(modes != 0, axis=1)]
    S = fsc.linear_sk(p, 2 * np.pi * modes / n)
    b = O.radial_bins_of((modes ** 2).sum(axis=1))
    ref = np.bincount(b, weights=S, minlength=nb)[:nb] / np.maximum(np.bincount(b, minlength=nb)[:nb], 1)
    assert np.array_equal(cnt, np.bincount(b, minlength=nb)[:nb])
    assert np.allclose(mean, ref, rtol=1e-11, atol=0)
    # and a few modes through the oracle directly
    for i in range(0, len(modes), max(1, len(modes) // 7)):
        r = T.sk_linear_stationary(2 * np.pi * modes[i] / n, D=D, kind=4, n0=0.55,
                                   G=T.coupling(0.85), kBT=1e-4)
        assert S[i] == pytest.approx(r, rel=1e-9)


def test_measured_3d_radial_structure_factor_matches_the_linear_theory():
    # metastable gas at T_hat = 0.8 (between binodal 0.431 and spinodal 0.645)
    n, nrep, T_hat, n0, kBT = 24, 16, 0.8, 0.55, 1e-13
    plist = [fsc.make_params(D=3, nx=n, ny=n, nz=n, stencil=4, precision="fp32", T_hat=T_hat,
                             rho0=n0, kBT=kBT, seed=31, replica=r) for r in range(nrep)]
    ens = fsc.Ensemble(plist)
    ens.init_uniform()
    ens.run(3000, 0)
    ens.sk_reset()
    ens.run(12000, 40)
    tot = cnt = None
    for r in range(nrep):
        s, _, c = ens.read_sk(r, fsc.FSC_SK_RADIAL)
        tot = s if tot is None else tot + s
        cnt = c if cnt is None else cnt + c
    ens.close()
    meas = tot / np.maximum(cnt, 1)
    nb = len(meas)
    theory, _ = fsc.linear_sk_radial(plist[0], nb)
    rel = meas[1:] / theory[1:] - 1
    print("relative deviation per shell", np.round(rel, 4))
    assert np.max(np.abs(rel)) < 0.05
    assert abs(np.mean(rel)) < 0.01


@pytest.mark.parametrize("D,stencil", [(2, 4), (2, 8), (3, 4)])
@pytest.mark.parametrize("nk", [1, 63, 64, 65, 130])
def test_unit_rates_equal_the_general_form(D, stencil, nk):
    # rates of exactly 1 take the conserved-moment sum, the next double below the
    # general one; both carry about 1e-16 / (1 - |eigenvalue|), 1e-11 at |k| = 0.01
    rng = np.random.default_rng(nk)
    kv = rng.uniform(-math.pi, math.pi, size=(nk, D))
    kv[0] = 0.0
    kv[0, -1] = math.pi  # a unit-modulus eigenvalue that the noise does not excite
    kv[nk // 2] = 0.01
    below = float(np.nextafter(1.0, 0.0))
    for T_hat, n0 in ((0.9, 0.5), (0.8, 2.2), (0.8, 1.0)):  # the last one unstable at small k
        got = fsc.linear_sk(_p(D, stencil, T_hat, n0, 1e-4), kv)
        ref = fsc.linear_sk(_p(D, stencil, T_hat, n0, 1e-4, (below,) * 3), kv)
        assert np.array_equal(np.isfinite(got), np.isfinite(ref))
        ok = np.isfinite(ref)
        assert np.allclose(got[ok], ref[ok], rtol=1e-9, atol=0), np.max(np.abs(got[ok] / ref[ok] - 1))


@pytest.mark.parametrize("lam", [(1, 1, 1), (0.8, 1.3, 1.7)])
@pytest.mark.parametrize("D,n", [(2, 2), (2, 3), (2, 65), (3, 2), (3, 5), (3, 14)])
def test_device_wave_vectors_of_the_radial_shells(D, n, lam):
    p = _p(D, 4, 0.85, 0.55, 1e-4, lam, n=n)
    m = np.arange(n)
    m = np.where(m > n // 2, m - n, m)
    modes = np.stack([g.ravel() for g in np.meshgrid(*([m] * D), indexing="ij")], axis=1)
    modes = modes[np.any(modes != 0, axis=1)]
    nb = O.radial_bin(D * (n // 2) ** 2) + 1
    mean, cnt = fsc.linear_sk_radial(p, nb)
    b = O.radial_bins_of((modes ** 2).sum(axis=1))
    S = fsc.linear_sk(p, 2 * np.pi * modes / n)
    assert np.array_equal(cnt, np.bincount(b, minlength=nb)[:nb])
    ref = np.bincount(b, weights=S, minlength=nb)[:nb] / np.maximum(cnt, 1)
    assert np.allclose(mean, ref, rtol=1e-11, atol=0)


@pytest.mark.parametrize("D,stencil", [(2, 4), (2, 8), (3, 4)])
def test_unstable_and_noise_free_states_at_unit_rates(D, stencil):
    # an unstable state has no stationary S(k) at small k (NaN), and without noise it is
    # 0; a wave vector that is no number gives NaN
    kv = np.concatenate([np.random.default_rng(2).uniform(-math.pi, math.pi, size=(100, D)),
                         np.full((1, D), 1e-3), np.zeros((1, D)), np.full((1, D), math.nan)])
    for n0, T_hat in ((1.0, 0.8), (1.0, 0.5), (0.5, 0.9)):
        quiet = fsc.linear_sk(_p(D, stencil, T_hat, n0, 0.0), kv)
        assert np.all(quiet[:-1] == 0.0) and np.isnan(quiet[-1])
        got = fsc.linear_sk(_p(D, stencil, T_hat, n0, 1e-4), kv)
        assert not np.any(np.isinf(got)) and np.isnan(got[-1])
        assert np.isnan(got[100]) == (n0 == 1.0)
    mean, _ = fsc.linear_sk_radial(_p(D, stencil, 0.5, 1.0, 0.0, n=8), 4)
    assert np.all(mean == 0.0)
