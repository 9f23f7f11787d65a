"""The block kernel (several steps per launch in LDS-resident tiles, the default
of small 2D lattices) against one launch per step (a fixed single-step tiling):
the per-node arithmetic is the same, so the states have to be equal bit for bit.

Shapes at the edges of its tiles: sides narrower than the stencil, one column
below and above the 64 and 128 columns a row of a tile holds (whole periodic rows
against tiles with halo columns), and heights below, at and above a tile's rows
and its halo.  Step counts that no launch's step count divides, and samples
between them.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

fsc = pytest.importorskip("paper_2212_07848_amd")
torch = pytest.importorskip("torch")


def _p(nx, ny, stencil, precision, kBT, r=0):
    return fsc.make_params(D=2, nx=nx, ny=ny, stencil=stencil, precision=precision, T_hat=0.8, rho0=0.62,
                           kBT=kBT, lam=(1.1, 0.9, 1.2), seed=5 + r, replica=r)


def _march(obj, stencil, precision):
    obj.set_tiling(*fsc.tile_shapes(2, stencil, precision)[0], 512)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("stencil", [4, 8])
@pytest.mark.parametrize("kBT", [0.0, 1e-5])
@pytest.mark.parametrize("nx,ny", [(1, 1), (2, 7), (5, 3), (63, 33), (64, 64), (65, 40), (127, 9),
                                   (128, 31), (129, 17), (300, 70), (513, 5)])
def test_block_kernel_equals_single_steps(nx, ny, stencil, precision, kBT):
    print(f"block kernel {nx}x{ny} E{stencil} {precision} kBT={kBT}", flush=True)
    states, sk = [], []
    for fixed in (False, True):
        with fsc.Lattice(_p(nx, ny, stencil, precision, kBT)) as lat:
            lat.init_uniform()
            rng = np.random.default_rng(3)
            lat.set_populations(lat.get_populations() * (1.0 + 0.05 * rng.uniform(-1, 1, (9, ny, nx))), 7)
            if fixed:
                _march(lat, stencil, precision)
            lat.step(1)
            lat.step(13)
            lat.run(33, 11)
            states.append(lat.get_populations())
            sk.append(lat.read_sk(fsc.FSC_SK_AXIS)[0])
            assert lat.t == 54
    assert np.array_equal(states[0], states[1])
    assert np.allclose(sk[0], sk[1], rtol=1e-12, atol=0.0)  # FP64 sums in another order


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_block_kernel_on_uneven_replicas_and_graph_chunks(precision):
    sides = [(64, 64), (100, 30), (128, 128), (31, 200), (190, 61)]
    got = []
    for fixed in (False, True):
        ens = fsc.Ensemble([_p(nx, ny, 4, precision, 1e-5, r) for r, (nx, ny) in enumerate(sides)])
        ens.init_uniform()
        if fixed:
            _march(ens, 4, precision)
        ens.run(300, 0)   # chunks replayed from a graph
        ens.run(35, 7)    # samples, an odd number of launches between them
        got.append([ens.get_populations(r) for r in range(len(sides))])
        ens.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)


def test_autotune_of_a_small_lattice_keeps_the_state_and_the_results():
    got = []
    for tune in (False, True):
        with fsc.Lattice(_p(96, 80, 4, "fp32", 1e-5)) as lat:
            lat.init_uniform()
            lat.step(5)
            if tune:
                lat.autotune()
            lat.step(40)
            got.append(lat.get_populations())
    assert np.array_equal(got[0], got[1])


def test_steps_captured_by_the_caller_replay_like_eager_ones():
    stream = torch.cuda.Stream()
    p = _p(96, 80, 4, "fp32", 1e-5)
    with fsc.Lattice(p, stream=stream) as lat, fsc.Lattice(p) as ref:
        for q in (lat, ref):
            q.init_uniform()
            q.step(3)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
            lat.step(10)
        for _ in range(3):
            with torch.cuda.stream(stream):
                g.replay()
            stream.synchronize()
            ref.step(10)
            assert np.array_equal(lat.get_populations(), ref.get_populations())


def test_samples_captured_by_the_caller_are_recorded_by_every_replay():
    stream = torch.cuda.Stream()
    p = _p(48, 48, 4, "fp64", 1e-5)
    with fsc.Lattice(p, stream=stream) as lat, fsc.Lattice(p) as ref:
        def rows():
            a, b = lat.read_series(), ref.read_series()
            assert np.array_equal(a["step"], b["step"])
            for key in ("L", "S"):  # FP64 sums in another order
                assert np.allclose(a[key], b[key], rtol=1e-12, atol=0.0)
            assert np.array_equal(lat.read_modes(), ref.read_modes())
            return len(a["step"])

        for q in (lat, ref):
            q.init_uniform()
            q.series_enable(8)
            q.modes_enable(3, 8)
            q.step(3)
            q.measure_sk()
        stream.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
            lat.run(2, 2)
            lat.measure_sk()
        assert rows() == 1  # a capture records nothing
        for k in range(1, 4):
            with torch.cuda.stream(stream):
                g.replay()
            ref.run(2, 2)
            ref.measure_sk()
            assert rows() == 1 + 2 * k
        for q in (lat, ref):  # eager samples go on from there, up to the capacity
            q.run(4, 2)
        assert rows() == 8
