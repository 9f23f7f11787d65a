"""The surrogate's BF16 matrix-core kernels element by element against the
BF16-emulating reference (oracle/surrogate.py with bf16=True), through the
C ABI.

The reference rounds exactly the operands the kernels keep in bfloat16 and
computes everything else in FP64.  What is left between the two is the
kernels' FP32 accumulation and SiLU (about 1e-6 relative per value) and the
few BF16 roundings that this moves across a rounding boundary: each such flip
changes one value by one bfloat16 step (2^-8 relative), and later layers pass
it on.  So the bulk of the elements must agree to FP32 precision (median
|d| <= 2e-5 of the largest element, where an FP64 reference without the
rounding is off by 5e-4 .. 9e-4 in the median), every element within 5e-3 of
the largest, and at most a few percent of the elements beyond 1e-3.  Deeper
networks pass more flips on: for 9 layers the bounds are 2e-4 (median) and
1e-2 (every element).  A CPU model of the kernels' FP32 arithmetic gives
medians of 1e-7 .. 1e-5 and maxima of 0.9e-3 .. 3.6e-3 for these networks;
measured on the GPU: medians 1e-7 .. 1.8e-5, maxima 1e-4 .. 5.1e-3.  Weight
gradients sum over every pixel: median 3e-6 .. 3e-4 and maximum <= 1.5e-3 of
the layer's largest gradient were measured; the bounds are 1e-3 and 5e-3.
"""
import numpy as np
import pytest

from oracle import surrogate as S

pytestmark = pytest.mark.gpu

fsc = pytest.importorskip("paper_2212_07848_amd")
torch = pytest.importorskip("torch")

from test_gpu_surrogate import _dev, _net  # noqa: E402


def test_device_bf16_conversion_is_round_to_nearest_even():
    # fsc_mfma_probe converts A and B to bfloat16 and multiplies them on the
    # matrix cores; with B a 0/1 selection matrix each output is one converted
    # element of A, exactly (products with 1 and sums with zeros are exact).
    rng = np.random.default_rng(9)
    # normal floats over a wide exponent range, plus bit patterns at and around
    # rounding ties (remainders 0x7FFF, 0x8000, 0x8001 with odd and even kept parts)
    mant = rng.integers(0, 2 ** 23, size=6000)
    expo = rng.integers(1, 254 - 10, size=6000)
    sign = rng.integers(0, 2, size=6000)
    bits = (sign << 31) | (expo << 23) | mant
    ties = []
    for kept in rng.integers(0x0080, 0x7F00, size=600):
        for rem in (0x7FFF, 0x8000, 0x8001):
            ties.append((int(kept) << 16) | rem)
    allbits = np.concatenate([bits, np.array(ties)]).astype(np.uint32)
    allv = allbits.view(np.float32).astype(np.float64)
    n = allv.size
    got = np.empty(n)
    sel_lo = np.zeros((32, 16), dtype=np.float32)
    sel_hi = np.zeros((32, 16), dtype=np.float32)
    for j in range(16):
        sel_lo[j, j] = 1.0
        sel_hi[16 + j, j] = 1.0
    k = 0
    while k < n:
        A = np.zeros((16, 32), dtype=np.float32)
        chunk = allv[k:k + 512]
        A.ravel()[: chunk.size] = chunk
        lo = fsc.mfma_probe(A, sel_lo)   # columns 0..15 of A
        hi = fsc.mfma_probe(A, sel_hi)   # columns 16..31 of A
        out = np.concatenate([lo, hi], axis=1).ravel()[: chunk.size]
        got[k:k + chunk.size] = out
        k += 512
    want = S.bf16_round(allv)
    assert np.array_equal(got, want), np.argwhere(got != want)[:5]


def _compare(got, ref, what, med_tol=2e-5, max_tol=5e-3, tail_tol=1e-3, tail_frac=0.05):
    scale = np.abs(ref).max()
    d = np.abs(got - ref) / scale
    med, mx, frac = float(np.median(d)), float(d.max()), float((d > tail_tol).mean())
    print(f"{what}: median {med:.1e}, max {mx:.1e}, beyond {tail_tol:.0e}: {frac:.3f}", flush=True)
    assert med <= med_tol, (what, med)
    assert mx <= max_tol, (what, mx)
    assert frac <= tail_frac, (what, frac)
    return med, mx


# shapes: rows of one tile of 16 pixels per wave and of two in the marching layers;
# the 8-row image makes every strip touch the periodic wrap in y
@pytest.mark.parametrize("layers,in_ch,shape", [(3, 1, (2, 32, 32)), (5, 1, (2, 32, 64)),
                                                (5, 2, (2, 16, 64)), (5, 2, (1, 8, 128)),
                                                (9, 2, (2, 32, 64))])
def test_forward_matches_bf16_reference_per_element(layers, in_ch, shape):
    B, H, W = shape
    rng = np.random.default_rng(11)
    p = _net(5, L=layers, in_ch=in_ch).astype(np.float32)
    rho = (1.0 + 0.3 * rng.normal(size=shape)).astype(np.float32)
    prev = (rho + 0.05 * rng.normal(size=shape)).astype(np.float32) if in_ch == 2 else None
    sur = fsc.Surrogate(layers, H, W, B, seed=0, in_ch=in_ch)
    sur.set_params(p)
    sur.set_norm(1.0, 0.3, 0.05)
    x = _dev(rho)
    out = torch.zeros_like(x)
    sur.forward(None if prev is None else _dev(prev), x, out, B)
    torch.cuda.synchronize()
    sur.close()
    got = (out.cpu().numpy().astype(np.float64) - rho) / 0.05
    kw = dict(prev=prev)
    ref = (S.forward(p.astype(np.float64), rho, 32, layers, 1.0, 0.3, 0.05, bf16=True, **kw)
           - rho) / 0.05
    plain = (S.forward(p.astype(np.float64), rho, 32, layers, 1.0, 0.3, 0.05, **kw) - rho) / 0.05
    deep = layers > 5
    _compare(got, ref, f"forward L={layers} K={in_ch} {shape}",
             med_tol=2e-4 if deep else 2e-5, max_tol=1e-2 if deep else 5e-3,
             tail_frac=0.3 if deep else 0.05)
    # the emulation matters: without the rounding the bulk is off by far more
    med_plain = float(np.median(np.abs(got - plain) / np.abs(plain).max()))
    print(f"  FP64 reference without rounding: median {med_plain:.1e}")
    assert med_plain > 5 * float(np.median(np.abs(got - ref) / np.abs(ref).max()))
    # the periodic edges are no worse than the interior
    d = np.abs(got - ref) / np.abs(ref).max()
    edge = np.zeros(shape, dtype=bool)
    edge[:, [0, -1], :] = True
    edge[:, :, [0, -1]] = True
    assert d[edge].max() <= (1e-2 if deep else 5e-3)
    assert np.median(d[edge]) <= (2e-4 if deep else 2e-5)


@pytest.mark.parametrize("in_ch,shape", [(1, (2, 32, 32)), (2, (2, 32, 32)), (2, (2, 16, 64)),
                                         (2, (1, 8, 128))])
def test_gradients_match_bf16_reference_per_element(in_ch, shape):
    B, H, W = shape
    layers = 5
    rng = np.random.default_rng(3)
    p = _net(4, L=layers, in_ch=in_ch).astype(np.float32)
    rho = (1.0 + 0.3 * rng.normal(size=shape)).astype(np.float32)
    prev = (rho + 0.05 * rng.normal(size=shape)).astype(np.float32) if in_ch == 2 else None
    tgt = (rho + 0.05 * rng.normal(size=shape)).astype(np.float32)
    sur = fsc.Surrogate(layers, H, W, B, seed=0, in_ch=in_ch)
    sur.set_params(p)
    sur.set_norm(1.0, 0.3, 0.05)
    loss, g = sur.grad(None if prev is None else _dev(prev), _dev(rho), _dev(tgt), B)
    sur.close()
    ref_loss, ref_g = S.loss_and_grad(p.astype(np.float64), rho, tgt, 32, layers, 1.0, 0.3, 0.05,
                                      prev=prev, bf16=True)
    assert loss == pytest.approx(ref_loss, rel=2e-3)
    o = 0
    for l, (co, ci) in enumerate(S.layer_shapes(32, layers, in_ch)):
        n = co * ci * 9
        for part, sl in (("W", slice(o, o + n)), ("b", slice(o + n, o + n + co))):
            gr, rr = g[sl].astype(np.float64), ref_g[sl]
            if l == layers - 1 and part == "b":
                # the mean-free output makes the loss independent of the last bias
                assert np.abs(rr).max() < 1e-12 * np.abs(ref_g).max()
                continue
            # each weight gradient sums over every pixel, which averages the
            # rounding flips: the bound is per element, relative to the layer's
            # largest gradient
            _compare(gr, rr, f"grad layer {l} {part} K={in_ch} {shape}", med_tol=1e-3,
                     max_tol=5e-3, tail_tol=2e-3, tail_frac=0.02)
        o += n + co


# rows of one and of several tiles, strips of one row and partial last strips, and
# the widths beyond 128 that keep the tiled and the generic layer
@pytest.mark.parametrize("shape", [(7, 5, 32), (100, 5, 32), (3, 11, 96), (2, 6, 160), (1, 8, 192)])
def test_gradients_on_edge_shapes(shape):
    test_gradients_match_bf16_reference_per_element(1, shape)


# images wider than 128 pixels: pairs of tiled layers and a single tiled one (192, 256),
# and the generic layer (160)
@pytest.mark.parametrize("layers,in_ch,shape", [(5, 1, (2, 8, 192)), (5, 2, (1, 4, 256)), (5, 1, (2, 6, 160))])
def test_forward_on_wide_images(layers, in_ch, shape):
    test_forward_matches_bf16_reference_per_element(layers, in_ch, shape)
