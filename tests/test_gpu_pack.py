"""Emission orders against each other and the oracle, at sizes around the pack
kernels' tiles: the tile-baseline order (16 baselines x 16 channels through LDS)
holds exactly the values of the triangle order, the raw sums equal the oracle's
integer X-engine, and emission averaged by F equals the average of the unaveraged
emission in FP64, rounded once (both computed from the same exact integers).
"""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2303_11557_amd import mwax  # noqa: E402
from paper_2303_11557_amd.mwax import Plan, make_config  # noqa: E402


@pytest.mark.parametrize("prec", ["int8", "fp32"])
@pytest.mark.parametrize("n_tiles,L", [(1, 1), (15, 2), (16, 16), (17, 32), (33, 64)])
def test_orders_agree(prec, n_tiles, L):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, T, ints = 2 * n_tiles, 9, 3
    rng = np.random.default_rng(n + L)
    x = rng.integers(-127, 128, size=(T, L, n, 2)).astype(np.int8 if prec == "int8" else np.float32)
    vis = {}
    with Plan(make_config(n_tiles, L=L, T=T, xprec=prec, max_samples=L * T)) as p:
        d = torch.from_numpy(x).cuda()
        for how in ("tri", "tile_bl", "raw" if prec == "int8" else "tri"):
            p.load_channelised(d)
            p.correlate()
            vis[how] = (p.integrate_raw(1)[0] if how == "raw" else p.integrate(1, order=how)).cpu().numpy()[0]
    ref = oracle.correlate_i64(x.astype(np.int8), T)[0]
    tri = vis["tri"]
    assert np.array_equal(tri, (ref[..., 0] + 1j * ref[..., 1]).astype(np.complex64))    # sums below 2^24 are exact
    if prec == "int8":
        assert np.array_equal(vis["raw"], ref)
    bl = 0
    for a in range(n_tiles):
        for b in range(a + 1):
            for q in range(4):
                r, s = 2 * a + q // 2, 2 * b + q % 2
                want = tri[:, mwax.pair_index(r, s)] if r >= s else np.conj(tri[:, mwax.pair_index(s, r)])
                assert np.array_equal(vis["tile_bl"][bl, :, q], want)
            bl += 1


@pytest.mark.parametrize("n_tiles,L", [(120, 64), (120, 128)])
def test_raw_with_several_channels_per_thread(n_tiles, L):
    # 113 x L / 2048 channels to a thread (3 and 7), the last run of them ragged
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, T = 2 * n_tiles, 3
    rng = np.random.default_rng(L)
    x = rng.integers(-127, 128, size=(T, L, n, 2)).astype(np.int8)
    s = (1.0 + rng.random(L)).astype(np.float32)
    with Plan(make_config(n_tiles, L=L, T=T, xprec="int8", max_samples=L * T)) as p:
        p.set_scales(s)
        p.load_channelised(torch.from_numpy(x).cuda())
        p.correlate()
        raw, sc = [t.cpu().numpy() for t in p.integrate_raw(1)]
        p.load_channelised(torch.from_numpy(x).cuda())
        p.correlate()
        tri = p.integrate(1).cpu().numpy()[0]
    assert np.array_equal(raw, oracle.correlate_i64(x, T)) and np.array_equal(sc[0], s)
    s2 = (s.astype(np.float64)[:, None, None]) * raw[0] * s.astype(np.float64)[:, None, None]
    assert np.allclose(tri, s2[..., 0] + 1j * s2[..., 1], rtol=2.0 ** -23, atol=0)


@pytest.mark.parametrize("prec", ["int8", "fp32"])
@pytest.mark.parametrize("n_tiles,L,F", [(1, 4, 2), (15, 32, 4), (33, 64, 1), (17, 64, 64)])
def test_emission_averaged_equals_average(prec, n_tiles, L, F):
    # sums below 2^24, exact also as the FP32 visibilities the oracle averages
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, T = 2 * n_tiles, 9
    rng = np.random.default_rng(n + F)
    x = rng.integers(-127, 128, size=(T, L, n, 2)).astype(np.int8)
    with Plan(make_config(n_tiles, L=L, T=T, xprec=prec, max_samples=L * T)) as p:
        p.load_channelised(torch.from_numpy(x.astype(np.int8 if prec == "int8" else np.float32)).cuda())
        p.correlate()
        got = p.integrate_averaged(F, 1).cpu().numpy()
    ref = oracle.correlate_i64(x, T).astype(np.float64)
    want = oracle.fscrunch(ref[..., 0] + 1j * ref[..., 1], F)
    assert got.shape == want.shape
    assert np.all(np.abs(got.real - want.real) <= 2.0 ** -24 * np.abs(want.real))
    assert np.all(np.abs(got.imag - want.imag) <= 2.0 ** -24 * np.abs(want.imag))
