"""Calls that span more integrations than one X-engine launch works on (eight
segments): FP32, small-array and averaging plans.  INT8 sums are equal to the
integer oracle; FP32 and binary16 ones within 2e-6 of the FP64 oracle (chains of a
few roundings of 2^-24), averages within one rounding per weighted term.
"""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2303_11557_amd import mwax  # noqa: E402
from paper_2303_11557_amd.mwax import Plan, make_config  # noqa: E402


@pytest.mark.parametrize("prec,n_tiles,F", [
    ("fp32", 3, 1), ("fp32", 40, 1),                    # both kernels' tile forms
    ("int8", 3, 1), ("fp16", 17, 1), ("int8", 32, 1),   # small arrays: one and three blocks
    ("int8", 20, 4), ("fp16", 40, 4),                   # averages
])
def test_twenty_segments_in_a_call(prec, n_tiles, F):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, L, T, ints = 2 * n_tiles, 16, 5, 20
    rng = np.random.default_rng(n + F)
    if prec == "int8":
        x = rng.integers(-127, 128, size=(ints * T, L, n, 2)).astype(np.int8)
    else:
        x = (rng.normal(size=(ints * T, L, n, 2)) * 30.0).astype(np.float16 if prec == "fp16" else np.float32)
    got = []
    with Plan(make_config(n_tiles, L=L, T=T, xprec=prec, max_samples=L * 94)) as p:
        if F > 1:
            p.set_averaging(F)
        d = torch.from_numpy(x).cuda()
        for a, b in ((0, 3), (3, 97), (97, 100)):       # 2 + 18 x 5 + 2 spectra in the second
            p.load_channelised(d[a:b])
            p.correlate()
            out = p.integrate_raw(ints)[0] if prec == "int8" and F == 1 else p.integrate(ints)
            got.append(out.cpu().numpy())
    assert [g.shape[0] for g in got] == [0, 19, 1]
    got = np.concatenate(got)
    if prec == "int8" and F == 1:
        assert np.array_equal(got, oracle.correlate_i64(x, T))
        return
    x = x.astype(np.float64)
    ref = oracle.correlate(x[..., 0] + 1j * x[..., 1], T) * (16.0 if prec == "fp16" else 1.0)   # 2^(2 e), e = 2
    if F > 1:
        ref = oracle.fscrunch(ref, F)
    err = np.linalg.norm(got - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
    assert got.shape == ref.shape and err.max() < 2e-6, err.max()
