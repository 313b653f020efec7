"""FP32 X-engine on the matrix cores against the FP64 oracle, at the edges of its
two kernels: 32 x 32 blocks with the K loop shared by eight waves (small
launches) and 64 x 64 tiles (at least four per CU).

Tolerance: the FP32 sums are chains of at most 32 + 128 roundings of 2^-24 of
the running sum, random in sign; sqrt(160) 2^-24 = 7.5e-7, so 2e-6 relative
Frobenius per channel.
"""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2303_11557_amd import mwax  # noqa: E402
from paper_2303_11557_amd.mwax import Plan, make_config  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    mwax.lib()
    yield


@pytest.mark.parametrize("n_tiles,L,T,split", [
    (1, 4, 1, 1),                  # one spectrum: one row group of one wave
    (17, 2, 130, 1),               # 34 inputs: a block of two; more stages than waves
    (16, 1, 16 * 128 * 8 + 37, 1),   # 32 inputs: past a wave's FP64 collection, ragged end
    (1, 1024, 2048 + 17, 1),       # 64 x 64 tiles, past the flush of the outer sums
    (33, 512, 37, 2),              # 66 inputs: a ragged tile; segments that store, then add
    (64, 512, 16, 1),              # 128 inputs: whole tiles, one whole stage
])
def test_matrix_core_fp32(n_tiles, L, T, split):
    n = 2 * n_tiles
    rng = np.random.default_rng(n * 5 + T)
    ints = 3                       # device slots are reused without being cleared
    x = (rng.normal(size=(ints * T, L, n, 2)) * 100.0).astype(np.float32)
    cuts = [0, T // 2, T] if split == 2 else [0, T]
    got = []
    with Plan(make_config(n_tiles, L=L, T=T, xprec="fp32", max_samples=L * T)) as p:
        d = torch.from_numpy(x).cuda()
        for j in range(ints):
            for a, b in zip(cuts, cuts[1:]):
                p.load_channelised(d[j * T + a:j * T + b])
                p.correlate()
            got.append(p.integrate(1).cpu().numpy().astype(np.complex128))
    got = np.concatenate(got)
    ref = oracle.correlate(x[..., 0].astype(np.float64) + 1j * x[..., 1], T)
    err = np.linalg.norm(got - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
    assert got.shape == ref.shape and err.max() < 2e-6, err.max()


@pytest.mark.parametrize("n_tiles", [116, 130])
def test_matrix_core_fp32_many_tiles(n_tiles):
    # 8 and 9 blocks of 32 along an edge, more than four workgroups per CU: four diagonal
    # tiles dealt to three workgroups; an odd last row of blocks
    n, L, T = 2 * n_tiles, 128, 33
    rng = np.random.default_rng(n)
    x = (rng.normal(size=(T, L, n, 2)) * 100.0).astype(np.float32)
    with Plan(make_config(n_tiles, L=L, T=T, xprec="fp32", max_samples=L * T)) as p:
        p.load_channelised(torch.from_numpy(x).cuda())
        p.correlate()
        got = p.integrate(1).cpu().numpy().astype(np.complex128)
    ref = oracle.correlate(x[..., 0].astype(np.float64) + 1j * x[..., 1], T)
    err = np.linalg.norm(got - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
    assert got.shape == ref.shape and err.max() < 2e-6, err.max()
