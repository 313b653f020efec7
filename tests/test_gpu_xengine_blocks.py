"""The X-engine's division of the triangle into 64 x 64 blocks, four to a workgroup:
odd block counts (strips of the last row), diagonal tiles packed four to three
workgroups (long INT8 launches) and left alone (short and FP16 ones).

INT8 sums are equal to the integer oracle; FP16 within the rounding of FP32 chains
of T / 8 matrix steps: sqrt(T / 8) 2^-24 < 1e-6 for T up to 2,100.
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


@pytest.mark.parametrize("prec,n_tiles,L,T", [
    ("int8", 33, 2, 40),         # 66 inputs: one tile, its second block of two rows
    ("int8", 65, 2, 40),         # 3 blocks: one strip of two columns
    ("fp16", 93, 2, 40),         # 186 inputs, as above
    ("int8", 150, 1, 2100),      # 5 blocks: strips of three columns and of one; chunks
    ("fp16", 200, 1, 100),       # 7 blocks: strips of three, three tiles left alone
    ("int8", 256, 1, 40),        # 8 blocks, the diagonal tiles alone
    ("int8", 250, 1, 2100),      # 8 blocks, the diagonal tiles in one set; chunks
    ("int8", 260, 1, 2100),      # 9 blocks: a set, and strips
    ("fp16", 300, 1, 40),        # 10 blocks: five tiles
])
def test_division_into_blocks(prec, n_tiles, L, T):
    n = 2 * n_tiles
    rng = np.random.default_rng(n + T)
    if prec == "int8":
        x = rng.integers(-127, 128, size=(T, L, n, 2)).astype(np.int8)
    else:
        x = (rng.normal(size=(T, L, n, 2)) * 100.0).astype(np.float16)
    with Plan(make_config(n_tiles, L=L, T=T, xprec=prec, max_samples=L * T)) as p:
        p.load_channelised(torch.from_numpy(x).cuda())
        p.correlate()
        got = (p.integrate_raw(1)[0] if prec == "int8" else p.integrate(1)).cpu().numpy()
    if prec == "int8":
        assert np.array_equal(got, oracle.correlate_i64(x, T))
        return
    x = x.astype(np.float64)
    ref = oracle.correlate(x[..., 0] + 1j * x[..., 1], T)
    got = got * 2.0 ** (-2 * ((int(np.log2(L)) + 1) // 2))
    assert np.linalg.norm(got - ref) / np.linalg.norm(ref) < 2e-6


@pytest.mark.parametrize("T", [5000, 70000])
def test_chunks_add_into_reused_slots(T):
    # long segments of few workgroups: two or more chunks to a tile, added atomically
    # into slots that earlier integrations left uncleared (int32 and int64 sums)
    n_tiles, L, ints = 35, 1, 4
    n = 2 * n_tiles
    x = np.random.default_rng(T).integers(-127, 128, size=(T, L, n, 2)).astype(np.int8)
    x[-1, :, :, :] = 127
    got = []
    with Plan(make_config(n_tiles, L=L, T=T, xprec="int8", max_samples=L * T)) as p:
        d = torch.from_numpy(x).cuda()
        for j in range(ints):
            p.load_channelised(d if j % 2 == 0 else -d)          # the same sums
            p.correlate()
            got.append(p.integrate_raw(1)[0].cpu().numpy()[0])
    ref = oracle.correlate_i64(x, T)[0]
    for g in got:
        assert np.array_equal(g, ref)
