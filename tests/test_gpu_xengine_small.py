"""X-engine of small arrays (32 x 32 blocks, a workgroup's waves sharing the K
loop) and of averages with few output channels, at the edges of their stages
(8 row groups: 128 INT8 or 64 FP16 spectra), slices (8 stages) and wave counts.

INT8 sums are equal to the integer oracle.  FP16: products of binary16 values are
exact in FP32 and a chain has at most n / 8 + 16 roundings of 2^-24 of the running
sum over n spectra, random in sign: sqrt(n / 8 + 16) 2^-24 < 2e-6 for n < 8,000.
"""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2303_11557_amd import mwax  # noqa: E402
from paper_2303_11557_amd.mwax import Batch, Plan, make_config  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    mwax.lib()
    yield


@pytest.mark.parametrize("prec", ["int8", "fp16"])
@pytest.mark.parametrize("n_tiles,L,T,split", [
    (1, 2, 1, 1),           # one spectrum
    (16, 2, 64, 1),         # 32 inputs: one whole block, one (half an INT8) stage
    (17, 4, 65, 2),         # 34 inputs: three blocks, one ragged; segments that store, then add
    (32, 2, 200, 1),        # 64 inputs: two (four) stages
    (3, 512, 500, 1),       # many channels: as few waves as stages
    (20, 256, 1100, 2),     # many channels: fewer waves than slices
    (32, 1, 2100, 1),       # eight waves, more stages than slices, ragged end
])
def test_small_arrays(prec, n_tiles, L, T, split):
    n = 2 * n_tiles
    rng = np.random.default_rng(n * 7 + T)
    ints = 3                # device slots are reused without being cleared
    if prec == "int8":
        x = rng.integers(-127, 128, size=(ints * T, L, n, 2)).astype(np.int8)
    else:
        x = (rng.normal(size=(ints * T, L, n, 2)) * 100.0).astype(np.float16)
    cuts = [0, T // 2, T] if split == 2 else [0, T]
    got = []
    with Plan(make_config(n_tiles, L=L, T=T, xprec=prec, max_samples=L * T)) as p:
        d = torch.from_numpy(x).cuda()
        for j in range(ints):
            for a, b in zip(cuts, cuts[1:]):
                p.load_channelised(d[j * T + a:j * T + b])
                p.correlate()
            out = p.integrate_raw(1)[0] if prec == "int8" else p.integrate(1)
            got.append(out.cpu().numpy())
    got = np.concatenate(got)
    if prec == "int8":
        assert np.array_equal(got, oracle.correlate_i64(x, T))
        return
    x = x.astype(np.float64)
    ref = oracle.correlate(x[..., 0] + 1j * x[..., 1], T)
    got = got * 2.0 ** (-2 * ((int(np.log2(L)) + 1) // 2))
    err = np.linalg.norm(got - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
    assert err.max() < 2e-6, err.max()


def test_small_batch_instances_equal_plans_of_their_own():
    # the number of waves that share a block differs between the two; the sums must not
    S = 32768
    shapes = [(16, 16, 2048), (32, 32, 700), (1, 64, 100), (9, 512, 64), (31, 1024, 32), (40, 32, 300)]
    cfgs = [make_config(t, L=L, T=T, xprec="fp16", max_samples=S) for t, L, T in shapes]
    volts = [torch.from_numpy(synth.gaussian_volts(2 * t, S, seed=40 + i)).cuda()
             for i, (t, _, _) in enumerate(shapes)]
    with Batch(cfgs) as b:
        b.run(volts)
        got = [p.integrate(64).cpu().numpy() for p in b.plans]
        b.sync()
    for c, v, g in zip(cfgs, volts, got):
        with Plan(c) as p:
            p.channelise(v)
            p.correlate()
            want = p.integrate(64).cpu().numpy()
        assert want.shape[0] >= 1 and np.array_equal(g, want)


@pytest.mark.parametrize("prec", ["int8", "fp16"])
@pytest.mark.parametrize("n_tiles,L,F,T", [
    (3, 16, 2, 1100),       # units of 64 row groups with a ragged last one; the centre channel
    (17, 32, 32, 300),      # one output channel over the whole band
    (33, 64, 4, 129),       # 66 inputs: six blocks, ragged
    (4, 512, 2, 70),        # one 64-edge workgroup per CU: the other kernel
])
def test_averages_of_few_output_channels(prec, n_tiles, L, F, T):
    n = 2 * n_tiles
    S = 2 * T * L           # one call: two segments
    v = torch.from_numpy(synth.gaussian_volts(n, S, seed=n + F, sources=[synth.Source(4.0, L // 5)], L=L)).cuda()
    cfg = make_config(n_tiles, L=L, T=T, xprec=prec, max_samples=S)
    outs = []
    for f in (1, F):
        with Plan(cfg) as p:
            if f > 1:
                p.set_averaging(f)
            p.channelise(v)
            p.correlate()
            if f == 1 and prec == "int8":
                raw, sc = [x.cpu().numpy().astype(np.float64) for x in p.integrate_raw(2)]
                outs.append((raw[..., 0] + 1j * raw[..., 1]) * (sc ** 2)[:, :, None])
            else:
                outs.append(p.integrate(2).cpu().numpy().astype(np.complex128))
    want = oracle.fscrunch(outs[0], F)
    assert outs[1].shape == want.shape == (2, L // F, n * (n + 1) // 2)
    err = np.linalg.norm(outs[1] - want, axis=-1) / np.linalg.norm(want, axis=-1)
    assert err.max() < max(2e-6, (F + 1) * 2.0 ** -24)
