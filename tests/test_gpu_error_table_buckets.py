"""Both ways the error table finds a 4-bit code (one threshold per bucket of [-1, 1]; bisection where a bucket holds two,
or a threshold lies above every ordinary normalised weight), and threshold averaging over several passes of its loop."""
import numpy as np
import pytest
import torch

from oracle import lowra_oracle as orc
from paper_2502_08141_amd import lowra, synth

pytestmark = pytest.mark.gpu

TABLES = {
    "spread": np.linspace(-0.93, 0.93, 15),
    "on the edges of buckets": (np.arange(15) - 7) / 8.0,
    "two in one bucket": np.concatenate([[-0.9, -0.899], np.linspace(-0.7, 0.9, 13)]),
    "equal neighbours": np.concatenate([[-0.5, -0.5, -0.5], np.linspace(-0.4, 0.9, 12)]),
    "below -1": np.concatenate([[-3.0], np.linspace(-0.8, 0.8, 14)]),
    "above 1": np.concatenate([np.linspace(-0.8, 0.8, 12), [1.0, 2.0, np.inf]]),
}


@pytest.mark.parametrize("name", list(TABLES))
@pytest.mark.parametrize("N,K", [(1, 64), (5, 4160), (3, 4032), (1, 4096), (2049, 4096)])   # bisection below 4096 features; pairs from 2048 channels
def test_error_table(name, N, K):
    print(f"[error table {name} {N}x{K}]", flush=True)
    thr, mp, _ = synth.shared_codebooks()
    thr = thr.copy()
    thr[2, :15] = TABLES[name].astype(np.float32)
    W = np.random.default_rng(N * K).normal(0, 0.02, (N, K)).astype(np.float32)
    edges = np.concatenate([thr[2, :15][np.abs(thr[2, :15]) <= 1], [-1.0, 1.0, 0.0, 0.03125, -0.03125]]).astype(np.float32)
    W[0, :edges.size] = edges                                 # a block whose absmax is 1: weights on thresholds and bucket edges
    W[0, edges.size:64] = 0.5
    if N > 2:
        W[2, :64] = 1e-41                                     # subnormal block: 1 / absmax is infinite
        W[2, 64:128] = 0.0
    got = lowra.lowra_channel_mse(torch.from_numpy(W).cuda(), torch.from_numpy(thr).cuda(), torch.from_numpy(mp).cuda())
    want = orc.channel_mse(W, thr, mp)
    assert np.allclose(got.cpu().numpy(), want, rtol=1e-5, atol=0)   # fp32 partial sums per thread against fp64


@pytest.mark.parametrize("seed", range(3))
def test_thresholds_out_of_order(seed):
    """A violated precondition: any code below 16 would do, and it is the one that the bisection ends at."""
    rng = np.random.default_rng(seed)
    thr, mp, _ = synth.shared_codebooks()
    thr = thr.copy()
    T = np.linspace(-0.93, 0.93, 15).astype(np.float32)       # one to a bucket
    T = rng.permutation(T) if seed else np.concatenate([T[:2], T[9:10], T[3:9], T[2:3], T[10:]])
    thr[2, :15] = T
    W = rng.normal(0, 0.02, (7, 640)).astype(np.float32)
    got = lowra.lowra_channel_mse(torch.from_numpy(W).cuda(), torch.from_numpy(thr).cuda(), torch.from_numpy(mp).cuda()).cpu().numpy()
    a = np.abs(W.reshape(7, 10, 64)).max(axis=2).repeat(64, axis=1)
    u = W * (np.float32(1) / a)
    c = np.zeros(W.shape, np.int64)
    for at in (lambda c: 8 * c + 7, lambda c: 8 * c + 3, lambda c: 4 * c + 1, lambda c: 2 * c):   # the code's bits from the top
        c = 2 * c + (T[at(c)] < u)
    want = np.square((W - mp[2][c] * a).astype(np.float64)).mean(axis=1)
    assert np.allclose(got[:, 2], want, rtol=1e-5, atol=0)


def test_decoded_weights_have_no_error():
    """Weights that are already decoded values (level times absmax, rounded to fp32) quantize to themselves: the error at
    their own width is exactly zero, so that an assignment of widths gains nothing by a wider one."""
    thr, mp, _ = synth.shared_codebooks()
    thr, mp = thr.copy(), mp.copy()
    rng = np.random.default_rng(3)
    for p, b in enumerate((1, 2, 4)):
        lv = np.linspace(-1, 1, 1 << b) * np.where(np.abs(np.linspace(-1, 1, 1 << b)) == 1, 1, 1 + 0.02 * rng.normal(size=1 << b))
        mp[p, :1 << b] = lv
        thr[p, :(1 << b) - 1] = (lv[1:] + lv[:-1]) / 2
        code = rng.integers(0, 1 << b, (37, 320))
        code[:, ::64] = 0                                     # level -1 in every block: its absmax is the scale itself
        a = rng.uniform(0.01, 0.1, (37, 5)).astype(np.float32).repeat(64, axis=1)
        W = mp[p][code] * a
        assert W.dtype == np.float32
        got = lowra.lowra_channel_mse(torch.from_numpy(W).cuda(), torch.from_numpy(thr).cuda(), torch.from_numpy(mp).cuda()).cpu()
        assert not got[:, p].any(), f"{b} bits: {got[:, p].max()}"


@pytest.mark.parametrize("fractions", [(0.4, 0.3, 0.3), (0.5, 0.5, 0.0), (1.0, 0.0, 0.0), (0.0, 0.0, 1.0)])
def test_average_thresholds_many_channels(fractions):
    N = 13001                                                 # past the 12288 channels of one pass
    bits = synth.assign_bits(N, fractions, np.random.default_rng(5))
    thr = np.sort(np.random.default_rng(6).uniform(-1, 1, (N, 16)).astype(np.float32), axis=1)
    thr[np.arange(16)[None, :] >= (1 << bits.astype(np.int64))[:, None] - 1] = np.inf
    lay = lowra.Layout(64, bits, np.arange(N, dtype=np.int32), bits)
    got = lowra.lowra_average_thresholds(lay, torch.from_numpy(thr).cuda()).cpu().numpy()
    want = orc.average_thresholds(bits, thr)
    fin = np.isfinite(want)
    assert np.array_equal(np.isfinite(got), fin) and np.abs(got[fin] - want[fin]).max() <= 2.0 ** -24   # both sums are fp64
