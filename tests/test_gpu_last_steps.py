"""Contractions that end inside a step: of 64 channels or features in the 256-column GEMMs, of 64 tokens in the adapter gradients."""
import pytest
import torch

from paper_2502_08141_amd import lowra, synth
from tests.gpu_util import DeviceLayer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K,M", [(8, 64, 40), (72, 320, 300), (584, 512, 40), (1096, 1088, 260)])
@pytest.mark.parametrize("fr", [(0.5, 0.5, 0.0), (0.4, 0.3, 0.3)])
@pytest.mark.parametrize("r", [0, 8])
def test_infinite_activations_in_the_last_step(N, K, M, fr, r):
    """256-column kernels, a last step that is not full: an infinity in a token's last features (input gradient: channels) makes
    its outputs infinite, of the weight's sign, and no other token's.  The rank-r term has the same sign."""
    print(f"[inf {N}x{K} M{M} r{r} {fr}]", flush=True)
    D = DeviceLayer(synth.make_custom(N, K, M, max(r, 1), fractions=fr, seed=910 + N))
    D.quantize()
    What = lowra.lowra_dequantize(D.layout, D.packed, D.absmax, D.mp)
    lowra.lowra_set_linear_path(lowra.PATH_GEMM)
    try:
        for call, act, W, fwd in ((lowra.lowra_linear_fwd, D.x, What, True), (lowra.lowra_linear_bwd_input, D.dY, What.T, False)):
            for at in (act.shape[1] - 1, act.shape[1] - 8, 3):
                a, A, B = act.clone(), None, None
                a[1, at] = float("inf")
                sign = torch.sign(W[:, at])
                assert (sign != 0).all()
                if r:
                    A, B = D.A.clone(), D.B.clone()
                    if fwd:
                        A[:, at], B[:] = 1.0, sign[:, None]
                    else:
                        B[at], A[:] = 1.0, sign
                out = call(D.layout, D.packed, D.absmax, D.mp, a, A, B, 1.0).float()
                assert torch.equal(out[1], sign.float() * float("inf")), (fwd, at)
                assert torch.isfinite(out[0]).all() and torch.isfinite(out[2:]).all(), (fwd, at)
    finally:
        lowra.lowra_set_linear_path(lowra.PATH_AUTO)


@pytest.mark.parametrize("N,K,M,r", [(40, 1088, 1, 5), (264, 1600, 17, 64), (8, 64, 65, 8), (136, 4096, 300, 24), (1544, 1088, 2100, 64)])
def test_infinite_activations_of_the_last_token(N, K, M, r):
    """Adapter gradients: an infinity in the last token's features or channels makes the gradients of that feature or channel
    infinite, of the rank-r intermediate's sign, and no other; likewise one in the intermediate, for its rank."""
    print(f"[inf token {N}x{K} M{M} r{r}]", flush=True)
    D = DeviceLayer(synth.make_custom(N, K, M, r, fractions=(0.5, 0.5, 0.0), seed=920 + r))
    gen = torch.Generator(device="cuda").manual_seed(M)
    side = [torch.randn(M, 64, generator=gen, device="cuda").bfloat16() for _ in range(2)]
    for s in side:
        s[:, r:] = 0
        assert (s[-1, :r] != 0).all()
    inf = float("inf")
    grads = lambda x=D.x, dY=D.dY, st=side[0], su=side[1]: lowra.lowra_adapter_grads_from_side(D.layout, x, dY, r, st, su)
    for hit in ("x", "dY", "st", "su"):
        t = {"x": D.x, "dY": D.dY, "st": side[0], "su": side[1]}[hit].clone()
        at = r - 1 if hit in ("st", "su") else t.shape[1] - 1
        t[-1, at] = inf
        dA, dB = grads(**{hit: t})
        other = {"x": side[1][-1, :r], "dY": side[0][-1, :r], "st": D.dY[-1], "su": D.x[-1]}[hit].float()
        g, rest = (dA, dB) if hit in ("x", "su") else (dB.T, dA)         # [r, features or channels]
        line, keep = (g[:, at], g[:, :at]) if hit in ("x", "dY") else (g[at], g[:at])
        nz = other != 0
        assert torch.equal(line[nz], (other.sign() * inf)[nz]), hit
        assert torch.isfinite(keep).all() and torch.isfinite(rest).all(), hit
