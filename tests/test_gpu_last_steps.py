"""The 256-column GEMMs where the contraction ends inside a step of 64 channels or features."""
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
