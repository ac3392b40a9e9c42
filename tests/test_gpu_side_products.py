"""The rank-r products of few tokens: contraction split between workgroups (with and without room for it), and B [N, r]
read in place at ranks below 64.  Checked where a caller sees them: in the workspaces of the two linear calls, against
fp64 products of the same bf16 inputs -- one rounding to bf16 (2^-9 relative, 2^-8 with the fp32 sum's share to spare)
of sums of up to 11008 products."""
import pytest
import torch

from paper_2502_08141_amd import lowra, synth
from tests.gpu_util import DeviceLayer

pytestmark = pytest.mark.gpu


def rel(got, want):
    rms = want.square().mean().sqrt()
    return ((got.double() - want).abs() / torch.maximum(want.abs(), rms)).max().item()


@pytest.mark.parametrize("N,K,M,r", [(1544, 1600, 17, 64), (4096, 1536, 100, 8), (11008, 64 * 25, 33, 16), (264, 4160, 333, 40),
                                     (1600, 2048, 700, 32), (1544, 1600, 40, 5), (2056, 1088, 2050, 56)])
def test_side_products(N, K, M, r):
    print(f"[side {N}x{K} M{M} r{r}]", flush=True)
    D = DeviceLayer(synth.make_custom(N, K, M, r, fractions=(0.5, 0.5, 0.0), seed=810 + r))
    D.quantize()
    L = D.L
    want = {lowra.OP_LINEAR_FWD: L.s * (D.x.double() @ D.A.double().T), lowra.OP_LINEAR_BWD_INPUT: L.s * (D.dY.double() @ D.B.double())}
    for op, w in want.items():
        full = D.layout.workspace_bytes(op, M, r)
        call = lowra.lowra_linear_fwd if op == lowra.OP_LINEAR_FWD else lowra.lowra_linear_bwd_input
        act = D.x if op == lowra.OP_LINEAR_FWD else D.dY
        for size in (full, full + 4096):
            ws = torch.full((size,), 0xff, dtype=torch.uint8, device="cuda")          # NaN in every format: nothing may be read before it is written
            out = call(D.layout, D.packed, D.absmax, D.mp, act, D.A, D.B, L.s, workspace=ws)
            side = lowra.lowra_linear_side_product(D.layout, op, M, r, ws)
            assert rel(side[:, :r], w) <= 2.0 ** -8
            assert not side[:, r:].any() and torch.isfinite(out.float()).all()
    dA, dB = lowra.lowra_adapter_grads(D.layout, D.x, D.dY, D.A, D.B, L.s)
    assert rel(dB, D.dY.double().T @ want[lowra.OP_LINEAR_FWD]) <= 2e-2 and rel(dA, want[lowra.OP_LINEAR_BWD_INPUT].T @ D.x.double()) <= 2e-2


@pytest.mark.parametrize("N,K,M,r", [(1536, 1536, 1300, 64), (1536, 2048, 700, 32), (1800, 1600, 500, 24), (4096, 1536, 20, 64)])
def test_adapter_gradients_form_the_same_products(N, K, M, r):
    """Where the contraction is split, the standalone call has the room to split it as the linear calls do: same bits."""
    print(f"[side grads {N}x{K} M{M} r{r}]", flush=True)
    D = DeviceLayer(synth.make_custom(N, K, M, r, fractions=(0.5, 0.5, 0.0), seed=830 + r))
    D.quantize()
    L, side = D.L, []
    for op, call, act in ((lowra.OP_LINEAR_FWD, lowra.lowra_linear_fwd, D.x), (lowra.OP_LINEAR_BWD_INPUT, lowra.lowra_linear_bwd_input, D.dY)):
        ws = torch.empty(D.layout.workspace_bytes(op, M, r), dtype=torch.uint8, device="cuda")
        call(D.layout, D.packed, D.absmax, D.mp, act, D.A, D.B, L.s, workspace=ws)
        side.append(lowra.lowra_linear_side_product(D.layout, op, M, r, ws))
    dA, dB = lowra.lowra_adapter_grads_from_side(D.layout, D.x, D.dY, r, *side)
    rA, rB = lowra.lowra_adapter_grads(D.layout, D.x, D.dY, D.A, D.B, L.s)
    assert torch.equal(dA, rA) and torch.equal(dB, rB)
