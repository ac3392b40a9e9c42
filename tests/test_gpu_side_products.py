"""The rank-r products of few tokens: contraction split between workgroups, and B [N, r] read in place at ranks below 64.
Checked where a caller sees them: in the workspaces of the two linear calls, the reported size and the smallest that is
accepted, against fp64 products of the same bf16 inputs -- one rounding to bf16 (2^-9 relative, 2^-8 with the fp32 sum's
share to spare) of sums of up to 11008 products."""
import pytest
import torch

from paper_2502_08141_amd import lowra, synth
from tests.gpu_util import DeviceLayer

pytestmark = pytest.mark.gpu


def rel(got, want):
    rms = want.square().mean().sqrt()
    return ((got.double() - want).abs() / torch.maximum(want.abs(), rms)).max().item()


def least_workspace(call, most):
    """The smallest workspace that `call` takes, found by its refusals (which launch nothing)."""
    lo, hi = 0, most                                          # in bytes: lo is refused, hi is taken
    while hi - lo > 256:
        mid = (lo + hi) // 512 * 256
        try:
            call(torch.empty(mid, dtype=torch.uint8, device="cuda"))
            hi = mid
        except lowra.LowraError as e:
            assert e.status in (lowra.WORKSPACE_TOO_SMALL, lowra.INVALID_ARG)
            lo = mid
    return hi


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
        for size in (full, least_workspace(lambda ws: call(D.layout, D.packed, D.absmax, D.mp, act, D.A, D.B, L.s, workspace=ws), full)):
            ws = torch.full((size,), 0xff, dtype=torch.uint8, device="cuda")          # NaN in every format: nothing may be read before it is written
            out = call(D.layout, D.packed, D.absmax, D.mp, act, D.A, D.B, L.s, workspace=ws)
            side = lowra.lowra_linear_side_product(D.layout, op, M, r, ws)
            assert rel(side[:, :r], w) <= 2.0 ** -8
            assert not side[:, r:].any() and torch.isfinite(out.float()).all()
    dA, dB = lowra.lowra_adapter_grads(D.layout, D.x, D.dY, D.A, D.B, L.s)
    assert rel(dB, D.dY.double().T @ want[lowra.OP_LINEAR_FWD]) <= 2e-2 and rel(dA, want[lowra.OP_LINEAR_BWD_INPUT].T @ D.x.double()) <= 2e-2


@pytest.mark.parametrize("N,K,M,r,path", [(1536, 1536, 1300, 64, lowra.PATH_AUTO), (1536, 2048, 700, 32, lowra.PATH_AUTO),
                                          (1800, 1600, 500, 24, lowra.PATH_AUTO), (4096, 1536, 20, 64, lowra.PATH_AUTO),
                                          (136, 4096, 40, 16, lowra.PATH_AUTO), (264, 1600, 300, 64, lowra.PATH_AUTO), (8, 9024, 37, 24, lowra.PATH_AUTO),
                                          (1544, 2112, 9, 64, lowra.PATH_GEMM), (4096, 1536, 16, 8, lowra.PATH_GEMM),
                                          (1536, 4096, 1, 5, lowra.PATH_GEMM)])
def test_adapter_gradients_form_the_same_products(N, K, M, r, path):
    """The split of the contraction follows from the shape: the linear calls, whatever workspace they have, and the
    standalone gradients form the same bits, for every token count whose intermediate a caller can get."""
    print(f"[side grads {N}x{K} M{M} r{r} path {path}]", flush=True)
    D = DeviceLayer(synth.make_custom(N, K, M, r, fractions=(0.5, 0.5, 0.0), seed=830 + r))
    D.quantize()
    L = D.L
    lowra.lowra_set_linear_path(path)
    try:
        rA, rB = lowra.lowra_adapter_grads(D.layout, D.x, D.dY, D.A, D.B, L.s)
        for least in (False, True):
            side = []
            for op, call, act in ((lowra.OP_LINEAR_FWD, lowra.lowra_linear_fwd, D.x), (lowra.OP_LINEAR_BWD_INPUT, lowra.lowra_linear_bwd_input, D.dY)):
                run = lambda ws: call(D.layout, D.packed, D.absmax, D.mp, act, D.A, D.B, L.s, workspace=ws)
                size = D.layout.workspace_bytes(op, M, r)
                ws = torch.empty(least_workspace(run, size) if least else size, dtype=torch.uint8, device="cuda")
                run(ws)
                side.append(lowra.lowra_linear_side_product(D.layout, op, M, r, ws))
            dA, dB = lowra.lowra_adapter_grads_from_side(D.layout, D.x, D.dY, r, *side)
            assert torch.equal(dA, rA) and torch.equal(dB, rB), f"least workspace: {least}"
    finally:
        lowra.lowra_set_linear_path(lowra.PATH_AUTO)


@pytest.mark.parametrize("N,K,M,r", [(264, 1600, 40, 8), (264, 4160, 333, 40), (1600, 2048, 700, 24), (264, 1024, 1200, 5)])
def test_infinite_activations_stay_in_their_ranks(N, K, M, r):
    """What fills the intermediate up to 64 ranks is zero whatever the activations hold: zeros of A or B times an infinity are none."""
    D = DeviceLayer(synth.make_custom(N, K, M, r, fractions=(0.5, 0.5, 0.0), seed=850 + r))
    D.quantize()
    What = lowra.lowra_dequantize(D.layout, D.packed, D.absmax, D.mp)
    for op, call, act, W in ((lowra.OP_LINEAR_FWD, lowra.lowra_linear_fwd, D.x, What), (lowra.OP_LINEAR_BWD_INPUT, lowra.lowra_linear_bwd_input, D.dY, What.T)):
        a, A, B = act.clone(), D.A.clone(), D.B.clone()
        a[1, 3] = float("inf")
        sign = torch.sign(W[:, 3]).bfloat16()                # a rank-r term of the weights' signs
        assert (sign != 0).all()
        if op == lowra.OP_LINEAR_FWD:
            A[:, 3], B[:] = 1.0, sign[:, None]
        else:
            B[3], A[:] = 1.0, sign
        full = D.layout.workspace_bytes(op, M, r)
        run = lambda ws: call(D.layout, D.packed, D.absmax, D.mp, a, A, B, 1.0, workspace=ws)
        for size in (full, least_workspace(run, full)):
            ws = torch.full((size,), 0xff, dtype=torch.uint8, device="cuda")
            out = run(ws).float()
            side = lowra.lowra_linear_side_product(D.layout, op, M, r, ws)
            assert torch.isposinf(side[1, :r]).all() and not side[:, r:].any()
            assert torch.equal(out[1], sign.float() * float("inf"))
            assert torch.isfinite(out[0]).all() and torch.isfinite(out[2:]).all()


@pytest.mark.parametrize("N,K,M,r", [(264, 1088, 33, 64), (264, 4096, 20, 8), (4096, 1088, 20, 64), (2048, 4096, 17, 16), (1536, 4096, 1, 8),
                                     (264, 1600, 1024, 8), (264, 1600, 1025, 8)])
def test_both_products_in_one_launch(N, K, M, r):
    """Neither, one and both of the two contractions split between workgroups, with the fewest tokens, the most that share a
    launch and one more: the same bits as the products of the linear calls, from a workspace of NaN."""
    test_adapter_gradients_form_the_same_products(N, K, M, r, lowra.PATH_GEMM)
    D = DeviceLayer(synth.make_custom(N, K, M, r, fractions=(0.5, 0.5, 0.0), seed=830 + r))
    ws = torch.full((D.layout.workspace_bytes(lowra.OP_ADAPTER_GRADS, M, r),), 0xff, dtype=torch.uint8, device="cuda")
    got = lowra.lowra_adapter_grads(D.layout, D.x, D.dY, D.A, D.B, D.L.s, workspace=ws)
    want = lowra.lowra_adapter_grads(D.layout, D.x, D.dY, D.A, D.B, D.L.s)
    assert all(torch.equal(a, b) and torch.isfinite(a).all() for a, b in zip(got, want))
