"""The calls that csrc/call.cpp makes without Python: the same bits as through lowra.py's own checks, and for everything but
plain tensors those checks and what they raise."""
import pytest
import torch
from torch.overrides import TorchFunctionMode

from paper_2502_08141_amd import lowra, synth
from tests.gpu_util import DeviceLayer

pytestmark = pytest.mark.gpu


class _Sub(torch.Tensor):
    pass


class _Mode(TorchFunctionMode):
    seen = 0

    def __torch_function__(self, func, types, args=(), kwargs=None):
        _Mode.seen += 1
        return func(*args, **(kwargs or {}))


def _layer(M, r, bf16_scales):
    D = DeviceLayer(synth.make_custom(264, 576, M, max(r, 1), fractions=(0.4, 0.3, 0.3), seed=31 + M))
    if bf16_scales:
        D.layout.set_scale_dtype(torch.bfloat16)
    packed, absmax = lowra.lowra_quantize(D.layout, D.W, D.thr)
    ws = {op: torch.empty(max(D.layout.workspace_bytes(op, M, max(r, 1)), 256), dtype=torch.uint8, device="cuda")
          for op in (lowra.OP_LINEAR_FWD, lowra.OP_LINEAR_BWD_INPUT, lowra.OP_ADAPTER_GRADS)}
    return D, packed, absmax, ws


@pytest.mark.parametrize("M,r,bf16_scales", [(1, 8, False), (16, 5, True), (40, 64, False), (40, 0, True), (0, 8, False)])
def test_same_results(M, r, bf16_scales, monkeypatch):
    D, packed, absmax, ws = _layer(M, r, bf16_scales)
    lay, s = D.layout, 1.5
    x, dY = D.x[:M].contiguous(), D.dY[:M].contiguous()
    A, B = (D.A, D.B) if r else (None, None)

    def run():
        out = [lowra.lowra_dequantize(lay, packed, absmax, D.mp),
               lowra.lowra_linear_fwd(lay, packed, absmax, D.mp, x, A, B, s, workspace=ws[0]),
               lowra.lowra_linear_bwd_input(lay, packed, absmax, D.mp, dY, A, B, s, workspace=ws[1])]
        if r:
            st, su = (lowra.lowra_linear_side_product(lay, op, M, r, ws[op]) for op in (0, 1))
            assert (st is None) == (M <= 16)
            out += list(lowra.lowra_adapter_grads(lay, x, dY, A, B, s, workspace=ws[2]))
            if st is not None and su is not None:
                out += [st.clone(), su.clone()]
                out += list(lowra.lowra_adapter_grads_from_side(lay, x, dY, r, st, su, workspace=ws[2]))
        torch.cuda.synchronize()
        return out

    native = run()
    with monkeypatch.context() as m:
        m.setattr(lowra, "_call", type("none", (), {k: staticmethod(lambda *a: None) for k in
                                                    ("linear", "grads", "grads_from_side", "side_product", "dequantize")}))
        plain = run()
    assert len(native) == len(plain)
    for a, b in zip(native, plain):
        assert a.dtype == b.dtype and a.shape == b.shape and a.device == b.device and not a.requires_grad
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


def test_everything_else_goes_through_the_checks():
    D, packed, absmax, ws = _layer(4, 8, False)
    lay = D.layout
    x = D.x[:4].contiguous()
    fwd = lambda x=x, A=D.A, B=D.B, s=1.0, ws=ws[0], lay=lay: lowra.lowra_linear_fwd(lay, packed, absmax, D.mp, x, A, B, s, workspace=ws)
    want = fwd()
    assert torch.equal(fwd(x=x.as_subclass(_Sub)), want) and torch.equal(fwd(s=1), want)
    with _Mode():
        assert torch.equal(fwd(), want) and _Mode.seen > 0    # a mode sees the allocation as before
    for bad, err in ((dict(x=x.float()), TypeError), (dict(x=x.cpu()), TypeError), (dict(x=x.t()), TypeError), (dict(x=x[:, :512].contiguous()), ValueError),
                     (dict(A=D.A[:4].contiguous()), ValueError), (dict(ws=ws[0][:16]), lowra.LowraError), (dict(ws=ws[0][1:]), lowra.LowraError)):
        with pytest.raises(err):
            fwd(**bad)
    with pytest.raises(ValueError):
        lowra.lowra_dequantize(lay, packed[:-1], absmax, D.mp)
    other = lowra.Layout(lay.K, lay.bits, lay.cb, lay.cb_bits)
    assert torch.equal(fwd(lay=other), want)
    other.close()
    with pytest.raises((lowra.LowraError, ValueError)):
        fwd(lay=other)
    torch.cuda.synchronize()
