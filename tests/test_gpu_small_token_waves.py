"""The small-token forward where its instantiation changes: 4, 8 or 16 wavefronts of one block of 256 features each, t = x A^T
formed by the workgroups themselves (up to 16 ranks and 32768 entries of A) or summed from partial sums."""
import pytest
import torch

from oracle import lowra_oracle as orc
from paper_2502_08141_amd import lowra, synth
from tests.gpu_util import REL_TOL, DeviceLayer, bf16_host_f64, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,r", [(64, 8), (192, 16), (1024, 16), (1024, 17), (1088, 16), (2048, 16), (2048, 24), (2112, 15), (2112, 16), (4096, 8),
                                 (4096, 9), (4032, 3), (4160, 8), (1088, 64), (2048, 100)])
@pytest.mark.parametrize("M,N", [(1, 264), (3, 8), (16, 40)])
def test_wavefronts_and_ranks(K, r, M, N):
    _check(K, r, M, N)


# Where the choice of the instantiation changes: token counts around those whose buffers fit 16 wavefronts, t formed in the
# workgroup or not, and more strips of channels than compute units.
@pytest.mark.parametrize("K,r,M,N,plan", [(4096, 8, 14, 40, (16, 1, True)), (4096, 8, 15, 40, (16, 1, False)), (4096, 16, 16, 40, (16, 1, False)),
                                          (2112, 8, 13, 40, (16, 1, True)), (2048, 16, 16, 40, (8, 1, True)), (1024, 16, 15, 40, (4, 1, True)),
                                          (4160, 16, 7, 40, (16, 2, False)), (4160, 16, 8, 40, (16, 2, False)), (11008, 8, 8, 24, (16, 3, False)),
                                          (11008, 64, 9, 24, (8, 6, False)), (13824, 32, 15, 8, (8, 7, False)), (1088, 8, 3, 4200, (4, 2, False)), (1088, 8, 13, 4200, (8, 1, False)),
                                          (1088, 16, 16, 4200, (8, 1, False)), (512, 16, 14, 4200, (4, 1, True)), (2112, 16, 15, 4200, (16, 1, False))])
def test_instantiations(K, r, M, N, plan):
    assert lowra.lowra_plan_small_fwd(N, K, M, r) == plan
    _check(K, r, M, N)


def _check(K, r, M, N):
    print(f"[small K {K} r {r} M {M} N {N}]", flush=True)
    L = synth.make_custom(N, K, M, r, fractions=(0.4, 0.3, 0.3), seed=K % 89 + r)
    D = DeviceLayer(L)
    D.quantize()
    rp, ra = orc.quantize(L.W, L.bits, L.cb, L.thresholds)
    ref = orc.linear_fwd(rp, ra, L.bits, L.cb, L.mappings, L.x, L.A, L.B, L.s)
    got = lowra.lowra_linear_fwd(D.layout, D.packed, D.absmax, D.mp, D.x, D.A, D.B, L.s)
    batch = lowra.FwdBatch([(D.layout, D.packed, D.absmax, D.x, D.A, D.B)] * 2, D.mp, L.s) if K >= 256 else None
    torch.cuda.synchronize()
    assert rel_err(bf16_host_f64(got), ref) <= REL_TOL
    if batch is not None:
        for y in batch.run():
            torch.cuda.synchronize()
            assert rel_err(bf16_host_f64(y), ref) <= REL_TOL
        batch.close()


def test_an_infinite_adapter_entry_stays_in_its_rank():
    """Lanes past the last rank repeat its row of A; what they form must not reach the result."""
    L = synth.make_custom(40, 512, 2, 5, fractions=(0.4, 0.3, 0.3), seed=3)
    D = DeviceLayer(L)
    D.quantize()
    A, B = D.A.clone(), D.B.clone()
    A[4, 7] = float("inf")
    B[:, 4] = 1.0
    x = D.x.clone()
    x[:, 7] = 1.0
    got = lowra.lowra_linear_fwd(D.layout, D.packed, D.absmax, D.mp, x, A, B, 1.0).float()
    assert torch.isposinf(got).all()


@pytest.mark.parametrize("K", [64, 192, 320, 1088, 2112, 4160])
@pytest.mark.parametrize("r", [0, 8, 24])
@pytest.mark.parametrize("M", [1, 16])
def test_an_infinite_last_feature_stays_infinite(K, r, M):
    """What fills up the last block of 256 features, and the ranks up to 16 or 32, must not make a NaN of an infinity."""
    N = 40
    L = synth.make_custom(N, K, M, max(r, 1), fractions=(0.4, 0.3, 0.3), seed=K + r)
    D = DeviceLayer(L)
    D.quantize()
    sign = torch.sign(lowra.lowra_dequantize(D.layout, D.packed, D.absmax, D.mp)[:, -1])
    assert (sign != 0).all()
    x, A, B = D.x.clone(), None, None
    x[:, -1] = float("inf")
    if r:                                                    # a term of the same sign
        A, B = D.A.clone(), sign[:, None].expand(N, r).contiguous()
        A[:, -1] = 1.0
    got = lowra.lowra_linear_fwd(D.layout, D.packed, D.absmax, D.mp, x, A, B, 1.0).float()
    want = (sign.float() * float("inf")).expand(M, N)
    assert torch.equal(got, want)


@pytest.mark.parametrize("path", [lowra.PATH_GEMV, lowra.PATH_GEMV_GENERAL])
@pytest.mark.parametrize("r", [0, 8, 24])
def test_an_infinite_feature_in_a_batch(path, r):
    """Either kernel of a batch: ranks past r, which it fills up, must not make a NaN of an infinity."""
    N, K, M = 40, 1024, 3
    L = synth.make_custom(N, K, M, max(r, 1), fractions=(0.4, 0.3, 0.3), seed=r)
    D = DeviceLayer(L)
    D.quantize()
    sign = torch.sign(lowra.lowra_dequantize(D.layout, D.packed, D.absmax, D.mp)[:, 5])
    x, A, B = D.x.clone(), None, None
    x[:, 5] = float("inf")
    if r:
        A, B = D.A.clone(), sign[:, None].expand(N, r).contiguous()
        A[:, 5] = 1.0
    lowra.lowra_set_linear_path(path)
    try:
        batch = lowra.FwdBatch([(D.layout, D.packed, D.absmax, x, A, B)] * 2, D.mp, 1.0)
    finally:
        lowra.lowra_set_linear_path(lowra.PATH_AUTO)
    want = (sign.float() * float("inf")).expand(M, N)
    for y in batch.run():
        assert torch.equal(y.float(), want)
    batch.close()
