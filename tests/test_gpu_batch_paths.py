"""A batched small-token forward takes the general or the streaming kernel by the size of the batch: both, and what
LOWRA_PATH_AUTO picks, against the oracle on batches around that choice, and with two workgroups per compute unit at 5120
features."""
import pytest
import torch

from oracle import lowra_oracle as orc
from paper_2502_08141_amd import lowra, synth
from tests.gpu_util import REL_TOL, DeviceLayer, bf16_host_f64, rel_err

pytestmark = pytest.mark.gpu

BATCHES = {
    "one small": [(136, 1024)],
    "attention": [(520, 4096)] * 3,
    "5120 features": [(1032, 5120), (264, 5120)],
    "mixed lengths": [(264, 2048), (136, 6144), (520, 4096)],
    "long rows": [(136, 11008)],
    "few strips, one launch": [(136, 512), (264, 1024), (136, 2816)],     # 4, 8 and 16 wavefronts by themselves
    "many strips": [(4200, 1024), (136, 2816)],
    "with one that only the general kernel takes": [(264, 2048), (136, 2112)],
}


@pytest.mark.parametrize("M,r", [(1, 16), (5, 8), (8, 0), (16, 32)])
@pytest.mark.parametrize("name", list(BATCHES))
def test_batch_paths(name, M, r):
    print(f"[batch {name} M{M} r{r}]", flush=True)
    layers = []
    for i, (N, K) in enumerate(BATCHES[name]):
        D = DeviceLayer(synth.make_custom(N, K, M, max(r, 1), fractions=(0.4, 0.3, 0.3), seed=900 + i))
        D.quantize()
        layers.append(D)
    refs = []
    for D in layers:
        L = D.L
        A, B = (L.A, L.B) if r else (None, None)
        refs.append(orc.linear_fwd(*orc.quantize(L.W, L.bits, L.cb, L.thresholds), L.bits, L.cb, L.mappings, L.x, A, B, L.s))
    for path in (lowra.PATH_AUTO, lowra.PATH_GEMV, lowra.PATH_GEMV_GENERAL):
        lowra.lowra_set_linear_path(path)
        try:
            batch = lowra.FwdBatch([(D.layout, D.packed, D.absmax, D.x, D.A if r else None, D.B if r else None) for D in layers], layers[0].mp, 2.0)
        finally:
            lowra.lowra_set_linear_path(lowra.PATH_AUTO)
        for _ in range(2):
            ys = batch.run()
            torch.cuda.synchronize()
            for y, ref in zip(ys, refs):
                assert rel_err(bf16_host_f64(y), ref) <= REL_TOL, path
        batch.close()
