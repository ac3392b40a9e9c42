"""The fused GEMMs for the token counts between the small-token kernels and the large output grids (17 to a few hundred
tokens, and 1 to 16 where no small-token kernel takes the shape), under LOWRA_PATH_AUTO.

Every case is held to the oracle by the 2e-2 rule of the linear outputs, and to the 256-column kernels
(LOWRA_PATH_GEMM), which multiply the same bf16 weights and activations: the two differ in the order of fp32 sums only,
so by at most one unit in the last place of the bf16 output, 2^-7 of the entry (or of the output's rms, where
cancellation leaves an entry smaller than its terms).

test_mid_token_linear runs the plans that the planner picks (at these sizes nearly always tiles of 32 tokens);
test_every_variant forces each tile height, split and width class in turn."""
import pytest
import torch

from oracle import lowra_oracle as orc
from paper_2502_08141_amd import lowra, synth
from tests.gpu_util import REL_TOL, bf16_host_f64, rel_err
from tests.gpu_util import DeviceLayer

pytestmark = pytest.mark.gpu

ORDER_TOL = 2.0 ** -7

MIXED, NARROW = (0.4, 0.3, 0.3), (0.5, 0.5, 0.0)
# N, K, M, r, shares of 1/2/4-bit rows, one table per channel, bf16 scales.  Group counts of every remainder by four (a
# superstep is four groups; odd counts leave the input gradient half a column tile); channels that leave partial tiles and
# steps; token counts that leave partial tiles; ranks below, across and above 64.
CASES = [
    (264, 128, 17, 8, MIXED, False, False),
    (136, 192, 33, 5, MIXED, True, True),
    (520, 320, 40, 64, NARROW, False, False),
    (8, 704, 100, 100, (0.0, 0.0, 1.0), False, False),
    (1136, 832, 66, 8, MIXED, False, True),
    (1000, 1088, 130, 12, (0.85, 0.15, 0.0), True, False),
    (72, 2112, 300, 0, (1.0, 0.0, 0.0), False, False),
    (200, 256, 257, 64, (0.0, 1.0, 0.0), False, True),
    (2056, 1024, 96, 128, MIXED, True, False),
    (4096, 2048, 31, 16, NARROW, False, False),
    (1032, 4160, 128, 64, MIXED, False, False),
    (328, 128, 9, 40, MIXED, False, False),
    (136, 576, 3, 64, NARROW, True, False),
    (512, 512, 500, 32, MIXED, False, False),
]


@pytest.mark.parametrize("shape", CASES, ids=lambda s: f"{s[0]}x{s[1]}m{s[2]}r{s[3]}")
def test_mid_token_linear(shape):
    N, K, M, r, fr, per_channel, bf16_scales = shape
    print(f"[mid {shape}]", flush=True)
    L = synth.make_custom(N, K, M, max(r, 1), fractions=fr, seed=700 + N % 97, per_channel_tables=per_channel)
    D = DeviceLayer(L)
    if bf16_scales:
        D.layout.set_scale_dtype(torch.bfloat16)
    packed, absmax = lowra.lowra_quantize(D.layout, D.W, D.thr)
    A, B = (D.A, D.B) if r else (None, None)
    rp, ra = orc.quantize(L.W, L.bits, L.cb, L.thresholds, **({"scale_dtype": "bf16"} if bf16_scales else {}))
    hA, hB = (L.A, L.B) if r else (None, None)
    calls = {
        "forward": (lambda ws: lowra.lowra_linear_fwd(D.layout, packed, absmax, D.mp, D.x, A, B, L.s, workspace=ws), lowra.OP_LINEAR_FWD,
                    orc.linear_fwd(rp, ra, L.bits, L.cb, L.mappings, L.x, hA, hB, L.s)),
        "input gradient": (lambda ws: lowra.lowra_linear_bwd_input(D.layout, packed, absmax, D.mp, D.dY, A, B, L.s, workspace=ws), lowra.OP_LINEAR_BWD_INPUT,
                           orc.linear_bwd_input(rp, ra, L.bits, L.cb, L.mappings, L.dY, hA, hB, L.s, L.K)),
    }
    for name, (call, op, ref) in calls.items():
        need = D.layout.workspace_bytes(op, M, r)
        ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
        got = call(ws)
        again = call(ws)
        lowra.lowra_set_linear_path(lowra.PATH_GEMM)
        try:
            gemm = call(ws)
        finally:
            lowra.lowra_set_linear_path(lowra.PATH_AUTO)
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int16), again.view(torch.int16)), name          # splits are added in a fixed order
        g, e = bf16_host_f64(got), rel_err(bf16_host_f64(got), ref)
        print(f"    {name}: rel {e:.2e}, against the 256-column kernel {rel_err(g, bf16_host_f64(gemm)):.2e}", flush=True)
        assert e <= REL_TOL, name
        if M > 16:                                            # (with fewer the forward is a small-token kernel: another decode)
            assert rel_err(g, bf16_host_f64(gemm)) <= ORDER_TOL, name


@pytest.mark.parametrize("rows,K", [(32, 1088), (64, 1152), (96, 1216), (128, 1280)])      # 17 to 20 groups: every remainder by four
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("tables", ["narrow", "shared", "channel"])                        # with 4-bit rows: up to 64 codebooks, or more
def test_every_variant(rows, K, splits, tables):
    """Every instantiation of both kernels, its contraction whole and split, on a ragged shape: two tiles of tokens, the second
    one not full, partial column tiles and steps."""
    N, M, r = 328, rows + 17, 40 if splits == 1 else 13
    bf16_scales = splits == 3 and rows in (64, 128)
    L = synth.make_custom(N, K, M, r, fractions=NARROW if tables == "narrow" else MIXED, seed=640 + rows, per_channel_tables=tables == "channel")
    D = DeviceLayer(L)
    if bf16_scales:
        D.layout.set_scale_dtype(torch.bfloat16)
    packed, absmax = lowra.lowra_quantize(D.layout, D.W, D.thr)
    rp, ra = orc.quantize(L.W, L.bits, L.cb, L.thresholds, **({"scale_dtype": "bf16"} if bf16_scales else {}))
    refs = {lowra.OP_LINEAR_FWD: orc.linear_fwd(rp, ra, L.bits, L.cb, L.mappings, L.x, L.A, L.B, L.s),
            lowra.OP_LINEAR_BWD_INPUT: orc.linear_bwd_input(rp, ra, L.bits, L.cb, L.mappings, L.dY, L.A, L.B, L.s, L.K)}
    for op, ref in refs.items():
        print(f"[mid variant rows {rows} splits {splits} {tables} op {op}]", flush=True)
        fn, act = (lowra.lowra_linear_fwd, D.x) if op == lowra.OP_LINEAR_FWD else (lowra.lowra_linear_bwd_input, D.dY)
        call = lambda: fn(D.layout, packed, absmax, D.mp, act, D.A, D.B, L.s)
        lowra.lowra_set_mid_tiling(rows, splits)
        try:
            assert lowra.lowra_plan_mid_tiling(op, N, K, M, tables != "narrow", L.mappings.shape[0]) == (rows, splits)
            got = call()
            lowra.lowra_set_mid_tiling()
            lowra.lowra_set_linear_path(lowra.PATH_GEMM)
            gemm = call()
        finally:
            lowra.lowra_set_mid_tiling()
            lowra.lowra_set_linear_path(lowra.PATH_AUTO)
        torch.cuda.synchronize()
        g = bf16_host_f64(got)
        assert rel_err(g, ref) <= REL_TOL and rel_err(g, bf16_host_f64(gemm)) <= ORDER_TOL


# Tiles of 192 tokens of the input gradient, in every class of tables (with 4-bit rows: up to 64 codebooks, or more).
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("tables", ["narrow", "shared", "channel"])
def test_input_gradient_of_192_token_tiles(splits, tables):
    N, K, M, r = 328, 1088, 209, 40
    L = synth.make_custom(N, K, M, r, fractions=NARROW if tables == "narrow" else MIXED, seed=600 + splits, per_channel_tables=tables == "channel")
    D = DeviceLayer(L)
    if splits == 3:
        D.layout.set_scale_dtype(torch.bfloat16)
    packed, absmax = lowra.lowra_quantize(D.layout, D.W, D.thr)
    rp, ra = orc.quantize(L.W, L.bits, L.cb, L.thresholds, **({"scale_dtype": "bf16"} if splits == 3 else {}))
    ref = orc.linear_bwd_input(rp, ra, L.bits, L.cb, L.mappings, L.dY, L.A, L.B, L.s, L.K)
    lowra.lowra_set_mid_tiling(192, splits)
    try:
        assert lowra.lowra_plan_mid_tiling(lowra.OP_LINEAR_BWD_INPUT, N, K, M, tables != "narrow", L.mappings.shape[0]) == (192, splits)
        got = lowra.lowra_linear_bwd_input(D.layout, packed, absmax, D.mp, D.dY, D.A, D.B, L.s)
    finally:
        lowra.lowra_set_mid_tiling()
    torch.cuda.synchronize()
    assert rel_err(bf16_host_f64(got), ref) <= REL_TOL


# The forward's instantiations of the other parity of the number of groups (with an odd one the codes are staged in pieces
# that start 8 bytes early, and the last superstep is not staged at all: three groups are that superstep alone), and its
# tiles of 192 tokens.
@pytest.mark.parametrize("rows,K", [(32, 1152), (64, 1216), (96, 1280), (128, 1088), (192, 1088), (192, 1152), (192, 1216), (192, 1280), (192, 192), (32, 192)])
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("tables", ["narrow", "shared"])
def test_forward_staged_codes(rows, K, splits, tables):
    if splits > (K // 64 + 3) // 4:
        splits = 1
    N, M, r = 328, rows + 17, 40
    bf16_scales = splits == 3 and K in (1088, 1152)
    print(f"[mid forward rows {rows} K {K} splits {splits} {tables}]", flush=True)
    L = synth.make_custom(N, K, M, r, fractions=NARROW if tables == "narrow" else MIXED, seed=610 + rows)
    D = DeviceLayer(L)
    if bf16_scales:
        D.layout.set_scale_dtype(torch.bfloat16)
    packed, absmax = lowra.lowra_quantize(D.layout, D.W, D.thr)
    rp, ra = orc.quantize(L.W, L.bits, L.cb, L.thresholds, **({"scale_dtype": "bf16"} if bf16_scales else {}))
    ref = orc.linear_fwd(rp, ra, L.bits, L.cb, L.mappings, L.x, L.A, L.B, L.s)
    call = lambda: lowra.lowra_linear_fwd(D.layout, packed, absmax, D.mp, D.x, D.A, D.B, L.s)
    lowra.lowra_set_mid_tiling(rows, splits)
    try:
        assert lowra.lowra_plan_mid_tiling(lowra.OP_LINEAR_FWD, N, K, M, tables != "narrow", 3) == (rows, splits)
        got = call()
        lowra.lowra_set_mid_tiling()
        lowra.lowra_set_linear_path(lowra.PATH_GEMM)
        gemm = call()
    finally:
        lowra.lowra_set_mid_tiling()
        lowra.lowra_set_linear_path(lowra.PATH_AUTO)
    torch.cuda.synchronize()
    g = bf16_host_f64(got)
    assert rel_err(g, ref) <= REL_TOL and rel_err(g, bf16_host_f64(gemm)) <= ORDER_TOL


@pytest.mark.parametrize("K", [320, 384, 448, 512])           # the last superstep of 256 features holds 1, 2, 3 or all 4 groups
@pytest.mark.parametrize("fr", [NARROW, MIXED])
def test_infinite_activations_at_the_end_of_a_row(K, fr):
    """An infinity in a token's last features (input gradient: channels) makes its outputs infinite, of the weight's sign, and no
    other token's: nothing that stands in for features past K or channels past N may be multiplied with it."""
    N, M = 200 + K // 8, 40                                   # 240, 248, 256, 264 channels
    D = DeviceLayer(synth.make_custom(N, K, M, 1, fractions=fr, seed=790 + K))
    D.quantize()
    What = lowra.lowra_dequantize(D.layout, D.packed, D.absmax, D.mp, out_dtype=torch.float32)
    for name, call, act, W in (("forward", lowra.lowra_linear_fwd, D.x, What), ("input gradient", lowra.lowra_linear_bwd_input, D.dY, What.T)):
        n = act.shape[1]
        a, at = act.clone(), {0: n - 1, 3: n - 8, 17: n - 5, 39: n - 64}
        for m, k in at.items():
            a[m, k] = float("inf") if m % 2 else float("-inf")
        got, plain = (call(D.layout, D.packed, D.absmax, D.mp, v, None, None, 1.0).float() for v in (a, act))
        for m in range(M):
            if m in at:
                w = W[:, at[m]]
                assert (w != 0).all() and torch.equal(got[m], a[m, at[m]].float() * torch.sign(w)), f"{name}, token {m}"
            else:
                assert torch.equal(got[m], plain[m]), f"{name}, token {m}"


def test_mid_token_less_workspace():
    """A workspace that holds less than lowra_workspace_bytes asks for, but what the call cannot do without, is taken: the
    contraction is then split between fewer workgroups, or not at all."""
    L = synth.make_custom(1032, 2048, 40, 64, fractions=MIXED, seed=771)
    D = DeviceLayer(L)
    D.quantize()
    want = lowra.lowra_linear_fwd(D.layout, D.packed, D.absmax, D.mp, D.x, D.A, D.B, L.s)
    need = D.layout.workspace_bytes(lowra.OP_LINEAR_FWD, L.M, L.r)
    side = (L.M * 64 * 2 + 255) // 256 * 256                  # the rank-r intermediate alone
    assert need > side                                        # 40 tokens of this shape are split
    for size in (need - 256, (need + side) // 2, side):
        got = lowra.lowra_linear_fwd(D.layout, D.packed, D.absmax, D.mp, D.x, D.A, D.B, L.s,
                                     workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        assert rel_err(bf16_host_f64(got), bf16_host_f64(want)) <= ORDER_TOL
    with pytest.raises(lowra.LowraError, match="workspace too small"):
        lowra.lowra_linear_fwd(D.layout, D.packed, D.absmax, D.mp, D.x, D.A, D.B, L.s,
                               workspace=torch.empty(side - 256, dtype=torch.uint8, device="cuda"))


def test_mid_token_unaligned_workspace():
    """Without a LoRA term the forward needs no workspace, so a pointer that is not aligned is no error: nothing is put there."""
    L = synth.make_custom(1032, 2048, 40, 1, fractions=MIXED, seed=772)
    D = DeviceLayer(L)
    D.quantize()
    call = lambda ws: lowra.lowra_linear_fwd(D.layout, D.packed, D.absmax, D.mp, D.x, None, None, L.s, workspace=ws)
    need = D.layout.workspace_bytes(lowra.OP_LINEAR_FWD, L.M, 0)
    assert need > 0                                           # an aligned one would hold partial tiles
    buf = torch.full((need + 16,), 0x5a, dtype=torch.uint8, device="cuda")
    got = call(buf[4:])
    assert torch.equal(got, call(torch.empty(0, dtype=torch.uint8, device="cuda")))
    assert (buf == 0x5a).all()


@pytest.mark.parametrize("N,K,M,r", [(4096, 4096, 128, 64), (11008, 4096, 66, 16), (4096, 11008, 300, 0), (1032, 4160, 40, 24), (5120, 13824, 1000, 16)])
def test_static_scratch_splits_the_same_way(N, K, M, r):
    """The forward without a workspace takes the same plan, its partial tiles in pieces where they exceed the static array:
    same bits."""
    print(f"[mid static {N}x{K} M{M} r{r}]", flush=True)
    D = DeviceLayer(synth.make_custom(N, K, M, r, fractions=(0.4, 0.3, 0.3), seed=870 + r))
    D.quantize()
    want = lowra.lowra_linear_fwd(D.layout, D.packed, D.absmax, D.mp, D.x, D.A, D.B, D.L.s)
    y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    assert torch.equal(lowra.lowra_linear_fwd_static(D.layout, D.packed, D.absmax, D.mp, D.x, D.A, D.B, D.L.s, y), want)
