"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every declared symbol,
plans rows like the oracle, and rejects bad arguments before touching a device."""
import ctypes as C
import os
import re

import numpy as np
import pytest

from oracle import lowra_oracle as orc
from paper_2502_08141_amd import lowra, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "lowra.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(lowra_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    L = lowra.lib()
    names = declared_symbols()
    assert set(names) == set(lowra.SYMBOLS)
    for name in names:
        assert getattr(L, name) is not None


def test_static_scratch_sizes_are_the_headers():
    text = open(os.path.join(ROOT, "include", "lowra.h")).read()
    for name in ("STATIC_SCRATCH_BYTES", "STATIC_ARRAY_BYTES"):
        n, shift = re.search(rf"#define LOWRA_{name} \((\d+)u << (\d+)\)", text).groups()
        assert int(n) << int(shift) == getattr(lowra, name)


def test_status_strings():
    assert lowra.status_string(0) == "ok"
    assert len({lowra.status_string(i) for i in range(6)}) == 6


def test_plan_rows_matches_oracle_and_rejects_bad_input():
    rng = np.random.default_rng(0)
    bits = rng.choice(np.array([1, 2, 4], np.uint8), size=1000)
    for K in (64, 4096, 13824):
        assert np.array_equal(lowra.lowra_plan_rows(K, bits), orc.row_offsets(K, bits))
    with pytest.raises(lowra.LowraError) as e:
        lowra.lowra_plan_rows(100, bits)
    assert e.value.status == lowra.UNSUPPORTED
    with pytest.raises(lowra.LowraError) as e:
        lowra.lowra_plan_rows(64, np.array([1, 3], np.uint8))
    assert e.value.status == lowra.UNSUPPORTED
    with pytest.raises(lowra.LowraError) as e:      # more than 4 GiB of codes
        lowra.lowra_plan_rows(1 << 20, np.full(1 << 13, 4, np.uint8))
    assert e.value.status == lowra.UNSUPPORTED


def test_layout_create_validates_on_host_first():
    """Every rejected argument is reported without a device; a valid one needs a device (HIP_ERROR here)."""
    _, _, cb_bits = synth.shared_codebooks()
    L = lowra.lib()
    h = C.c_void_p()

    def create(N, K, group, bits, cb, Cn, cbb):
        b = np.ascontiguousarray(bits, np.uint8); c = np.ascontiguousarray(cb, np.int32)
        q = np.ascontiguousarray(cbb, np.uint8)
        return L.lowra_layout_create(N, K, group, b.ctypes.data, c.ctypes.data, Cn, q.ctypes.data, C.byref(h))

    assert create(4, 128, 32, [1] * 4, [0] * 4, 3, cb_bits) == lowra.UNSUPPORTED      # group != 64
    assert create(4, 96, 64, [1] * 4, [0] * 4, 3, cb_bits) == lowra.UNSUPPORTED       # K % 64
    assert create(4, 128, 64, [1, 2, 8, 1], [0, 1, 2, 0], 3, cb_bits) == lowra.UNSUPPORTED
    assert create(4, 128, 64, [1] * 4, [0, 0, 3, 0], 3, cb_bits) == lowra.INVALID_ARG  # table index out of range
    assert create(4, 128, 64, [1, 2, 4, 1], [0, 1, 1, 0], 3, cb_bits) == lowra.INVALID_ARG  # width/table mismatch
    assert create(-1, 128, 64, [1], [0], 3, cb_bits) == lowra.INVALID_ARG
    assert L.lowra_layout_create(4, 128, 64, None, None, 3, None, C.byref(h)) == lowra.INVALID_ARG
    assert L.lowra_packed_bytes(None) == 0
    assert L.lowra_set_linear_path(7) == lowra.INVALID_ARG
    for bad in [(256, 100, 0), (128, 256, 1), (64, 64, 0), (256, 192, -1), (0, 128, 0)]:
        assert L.lowra_set_fwd_tiling(*bad) == lowra.INVALID_ARG, bad
    assert L.lowra_set_fwd_tiling(256, 192, 3) == lowra.OK and L.lowra_set_fwd_tiling(0, 0, 0) == lowra.OK
    assert L.lowra_quantize(None, None, None, None, None, None) == lowra.INVALID_ARG
    # the batched quantizer checks every entry on the host before it launches anything
    nul = (C.c_void_p * 2)(C.c_void_p(0), C.c_void_p(0))
    assert L.lowra_quantize_batch(0, None, None, None, None, None, None) == lowra.OK
    assert L.lowra_quantize_batch(-1, nul, nul, nul, nul, nul, None) == lowra.INVALID_ARG
    assert L.lowra_quantize_batch(2, None, nul, nul, nul, nul, None) == lowra.INVALID_ARG
    assert L.lowra_quantize_batch(2, nul, nul, nul, nul, nul, None) == lowra.INVALID_ARG      # null layouts


def test_assign_precisions_matches_the_oracle_rule():
    """Host-only entry point: the library's heap-based greedy assignment takes the same decisions as
    the oracle's plain scan (both in fp64), including ties and upgrades that do not help."""
    rng = np.random.default_rng(12)
    for N in (1, 7, 300):
        params = rng.choice([4096, 11008, 13824], N).astype(np.int64)
        m4 = rng.uniform(1e-6, 2e-6, N); m2 = m4 * rng.uniform(0.8, 6, N); m1 = m2 * rng.uniform(0.9, 4, N)
        mse = np.stack([m1, m2, m4], axis=1).astype(np.float32)
        mse[::5] = mse[0]                                           # exact ties between channels
        for bpp in (1.0, 1.15, 1.5, 2.0, 2.25, 3.1, 4.0):
            assert np.array_equal(lowra.lowra_assign_precisions(params, mse, bpp), orc.assign_greedy(params, mse, bpp)), (N, bpp)
    with pytest.raises(lowra.LowraError):
        lowra.lowra_assign_precisions(np.array([64], np.int64), np.ones((1, 3), np.float32), 0.5)
    with pytest.raises(lowra.LowraError):
        lowra.lowra_assign_precisions(np.array([0], np.int64), np.ones((1, 3), np.float32), 2.0)


def test_forward_tiling_planner():
    """Host only: the forward GEMM's planner.  A compute unit runs one 256-channel tile at a time, a tile of 256 / 192 /
    128 token rows costs 1 / 0.80 / 0.62: the plan must cover every token row, never finish later than the plain
    256-row tiling, and on the configs' shapes pick what the rounds arithmetic says."""
    import itertools
    import math

    cost = {256: 1.0, 192: 0.80, 128: 0.62}

    def finish(N, M, units, ra, rb, ca):
        cols = -(-N // 256)
        jobs = [cost[ra]] * (ca * -(-M // ra)) + [cost[rb]] * ((cols - ca) * -(-M // rb))
        free = [0.0] * units
        for j in jobs:                                   # launch order, each tile to the unit that is free first
            k = min(range(units), key=free.__getitem__)
            free[k] += j
        return max(free)

    for N, M, units in itertools.product([256, 1000, 4096, 5120, 11008], [17, 300, 2048, 4096], [64, 256]):
        ra, rb, ca = lowra.lowra_plan_fwd_tiling(N, M, units)
        cols = -(-N // 256)
        assert ra in cost and rb in cost and rb <= ra and 0 <= ca <= cols, (N, M, units, ra, rb, ca)
        assert finish(N, M, units, ra, rb, ca) <= finish(N, M, units, 256, 256, cols) + 1e-9, (N, M, units, ra, rb, ca)
    # config 3: 688 tiles of 256 rows are three rounds on 256 units; 256-row tiles for the first columns and 192-row
    # tiles for the rest finish at 2.8 (e.g. 30 columns = 480 tiles, then 13 x 22 = 286 tiles)
    ra, rb, ca = lowra.lowra_plan_fwd_tiling(11008, 4096, 256)
    assert (ra, rb) == (256, 192) and abs(finish(11008, 4096, 256, ra, rb, ca) - 2.8) < 1e-9
    # config 2: 128 tiles of 256 rows leave half the units idle; 256 tiles of 128 rows fill them
    assert lowra.lowra_plan_fwd_tiling(4096, 2048, 256) == (128, 128, 16)
    # config 4: 320 tiles of 256 rows are two rounds; 440 tiles of 192 rows are two shorter ones
    assert lowra.lowra_plan_fwd_tiling(5120, 4096, 256) == (192, 192, 20)
    L = lowra.lib()
    assert L.lowra_plan_fwd_tiling(0, 4, 256, None, None, None) == lowra.INVALID_ARG


def test_mid_token_planner():
    """Host only: the mid-token GEMMs' planner and the hook that forces a plan."""
    FWD, BWD = lowra.OP_LINEAR_FWD, lowra.OP_LINEAR_BWD_INPUT
    L = lowra.lib()
    for bad in [(2, 256, 256, 40, 0, 3), (FWD, 0, 256, 40, 0, 3), (FWD, 256, 100, 40, 0, 3), (BWD, 256, 256, 0, 0, 3), (BWD, 256, 256, 40, 0, 0)]:
        with pytest.raises(lowra.LowraError):
            lowra.lowra_plan_mid_tiling(*bad)
    for bad in [(0, 1), (32, 0), (48, 1), (160, 1), (64, 33), (-32, 1), (64, -1)]:
        assert L.lowra_set_mid_tiling(*bad) == lowra.INVALID_ARG, bad
    assert lowra.lowra_plan_mid_tiling(FWD, 4096, 64, 40, True, 3) == (0, 0)               # one group: no mid-token kernel
    for op in (FWD, BWD):
        for wide, books in ((False, 3), (True, 3), (True, 4096)):
            rows, splits = lowra.lowra_plan_mid_tiling(op, 4096, 4096, 128, wide, books)
            assert rows in (32, 64, 96, 128) and splits > 1                                # 32 tiles at most: the contraction is split
            assert lowra.lowra_plan_mid_tiling(op, 11008, 4096, 4096, wide, books) == (0, 0)   # the 256-column kernels' tiles fill the chip
    lowra.lowra_set_mid_tiling(96, 3)
    try:
        assert lowra.lowra_plan_mid_tiling(FWD, 328, 1088, 40, True, 3) == (96, 3)         # 5 supersteps: 2 + 2 + 1
        assert lowra.lowra_plan_mid_tiling(FWD, 328, 832, 40, True, 3) == (96, 2)          # 4: 2 + 2
        assert lowra.lowra_plan_mid_tiling(BWD, 328, 832, 40, True, 3) == (96, 3)          # 6 steps
        assert lowra.lowra_plan_mid_tiling(BWD, 64, 832, 40, True, 3) == (96, 1)
        assert lowra.lowra_plan_mid_tiling(FWD, 1 << 15, 1088, 4096, False, 3) == (96, 1)  # the partial tiles would exceed 64 MiB
    finally:
        lowra.lowra_set_mid_tiling()
    assert lowra.lowra_plan_mid_tiling(FWD, 11008, 4096, 4096, True, 3) == (0, 0)


def test_mid_token_planner_odd_groups():
    """Host only: with an odd number of groups the 256-column forward takes three to six times the mid-token kernel's time per
    step, so no call goes there that the planner compares (up to 16 workgroups of 128 x 128 outputs per unit)."""
    for N in (3000, 4096, 8184, 13824):
        for K in range(192, 6000, 128):
            for M in (*range(64, 4200, 224), 3072, 6000, 8192):
                if -(-N // 128) * -(-M // 128) <= 16 * 256:
                    for wide, books in ((False, 3), (False, N), (True, 3), (True, N)):
                        assert lowra.lowra_plan_mid_tiling(lowra.OP_LINEAR_FWD, N, K, M, wide, books) != (0, 0), (N, K, M, wide, books)


def test_mid_token_planner_input_gradient():
    """Host only: a round of the 256-column input gradient costs about ten steps beside its steps, and a step outside its pipeline
    (features that are no multiple of 256, fewer than eight full steps) 2.4 pipelined ones.  So few channels and such features stay
    with the mid-token kernel where the tiles do not fill the chip evenly (measured 1.2 to 1.9 times as fast)."""
    plan = lambda N, K, M, wide=False: lowra.lowra_plan_mid_tiling(lowra.OP_LINEAR_BWD_INPUT, N, K, M, wide, 3)
    for N, K, M in [(264, 5504, 3072), (264, 5120, 4096), (264, 13824, 1200), (264, 4096, 3072), (264, 2752, 3000), (520, 4160, 2048), (520, 8192, 1025),
                    (1024, 13824, 1025), (3072, 11008, 513), (4096, 4160, 2048)]:
        assert plan(N, K, M) != (0, 0), (N, K, M)
    assert plan(264, 5120, 4096, True) != (0, 0) and plan(264, 8192, 2500, True) != (0, 0)
    assert plan(4096, 4096, 2048) == plan(4096, 4096, 4096) == plan(13824, 5120, 4096) == (0, 0)      # tiles that fill the chip


def test_small_forward_planner():
    """Host only: the general small-token forward's wavefronts.  A low rank needs no more of a workgroup's memory than a high one
    where its t comes from a launch of its own, so it must not run through fewer wavefronts; and where the form that makes t
    itself is the only one that does not fit, the other is taken before fewer wavefronts are."""
    plan = lowra.lowra_plan_small_fwd
    assert plan(4096, 4096, 16, 8) == plan(4096, 4096, 15, 8) == (16, 1, False)     # the sums of 16 wavefronts do not fit beside 16 tokens
    assert plan(4096, 4096, 14, 8) == (16, 1, True)
    assert plan(4096, 4096, 16, 16) == plan(4096, 4096, 16, 32) == (16, 1, False)
    assert plan(4096, 2048, 16, 16) == (8, 1, True)
    assert plan(4096, 11008, 8, 16) == (16, 3, False) and plan(4096, 11008, 9, 16) == (8, 6, False)
    assert plan(11008, 4096, 4, 16) == (8, 2, False) and plan(11008, 4096, 16, 16) == (16, 1, False)
    for K in list(range(64, 4096, 192)) + list(range(4096, 16385, 1024)):
        for M in range(1, 17):
            for N, strips in ((8, 0), (4096, 0), (4104, 0), (4096, 768)):
                # (with many strips a rank's few KB also decide whether two smaller workgroups share a unit)
                waves = [plan(N, K, M, r, strips)[0] for r in ((0, 8, 16, 17, 64, 128) if N <= 4096 and not strips else (8, 16, 17))]
                assert all(a >= b for a, b in zip(waves, waves[1:])), (N, K, M, strips, waves)
                for r in (0, 8, 16, 64):
                    if N <= 4096:                            # a batch whose strips have a unit each takes what a call does
                        assert plan(N, K, M, r, -(-N // 16)) == plan(N, K, M, r), (N, K, M, r)
                    w, rounds, fused = plan(N, K, M, r, strips)
                    assert w * rounds * 256 >= K and (not fused or (rounds == 1 and 0 < r <= 16)), (N, K, M, r, strips)
    for bad in [(0, 256, 1, 0, 0), (8, 100, 1, 0, 0), (8, 256, 17, 0, 0), (8, 256, 1, -1, 0), (8, 256, 1, 0, -1)]:
        with pytest.raises(lowra.LowraError):
            plan(*bad)
    assert pytest.raises(lowra.LowraError, plan, 8, 16448, 1, 0).value.status == lowra.UNSUPPORTED
