"""Every kernel family that stage 2 can be served by, on shapes that the
library itself says it serves by that family (asserted, so that a change of
the selection cannot quietly move a test to another kernel)."""
import numpy as np
import pytest

import oracle
from helpers import (Case, bf16_to_f64, identical_share, mirror_err_rows, rel_err_rows, tile_sample, to_host)

pytestmark = pytest.mark.gpu

# the bars of test_gpu_moe.py for tests that compare hundreds of rows: exact
# mode (fp8: h is re-quantised to e4m3, up to 2^-4 per value), mirror mode (bf16:
# y passes two bf16 roundings in series, 2^-8), share of identical values
TOL = {"exact": {"bf16": 1e-2, "fp8": 8e-2, "fp8mx": 8e-2}, "mirror": {"bf16": 4e-3, "fp8": 2e-2, "fp8mx": 2e-2}}
IDENTICAL = {"bf16": 0.995, "fp8": 0.85, "fp8mx": 0.85}

# rows of the experts held here: few (of 64 experts in all, the other pairs
# nobody's), every number of live 32-row blocks of a 256-row tile, and full tiles
FEW = [150, 0, 1, 31, 70, 129, 300]
BLOCKS = [0, 1, 31, 33, 64, 65, 97, 129, 161, 193, 225, 255, 256, 257, 300, 520, 900]
FULL = [300, 520, 900, 257, 256, 700, 33, 0]


def _workload(dtype, ids, E, n_local, H, I, T_valid=None):
    from paper_2608_13057_amd import synth

    T, K = ids.shape
    pl = synth.placement_local_hot(E, n_local, 1)  # a second slot for expert 0
    w = np.random.default_rng(5).uniform(0.1, 1.0, (T, K)).astype(np.float32)
    return synth.Workload("routes", dtype, T, T if T_valid is None else T_valid, K, E, H, I, 0.0, pl,
                          {"uniform": synth.plan_uniform(pl, E)}, ids, w, 0)


def _forward(c):
    import torch
    from paper_2608_13057_amd import moe

    y = torch.empty(c.wl.T, c.wl.H, dtype=torch.int16, device="cuda")
    moe.forward(c.shape, c.d_plan, c.d_ids, c.d_w, c.d_x, c.d_xs, c.d_weights, c.disp, y, c.ws)
    torch.cuda.synchronize()
    return to_host(y)


def _check(c, what, rng, extra=200):
    """Stage 1 bit for bit; y on one row of every M-tile, every slot's last
    row and `extra` random tokens against the fp64 oracle (exact and mirror
    modes); tokens without a local pair exactly zero."""
    print(f"[{what}] running, T={c.wl.T} S={c.wl.S}", flush=True)
    y = _forward(c)
    d = c.oracle_dispatch()
    assert np.array_equal(to_host(c.disp.slot_counts), d["slot_counts"])
    assert np.array_equal(to_host(c.disp.pair_row), d["pair_row"])
    has = (d["pair_row"] >= 0).any(axis=1)
    assert np.all(y[~has] == 0)
    loc = np.nonzero(has)[0]
    pick = np.union1d(tile_sample(d, c.m_tile, rng), rng.choice(loc, min(len(loc), extra), replace=False))
    sel = np.zeros(c.wl.T, np.uint8)
    sel[pick] = 1
    got = bf16_to_f64(y)
    for mode in ("exact", "mirror"):
        ref = oracle.moe(c.x, c.wl.topk_w, oracle.pair_slot(d), c.w13, c.w2, c.dtype, mode, c.xs, c.s13, c.s2,
                         token_sel=sel)
        err = (rel_err_rows if mode == "exact" else mirror_err_rows)(got, ref, pick)
        print(f"[{what}] sampled {len(pick)} {mode} err={err:.2e}")
        assert err <= TOL[mode][c.dtype]
    assert identical_share(got[pick], ref[pick]) >= IDENTICAL[c.dtype]
    return y, d


@pytest.mark.parametrize("route,dtype,m_tile,counts,H,I", [
    ("big", "bf16", 256, FEW, 512, 384), ("big", "bf16", 256, FEW, 1280, 128), ("big", "bf16", 256, FULL, 512, 1152),
    ("stream", "bf16", 256, FEW, 1152, 384), ("stream", "fp8", 256, FEW, 1152, 384),
    ("stream", "fp8mx", 256, FEW, 1152, 384), ("stream", "fp8", 256, FEW, 128, 640),
    ("stream", "bf16", 128, FEW, 1152, 640), ("stream", "fp8", 192, FEW, 2048, 640),
    ("wide", "bf16", 192, BLOCKS, 640, 1152), ("wide", "fp8", 192, BLOCKS, 640, 1152),
    ("wide", "fp8mx", 192, BLOCKS, 640, 1152)])
def test_route(route, dtype, m_tile, counts, H, I):
    """Slots of no row, one row, ragged tiles, full tiles and several tiles."""
    from paper_2608_13057_amd import measure

    E = 64 if counts is FEW else len(counts)
    ids = np.repeat(np.arange(len(counts), dtype=np.int32), counts)
    if counts is FEW:
        ids = np.concatenate([ids, np.full(9, 40, np.int32)])
    rng = np.random.default_rng(17)
    rng.shuffle(ids)
    c = Case(_workload(dtype, ids.reshape(-1, 1), E, len(counts), H, I), "uniform", m_tile)
    assert measure.stage2_route(c.shape) == route
    _check(c, f"{route} {dtype} M={m_tile} H={H} I={I}", rng)


@pytest.mark.parametrize("dtype,m_tile", [("bf16", 128), ("fp8", 64), ("fp8mx", 64)])
def test_wide_tiles_beyond_the_sorted_list(dtype, m_tile):
    """More wide tiles than the kernel's cost-ordered list holds (768), so
    that items are dealt in tile order: 256 slots of three to five 256-row
    tiles.  I 512: the mirror bar is that of rows whose outputs sum a thousand
    terms and more (K I; the tiny shape has 2 x 512); one flipped e4m3 code of
    h, at most 2^-3 of its term, weighs 1 / sqrt(K I) of a row's output, twice
    as much in 4 x 128 terms (2.4e-2 seen) as in 4 x 512."""
    from paper_2608_13057_amd import measure

    E, K, T = 255, 4, 57600
    rng = np.random.default_rng(29)
    ids = ((rng.integers(0, E, (T, 1)) + np.cumsum(rng.integers(1, 60, (T, K)), axis=1)) % E).astype(np.int32)
    c = Case(_workload(dtype, ids, E, E, 128, 512), "uniform", m_tile)
    assert measure.stage2_route(c.shape) == "wide"
    _, d = _check(c, f"unsorted {dtype} M={m_tile}", rng, extra=50)
    tiles = sum(-(-int(n) // 256) for n in d["slot_counts"])
    assert tiles > 768, tiles


@pytest.mark.parametrize("dtype", ["bf16", "fp8", "fp8mx"])
def test_tokens_across_the_line_between_kernels(dtype):
    """The first 40 tokens alone (streaming GEMM) and among 800 (wide tiles):
    the sums run in another order, so the results are equal to rounding only.
    Both are within the mirror bars of the same reference, hence within twice
    the bar of each other."""
    from paper_2608_13057_amd import measure, synth

    E, K, H, I = 12, 2, 640, 1536
    rng = np.random.default_rng(7)
    ids = np.stack([rng.permutation(E)[:K] for _ in range(800)]).astype(np.int32)
    out = {}
    for T, route in ((40, "stream"), (800, "wide")):
        c = Case(_workload(dtype, ids[:T], E, E, H, I), "uniform", 64)
        assert measure.stage2_route(c.shape) == route
        x, _ = synth.activations(800, H, 0, dtype)  # drawn row by row
        assert np.array_equal(c.x, x[:T])
        print(f"[across {dtype} T={T}] running", flush=True)
        out[T] = bf16_to_f64(_forward(c)[:40])
    err = mirror_err_rows(out[40], out[800], np.arange(40))
    print(f"[across {dtype}] err={err:.2e} identical={identical_share(out[40], out[800]):.4f}")
    assert np.any(out[40] != 0) and err <= 2 * TOL["mirror"][dtype]


@pytest.mark.parametrize("dtype,T_valid", [("bf16", 40), ("bf16", 800), ("fp8", 40), ("fp8", 800), ("fp8mx", 40),
                                           ("fp8mx", 800)])
def test_padding_changes_no_bit(dtype, T_valid):
    """A padded batch gives the bits of the batch it holds, whichever kernel
    serves that one and whichever its size with padding would have; padding
    rows are zero."""
    from paper_2608_13057_amd import measure

    E, K, H, I = 12, 2, 640, 1536
    rng = np.random.default_rng(7)
    ids = np.stack([rng.permutation(E)[:K] for _ in range(1000)]).astype(np.int32)
    out = {}
    for T in (T_valid, 1000):
        c = Case(_workload(dtype, ids[:T], E, E, H, I, T_valid), "uniform", 64)
        assert measure.stage2_route(c.shape) == ("stream" if T_valid == 40 else "wide")
        print(f"[padding {dtype} T={T} valid {T_valid}] running", flush=True)
        out[T] = _forward(c)
    assert np.any(out[T_valid] != 0)
    assert np.array_equal(out[1000][:T_valid], out[T_valid])
    assert np.all(out[1000][T_valid:] == 0)
