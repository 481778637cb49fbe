"""The streaming GEMM's two ways of dealing a gate/up item's two contraction
chunks to the workgroups: whole items, or ranges that end inside an item (which
the fixup kernel completes).  Both sum a row's products in the same order, so
which one a batch takes shows in no bit of its result."""
import numpy as np
import pytest

import oracle
from helpers import (Case, bf16_to_f64, identical_share, mirror_err_rows, mirror_stats, rel_err_rows, to_host)

pytestmark = pytest.mark.gpu

# the bars of test_gpu_moe.py for tests that compare hundreds of rows: exact
# mode (fp8: h is re-quantised to e4m3, up to 2^-4 per value), mirror mode (bf16:
# y passes two bf16 roundings in series, 2^-8), share of identical values
TOL = {"exact": {"bf16": 1e-2, "fp8": 8e-2, "fp8mx": 8e-2}, "mirror": {"bf16": 4e-3, "fp8": 2e-2, "fp8mx": 2e-2}}
IDENTICAL = {"bf16": 0.995, "fp8": 0.85, "fp8mx": 0.85}


def _forward(c):
    import torch
    from paper_2608_13057_amd import moe

    y = torch.empty(c.wl.T, c.wl.H, dtype=torch.int16, device="cuda")
    moe.forward(c.shape, c.d_plan, c.d_ids, c.d_w, c.d_x, c.d_xs, c.d_weights, c.disp, y, c.ws)
    torch.cuda.synchronize()
    return to_host(y)


def _workload(dtype, ids, E, n_local, n_extra, H, I, plan=None):
    """Experts 0 .. n_local - 1 held here, second slots for the first n_extra;
    the other experts' pairs are nobody's."""
    from paper_2608_13057_amd import synth

    T, K = ids.shape
    pl = synth.placement_local_hot(E, n_local, n_extra)
    uni = synth.plan_uniform(pl, E)
    if plan is not None:
        uni = synth.Plan(np.array(plan, np.uint32), uni.remote_weight, uni.remote_replicas, "p")
    w = np.random.default_rng(5).uniform(0.1, 1.0, (T, K)).astype(np.float32)
    return synth.Workload("ranges", dtype, T, T, K, E, H, I, 0.0, pl, {"p": uni}, ids, w, 0)


@pytest.mark.parametrize("dtype,H,I", [("bf16", 2176, 384), ("bf16", 2176, 1024), ("fp8", 3200, 384),
                                       ("fp8mx", 3200, 384), ("fp8mx", 3200, 640)])
@pytest.mark.parametrize("m_tile", [64, 128, 192, 256])
def test_split_items(dtype, H, I, m_tile):
    """Items of two chunks (34 or 25 steps: the second chunk is padded to the
    pipeline depth) of slots with no row, one row, a ragged tile and several
    tiles, split over the workgroups: a chunk each where there are fewer
    chunks than workgroups, ranges of more where I is 1024.  y against the
    fp64 oracle (exact and mirror modes), the same bits for another split of
    the expert with two slots, tokens without a local pair exactly zero."""
    from paper_2608_13057_amd import measure

    counts = [150, 0, 1, 31, 70, 129, 200]
    ids = np.concatenate([np.repeat(np.arange(len(counts), dtype=np.int32), counts), np.full(9, 40, np.int32)])
    np.random.default_rng(3).shuffle(ids)
    outs = []
    for plan in (None, [1] * 7 + [4]):
        c = Case(_workload(dtype, ids.reshape(-1, 1), 64, 7, 1, H, I, plan), "p", m_tile)
        assert measure.stage2_route(c.shape) == "stream_split"
        print(f"[split items {dtype} M={m_tile} H={H} I={I}] running", flush=True)
        outs.append(_forward(c))
    d = c.oracle_dispatch()
    assert np.array_equal(to_host(c.disp.slot_counts), d["slot_counts"])
    assert np.array_equal(outs[0], outs[1])
    has = (d["pair_row"] >= 0).any(axis=1)
    assert np.all(outs[1][~has] == 0) and (~has).sum() == 9
    got, loc = bf16_to_f64(outs[1]), np.nonzero(has)[0]
    for mode in ("exact", "mirror"):
        ref = oracle.moe(c.x, c.wl.topk_w, oracle.pair_slot(d), c.w13, c.w2, dtype, mode, c.xs, c.s13, c.s2)
        err = (rel_err_rows if mode == "exact" else mirror_err_rows)(got, ref, loc)
        print(f"[split items {dtype} M={m_tile}] {mode} err={err:.2e} {mirror_stats(got[loc], ref[loc])}")
        assert err <= TOL[mode][dtype]
    assert identical_share(got[loc], ref[loc]) >= IDENTICAL[dtype]


@pytest.mark.parametrize("dtype,H", [("bf16", 2048), ("fp8", 4096), ("fp8mx", 4096)])
def test_tokens_keep_their_bits_in_a_larger_batch(dtype, H):
    """The first three tokens of a batch of 64 give the same bits as a batch
    of those three alone, though at 64-row M-tiles the small batch splits its
    items and the large one deals them whole, and at 128 and 192 rows both
    split (H 4096) or neither (H 2048)."""
    from paper_2608_13057_amd import measure, synth

    E, I = 12, 1024
    rng = np.random.default_rng(7)
    ids = np.stack([rng.permutation(E)[:2] for _ in range(64)]).astype(np.int32)
    outs = {}
    for T in (3, 64):
        for m_tile in (64, 128, 192):
            c = Case(_workload(dtype, ids[:T], E, E, 0, H, I), "p", m_tile)
            whole = T == 64 if m_tile == 64 else H == 2048
            assert measure.stage2_route(c.shape) == ("stream" if whole else "stream_split")
            # (the generators draw row by row: the same x and weights for the first tokens)
            x, xs = synth.activations(64, H, 0, dtype)
            assert np.array_equal(c.x, x[:T])
            print(f"[batch size {dtype} T={T} M={m_tile}] running", flush=True)
            outs[T, m_tile] = _forward(c)[:3]
    first = outs[3, 64]
    assert np.any(first != 0)
    for k, y in outs.items():
        assert np.array_equal(y, first), k
