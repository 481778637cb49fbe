"""Performance cases of the per-GPU MoE block, through its public Python entry
points (paper_2608_13057_amd.moe).

A case is one GPU's share of an expert-parallel MoE layer: a batch of routed
tokens, the local expert slots with their packed weights, and the split plan.
The cases go from a handful of decode tokens, where launches and the streaming
of the activated experts' weights count, over mixed batches, where a slot sees
some dozens to hundreds of rows, to prefill batches bound by the matrix cores;
in bf16, fp8 with fp32 block scales and fp8 with power-of-two block scales.

Fields of a case: T tokens of which the first T_valid count, top-K of E
experts, hidden size H, expert width I, Zipf exponent of the popularity,
placement of the slots (local_hot / strided / remote_hot with home and extra
slots, see synth), plan, m_tile, call (prepared: a PreparedForward; forward:
moe.forward; stages: dispatch, experts and combine one by one) and shared
(slots reach their weights through a per-slot table, replicas of one expert
sharing a copy).
"""
import math

import numpy as np
import torch

from paper_2608_13057_amd import moe, synth

SHAPES = {
    # E, K, H, I, zipf, placement, home slots, extra slots
    "qwen3": (128, 8, 4096, 1536, 1.0, "remote_hot", 16, 2),
    "qwen3_home": (128, 8, 4096, 1536, 1.2, "strided", 16, 2),
    "dsv3": (256, 8, 7168, 2048, 0.8, "remote_hot", 32, 4),
    "fine": (64, 6, 2048, 1408, 1.0, "remote_hot", 8, 2),
    "tiny": (6, 2, 256, 512, 1.2, "local_hot", 6, 2),
}


def _tile(T, K, E, dtype):
    """M-tile by rows per expert: 64 for decode batches, 128 up to 128 rows
    per expert, then 256 (128 for fp8 with fp32 scales)."""
    rows = T * K / E
    return 64 if rows <= 64 else 128 if rows <= 128 or dtype == "fp8" else 256


def _case(shape, dtype, T, plan, T_valid=None, m_tile=None, call="prepared", shared=False):
    E, K, H, I, zipf, placement, home, extra = SHAPES[shape] if isinstance(shape, str) else shape
    return dict(dtype=dtype, T=T, T_valid=T if T_valid is None else T_valid, K=K, E=E, H=H, I=I, zipf=zipf,
                placement=placement, home=home, extra=extra, plan=plan,
                m_tile=m_tile or _tile(T, K, E, dtype), call=call, shared=shared)


def listed():
    c = []

    def add(name, *a, **k):
        c.append(dict(name=name, **_case(*a, **k)))

    # the smallest layer of the tests and the smoke run: launches and latency
    add("tiny_bf16_96", "tiny", "bf16", 96, "uniform")
    # a nearly idle server: few tokens, each activating experts of its own, replicas sampled per pair
    add("decode_bf16_16", "qwen3", "bf16", 16, "sampled", call="forward")
    # an ordinary bf16 decode batch
    add("decode_bf16_512", "qwen3", "bf16", 512, "token_balancing")
    # decode of a Qwen3-FP8-like checkpoint (fp32 block scales), experts homed here with local replicas
    add("decode_fp8_1024", "qwen3_home", "fp8", 1024, "uniform")
    # decode of a DeepSeek-V3-like checkpoint: many slots, few rows each
    add("decode_dsv3_fp8_256", "dsv3", "fp8", 256, "uniform")
    # a padded graph batch with power-of-two scales, tile-aware split, replicas sharing their weights
    add("decode_fp8mx_999", "qwen3", "fp8mx", 999, "snap", T_valid=871, shared=True)
    # mixed batches (chunked prefill beside decode): some 90 to 125 rows per expert
    add("mixed_bf16_1499", "qwen3", "bf16", 1499, "uniform")
    add("mixed_dsv3_fp8_3001", "dsv3", "fp8", 3001, "uniform")
    # prefill in the three element types
    add("prefill_bf16_8192", "qwen3", "bf16", 8192, "uniform")
    add("prefill_fp8_8192", "qwen3", "fp8", 8192, "uniform")
    add("prefill_fp8mx_8192", "qwen3", "fp8mx", 8192, "uniform")
    # a fine-grained MoE (expert width an odd multiple of 128), stages called one by one around an all-to-all
    add("stages_fine_fp8mx_4097", "fine", "fp8mx", 4097, "replica_min", call="stages")
    return c


def _cost(case):
    """Rough seconds of a pass, to keep drawn cases below the largest listed one."""
    w = work(case)
    return w["bytes"] / 5e12 + w["flops"] / {"bf16": 0.8e15, "fp8": 0.55e15, "fp8mx": 1.6e15}[case["dtype"]]


def draw(rng):
    shape = rng.choice(["qwen3", "qwen3_home", "dsv3", "fine", "tiny", "any", "any"])
    if shape == "any":
        E = rng.choice([16, 24, 32, 64, 96])
        shape = (E, rng.randint(1, 8), 128 * rng.randint(2, 40), 128 * rng.randint(1, 16), rng.uniform(0.5, 1.2),
                 rng.choice(["strided", "remote_hot"]), E // 8, rng.randint(0, min(4, E // 8)))
    dtype = rng.choice(["bf16", "fp8", "fp8mx"])
    T = int(round(math.exp(rng.uniform(math.log(4), math.log(8192)))))
    call = rng.choice(["prepared", "prepared", "forward", "stages"])
    shared = rng.random() < 0.25
    plan = rng.choice(["uniform", "uniform", "token_balancing", "replica_min", "snap", "sampled"])
    padded = rng.random() < 0.3
    pad = rng.uniform(0.7, 1.0)
    largest = max(_cost(c) for c in listed() if c["T"] == 8192)
    while True:
        K, E = (SHAPES[shape] if isinstance(shape, str) else shape)[1::-1]
        p = "uniform" if plan == "sampled" and T * K > 8192 else plan
        case = _case(shape, dtype, T, p, T_valid=max(1, int(T * pad)) if padded else None, call=call, shared=shared)
        if _cost(case) <= largest or T <= 4:
            return case
        T = max(4, T * 2 // 3)


def _placement(case):
    if case["placement"] == "local_hot":
        return synth.placement_local_hot(case["E"], case["home"], case["extra"])
    if case["placement"] == "strided":
        return synth.placement_local_hot_strided(case["E"], case["home"], case["extra"])
    return synth.placement_remote_hot(case["E"], case["extra"])


def _plan(case, pl, ids):
    if case["plan"] == "token_balancing":
        return synth.plan_token_balancing(pl, case["E"], ids, case["T_valid"])
    return synth.plan_replica_min(pl, case["E"]) if case["plan"] == "replica_min" else synth.plan_uniform(pl, case["E"])


def _entries(pl, plan, E):
    """Per expert: its local slots and the integer weights of its entries
    (local slots in order, then the remote share), after the fallback of a
    row of zeros to equal weights."""
    slots = [[] for _ in range(E)]
    for s, e in enumerate(pl.slot_expert.tolist()):
        slots[e].append(s)
    rows = []
    for e in range(E):
        w = [int(plan.slot_weight[s]) for s in slots[e]] + [int(plan.remote_weight[e])]
        if sum(w) == 0:
            w = [1] * len(slots[e]) + [int(plan.remote_replicas[e])]
        rows.append(w)
    return slots, rows


def _split(case, n, slots, weights):
    """Pairs of one expert that each of its local slots takes, of n in all."""
    W, C, out = sum(weights), 0, []
    for w in weights[:len(slots)]:
        b = []
        for x in (n * C // W, n * (C + w) // W) if W else (0, 0):
            if case["plan"] == "snap" and x != n:
                x = min(n, (x + case["m_tile"] // 2) // case["m_tile"] * case["m_tile"])
            b.append(x)
        out.append((b[0], b[1]))
        C += w
    return out


def work(case):
    """Routing of a fixed seed: weights of the slots that get pairs, the rows
    of tokens with a local pair, ids and routing weights read once; y and the
    index outputs written once; 6 H I operations per local pair."""
    T, K, E, H, I = (case[k] for k in ("T", "K", "E", "H", "I"))
    ids, _ = synth.routing(T, K, E, case["zipf"], 0)
    pl = _placement(case)
    plan = _plan(case, pl, ids)
    slots, rows = _entries(pl, plan, E)
    n = np.bincount(ids[:case["T_valid"]].reshape(-1), minlength=E)
    counts = [hi - lo for e in range(E) for lo, hi in _split(case, int(n[e]), slots[e], rows[e])]
    G, N = sum(c > 0 for c in counts), sum(counts)
    es = 2 if case["dtype"] == "bf16" else 1
    held = np.isin(ids[:case["T_valid"]], [e for e in range(E) if slots[e] and sum(rows[e][:len(slots[e])])])
    scales = 0 if es == 2 else G * 3 * (H // 128) * (I // 128) * 4 + int(held.any(1).sum()) * (H // 128) * 4
    nbytes = G * 3 * H * I * es + int(held.any(1).sum()) * H * es + scales + T * K * 8 + T * H * 2 + T * K * 4
    return {"bytes": nbytes, "flops": 6 * H * I * N}


def tolerance(case):
    """About four times what two correct computations differ by: the kernels
    against a torch computation in fp32 that rounds h, y_perm and y where they
    do (bf16: flips of one ulp, at most 3.0e-4 and 2.0e-2 seen; fp8: flips of
    an e4m3 code of h, which move a whole down sum, at most 2.0e-3 and
    1.3e-1 seen)."""
    if case["dtype"] == "bf16":
        return {"rel": 1.2e-3, "max": 8e-2}
    return {"rel": 8e-3, "max": 5e-1}


def _generator(seed, stream):
    return torch.Generator(device="cuda").manual_seed(seed * 4099 + stream)


def _quantise(v, blocks, pow2):
    """fp32 [R, C] -> e4m3 bytes and fp32 scales, over blocks (rows, 128)."""
    R, C = v.shape
    b = v.view(R // blocks, blocks, C // 128, 128)
    amax = b.abs().amax(dim=(1, 3))
    sc = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
    if pow2:
        m, e = torch.frexp(sc)
        sc = torch.ldexp(torch.ones_like(sc), torch.where(m == 0.5, e - 1, e))
    q = (b / sc[:, None, :, None]).clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
    return q.view(R, C).view(torch.uint8), sc


def _routing(case, seed):
    """Top-K ids and softmax weights of Gaussian logits with a Zipf bias."""
    T, K, E = case["T"], case["K"], case["E"]
    bias = torch.from_numpy(np.log(synth.zipf_popularity(E, case["zipf"]))).float().cuda()
    z = torch.randn(T, E, generator=_generator(seed, 0), device="cuda") * synth.SIGMA + bias
    top = torch.topk(z, K, dim=1)
    return top.indices.to(torch.int32), torch.softmax(top.values, dim=1)


def _inputs(case, seed):
    T, H, I, dtype = case["T"], case["H"], case["I"], case["dtype"]
    ids, w = _routing(case, seed)
    pl = _placement(case)
    plan = _plan(case, pl, ids.cpu().numpy() if case["plan"] == "token_balancing" else None)
    x = torch.randn(T, H, generator=_generator(seed, 1), device="cuda")
    xs = None
    if dtype == "bf16":
        x = x.to(torch.bfloat16)
    else:
        x, xs = _quantise(x, 1, dtype == "fp8mx")
    return ids, w, pl, plan, x, xs


def _expert(case, seed, e):
    """Weights of logical expert e: w13 [2I, H], w2 [H, I] and their scales."""
    g, out = _generator(seed, 2 + e), []
    for R, C in ((2 * case["I"], case["H"]), (case["H"], case["I"])):
        v = torch.randn(R, C, generator=g, device="cuda") * 0.02
        out += [v.to(torch.bfloat16), None] if case["dtype"] == "bf16" else _quantise(v, 128, case["dtype"] == "fp8mx")
    return out


def _natural(case, seed, experts):
    """Weights of the slots in the natural layout."""
    parts = {e: _expert(case, seed, e) for e in set(experts)}
    col = [None if parts[experts[0]][i] is None else torch.stack([parts[e][i] for e in experts]) for i in range(4)]
    if case["dtype"] == "bf16":
        col[0], col[2] = col[0].view(torch.int16), col[2].view(torch.int16)
    return moe.WeightTensors(col[0], col[2], col[1], col[3])


def _shape(case, S, **k):
    return moe.MoEShape(T=k.get("T", case["T"]), T_valid=k.get("T_valid", case["T_valid"]), K=case["K"], E=case["E"],
                        S=S, H=case["H"], I=case["I"], m_tile=case["m_tile"], dtype=case["dtype"])


def prepare(case, seed):
    ids, w, pl, plan, x, xs = _inputs(case, seed)
    experts = pl.slot_expert.tolist()
    shape = _shape(case, len(experts))
    td = moe.to_device
    pt = moe.PlanTensors(td(pl.slot_expert), td(plan.slot_weight), td(plan.remote_weight), td(plan.remote_replicas),
                         snap_tiles=case["plan"] == "snap", sample_seed=seed if case["plan"] == "sampled" else None)
    if case["shared"]:
        one = {e: moe.pack_weights(_shape(case, 1), _natural(case, seed, [e])) for e in set(experts)}
        weights = moe.slot_table([one[e] for e in experts])
    else:
        weights = moe.pack_weights(shape, _natural(case, seed, experts))
    ws = moe.Workspace(shape)
    disp = moe.DispatchBuffers.allocate(shape, ws.row_cap)
    y = torch.empty(case["T"], case["H"], dtype=torch.int16, device="cuda")
    if case["dtype"] == "bf16":
        x = x.view(torch.int16)
    s = dict(call=case["call"], shape=shape, plan=pt, ids=ids, w=w, x=x, xs=xs, weights=weights, ws=ws, disp=disp, y=y)
    if case["call"] == "prepared":
        s["fwd"] = moe.PreparedForward(shape, pt, ids, w, x, xs, weights, disp, y, ws)
    elif case["call"] == "stages":
        s["y_perm"] = torch.empty(ws.row_cap, case["H"], dtype=torch.int16, device="cuda")
    return s


def run(s):
    if s["call"] == "prepared":
        s["fwd"]()
    elif s["call"] == "forward":
        moe.forward(s["shape"], s["plan"], s["ids"], s["w"], s["x"], s["xs"], s["weights"], s["disp"], s["y"], s["ws"])
    else:
        moe.dispatch(s["shape"], s["plan"], s["ids"], s["x"], s["xs"], s["disp"], s["ws"])
        moe.experts(s["shape"], s["disp"], s["weights"], s["y_perm"], s["ws"])
        moe.combine(s["shape"], s["disp"].pair_row, s["w"], s["y_perm"], s["y"])
    d = s["disp"]
    return s["y"].view(torch.bfloat16), d.expert_counts, d.slot_counts, d.slot_offsets, d.pair_row


def _assign(case, seed, ids, pl, plan):
    """Local slot of every pair (-1: remote or not held here), in numpy."""
    E, Pv = case["E"], case["T_valid"] * case["K"]
    flat = ids.reshape(-1).copy()
    flat[Pv:] = -1
    slots, rows = _entries(pl, plan, E)
    slot = np.full(flat.size, -1, np.int64)
    for e in range(E):
        p = np.flatnonzero(flat == e)
        if not slots[e] or not p.size:
            continue
        if case["plan"] != "sampled":
            for s, (lo, hi) in zip(slots[e], _split(case, p.size, slots[e], rows[e])):
                slot[p[lo:hi]] = s
            continue
        C = np.cumsum(rows[e])
        for i in p.tolist():  # numpy advances its counter before a block, so the block of counter i starts from i - 1
            c = [(i - 1) % 2**64] + [0 if i else 2**64 - 1] * 3
            bits = np.random.Philox(key=np.array([seed, 0], np.uint64), counter=np.array(c, np.uint64)).random_raw()
            j = int(np.searchsorted(C, ((int(bits) >> 32) * int(C[-1])) >> 32, side="right"))
            slot[i] = slots[e][j] if j < len(slots[e]) else -1
    return flat, slot


def _dequantise(q, sc, blocks):
    v = q.view(torch.float8_e4m3fn).double()
    return v * sc.double().repeat_interleave(blocks, 0).repeat_interleave(128, 1)


def exact(case, seed):
    ids, w, pl, plan, x, xs = _inputs(case, seed)
    E, S, M, K = case["E"], len(pl.slot_expert), case["m_tile"], case["K"]
    flat, slot = _assign(case, seed, ids.cpu().numpy(), pl, plan)
    counts = np.bincount(slot[slot >= 0], minlength=S)
    offsets = np.concatenate([[0], np.cumsum((counts + M - 1) // M * M)])
    row = np.full(flat.size, -1, np.int64)
    for s in range(S):
        p = np.flatnonzero(slot == s)
        row[p] = offsets[s] + np.arange(p.size)
    xd = x.double() if xs is None else _dequantise(x, xs, 1)
    y = torch.zeros(case["T"], case["H"], dtype=torch.float64, device="cuda")
    for e in sorted(set(pl.slot_expert.tolist())):
        p = torch.from_numpy(np.flatnonzero((flat == e) & (slot >= 0))).cuda()
        if not p.numel():
            continue
        a, sa, b, sb = _expert(case, seed, e)
        a = a.double() if sa is None else _dequantise(a, sa, 128)
        b = b.double() if sb is None else _dequantise(b, sb, 128)
        t = p // K
        g = xd[t] @ a.t().contiguous()
        g, u = g[:, :case["I"]], g[:, case["I"]:]
        o = (g / (1 + torch.exp(-g)) * u) @ b.t().contiguous()
        y.index_add_(0, t, o * w.reshape(-1)[p].double()[:, None])
    i32 = [torch.from_numpy(v.astype(np.int32)) for v in
           (np.bincount(flat[flat >= 0], minlength=E), counts, offsets, row.reshape(case["T"], K))]
    return (y, *i32)
