"""The work that a tuner has this library do, as cases that can be timed and compared.

One exploration round is: draw or keep a population of candidate schedules per tuned subgraph, score it with the draft
model and keep the best k (`prior_filter`, or the whole explorer loop `random_init` + `lse`), score the drafted set with
the learned cost model (`verify_score`, or `pacm_score` for the model with both branches), keep the best few (`topk`) and,
after training, let the Siamese weights follow (`moa_update`).  The cases are these calls over the sizes they are made
at: from one task of a few thousand candidates to twenty million candidates at once.

A case is a dict of plain values; `prepare` makes on the GPU what a tuner holds before the call (populations, features,
weights, preallocated outputs and workspaces), `run` is one pass through the public entry points.
"""
import numpy as np
import torch

import paper_2402_02361_amd as P
import workloads as W

MIB = 1 << 20


def listed():
    return [
        # one task, the smallest population a round scores: a handful of microseconds of GPU work, so launches and latency count
        {"name": "filter_gemm_4k", "kind": "filter", "tasks": "gemm", "n_tasks": 1, "each": 4096, "ragged": False, "k": 64, "flags": 0},
        # one convolution task with a large population: many tile slots, still a single short launch per stage
        {"name": "filter_conv_64k", "kind": "filter", "tasks": "conv", "n_tasks": 1, "each": 65536, "ragged": False, "k": 128, "flags": 0},
        # all twenty subgraphs of an encoder layer scored in one call: the ordinary whole-network round
        {"name": "filter_bert_20x50k", "kind": "filter", "tasks": "bert", "n_tasks": 20, "each": 50000, "ragged": False, "k": 512, "flags": 0},
        # tasks of every loop-nest class with odd population sizes, so that segments start at any alignment
        {"name": "filter_mixed_ragged_3m", "kind": "filter", "tasks": "mixed", "n_tasks": 10, "each": 333333, "ragged": True, "k": 512, "flags": 0},
        # the largest population: exhaustive-style scoring of two subgraphs, bound by memory bandwidth
        {"name": "filter_stress_21m", "kind": "filter", "tasks": "stress", "n_tasks": 2, "each": 10 * MIB, "ragged": False, "k": 4096, "flags": 0},
        # the explorer loop on one task at the population that a tuning round uses (8,000 explored, 512 drafted)
        {"name": "explore_gemm_8k", "kind": "explore", "tasks": "gemm", "n_tasks": 1, "each": 8000, "ragged": False, "k": 512, "steps": 4, "flags": 0},
        # the explorer loop with a population that fills the device
        {"name": "explore_stress_21m", "kind": "explore", "tasks": "stress", "n_tasks": 2, "each": 10 * MIB, "ragged": False, "k": 4096, "steps": 4, "flags": 0},
        # the learned model on one task's drafted set
        {"name": "verify_512", "kind": "verify", "n_d": 512, "group": 512},
        # the learned model on the drafted sets of many tasks in one call
        {"name": "verify_131k", "kind": "verify", "n_d": 131072, "group": 4096},
        # the model with both branches on the drafted sets of two tasks, and of many
        {"name": "pacm_8k", "kind": "pacm", "n_d": 8192, "group": 4096},
        {"name": "pacm_131k", "kind": "pacm", "n_d": 131072, "group": 4096},
        # a whole round over twenty tasks: draft, verify, the final selection, the momentum update of the weights
        {"name": "round_bert_20x50k", "kind": "round", "tasks": "bert", "n_tasks": 20, "each": 50000, "ragged": False, "k": 512, "flags": 0, "k_final": 32},
    ]


def _log_int(rng, lo, hi):
    return int(round(float(lo) * (float(hi) / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["filter"] * 4 + ["explore"] * 2 + ["verify"] * 2 + ["pacm"] * 2 + ["round"])
    if kind in ("verify", "pacm"):
        return {"kind": kind, "n_d": _log_int(rng, 200, 131072), "group": rng.choice([100, 512, 1000, 4096])}
    tasks = rng.choice(["gemm", "conv", "bert", "mixed", "stress"])
    n_tasks = {"gemm": 1, "conv": 1, "stress": 2}.get(tasks) or rng.randint(2, 20)
    if kind == "filter":
        n = _log_int(rng, max(4096, 500 * n_tasks), 11 * MIB)
    elif kind == "explore":
        n = _log_int(rng, max(4000, 500 * n_tasks), 4 * MIB)
    else:
        n = _log_int(rng, 2000 * n_tasks, 2 * MIB)
    case = {"kind": kind, "tasks": tasks, "n_tasks": n_tasks, "each": max(300, n // n_tasks), "ragged": rng.random() < 0.5,
            "flags": rng.choice([0, 0, 0, P.REFERENCE_ROUNDING, P.NO_COMPUTE_PENALTY, P.NO_MEMORY_PENALTY]) if kind != "round" else 0}
    smallest = min(_counts(case))
    case["k"] = max(k for k in (rng.choice([32, 64, 128]), rng.choice([64, 256, 500]), rng.choice([32, 512, 1000, 4096])) if k <= smallest // 4 or k <= 64)
    if kind == "explore":
        case["steps"] = rng.randint(2, 5)
    if kind == "round":
        case["k_final"] = rng.choice([10, 32])
    return case


# ---- the tasks of a population


def _subgraphs(tasks, n_tasks):
    frag = W.gemm(4096, 4096, 4096, dtype_bytes=2, sp_levels=4, rd_levels=3, frag=(16, 16, 16), name="gemm4096_fp16_frag16")
    depthwise = W.depthwise_conv2d(1, 512, 28, 28, 3, 3, stride=1, pad=1)
    conv = W.conv2d(1, 64, 56, 56, 64, 3, 3, stride=1, pad=1)
    if tasks == "gemm":
        return [W.gemm(512, 512, 512)] * n_tasks
    if tasks == "conv":
        return [conv] * n_tasks
    if tasks == "bert":
        return list(W.bert_base_subgraphs(n_tasks))
    if tasks == "stress":
        return [frag, depthwise]
    mixed = [conv, W.gemm(128, 3072, 768), depthwise, W.batched_gemm(12, 128, 128, 64), frag]
    return [mixed[t % len(mixed)] for t in range(n_tasks)]


def _counts(case):
    each, n_tasks = case["each"], case["n_tasks"]
    if case["tasks"] == "stress":   # four parts of the first subgraph to one of the second
        counts = [2 * each * 4 // 5, 2 * each // 5]
    else:
        counts = [each] * n_tasks
    if case["ragged"]:
        counts = [c + (t * 7919 + 5) % 97 - 48 for t, c in enumerate(counts)]
    return counts


def _population(case):
    sgs = _subgraphs(case["tasks"], case["n_tasks"])
    seg = np.zeros(len(sgs) + 1, dtype=np.int64)
    seg[1:] = np.cumsum(_counts(case))
    return sgs, seg, max(W.n_slots(s) for s in sgs)


def _generator(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + stream) & 0x7FFFFFFFFFFFFFFF)
    return g


def _draw_tiles(sgs, seg, rows, seed):
    """Per axis an ordered factorisation drawn uniformly from all of them (what RandomInitSch does), uint16 [rows, n]."""
    g = _generator(seed, 1)
    tiles = torch.zeros((rows, int(seg[-1])), dtype=torch.int16, device="cuda")
    for t, sg in enumerate(sgs):
        lo, hi = int(seg[t]), int(seg[t + 1])
        slot = 0
        for table in W.axis_tables(sg):
            columns = torch.from_numpy(np.ascontiguousarray(table.T).astype(np.int16)).cuda()
            pick = torch.randint(len(table), (hi - lo,), generator=g, device="cuda", dtype=torch.int32)
            for level in range(table.shape[1]):
                tiles[slot + level, lo:hi] = columns[level][pick]
            slot += table.shape[1]
    return tiles.view(torch.uint16)


def _statements(n_d, group):
    """Statements per candidate: 3 to 8, the same for the candidates that one task drafted."""
    return 3 + torch.div(torch.arange(n_d, device="cuda"), group, rounding_mode="floor") % 6


def _blocks(n_d, group):
    """Data-movement blocks per candidate; every sixth task is an element-wise operator and has none."""
    t = torch.div(torch.arange(n_d, device="cuda"), group, rounding_mode="floor")
    return (5 * t + 4) % 6 + 2 * (t % 6 == 2)


def _features(n_d, valid, rows, width, g):
    """Rows of log-scaled counters: half of the values zero, the others below 24; rows past a candidate's own are zero."""
    x = torch.rand((n_d, rows, width), generator=g, device="cuda")
    x = (x * 48.0 - 24.0).clamp_(min=0.0)
    x *= (torch.arange(rows, device="cuda")[None, :] < valid[:, None])[:, :, None]
    return x


def _to_gpu(weights):
    return {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() if isinstance(v, np.ndarray) else v for k, v in weights.items()}


def _workspace(which, n, n_sg, k):
    return torch.empty(max(256, P.workspace_bytes(which, n, n_sg, k)), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind, "seed": int(seed)}
    if kind in ("filter", "round", "explore"):
        sgs, seg, rows = _population(case)
        n, n_sg, k = int(seg[-1]), len(sgs), case["k"]
        s.update(csg=P.to_c_subgraphs(sgs), seg=seg, k=k, flags=case["flags"], rows=rows)
        s["score"] = torch.empty(n, dtype=torch.float32, device="cuda")
    if kind in ("filter", "round"):
        s["tiles"] = _draw_tiles(sgs, seg, rows, seed)
        s["idx"] = torch.empty((n_sg, k), dtype=torch.int32, device="cuda")
        s["val"] = torch.empty((n_sg, k), dtype=torch.float32, device="cuda")
        s["ws"] = _workspace(P.WS_PRIOR_FILTER, n, n_sg, k)
    if kind == "explore":
        s["steps"] = case["steps"]
        s["tiles"] = torch.empty((rows, n), dtype=torch.uint16, device="cuda")
        s["ws"] = _workspace(P.WS_LSE, n, n_sg, k)
        s["ws_init"] = torch.empty(max(256, int(P.load_library().pruner_random_init_workspace_bytes(s["csg"], n_sg))), dtype=torch.uint8, device="cuda")
    if kind == "round":
        n_d = n_sg * k
        s["seg_drafted"] = np.arange(n_sg + 1, dtype=np.int64) * k
        s["k_final"] = case["k_final"]
        s["fin"] = torch.empty((n_sg, case["k_final"]), dtype=torch.int32, device="cuda")
        s["fin_val"] = torch.empty((n_sg, case["k_final"]), dtype=torch.float32, device="cuda")
        s["ws_final"] = _workspace(P.WS_TOPK, n_d, n_sg, case["k_final"])
        g = _generator(seed, 3)
        n_w = 256 * 164 + 256 * 256 + 256   # the matrices that the momentum update adapts
        s["phi"] = torch.randn(n_w, generator=g, device="cuda") * 0.06
        s["phi_target"] = s["phi"] + torch.randn(n_w, generator=g, device="cuda") * 1e-3
        s["phi_bf16"] = torch.empty(n_w, dtype=torch.uint16, device="cuda")
    if kind in ("verify", "pacm", "round"):
        n_d, group = (case["n_d"], case["group"]) if kind != "round" else (n_d, k)
        g = _generator(seed, 2)
        s["n_stmt"] = _statements(n_d, group).to(torch.int32)
        s["feat"] = _features(n_d, s["n_stmt"], 8, 164, g)
        s["out"] = torch.empty(n_d, dtype=torch.float32, device="cuda")
        if kind == "pacm":
            s["n_blk"] = _blocks(n_d, group).to(torch.int32)
            s["flow"] = _features(n_d, s["n_blk"], 8, 23, g)
            s["weights"] = _to_gpu(W.make_pacm_weights(seed))
            s["ws_model"] = _workspace(P.WS_PACM, n_d, 0, 0)
        else:
            s["weights"] = _to_gpu(W.make_mlp_weights(seed))
            s["ws_model"] = _workspace(P.WS_VERIFY, n_d, 0, 0)
    return s


def run(s):
    kind = s["kind"]
    if kind == "explore":
        # a fresh population, then the loop on it: all on the device
        P.random_init(s["csg"], s["seg"], s["rows"], s["seed"], tiles=s["tiles"], workspace=s["ws_init"])
        score, spec_tiles, spec_score, spec_count = P.lse(s["csg"], s["seg"], s["tiles"], s["k"], s["steps"], s["seed"], 52429,
                                                          flags=s["flags"], score=s["score"], workspace=s["ws"])
        return {"score": score, "spec_tiles": spec_tiles.view(torch.int16), "spec_score": spec_score, "spec_count": spec_count,
                "population": s["tiles"].view(torch.int16)}
    out = {}
    if kind in ("filter", "round"):
        score, idx, val = P.prior_filter(s["csg"], s["seg"], s["tiles"], s["k"], flags=s["flags"], score=s["score"], idx_out=s["idx"],
                                         val_out=s["val"], workspace=s["ws"])
        out.update(score=score, idx=idx, val=val)
    if kind in ("verify", "round"):
        out["verify"] = P.verify_score(s["feat"], s["n_stmt"], s["weights"], vscore=s["out"], workspace=s["ws_model"])
    if kind == "pacm":
        out["pacm"] = P.pacm_score(s["feat"], s["n_stmt"], s["flow"], s["n_blk"], s["weights"], y=s["out"], workspace=s["ws_model"])
    if kind == "round":
        out["final"], out["final_val"] = P.topk(out["verify"], s["seg_drafted"], s["k_final"], idx_out=s["fin"], val_out=s["fin_val"],
                                                workspace=s["ws_final"])
        # the round's weights stay as they are beside the updated ones
        out["phi"] = P.moa_update(s["phi"].clone(), s["phi_target"], 0.99, bf16=s["phi_bf16"])
        out["phi_bf16"] = s["phi_bf16"].view(torch.int16)
    return out


# ---- what a pass cannot do without


def work(case):
    kind = case["kind"]
    b = f = 0.0
    if kind in ("filter", "round", "explore"):
        sgs, seg, rows = _population(case)
        for sg, c in zip(sgs, np.diff(seg)):
            slots = W.n_slots(sg)
            if kind == "explore":   # the last population and its scores go out; every step mutates and scores each candidate
                b += float(c) * (2 * rows + 4) + case["k"] * (2.0 * rows + 4)
                f += float(c) * case["steps"] * (2 * slots + 60 + 60)
            else:                   # tile factors in, a score out, the k best out
                b += float(c) * (2 * slots + 4) + 8.0 * case["k"]
                f += float(c) * (2 * slots + 60)
    if kind in ("verify", "pacm", "round"):
        n_d, group = (case["n_d"], case["group"]) if kind != "round" else (case["n_tasks"] * case["k"], case["k"])
        t = np.arange(n_d) // group
        rows = float((3 + t % 6).sum())
        b += rows * 656 + n_d * 8.0 + 2 * (256 * 164 + 256 * 256)
        f += rows * 2 * (164 * 256 + 256 * 256)
        if kind == "pacm":
            blk = ((5 * t + 4) % 6 + 2 * (t % 6 == 2)).astype(np.float64)
            b += float(blk.sum()) * 92 + n_d * 4.0 + 2 * (64 * 23 + 4 * 64 * 64 + 320 * 256)
            f += float(blk.sum()) * 2 * (23 * 64 + 4 * 64 * 64) + float((blk ** 2).sum()) * 4 * 64 + n_d * 2.0 * (320 * 256 + 256)
        else:
            f += rows * 2 * 256
    if kind == "round":
        b += (256 * 164 + 256 * 256 + 256) * 14.0 + case["n_tasks"] * case["k_final"] * 8.0
    return {"bytes": b, "flops": f}


def tolerance(case):
    kind = case["kind"]
    if kind == "explore":
        # integer draws, and selections that decide what the next step draws from: another last bit of one score is another run
        return "exact"
    if kind == "filter":
        if case["flags"] & P.REFERENCE_ROUNDING or sum(_counts(case)) < MIB:
            return "exact"   # one correctly rounded operation per step of Eq. 1
        # the two binary32 forms of Eq. 1 are 1.0e-7 apart in norm and 3.4e-7 in the worst candidate; candidates that far apart may trade ranks
        return {"rel": 4e-7, "max": 1.4e-6, "differ": 0.01}
    if kind == "pacm":
        # against the same roundings to bfloat16 with binary64 sums: up to 3.7e-3 in norm, 2.1e-2 in the worst candidate
        # (a pooled sum of eight activations that falls on the other side of a rounding boundary moves the whole candidate)
        return {"rel": 1.5e-2, "max": 8e-2}
    # against the same roundings to bfloat16 with binary64 sums: up to 4.9e-5 in norm, 2.4e-3 in the worst candidate
    return {"rel": 2e-4, "max": 1e-2, "differ": 0.005}


# ---- the same results in 64 bits, in plain torch


def _exact_scores(sg, tiles, flags):
    """-L_total of every column: symbols as integers, penalties and Eq. 1 in binary64 (the order of Alg. 2)."""
    hw, n_sp, n_rd = sg.hw, sg.n_sp, sg.n_rd
    spatial = [[tiles[4 * a + l].to(torch.int64) for l in range(4)] for a in range(n_sp)]
    at = 4 * n_sp
    reduction = [[tiles[at + sg.rd_levels * r + l].to(torch.int64) for l in range(sg.rd_levels)] for r in range(n_rd)]
    block = [v * t * i for _, v, t, i in spatial] + [f[1] * f[2] if sg.rd_levels == 3 else f[1] for f in reduction]
    register = [v * i for _, v, _, i in spatial] + [f[2] if sg.rd_levels == 3 else torch.ones_like(f[1]) for f in reduction]

    def product(v):
        p = torch.ones_like(tiles[0], dtype=torch.int64)
        for x in v:
            p = p * x
        return p

    def extent(dim, e):
        return 1 + sum(coef * (e[axis] - 1) for axis, coef in dim)

    def footprint(buffer, e):
        return product([extent(d, e) for d in buffer.dims])

    def up(a, b):
        return torch.div(a + (b - 1), b, rounding_mode="floor")

    outer = product([f[0] for f in reduction])
    lanes = product(register[:n_sp])
    s1 = lanes + sum(footprint(x, register) for x in sg.inputs)
    s2 = 2 * lanes * product(register[n_sp:])
    s3 = sg.dtype_bytes * sum(footprint(x, block) for x in sg.inputs)
    s4 = product([t for _, _, t, _ in spatial])
    s6 = product([g for g, _, _, _ in spatial])
    whole = 1
    for e in sg.extent:
        whole *= e
    fragments = 1.0
    if tuple(sg.frag) != (0, 0, 0):
        s4, s1 = s4 * hw.n_l1, up(s1, hw.n_l1)
        inner = (spatial[n_sp - 2][3], spatial[n_sp - 1][3], register[-1])
        for x, f in zip(inner, sg.frag):
            fragments = fragments * (x.double() / (up(x, f) * f).double())
    warps = up(s4, hw.n_l1)
    u_p, u_m = float(hw.T_p), float(hw.T_m)
    if not flags & P.NO_COMPUTE_PENALTY:
        u_p = u_p * (1 + s2.double() / s1.double()) * (warps.double() / (up(warps, hw.pu_l1) * hw.pu_l1).double())
        u_p = u_p * (s4.double() / (warps * hw.n_l1).double()) * (s6.double() / (up(s6, hw.pu_l2) * hw.pu_l2).double()) * fragments
    total = 2.0 * whole / u_p
    spatial_whole = 1
    for e in sg.extent[:n_sp]:
        spatial_whole *= e
    moved = [(sg.dtype_bytes * s6 * outer * footprint(x, block), extent(x.dims[-1], block)) for x in sg.inputs]
    moved.append((torch.full_like(s6, sg.dtype_bytes * spatial_whole), extent(sg.out.dims[-1], block)))
    for s5, s7 in moved:
        u = u_m
        if not flags & P.NO_MEMORY_PENALTY:
            u = u_m * torch.clamp(hw.m_l0 / s1.double(), max=1.0) * torch.clamp(hw.m_l1 / s3.double(), max=1.0)
            u = u * (s7.double() / (up(s7, hw.n_l2) * hw.n_l2).double())
        total = total + s5.double() / u
    return -total


def _bf16_bits(t):
    return (t.view(torch.int16).to(torch.int32) << 16).view(torch.float32).double()


def _hidden(s, lo, hi):
    w = s["weights"]
    x = s["feat"][lo:hi].double()
    x = torch.relu(x @ _bf16_bits(w["W1"]).T + w["b1"].double())
    return torch.relu(x @ _bf16_bits(w["W2"]).T + w["b2"].double())


def _exact_verify(s):
    w, parts = s["weights"], []
    for lo in range(0, len(s["n_stmt"]), 16384):
        hi = min(lo + 16384, len(s["n_stmt"]))
        y = (_hidden(s, lo, hi) * _bf16_bits(w["w3"])).sum(-1) + w["b3"]
        parts.append((y * (torch.arange(8, device="cuda")[None] < s["n_stmt"][lo:hi, None])).sum(1))
    return torch.cat(parts)


def _exact_pacm(s):
    w, parts = s["weights"], []
    for lo in range(0, len(s["n_stmt"]), 16384):
        hi = min(lo + 16384, len(s["n_stmt"]))
        place = torch.arange(8, device="cuda")[None]
        v_s = (_hidden(s, lo, hi) * (place < s["n_stmt"][lo:hi, None])[:, :, None]).sum(1)
        there = place < s["n_blk"][lo:hi, None]
        e = torch.relu(s["flow"][lo:hi].double() @ _bf16_bits(w["We"]).T + w["be"].double())
        q, k, v = (e @ _bf16_bits(w[m]).T for m in ("Wq", "Wk", "Wv"))
        a = (q[:, :, None, :] * k[:, None, :, :]).sum(-1) / 8
        a = torch.softmax(torch.where(there[:, None, :], a, torch.full_like(a, -1e300)), dim=-1)
        o = (a[:, :, :, None] * v[:, None, :, :]).sum(2)
        z = (e + o @ _bf16_bits(w["Wo"]).T) * there[:, :, None]
        g = torch.relu(torch.cat([v_s, z.sum(1)], 1) @ _bf16_bits(w["Wh"]).T + w["bh"].double())
        parts.append((g * _bf16_bits(w["wo"])).sum(-1) + w["bo"])
    return torch.cat(parts)


def _best(x, seg, k):
    return torch.stack([torch.topk(x[int(seg[t]):int(seg[t + 1])], k, sorted=True).values for t in range(len(seg) - 1)])


def exact(case, seed):
    kind = case["kind"]
    if kind == "explore":
        return None   # a loop of integer draws and selections: every bit is compared instead
    s = prepare(case, seed)
    out = {}
    if kind in ("filter", "round"):
        sgs, seg, _ = _population(case)
        tiles = s["tiles"].view(torch.int16)
        parts = []
        for t, sg in enumerate(sgs):
            for lo in range(int(seg[t]), int(seg[t + 1]), MIB):
                parts.append(_exact_scores(sg, tiles[:, lo:min(lo + MIB, int(seg[t + 1]))], case["flags"]))
        score = torch.cat(parts)
        out.update(score=score, idx=None, val=_best(score, seg, case["k"]))
    if kind in ("verify", "round"):
        out["verify"] = _exact_verify(s)
    if kind == "pacm":
        out["pacm"] = _exact_pacm(s)
    if kind == "round":
        out["final"], out["final_val"] = None, _best(out["verify"], s["seg_drafted"], case["k_final"])
        m = float(np.float32(0.99))
        out["phi"] = m * s["phi"].double() + (1.0 - m) * s["phi_target"].double()
        out["phi_bf16"] = None
    return out
