"""The plan-search workloads that stand for the use of this library, for timing.

A case is one call pattern of a planner: a model's layers and a cluster's GPU
islands come in, scores, surviving candidates and a pipeline plan come out.
Every case goes through the public entry points of
`paper_2606_16907_amd.tangram`.  `listed()` holds the named cases, `draw()`
gives more of the same ranges, and `exact()` recomputes the floating-point
results with plain numpy and torch in 64 bits.

Kinds (the field "kind" of a case):
  search   score every candidate, prune, compose, on kept buffers: a planner
           that re-evaluates one cluster (bench.py's step)
  replan   the cluster changed (a node failed, a link was re-measured): build
           the problem from host tables, search, release
  prune    the surviving set of scores that are on the device already
  relaxed  composition with the bound relaxed (step (4)) of a kept surviving set
  orders   composition over every island order of a kept surviving set
  classes  the search with redundancy pruning (one score per slice class)
  islands  island construction from node measurements

Island sizes belong to the case (drawn from its "cluster" number); GPU rates,
memory sizes, link speeds, the efficiency and memory fractions and node
measurements are drawn from the seed.
"""
import random

import numpy as np
import torch

from paper_2606_16907_amd import tangram as T

LAYER_FIELDS = ("fwd_flops", "dense_params", "expert_params", "act_stash_bytes", "tp_comm_bytes", "a2a_bytes",
                "out_act_bytes", "cp_comm_bytes")
STAGE_INTS = ("island", "first_layer", "end_layer", "tp", "cp", "dp", "ep", "zero", "recompute", "offload", "mb",
              "depth", "pair_index")
STAGE_FLOATS = ("cost", "mem_bytes", "link_out")

DENSE = {"hidden": 4096, "heads": 32, "kv": 8, "ffn": 14336, "swiglu": True, "seq": 4096, "experts": 0, "top_k": 0,
         "uneven": False}
MOE = {"hidden": 6144, "heads": 48, "kv": 8, "ffn": 4096, "swiglu": True, "seq": 4096, "experts": 64, "top_k": 2,
       "uneven": False}
SPACE = {"tp": "1,2,4,8", "mb": "1,2,4,8", "ep": "1", "zero": "0,1,2,3", "cp": "1", "rc": "0", "of": "0", "eps": 0.0}
EXTENDED = {"cp": "1,2,4", "rc": "0,1", "of": "0,1"}
# the 70B-class decoder and the 128-layer decoder of bench.py
D70 = dict(DENSE, hidden=8192, heads=64, ffn=28672, seq=8192)
D128 = dict(DENSE, hidden=12288, heads=96, kv=96, ffn=49152, swiglu=False, seq=8192)


def _case(name, kind, model, layers, islands, nodes, gpus, types, fabric, batch, cluster, **space):
    c = {"name": name, "kind": kind, "layers": layers, "islands": islands, "nodes": nodes, "gpus": gpus,
         "types": types, "fabric": fabric, "batch": batch, "cluster": cluster}
    c.update(model)
    c.update(SPACE)
    c.update(space)
    return c


def listed():
    return [
        # the smallest call: a laptop-size what-if, two islands of 4 GPUs; latency and launches
        _case("search_tiny", "search", dict(DENSE, hidden=1024, heads=16, kv=16, ffn=4096, swiglu=False, seq=2048),
              8, 2, 1, 4, 2, False, 64, 1, tp="1,2,4", mb="1,2,4"),
        # an 8B-class model on four 8-GPU nodes of different generations
        _case("search_8b", "search", DENSE, 32, 4, 1, 8, 4, False, 512, 2),
        # a mixture-of-experts model on 32 islands, expert parallelism searched
        _case("search_moe", "search", MOE, 48, 32, 4, 8, 4, False, 2048, 4, ep="1,2,4,8,16"),
        # uneven layers (embedding, head, alternating expert layers), an odd layer count, 27 islands of odd
        # sizes, a batch with a factor of 3, imbalance pruning on
        _case("search_uneven", "search", dict(MOE, hidden=5120, heads=40, ffn=3072, uneven=True), 61, 27, 5, 6, 3,
              False, 1536, 6, ep="1,2,4,8", eps=1.0),
        # a 70B-class model with context parallelism, recomputation and offloading searched as well
        _case("search_70b_extended", "search", D70, 80, 16, 8, 8, 3, False, 1024, 3, **EXTENDED),
        # the largest: 128 layers on 128 islands behind a three-level fabric, 1e9 candidates
        _case("search_128", "search", D128, 128, 128, 8, 8, 5, True, 4096, 5),
        # a node failed or joined: the problem is built anew from host tables, then searched
        _case("replan_70b", "replan", D70, 80, 16, 8, 8, 3, False, 1024, 3),
        # the surviving set of a large group space (expert parallelism with the extended space)
        _case("prune_moe_extended", "prune", MOE, 48, 32, 4, 8, 4, False, 2048, 4, ep="1,2,4,8,16", **EXTENDED),
        # composition with the bound relaxed, for the least iteration time, 96 layers on 64 islands
        _case("relaxed_96", "relaxed", dict(D128, hidden=8192, heads=64, kv=64, ffn=32768), 96, 64, 6, 8, 4, True,
              2048, 7),
        # composition over every order of 16 islands
        _case("orders_70b", "orders", D70, 80, 16, 8, 8, 3, False, 1024, 3),
        # the search with redundancy pruning on the largest instance
        _case("classes_128", "classes", D128, 128, 128, 8, 8, 5, True, 4096, 5),
        # grouping the 1024 nodes of a cluster into islands
        {"name": "islands_1024", "kind": "islands", "n": 1024, "types": 5, "leaf": 8, "asym": 0.0},
    ]


# no drawn case is larger than the listed case of its kind: candidates, then table cells times micro-batch sizes
MOST = {"search": (1.0e9, 1.05e7), "classes": (1.0e9, 1.05e7), "replan": (6.0e7, 5.1e5), "prune": (2.5e8, 1.0e7),
        "relaxed": (2.3e8, 2.6e6), "orders": (6.0e7, 5.1e5)}


def draw(rng):
    def log_int(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    while True:
        kind = rng.choice(["search", "search", "search", "search", "replan", "prune", "relaxed", "orders", "classes",
                           "islands"])
        if kind == "islands":
            # links measured one by one ("asym") leave many small islands, at a far higher cost per node
            asym = rng.choice([0.0, 0.0, 0.0, 0.01])
            return {"kind": kind, "n": log_int(40, 400 if asym else 1000), "types": rng.randint(2, 6),
                    "leaf": rng.choice([4, 8, 16]), "asym": asym}
        moe = rng.random() < 0.35
        heads = rng.choice([32, 40, 48, 64, 80, 96] if kind == "prune" else [16, 24, 32, 40, 48, 64, 80, 96])
        hidden = 128 * heads
        model = {"hidden": hidden, "heads": heads, "kv": rng.choice([8, heads]), "swiglu": rng.random() < 0.6,
                 "ffn": int(hidden * rng.choice([0.5, 0.75, 1.0])) if moe else int(hidden * rng.choice([2.67, 3.5, 4])),
                 "seq": rng.choice([2048, 4096, 8192]), "experts": rng.choice([8, 16, 64, 96]) if moe else 0,
                 "top_k": rng.choice([1, 2, 4]) if moe else 0, "uneven": rng.random() < 0.3}
        c = _case("", kind, model, log_int(24 if kind == "prune" else 6, 128),
                  log_int(2, 16 if kind == "orders" else 128), rng.randint(1, 8), rng.choice([4, 6, 8, 8, 8]),
                  rng.randint(2 if kind == "prune" else 1, 5), rng.random() < 0.5,
                  rng.choice([1, 1, 3, 5]) * 2 ** rng.randint(6, 11), rng.randrange(1 << 20),
                  ep=rng.choice(["1,2,4,8", "1,2,4,8,16"]) if moe else "1",
                  tp=rng.choice(["1,2,4", "1,2,4,8", "1,2,4,8", "1,2,3,4,6"]),
                  mb=rng.choice(["1,2,4", "1,2,4,8", "1,2,3,4,6"]), zero=rng.choice(["0,1,2,3", "0,1,2,3", "1,3"]),
                  eps=rng.choice([0.0, 0.0, 0.0, 1.0, 2.0]))
        del c["name"]
        if rng.random() < 0.25:
            c.update(EXTENDED)
        if not _holds(c):
            continue
        ns, n, _ = _sizes(c)
        if kind == "replan" and n > 4e4 * ns:  # configs: a problem's tables grow with them
            continue
        if n <= MOST[kind][0] and _b_count(c) * ns * c["islands"] <= MOST[kind][1]:
            return c


def _holds(c):
    """A model this cluster is bought for: its training state is well under the
    cluster's memory, the activations a GPU keeps are under a card's, and, with
    imbalance pruning, a layer is no larger than an island's share."""
    rows, counts = _layers(c), _gpu_counts(c)
    split = min(max(_ints(c["tp"])), c["gpus"])
    state = 16.0 * (sum(rows["dense_params"]) + sum(rows["expert_params"]))
    per_layer = max(16.0 * (d / split + e / min(counts)) for d, e in zip(rows["dense_params"], rows["expert_params"]))
    return (state <= 0.35 * 80e9 * sum(counts) and per_layer <= 24e9
            and sum(rows["act_stash_bytes"]) / split <= 60e9
            and (c["eps"] == 0 or 2 * c["islands"] <= c["layers"]))


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------
def _ints(text):
    return [int(x) for x in str(text).split(",")]


def _gpu_counts(case):
    rng = random.Random(case["cluster"])
    return [case["gpus"] * rng.randint(1, case["nodes"]) for _ in range(case["islands"])]


def _layer(case, moe):
    s, h, f = case["seq"], case["hidden"], case["ffn"]
    h_kv = case["kv"] * (h // case["heads"])
    mats = 3 if case["swiglu"] else 2
    flops = 2 * s * h * (h + 2 * h_kv) + 2 * s * h * h + 4 * s * s * h
    params = h * (h + 2 * h_kv) + h * h + 2 * h
    stash = 10 * s * h + 2 * s * (h + 2 * h_kv) + 2 * s * h
    if moe:
        e, k = case["experts"], case["top_k"]
        return [flops + 2 * s * h * e + k * 3 * 2 * s * h * f, params + h * e, e * 3 * h * f,
                stash + k * (6 * s * f + 2 * s * h), 4 * s * h, 2 * (k * s) * h * 2, 2 * s * h, 4 * s * h_kv]
    return [flops + mats * 2 * s * h * f, params + mats * h * f, 0, stash + (6 if case["swiglu"] else 4) * s * f,
            4 * s * h, 0, 2 * s * h, 4 * s * h_kv]


def _layers(case):
    """Per-layer integers.  An uneven model has an embedding before its first
    layer, a head after its last, and experts on every second layer only."""
    rows = []
    for l in range(case["layers"]):
        row = _layer(case, case["experts"] > 0 and (not case["uneven"] or l % 2 == 1))
        if case["uneven"] and l in (0, case["layers"] - 1):
            row[1] += 65536 * case["hidden"]
            if l:
                row[0] += 2 * case["seq"] * case["hidden"] * 65536
                row[3] += 4 * case["seq"] * 65536
        rows.append(row)
    return {f: [r[q] for r in rows] for q, f in enumerate(LAYER_FIELDS)}


def _instance(case, seed):
    rng = np.random.default_rng([int(seed), 17])
    K = case["islands"]
    kinds = [(round(float(rng.uniform(100.0, 1000.0)), 1) * 1e12, float(rng.choice([40, 80, 141, 192])) * 1e9,
              round(float(rng.uniform(300.0, 900.0)), 1) * 1e9) for _ in range(case["types"])]
    if max(k[1] for k in kinds) < 100e9:  # a cluster bought for this model has some large-memory GPUs
        kinds[0] = (kinds[0][0], 141e9, kinds[0][2])
    of = [k if k < len(kinds) else int(rng.integers(0, len(kinds))) for k in range(K)]
    rng.shuffle(of)
    islands = {"n_gpus": _gpu_counts(case), "peak_flops": [kinds[t][0] for t in of],
               "hbm_bytes": [kinds[t][1] for t in of], "intra_bw": [kinds[t][2] for t in of],
               "host_bw": [64e9 if kinds[t][1] >= 100e9 else 32e9 for t in of]}
    place = [0] * K
    if case["fabric"]:  # leaves of 4 islands, spines of 16
        for slot, k in enumerate(rng.permutation(K)):
            place[int(k)] = slot
        inter = [[0.0 if a == b else 400e9 if place[a] // 4 == place[b] // 4 else
                  100e9 if place[a] // 16 == place[b] // 16 else 25e9 for b in range(K)] for a in range(K)]
    else:
        nic = [round(float(rng.uniform(12.5, 50.0)), 2) * 1e9 for _ in range(K)]
        inter = [[0.0 if a == b else min(nic[a], nic[b]) for b in range(K)] for a in range(K)]
    order = sorted(range(K), key=lambda k: ((place[k] // 16, place[k] // 4) if case["fabric"] else ()) + (
        -islands["hbm_bytes"][k], -islands["peak_flops"][k], -islands["n_gpus"][k], k))
    space = {"global_batch": case["batch"], "n_experts": case["experts"], "tp": _ints(case["tp"]),
             "ep": _ints(case["ep"]), "mb": _ints(case["mb"]), "zero": _ints(case["zero"]), "cp": _ints(case["cp"]),
             "recompute": _ints(case["rc"]), "offload": _ints(case["of"]), "eta": round(float(rng.uniform(0.35, 0.65)), 3),
             "mem_frac": round(float(rng.uniform(0.8, 0.95)), 3), "imbalance_eps": case["eps"]}
    return {"layers": _layers(case), "islands": islands, "inter_bw": inter, "space": space, "island_order": order}


def _cluster(case, seed):
    """Nodes bought in runs of one GPU type, measured with 2% spread, behind a
    leaf/pod fabric; with "asym" each direction of each link deviates."""
    n = case["n"]
    rng = np.random.default_rng([int(seed), 29])
    kinds = [(round(float(rng.uniform(100.0, 1000.0)), 1) * 1e12, float(rng.choice([40, 80, 141, 192])) * 1e9,
              round(float(rng.uniform(300.0, 900.0)), 1) * 1e9) for _ in range(case["types"])]
    of = []
    while len(of) < n:
        of += [int(rng.integers(0, len(kinds)))] * int(rng.integers(4, 49))
    jitter = rng.uniform(-0.02, 0.02, size=(n, 2))
    nodes = {"gpus": [8] * n,
             "peak_flops": [round(kinds[of[u]][0] * (1.0 + jitter[u, 0]), -6) for u in range(n)],
             "hbm_bytes": [kinds[of[u]][1] for u in range(n)],
             "intra_bw": [round(kinds[of[u]][2] * (1.0 + jitter[u, 1]), -3) for u in range(n)],
             "host_bw": [64e9 if kinds[of[u]][1] >= 100e9 else 32e9 for u in range(n)]}
    u = np.arange(n)
    leaf, pod = u // case["leaf"], u // (4 * case["leaf"])
    e = np.where(leaf[:, None] == leaf[None, :], 400e9, np.where(pod[:, None] == pod[None, :], 100e9, 25e9))
    if case["asym"]:
        e = np.round(e * (1.0 + case["asym"] * rng.uniform(-1.0, 1.0, size=(n, n))), -3)
    np.fill_diagonal(e, 0.0)
    return {"nodes": nodes, "node_bw": e, "eps": {"compute": 0.1, "memory": 0.1, "intra": 0.1}}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "islands":
        n = case["n"]
        ws = T.load_library().tg_build_islands_workspace_bytes(n)
        return {"kind": kind, "cluster": _cluster(case, seed),
                "ws": torch.empty(int(ws), dtype=torch.uint8, device="cuda"), "bw": np.zeros((n, n)),
                "islands": np.zeros((5, n))}
    inst = _instance(case, seed)
    ns, n, ok = _sizes(case)
    p = T.Problem(inst)
    depth = min(case["layers"], case["islands"])
    s = {"kind": kind, "p": p, "inst": inst, "order": inst["island_order"], "depth": depth}
    # the buffers a planner sizes once and keeps; eight survivors for every (slice, island, micro-batch size)
    room = min(ok, 8 * _b_count(case) * ns * case["islands"])
    s["surv"] = torch.zeros(max(room, 1), dtype=torch.int64, device="cuda")
    if kind == "classes":
        s["cost"], s["dmax"] = p.tg_score_classes()
        s["pws"] = p.prune_classes_workspace()
        found = p.tg_prune_classes(s["cost"], s["dmax"], survivors=s["surv"], workspace=s["pws"])
    else:
        s["cost"], s["dmax"] = p.tg_score_pairs()
        s["pws"] = p.prune_workspace()
        found = p.tg_prune(s["cost"], s["dmax"], survivors=s["surv"], workspace=s["pws"])
    s["n"] = int(found.numel())
    if kind in ("search", "classes", "replan"):
        s["cws"] = p.compose_workspace(s["n"])
    elif kind == "relaxed":
        s["cws"] = p.compose_relaxed_workspace(s["n"])
    elif kind == "orders":
        s["cws"] = p.compose_all_orders_workspace(s["n"])
    if kind == "replan":  # the cluster changes: the old problem goes, the buffers stay
        p.close()
        s["p"] = None
    return s


# ----------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------
def _plan(s, status, plan):
    ints = np.zeros((s["depth"], len(STAGE_INTS)), dtype=np.int64)
    floats = np.zeros((s["depth"], len(STAGE_FLOATS)))
    st = plan["stages"]
    if st:
        ints[:len(st)] = [[x[f] for f in STAGE_INTS] for x in st]
        floats[:len(st)] = [[x[f] for f in STAGE_FLOATS] for x in st]
    return {"head": np.array([status, plan["b"], plan["m"], plan["S"]], dtype=np.int64),
            "pft": np.array([plan["P"], plan["F"], plan["T"]], dtype=np.float64),
            "stage_int": ints, "stage_float": floats}


def run(s):
    kind = s["kind"]
    if kind == "islands":
        r = T.build_islands(s["cluster"], workspace=s["ws"])
        k = r["K"]
        s["bw"][:k, :k] = r["inter_bw"]
        for q, f in enumerate(("n_gpus", "peak_flops", "hbm_bytes", "intra_bw", "host_bw")):
            s["islands"][q, :k] = r["islands"][f]
        return {"K": k, "island_of": np.array(r["island_of"]), "islands": s["islands"], "inter_bw": s["bw"]}
    p, cost, dmax = s["p"], s["cost"], s["dmax"]
    if kind == "search":
        p.tg_score_pairs(0, p.N, cost, dmax)
        found = p.tg_prune(cost, dmax, survivors=s["surv"], workspace=s["pws"])
        plan = _plan(s, *p.tg_compose_pipeline(found, cost, dmax, s["order"], workspace=s["cws"]))
        return {"cost": cost, "dmax": dmax, "n": found.numel(), "survivors": s["surv"], "plan": plan}
    if kind == "replan":
        p = T.Problem(s["inst"])
        p.tg_score_pairs(0, p.N, cost, dmax)
        found = p.tg_prune(cost, dmax, survivors=s["surv"], workspace=s["pws"])
        plan = _plan(s, *p.tg_compose_pipeline(found, cost, dmax, s["order"], workspace=s["cws"]))
        p.close()
        return {"cost": cost, "dmax": dmax, "n": found.numel(), "survivors": s["surv"], "plan": plan}
    if kind == "classes":
        p.tg_score_classes(0, cost.numel(), cost, dmax)
        found = p.tg_prune_classes(cost, dmax, survivors=s["surv"], workspace=s["pws"])
        plan = _plan(s, *p.tg_compose_pipeline_classes(found, cost, dmax, s["order"], workspace=s["cws"]))
        return {"cost": cost, "dmax": dmax, "n": found.numel(), "survivors": s["surv"], "plan": plan}
    if kind == "prune":
        found = p.tg_prune(cost, dmax, survivors=s["surv"], workspace=s["pws"])
        return {"n": found.numel(), "survivors": s["surv"]}
    found = s["surv"][:s["n"]]
    if kind == "relaxed":
        return {"plan": _plan(s, *p.tg_compose_pipeline_relaxed(found, cost, dmax, s["order"], workspace=s["cws"]))}
    return {"plan": _plan(s, *p.tg_compose_pipeline_all_orders(found, cost, dmax, workspace=s["cws"]))}


# ----------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------
def _configs(case):
    """Every island's configs in candidate order: rows (k, tp, cp, dp, ep, z, rc, of, mb)."""
    out = []
    cps, rcs, ofs, zs, mbs = (_ints(case[f]) for f in ("cp", "rc", "of", "zero", "mb"))
    for k, n in enumerate(_gpu_counts(case)):
        for tp in _ints(case["tp"]):
            for cp in cps:
                for dp in range(1, n // (tp * cp) + 1):
                    for ep in _ints(case["ep"]):
                        if dp % ep or (ep != 1 if case["experts"] == 0 else case["experts"] % ep):
                            continue
                        out += [(k, tp, cp, dp, ep, z, rc, of, mb) for z in zs for rc in rcs for of in ofs for mb in mbs]
    return np.array(out, dtype=np.int64).reshape(-1, 9)


def _sizes(case):
    """Slices, candidates, candidates whose micro-batch divides the batch."""
    ns = case["layers"] * (case["layers"] + 1) // 2
    cfg = _configs(case)
    ok = int(np.sum(case["batch"] % (cfg[:, 3] * cfg[:, 8]) == 0))
    return ns, len(cfg) * ns, ok * ns


def _b_count(case):
    cfg = _configs(case)
    b = np.unique(cfg[:, 3] * cfg[:, 8])
    return int(np.sum(case["batch"] % b == 0))


def _class_of_slices(case):
    """Class of each slice (equal sums of every layer field), classes numbered
    by their first slice, and each class's first slice."""
    pre = _prefix(case)
    i, j = _slices(case)
    _, first, inv = np.unique((pre[:, j] - pre[:, i]).T, axis=0, return_index=True, return_inverse=True)
    rank = np.empty(len(first), dtype=np.int64)
    rank[np.argsort(first)] = np.arange(len(first))
    return rank[inv.reshape(-1)], np.sort(first)


def work(case):
    """Bytes: outputs written once and device inputs read once.  Operations:
    the transitions of the set dynamic program of the all-orders search, four
    per (state, cut, next island); elsewhere the stated step-time model, about
    twenty per candidate."""
    kind = case["kind"]
    if kind == "islands":
        return {"bytes": 8.0 * case["n"] ** 2, "flops": 0.0}
    ns, n, ok = _sizes(case)
    groups = float(_b_count(case)) * ns * case["islands"]
    if kind in ("search", "replan"):
        return {"bytes": 9.0 * n, "flops": 20.0 * n}
    if kind == "classes":
        nc = len(_class_of_slices(case)[1])
        return {"bytes": 9.0 * n / ns * nc + 8.0 * groups, "flops": 20.0 * n / ns * nc}
    if kind == "prune":
        return {"bytes": 9.0 * ok, "flops": 0.0}
    if kind == "relaxed":  # about one survivor a group: its index, cost and depth
        return {"bytes": 17.0 * groups, "flops": 0.0}
    k = case["islands"]
    return {"bytes": 17.0 * groups, "flops": 4.0 * _b_count(case) * case["layers"] * k * (k - 1) * 2.0 ** (k - 2)}


def tolerance(case):
    """Costs, depths, survivors and plans are defined one IEEE rounding at a
    time, ties included: another correct implementation returns the same bits."""
    return "exact"


# ----------------------------------------------------------------------------
# the same results in plain numpy and torch
# ----------------------------------------------------------------------------
def _prefix(case):
    lay = _layers(case)
    return np.array([np.concatenate([[0], np.cumsum(np.array(lay[f], dtype=np.int64))]) for f in LAYER_FIELDS])


def _slices(case):
    i, j = np.triu_indices(case["layers"])
    return i, j + 1


def _coefficients(case, inst, cfg):
    k, tp, cp, dp, ep, z, rc, of, mb = (cfg[:, q].astype(np.float64) for q in range(9))
    isl = {f: np.array(v, dtype=np.float64)[cfg[:, 0]] for f, v in inst["islands"].items()}
    F, W, Hb = isl["peak_flops"], isl["intra_bw"], isl["host_bw"]
    q, zi = tp * cp, cfg[:, 5]
    nc, nt = np.where(rc > 0, 4.0, 3.0), np.where(rc > 0, 3.0, 2.0)
    m = float(case["batch"]) / (dp * mb)

    def sync(D, qe):
        r = (D - 1.0) / D
        zm = np.where(zi <= 1, 0.0, np.where(zi == 2, 2.0 * r, 6.0 * r))
        zit = np.where(zi <= 1, 4.0 * r, np.where(zi == 2, 2.0 * r, 0.0))
        state = np.choose(zi, [np.full_like(D, 16.0), 4.0 + 12.0 / D, 2.0 + 14.0 / D, 16.0 / D])
        return ((zm / qe) / W) + (((zit / qe) / W) / m), state / qe

    dd, mud = sync(dp * cp, tp)
    de, mue = sync(np.floor(dp / ep) * cp, tp * ep)
    return {"alpha": (nc * mb) / ((q * F) * inst["space"]["eta"]),
            "beta": np.where(tp > 1, (((2.0 * nt) * mb) * (tp - 1.0)) / (q * W), 0.0),
            "gamma": np.where(ep > 1, ((nt * mb) * (ep - 1.0)) / ((ep * q) * W), 0.0),
            "kappa": np.where(cp > 1, (((nt + 1.0) * mb) * (cp - 1.0)) / ((cp * tp) * W), 0.0),
            "omega": np.where(of > 0, (2.0 * mb) / (q * Hb), 0.0), "dd": dd, "de": de, "mud": mud, "mue": mue,
            "rho": mb / q, "H": isl["hbm_bytes"] * inst["space"]["mem_frac"], "m": m, "rc": rc, "of": of}


def _scores(case, cfg, co, sums, lo, hi):
    """Costs and depths of configs [lo, hi) over the slices whose sums are given."""
    def col(f):
        return torch.from_numpy(np.ascontiguousarray(co[f][lo:hi])).cuda()[:, None]

    Fl, Pd, Pe, Act, Tb, Ab, Oa, Cb = (torch.from_numpy(x.astype(np.float64)).cuda()[None, :] for x in sums)
    S = torch.where(col("rc") > 0, Oa, Act)
    v = col("alpha") * Fl
    for c, x in (("beta", Tb), ("gamma", Ab), ("dd", Pd), ("de", Pe), ("kappa", Cb), ("omega", S)):
        t = col(c) * x
        v = v + t
    state = col("mud") * Pd
    state = state + col("mue") * Pe
    A1 = col("rho") * S
    d = torch.zeros_like(v)
    step = 1 << (case["islands"].bit_length() - 1)
    while step:  # the largest depth that fits: fits() is monotone in the depth
        t = d + step
        at = torch.where(col("of") > 0, torch.ones_like(t), t)
        use = state + torch.minimum(at, col("m")) * A1
        d = torch.where((t <= case["islands"]) & (use <= col("H")), t, d)
        step >>= 1
    return v, d


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("search", "replan", "classes"):
        return None  # whole numbers, selected inputs, or a search too long to repeat here
    inst, cfg = _instance(case, seed), _configs(case)
    co, pre = _coefficients(case, inst, cfg), _prefix(case)
    si, sj = _slices(case)
    sums = pre[:, sj] - pre[:, si]
    L, K, NS = case["layers"], case["islands"], len(si)
    b = cfg[:, 3] * cfg[:, 8]
    bvals = np.unique(b[case["batch"] % b == 0])
    D, nb = min(K, L), len(bvals)
    n_scored, cls = NS, None
    if kind == "classes":
        cls, first = _class_of_slices(case)
        sums, n_scored = sums[:, first], len(first)
    balanced = np.ones((K, n_scored), dtype=bool)
    if case["eps"] > 0:
        share = sums[0].astype(np.float64) / float(pre[0, L])
        power = np.array(inst["islands"]["n_gpus"], dtype=np.float64) * np.array(inst["islands"]["peak_flops"])
        total = 0.0
        for x in power:
            total = total + x
        c, r = (power / total)[:, None], 1.0 + case["eps"]
        balanced = (share <= c * r) & (share * r >= c)
    balanced = torch.from_numpy(balanced).cuda()
    # least cost of a group by the depth it fits at, then by the depth it reaches
    inf = float("inf")
    tab = torch.full((nb * K * n_scored, D), inf, dtype=torch.float64, device="cuda")
    cost = torch.empty(len(cfg) * n_scored, dtype=torch.float64, device="cuda")
    group = np.searchsorted(bvals, b) * K + cfg[:, 0]
    fits_b = case["batch"] % b == 0
    per = max(1, (1 << 24) // n_scored)
    s_at = torch.arange(n_scored, device="cuda")
    for lo in range(0, len(cfg), per):
        hi = min(len(cfg), lo + per)
        v, d = _scores(case, cfg, co, sums, lo, hi)
        cost[lo * n_scored:hi * n_scored] = v.reshape(-1)
        at = torch.from_numpy(group[lo:hi]).cuda()[:, None] * n_scored + s_at[None, :]
        keep = (d > 0) & torch.from_numpy(fits_b[lo:hi]).cuda()[:, None] & balanced[torch.from_numpy(
            np.ascontiguousarray(cfg[lo:hi, 0])).cuda()]
        cell = at[keep] * D + (d[keep].long().clamp(max=D) - 1)
        tab.view(-1).scatter_reduce_(0, cell, v[keep], "amin")
    for x in range(D - 2, -1, -1):
        tab[:, x] = torch.minimum(tab[:, x], tab[:, x + 1])
    tab = tab.view(nb, K, n_scored, D)
    return {"cost": cost, "dmax": None, "n": None, "survivors": None, "plan": {
        "head": None, "pft": _least_plan(case, inst, bvals, tab, cls, si, sj, D), "stage_int": None,
        "stage_float": None}}


def _least_plan(case, inst, bvals, tab, cls, si, sj, D):
    """(P, F, T) of the least plan: per b the least bottleneck, then the least
    fill at it; across b the least T."""
    L, K, inf = case["layers"], case["islands"], float("inf")
    order = inst["island_order"]
    E = torch.tensor(inst["inter_bw"], dtype=torch.float64, device="cuda")[order][:, order]
    oa = torch.tensor(inst["layers"]["out_act_bytes"], dtype=torch.float64, device="cuda")
    after = torch.ones(K, K, dtype=torch.bool, device="cuda").triu(1)
    cut = torch.from_numpy(si * (L + 1) + sj).cuda()
    best = (inf, inf, inf)
    for x, b in enumerate(bvals):
        t = tab[x][order]
        if cls is not None:
            t = t[:, torch.from_numpy(cls).cuda()]

        def stage(d):  # [i][j][position], +inf where nothing fits
            full = torch.full((L * (L + 1), K), inf, dtype=torch.float64, device="cuda")
            full[cut] = t[:, :, d - 1].T
            return full.view(L, L + 1, K)

        link = ((2.0 * float(b)) * oa)[:, None, None] / E[None]  # after layer j - 1, from o to o2
        link = torch.where(after[None] & (E[None] != 0), link, torch.full_like(link, inf))
        bound = None
        for fill in (False, True):
            lim = bound if fill else inf
            root, cont = inf, None
            for d in range(1, D + 1):
                S = stage(d)
                if fill:
                    S = torch.where(S <= lim, S, torch.full_like(S, inf))
                if d == 1:
                    V = S[:, L]
                else:
                    V = (S[:, 1:] + cont[None] if fill else torch.maximum(S[:, 1:], cont[None])).amin(1)
                root = min(root, float(V[0].min()))
                nxt = V[1:, None, :]  # rows j = 1 .. L - 1
                X = link[:L - 1]
                if fill:
                    W = (torch.where(X <= lim, X, torch.full_like(X, inf)) + nxt).amin(2)
                else:
                    W = torch.maximum(X, nxt).amin(2)
                cont = torch.cat([W, torch.full((1, K), inf, dtype=torch.float64, device="cuda")])
            if not fill:
                bound = root
                if not bound < inf:
                    break
        if bound < inf and root < inf:
            total = ((float(case["batch"] // int(b)) - 1.0) * bound) + root
            if total < best[2]:
                best = (bound, root, total)
    return np.array(best, dtype=np.float64)
