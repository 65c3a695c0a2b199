"""tg_compose_pipeline on both sides of each limit between the small composition
(one block per micro-batch size) and the level launches, against the CPU
oracle: the work of a level (K^2 (L + 1) = 7000), the stage table of every depth
(256 K cells), the list length (32768) and the entries the plan's groups may
hold (2048).  Lists are surviving sets and supersets of them (every compatible
candidate that fits, with exact ties in cost and depth inside a group), uneven
layers, with and without imbalance pruning."""
import collections

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle.oracle import Oracle  # noqa: E402
from tests.inst_util import instance  # noqa: E402
from tests.test_gpu_imbalance import with_eps  # noqa: E402
from tests.test_gpu_parity import plan_equal  # noqa: E402
from tests.test_gpu_superset import superset  # noqa: E402
from workloads import random_tiny  # noqa: E402

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2606_16907_amd import tangram as T  # noqa: E402


def _same(p, o, lst, cost, dmax):
    st, plan = p.tg_compose_pipeline(torch.from_numpy(lst).cuda(), cost, dmax)
    ost, oplan = o.compose(lst)[:2]
    assert st == (T.TG_ENOPLAN if ost != 0 else 0)
    if ost == 0:
        plan_equal(plan, oplan)
    return plan


# with three micro-batch sizes: slices * 3 * K * min(K, L) cells 262,080 and 267,120,
# 257,040 and 272,160; K^2 (L + 1) 6,804 and 7,128, 6,561 and 7,056; then well past
SIZES = [(4, 104), (4, 105), (12, 34), (12, 35), (18, 20), (18, 21), (27, 8), (28, 8), (14, 70), (16, 61), (33, 30)]


# imbalance pruning leaves plans where islands can hold a balanced share of the layers
@pytest.mark.parametrize("K,L,eps", [(K, L, e) for e in (0.0, 2.0) for K, L in SIZES if e == 0.0 or 2 * K <= L])
def test_sizes(K, L, eps):
    print("case", K, L, eps, flush=True)
    inst = with_eps(random_tiny(4000 + 100 * K + L, L_range=(L, L), K_range=(K, K), tight=L < 40), eps)
    f = 16 if L > 100 else 4  # long models get smaller layers, so that plans exist
    inst["layers"] = {k: [x // f for x in v] for k, v in inst["layers"].items()}
    inst["space"]["global_batch"] = 4
    p, o = T.Problem(inst), Oracle(inst)
    assert p.n_b == 3
    cost, dmax = p.tg_score_pairs()
    surv = p.tg_prune(cost, dmax).cpu().numpy()
    assert np.array_equal(surv, o.prune())
    plan = _same(p, o, surv, cost, dmax)
    if eps == 0.0:  # a superset may hold no unbalanced pair
        idx = superset(p, inst, dmax)[0]
        assert len(idx) > len(surv)
        again = _same(p, o, idx, cost, dmax)
        assert (again["T"], again["b"], again["S"]) == (plan["T"], plan["b"], plan["S"])


def _members(o):
    B = o.inst["space"]["global_batch"]
    c = collections.Counter()
    for g in range(o.n_configs):
        d = o.decode(g * o.NS)
        if B % (d["dp"] * d["mb"]) == 0:
            c[(d["island"], d["dp"] * d["mb"])] += 1
    return max(c.values())


def _uneven(L, unit=10**7):
    return {"fwd_flops": [(7 * l % 5 + 1) * 10**12 for l in range(L)],
            "dense_params": [(l % 3 + 1) * unit for l in range(L)], "expert_params": [unit] * L,
            "act_stash_bytes": [10**8 + 10**7 * (l % 4) for l in range(L)],
            "tp_comm_bytes": [10**6] * L, "a2a_bytes": [10**6] * L, "out_act_bytes": [10**7] * L,
            "cp_comm_bytes": [10**6] * L}


def test_list_length():
    """32,768 entries, the longest list of the small composition, and one more."""
    inst = instance(K=6, layers=_uneven(16), n_gpus=[8, 6, 8, 4, 8, 8], peak=[(3 + k) * 1e13 for k in range(6)],
                    hbm=40e9, intra=300e9, inter=25e9, B=16, tp=(1, 2), mb=(1, 2, 4), zero=(0, 1, 2, 3), host=32e9,
                    recompute=(0, 1), offload=(0, 1))
    p, o = T.Problem(inst), Oracle(inst)
    assert _members(o) * 6 <= 2048
    cost, dmax = p.tg_score_pairs()
    surv = p.tg_prune(cost, dmax).cpu().numpy()
    rest = np.setdiff1d(superset(p, inst, dmax)[0], surv)
    rng = np.random.default_rng(5)
    for n in (32767, 32768, 32769):  # the surviving set and some more
        print("case", n, len(surv), flush=True)
        lst = np.union1d(surv, rng.choice(rest, size=n - len(surv), replace=False))
        assert len(lst) == n
        assert _same(p, o, lst, cost, dmax)["S"] >= 1


# 1,008 and 1,072 members in the largest group of an island: 2,016 and 2,144
# entries in the groups of a plan of two stages
@pytest.mark.parametrize("tp,members", [((1, 2, 4), 1008), ((1, 2, 4, 8), 1072)])
def test_matches(tp, members):
    print("case", tp, flush=True)
    inst = instance(K=2, layers=_uneven(2, 10**8), n_gpus=16, peak=1e14, hbm=[4e9, 5e9], intra=300e9, inter=200e9,
                    B=32, tp=tp, cp=(1, 2, 4, 8), ep=(1, 2, 4, 8), mb=(1, 2, 4, 8, 16), zero=(0, 1, 2, 3), n_experts=16,
                    recompute=(0, 1), offload=(0, 1), host=32e9)
    p, o = T.Problem(inst), Oracle(inst)
    assert _members(o) == members
    cost, dmax = p.tg_score_pairs()
    idx, _, b = superset(p, inst, dmax)
    stages = set()
    for bv in sorted(set(b.tolist())):  # alone: b does not matter to another's plan
        lst = idx[b == bv]
        assert len(lst) <= 32768
        stages.add(_same(p, o, lst, cost, dmax)["S"])
    assert 2 in stages  # a plan whose two groups the finish picks out of the list
