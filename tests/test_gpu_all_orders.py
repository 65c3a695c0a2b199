"""Parity of the HIP composition over every island subset and order
(tg_compose_pipeline_all_orders, through the C ABI) with the CPU oracle's
tgo_compose_all_orders: the plan (b, stages, islands, cuts, configs, pair
indices, P, F, T and per-stage values) compared bit for bit.  Cases: the
named instances with at most 16 islands (the 16-island 70B instance against
the oracle's stored result), random instances from one to eight islands,
instances with exact ties, models longer than one block of threads, fewer
layers than islands, the extended config space, an empty list and the
16-island limit."""
import ctypes
import sys

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle.oracle import Oracle  # noqa: E402
from workloads import extended, load_instance, random_tiny  # noqa: E402
from tests.inst_util import instance, scaled, tiny_tight  # noqa: E402
from tests.golden.make_golden import load as load_golden  # noqa: E402
from tests.test_gpu_parity import plan_equal  # noqa: E402
from tests.test_oracle_all_orders import _symmetric  # noqa: E402

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2606_16907_amd import tangram as T  # noqa: E402


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


CASES = ([("tiny", lambda: load_instance("tiny")), ("tiny_tight", tiny_tight),
          ("dense8b", lambda: load_instance("dense8b")),
          ("dense8b_ext", lambda: extended(load_instance("dense8b")))]
         + [(f"rand{s}", lambda s=s: random_tiny(s, tight=(s % 2 == 1))) for s in range(16)]
         + [(f"sym{s}", lambda s=s: _symmetric(s)) for s in range(8)]
         + [(f"wide{s}", lambda s=s: random_tiny(2000 + s, L_range=(6, 12), K_range=(5, 8), tight=(s % 2 == 1)))
            for s in range(6)]
         + [("long70", lambda: random_tiny(3000, L_range=(70, 70), K_range=(3, 3))),
            ("long140", lambda: random_tiny(3001, L_range=(140, 140), K_range=(2, 2), tight=True)),
            ("long300", lambda: scaled(random_tiny(3006, L_range=(300, 300), K_range=(3, 3)), memory=64.0)),
            ("few_layers", lambda: random_tiny(3002, L_range=(2, 3), K_range=(5, 6))),
            ("one_island", lambda: random_tiny(3003, L_range=(5, 5), K_range=(1, 1)))])


def _gpu(p):
    cost, dmax = p.tg_score_pairs()
    surv = p.tg_prune(cost, dmax)
    return surv, cost, dmax


@pytest.mark.parametrize("name,make", CASES, ids=[n for n, _ in CASES])
def test_all_orders_parity(name, make):
    inst = make()
    say("case", name)
    o = Oracle(inst)
    ost, oplan, _ = o.compose_all_orders(o.prune())
    p = T.Problem(inst)
    surv, cost, dmax = _gpu(p)
    ws = p.compose_all_orders_workspace(int(surv.numel()))
    for rep in range(2):  # the same workspace twice: nothing carries over
        st, plan = p.tg_compose_pipeline_all_orders(surv, cost, dmax, workspace=ws)
        if ost != 0:
            assert st == T.TG_ENOPLAN and plan["S"] == 0
            continue
        assert st == 0
        plan_equal(plan, oplan)
    # the fixed-order composition on the same buffers is unaffected
    st3, plan3 = p.tg_compose_pipeline(surv, cost, dmax)
    ost3, oplan3, _ = o.compose(o.prune())
    assert st3 == ost3
    if st3 == 0:
        plan_equal(plan3, oplan3)


@pytest.mark.parametrize("name", ["tiny", "dense8b", "dense70b"])
def test_all_orders_named_against_stored(name):
    g = load_golden(name)["all_orders"]
    say("case", name)
    p = T.Problem(load_instance(name))
    surv, cost, dmax = _gpu(p)
    st, plan = p.tg_compose_pipeline_all_orders(surv, cost, dmax)
    assert st == g["status"] == 0
    g["plan"]["status"] = 0
    plan_equal(plan, g["plan"])
    assert plan["T"] == min(row[2] for row in g["per_b"])


def test_all_orders_empty_list_has_no_plan():
    p = T.Problem(load_instance("tiny"))
    _, cost, dmax = _gpu(p)
    st, plan = p.tg_compose_pipeline_all_orders(torch.empty(0, dtype=torch.int64, device="cuda"), cost, dmax)
    assert st == T.TG_ENOPLAN and plan["S"] == 0


def test_all_orders_rejects_more_than_16_islands():
    p = T.Problem(load_instance("moe"))  # 32 islands
    assert T.load_library().tg_compose_all_orders_workspace_bytes(p.h, 0) == 0
    cost = torch.empty(1, dtype=torch.float64, device="cuda")
    dmax = torch.empty(1, dtype=torch.uint8, device="cuda")
    ws = torch.empty(256, dtype=torch.uint8, device="cuda")
    # the library refuses before it reads any buffer (called directly: the
    # binding already refuses score arrays shorter than N)
    vp = ctypes.c_void_p
    plan = T.TgPlan()
    st = T.load_library().tg_compose_pipeline_all_orders(p.h, None, 0, vp(cost.data_ptr()), vp(dmax.data_ptr()),
                                                         ctypes.byref(plan), vp(ws.data_ptr()), ws.numel(), None)
    assert st == T.TG_EINVAL and "16 islands" in T.last_error()
    with pytest.raises(ValueError, match="at least"):
        p.tg_compose_pipeline_all_orders(torch.empty(0, dtype=torch.int64, device="cuda"), cost, dmax,
                                         workspace=ws)


def _banded(seed, L, K, memory, eps, tight):
    """Large enough (7 b x K 2^(K-1) states x rows) for the bounds from a few
    island orders and the bands of rows they leave."""
    inst = scaled(random_tiny(seed, L_range=(L, L), K_range=(K, K), tight=tight), memory=memory)
    inst["space"].update(global_batch=24, mb=[1, 2, 3, 4], imbalance_eps=eps)
    return inst


@pytest.mark.parametrize("seed,L,K,memory,eps,tight", [
    (4101, 28, 12, 4.0, 0.0, False),   # uneven layers, some links absent
    (4102, 30, 12, 3.0, 0.0, True),    # depth limits bind
    (4103, 31, 12, 8.0, 3.0, False),   # imbalance pruning: stage costs not monotone from the first cut
    (4104, 60, 11, 20.0, 0.0, False),
    (4105, 28, 12, 1.0, 0.0, True)])   # few plans: the memory order alone has none
def test_all_orders_bands(seed, L, K, memory, eps, tight):
    say("banded", seed)
    inst = _banded(seed, L, K, memory, eps, tight)
    o, p = Oracle(inst), T.Problem(inst)
    assert p.n_b * K * 2 ** (K - 1) * (L + 1) >= 1 << 22
    ost, oplan, _ = o.compose_all_orders(o.prune())
    surv, cost, dmax = _gpu(p)
    ws = p.compose_all_orders_workspace(int(surv.numel()))
    for rep in range(2):
        st, plan = p.tg_compose_pipeline_all_orders(surv, cost, dmax, workspace=ws)
        assert st == (T.TG_ENOPLAN if ost != 0 else 0)
        if ost == 0:
            plan_equal(plan, oplan)


def _many_b(K, L):
    """More micro-batch sizes than one run of the fill covers (32)."""
    layers = {"fwd_flops": [(7 * l % 5 + 1) * 10**12 for l in range(L)],
              "dense_params": [10**7 * (l % 3) for l in range(L)], "act_stash_bytes": [10**6] * L,
              "tp_comm_bytes": [10**6] * L, "out_act_bytes": [10**7] * L}
    return instance(K=K, layers=layers, n_gpus=[4 + 3 * k for k in range(K)], peak=[(3 + k) * 1e13 for k in range(K)],
                    hbm=40e9, intra=300e9, inter=25e9, B=720720, mb=(1, 2, 3, 5, 7, 11, 13), tp=(1, 2), zero=(0, 3))


@pytest.mark.parametrize("name,make,bounded", [
    # every b filled at once: rows staged at no level, at some, at all
    ("unstaged", lambda: scaled(random_tiny(3011, L_range=(512, 512), K_range=(3, 3)), memory=99.0), False),
    ("staged_some", lambda: scaled(random_tiny(3012, L_range=(306, 306), K_range=(5, 5)), memory=99.0), False),
    ("staged_all", lambda: random_tiny(3013, L_range=(40, 40), K_range=(9, 9)), False),
    ("eps", lambda: _banded(3014, 33, 7, 4.0, 1.0, False), False),
    # rows without bands, the fill only for the b that can win
    ("whole", lambda: _banded(3015, 118, 10, 40.0, 0.0, False), True),
    ("whole_eps", lambda: _banded(3016, 60, 11, 40.0, 2.0, False), True),
    ("whole_tight", lambda: _banded(3017, 57, 11, 2.0, 0.0, True), True),
    ("many_b", lambda: _many_b(4, 7), False)])
def test_all_orders_without_bands(name, make, bounded):
    say("whole rows", name)
    inst = make()
    o, p = Oracle(inst), T.Problem(inst)
    assert (p.n_b * p.K * 2 ** (p.K - 1) * (p.L + 1) >= 1 << 22) == bounded
    assert name != "many_b" or p.n_b > 32
    ost, oplan, _ = o.compose_all_orders(o.prune())
    surv, cost, dmax = _gpu(p)
    ws = p.compose_all_orders_workspace(int(surv.numel()))
    ws.fill_(0xFF)
    for rep in range(2):
        st, plan = p.tg_compose_pipeline_all_orders(surv, cost, dmax, workspace=ws)
        assert st == (T.TG_ENOPLAN if ost != 0 else 0)
        if ost == 0:
            plan_equal(plan, oplan)
