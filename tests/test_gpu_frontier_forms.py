"""The survivor definition on score arrays that no instance produces, for both
frontier kernels: depths and costs drawn at random with many exact ties, +inf
costs, groups without a fitting member, one island up to the widest cluster the
depth buckets take (32) and past it, and groups larger than a round of the
bitmap's mask.  The expected list is the definition itself: within a group a
member survives iff no member at least as deep has a smaller key (cost, -depth,
index)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from workloads.gen import _space, uniform_layers  # noqa: E402

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2606_16907_amd import tangram as T  # noqa: E402


def _problem(L, K, gpus, batch, cp=(1,)):
    layers = uniform_layers(L, s=2048, h=1024, n_heads=16, n_kv=16, ffn=4096, act="gelu")
    isl = {"n_gpus": [gpus] * K, "peak_flops": [300e12] * K, "hbm_bytes": [80e9] * K, "intra_bw": [600e9] * K,
           "host_bw": [32e9] * K}
    E = [[0.0 if a == b else 25e9 for b in range(K)] for a in range(K)]
    return T.Problem({"layers": layers, "islands": isl, "inter_bw": E, "island_order": list(range(K)),
                      "space": _space(batch, tp=(1, 2), mb=(1, 2), cp=cp, recompute=(0, 1), offload=(0, 1))})


def _survivors(p, batch, cost, dmax):
    pairs = p.tg_enumerate_pairs().cpu().numpy()
    b = pairs[:, 5].astype(np.int64) * pairs[:, 10]
    ok = (batch % b == 0) & (dmax > 0)
    idx = np.nonzero(ok)[0]
    key = (pairs[idx, 0].astype(np.int64) * 1000 + pairs[idx, 1]) * 1000 + pairs[idx, 2]
    order = np.lexsort((idx, -dmax[idx].astype(np.int64), cost[idx], b[idx], key))
    keep, last, deepest = [], None, 0
    for t in idx[order]:  # ascending key inside each group: survives iff deeper than every earlier one
        g = (pairs[t, 0], pairs[t, 1], pairs[t, 2], b[t])
        if g != last:
            last, deepest = g, 0
        if dmax[t] > deepest:
            deepest = int(dmax[t])
            keep.append(int(t))
    return np.array(sorted(keep), dtype=np.int64)


@pytest.mark.parametrize("L,K,gpus,batch,cp", [
    (3, 1, 2, 4, (1,)), (11, 2, 4, 8, (1,)), (12, 5, 3, 6, (1, 2)), (4, 31, 4, 4, (1,)), (4, 32, 4, 4, (1,)),
    (4, 33, 4, 4, (1,)), (3, 64, 3, 4, (1,)), (11, 3, 64, 64, (1, 2, 4, 8)), (2, 32, 32, 64, (1, 2, 4)),
    (2, 33, 32, 64, (1, 2, 4))])
@pytest.mark.parametrize("seed", range(3))
def test_frontier(L, K, gpus, batch, cp, seed):
    print("case", L, K, gpus, batch, seed, flush=True)
    p = _problem(L, K, gpus, batch, cp)
    rng = np.random.default_rng([seed, L, K])
    n = p.N
    few = rng.integers(0, 6, size=n) * 0.5            # many exact ties
    cost = np.where(rng.random(n) < 0.5, few, rng.random(n) * 3)
    cost[rng.random(n) < 0.05] = np.inf
    dmax = rng.integers(0, K + 1, size=n).astype(np.uint8)
    if seed == 1:                                      # depths follow costs: long staircases
        dmax = np.clip((cost * K / 3).round(), 0, K).astype(np.uint8)
    if seed == 2:
        dmax[rng.random(n) < 0.9] = 0
    got = p.tg_prune(torch.from_numpy(cost).cuda(), torch.from_numpy(dmax).cuda()).cpu().numpy()
    assert np.array_equal(got, _survivors(p, batch, cost, dmax))


@pytest.mark.parametrize("L,K,gpus,batch", [(11, 3, 64, 64), (4, 5, 6, 12), (4, 33, 4, 4)])
def test_scores_out_of_the_model(L, K, gpus, batch):
    """Depths past the island count are compared like any other; members whose
    cost is no number all survive where they fit, many to a group and depth
    among them, and beat nobody."""
    print("case", L, K, gpus, batch, flush=True)
    p = _problem(L, K, gpus, batch)
    rng = np.random.default_rng([7, L, K])
    n = p.N
    cost = rng.integers(0, 40, size=n) * 0.25
    dmax = rng.integers(0, 256, size=n).astype(np.uint8)
    got = p.tg_prune(torch.from_numpy(cost).cuda(), torch.from_numpy(dmax).cuda()).cpu().numpy()
    assert np.array_equal(got, _survivors(p, batch, cost, dmax))
    dmax = np.minimum(dmax, K).astype(np.uint8)
    nan = rng.random(n) < 0.5
    pairs = p.tg_enumerate_pairs().cpu().numpy()
    fits = (batch % (pairs[:, 5].astype(np.int64) * pairs[:, 10]) == 0) & (dmax > 0)
    want = np.union1d(_survivors(p, batch, cost, np.where(nan, 0, dmax).astype(np.uint8)), np.nonzero(nan & fits)[0])
    cost[nan] = np.nan
    got = p.tg_prune(torch.from_numpy(cost).cuda(), torch.from_numpy(dmax).cuda()).cpu().numpy()
    assert np.array_equal(got, want)
