"""The survivor compaction's three ways of counting the bits before a tile, and
the class expansion, against the oracle's list: bitmaps just below and above
the size from which a count pass runs (8192 words), rows that survive on every
slice, a bitmap of one partial word, rows cut into several pieces, and
capacities that cut the list inside a tile.  And tiles of every density, dealt
output by output or walked word by word, with one and four words a thread."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle.oracle import Oracle  # noqa: E402
from tests.inst_util import instance, scaled  # noqa: E402
from workloads import load_instance, random_tiny  # noqa: E402

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2606_16907_amd import tangram as T  # noqa: E402


def _dense8b(L, memory=1.0):
    inst = load_instance("dense8b")
    inst["layers"] = {f: (v * 4)[:L] for f, v in inst["layers"].items()}
    return scaled(inst, memory=memory)


def _long(L, memory=1.0):
    """Two kinds of layer on three islands, the last too small for any layer."""
    layers = {"fwd_flops": [10**11 * (1 + l % 2) for l in range(L)], "dense_params": [10**6] * L,
              "act_stash_bytes": [10**6 * (1 + l % 2) for l in range(L)], "tp_comm_bytes": [10**5] * L,
              "out_act_bytes": [10**5] * L}
    return instance(K=3, layers=layers, n_gpus=[4, 2, 3], peak=[1e14, 2e14, 1e14],
                    hbm=[1e9 * memory, 2e9 * memory, 1e5], intra=300e9, inter=25e9, B=8, tp=(1, 2), mb=(1, 2),
                    zero=(0, 3))


CASES = [("w7680", lambda: _dense8b(38)), ("w8320", lambda: _dense8b(40)), ("dense", lambda: _dense8b(40, 1e6)),
         ("w30000", lambda: _dense8b(77)), ("one_word", lambda: random_tiny(5, L_range=(2, 2), K_range=(1, 1))),
         ("none", lambda: _dense8b(24, 1e-6)),
         # 5,050, 5,151, 16,110 and 45,150 slices a row: one piece of the expansion, two, four, nine
         ("pieces100", lambda: _long(100)), ("pieces101", lambda: _long(101)), ("pieces179", lambda: _long(179)),
         ("pieces300", lambda: _long(300, 0.3))]


@pytest.mark.parametrize("name,make", CASES, ids=[n for n, _ in CASES])
def test_compaction(name, make):
    print("case", name, flush=True)
    inst = make()
    p, want = T.Problem(inst), Oracle(inst).prune()
    cost, dmax = p.tg_score_pairs()
    assert np.array_equal(p.tg_prune(cost, dmax).cpu().numpy(), want)
    assert np.array_equal(p.tg_prune_classes(*p.tg_score_classes()).cpu().numpy(), want)
    for cap in [c for c in sorted({0, 1, len(want) // 3, len(want) - 1}) if 0 <= c < len(want)]:
        buf = torch.full((max(cap, 1) + 64,), -7, dtype=torch.int64, device="cuda")
        with pytest.raises(T.TangramError) as err:
            p.tg_prune(cost, dmax, survivors=buf[:cap])
        assert err.value.status == T.TG_ECAPACITY and err.value.required == len(want)
        got = buf.cpu().numpy()
        assert np.array_equal(got[:cap], want[:cap]) and (got[cap:] == -7).all()


# one config a group, so that what fits survives: 3 rows an island, 30, 129 and
# 2,052 words a row; 3,600 words (counted by each block), 46,440 (count pass) and
# 1.05 million (four words a thread)
@pytest.mark.parametrize("L,K", [(61, 40), (128, 120), (512, 171)])
def test_compaction_densities(L, K):
    print("case", L, K, flush=True)
    one = {"fwd_flops": 10**11, "dense_params": 10**6, "act_stash_bytes": 10**6, "out_act_bytes": 10**5}
    p = T.Problem(instance(K=K, L=L, layer=one, n_gpus=4, hbm=80e9, B=4, tp=(1,), mb=(1,), zero=(3,)))
    gen = torch.Generator(device="cuda").manual_seed(L)
    rows = torch.arange(p.N, device="cuda") // p.NS
    cost = torch.ones(p.N, dtype=torch.float64, device="cuda")
    ok = torch.zeros(p.n_configs, dtype=torch.bool)
    for g in range(p.n_configs):
        row = p.tg_enumerate_pairs(g * p.NS, 1)[0].tolist()
        ok[g] = 4 % (row[5] * row[10]) == 0
    ok = ok.cuda()[rows]
    # stretches of every density, among them 8 bits a word and a little to either side
    share = torch.tensor([0.0, 0.001, 0.05, 0.12, 0.125, 0.13, 0.5, 1.0], device="cuda")
    for stretch in (64 * 256, 64 * 100 + 7):
        pick = torch.randint(0, 8, (p.N // stretch + 1,), generator=gen, device="cuda")
        odds = share[pick[torch.arange(p.N, device="cuda") // stretch]]
        want_bits = torch.rand(p.N, generator=gen, device="cuda") < odds
        dmax = (want_bits & ok).to(torch.uint8)
        got = p.tg_prune(cost, dmax)
        want = torch.nonzero(dmax).flatten()
        assert torch.equal(got, want)
        cap = int(want.numel()) * 2 // 3
        buf = torch.full((cap + 64,), -7, dtype=torch.int64, device="cuda")
        with pytest.raises(T.TangramError) as err:
            p.tg_prune(cost, dmax, survivors=buf[:cap])
        assert err.value.status == T.TG_ECAPACITY and err.value.required == want.numel()
        assert torch.equal(buf[:cap], want[:cap]) and bool((buf[cap:] == -7).all())
