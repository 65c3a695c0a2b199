"""The score kernel that evaluates the model once per slice class, against the
CPU oracle bit for bit: layer patterns with few classes (equal layers, a
repeating pair, a head and a tail), slice counts of every alignment, one
configuration per block and several, rows cut into pieces, and score ranges
that start and end inside rows, into buffers at odd byte offsets: 31 configs'
rows and fewer, which the general kernel takes, and more."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle.oracle import Oracle  # noqa: E402
from workloads import extended, load_instance  # noqa: E402
from workloads.gen import _space, make_moe, uniform_layers  # noqa: E402

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2606_16907_amd import tangram as T  # noqa: E402


def _instance(L, pattern, gpus=(4, 6), moe=False, ext=False):
    shape = dict(s=2048, h=1024, n_heads=16, n_kv=16, ffn=4096, act="gelu")
    layers = uniform_layers(L, **shape)
    if moe:
        layers = uniform_layers(L, **dict(shape, n_experts=8, top_k=2, ffn_expert=1024))
    for f, v in layers.items():
        for l in range(L):
            if pattern == "pair" and l % 2:
                v[l] = v[l] * 3 + 7
            if pattern == "ends" and l in (0, L - 1):
                v[l] = v[l] * 5 + l
    K = len(gpus)
    isl = {"n_gpus": list(gpus), "peak_flops": [300e12 + 1e12 * k for k in range(K)],
           "hbm_bytes": [(12 + 9 * k) * 1e9 for k in range(K)], "intra_bw": [600e9] * K, "host_bw": [32e9] * K}
    E = [[0.0 if a == b else 25e9 for b in range(K)] for a in range(K)]
    inst = {"name": f"{pattern}{L}", "layers": layers, "islands": isl, "inter_bw": E, "island_order": list(range(K)),
            "space": _space(48, tp=(1, 2, 4), mb=(1, 2, 3), ep=(1, 2) if moe else (1,), n_experts=8 if moe else 0)}
    return extended(inst) if ext else inst


# slices 28 to 45150: odd counts, counts of every residue mod 16, more than one piece (L = 300)
CASES = [(7, "equal", False, False), (8, "equal", False, False), (9, "equal", True, False), (13, "equal", False, True),
         (21, "pair", False, False), (22, "pair", True, True), (23, "ends", False, False), (33, "ends", True, False),
         (127, "equal", False, False), (128, "ends", False, False), (130, "equal", True, True),
         (300, "equal", False, False)]


@pytest.mark.parametrize("L,pattern,moe,ext", CASES)
def test_score_by_class(L, pattern, moe, ext):
    print("case", L, pattern, moe, ext, flush=True)
    inst = _instance(L, pattern, moe=moe, ext=ext)
    p, o = T.Problem(inst), Oracle(inst)
    assert 4 * p.NC <= p.NS  # few classes: the path under test
    oc, od = o.score()
    cost, dmax = p.tg_score_pairs()
    assert np.array_equal(cost.cpu().numpy().view(np.uint64), oc.view(np.uint64))
    assert np.array_equal(dmax.cpu().numpy(), od)
    # parts of the range, into buffers 8 bytes (costs) and any byte (depths) off an aligned address
    for first, count, off in ((1, 2 * p.NS + 3, 1), (p.NS - 1, 2, 3), (p.NS // 2, 1, 15), (5 * p.NS, p.NS, 8),
                              (p.N - p.NS - 5, p.NS + 5, 17), (p.NS - 3, 33 * p.NS + 7, 1), (3, 40 * p.NS, 9),
                              (p.NS // 3, 31 * p.NS, 2)):
        first, count = max(first, 0), min(count, p.N - max(first, 0))
        cbuf = torch.full((count + off + 16,), -1.0, dtype=torch.float64, device="cuda")
        dbuf = torch.full((count + off + 32,), 255, dtype=torch.uint8, device="cuda")
        p.tg_score_pairs(first, count, cbuf[off:off + count], dbuf[off:off + count])
        c, d = cbuf.cpu().numpy(), dbuf.cpu().numpy()
        assert np.array_equal(c[off:off + count].view(np.uint64), oc[first:first + count].view(np.uint64))
        assert np.array_equal(d[off:off + count], od[first:first + count])
        assert (c[:off] == -1).all() and (c[off + count:] == -1).all()  # nothing outside the range
        assert (d[:off] == 255).all() and (d[off + count:] == 255).all()


# at 24 layers a block of four configs writes 1,200 candidates; at 12 (312), with so
# many configs, the general kernel takes over
@pytest.mark.parametrize("L", [12, 24])
def test_score_by_class_shared_blocks(L):
    """Enough configs that several share a block, in the expert variant."""
    inst = make_moe()
    inst["layers"] = {f: v[:L] for f, v in inst["layers"].items()}
    p, o = T.Problem(inst), Oracle(inst)
    assert p.n_configs >= 2 * 4 * 1024 and 4 * p.NC <= p.NS
    oc, od = o.score()
    cost, dmax = p.tg_score_pairs()
    assert np.array_equal(cost.cpu().numpy().view(np.uint64), oc.view(np.uint64))
    assert np.array_equal(dmax.cpu().numpy(), od)
    assert load_instance("moe")["islands"] == inst["islands"]


@pytest.mark.parametrize("L,islands", [(63, 40), (127, 115), (128, 113), (136, 3), (137, 3)])
def test_score_by_class_large(L, islands):
    """Slice counts that are a multiple of 64, just past 32 Mi candidates (fewer
    go to the general kernel), and the longest row of one piece and the next,
    over the whole range and from odd starts."""
    print("case", L, islands, flush=True)
    inst = _instance(L, "equal", gpus=(8,) * islands)
    p, o = T.Problem(inst), Oracle(inst)
    assert (p.NS % 64 == 0) == (L in (127, 128))
    assert p.N > 32 << 20 or L not in (127, 128)
    oc, od = o.score()
    for first, count in ((0, p.N), (5, p.N - 11)):
        cost, dmax = p.tg_score_pairs(first, count)
        assert np.array_equal(cost.cpu().numpy().view(np.uint64), oc[first:first + count].view(np.uint64))
        assert np.array_equal(dmax.cpu().numpy(), od[first:first + count])
