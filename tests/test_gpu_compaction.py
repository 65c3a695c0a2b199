"""The survivor compaction's three ways of counting the bits before a tile, and
the class expansion, against the oracle's list: bitmaps just below and above
the size from which a count pass runs (8192 words), rows that survive on every
slice, a bitmap of one partial word, and capacities that cut the list inside a
tile."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle.oracle import Oracle  # noqa: E402
from tests.inst_util import scaled  # noqa: E402
from workloads import load_instance, random_tiny  # noqa: E402

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2606_16907_amd import tangram as T  # noqa: E402


def _dense8b(L, memory=1.0):
    inst = load_instance("dense8b")
    inst["layers"] = {f: (v * 4)[:L] for f, v in inst["layers"].items()}
    return scaled(inst, memory=memory)


CASES = [("w7680", lambda: _dense8b(38)), ("w8320", lambda: _dense8b(40)), ("dense", lambda: _dense8b(40, 1e6)),
         ("w30000", lambda: _dense8b(77)), ("one_word", lambda: random_tiny(5, L_range=(2, 2), K_range=(1, 1))),
         ("none", lambda: _dense8b(24, 1e-6))]


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
