"""The binding's host tables hold what a field-by-field ctypes assignment of
the converted values holds, for every form of column it takes: lists, tuples,
arrays and tensors, whole numbers of any size (a field keeps the low bits, as
a ctypes field does, and the library then judges the value), floats in integer
columns and numbers as text.  No device is needed: the tables are filled, and
bad values refused, before the first device call."""
import copy
import ctypes

import numpy as np
import pytest
import torch

from paper_2606_16907_amd import tangram as T
from tests.inst_util import instance

INTS = [
    [3, 0, 2**62, 7], (1, 2, 3, 4), np.array([5, 6, 7, 8]), np.array([1, 2, 3, 255], dtype=np.uint8),
    [2**63, 1, 2, 3], [2**64 + 5, 1, 2, 3], [-2**63 - 1, 2**63, -1, 0], [2**40 + 1, 2**32 + 2, -1, 0],
    [True, False, 1, 0], [1.9, 2.0, 3, 4], [2**53 + 1, 1.0, 2, 3], ["3", "4", 5, "6"],
    [np.uint64(2**64 - 1), np.int32(-1), 1, 2], torch.arange(4), [torch.tensor(3), torch.tensor(4.5), 1, 2],
    [1, 2, 3, 4, "past the table"], {0: 1, 1: 2, 2: 3, 3: 4},
]
FLOATS = [
    [1.5, -0.0, float("inf"), float("nan")], (1, 2, 3, 4), [2**63, 2**53 + 1, 1, 0.1], [10**300, 1, 2, 3],
    np.array([0.1, 0.2, 0.3, 0.4], dtype=np.float32), ["1.5", "inf", 2, "1e300"], [True, 2.5, 1, 0],
    torch.tensor([1.25, 2, 3, 4]), [torch.tensor(0.1, requires_grad=True)] * 4,
    [torch.tensor(0.1, dtype=torch.bfloat16)] * 4,
]
BAD = [(int, [1, [2], 3, 4]), (float, [1.0, [2.0, 3.0], 3, 4]), (int, [None, 1, 2, 3]), (int, [1, 2]),
       (float, [10**400, 1, 2, 3]), (int, [float("inf"), 1, 2, 3]), (float, ["a", 1, 2, 3]), (float, [1j, 1, 2, 3])]


def _one_by_one(struct, field, conv, column, n=4):
    table = (struct * n)()
    for r in range(n):
        setattr(table[r], field, conv(column[r]))
    return bytes(table)


@pytest.mark.parametrize("struct,field,conv,column",
                         [(T.TgLayer, "fwd_flops", int, c) for c in INTS]
                         + [(T.TgIsland, "n_gpus", int, c) for c in INTS]
                         + [(T.TgIsland, "peak_flops", float, c) for c in FLOATS])
def test_columns(struct, field, conv, column):
    table = (struct * 4)()
    T._fill_table(table, struct, {"c": column}, [(field, conv, "c")])
    assert bytes(table) == _one_by_one(struct, field, conv, column)


@pytest.mark.parametrize("conv,column", BAD)
def test_bad_columns_raise_alike(conv, column):
    field = "n_gpus" if conv is int else "peak_flops"
    with pytest.raises(Exception) as want:
        _one_by_one(T.TgIsland, field, conv, column)
    with pytest.raises(want.type):
        T._fill_table((T.TgIsland * 4)(), T.TgIsland, {"c": column}, [(field, conv, "c")])


def test_empty_table_reads_no_column():
    T._fill_table((T.TgIsland * 0)(), T.TgIsland, {}, [("n_gpus", int, "missing")])


@pytest.mark.parametrize("value", [2**63, 2**63 + 1, -1, -2**62])
def test_library_judges_wide_values(value):
    inst = copy.deepcopy(instance(K=2, L=3, layer={"fwd_flops": 2**40}))
    inst["layers"]["fwd_flops"][1] = value
    with pytest.raises(T.TangramError) as err:
        T.Problem(inst)
    assert err.value.status == T.TG_EINVAL
