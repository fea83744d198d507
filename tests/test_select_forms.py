"""The shapes of the GPU tests are those of the form of the selection that each test is about: a line of the dispatch that moves must not empty
a test.  (The rules are asked on the host.)"""
import pytest

pytest.importorskip("torch")
sv = pytest.importorskip("paper_2602_13836_amd")

import test_gpu_code_select as codes
import test_gpu_key_select as keys
import test_gpu_parity as parity
from forms import form_of


@pytest.mark.parametrize("form,shapes", [
    ("codes", codes.EDGES), ("codes", codes.LONG_LISTS), ("codes", [(*s, 100) for s in codes.HARD]), ("codes", [(*s, 20000) for s in codes.HARD]),
    ("codes", [(*s, s[1] // 20) for s in codes.ONE_SUM]),
    ("keys", keys.EDGES), ("keys", keys.TOGETHER), ("keys", keys.OFFSET), ("keys", [(20, V, 32, k) for V, k in keys.MISLED]),
    ("keys", [(15, 3 * keys.PART, 32, k) for k in (1000, 12000, 40000)]), ("keys", [(*s, s[1] // 20) for s in keys.ONE_SUM]),
    ("codes", [(rows, V, 16, k) for rows, V, k in parity.USELESS_SAMPLE]), ("codes", [(67, 50000, 16, 3000)]),
])
def test_form(form, shapes):
    assert [s for s in shapes if form_of(*s) != form] == []


def test_forms_of_a_batch():
    got = [form_of(rows, V, dp, k) for rows, d, dp, V, k in parity.BATCH_SELECT_SHAPES]
    assert got.count("codes") >= 8 and "keys" in got and got[-1] == "scores"
