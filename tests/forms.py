"""Which form of the selection serves a bf16 call without scores_out and without a threshold, as the library itself decides it: the rules of its
dispatch are functions of the shared object (C++ names) and need no GPU."""
import ctypes

import paper_2602_13836_amd as sv

_INT, _I64 = ctypes.c_int, ctypes.c_int64


def _ask(name, argtypes, *args):
    f = getattr(sv.load_library(), name)
    f.restype, f.argtypes = ctypes.c_bool, argtypes
    return f(*args)


def form_of(rows, V, d_prime, k):
    """"keys" (two bytes per score), "codes" (one), "bracket" (wide selectors), "rows" (scores in memory, one launch after them) or
    "scores" (in memory, through a histogram)."""
    shape = (_INT, _INT, _I64, _I64, _I64), sv.SV_BF16, d_prime // 8, rows, V, k
    if _ask("_ZN2sv20key_select_supportedEiilll", *shape):
        return "keys"
    if _ask("_ZN2sv21code_select_supportedEiilll", *shape):
        return "codes"
    if _ask("_ZN2sv24bracket_select_supportedEill", (_INT, _I64, _I64), sv.SV_BF16, rows, V):
        return "bracket"
    return "rows" if _ask("_ZN2sv20row_select_supportedEl", (_I64,), V) else "scores"
