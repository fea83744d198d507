"""The bracketed selection: batches of 65 rows and more, selectors wider than 512 elements, 32768 to 393216 tokens.  Scores are exact
(whole numbers in steps of 2^-6), so the ids must be those of a full sort, ties to the smaller id."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
sv = pytest.importorskip("paper_2602_13836_amd")

pytestmark = pytest.mark.gpu


def _bf16(a):
    return torch.from_numpy(a.astype(np.float32)).cuda().to(torch.bfloat16)


def _inputs(rows, V, d_prime, seed, d=64):
    rng = np.random.default_rng(seed)
    return rng.integers(-1, 2, (rows, d)), rng.integers(-1, 2, (d_prime, d)), rng.integers(-2, 3, (V, d_prime), dtype=np.int8) / np.float32(64)


def _check(h, Wd, Wv, k):
    h, Wd, Wv = _bf16(h), _bf16(Wd), _bf16(Wv)
    idx, _ = sv.select(h, Wd, Wv, k)
    s = (h.double() @ Wd.double().t()).float() @ Wv.float().t()                 # (exact in float32)
    want = torch.sort(s, dim=1, descending=True, stable=True).indices[:, :k].sort(dim=1).values
    assert torch.equal(idx.long(), want)


# tiles of 128 and of 256 hidden rows, one, part of one and several; lists of 256-token tiles that the resolve step requests in 8, 16 and 24
# pairs per thread (up to 47662, 95325 and more tokens) and beyond (143000), packed into LDS and walked in memory; k = 1 and k = V
@pytest.mark.parametrize("rows,V,d_prime,k", [(65, 32768, 520, 1), (66, 40007, 2048, 300), (129, 33001, 1024, 33001), (140, 47700, 520, 9000),
                                              (257, 60000, 576, 30000), (300, 95326, 520, 5000), (513, 65537, 520, 65536),
                                              (400, 140000, 520, 8192), (70, 200001, 640, 100000), (65, 393216, 520, 20000)])
def test_edges(rows, V, d_prime, k):
    _check(*_inputs(rows, V, d_prime, rows + k), k)


def _misleading(rows, V, d_prime, seed, sampled):
    """Inputs whose first product, the same in every row, sets the sampled tokens apart from all others."""
    h, Wd, Wv = _inputs(rows, V, d_prime, seed)
    h[:, 1] = 1
    Wd[:, 1] = 0
    Wd[0, :] = 0
    Wd[0, 1] = 1                                   # h'[0] = 1 in every row
    Wv[:, 0] = 0
    Wv[np.arange(sv.SELECT_SAMPLE) * V // sv.SELECT_SAMPLE, 0] = sampled
    return h, Wd, Wv


@pytest.mark.parametrize("rows,V,k", [(65, 40000, 2000), (140, 65536, 8192), (300, 33001, 24000), (66, 150000, 9000)])
def test_rows_whose_bracket_misses_are_redone(rows, V, k):
    """The sampled tokens score below all others: more than k scores lie above every row's bracket."""
    _check(*_misleading(rows, V, 520, V + rows, -1024.0), k)


@pytest.mark.parametrize("rows,V,k", [(65, 40000, 9000), (140, 65536, 30000), (300, 33001, 33001), (66, 150000, 70000)])
def test_rows_whose_bracket_is_too_high_are_redone(rows, V, k):
    """The sampled tokens score above all others, and more than they are wanted."""
    _check(*_misleading(rows, V, 520, V + rows, 1024.0), k)


@pytest.mark.parametrize("rows", [67, 300])
def test_ties_of_the_sampled_tokens(rows):
    """The sampled tokens are the best and all score the same: the bracket holds, and the tie rule decides among thousands."""
    V, k, d_prime = 50000, 3000, 520
    h, Wd, Wv = _misleading(rows, V, d_prime, rows, 1024.0)
    Wv[np.arange(sv.SELECT_SAMPLE) * V // sv.SELECT_SAMPLE, 1:] = 0
    _check(h, Wd, Wv, k)


def test_some_rows_redone():
    """Rows with and without a bracket that holds, in one call."""
    rows, V, d_prime, k = 200, 40000, 520, 2000
    h, Wd, Wv = _misleading(rows, V, d_prime, 9, -1024.0)
    h[::3, 1] = 0                                  # every third row does not see what sets the sampled tokens apart
    _check(h, Wd, Wv, k)
