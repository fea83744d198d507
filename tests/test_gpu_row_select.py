"""The selection from rows of up to 16384 scores in one launch, and h' made by the launch that makes the scores.  Scores are exact (whole numbers
times a power of two), so ids and scores must be those of a full sort, ties to the smaller id."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
sv = pytest.importorskip("paper_2602_13836_amd")

pytestmark = pytest.mark.gpu


def _dev(a, dtype):
    return torch.from_numpy(a.astype(np.float32)).cuda().to(dtype)


def _inputs(rows, V, d_prime, seed, d=64, values=3):
    rng = np.random.default_rng(seed)
    return (rng.integers(-1, 2, (rows, d)), rng.integers(-1, 2, (d_prime, d)), rng.integers(-values + 1, values, (V, d_prime)) / 64.0)


def _check(h, Wd, Wv, k, dtype, tau=None):
    h, Wd, Wv = (_dev(a, dtype) for a in (h, Wd, Wv))
    s = (h.double() @ Wd.double().t()) @ Wv.double().t()
    want = torch.sort(s, dim=1, descending=True, stable=True).indices[:, :k].sort(dim=1).values
    score = s.gather(1, want)
    if tau is not None:
        want = torch.where(score >= tau, want, -1)
        score = torch.where(score >= tau, score, -np.inf)
    idx, sc = sv.select(h, Wd, Wv, k, want_scores=True, tau=tau)
    assert torch.equal(idx.long(), want) and torch.equal(sc.double(), score)
    assert torch.equal(sv.select(h, Wd, Wv, k, tau=tau)[0], idx)


# groups of 4096 scores at their edges, rows that do not start on 16 bytes, a row of less than four
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,V,k", [(1, 1, 1), (3, 3, 2), (2, 257, 256), (5, 4095, 100), (1, 4096, 4096), (9, 4097, 1), (40, 8191, 700),
                                      (1, 8193, 8192), (70, 12289, 3000), (3, 16383, 5000), (8, 16384, 16384), (260, 10001, 1000)])
def test_edges(dtype, rows, V, k):
    _check(*_inputs(rows, V, 16, rows + V, values=40), k, dtype)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("values,d_prime", [(1, 8), (2, 8), (3, 16)])
@pytest.mark.parametrize("k", [1, 77, 3000, 9999])
def test_many_equal_scores(dtype, values, d_prime, k):
    """A few different scores (or one) among ten thousand: more of the deciding one than are ranked by counting."""
    h, Wd, Wv = _inputs(4, 10000, d_prime, k, values=values)
    h[1] = 0
    _check(h, Wd, Wv, k, dtype)
    _check(h, Wd, Wv, k, dtype, tau=0.0)


@pytest.mark.parametrize("k", [5, 900, 7000])
def test_infinite_scores(k):
    h, Wd, Wv = _inputs(3, 9000, 16, k)
    h[:, 1] = 1
    Wd[:, 1] = 0
    Wd[0, :] = 0
    Wd[0, 1] = 1                                   # h'[0] = 1 in every row
    Wv[:, 0] = 0
    Wv[::100, 0] = np.inf
    Wv[5::70, 0] = -np.inf
    _check(h, Wd, Wv, k, torch.float32)


# W_down of one to 4096 units of 16 bytes, rows of one unit to 128: h' made on the way, and just not
@pytest.mark.parametrize("dtype,d,d_prime,V", [(torch.float32, 4, 4, 300), (torch.float32, 256, 32, 8192), (torch.float32, 512, 32, 16384),
                                               (torch.float32, 252, 64, 5000), (torch.float32, 512, 36, 5000), (torch.float32, 516, 28, 700),
                                               (torch.bfloat16, 8, 8, 2048), (torch.bfloat16, 1024, 32, 9000), (torch.bfloat16, 520, 40, 3000),
                                               (torch.bfloat16, 1024, 40, 3000), (torch.float32, 64, 256, 3000)])
def test_down_projection_on_the_way(dtype, d, d_prime, V):
    for rows in (1, 4):
        _check(*_inputs(rows, V, d_prime, d, d=d), min(V, 200), dtype)
    wide = _dev(_inputs(2, V, d_prime, 1, d=2 * d)[0], dtype)[:, :d]           # hidden rows further apart than their length
    _, Wd, Wv = _inputs(2, V, d_prime, 2, d=d)
    Wd, Wv = _dev(Wd, dtype), _dev(Wv, dtype)
    assert torch.equal(sv.select(wide, Wd, Wv, 100)[0], sv.select(wide.contiguous(), Wd, Wv, 100)[0])
