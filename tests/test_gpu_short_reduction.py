"""The kernel that keeps the hidden rows in registers (more than 64 rows, selectors of up to 512 elements), at the edges of
its panels, runs and steps."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
sv = pytest.importorskip("paper_2602_13836_amd")

pytestmark = pytest.mark.gpu


def _exact_inputs(rows, V, d_prime, seed, d=64):
    """Weights and states whose products and sums are exact in every precision used: h' is a whole number of at most 64
    (exact in bf16), a score a multiple of 2^-6 below 2^10."""
    rng = np.random.default_rng(seed)

    def bf16(a):
        return torch.from_numpy(a.astype(np.float32)).cuda().to(torch.bfloat16)

    h = bf16(rng.integers(-1, 2, (rows, d)))
    Wd = bf16(rng.integers(-1, 2, (d_prime, d)))
    Wv = bf16(rng.integers(-2, 3, (V, d_prime)) / 64.0)
    return h, Wd, Wv


def _scores(h, Wd, Wv):
    return (h.double() @ Wd.double().t()) @ Wv.double().t()


# rows: one panel and a bit more of each size (128, 256, 512), both sides; d_prime: one unit, odd numbers of units, whole
# steps, the two widths that registers hold (256, 512) and one past the second; V: whole runs, a run of one item more, one less
SHAPES = [(65, 32768, 256), (127, 32769, 8), (128, 33000, 24), (129, 40001, 256), (255, 32831, 200), (256, 65536, 248),
          (257, 32832, 256), (300, 33023, 136), (511, 32895, 256), (512, 65537, 16), (513, 32770, 256), (65, 32768, 264),
          (200, 33001, 512), (300, 40960, 504), (100, 33333, 520), (1030, 32800, 64)]
# numbers of panels that do not divide an XCD's 32 compute units, and more of them than there are: several rounds of workgroups,
# runs of few and of many steps
SHAPES += [(700, 40000, 64), (1300, 32790, 256), (2100, 32769, 128), (8500, 32768, 32), (17000, 32800, 16)]


# one run shorter than a step, fewer items than a sub-tile has, wavefronts along the matrix that see none
SMALL = [(65, 1, 8), (130, 31, 256), (200, 33, 264), (300, 63, 64), (513, 65, 256)]


@pytest.mark.parametrize("rows,V,d_prime", SHAPES + SMALL)
def test_log_probabilities_of_a_batch(rows, V, d_prime):
    h, Wd, Wv = _exact_inputs(rows, V, d_prime, rows + d_prime)
    s = _scores(h, Wd, Wv)
    ref = torch.log_softmax(s, dim=1)
    out = torch.full((rows, V), float("nan"), device="cuda")
    sv.aux_log_softmax(h, Wd, Wv, out=out)
    # The scores are exact.  In units of 2^-24: an exponential e^-x is off by at most 2 x + 2 (its argument is scaled to base
    # two), which counts with its weight in the sum, and so are the factors that move a partial sum to a larger maximum
    # (together no further than the mean x, and 2); a lane's sum, the runs' and the rows' are fewer than 128 additions one after
    # the other, whose roundings of half a unit each are independent (six standard deviations of their sum); the
    # logarithm, its sum with the maximum and the last subtraction round once each.
    x = s.amax(dim=1, keepdim=True) - s
    mean_x = (ref.exp() * x).sum(dim=1, keepdim=True)
    lse = s[:, :1] - ref[:, :1]
    tol = 2.0 ** -24 * (6 * 0.5 * 128 ** 0.5 + 4 * mean_x + 4 + ref.abs() + 2 * lse.abs())
    ratio = float(((out.double() - ref).abs() / tol).max())
    assert ratio <= 1, ratio                       # (false for NaN)


@pytest.mark.parametrize("rows,V,d_prime", SHAPES)
@pytest.mark.parametrize("share", [0.5, 0.05, 0.0005])
def test_selection_of_a_batch(rows, V, d_prime, share):
    """Exact scores with many ties: the ids must be those of a full sort, ties to the smaller id."""
    h, Wd, Wv = _exact_inputs(rows, V, d_prime, 7 * rows + d_prime)
    k = max(1, int(V * share))
    idx, _ = sv.select(h, Wd, Wv, k)
    s = _scores(h, Wd, Wv)
    # (stable sort by descending score: equal scores stay in ascending id order)
    want = torch.sort(s, dim=1, descending=True, stable=True).indices[:, :k].sort(dim=1).values
    assert torch.equal(idx.long(), want)
