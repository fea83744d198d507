"""The selection by two-byte keys at the edges of its parts (32768 tokens), where its sample misleads, where its lists or ties leave
their room and where half precision says nothing.  Scores are exact (whole numbers times a power of two), so the ids must be those of a
full sort, ties to the smaller id."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
sv = pytest.importorskip("paper_2602_13836_amd")

pytestmark = pytest.mark.gpu

PART = 32768
# a part, one token more or less, several parts a workgroup, the largest vocabulary; panels of 64, 128 and 256 hidden rows
EDGES = [(65, 16384, 256, 4), (16, PART, 128, 900), (33, PART + 1, 40, PART + 1), (64, 2 * PART - 1, 8, 20000),
         (24, 2 * PART + 33, 256, 30000), (64, 8 * PART, 128, 6000), (50, 12 * PART, 64, 90000), (64, 11 * PART + 7, 256, 1),
         (2, 16385, 128, 2000), (8, 131072, 16, 16384), (65, PART, 256, 5000), (128, 65536, 200, 8000), (200, 20000, 264, 3000),
         (70, 100001, 512, 2500), (130, 70000, 264, 69999)]
TOGETHER = [(60, 128256, 256, 16384), (20, 32768, 64, 3000), (70, 50000, 136, 6000), (9, 262144, 128, 9000), (3, 70001, 48, 8000)]
OFFSET = [(60, 128256, 256, 4096), (20, 32768, 64, 3000), (3, 70001, 40, 8000), (100, 40000, 256, 1500), (150, 20000, 304, 700),
          (66, 100000, 512, 3000)]
MISLED = [(20000, 900), (40000, 200), (40000, 9000), (150001, 4000)]
ONE_SUM = [(2, 40000, 128), (8, 128256, 64), (9, 32768, 256), (64, 50000, 200), (66, 60000, 256), (130, 40000, 512)]


def _bf16(a):
    return torch.from_numpy(a.astype(np.float32)).cuda().to(torch.bfloat16)


def _inputs(rows, V, d_prime, seed, d=64):
    rng = np.random.default_rng(seed)
    return (rng.integers(-1, 2, (rows, d)), rng.integers(-1, 2, (d_prime, d)), rng.integers(-2, 3, (V, d_prime)) / 64.0)


def _check(h, Wd, Wv, k, scale=1.0):
    h, Wd, Wv = _bf16(h), _bf16(Wd), _bf16(Wv * scale)
    need = sv.workspace_bytes(sv.SV_OP_SELECT, h.shape[0], h.shape[1], Wv.shape[0], k, Wd.shape[0], 0, sv.SV_BF16, 0)
    ws = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    idx, _ = sv.select(h, Wd, Wv, k, ws=ws[:need])
    s = (h.double() @ Wd.double().t()) @ Wv.double().t()
    want = torch.sort(s, dim=1, descending=True, stable=True).indices[:, :k].sort(dim=1).values
    assert torch.equal(idx.long(), want)
    assert bool((ws[need:] == 0x5A).all())             # nothing past the workspace is written


@pytest.mark.parametrize("rows,V,d_prime,k", EDGES)
def test_edges(rows, V, d_prime, k):
    _check(*_inputs(rows, V, d_prime, rows + k), k)


def _sampled(V):
    """Ids of the sampled tokens: of every 32 the same two, four or eight."""
    places = np.array([0, 2, 8, 10] if V <= 32768 else [0, 10] if V <= 65536 else [0])
    ids = np.arange(0, V, 32)[:, None] + np.concatenate((places, places + 16))
    return ids[ids < V]


def _records(ws, rows, V, d_prime):
    """What a call leaves in its workspace: the rows' keys, and how many scores were above their bracket and in it."""
    units, parts = (V + 31) // 32, (V + PART - 1) // PART
    at, stride = (rows * d_prime * 2 + 255) // 256 * 256, (units * 64 + 255) // 256 * 256 | 256
    keys = ws[at: at + rows * stride].view(rows, stride)[:, : units * 64].cpu().numpy().view(np.uint16)
    at += rows * stride
    return keys, ws[at: at + rows * parts * 8].cpu().numpy().view(np.uint32).reshape(rows, parts, 2).sum(1)


def _ids_and_records(h, Wd, Wv, k):
    (rows, d), (V, d_prime) = h.shape, Wv.shape
    ws = torch.empty(sv.workspace_bytes(sv.SV_OP_SELECT, rows, d, V, k, d_prime, 0, sv.SV_BF16, 0), dtype=torch.uint8, device="cuda")
    idx, _ = sv.select(h, Wd, Wv, k, ws=ws)
    records = _records(ws, rows, V, d_prime)
    assert torch.equal(idx, sv.select(h, Wd, Wv, k, want_scores=True)[0])      # (the scores in memory)
    return records


@pytest.mark.parametrize("rows,V,d_prime,k", TOGETHER)
@pytest.mark.parametrize("together", [1, 32, 700])
def test_neighbours_with_much_in_common(rows, V, d_prime, k, together):
    """Seven tenths of a score's variance is shared by `together` neighbouring tokens: the bracket has the k-th score of every row all
    the same (within 6 standard deviations of a sample of independent ones)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(together)
    randn = lambda *n: torch.randn(n, generator=gen, device="cuda")
    Wv = randn(V, d_prime)
    if together > 1:
        Wv = 0.3 ** 0.5 * Wv + 0.7 ** 0.5 * randn(V // together + 1, d_prime).repeat_interleave(together, 0)[:V]
    _, counts = _ids_and_records(randn(rows, 512).bfloat16(), randn(d_prime, 512).bfloat16(), Wv.bfloat16(), k)
    assert ((counts[:, 0] < k) & (k <= counts.sum(1))).all()


@pytest.mark.parametrize("rows,V,d_prime,k", OFFSET)
@pytest.mark.parametrize("offset", [-30.0, 0.0, 30.0, 1000.0])
def test_scores_with_a_common_offset(rows, V, d_prime, k, offset):
    """All scores of a row lie `offset` standard deviations from zero.  A key says where a score lies among those of its row, so few share
    the k-th one's (half precision has 2048 numbers between one and three deviations)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows)
    randn = lambda *n: torch.randn(n, generator=gen, device="cuda")
    h, Wd, Wv = randn(rows, 512), randn(d_prime, 512) / 16, randn(V, d_prime)
    h[:, 0] = 8.0
    Wd[:, 0] = 0.0
    Wd[0, 0] = 1.0                                     # h'[0] = 8 and nothing else in every row, against sums of 512 / 256 in the others
    Wv[:, 0] = offset * (2.0 * d_prime) ** 0.5 / 8
    keys, _ = _ids_and_records(h.bfloat16(), Wd.bfloat16(), Wv.bfloat16(), k)
    kth = -np.partition(-keys.astype(np.int32), k - 1, axis=1)[:, k - 1: k]
    assert (keys == kth).sum(1).max() <= 64            # (what the quick choice among them takes)


@pytest.mark.parametrize("V,k", MISLED)
@pytest.mark.parametrize("best", [True, False])
def test_samples_that_mislead(V, k, best):
    """The sampled tokens are the best of all, or the worst: the k-th score lies outside of the bracket."""
    rows, d_prime = 20, 32
    h, Wd, Wv = _inputs(rows, V, d_prime, k)
    h[:, 1] = 1
    Wd[:, 1] = 0
    Wd[0, :] = 0
    Wd[0, 1] = 1                                       # h'[0] = 1 in every row
    Wv[:, 0] = 0
    Wv[_sampled(V), 0] = 64.0 if best else -64.0
    _check(h, Wd, Wv, k)


@pytest.mark.parametrize("k", [1000, 12000, 40000])
def test_parts_of_one_score(k):
    """Nearly all tokens of the second part share a score that decides in some of the rows: more than a part's list holds, and than LDS
    holds ties."""
    rows, V, d_prime = 15, 3 * PART, 32
    h, Wd, Wv = _inputs(rows, V, d_prime, k)
    h[:, 1:] = 0
    h[:, 0] = np.arange(rows) % 5 - 2                  # h' = (h[0], 0, ...), zeros among them
    Wd[:, 0] = 0
    Wd[0, 0] = 1
    Wv[PART: 2 * PART - 100, 0] = 1 / 64.0
    _check(h, Wd, Wv, k)


# scores that half precision rounds to zero or to its largest number: ties by the tens of thousands
@pytest.mark.parametrize("scale", [2.0 ** -100, 2.0 ** -20, 2.0 ** 18, 2.0 ** 100])
@pytest.mark.parametrize("k", [77, 30000])
def test_scores_out_of_the_range_of_halves(scale, k):
    _check(*_inputs(12, 70000, 64, k), k, scale)


def test_hidden_rows_of_any_size():
    """Every row's keys are relative to the row's largest element."""
    rows, V, d_prime, k = 40, 50000, 128, 1500
    h, Wd, Wv = _inputs(rows, V, d_prime, 7)
    _check(h * 2.0 ** np.linspace(-60, 60, rows).astype(int)[:, None], Wd, Wv, k)


@pytest.mark.parametrize("rows,V,d_prime", ONE_SUM)
def test_one_sum_per_score(rows, V, d_prime):
    """All rows of W_vocab hold the same numbers in different orders and h' is one number d' times, so all scores are equal but for their
    rounding, which decides what is selected: the same, whether or not the scores go through memory."""
    rng = np.random.default_rng(rows + V)
    Wv = _bf16(rng.permuted(np.tile(rng.normal(size=d_prime) + 1.0, (V, 1)), axis=1))
    h, Wd = _bf16(rng.normal(size=(rows, 64)) + 2.0), _bf16(np.full((d_prime, 64), 1 / 64))
    _ids_and_records(h, Wd, Wv, V // 20)
