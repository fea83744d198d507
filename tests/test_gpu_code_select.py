"""The selection of a batch by one-byte codes, where its map is of no use or its lists leave LDS.  Scores are exact (whole
numbers in steps of 2^-6), so the ids must be those of a full sort, ties to the smaller id."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
sv = pytest.importorskip("paper_2602_13836_amd")

pytestmark = pytest.mark.gpu

SAMPLE = sv.SELECT_CODE_SAMPLE


def _bf16(a):
    return torch.from_numpy(a.astype(np.float32)).cuda().to(torch.bfloat16)


def _inputs(rows, V, d_prime, seed, d=64):
    rng = np.random.default_rng(seed)
    return (rng.integers(-1, 2, (rows, d)), rng.integers(-1, 2, (d_prime, d)), rng.integers(-2, 3, (V, d_prime)) / 64.0)


# for inputs that are hard on codes: rows, V, d'; panels of 128, of 512, and selectors of more than 256 elements
HARD = [(70, 50000, 64), (300, 33000, 256), (258, 40000, 512)]
EDGES = [(65, 16384, 128, 100), (65, 32768, 64, 1), (66, 32769, 8, 32769), (90, 98303, 256, 9000), (129, 65536, 256, 64), (70, 65537, 40, 3000),
         (257, 16384, 512, 300), (300, 65537, 512, 40000), (65, 262144, 512, 500), (512, 24576, 200, 2000)]
LONG_LISTS = [(300, 200000, 256, 100000), (65, 393216, 256, 196608)]
ONE_SUM = [(70, 40000, 128), (140, 60000, 256), (100, 70000, 200), (257, 33000, 512)]


def _check(h, Wd, Wv, k):
    h, Wd, Wv = _bf16(h), _bf16(Wd), _bf16(Wv)
    idx, _ = sv.select(h, Wd, Wv, k)
    s = (h.double() @ Wd.double().t()) @ Wv.double().t()
    want = torch.sort(s, dim=1, descending=True, stable=True).indices[:, :k].sort(dim=1).values
    assert torch.equal(idx.long(), want)


# units of 32 codes and rounds of 1024 of them at their edges, d' of one unit to the widest
@pytest.mark.parametrize("rows,V,d_prime,k", [(65, 32768, 256, 1), (66, 32769, 8, 32769), (70, 65536, 512, 64), (65, 65537, 40, 3000),
                                              (65, 98303, 256, 9000), (260, 40000, 128, 500), (65, 393216, 16, 20000),
                                              (65, 262145, 24, 131072),
                                              # panels of 64 rows: steps of 128 rows of W_vocab, runs shorter than that and of one and a half
                                              (40, 16384, 256, 300), (64, 16385, 200, 5000), (16, 49000, 128, 1500), (41, 40960, 256, 2000),
                                              (60, 262144, 248, 8192), (17, 24001, 8, 700), (9, 16384, 256, 100), (24, 70000, 256, 900),
                                              # ids a lane per token: from less to more than that many in 64 units, few units, the last one cut
                                              (12, 16385, 128, 16000), (9, 32768, 40, 9300), (30, 20001, 64, 5200), (64, 200000, 256, 100000),
                                              (300, 50017, 256, 14000)])
def test_edges(rows, V, d_prime, k):
    _check(*_inputs(rows, V, d_prime, rows + k), k)


@pytest.mark.parametrize("rows,V,d_prime,k", EDGES)
def test_edges_of_codes(rows, V, d_prime, k):
    _check(*_inputs(rows, V, d_prime, rows + k), k)


def test_static_scratch_nearly_full():
    """20 rows of 33500 tokens: what the library's static scratch just holds.  The sums of real numbers round, so equal ids also say
    that both calls ran the same kernels."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    h, Wd, Wv = (torch.randn(n, generator=gen, device="cuda").to(torch.bfloat16) for n in ((20, 512), (64, 512), (33500, 64)))
    assert 8 << 20 > sv.workspace_bytes(sv.SV_OP_SELECT, 20, 512, 33500, 1000, 64, 0, sv.SV_BF16, 0) > 7.5 * 2 ** 20
    idx, _ = sv.select(h, Wd, Wv, 1000)
    idx_static = torch.full_like(idx, -1)
    sv.select_static(h, Wd, Wv, 1000, idx_static)
    assert torch.equal(idx, idx_static)


# a list of entries that is longer than its LDS (wide intervals: half of the tokens are wanted), more rows than CUs among them
@pytest.mark.parametrize("rows,V,d_prime,k", LONG_LISTS)
def test_lists_longer_than_lds(rows, V, d_prime, k):
    _check(*_inputs(rows, V, d_prime, rows), k)


@pytest.mark.parametrize("rows,V,d_prime", HARD)
def test_rows_of_zeros_and_plateaus(rows, V, d_prime):
    """Rows without any difference between tokens; rows with two, three or a few different scores, so that tens of thousands
    share the code that decides."""
    h, Wd, Wv = _inputs(rows, V, d_prime, 3)
    h[10] = 0
    h[69] = 0
    h[20:30] = 0
    h[20:30, 0] = np.arange(10) % 3 - 1
    Wd[:, 0] = 0
    Wd[0, 0] = 1                                   # rows 20 to 29 see only the first column of W_vocab
    Wv[:, 0] = np.sign(Wv[:, 0]) / 64.0
    for k in (1, 100, 16000, 33000, V):
        _check(h, Wd, Wv, k)


@pytest.mark.parametrize("share", [1.0, 0.9, 0.55])
@pytest.mark.parametrize("k", [1, 9000, 20000, 39999])
@pytest.mark.parametrize("rows,V,d_prime", [(68, 40000, 32), HARD[2]])
def test_lists_longer_than_their_memory(rows, V, d_prime, share, k):
    """More than half of the tokens share a score that the map has an interval for, and most of their codes do not fit the list; some
    rows select among them, some have them above or below the k-th score.  Nothing past the workspace is written."""
    h, Wd, Wv = _inputs(rows, V, d_prime, k)
    h[:, 1:] = 0
    h[:, 0] = np.arange(rows) % 5 - 2              # h' = (h[0], 0, ...)
    Wd[:, 0] = 0
    Wd[0, 0] = 1
    Wv[np.random.default_rng(k).random(V) < share, 0] = 1 / 64.0
    _check(h, Wd, Wv, k)
    h, Wd, Wv = _bf16(h), _bf16(Wd), _bf16(Wv)
    need = sv.workspace_bytes(sv.SV_OP_SELECT, rows, 64, V, k, d_prime, 0, sv.SV_BF16, 0)
    ws = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    idx, _ = sv.select(h, Wd, Wv, k, ws=ws[:need])
    assert torch.equal(idx, sv.select(h, Wd, Wv, k)[0]) and bool((ws[need:] == 0x5A).all())


@pytest.mark.parametrize("k", [200, 5000, 20000])
@pytest.mark.parametrize("best", [True, False])
@pytest.mark.parametrize("rows,V,d_prime", [(66, 40000, 32)] + HARD[1:])
def test_samples_that_mislead(rows, V, d_prime, k, best):
    """The sampled tokens are the best of all, or the worst: the k-th score lies outside of what the sample says."""
    h, Wd, Wv = _inputs(rows, V, d_prime, k)
    h[:, 1] = 1
    Wd[:, 1] = 0
    Wd[0, :] = 0
    Wd[0, 1] = 1                                   # h'[0] = 1 in every row
    Wv[:, 0] = 0
    Wv[np.arange(SAMPLE) * V // SAMPLE, 0] = 64.0 if best else -64.0
    _check(h, Wd, Wv, k)


@pytest.mark.parametrize("far", [2.0 ** 6, 2.0 ** 20, 2.0 ** 50])
@pytest.mark.parametrize("k", [300, 4000])
@pytest.mark.parametrize("rows,V,d_prime", [(65, 33000, 64)] + HARD[1:])
def test_scores_far_from_all_others(rows, V, d_prime, k, far):
    """A few tokens of every row score far above and far below the rest, sampled ones among them: one step of the map's first
    histogram holds nearly the whole sample.  (Their own scores round; all of those above are selected, none of those below.)"""
    h, Wd, Wv = _inputs(rows, V, d_prime, k)
    h[:, 1] = 1
    Wd[:, 1] = 0
    Wd[0, :] = 0
    Wd[0, 1] = 1                                   # h'[0] = 1 in every row
    Wv[:, 0] = 0
    Wv[::1009, 0] = far
    Wv[5::2003, 0] = -far
    _check(h, Wd, Wv, k)


# (12 and 40 rows: two bytes per score)
@pytest.mark.parametrize("rows,V,d_prime", [(12, 33000, 64), (40, 33000, 64), (70, 33000, 64), HARD[2]])
@pytest.mark.parametrize("up,down,none", [(1009, 2003, 3001), (2, 2003, 3001), (1009, 2, 3001), (1009, 2003, 4), (1, 2003, 3001)])
@pytest.mark.parametrize("k", [20, 300, 20000])
def test_scores_that_are_infinite(rows, V, d_prime, up, down, none, k):
    """Every `up`-th token scores infinity, every `down`-th minus infinity, every `none`-th no number, which is never selected (as where
    the scores go through memory) as long as there are k others."""
    h, Wd, Wv = _inputs(rows, V, d_prime, k)
    h[:, 1] = 1
    Wd[:, 1] = 0
    Wd[0, :] = 0
    Wd[0, 1] = 1                                   # h'[0] = 1 in every row
    Wv[:, 0] = 0
    Wv[::up, 0] = np.inf
    Wv[5::down, 0] = -np.inf
    Wv[7::none, 0] = np.nan
    h, Wd, Wv = _bf16(h), _bf16(Wd), _bf16(Wv)
    s = ((h.double() @ Wd.double().t()) @ Wv.double().t()).nan_to_num(nan=-1e39, posinf=1e38, neginf=-1e38)
    want = torch.sort(s, dim=1, descending=True, stable=True).indices[:, :k].sort(dim=1).values
    idx, _ = sv.select(h, Wd, Wv, k)
    assert torch.equal(idx.long(), want)


@pytest.mark.parametrize("rows", [40, 300])
def test_replays_of_a_captured_call(rows):
    V, d_prime, k = 40000, 128, 1500
    h, Wd, Wv = (_bf16(a) for a in _inputs(rows, V, d_prime, rows))
    idx = torch.zeros((rows, k), dtype=torch.int32, device="cuda")
    ws = torch.empty(sv.workspace_bytes(sv.SV_OP_SELECT, rows, 64, V, k, d_prime, 0, sv.SV_BF16, 0), dtype=torch.uint8, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        sv.select(h, Wd, Wv, k, idx_out=idx, ws=ws)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sv.select(h, Wd, Wv, k, idx_out=idx, ws=ws)
    for seed in range(3):
        h.copy_(_bf16(_inputs(rows, V, d_prime, 100 + seed)[0]))
        ws.fill_(seed * 85)
        graph.replay()
        got = idx.clone()
        want, _ = sv.select(h, Wd, Wv, k)
        torch.cuda.synchronize()
        assert torch.equal(got, want)


@pytest.mark.parametrize("rows,V,d_prime", [(9, 32768, 256), (16, 40000, 128), (17, 16384, 256), (24, 60000, 200), (32, 90112, 128), (20, 90113, 64),
                                            (32, 128256, 256), (33, 100000, 256), (60, 33000, 248), (65, 20000, 512), (130, 40000, 512)] + ONE_SUM)
def test_one_sum_per_score(rows, V, d_prime):
    """A call adds a score's products the same way whether or not it is asked for the scores.  All rows of W_vocab hold the same numbers in
    different orders and h' is one number d' times, so all scores are equal but for their rounding, which decides what is selected."""
    rng = np.random.default_rng(rows + V)
    base = rng.normal(size=d_prime) + 1.0
    Wv = _bf16(rng.permuted(np.tile(base, (V, 1)), axis=1))
    h = _bf16(rng.normal(size=(rows, 64)) + 2.0)
    Wd = _bf16(np.full((d_prime, 64), 1 / 64))
    k = V // 20
    idx, _ = sv.select(h, Wd, Wv, k)
    with_scores, sc = sv.select(h, Wd, Wv, k, want_scores=True)
    # (they do round differently, by more than h' does: rows whose h' is the same have the same scores)
    assert len(sc.unique()) > len((h.double() @ Wd.double().t())[:, 0].bfloat16().unique())
    assert torch.equal(idx, with_scores)
