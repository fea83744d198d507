"""The tiled product with a last tile of hidden rows that some wavefronts have few groups of 32 of, or none.  Whole-numbered inputs
whose sums are exact in float32, so results are compared for equality."""
import pytest

torch = pytest.importorskip("torch")
sv = pytest.importorskip("paper_2602_13836_amd")

pytestmark = pytest.mark.gpu


def _numbers(rows, V, d):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows + V)
    return (torch.randint(-4, 5, (n, d), device="cuda", generator=gen).to(torch.bfloat16) for n in (rows, V))


def _check(h, U):
    out = torch.full((h.shape[0], U.shape[0]), float("nan"), device="cuda")
    assert torch.equal(sv.dense_logits(h, U, out=out).double(), h.double() @ U.double().t())


# rows one past a group, a wavefront's half and a tile, and one short of them; V: 256 x 256, 128 x 256 and 128 x 128 tiles
@pytest.mark.parametrize("rows", [97, 161, 191, 193, 225, 257, 289, 385, 417, 511])
@pytest.mark.parametrize("V,d", [(66001, 72), (20000, 200), (700, 1032)])
def test_last_tile(rows, V, d):
    _check(*_numbers(rows, V, d))


def test_last_tile_of_rows_far_apart():
    """Hidden rows 16 MB apart, which are named by address (2.7 GB of them)."""
    h, U = _numbers(161, 300, 72)
    apart = torch.empty((161, 8 << 20), dtype=torch.bfloat16, device="cuda")
    apart[:, :72] = h
    _check(apart[:, :72], U)


@pytest.mark.parametrize("rows,V,d", [(129, 28000, 200), (160, 31000, 4096), (130, 32768, 136)])
def test_one_group_of_a_last_tile(rows, V, d):
    """128 x 256 tiles in one round of workgroups whose last tile of hidden rows has 32 of them at most.  The group beside
    them is multiplied too, and stores nothing."""
    h, U = _numbers(rows, V, d)
    out = torch.full((rows + 1, V), float("nan"), device="cuda")
    sv.dense_logits(h, U, out=out[:rows])
    assert torch.equal(out[:rows].double(), h.double() @ U.double().t()) and bool(out[rows].isnan().all())
