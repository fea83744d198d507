"""The tiled product with a last tile of hidden rows that some wavefronts have few groups of 32 of, or none.  Whole-numbered inputs
whose sums are exact in float32, so results are compared for equality."""
import pytest

torch = pytest.importorskip("torch")
sv = pytest.importorskip("paper_2602_13836_amd")

pytestmark = pytest.mark.gpu


# rows one past a group, a wavefront's half and a tile, and one short of them; V: 256 x 256, 128 x 256 and 128 x 128 tiles;
# far: hidden rows 16 MB apart, which are named by address
@pytest.mark.parametrize("rows", [97, 161, 191, 193, 225, 257, 289, 385, 417, 511])
@pytest.mark.parametrize("V,d,far", [(66001, 72, False), (20000, 200, False), (700, 1032, False), (300, 72, True)])
def test_last_tile(rows, V, d, far):
    if far and rows != 161:
        pytest.skip("one count of rows is enough for 2.7 GB of hidden states")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows + V)
    h, U = (torch.randint(-4, 5, (n, d), device="cuda", generator=gen).to(torch.bfloat16) for n in (rows, V))
    ref = h.double() @ U.double().t()
    if far:
        apart = torch.empty((rows, 8 << 20), dtype=torch.bfloat16, device="cuda")
        apart[:, :d] = h
        h = apart[:, :d]
    out = torch.full((rows, V), float("nan"), device="cuda")
    assert torch.equal(sv.dense_logits(h, U, out=out).double(), ref)


@pytest.mark.parametrize("rows,V,d", [(129, 28000, 200), (160, 31000, 4096), (130, 32768, 136)])
def test_one_group_of_a_last_tile(rows, V, d):
    """128 x 256 tiles in one round of workgroups whose last tile of hidden rows has 32 of them at most.  The group beside them is multiplied too, and stores nothing."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows + V)
    h, U = (torch.randint(-4, 5, (n, d), device="cuda", generator=gen).to(torch.bfloat16) for n in (rows, V))
    out = torch.full((rows + 1, V), float("nan"), device="cuda")
    sv.dense_logits(h, U, out=out[:rows])
    assert torch.equal(out[:rows].double(), h.double() @ U.double().t()) and bool(out[rows].isnan().all())
