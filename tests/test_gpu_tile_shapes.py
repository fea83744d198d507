"""The tiled product for more than 64 hidden rows at the edges of its tiles: every tile shape, ragged rows, item counts and
reductions, by matrix, by list and by list per row.  Whole-numbered inputs whose sums are exact in float32, so results
are compared for equality."""
import pytest

torch = pytest.importorskip("torch")
sv = pytest.importorskip("paper_2602_13836_amd")

pytestmark = pytest.mark.gpu


def _whole(gen, rows, cols, top):
    return torch.randint(-top, top + 1, (rows, cols), device="cuda", generator=gen).to(torch.bfloat16)


def _inputs(rows, d, V, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    # |sum| <= 16384 * 4 * 4 < 2^24: every partial sum is exact
    h, U = _whole(gen, rows, d, 4), _whole(gen, V, d, 4)
    return gen, h, U, h.double() @ U.double().t()


# items: around one and two tiles of 128 and 256; then enough of them for the wider tiles (128 x 256: several hundred to a
# round's worth; 256 x 256: full rounds).  d: one 16-byte unit, less than a 64-element slice, one, one and a unit, odd numbers
# of slices, more slices than stages, rotated walks (16 slices and more), ragged ones among them
@pytest.mark.parametrize("rows,d,V", [
    (65, 8, 127), (65, 64, 128), (66, 72, 129), (127, 56, 255), (128, 128, 256), (129, 136, 257), (192, 192, 511),
    (255, 200, 513), (256, 320, 300), (257, 264, 130), (300, 1024, 777), (384, 1096, 1000), (512, 4096, 515), (513, 520, 259),
    # the ring of four stages (17 to 64 rows): fewer slices than stages, ragged ones, 32 x 64 to 64 x 256 tiles,
    # rows of M on cache lines (multiples of 64 elements) and off them
    (17, 520, 129), (32, 1032, 300), (24, 584, 57345), (33, 8, 127), (40, 72, 129), (60, 136, 1000), (64, 200, 32769), (48, 1096, 65537),
    (33, 136, 65567), (64, 1096, 90112), (40, 264, 90113), (50, 72, 131073), (64, 72, 155648), (48, 200, 155649),
    (60, 2056, 70000), (34, 264, 40001),
    (17, 576, 129), (32, 1088, 300), (24, 1048, 65), (20, 576, 20001), (32, 584, 20001), (24, 576, 57345), (33, 64, 16384), (64, 1024, 16383), (40, 1088, 257), (40, 1096, 20001), (64, 136, 30000),
    (130, 72, 33000), (128, 328, 70001), (256, 64, 66000), (400, 200, 66049), (520, 1032, 40003), (700, 136, 50000)])
def test_dense_product(rows, d, V):
    _, h, U, ref = _inputs(rows, d, V, rows + d)
    assert torch.equal(sv.dense_logits(h, U).double(), ref)


@pytest.mark.parametrize("rows,d,V,k", [(65, 72, 3000, 129), (200, 520, 5000, 1000), (256, 1032, 40000, 35001), (300, 64, 70000, 66000)])
def test_shared_list(rows, d, V, k):
    gen, h, U, ref = _inputs(rows, d, V, k)
    idx = torch.randint(0, V, (k,), device="cuda", generator=gen).to(torch.int32)
    assert torch.equal(sv.subset_logits(h, U, idx).double(), ref[:, idx.long()])


# short lists and long rows: the reduction split over the wavefronts of a workgroup (16 items by 16 or 32 hidden rows), with
# fewer slices of 256 than twice the wavefronts, ragged last slices, and rings deeper than what is left to read; rows of M on cache
# lines and off them (two forms)
@pytest.mark.parametrize("rows,d,V,k", [(2, 2048, 400, 1), (3, 2056, 400, 15), (16, 2104, 5000, 4101), (17, 2296, 700, 17),
                                        (31, 4096, 700, 333), (33, 2304, 700, 300), (64, 6152, 900, 513), (48, 16384, 300, 50),
                                        (9, 2112, 700, 30), (16, 4160, 5000, 4101), (40, 2240, 900, 333), (20, 4288, 700, 100)])
def test_shared_list_of_long_rows(rows, d, V, k):
    gen, h, U, ref = _inputs(rows, d, V, k + d)
    idx = torch.randint(0, V, (k,), device="cuda", generator=gen).to(torch.int32)
    assert torch.equal(sv.subset_logits(h, U, idx).double(), ref[:, idx.long()])


@pytest.mark.parametrize("rows,d,V,k", [(65, 72, 257, 200), (100, 520, 5000, 1000), (129, 1032, 3001, 500), (300, 64, 1024, 300),
                                        (512, 136, 2047, 64)])
@pytest.mark.parametrize("ascending", [True, False])
def test_list_per_row(rows, d, V, k, ascending):
    gen, h, U, ref = _inputs(rows, d, V, k + rows)
    idx = torch.rand((rows, V), device="cuda", generator=gen).topk(k, dim=1).indices.to(torch.int32)
    if ascending:
        idx = idx.sort(dim=1).values
    got = sv.subset_logits(h, U, idx.contiguous(), sorted_lists=ascending)
    assert torch.equal(got.double(), ref.gather(1, idx.long()))


# lists that crowd into a few item tiles: slices around eight and sixteen entries for each of a row's eight threads, whole tiles
# (of 256 items), none in the next, on tiles of 128 and of 256 hidden rows
@pytest.mark.parametrize("rows,d,V", [(70, 72, 1100), (128, 520, 1100), (200, 136, 1100), (513, 200, 1100)])
@pytest.mark.parametrize("ascending", [True, False])
def test_list_per_row_in_crowded_tiles(rows, d, V, ascending):
    gen, h, U, ref = _inputs(rows, d, V, rows + V)
    for at, n in ((0, 63), (256, 64), (512, 65), (256, 127), (0, 129), (768, 191), (0, 256), (200, 800), (844, 256)):
        idx = at + torch.rand((rows, n), device="cuda", generator=gen).argsort(dim=1).to(torch.int32)
        idx = idx.sort(dim=1).values if ascending else idx
        got = sv.subset_logits(h, U, idx.contiguous(), sorted_lists=ascending)
        assert torch.equal(got.double(), ref.gather(1, idx.long())), (at, n)


# large products whose lists have a little more than twice, or three or four times, as many entries as the matrix has rows: all of the
# matrix is multiplied, which takes room for a table of slices; with less the call is refused
@pytest.mark.parametrize("rows,d,V,k", [(129, 4096, 80000, 1801), (129, 4096, 80000, 1900), (260, 2048, 76000, 1160), (260, 2048, 76000, 1180)])
def test_list_per_row_of_a_large_product(rows, d, V, k):
    gen, h, U, ref = _inputs(rows, d, V, k)
    race = torch.empty((rows, V), device="cuda").exponential_(1.0, generator=gen) * torch.arange(1, V + 1, device="cuda") ** 1.1
    idx = race.topk(k, dim=1, largest=False).indices.to(torch.int32)
    want = ref.gather(1, idx.long())
    assert torch.equal(sv.subset_logits(h, U, idx).double(), want)
    idx, order = idx.sort(dim=1)
    want = want.gather(1, order)
    table = (rows * (-(-V // 256) + 1) + 3) // 4 * 16
    assert table == sv.workspace_bytes(sv.SV_OP_SUBSET_LOGITS, rows, d, V, k, idx_mode=sv.SV_IDX_SORTED)
    room, out = torch.empty(table, dtype=torch.uint8, device="cuda"), torch.empty((rows, k), dtype=torch.float32, device="cuda")

    def within(nbytes):
        return sv.load_library().specvocab_subset_logits(h.data_ptr(), rows, d, d, U.data_ptr(), V, d, sv.SV_BF16, idx.data_ptr(), k,
                                                         sv.SV_IDX_PER_ROW | sv.SV_IDX_SORTED, out.data_ptr(), room.data_ptr(), nbytes, None)
    torch.cuda.synchronize()
    assert within(table - 16) == 5 and within(table) == 0
    torch.cuda.synchronize()
    assert torch.equal(out.double(), want)


# several float32 rows over one set of rows of M, large enough that M is read once for all of them: rows of M of one to sixteen
# KB with ragged ends, more hidden rows than LDS holds at a time, more than a wavefront has lanes, items that do not divide;
# few items, which make smaller groups of hidden rows (of eight, of a last group of one, of uneven numbers)
@pytest.mark.parametrize("rows,d,V", [(2, 260, 70001), (5, 1028, 20003), (8, 2052, 9000), (70, 64, 5001), (130, 512, 4099),
                                      (3, 4096, 3001), (37, 3072, 2049), (9, 512, 4097), (65, 256, 4096), (41, 260, 6001)])
def test_float32_rows_share_one_pass(rows, d, V):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows + d)
    h, U = (torch.randint(-4, 5, (n, d), device="cuda", generator=gen).float() for n in (rows, V))
    ref = (h.double() @ U.double().t())
    assert torch.equal(sv.dense_logits(h, U).double(), ref)
    idx = torch.randint(0, V, (V,), device="cuda", generator=gen).to(torch.int32)
    idx[::3] = -1
    want = ref[:, idx.long().clamp(min=0)].masked_fill(idx < 0, float("-inf"))
    assert torch.equal(sv.subset_logits(h, U, idx, padded=True).double(), want)


# rows whose last 16-byte units do not fill a wavefront: what stands in for the missing ones must not meet an infinity
@pytest.mark.parametrize("rows,d,V", [(130, 100, 20003), (5, 1028, 20003), (8, 2052, 9000)])
def test_float32_rows_with_infinities_at_their_end(rows, d, V):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows + d)
    h, U = (torch.randint(1, 5, (n, d), device="cuda", generator=gen).float() for n in (rows, V))
    h[1, -1], h[2, -3], U[7, -2] = float("inf"), float("-inf"), float("inf")
    ref = h.double() @ U.double().t()
    torch.testing.assert_close(sv.dense_logits(h, U).double(), ref, rtol=0, atol=0, equal_nan=True)


def _far_rows(gen, n, d, apart):
    """n rows of d elements, `apart` elements from one to the next."""
    t = torch.empty((n - 1) * apart + d, dtype=torch.bfloat16, device="cuda").as_strided((n, d), (apart, 1))
    return t.copy_(_whole(gen, n, d, 4))


# Byte offsets past 32 bits: lanes name their sources by address.  The split reduction (16 and 32 hidden rows per workgroup, a
# ring of each depth), the ring on each of its tiles, and the alternating loop, with whole and ragged reductions
@pytest.mark.parametrize("rows,d,k", [(2, 2048, 700), (9, 2056, 9000), (16, 4096, 40), (20, 2048, 700), (60, 2328, 1500),
                                      (20, 584, 9000), (24, 1032, 60000), (40, 72, 700), (48, 1096, 30000), (64, 264, 50000),
                                      (70, 72, 700), (100, 520, 9000), (128, 1096, 40000), (300, 200, 9000), (513, 1032, 30000)])
def test_list_into_a_matrix_past_four_gigabytes(rows, d, k):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows + d)
    V = 70000
    U = _far_rows(gen, V, d, 32768)                                                  # 64 KB between rows: 4.6 GB
    h = _whole(gen, rows, d, 4)
    idx = torch.randint(0, V, (k,), device="cuda", generator=gen).to(torch.int32)
    idx[0], idx[1] = V - 1, 0
    ref = h.double() @ U[idx.long()].double().t()
    assert torch.equal(sv.subset_logits(h, U, idx).double(), ref)


# unions of so many tokens that a tile of 256 is as wide as its share of the chip makes it: one 32 of it, an odd number, seven of
# eight, all, and a second round, a token less and more each; requests of a wavefront that are partly, or all, past the width
@pytest.mark.parametrize("rows,d,n", [(rows, d, n + by) for rows, d, n in ((33, 72, 8192), (64, 136, 24576), (40, 1096, 40960), (60, 264, 57344),
                                                                          (48, 200, 65536)) for by in (-1, 0, 1)] + [(40, 2056, 5200), (64, 2304, 16385)])
def test_union_of_a_size(rows, d, n):
    V = 70001
    gen, h, U, ref = _inputs(rows, d, V, rows + n)
    step = n // rows
    k = max(n - (rows - 1) * step, 513)                                              # the last row's reaches the end
    at = (torch.arange(rows, device="cuda")[:, None] * step + torch.arange(k, device="cuda")) % n
    tokens = torch.randperm(V, device="cuda", generator=gen)[:n].to(torch.int32)
    idx = tokens[at].contiguous()
    assert torch.unique(idx).numel() == n
    assert torch.equal(sv.subset_logits(h, U, idx).double(), ref.gather(1, idx.long()))


def test_lists_of_their_own_into_a_matrix_past_four_gigabytes():
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2)
    rows, d, V, k = 40, 520, 70000, 500
    U, h = _far_rows(gen, V, d, 32768), _whole(gen, rows, d, 4)
    idx = torch.rand((rows, V), device="cuda", generator=gen).topk(k, dim=1).indices.to(torch.int32)
    ref = (h.double() @ U.double().t()).gather(1, idx.long())
    assert torch.equal(sv.subset_logits(h, U, idx.contiguous()).double(), ref)


# hidden states (the last positions of long sequences, say) or rows of the matrix whose distance times a tile's rows is past 32
# bits: 16 MB for the tiled kernel, 128 MB for the split reduction
@pytest.mark.parametrize("rows,d,V,h_apart,u_apart", [(20, 1032, 300, 8400000, 1032), (40, 520, 1000, 8400000, 520), (70, 136, 1000, 8400000, 136),
                                                      (257, 72, 700, 8400000, 80), (40, 200, 100, 200, 8400000), (70, 520, 130, 528, 8400000),
                                                      (9, 2056, 300, 67200000, 2056), (18, 2104, 40, 2104, 134400000)])
def test_rows_far_apart(rows, d, V, h_apart, u_apart):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows + d)
    h, U = _far_rows(gen, rows, d, h_apart), _far_rows(gen, V, d, u_apart)
    ref = h.double() @ U.double().t()
    assert torch.equal(sv.dense_logits(h, U).double(), ref)
    idx = torch.rand((rows, V), device="cuda", generator=gen).topk(V // 2 + 1, dim=1).indices.to(torch.int32)
    for ordered in (False, True):
        idx = idx.sort(dim=1).values if ordered else idx.contiguous()
        assert torch.equal(sv.subset_logits(h, U, idx, sorted_lists=ordered).double(), ref.gather(1, idx.long()))
