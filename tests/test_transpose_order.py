"""The order in which tile transposes take their tiles: lists of neighbouring tiles for every XCD, or diagonals."""
import ctypes

import pytest
import torch

from tests.test_transpose import pure_transpose
from tests.util import device_header, host_build
from workloads.configs import TORCH_DTYPE


@pytest.fixture(scope="module")
def place(tmp_path_factory):
    """transpose_place of the device header, built for the CPU: block -> (batch entry, tile row, tile column)"""
    lib = host_build(device_header("constexpr u32 kTransposeNear", "transpose_place") + """
extern "C" i64 place(i64 t, i64 batch, i64 tiles_p, i64 tiles_q, int lists, i64* pq) {
  return transpose_place(t, batch, tiles_p, tiles_q, 1, 1, lists != 0, pq[0], pq[1]);
}
""", tmp_path_factory.mktemp("place") / "transpose")
    lib.place.restype = ctypes.c_int64
    lib.place.argtypes = [ctypes.c_int64] * 4 + [ctypes.c_int, ctypes.c_void_p]
    pq = (ctypes.c_int64 * 2)()

    def call(t, batch, tiles_p, tiles_q, lists):
        b = lib.place(t, batch, tiles_p, tiles_q, lists, pq)
        return b, pq[0], pq[1]
    return call


def _listed(t, batch, tiles_p, tiles_q, near=4):
    """The tile that block t takes from the lists, in unbounded integers."""
    per_batch = tiles_p * tiles_q
    n, x = batch * per_batch, t % 8
    k = x * (n // 8) + min(x, n % 8) + t // 8
    b, r = divmod(k, per_batch)
    g, i = divmod(r, near * tiles_q)
    w = min(near, tiles_p - g * near)
    return b, g * near + i % w, i // w


@pytest.mark.parametrize("lists", [0, 1])
def test_every_tile_once(place, lists):
    for batch, tiles_p, tiles_q in [(1, 1, 1), (1, 5, 3), (3, 4, 7), (2, 3, 3), (1, 33, 94), (7, 1, 1), (1, 9, 1), (5, 2, 11), (1, 3, 40)]:
        n = batch * tiles_p * tiles_q
        seen = [place(t, batch, tiles_p, tiles_q, lists) for t in range(n)]
        assert sorted(seen) == [(b, p, q) for b in range(batch) for p in range(tiles_p) for q in range(tiles_q)]
        if lists:
            assert seen == [_listed(t, batch, tiles_p, tiles_q) for t in range(n)]


def test_tiles_of_the_largest_launches(place):
    """Up to the 2^29 tiles that lists are used for; diagonals beyond, in 32 bits and from 2^31 tiles on in 64."""
    for tiles_p, tiles_q in [(1, (1 << 29) - 1), ((1 << 29) - 1, 1), (3, (1 << 29) // 3), (5, (1 << 29) // 5), (1 << 14, (1 << 15) - 1)]:
        n = tiles_p * tiles_q
        for t in [*range(16), *range(n // 2, n // 2 + 16), *range(n - 16, n)]:
            assert place(t, 1, tiles_p, tiles_q, 1) == _listed(t, 1, tiles_p, tiles_q), (tiles_p, tiles_q, t)
    for batch, tiles_p, tiles_q in [(1, 1, 1 << 30), (1, 1, (1 << 31) - 1), (1, (1 << 31) - 1, 1), (1, 3, 1 << 29), (3, 1 << 15, 1 << 14), (1, 3, 1 << 30), (1 << 31, 2, 3)]:
        n = batch * tiles_p * tiles_q
        for t in [0, 1, 7, n // 3, n // 2 + 1, n - 2, n - 1]:
            b, r = divmod(t, tiles_p * tiles_q)
            q, p = divmod(r, tiles_p)
            assert place(t, batch, tiles_p, tiles_q, 0) == (b, (p + q) % tiles_p, q), (batch, tiles_p, tiles_q, t)


def test_lists_end_before_their_indices_do():
    """One tile row of 2^29 half tiles, and one tile less: the order is an argument of a single-shape module."""
    from paper_2103_05288_amd import Context
    ctx = Context(-1)
    for cols, lists in (((1 << 29) - 1, 1), (1 << 29, 0), ((1 << 30), 0)):
        assert f"A.aux0 = {lists}LL;" in ctx.register_static(pure_transpose("bf16", (1, 0)), [64 * cols, 1]).source, cols
    ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f32", "bool"])
def test_copies(dtype):
    """Operand rows off and on whole lines (lists and diagonals), every number of tiles mod 8, one to six tile rows, and
    every tile row count of the last band; batches whose tiles do not start on a multiple of 8; more tiles than were walked by
    a resident grid.  Copies: exact."""
    from paper_2103_05288_amd import Context
    ctx = Context(0)
    try:
        shapes = [([q, p], (1, 0)) for q in (1, 65, 513, 1100) for p in (1, 129, 300, 400, 513, 700, 1281)]
        shapes += [([64 * k + 3, 128 * k], (1, 0)) for k in (1, 3, 7)] + [([4100, 5001], (1, 0)), ([130, 70000], (1, 0)), ([70001, 257], (1, 0))]
        shapes += [([b, 130, 515], (0, 2, 1)) for b in (2, 3, 7)] + [([1000, 3, 65], (0, 2, 1))]
        for dims, perm in shapes:
            h = ctx.register(pure_transpose(dtype, perm))
            n = 1
            for d in dims:
                n *= d
            x = torch.arange(n, device="cuda") * 40503
            x = (x % 2).to(torch.uint8) if dtype == "bool" else x.to(torch.int32).view(torch.float32) if dtype == "f32" else \
                (x % 65536).to(torch.uint16).view(TORCH_DTYPE[dtype])
            x = x.reshape(dims)
            raw = {"bool": torch.uint8, "f32": torch.int32, "bf16": torch.int16}[dtype]
            want = x.view(raw).permute(perm).contiguous()
            out = torch.full((n + 32,), 5, dtype=raw, device="cuda")
            h.launch(dims, [x], [out[16:n + 16].view(x.dtype).reshape(want.shape)])
            torch.cuda.synchronize()
            assert torch.equal(out[16:n + 16], want.reshape(-1)), (dtype, dims)
            assert bool((out[:16] == 5).all()) and bool((out[n + 16:] == 5).all()), (dtype, dims)
    finally:
        ctx.close()


def _softmax_graph(ctx):
    from tests.test_transposed_rows import softmax
    return ctx.register_graph(softmax("bf16"))


def test_one_strip_of_long_rows_for_most_cus():
    """Rows beyond 4096 elements: one kernel where strips of 16 give between two thirds of the CUs and all of them one."""
    from paper_2103_05288_amd import Context
    ctx = Context(-1)
    g = _softmax_graph(ctx)
    for cols, one in ((16 * 170, False), (16 * 171, True), (3000, True), (16 * 255, True), (16 * 255 + 1, True), (4096, True), (4097, False)):
        assert ("k_row_xpose" in g.plan([6000, cols], 1)["kernels"][0]) == one, cols
    ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("dims", [[4097, 2737], [6000, 3001], [8192, 4080], [4500, 4096]])
def test_one_strip_of_long_rows_matches_oracle(dims):
    from paper_2103_05288_amd import Context
    from tests.test_transposed_rows import check, softmax
    ctx = Context(0)
    check(ctx, _softmax_graph(ctx), softmax("bf16"), dims, 1, 7)
    ctx.close()
