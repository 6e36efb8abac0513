"""The order in which tile transposes take their tiles: lists of neighbouring tiles for every XCD, or diagonals."""
import pytest
import torch

from tests.test_transpose import pure_transpose
from workloads.configs import TORCH_DTYPE


def _place(t, batch, tiles_p, tiles_q, near=4):
    """The tile that block t takes from the lists."""
    per_batch = tiles_p * tiles_q
    n, x = batch * per_batch, t % 8
    k = x * (n // 8) + min(x, n % 8) + t // 8
    b, r = divmod(k, per_batch)
    g, i = divmod(r, near * tiles_q)
    w = min(near, tiles_p - g * near)
    return b, g * near + i % w, i // w


def test_lists_hold_every_tile_once():
    for batch, tiles_p, tiles_q in [(1, 1, 1), (1, 5, 3), (3, 4, 7), (2, 3, 3), (1, 33, 94), (7, 1, 1), (1, 9, 1), (5, 2, 11)]:
        n = batch * tiles_p * tiles_q
        seen = {_place(t, batch, tiles_p, tiles_q) for t in range(n)}
        assert seen == {(b, p, q) for b in range(batch) for p in range(tiles_p) for q in range(tiles_q)}


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
    for cols, one in ((16 * 170, False), (16 * 171, True), (3000, True), (16 * 255, True), (16 * 255 + 1, False), (4097, False)):
        assert ("k_row_xpose" in g.plan([6000, cols], 1)["kernels"][0]) == one, cols
    ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("dims", [[4097, 2737], [6000, 3001], [8192, 4080]])
def test_one_strip_of_long_rows_matches_oracle(dims):
    from paper_2103_05288_amd import Context
    from tests.test_transposed_rows import check, softmax
    ctx = Context(0)
    check(ctx, _softmax_graph(ctx), softmax("bf16"), dims, 1, 7)
    ctx.close()
