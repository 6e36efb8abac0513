"""Compaction in one pass: which calls take it (host), and its results at the edges of its tiles and iterations on the GPU,
with counts of other blocks awaited and with every one that is not there yet counted by the block that misses it."""
import pytest
import torch

from tests.test_compact_gpu import check, filtered, unique_sorted
from tests.util import run_gpu
from workloads import PatternBuilder


def _kernels(plan):
    return [k.split("_k_compact_")[1] for k in plan["kernels"]]


def test_which_calls_take_one_pass():
    from paper_2103_05288_amd import VARIANTS, Context
    ctx = Context(-1)
    h = ctx.register(unique_sorted("i32"))
    line = (64 << 20) // 12                                   # input, values and ranks of 4 bytes an element
    assert _kernels(h.plan([line - 8])) == ["count_vec", "scatter_vec"]
    p = h.plan([line + 8])
    assert _kernels(p) == ["clear", "chain_vec"] and p["n_launches"] == 2
    tiles = -(-(line + 8) // 4096)
    assert p["workspace_bytes"] == max(4 * tiles, 1024 * 16) and p["grid"][1][0] == 1024 and p["grid"][0][0] == -(-tiles // 256)
    assert _kernels(h.plan([1 << 25], VARIANTS.index("compact_scalar"))) == ["count_scalar", "scatter_scalar"]
    ctx.test_option("non_temporal", 0)                        # its stores are: without them two launches
    assert _kernels(h.plan([1 << 25])) == ["count_vec", "scatter_vec"]
    ctx.test_option("non_temporal", -1)
    # kept values that take more LDS than four blocks a CU have
    assert _kernels(ctx.register(filtered()).plan([1 << 25])) == ["count_vec", "scatter_vec_nt"]
    # tests: from the line of two launches on, not below it
    ctx.test_option("compact_looks", 3)
    assert _kernels(h.plan([32 * 4096])) == ["clear", "chain_vec"] and len(_kernels(h.plan([31 * 4096]))) == 3
    ctx.close()


def _one_output(dtype):
    """keep = x > thr: the kept x alone, with the count"""
    pb = PatternBuilder("one_output")
    n = pb.dim()
    x = pb.param(dtype, [n])
    keep = pb.op("gt", pb.cast(x, "f32"), pb.param("f32", []), dims=[n])
    pb.output(pb.compact(x, keep))
    pb.output(pb.compact_count(keep, "i32"))
    return pb.build()


@pytest.mark.parametrize("dtype", ["i32", "i64"])
def test_the_workspace_of_the_most_elements_serves_fewer(dtype):
    from paper_2103_05288_amd import Context
    ctx = Context(-1)
    h = ctx.register(unique_sorted(dtype))
    sizes = [h.plan([int(2 ** (k / 8))])["workspace_bytes"] for k in range(80, 208)]
    assert sizes == sorted(sizes)
    ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("looks", [0, 500])
@pytest.mark.parametrize("what", ["i32", "i64", "f32", "bf16"])
def test_results(what, looks):
    """Whole tiles and an element more or less, blocks with one, two and three tiles (1024 blocks of four parts), a last
    tile that ends inside a slot; few and many kept.  Whole numbers and copied values: exact."""
    from paper_2103_05288_amd import Context
    ctx = Context(0)
    ctx.test_option("compact_looks", looks)
    pat = _one_output("bf16") if what == "bf16" else unique_sorted(what)
    h = ctx.register(pat)
    vec = {"i32": 4, "f32": 4, "i64": 2, "bf16": 8}[what]
    tile = 1024 * vec
    g = torch.Generator().manual_seed(17)
    for n in (32 * tile - 1, 32 * tile, 33 * tile + 1, 1024 * tile + 1, 2049 * tile + tile // 2 + 3 * vec + 1):
        assert _kernels(h.plan([n])) == ["clear", "chain_vec"]
        print(f"[one pass] {what} looks={looks} n={n}", flush=True)
        if what == "bf16":
            if n > 40 * tile:
                n = 1025 * tile + 77 if looks else 1024 * tile + 1
            x = torch.round(torch.randn(n, generator=g) * 4).to(torch.bfloat16)
            for thr in (-1e9, 1e9, 2.0):
                check(ctx, pat, [n], [x, torch.tensor(thr)], f"{what} thr={thr}")
        else:
            for spread in (2, 3 * n):
                x = torch.sort(torch.randint(-spread, spread + 1, (n,), generator=g, dtype=torch.int64)).values
                x = x * 3000000007 if what == "i64" else x.to(torch.int32) if what == "i32" else (x % (1 << 24)).sort().values.to(torch.float32)
                check(ctx, pat, [n], [x], f"{what} spread={spread}")
    ctx.close()


@pytest.mark.gpu
def test_captured_and_replayed():
    """The cells are cleared by the call itself: replays with other inputs, and eager calls on the same workspace between them."""
    from paper_2103_05288_amd import Context
    ctx = Context(0)
    pat = unique_sorted("i32")
    h = ctx.register(pat)
    n = 6000007
    g = torch.Generator().manual_seed(5)
    xs = [torch.sort(torch.randint(0, k, (n,), generator=g, dtype=torch.int32)).values for k in (1000, 10 ** 6, 10 ** 8)]
    want = [run_gpu(h, pat, [n], [x]) for x in xs]
    assert _kernels(h.plan([n])) == ["clear", "chain_vec"]
    x = xs[0].cuda()
    outs = [torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda"),
            torch.empty(1, dtype=torch.int64, device="cuda")]
    ws = torch.empty(ctx.workspace_bytes(h.id, [n]), dtype=torch.uint8, device="cuda")
    h.launch([n], [x], outs, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        h.launch([n], [x], outs, workspace=ws)
    for k in (1, 2, 0, 1):
        x.copy_(xs[k])
        for t in outs:
            t.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        m = int(outs[2][0])
        assert m == int(want[k][2].reshape(-1)[0]) and torch.equal(outs[1].cpu(), want[k][1])
        assert torch.equal(outs[0][:m].cpu(), want[k][0][:m]) and bool((outs[0][m:] == -7).all())
        h.launch([n], [x], outs, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(outs[1].cpu(), want[k][1])
    ctx.close()


def _wide_values(pred, value, outputs=1):
    """keep = x > thr for a narrow x; kept: operands of a wider type"""
    pb = PatternBuilder("wide_values")
    n = pb.dim()
    x = pb.param(pred, [n])
    values = [pb.param(value, [n]) for _ in range(outputs)]
    keep = pb.op("gt", pb.cast(x, "f32"), pb.param("f32", []), dims=[n])
    for v in values:
        pb.output(pb.compact(v, keep))
    pb.output(pb.compact_rank(keep, "i32"))
    pb.output(pb.compact_count(keep, "i32"))
    return pb.build()


def test_kept_values_take_8_kb_of_a_wavefront():
    """All four slots of a lane leave together, or as many as that holds."""
    from paper_2103_05288_amd import Context
    ctx = Context(-1)
    for pat, slots in ((unique_sorted("i32"), 4), (unique_sorted("i64"), 4), (filtered(), 4), (_wide_values("bf16", "i64"), 2)):
        assert f"COMPACT_STRETCH = {slots};" in ctx.register(pat).source
    ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("outputs", [1, 2])
def test_wide_values_of_narrow_operands(outputs):
    """A wavefront's kept values in two stretches: tiles of 8192 elements, whole ones and one element more or less, one slot and
    one stretch of a last part; none, some and all kept.  Copied values: exact."""
    from paper_2103_05288_amd import Context
    ctx = Context(0)
    pat = _wide_values("bf16", "i64", outputs)
    g = torch.Generator().manual_seed(23)
    for n in (1, 511, 513, 1025, 8191, 8193, 32 * 8192 - 1, 33 * 8192 + 1025, 260 * 8192 + 1537):
        x = torch.round(torch.randn(n, generator=g) * 4).to(torch.bfloat16)
        values = [torch.randint(-2 ** 62, 2 ** 62, (n,), generator=g) for _ in range(outputs)]
        for thr in (-1e9, 1e9, 2.0):
            print(f"[wide values] n={n} thr={thr}", flush=True)
            check(ctx, pat, [n], [x, *values, torch.tensor(thr)], f"n={n} thr={thr}")
    ctx.close()


@pytest.mark.gpu
def test_counting_for_others_is_shared():
    """Every cell that is not there at once counted by who misses it, as if its block were never resident: wavefronts take different
    cells and find what the others have counted.  At most three times the call's ordinary time (1.6 times; 5.6 where every block
    counted all of them)."""
    from paper_2103_05288_amd import Context
    ctx = Context(0)
    pat = unique_sorted("i32")
    h = ctx.register(pat)
    n = 33555445
    g = torch.Generator(device="cuda").manual_seed(29)
    x = torch.sort(torch.randint(0, n // 4, (n,), generator=g, device="cuda", dtype=torch.int32)).values
    outs = [torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(1, dtype=torch.int64, device="cuda")]
    ws = torch.empty(ctx.workspace_bytes(h.id, [n]), dtype=torch.uint8, device="cuda")
    best, results = {}, {}
    for looks in (500, 0, 500, 0):
        ctx.test_option("compact_looks", looks)
        call = h.bind([n], [x], outs, workspace=ws)
        for _ in range(4):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(5):
                call()
            end.record()
            torch.cuda.synchronize()
            best[looks] = min(best.get(looks, 1e9), start.elapsed_time(end))
        results[looks] = [outs[0][:int(outs[2][0])].clone(), outs[1].clone(), outs[2].clone()]
    assert all(torch.equal(a, b) for a, b in zip(results[0], results[500]))
    assert best[0] < 3 * best[500], best
    ctx.close()
