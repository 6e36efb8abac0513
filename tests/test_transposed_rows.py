"""Row reduces whose operand arrives transposed: an op graph launches them as one kernel where that is faster, as a tile
transpose and a row kernel elsewhere.  Both routes against the oracle, and which one a call takes."""
import pytest
import torch

from workloads import PatternBuilder
from workloads.configs import TORCH_DTYPE


def softmax(dtype, rank3=False):
    pb = PatternBuilder("transposed_softmax_" + dtype)
    dims = pb.dims(3 if rank3 else 2)
    P, Q = dims[-2:]
    lead = list(dims[:-2])
    shape, axes = lead + [Q, P], list(range(len(dims) - 1))
    perm = (0, 2, 1) if rank3 else (1, 0)
    x = pb.transpose(pb.param(dtype, lead + [P, Q]), perm)
    x = x if dtype == "f32" else pb.cast(x, "f32")
    last = len(shape) - 1
    m = pb.reduce("max", x, last)
    e = pb.op("exp", pb.op("sub", x, pb.broadcast(m, shape, axes)))
    y = pb.op("div", e, pb.broadcast(pb.reduce("sum", e, last), shape, axes))
    pb.output(y if dtype == "f32" else pb.cast(y, dtype))
    pb.output(m)                                   # one value per row
    return pb.build()


def weighted_sums(dtype):
    """No element outputs; a row vector and a value per row beside the transposed operand."""
    pb = PatternBuilder("transposed_weighted_" + dtype)
    P, Q = pb.dims(2)
    x = pb.cast(pb.transpose(pb.param(dtype, [P, Q]), (1, 0)), "f32")
    w = pb.param("f32", [P])
    r = pb.param("f32", [Q])
    v = pb.op("mul", pb.op("add", x, pb.broadcast(r, [Q, P], [0])), pb.broadcast(w, [Q, P], [1]))
    pb.output(pb.reduce("sum", v, 1))
    return pb.build()


def distance_to_max_i32():
    pb = PatternBuilder("transposed_i32")
    P, Q = pb.dims(2)
    x = pb.transpose(pb.param("i32", [P, Q]), (1, 0))
    m = pb.reduce("max", x, 1)
    pb.output(pb.op("sub", x, pb.broadcast(m, [Q, P], [0])))
    pb.output(pb.reduce("sum", x, 1))
    return pb.build()


def two_operands():
    """A second operand with an element per element: not one kernel."""
    pb = PatternBuilder("transposed_plus")
    P, Q = pb.dims(2)
    x = pb.op("add", pb.transpose(pb.param("f32", [P, Q]), (1, 0)), pb.param("f32", [Q, P]))
    pb.output(pb.op("sub", x, pb.broadcast(pb.reduce("max", x, 1), [Q, P], [0])))
    return pb.build()


def test_registered_again_compiles_nothing():
    """The kernels of a row reduce over a transposed operand are compiled once in a context, whatever graphs use them."""
    from paper_2103_05288_amd import Context
    c = Context(-1)
    try:
        c.register_graph(softmax("bf16"))
        before = c.stats()["compile_events"]
        assert before == 3                         # transpose, row reduce, row reduce over the transposed operand
        c.register_graph(softmax("bf16"))
        assert c.stats()["compile_events"] == before
        c.register_graph(softmax("f32"))           # another pattern
        assert c.stats()["compile_events"] == before + 3
        c.register_graph(softmax("f32"))
        c.register_graph(softmax("bf16"))
        assert c.stats()["compile_events"] == before + 3
    finally:
        c.close()


def test_which_calls_take_one_kernel():
    """By the plan: all eight versions are reached; very short rows in great number, and launches of 2^32 threads and more
    (which the device refuses), take two kernels."""
    from paper_2103_05288_amd import Context
    c = Context(-1)
    try:
        g = c.register_graph(softmax("bf16"))
        seen = set()
        for dims in ([8, 15], [64 * 8 * 4, 8], [64 * 8 * 4 + 1, 13], [64 * 8 * 8, 16], [32 * 8 * 12, 7201], [32 * 8 * 12 - 1, 7201],
                     [64 * 8 * 12 + 8, 6145], [64 * 8 * 12 + 3, 6145], [40, 200000], [5, 65537], [3, 40000]):
            first, second = g.plan(dims, 0), g.plan(dims, 1)
            assert first["n_launches"] == 0 and second["n_launches"] == 1, dims
            assert second["grid"][0][0] * second["block"][0][0] < 1 << 32
            seen.add(second["kernels"][0].split("_k_row_xpose_")[1])
        assert seen == {"nv%d%s" % (n, e) for n in (4, 8, 12, 16) for e in ("", "_e")}
        for dims in ([3, 200000], [1, 154872], [8, 200000], [7, 7], [64 * 8 * 8 + 1, 16], [3527, 65]):
            first, second = g.plan(dims, 0), g.plan(dims, 1)
            assert first["n_launches"] == 1 and "k_transpose_tile" in first["kernels"][0] and second["n_launches"] == 1, dims
            assert "k_row_xpose" not in second["kernels"][0]
        g = c.register_graph(softmax("bf16", rank3=True))
        for dims in ([500, 2, 64], [4000, 2, 1500], [8252, 2, 908], [500, 24, 1500], [1 << 20, 33, 256]):
            assert g.plan(dims, 0)["n_launches"] == 1 and "k_row_xpose" not in g.plan(dims, 1)["kernels"][0], dims
        for dims in ([500, 50, 300], [16, 12, 1500], [1 << 20, 33, 224]):
            p = g.plan(dims, 1)
            assert g.plan(dims, 0)["n_launches"] == 0 and p["grid"][0][0] * p["block"][0][0] < 1 << 32, dims
    finally:
        c.close()


def test_a_failing_compile_of_the_one_kernel_leaves_two(tmp_path):
    """The module of the fused kernel is an option: where it cannot be compiled the graph is registered all the same."""
    import os
    import struct
    import subprocess
    from paper_2103_05288_amd.binding import lib_path, marshal_pattern
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    exe, path = tmp_path / "optional_compile_fails", tmp_path / "graph"
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(root, "include"),
                    "-o", str(exe), os.path.join(root, "tests", "cpp", "optional_compile_fails.cpp"), lib_path(), "-L/opt/rocm/lib", "-lhiprtc",
                    "-ldl", "-Wl,-rpath," + os.path.dirname(lib_path()), "-Wl,-rpath,/opt/rocm/lib"], check=True)
    pat = softmax("bf16")
    ops, n_ops, cs, n_cs = marshal_pattern(pat)
    path.write_bytes(struct.pack("<iii", n_ops, n_cs, pat.n_dims) + bytes(ops) + (bytes(cs)[: n_cs * 20] if n_cs else b""))
    r = subprocess.run([str(exe), str(path)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stderr)
    assert r.stdout.strip() == "compiles=3 failed=1 again=0"


@pytest.fixture(scope="module")
def ctx():
    from paper_2103_05288_amd import Context
    c = Context(0)
    yield c
    c.close()


def run(ctx, g, pat, dims, ins, off=0):
    """-> (outputs, device launches); off: elements the first operand lies past a 256-byte boundary"""
    dev = [t.cuda() for t in ins]
    if off:
        buf = torch.empty(dev[0].numel() + off, dtype=dev[0].dtype, device="cuda")
        buf[off:].copy_(dev[0].reshape(-1))
        dev[0] = buf[off:].view(dev[0].shape)
    outs = [torch.zeros(pat.shape_of(i, dims), dtype=TORCH_DTYPE[pat.ops[i].dtype], device="cuda") for i in pat.outputs]
    for o in outs:
        o.fill_(float("nan") if o.dtype.is_floating_point else -7)
    before = ctx.stats()["device_launches"]
    g.launch(dims, dev, outs, workspace=torch.empty(max(16, g.workspace_bytes(dims)), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    return outs, ctx.stats()["device_launches"] - before


def check(ctx, g, pat, dims, launches, seed, off=0, positive=False):
    from oracle import run as oracle_run
    from tests.util import assert_close, to_oracle_input
    gen = torch.Generator().manual_seed(seed)
    ins = [torch.randn(pat.shape_of(i, dims), generator=gen).to(TORCH_DTYPE[pat.ops[i].dtype]) for i in pat.params]
    if positive:      # (sums of n fp32 terms err by up to n 2^-24 sum |term|, which the bar measures against the sum: one sign)
        ins = [t.abs() for t in ins]
    outs, n = run(ctx, g, pat, dims, ins, off)
    assert n == launches, (dims, n)
    want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0]
    for k, (o, w) in enumerate(zip(outs, want)):
        assert_close(o.cpu(), w, f"{pat.name if hasattr(pat, 'name') else ''} {dims} out{k}")


# columns of the operand (rows of the result) around the strips of 8, 16 and 32; rows of the operand around the slots of
# a lane, the slots that a kernel holds (4, 8, 12, 16 of 64, 32 or 16 lanes) and the line to two kernels
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_strips_and_row_lengths(ctx, dtype):
    pat = softmax(dtype)
    g = ctx.register_graph(pat)
    V = 4 if dtype == "f32" else 8
    odd = 1 if dtype == "f32" else 2               # few long rows off dword boundaries
    for i, (p, q, n) in enumerate([(1, 8, 1), (3, 9, 1), (7, 7, 2), (8, 1, 2), (8, 15, 1), (9, 17, 1), (64 * V, 31, 1), (64 * V + 1, 33, 1),
                                   (64 * V * 4, 8, 1), (64 * V * 4 + 1, 13, 1), (64 * V * 8 - 1, 22, 1), (64 * V * 8 - 1, 21, odd), (64 * V * 8, 16, 1), (64 * V * 5 + 3, 513, 1),
                                   (64 * V * 8 + 1, 16, 2), (64 * V * 16 + 1, 40, 2), (37, 7168, 1), (16 * V + 5, 32801, 1), (5, 65537, 1),
                                   (16 * V * 12, 32800, 1), (16 * V * 12 + 1, 32800, 1), (32 * V * 12, 7201, 1), (32 * V * 12 + 3, 7169, 1),
                                   (64 * V * 8 + 3, 6145, 1), (64 * V * 12 + 8, 6145, 1), (64 * V * 12, 6144 - 16, 2)]):
        if dtype == "bf16" or p * q <= 1 << 23:     # (the largest ones once)
            check(ctx, g, pat, [p, q], n, i)
    for off in (1, 3, 8):                           # bases off every boundary of an access
        check(ctx, g, pat, [100, 77], 1, 90 + off, off)
        check(ctx, g, pat, [301, 8], 1, 90 + off, off)


@pytest.mark.gpu
def test_batches_row_vectors_and_what_stays_two_kernels(ctx):
    pat = softmax("bf16", rank3=True)
    g = ctx.register_graph(pat)
    for i, (b, p, q) in enumerate([(1, 30, 40), (5, 64, 19), (33, 9, 8), (7, 513, 257), (300, 100, 33), (1100, 40, 129)]):
        check(ctx, g, pat, [b, p, q], 1, 20 + i)
    check(ctx, g, pat, [4, 50, 5], 2, 30)           # fewer rows than a strip
    check(ctx, g, pat, [2, 5000, 40], 2, 31)        # long rows, few strips
    for dtype in ("bf16", "f16"):
        pat = weighted_sums(dtype)
        g = ctx.register_graph(pat)
        for i, (p, q) in enumerate([(8, 8), (63, 100), (2050, 31), (4096, 10), (515, 7300)]):
            check(ctx, g, pat, [p, q], 1, 40 + i, positive=True)
    pat = distance_to_max_i32()
    g = ctx.register_graph(pat)
    for p, q in ((1, 8), (50, 33), (257, 100), (2048, 17), (1025, 9)):
        x = torch.randint(-1000, 1000, (p, q), dtype=torch.int32, generator=torch.Generator().manual_seed(p))
        outs, n = run(ctx, g, pat, [p, q], [x])
        t = x.t()
        assert n == 1 and torch.equal(outs[0].cpu(), t - t.max(1, keepdim=True)[0]) and torch.equal(outs[1].cpu(), t.sum(1, dtype=torch.int32))
    pat = two_operands()
    check(ctx, ctx.register_graph(pat), pat, [60, 70], 2, 50)


@pytest.mark.gpu
@pytest.mark.parametrize("p, q", [(1014, 49800), (4096, 8000), (2400, 6000)])
def test_sums_are_no_further_off_than_the_row_kernels(ctx, p, q):
    """Sums of squares (of one sign) against the same sums of the transposed tensor through the row kernels."""
    def build(transposed):
        pb = PatternBuilder("squares")
        P, Q = pb.dims(2)
        x = pb.param("bf16", [P, Q] if transposed else [Q, P])
        x = pb.cast(pb.transpose(x, (1, 0)) if transposed else x, "f32")
        pb.output(pb.reduce("sum", pb.op("mul", x, x), 1))
        return pb.build()
    one, rows = build(True), build(False)
    x = torch.randn(p, q, generator=torch.Generator().manual_seed(p)).bfloat16()
    outs, n = run(ctx, ctx.register_graph(one), one, [p, q], [x])
    assert n == 1
    h = ctx.register(rows)
    ref, dims = torch.empty(q, device="cuda"), [0, 0]
    dims[rows.ops[rows.params[0]].dims[0]], dims[rows.ops[rows.params[0]].dims[1]] = q, p
    h.launch(dims, [x.cuda().t().contiguous()], [ref])
    torch.cuda.synchronize()
    want = (x.cuda().double() ** 2).sum(0)
    off = lambda v: float((v.double() - want).norm() / want.norm())
    assert off(outs[0]) <= 1.05 * off(ref), (off(outs[0]), off(ref))


@pytest.mark.gpu
def test_result_over_its_operand_and_forced_versions(ctx):
    """Through two kernels the operand is read before anything is written; a call that relies on it still goes that way."""
    from oracle import run as oracle_run
    from paper_2103_05288_amd import DiscError, VARIANTS
    from tests.util import assert_close, to_oracle_input
    pat = softmax("bf16")
    g = ctx.register_graph(pat)
    x = torch.randn(96, 96, generator=torch.Generator().manual_seed(1)).bfloat16()
    buf, m = x.cuda(), torch.empty(96, dtype=torch.float32, device="cuda")
    ws = torch.empty(g.workspace_bytes([96, 96]), dtype=torch.uint8, device="cuda")
    before = ctx.stats()["device_launches"]
    g.launch([96, 96], [buf], [buf, m], workspace=ws)
    torch.cuda.synchronize()
    assert ctx.stats()["device_launches"] == before + 2
    want = oracle_run(pat, [96, 96], [to_oracle_input(x)])[0]
    assert_close(buf.cpu(), want[0], "in place")
    ctx.force_variant(VARIANTS.index("row_reg_vec"))
    try:
        with pytest.raises(DiscError):              # (the transpose has no such version)
            g.launch([96, 96], [buf], [torch.empty_like(buf), m], workspace=ws)
    finally:
        ctx.force_variant(-1)


@pytest.mark.gpu
def test_captured_and_replayed(ctx):
    pat = softmax("bf16")
    g = ctx.register_graph(pat)
    dims = [700, 300]
    x = torch.randn(dims, device="cuda").bfloat16()
    out, m = torch.empty(300, 700, dtype=torch.bfloat16, device="cuda"), torch.empty(300, device="cuda")
    ws = torch.empty(g.workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        g.launch(dims, [x], [out, m], workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.launch(dims, [x], [out, m], workspace=ws)
    for k in range(3):
        x.copy_(torch.randn(dims, device="cuda").bfloat16())
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        g.launch(dims, [x], [out, m], workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(got, out), k
