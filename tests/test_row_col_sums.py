"""Sums over the rows fused into a row-reduce pattern (the weight gradients of a normalisation next
to its input gradient, Section 4.3's input fusion with both reduction kinds in one kernel): the
checker's acceptance rule, the launch plan, and parity with the oracle through the C ABI."""
import numpy as np
import pytest
import torch

from workloads.configs import TORCH_DTYPE
from workloads.extras import gelu_backward_bias_gradient, layernorm_backward_graph, logsumexp_with_total_and_amax
from workloads.pattern import PatternBuilder


@pytest.fixture(scope="module")
def hctx():
    from paper_2103_05288_amd import Context
    c = Context(device=-1)
    yield c
    c.close()


def softmax_backward_with_bias_gradient():
    """dx of a row softmax (one row reduction) and the column sum of dx's upstream gradient."""
    pb = PatternBuilder("softmax_bwd_bias")
    t, h = pb.dims(2)
    y = pb.cast(pb.param("bf16", [t, h]), "f32")
    dy = pb.cast(pb.param("bf16", [t, h]), "f32")
    dot = pb.reduce("sum", pb.op("mul", dy, y), 1)
    dx = pb.op("mul", y, pb.op("sub", dy, pb.broadcast(dot, [t, h], [0])))
    pb.output(pb.cast(dx, "bf16"))
    pb.output(pb.reduce("sum", dx, 0))
    return pb.build()


def test_one_pattern_two_launches(hctx):
    pat = layernorm_backward_graph()
    h = hctx.register(pat)
    assert h.info["template"] == "row_reduce" and h.info["n_phases"] == 3 and h.info["n_outputs"] == 3
    pl = h.plan([4096, 1024])
    assert pl["n_launches"] == 2 and pl["kernels"][0].split("k_row_")[1].startswith("vec_nv2") and pl["kernels"][1].endswith("k_colsum_finish")
    # one row of fp32 partial sums per block and summed output
    assert pl["workspace_bytes"] == pl["grid"][0][0] * 1024 * 4 * 2
    assert pl["grid"][1][0] == 1024 // 16 and pl["block"][1][0] == 256
    # rows too long for registers: the streaming version keeps the partial sums in the workspace
    pl = h.plan([100, 30000])
    assert pl["kernels"][0].endswith("k_row_stream_vec") and pl["workspace_bytes"] == 100 * 30000 * 4 * 2
    # wide blocks (one lane group per block): still one row of partial sums per block
    pl = h.plan([3000, 8192])
    assert pl["block"][0][0] == 512 and pl["workspace_bytes"] == pl["grid"][0][0] * 8192 * 4 * 2
    # the graph front end now keeps the whole backward pass in this one pattern
    g = hctx.register_graph(pat)
    assert g.info["n_patterns"] == 1 and g.info["n_intermediates"] == 0
    # a sum over zero rows has no value
    from paper_2103_05288_amd import DiscError
    with pytest.raises(DiscError) as e:
        h.plan([0, 64])
    assert "size 0" in str(e.value)


def test_acceptance_rule(hctx):
    from paper_2103_05288_amd import DiscError

    def build(kind="sum", consume=False, rank3=False, integer=False):
        pb = PatternBuilder("rule")
        if rank3:
            b, t, h = pb.dims(3)
            shape, rows_axes = [b, t, h], [0, 1]
        else:
            t, h = pb.dims(2)
            shape, rows_axes = [t, h], [0]
        x = pb.param("i32" if integer else "f32", shape)
        m = pb.reduce("max", x, len(shape) - 1)
        d = pb.op("sub", x, pb.broadcast(m, shape, rows_axes))
        pb.output(d)
        s = pb.reduce(kind, d, 0)
        if consume:
            s = pb.op("neg", s)
        pb.output(s)
        return pb.build()

    assert hctx.register(build()).info["template"] == "row_reduce"
    for kw, word in ((dict(kind="max"), "floating-point sum"), (dict(consume=True), "outputs alone"),
                     (dict(rank3=True), "two-dimensional"), (dict(integer=True), "floating-point sum")):
        with pytest.raises(DiscError) as e:
            hctx.register(build(**kw))
        assert e.value.status == "UNFUSIBLE" and word in str(e.value), (kw, str(e.value))


def test_sum_over_rows_beside_a_loop_fusion(hctx):
    """No row reduction at all: an element-wise backward with its bias gradient runs in the row
    template without reduction phases (operands read once); a pattern whose element-wise output
    needs the column sum keeps the column-reduce template."""
    h = hctx.register(gelu_backward_bias_gradient())
    assert h.info["template"] == "row_reduce" and h.info["n_phases"] == 0 and h.info["n_outputs"] == 2
    pl = h.plan([4096, 1024])
    assert pl["n_launches"] == 2 and pl["kernels"][1].endswith("k_colsum_finish")
    assert pl["workspace_bytes"] == pl["grid"][0][0] * 1024 * 4
    assert h.plan([5, 0])["n_launches"] == 0           # nothing to compute, and no reduction over an empty axis
    pb = PatternBuilder("centre")
    t, hh = pb.dims(2)
    x = pb.param("f32", [t, hh])
    m = pb.op("div", pb.reduce("sum", x, 0), pb.dim_size(t))
    pb.output(pb.op("sub", x, pb.broadcast(m, [t, hh], [1])))
    assert hctx.register(pb.build()).info["template"] == "col_reduce"
    # a column sum alone (no full-shape output) also stays a column reduce: more parallel over the rows
    pb = PatternBuilder("bias_grad_alone")
    t, hh = pb.dims(2)
    pb.output(pb.reduce("sum", pb.op("tanh", pb.param("f32", [t, hh])), 0))
    assert hctx.register(pb.build()).info["template"] == "col_reduce"


def test_per_row_values_reduced_over_the_rows(hctx):
    """Rank-0 outputs: a sum / maximum / minimum of per-row values over the rows rides along in the
    row kernels (one partial result per block, a last one-block launch)."""
    from paper_2103_05288_amd import DiscError
    pat = logsumexp_with_total_and_amax()
    h = hctx.register(pat)
    assert h.info["template"] == "row_reduce" and h.info["n_phases"] == 2 and h.info["n_outputs"] == 3
    pl = h.plan([4096, 1024])
    assert pl["n_launches"] == 2 and pl["kernels"][1].endswith("k_rowred_finish") and pl["grid"][1] == [1, 1, 1]
    assert pl["workspace_bytes"] == 2 * pl["grid"][0][0] * 4
    assert h.plan([100, 30000])["kernels"][0].endswith("k_row_stream_vec")
    with pytest.raises(DiscError) as e:
        h.plan([0, 64])
    assert e.value.status == "EMPTY_REDUCE"
    assert pat.shape_of(pat.outputs[1], [7, 5]) == ()
    # with sums over the rows of full-size values in the same pattern: three launches
    pb = PatternBuilder("both")
    t, hh = pb.dims(2)
    x = pb.param("f32", [t, hh])
    m = pb.reduce("max", x, 1)
    d = pb.op("sub", x, pb.broadcast(m, [t, hh], [0]))
    pb.output(d)
    pb.output(pb.reduce("sum", d, 0))
    pb.output(pb.reduce("min", m, 0))
    hb = hctx.register(pb.build())
    pl = hb.plan([4096, 1024])
    assert [k.split("_k_")[1] for k in pl["kernels"]][1:] == ["colsum_finish", "rowred_finish"]
    assert pl["workspace_bytes"] == (pl["grid"][0][0] * 1024 * 4 + 255) // 256 * 256 + pl["grid"][0][0] * 4
    # what is not fused: a rank-0 result of anything else
    for build in ("prod_like_argmax", "consumed", "column_vector", "no_row_reduce"):
        pb = PatternBuilder(build)
        t, hh = pb.dims(2)
        x = pb.param("f32", [t, hh])
        m = pb.reduce("max", x, 1)
        pb.output(pb.op("sub", x, pb.broadcast(m, [t, hh], [0])))
        if build == "prod_like_argmax":
            pb.output(pb.reduce("argmax", m, 0))
        elif build == "consumed":
            s = pb.reduce("sum", m, 0)
            pb.output(pb.op("sub", m, pb.broadcast(s, [t], [])))
        elif build == "column_vector":
            pb.output(pb.reduce("sum", pb.reduce("sum", x, 0), 0))
        else:
            pb = PatternBuilder(build)
            t = pb.dim()
            pb.output(pb.reduce("sum", pb.param("f32", [t]), 0))
        with pytest.raises(DiscError) as e:
            hctx.register(pb.build())
        assert e.value.status in ("UNFUSIBLE", "BAD_PATTERN"), (build, str(e.value))


def _inputs(pat, dims, gen):
    ins = []
    for pi in pat.params:
        shp = pat.shape_of(pi, dims)
        ins.append(torch.randn(shp, generator=gen).to(TORCH_DTYPE[pat.ops[pi].dtype]))
    return ins


def _check_sum(got, want, terms_abs, rows_per_block, what):
    """A sum of T terms of mixed sign cannot meet a bar relative to the (cancelled) result.  Each
    term carries at most 8 fp32 roundings from the element-wise arithmetic; a lane then adds the
    terms of its block's rows in fp32 (rows_per_block additions), the lane groups of a block meet in
    at most 8 more fp32 additions, and the partial rows are added in fp64:
    |err| <= (16 + rows_per_block) * 2^-24 * sum_t |term_t| + 1e-6."""
    lim = (16 + rows_per_block) * 2.0 ** -24 * terms_abs.sum(0) + 1e-6
    err = np.abs(got.double().numpy() - np.asarray(want, dtype=np.float64))
    assert (err <= lim).all(), (what, float((err / lim).max()))


LN_SHAPES = [[7, 5], [300, 1], [1000, 77], [20000, 16], [4096, 1024], [513, 2050], [1500, 1021], [300, 4100],
             [65, 8200], [40, 30000], [3, 40000]]


@pytest.mark.gpu
@pytest.mark.parametrize("dims", LN_SHAPES, ids=lambda d: f"{d[0]}x{d[1]}")
def test_layernorm_backward_single_pattern_matches_oracle(dims):
    from oracle import run as oracle_run
    from paper_2103_05288_amd import Context
    from tests.util import assert_close, run_gpu, to_oracle_input
    pat = layernorm_backward_graph()
    ctx = Context(0)
    try:
        h = ctx.register(pat)
        gen = torch.Generator().manual_seed(dims[0] * 7919 + dims[1])
        ins = _inputs(pat, dims, gen)
        pl = h.plan(dims)
        assert pl["n_launches"] == 2
        got = run_gpu(h, pat, dims, ins)
        want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0]
        assert_close(got[0], want[0], f"dx dims={dims}")
        x64, dy64 = ins[0].double().numpy(), ins[1].double().numpy()
        xc = x64 - x64.mean(1, keepdims=True)
        xhat = xc / np.sqrt((xc * xc).mean(1, keepdims=True) + 1e-5)
        rpb = -(-dims[0] // pl["grid"][0][0])
        _check_sum(got[1], want[1], np.abs(dy64 * xhat), rpb, f"dgamma dims={dims} {pl['kernels'][0]}")
        _check_sum(got[2], want[2], np.abs(dy64), rpb, f"dbeta dims={dims} {pl['kernels'][0]}")
        # the same call again on the same workspace gives the same bits (fixed summation order)
        again = run_gpu(h, pat, dims, ins)
        for a, b in zip(got, again):
            assert torch.equal(a, b)
    finally:
        ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("dims", [[508, 1000], [509, 1000], [516, 1000], [2043, 1000], [2300, 13]], ids=lambda d: f"{d[0]}x{d[1]}")
def test_adding_up_the_partial_rows(dims):
    """The second launch with whole batches of loads, with and without a last one, and numbers of partial rows that its
    lanes do not divide."""
    from paper_2103_05288_amd import Context
    ctx = Context(0)
    try:
        pl = ctx.register(layernorm_backward_graph()).plan(dims)
        assert pl["block"][1][0] == 256
    finally:
        ctx.close()
    test_layernorm_backward_single_pattern_matches_oracle(dims)


@pytest.mark.gpu
def test_forced_versions_and_one_phase_pattern():
    """Every row-kernel version carries the sums (scalar and streaming versions forced on shapes the
    host would give to the vector version), and a one-phase pattern (softmax backward) with a single
    summed output."""
    from oracle import run as oracle_run
    from paper_2103_05288_amd import Context
    from paper_2103_05288_amd.binding import VARIANTS
    from tests.util import assert_close, run_gpu, to_oracle_input
    ctx = Context(0)
    try:
        pat = layernorm_backward_graph()
        h = ctx.register(pat)
        gen = torch.Generator().manual_seed(5)
        for force in ("row_reg_vec", "row_reg_scalar", "row_stream_vec", "row_stream_scalar"):
            for dims in ([33, 768], [600, 100]):
                ins = _inputs(pat, dims, gen)
                ctx.force_variant(VARIANTS.index(force))
                try:
                    pl = h.plan(dims, force_variant=VARIANTS.index(force))
                    got = run_gpu(h, pat, dims, ins)
                finally:
                    ctx.force_variant(-1)
                want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0]
                assert_close(got[0], want[0], f"dx {force} {dims}")
                x64, dy64 = ins[0].double().numpy(), ins[1].double().numpy()
                xc = x64 - x64.mean(1, keepdims=True)
                xhat = xc / np.sqrt((xc * xc).mean(1, keepdims=True) + 1e-5)
                rpb = -(-dims[0] // pl["grid"][0][0])
                _check_sum(got[1], want[1], np.abs(dy64 * xhat), rpb, f"dgamma {force} {dims}")
                _check_sum(got[2], want[2], np.abs(dy64), rpb, f"dbeta {force} {dims}")
        pat = softmax_backward_with_bias_gradient()
        h = ctx.register(pat)
        assert h.info["template"] == "row_reduce" and h.info["n_phases"] == 1
        for dims in ([3, 7], [2000, 1000], [9, 5739], [5000, 48]):
            probs = torch.softmax(torch.randn(*dims, generator=gen), dim=1).bfloat16()
            ins = [probs, torch.randn(*dims, generator=gen).bfloat16()]
            pl = h.plan(dims)
            got = run_gpu(h, pat, dims, ins)
            want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0]
            assert_close(got[0], want[0], f"softmax backward dx {dims}")
            y64, dy64 = ins[0].double().numpy(), ins[1].double().numpy()
            dx = y64 * (dy64 - (dy64 * y64).sum(1, keepdims=True))
            _check_sum(got[1], want[1], np.abs(dx) + np.abs(y64 * dy64), -(-dims[0] // pl["grid"][0][0]), f"sum of dx {dims}")
    finally:
        ctx.close()


@pytest.mark.gpu
def test_gelu_backward_with_bias_gradient_matches_oracle():
    from oracle import run as oracle_run
    from paper_2103_05288_amd import Context
    from tests.util import assert_close, run_gpu, to_oracle_input
    pat = gelu_backward_bias_gradient()
    ctx = Context(0)
    try:
        h = ctx.register(pat)
        gen = torch.Generator().manual_seed(17)
        for dims in ([1, 1], [7, 5], [1000, 77], [20000, 16], [4096, 1024], [513, 2050], [300, 4100], [65, 8200], [40, 30000]):
            ins = _inputs(pat, dims, gen)
            pl = h.plan(dims)
            got = run_gpu(h, pat, dims, ins)
            want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0]
            assert_close(got[0], want[0], f"gelu backward dx dims={dims}")
            dy, x, b = (t.double().numpy() for t in ins)
            a = 1.702 * (x + b)
            s = 1.0 / (1.0 + np.exp(-a))
            dx = dy * s * (1.0 + a * (1.0 - s))
            _check_sum(got[1], want[1], np.abs(dx), -(-dims[0] // pl["grid"][0][0]), f"bias gradient dims={dims} {pl['kernels'][0]}")
    finally:
        ctx.close()


@pytest.mark.gpu
def test_single_shape_build_of_a_pattern_with_sums_over_rows():
    """The shape-specialised build (every extent and plan member a constant, Section 5.3's static
    counterpart) of LayerNorm backward: the number of partial-sum rows follows the grid of the
    launch, not the one planned at registration."""
    from oracle import run as oracle_run
    from paper_2103_05288_amd import Context
    from tests.util import assert_close, run_gpu, to_oracle_input
    pat = layernorm_backward_graph()
    ctx = Context(0)
    try:
        gen = torch.Generator().manual_seed(23)
        for dims in ([20000, 768], [3000, 2050]):
            ins = _inputs(pat, dims, gen)
            hs = ctx.register_static(pat, dims)
            pl = hs.plan(dims)
            got = run_gpu(hs, pat, dims, ins)
            want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0]
            assert_close(got[0], want[0], f"static dx dims={dims}")
            x64, dy64 = ins[0].double().numpy(), ins[1].double().numpy()
            xc = x64 - x64.mean(1, keepdims=True)
            xhat = xc / np.sqrt((xc * xc).mean(1, keepdims=True) + 1e-5)
            rpb = -(-dims[0] // pl["grid"][0][0])
            _check_sum(got[1], want[1], np.abs(dy64 * xhat), rpb, f"static dgamma dims={dims}")
            _check_sum(got[2], want[2], np.abs(dy64), rpb, f"static dbeta dims={dims}")
    finally:
        ctx.close()


@pytest.mark.gpu
def test_logsumexp_total_and_amax_match_oracle():
    from oracle import run as oracle_run
    from paper_2103_05288_amd import Context
    from paper_2103_05288_amd.binding import VARIANTS
    from tests.util import assert_close, run_gpu, to_oracle_input
    pat = logsumexp_with_total_and_amax()
    ctx = Context(0)
    try:
        h = ctx.register(pat)
        gen = torch.Generator().manual_seed(29)
        cases = [([1, 1], None), ([7, 5], None), ([1000, 77], None), ([20000, 16], None), ([4096, 1024], None), ([513, 2050], None),
                 ([300, 4100], None), ([65, 8200], None), ([40, 30000], None),
                 ([33, 768], "row_reg_scalar"), ([600, 100], "row_stream_vec"), ([600, 100], "row_stream_scalar")]
        for dims, force in cases:
            ins = [(3 * torch.randn(*dims, generator=gen)).bfloat16()]
            fv = VARIANTS.index(force) if force else -1
            ctx.force_variant(fv)
            try:
                pl = h.plan(dims, force_variant=fv)
                got = run_gpu(h, pat, dims, ins)
            finally:
                ctx.force_variant(-1)
            want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0]
            assert_close(got[0], want[0], f"lse dims={dims} {force}")
            # the total: terms of either sign, each with fp32 roundings of its own; a lane adds the
            # rows of its block in fp32, the blocks are added in fp64
            lse = np.asarray(want[0], dtype=np.float64)
            rpb = -(-dims[0] // pl["grid"][0][0])
            lim = (16 + rpb) * 2.0 ** -24 * np.abs(lse).sum() + 1e-6
            assert abs(float(got[1]) - float(want[1])) <= lim, (dims, force, float(got[1]), float(want[1]), lim)
            # the amax of bf16 inputs is exact
            assert float(got[2]) == float(want[2]) == float(ins[0].float().abs().max()), (dims, force)
    finally:
        ctx.close()


@pytest.mark.gpu
def test_column_sums_and_scalar_reductions_together():
    from oracle import run as oracle_run
    from paper_2103_05288_amd import Context
    from tests.util import assert_close, run_gpu, to_oracle_input
    pb = PatternBuilder("both")
    t, hh = pb.dims(2)
    x = pb.param("f32", [t, hh])
    m = pb.reduce("max", x, 1)
    e = pb.op("exp", pb.op("sub", x, pb.broadcast(m, [t, hh], [0])))        # in (0, 1]
    pb.output(pb.cast(e, "bf16"))
    pb.output(pb.reduce("sum", e, 0))                                      # non-negative terms: the element-wise bar applies
    pb.output(pb.reduce("min", m, 0))
    pb.output(pb.reduce("sum", pb.reduce("sum", e, 1), 0))
    pat = pb.build()
    ctx = Context(0)
    try:
        h = ctx.register(pat)
        assert h.info["n_phases"] == 2
        gen = torch.Generator().manual_seed(37)
        for dims in ([5, 3], [3000, 130], [700, 1024], [129, 5000], [50, 26000]):
            ins = [torch.randn(*dims, generator=gen)]
            assert h.plan(dims)["n_launches"] == 3
            got = run_gpu(h, pat, dims, ins)
            want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0]
            for k, (g, w) in enumerate(zip(got, want)):
                assert_close(g, w, f"dims={dims} out{k}")
    finally:
        ctx.close()


def scaled_squares_with_sums():
    """No reduction along the rows: y = x * s[t] + b[h] with x a window of a wider input padded on the left, and
    two sums over the rows (non-negative terms)."""
    pb = PatternBuilder("scaled_squares")
    t, h, wide, low = pb.dims(4)
    x = pb.cast(pb.pad(pb.param("bf16", [t, wide]), [pb.static_start(0), low], [t, h], 0.5), "f32")
    s = pb.param("f32", [t])
    b = pb.param("f32", [h])
    y = pb.op("add", pb.op("mul", x, pb.broadcast(s, [t, h], [0])), pb.broadcast(b, [t, h], [1]))
    pb.output(pb.cast(y, "bf16"))
    pb.output(pb.reduce("sum", pb.op("mul", y, y), 0))
    pb.output(pb.reduce("sum", pb.op("abs", y), 0))
    return pb.build()


def test_single_shape_build_by_column_tiles(hctx):
    """The single-shape module of a non-temporal launch also holds the plain version for misaligned operands."""
    h = hctx.register_static(gelu_backward_bias_gradient(), [16384, 1024])
    assert h.info["n_variants"] == 3
    assert h.plan([16384, 1024])["kernels"][0].endswith("k_row_cols_vec_nt")
    q = h.plan([16384, 1024], inputs=[4096, 4098, 4096], outputs=[4096, 4096])
    assert q["kernels"][0].endswith("k_row_cols_vec") and q["workspace_bytes"] <= 16 << 20
    # the workspace a caller asked for without showing its operands is enough for any alignment
    assert q["workspace_bytes"] == hctx.workspace_bytes(h.id, [16384, 1024]) == h.plan([16384, 1024])["workspace_bytes"]


@pytest.mark.gpu
@pytest.mark.parametrize("nt", [0, 1])
def test_version_by_column_tiles(nt):
    """Element-wise patterns with sums over the rows run in k_row_cols: every number of lanes along the columns
    (1 .. 64) at its edges, several column tiles, fewer rows than a batch, and more than a block sums up in
    one go; plain accesses, and the version for rows of whole slots with non-temporal ones."""
    from oracle import run as oracle_run
    from paper_2103_05288_amd import Context
    from tests.util import assert_close, run_gpu, to_oracle_input
    ctx = Context(0)
    ctx.test_option("non_temporal", nt)
    try:
        gen = torch.Generator().manual_seed(41)
        plain, padded = gelu_backward_bias_gradient(), scaled_squares_with_sums()
        hp, hq = ctx.register(plain), ctx.register(padded)
        assert (hp.info["template"], hp.info["n_phases"]) == (hq.info["template"], hq.info["n_phases"]) == ("row_reduce", 0)
        lanes = set()
        for i, h in enumerate((4, 8, 9, 17, 24, 64, 65, 128, 129, 255, 256, 504, 513, 1024, 1032, 2041, 2048, 2049, 4104)):
            for t in ((1, 3 + i, 200 + 7 * i) if h > 64 else (1, 5000 + i)):
                pl = hp.plan([t, h])
                lanes.add(pl["lanes_per_row"])
                assert pl["kernels"][0].endswith("k_row_cols_vec_nt" if nt and h % 8 == 0 else "k_row_cols_vec"), pl["kernels"]
                assert pl["workspace_bytes"] >= pl["grid"][0][0] * h * 4 and pl["workspace_bytes"] == ctx.workspace_bytes(hp.id, [t, h])
                ins = _inputs(plain, [t, h], gen)
                got = run_gpu(hp, plain, [t, h], ins)
                want = oracle_run(plain, [t, h], [to_oracle_input(x) for x in ins])[0]
                assert_close(got[0], want[0], f"dx {t}x{h} nt={nt}")
                dy, x, b = (v.double().numpy() for v in ins)
                a = 1.702 * (x + b)
                s = 1.0 / (1.0 + np.exp(-a))
                _check_sum(got[1], want[1], np.abs(dy * s * (1.0 + a * (1.0 - s))), -(-t // pl["grid"][0][0]), f"db {t}x{h} nt={nt}")
                dims = [t, h, max(1, h - 3), min(2, h - 1)] if i % 2 else [t, h, h, 0]
                ins = [torch.randn(t, dims[2], generator=gen).bfloat16(), torch.randn(t, generator=gen), torch.randn(h, generator=gen)]
                got = run_gpu(hq, padded, dims, ins)
                want = oracle_run(padded, dims, [to_oracle_input(v) for v in ins])[0]
                for k, (g, w) in enumerate(zip(got, want)):
                    assert_close(g, w, f"padded {dims} out{k} nt={nt}")
        assert lanes == {1, 2, 4, 8, 16, 32, 64}          # (more of them for large ragged rows only, see the next test)
    finally:
        ctx.close()


def plain_sums(second):
    """Sums over the rows of the values as they are stored: nothing is rounded before it is added."""
    pb = PatternBuilder("plain_sums2" if second else "plain_sums")
    t, h = pb.dims(2)
    x = pb.param("f32", [t, h])
    pb.output(pb.cast(x, "bf16"))
    pb.output(pb.reduce("sum", x, 0))
    if second:
        pb.output(pb.reduce("sum", pb.op("neg", x), 0))
    return pb.build()


@pytest.mark.gpu
@pytest.mark.parametrize("second", [False, True])
def test_sums_by_column_tiles_are_rounded_once(second):
    """k_row_cols adds up in fp64.  With partial rows in fp64 (fewer than 256 of them, or fewer than 4096 rows) a sum is
    the exact one rounded to fp32: half an ulp, against 64 bits in plain torch, on values of both signs (where
    every earlier rounding shows).  Otherwise every partial row is rounded once as well.  From one row per lane to
    more than a hundred, whole and odd batches, lanes without a row, one partial row, 1 to 256 lanes along
    the columns, plain and non-temporal accesses; a small workspace limit (more columns than 2 MiB of fp64)."""
    from paper_2103_05288_amd import Context
    ctx = Context(0)
    try:
        pat = plain_sums(second)
        h = ctx.register(pat)
        gen = torch.Generator(device="cuda").manual_seed(47)
        seen, reached, kinds = set(), set(), set()
        cases = [[1, 36], [2, 36], [700, 4096], [513, 4096], [3, 2200001], [11000, 1101], [25000, 500], [16003, 1001]]
        for H, big in ((8, 1 << 23), (13, 1 << 22), (24, 1 << 22), (40, 1 << 22), (100, 1 << 22), (250, 1 << 20), (504, 1 << 20), (20001, 1 << 14)):
            p = h.plan([big, H])
            rows = p["grid"][0][0] * (256 // p["lanes_per_row"])        # one row per lane
            for k, r in ((2, 0), (15, 1), (16, 0), (17, rows - 1), (31, 5), (33, 0), (110, 3)):
                if rows * (k + 1) * H < 1 << 28:
                    cases.append([rows * k + r, H])
        for T, H in cases:
            p = h.plan([T, H])
            print(f"[rounded once] {T}x{H} {p['kernels'][0]} {p['grid'][0]}", flush=True)
            seen.add((p["lanes_per_row"], p["kernels"][0].endswith("_nt")))
            reached.add(-(-T // (p["grid"][0][0] * (256 // p["lanes_per_row"]))))
            x = torch.empty((T, H), device="cuda").normal_(generator=gen)
            outs = [torch.full((T, H), float("nan"), device="cuda", dtype=torch.bfloat16)]
            outs += [torch.full((H,), float("nan"), device="cuda") for _ in range(2 if second else 1)]
            ws = torch.full((ctx.workspace_bytes(h.id, [T, H]),), 255, dtype=torch.uint8, device="cuda")
            h.launch([T, H], [x], outs, workspace=ws)
            torch.cuda.synchronize()
            P, TY = p["grid"][0][0], 256 // p["lanes_per_row"]
            part = torch.zeros((P, H), dtype=torch.float64, device="cuda")         # the blocks' shares
            for i in range(0, T, 1 << 14):
                rows = torch.arange(i, min(T, i + (1 << 14)), device="cuda")
                part.index_add_(0, rows // TY % P, x[i : i + (1 << 14)].double())
            want = part.sum(0)
            few = P < 256 or T < 4096
            kinds.add(few)
            assert torch.equal(outs[0], x.bfloat16())
            # half an ulp of the result (and of the partial rows), and what the order of the fp64 additions
            # changes (T * 2^-53 of the terms)
            lim = (want.abs() + (0 if few else part.abs().sum(0))) * 2.0 ** -24 + T * 2.0 ** -50
            for sign, o in zip((1, -1), outs[1:]):
                assert bool(((o.double() - sign * want).abs() <= lim).all()), (T, H, (o.double() - sign * want).abs().max())
            del x, outs, ws, part
        assert kinds == {True, False}
        assert {s[0] for s in seen} == {1, 2, 4, 8, 16, 32, 64, 128, 256} and {s[1] for s in seen} == {False, True}
        assert {1, 2, 16, 18, 32, 33} <= reached and max(reached) > 100, reached
    finally:
        ctx.close()


@pytest.mark.gpu
def test_wide_rows_of_patterns_with_and_without_element_outputs():
    """Rows beyond blocks of 256 threads: LayerNorm backward never takes three slots per lane there (two on twice the
    lanes, else the streaming version); a pattern without per-element outputs takes the streaming version."""
    from oracle import run as oracle_run
    from paper_2103_05288_amd import Context
    from tests.util import assert_close, run_gpu, to_oracle_input
    ctx = Context(0)
    try:
        gen = torch.Generator().manual_seed(43)
        pat = layernorm_backward_graph()
        h = ctx.register(pat)
        for dims, want_kernel in (([300, 8201], "nv2w_s"), ([270, 12289], "nv2w"), ([40, 16385], "stream_vec"), ([261, 24576], "stream_vec"),
                                  ([5, 33000], "stream_vec")):
            ins = _inputs(pat, dims, gen)
            pl = h.plan(dims)
            assert pl["kernels"][0].endswith(want_kernel), (dims, pl["kernels"])
            got = run_gpu(h, pat, dims, ins)
            want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0]
            assert_close(got[0], want[0], f"dx {dims}")
            x64, dy64 = ins[0].double().numpy(), ins[1].double().numpy()
            xc = x64 - x64.mean(1, keepdims=True)
            xhat = xc / np.sqrt((xc * xc).mean(1, keepdims=True) + 1e-5)
            rpb = -(-dims[0] // pl["grid"][0][0])
            _check_sum(got[1], want[1], np.abs(dy64 * xhat), rpb, f"dgamma {dims}")
            _check_sum(got[2], want[2], np.abs(dy64), rpb, f"dbeta {dims}")
        pat = logsumexp_with_total_and_amax()
        h = ctx.register(pat)
        assert h.plan([50, 6144])["variant_name"] == "row_reg_vec"
        for dims in ([50, 6145], [600, 8191], [9, 8193], [9, 16384], [9, 16391], [513, 32768], [7, 32769], [3, 65543]):
            ins = [(3 * torch.randn(*dims, generator=gen)).bfloat16()]
            pl = h.plan(dims)
            assert pl["variant_name"] == "row_stream_vec"
            got = run_gpu(h, pat, dims, ins)
            want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0]
            assert_close(got[0], want[0], f"lse {dims}")
            lim = (16 + -(-dims[0] // pl["grid"][0][0])) * 2.0 ** -24 * np.abs(np.asarray(want[0])).sum() + 1e-6
            assert abs(float(got[1]) - float(want[1])) <= lim
            assert float(got[2]) == float(want[2])
    finally:
        ctx.close()


@pytest.mark.gpu
def test_misaligned_operands_fit_the_workspace_asked_for():
    """A launch whose operands lie off the boundaries that the plan without pointers assumes runs another grid; the
    workspace asked for beforehand is enough for it."""
    from oracle import run as oracle_run
    from paper_2103_05288_amd import Context
    from tests.util import assert_close, to_oracle_input
    ctx = Context(0)
    try:
        pat = logsumexp_with_total_and_amax()
        h = ctx.register(pat)
        gen = torch.Generator().manual_seed(3)
        for dims in ([110, 4183], [1020, 5740]):
            x = torch.randn(*dims, generator=gen).bfloat16()
            want = oracle_run(pat, dims, [to_oracle_input(x)])[0]
            n = dims[0] * dims[1]
            for off in (0, 1, 8):                       # elements past a 256-byte boundary
                dev = torch.zeros(n + 64, dtype=torch.bfloat16, device="cuda")
                dev[off : off + n] = x.reshape(-1).cuda()
                outs = [torch.full((dims[0],), float("nan"), device="cuda")] + [torch.full((), float("nan"), device="cuda") for _ in range(2)]
                ws = torch.empty(ctx.workspace_bytes(h.id, dims), dtype=torch.uint8, device="cuda")
                h.launch(dims, [dev[off:]], outs, workspace=ws)
                torch.cuda.synchronize()
                assert_close(outs[0].cpu(), want[0], f"lse {dims} off={off}")
                lim = 2.0 ** -20 * np.abs(np.asarray(want[0])).sum()
                assert abs(float(outs[1]) - float(want[1])) <= lim and float(outs[2]) == float(want[2])
                outs2 = [torch.full_like(o, float("nan")) for o in outs]
                ctx.launch_static_scratch(h.id, dims, [dev[off:]], outs2)
                torch.cuda.synchronize()
                assert all(torch.equal(a, b) for a, b in zip(outs, outs2))
    finally:
        ctx.close()


def test_narrow_rows_keep_every_lane_busy(hctx):
    """The version by column tiles has the fewest lanes along the columns that hold a row (a power of two), one for a
    row of one slot: with more of them the rest would idle for the whole kernel."""
    h = hctx.register(gelu_backward_bias_gradient())
    for width, lanes in ((4, 1), (8, 1), (9, 2), (16, 2), (24, 4), (32, 4), (40, 8), (64, 8), (128, 16), (512, 64), (4096, 64)):
        for rows in (100, 1 << 20):
            p = h.plan([rows, width])
            assert p["lanes_per_row"] == lanes and "row_cols" in p["kernels"][0], (rows, width)


def softmax_with_column_sums():
    """Row softmax of bf16 scores and the sum over the rows of the probabilities: one reduction over the rows."""
    pb = PatternBuilder("softmax_col_sums")
    t, h = pb.dims(2)
    x = pb.cast(pb.param("bf16", [t, h]), "f32")
    e = pb.op("exp", pb.op("sub", x, pb.broadcast(pb.reduce("max", x, 1), [t, h], [0])))
    y = pb.op("div", e, pb.broadcast(pb.reduce("sum", e, 1), [t, h], [0]))
    pb.output(pb.cast(y, "bf16"))
    pb.output(pb.reduce("sum", y, 0))
    return pb.build()


def test_partial_rows_of_wide_blocks(hctx):
    """A row of partial sums holds no more rows of the tensor where the rows need blocks of 1024 threads than where
    they fit blocks of 512, as long as three slots per lane would have fitted those."""
    h = hctx.register(layernorm_backward_graph())
    narrow = h.plan([32768, 8192])
    assert narrow["block"][0][0] == 512
    for width in (8193, 9000, 12288):
        p = h.plan([32768, width])
        assert p["block"][0][0] == 1024 and p["grid"][0][0] >= narrow["grid"][0][0], width
        assert p["workspace_bytes"] >= 2 * 4 * width * p["grid"][0][0]
        assert h.plan([300, width])["grid"][0][0] >= 299


@pytest.mark.gpu
def test_wide_blocks_with_little_scratch():
    """The static scratch array holds one row of partial sums per CU, not two, of rows of 10000 columns: the call is
    accepted and runs one round of blocks."""
    from oracle import run as oracle_run
    from paper_2103_05288_amd import Context
    from tests.util import assert_close, run_gpu, to_oracle_input
    ctx = Context(0)
    try:
        pat = softmax_with_column_sums()
        h = ctx.register(pat)
        gen = torch.Generator().manual_seed(7)
        for dims in ([600, 10000], [257, 12283]):
            x = (2 * torch.randn(*dims, generator=gen)).bfloat16()
            assert ctx.workspace_bytes(h.id, dims) > 16 << 20 or dims[0] < 400
            want = oracle_run(pat, dims, [to_oracle_input(x)])[0]
            terms = np.asarray(want[0], dtype=np.float64)
            outs = [torch.full(dims, float("nan"), dtype=torch.bfloat16, device="cuda"), torch.full((dims[1],), float("nan"), device="cuda")]
            ctx.launch_static_scratch(h.id, dims, [x.cuda()], outs)
            torch.cuda.synchronize()
            for got, rows in ((run_gpu(h, pat, dims, [x]), 2), ([o.cpu() for o in outs], 3)):
                assert_close(got[0], want[0], f"softmax {dims}")
                _check_sum(got[1], want[1], terms, rows, f"column sums {dims}")
    finally:
        ctx.close()
