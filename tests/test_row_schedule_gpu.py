"""GPU parity over the row-reduce schedules: every class of (lanes per row, slots per lane), ragged
tails of every length, row counts that leave the last block partly filled, rows of several
wavefronts whose slot grid turns from row to row, the staged (LDS) and unstaged kernel versions,
and the streaming version behind the longest register-resident class."""
import os

import numpy as np
import pytest
import torch

from oracle import run as oracle_run
from workloads import PatternBuilder
from workloads.configs import CONFIGS
from tests.util import assert_close, run_gpu, to_oracle_input
from paper_2103_05288_amd import VARIANTS

pytestmark = pytest.mark.gpu

# row lengths chosen around the capacity steps 2 * 2^k and 3 * 2^k slots of 8 elements, plus ragged
# tails 1..7 past a slot boundary
ROW_LENGTHS = [1, 3, 7, 8, 9, 15, 17, 31, 33, 47, 63, 65, 97, 100, 127, 128, 129, 191, 200, 255, 256, 257, 385, 511, 513,
               768, 770, 1023, 1024, 1025, 1100, 1537, 2047, 2048, 2049, 3000, 3073, 4096, 4097, 5739, 6144, 6145, 8191,
               8193, 12289, 16386, 20003, 24576, 24577]


@pytest.fixture(scope="module")
def ctx():
    from paper_2103_05288_amd import Context
    c = Context(0)
    yield c
    c.close()


def check(ctx, cfg_name, dims, seed, handle=None):
    cfg = CONFIGS[cfg_name]
    pat = cfg.pattern()
    h = handle or ctx.register(pat)
    ins = cfg.inputs(dims, seed=seed)
    got = run_gpu(h, pat, dims, ins)
    want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0]
    plan = h.plan(dims)
    for k, (g, w) in enumerate(zip(got, want)):
        assert_close(g, w, f"{cfg_name} dims={dims} out{k} G={plan['lanes_per_row']} nv={plan['slots_per_lane']} "
                           f"kernel={plan['kernels'][0]}")
    return plan


@pytest.mark.parametrize("cfg_name", ["C2", "C4"])
def test_every_capacity_class_and_tail(ctx, cfg_name):
    h = ctx.register(CONFIGS[cfg_name].pattern())
    seen = set()
    suffixes = set()
    for i, H in enumerate(ROW_LENGTHS):
        T = 1 + (i * 5) % 23            # 1 .. 23 rows: every residue of rows per block shows up
        plan = check(ctx, cfg_name, [T, H], seed=100 + i, handle=h)
        seen.add((plan["variant_name"], plan["lanes_per_row"], plan["slots_per_lane"]))
        name = plan["kernels"][0]
        suffixes.add(name.rsplit("_", 1)[1] if name.rsplit("_", 1)[1] in ("e", "t", "nt") else "")
        # a ragged end on at least 8 lanes in a block of 256 threads is taken as single elements (_t)
        if plan["variant_name"] == "row_reg_vec" and plan["block"][0][0] == 256:
            assert name.endswith("_t") == (H % 8 != 0 and plan["lanes_per_row"] >= 8), (H, name)
    assert {"", "e", "t"} <= suffixes
    lanes = {g for v, g, n in seen if v == "row_reg_vec"}
    assert {4, 8, 16, 32, 64, 128, 256, 512, 1024} <= lanes
    assert {n for v, g, n in seen if v == "row_reg_vec"} >= {1, 2, 3}
    assert any(v == "row_stream_vec" for v, g, n in seen)
    # large launches of rows that start and end on 16-byte boundaries run the non-temporal versions
    rows = lambda H: (100 << 20) // (4 * H)
    assert all(h.plan([rows(H), H])["kernels"][0].endswith("_nt") for H in (128, 768, 2048, 6144))
    assert not any(h.plan([rows(H), H])["kernels"][0].endswith("_nt") for H in (64, 127, 2047, 8192))
    assert not any(h.plan([5, H])["kernels"][0].endswith("_nt") for H in (128, 768, 2048, 6144))


@pytest.mark.parametrize("cfg_name", ["C2", "C4"])
def test_many_rows_per_block_and_turning_grid(monkeypatch, cfg_name):
    """Enough rows that blocks walk several of them (the software pipeline runs past its first row)
    and, for rows of several wavefronts, the slot grid keeps turning.  One round of resident blocks
    keeps the row counts this needs small."""
    from paper_2103_05288_amd import Context
    c = Context(0)
    c.test_option("row_rounds", 1)
    try:
        h = c.register(CONFIGS[cfg_name].pattern())
        for H, T in [(127, 70001), (1100, 9001), (2047, 6000), (3001, 5003), (5739, 6007), (8190, 4500), (20003, 700)]:
            plan = check(c, cfg_name, [T, H], seed=H, handle=h)
            rows_per_block = plan["block"][0][0] // plan["lanes_per_row"]
            assert T > plan["grid"][0][0] * rows_per_block, (H, T, plan["grid"], rows_per_block)
    finally:
        c.close()


def test_non_temporal_versions_any_alignment(monkeypatch):
    """The non-temporal kernel versions forced wherever they exist (rows of whole slots, also small
    launches and short rows that the host rule would leave to the plain versions), and the host rule
    with operands that are not 16-byte aligned: it must fall back to a plain version."""
    from paper_2103_05288_amd import Context
    c = Context(0)
    c.test_option("non_temporal", 1)
    try:
        for cfg_name in ("C2", "C4"):
            h = c.register(CONFIGS[cfg_name].pattern())
            for H, T in [(8, 40), (127, 300), (1000, 77), (2047, 500), (3000, 2003), (6144, 300), (72, 5000)]:
                plan = check(c, cfg_name, [T, H], seed=H + 2, handle=h)
                # (the non-temporal versions are built for rows of whole slots: 8 elements here)
                assert plan["kernels"][0].endswith("_nt") == (H % 8 == 0), plan["kernels"]
        # the loop-fusion kernel and the epilogue of a column reduce have such versions too
        plan = check(c, "C0", [300, 768], seed=9)
        assert plan["kernels"][0].endswith("k_loop_vec_nt"), plan["kernels"]
        plan = check(c, "C3", [3000, 1024], seed=10)
        assert plan["kernels"][-1].endswith("k_col_epi2_vec_nt"), plan["kernels"]
        c.force_variant(VARIANTS.index("col_3stage_vec"))
        check(c, "C3", [3000, 1024], seed=10)
        c.force_variant(-1)
        plan = c.register(CONFIGS["C3"].pattern()).plan([3000, 1024], VARIANTS.index("col_3stage_vec"))
        assert plan["kernels"][-1].endswith("k_col_epi_vec_nt"), plan["kernels"]
    finally:
        c.close()
    c = Context(0)
    try:
        # host rule for the loop kernels: large launches only
        h0 = c.register(CONFIGS["C0"].pattern())
        assert h0.plan([20000, 768])["kernels"][0].endswith("_nt") and not h0.plan([300, 768])["kernels"][0].endswith("_nt")
        # one real launch above the size threshold under the host rule (C2: 6 bytes per element)
        plan = check(c, "C2", [14000, 1024], seed=21)
        assert plan["kernels"][0].endswith("_nt"), plan["kernels"]
        cfg = CONFIGS["C4"]
        pat = cfg.pattern()
        h = c.register(pat)
        dims = [33, 1024]
        ins = cfg.inputs(dims, seed=3)
        want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0]
        dev = []
        for t in ins:                       # every operand 2 bytes (bf16) or 1 byte past a 16-byte boundary
            flat = torch.empty(t.numel() + 16, dtype=t.dtype, device="cuda")
            view = flat[1:1 + t.numel()].view(t.shape)
            view.copy_(t)
            dev.append(view)
        out_flat = torch.zeros(dims[0] * dims[1] + 16, dtype=torch.bfloat16, device="cuda")
        out = out_flat[1:1 + dims[0] * dims[1]].view(dims)
        # the rule at a size where it applies: aligned (or no) pointers take the version, these do not
        big = [20000, 1024]
        assert h.plan(big)["kernels"][0].endswith("_nt")
        assert not h.plan(big, inputs=[t.data_ptr() for t in dev], outputs=[out.data_ptr()])["kernels"][0].endswith("_nt")
        h.launch(dims, dev, [out])
        torch.cuda.synchronize()
        assert_close(out.cpu(), want[0], "misaligned bases")
        assert float(out_flat[0]) == 0.0 and float(out_flat[-1]) == 0.0
    finally:
        c.close()


def test_unstaged_versions(monkeypatch):
    """The same shapes with LDS staging switched off: the kernel versions that read row vectors from
    global memory in every slot."""
    from paper_2103_05288_amd import Context
    c = Context(0)
    c.test_option("stage_row_vectors", 0)
    try:
        for cfg_name in ("C2", "C4"):
            h = c.register(CONFIGS[cfg_name].pattern())
            for H, T in [(9, 40), (127, 300), (1100, 77), (3001, 2003), (8190, 600), (20003, 40)]:
                plan = check(c, cfg_name, [T, H], seed=H + 1, handle=h)
                assert not plan["kernels"][0].endswith("_s") and plan["lds_bytes"][0] == 0
    finally:
        c.close()


def test_ragged_pieces_every_storage_width(ctx):
    """One pattern with 1-, 2- and 4-byte operands and outputs of each width, so the ragged tail of a
    row moves through the power-of-two pieces of every vector type; the last row ends the tensors, so
    its tail cannot be over-read."""
    pb = PatternBuilder("widths")
    T, H = pb.dims(2)
    a = pb.param("bf16", [T, H])
    b = pb.param("f32", [T, H])
    m = pb.param("bool", [T, H])
    a32 = pb.cast(a, "f32")
    s = pb.reduce("max", pb.op("mul", a32, b), 1)      # a max: no accumulated rounding to cancel against
    y = pb.op("select", m, b, pb.op("add", a32, pb.broadcast(s, [T, H], [0])), dims=[T, H])
    pb.output(y)                                        # f32
    pb.output(pb.cast(y, "f16"))                        # 2 bytes
    pb.output(pb.op("gt", y, pb.const(0.0), dims=[T, H]))   # bool, 1 byte
    pat = pb.build()
    h = ctx.register(pat)
    rng = np.random.default_rng(5)
    for H_ in list(range(1, 18)) + [63, 127, 129, 250, 1001, 4099]:
        for T_ in (1, 5):
            ins = [torch.from_numpy(rng.standard_normal((T_, H_)).astype(np.float32)).to(torch.bfloat16),
                   torch.from_numpy(rng.standard_normal((T_, H_)).astype(np.float32)),
                   torch.from_numpy((rng.random((T_, H_)) < 0.3).astype(np.uint8))]
            got = run_gpu(h, pat, [T_, H_], ins)
            want = oracle_run(pat, [T_, H_], [to_oracle_input(t) for t in ins])[0]
            # the comparison output flips where y is within rounding of zero: compare it only away from 0
            y64 = np.asarray(want[0])
            safe = np.abs(y64) > 1e-4
            assert_close(got[0], want[0], f"widths f32 dims={[T_, H_]}")
            assert_close(got[1], want[1], f"widths f16 dims={[T_, H_]}")
            assert np.array_equal(got[2].numpy()[safe] != 0, np.asarray(want[2])[safe] != 0), [T_, H_]


def test_odd_rows_of_two_byte_elements_any_base_alignment():
    """Rows of an odd number of 2-byte elements start alternately on and two bytes off a dword
    boundary.  A pattern with 2-byte and 1-byte full-size operands and results, an fp32 row vector
    (staged in LDS or not), a sum, a max and an argmax per row; guard cells around every result show
    that nothing is written outside, with bases on a 16-byte boundary and one element past it."""
    from paper_2103_05288_amd import Context
    pb = PatternBuilder("odd_rows")
    T, H = pb.dims(2)
    x = pb.param("bf16", [T, H])
    m = pb.param("bool", [T, H])
    g = pb.param("f32", [H])
    x32 = pb.cast(x, "f32")
    v = pb.op("mul", x32, pb.broadcast(g, [T, H], [1]))
    mx = pb.reduce("max", v, 1)
    am = pb.reduce("argmax", v, 1)
    e = pb.op("exp", pb.op("sub", v, pb.broadcast(mx, [T, H], [0])))
    s = pb.reduce("sum", e, 1)
    y = pb.op("select", m, x32, pb.op("div", e, pb.broadcast(s, [T, H], [0])), dims=[T, H])
    pb.output(pb.cast(y, "bf16"))
    pb.output(pb.cast(pb.op("add", y, v), "f16"))
    pb.output(pb.op("gt", v, pb.const(0.25), dims=[T, H]))
    pb.output(am)
    pb.output(s)
    pat = pb.build()
    rng = np.random.default_rng(11)
    out_dt = [torch.bfloat16, torch.float16, torch.bool, torch.int32, torch.float32]

    def run(c, h, dims, ins, skew):
        """Launch with every full-size tensor `skew` elements past a 16-byte boundary and guards around the results."""
        T_, H_ = dims
        dev = []
        for t in ins:
            if t.dim() == 2:
                flat = torch.zeros(t.numel() + 32, dtype=t.dtype, device="cuda")
                view = flat[16 + skew:16 + skew + t.numel()].view(t.shape)
                view.copy_(t)
                dev.append(view)
            else:
                dev.append(t.cuda())
        flats, outs = [], []
        for dt, full in zip(out_dt, (True, True, True, False, False)):
            n = T_ * H_ if full else T_
            flat = torch.full((n + 32,), 1, dtype=dt, device="cuda")
            flats.append(flat)
            outs.append(flat[16 + skew:16 + skew + n].view((T_, H_) if full else (T_,)))
        h.launch(dims, dev, outs)
        torch.cuda.synchronize()
        for f, o in zip(flats, outs):
            fc = f.cpu()
            assert bool((fc[:16 + skew] == 1).all()) and bool((fc[16 + skew + o.numel():] == 1).all()), f"guard cells dims={dims} skew={skew}"
        return [o.cpu() for o in outs]

    for stage in (1, 0):
        c = Context(0)
        c.test_option("stage_row_vectors", stage)
        c.test_option("row_rounds", 1)
        try:
            h = c.register(pat)
            shapes = [(2, 5), (3, 9), (5, 33), (64, 127), (1001, 129), (7, 511), (300, 1023), (33, 1025), (4100, 3001),
                      (6000, 4095), (9, 6143), (2500, 8191), (5, 24575), (70001, 127)]
            for T_, H_ in shapes:
                ins = [torch.from_numpy(rng.standard_normal((T_, H_)).astype(np.float32)).to(torch.bfloat16),
                       torch.from_numpy((rng.random((T_, H_)) < 0.3)),
                       torch.from_numpy((0.5 + rng.random(H_)).astype(np.float32))]
                print(f"[odd rows] stage={stage} dims={[T_, H_]}", flush=True)
                want = oracle_run(pat, [T_, H_], [to_oracle_input(t) for t in ins])[0]
                v64 = np.asarray(ins[0].float().numpy(), dtype=np.float64) * np.asarray(ins[2].numpy(), dtype=np.float64)[None, :]
                for skew in (0, 1):          # bf16 / f16 tensors: dword aligned, then two bytes off
                    got = run(c, h, [T_, H_], ins, skew)
                    what = f"odd rows dims={[T_, H_]} stage={stage} skew={skew}"
                    assert_close(got[0], want[0], what + " out0")
                    assert_close(got[1], want[1], what + " out1")
                    safe = np.abs(v64 - 0.25) > 1e-5
                    assert np.array_equal(got[2].numpy()[safe], np.asarray(want[2])[safe] != 0), what + " out2"
                    # argmax: the position may differ only where two products tie to fp32 rounding
                    ga = got[3].numpy().astype(np.int64)
                    wa = np.asarray(want[3]).astype(np.int64)
                    rows_ = np.arange(T_)
                    assert np.all((ga >= 0) & (ga < H_)), what
                    assert np.all(np.abs(v64[rows_, ga] - v64[rows_, wa]) <= 1e-6 * np.abs(v64[rows_, wa])), what + " argmax"
                    assert_close(got[4], want[4], what + " out4")
        finally:
            c.close()


def test_single_element_ends_in_fp32_and_f16_patterns(ctx):
    """The versions that take the ragged ends of a row as single elements, at other vector widths
    than the benchmark patterns': an fp32 softmax (4 elements per slot, up to 3 single elements at
    either end -- fp32 rows always start on dword boundaries, so they are never shifted) and an f16
    one with a row-group mask (8 per slot; odd rows are shifted), at seeded random row lengths."""
    rng = np.random.default_rng(23)
    for dt, tdt in (("f32", torch.float32), ("f16", torch.float16)):
        pb = PatternBuilder("softmax_" + dt)
        B, S, H = pb.dims(3)
        x = pb.param(dt, [B, S, H])
        m = pb.param(dt, [B, pb.static(1), H])
        v = pb.op("add", pb.cast(x, "f32"), pb.cast(pb.broadcast(m, [B, S, H], [0, 1, 2]), "f32"))
        mx = pb.reduce("max", v, 2)
        e = pb.op("exp", pb.op("sub", v, pb.broadcast(mx, [B, S, H], [0, 1])))
        s = pb.reduce("sum", e, 2)
        pb.output(pb.cast(pb.op("div", e, pb.broadcast(s, [B, S, H], [0, 1])), dt))
        pb.output(mx)
        pat = pb.build()
        h = ctx.register(pat)
        seen_t = 0
        for _ in range(14):
            Hh = int(rng.integers(33, 3000))
            Bb, Ss = int(rng.integers(1, 4)), int(rng.integers(1, 300))
            dims = [Bb, Ss, Hh]
            xs = torch.from_numpy(rng.standard_normal((Bb, Ss, Hh)).astype(np.float32)).to(tdt)
            ms = torch.from_numpy((rng.random((Bb, 1, Hh)) < 0.2).astype(np.float32) * -50.0).to(tdt)
            got = run_gpu(h, pat, dims, [xs, ms])
            want = oracle_run(pat, dims, [to_oracle_input(xs), to_oracle_input(ms)])[0]
            plan = h.plan(dims)
            seen_t += plan["kernels"][0].endswith("_t")
            for k, (g, w) in enumerate(zip(got, want)):
                assert_close(g, w, f"softmax {dt} dims={dims} out{k} kernel={plan['kernels'][0]}")
        assert seen_t >= 5


@pytest.mark.parametrize("cfg_name", ["C2", "C4"])
def test_streaming_rows_and_piped_wide_rows(ctx, cfg_name):
    """The streaming version at the edges of what its blocks hold in registers (4 slots of 8 elements per lane,
    blocks of up to 1024 threads; longer rows are read again; far longer ones in blocks of 256), ragged ends of
    every kind, and blocks of 1024 threads that walk several rows."""
    h = ctx.register(CONFIGS[cfg_name].pattern())
    blocks = set()
    for i, H in enumerate((24577, 24584, 24583, 32760, 32767, 32768, 32769, 32777, 40004, 65535, 65536, 65537, 70003)):
        plan = check(ctx, cfg_name, [2 + i % 3, H], seed=300 + i, handle=h)
        assert plan["variant_name"] == "row_stream_vec"
        blocks.add((H > 65536, plan["block"][0][0]))
    assert blocks == {(False, 1024), (True, 256)}
    for H in (8, 100, 8191, 8192, 8200, 16385):      # forced: blocks of 256 to 1024 threads
        ctx.force_variant(VARIANTS.index("row_stream_vec"))
        try:
            check(ctx, cfg_name, [7, H], seed=H, handle=h)
        finally:
            ctx.force_variant(-1)
    plan = check(ctx, cfg_name, [2060, 12296], seed=5, handle=h)
    assert plan["kernels"][0].endswith("k_row_vec_nv3w") and plan["lanes_per_row"] == 1024 and plan["slots_per_lane"] == 2


@pytest.mark.parametrize("nt", [0, 1])
def test_held_rows(ctx, nt):
    """Patterns that write nothing per element: the edges of what the blocks of the streaming version hold (8 slots of 8
    elements a lane in 64 to 512 threads, 4 in 1024 and where rows are few; longer rows are read again), ragged ends, plain
    and non-temporal."""
    from workloads.extras import logsumexp_with_total_and_amax
    pat = logsumexp_with_total_and_amax()
    h = ctx.register(pat)
    seen = set()
    ctx.test_option("non_temporal", nt)
    try:
        for i, (T, H) in enumerate([(4097, 1538), (4100, 4096), (4097, 4102), (1030, 6145), (1025, 8192), (1027, 8193), (1026, 16391),
                                    (3, 6145), (2, 8193), (2, 16384), (3, 16391), (2, 32768), (3, 32769), (1, 65536), (2, 65537), (1, 70003),
                                    (1300, 8193)]):
            x = (torch.randn(T, H, generator=torch.Generator().manual_seed(i)) * 2).to(torch.bfloat16)
            x[T - 1, H - 1] = 40.0 + i                      # the last single element decides the last row
            plan = h.plan([T, H])
            assert plan["variant_name"] == "row_stream_vec"
            seen.add((plan["kernels"][0].split("_k_")[1], plan["block"][0][0]))
            assert plan["reg_slots"] == (4 if plan["kernels"][0].endswith("_vecw") else 8)
            got = run_gpu(h, pat, [T, H], [x])
            want = oracle_run(pat, [T, H], [to_oracle_input(x)])[0]
            for k, (g, w) in enumerate(zip(got, want)):
                assert_close(g, w, f"held rows {T}x{H} out{k}")
    finally:
        ctx.test_option("non_temporal", -1)
    for T, H, block in ((4097, 1538, 64), (7180, 6145, 128), (1030, 6145, 256), (3, 6145, 256), (1026, 16391, 512), (3, 16391, 512), (3, 16384, 512),
                        (1026, 32769, 1024)):
        assert h.plan([T, H])["block"][0][0] == block
    assert seen == {("row_stream_vec", b) for b in (64, 128, 256, 512)} | {("row_stream_vecw", b) for b in (256, 512, 1024)}


@pytest.mark.parametrize("dims, lanes, slots", [((1903, 16013), 512, 4), ((4100, 32000), 1024, 4), ((9000, 4096), 256, 2)], ids=lambda v: str(v))
def test_held_rows_add_up_in_chains_no_longer_than_the_other_versions(ctx, dims, lanes, slots):
    """Sums of squares (of one sign: the error is that of the additions) against the same sum in fp32 as `lanes` lanes of
    `slots` slots of eight elements take it, one chain of additions a lane, the lanes by halves: no further off."""
    pb = PatternBuilder()
    t, h = pb.dims(2)
    x = pb.cast(pb.param("bf16", [t, h]), "f32")
    pb.output(pb.reduce("sum", pb.op("mul", x, x), 1))
    hd = ctx.register(pb.build())
    assert hd.plan(list(dims))["variant_name"] == "row_stream_vec" and hd.plan(list(dims))["slots_per_lane"] > slots
    T, H = dims
    x = torch.randn(T, H, generator=torch.Generator().manual_seed(H)).to(torch.bfloat16).cuda()
    out = torch.empty(T, device="cuda")
    hd.launch(list(dims), [x], [out])
    sq = torch.zeros(T, slots * lanes * 8, device="cuda")
    sq[:, :H] = x.float() ** 2                      # (exact: eight significant bits squared)
    sq = sq.view(T, slots, lanes, 8)
    lane = torch.zeros(T, lanes, device="cuda")
    for j in range(slots):
        for e in range(8):
            lane = lane + sq[:, j, :, e]
    while lane.shape[1] > 1:
        half = lane.shape[1] // 2
        lane = lane[:, :half] + lane[:, half:]
    want = (x.double() ** 2).sum(1)
    off = lambda v: float((v.double() - want).norm() / want.norm())
    assert off(out) <= 1.05 * off(lane[:, 0]), (off(out), off(lane[:, 0]))


def test_ragged_rows_on_whole_lines():
    """Ragged rows with non-temporal accesses: vector slots on boundaries of 32, 64 or 128 elements of the tensor, up to
    127 + 7 single elements per row.  Odd and even lengths, a last slot that ends exactly at the row's end, the least
    and the most single elements, two rows per block; bases off a line fall back to 16-byte boundaries; too few rows
    for a grid of one alignment per lane group leave the slots where they are."""
    from paper_2103_05288_amd import Context
    c = Context(0)
    c.test_option("non_temporal", 1)
    try:
        h = c.register(CONFIGS["C4"].pattern())
        for H, T, al in ((777, 1100, 32), (1023, 700, 32), (1537, 400, 32), (1601, 600, 64), (2046, 515, 64), (2047, 515, 64), (3001, 390, 64),
                         (3073, 300, 128), (4095, 300, 128), (4097, 390, 128), (5739, 260, 128), (6150, 257, 128), (8185, 259, 128)):
            plan = check(c, "C4", [T, H], seed=H, handle=h)
            rpb = plan["block"][0][0] // plan["lanes_per_row"]
            assert plan["kernels"][0].endswith("_t") and plan["grid"][0][0] * rpb * H % al == 0, (H, plan["grid"])
        check(c, "C4", [20, 4095], seed=6, handle=h)
        cfg = CONFIGS["C4"]
        pat, dims = cfg.pattern(), [260, 4095]
        ins = cfg.inputs(dims, seed=8)
        for shift in (8, 1):                       # 16 bytes (bf16) or one element past a line
            dev = [torch.cat([torch.zeros(shift, dtype=t.dtype), t.reshape(-1)]).cuda()[shift:] for t in ins]
            out = torch.full((dims[0] * dims[1] + 64,), float("nan"), dtype=torch.bfloat16, device="cuda")
            h.launch(dims, dev, [out[32:]])
            torch.cuda.synchronize()
            want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0][0]
            assert_close(out[32:-32].reshape(dims).cpu(), want, f"base shifted by {shift}")
            assert bool(torch.isnan(out[:32]).all()) and bool(torch.isnan(out[-32:]).all())
        h1 = c.register(CONFIGS["C1"].pattern())   # a row-group operand read at the shifted columns
        for S in (777, 1023):
            plan = check(c, "C1", [1, 2, S], seed=S, handle=h1)
            assert plan["lanes_per_row"] == 64 and plan["kernels"][0].endswith("_t")
    finally:
        c.close()


def test_short_ragged_rows_on_eight_lanes(ctx):
    """Ragged rows of 10 to 12 slots: four lanes and a ragged last slot when there are few of them, eight lanes and single
    elements (up to seven, one to a lane) from 1024 rows on."""
    h = ctx.register(CONFIGS["C4"].pattern())
    for H in (73, 78, 79, 85, 93, 95):
        few, many = h.plan([1023, H]), h.plan([1024, H])
        assert few["lanes_per_row"] == 4 and not few["kernels"][0].endswith("_t")
        assert many["lanes_per_row"] == 8 and many["kernels"][0].endswith("_t")
        check(ctx, "C4", [1031, H], seed=H, handle=h)
    h1 = ctx.register(CONFIGS["C1"].pattern())
    for S in (73, 77, 93):
        assert check(ctx, "C1", [4, 4, S], seed=S, handle=h1)["lanes_per_row"] == 8


def test_ragged_rows_of_nine_slots_on_eight_lanes(ctx):
    """The same for rows of eight whole slots and two to seven elements."""
    h = ctx.register(CONFIGS["C4"].pattern())
    for H in (66, 68, 71):
        few, many = h.plan([1023, H]), h.plan([1024, H])
        assert few["lanes_per_row"] == 4 and not few["kernels"][0].endswith("_t")
        assert many["lanes_per_row"] == 8 and many["kernels"][0].endswith("_t")
        check(ctx, "C4", [1031, H], seed=H, handle=h)
    h1 = ctx.register(CONFIGS["C1"].pattern())
    for S in (66, 71):
        assert check(ctx, "C1", [4, 4, S], seed=S, handle=h1)["lanes_per_row"] == 8



def test_single_shape_module_with_operands_off_a_line():
    """Ragged rows on whole lines in a module for one shape: operands on a line, on 16 bytes and off them."""
    from paper_2103_05288_amd import Context
    c = Context(0)
    c.test_option("non_temporal", 1)
    try:
        cfg, dims = CONFIGS["C4"], [260, 4095]
        pat, ins = cfg.pattern(), cfg.inputs([260, 4095], seed=9)
        h = c.register_static(pat, dims)
        want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0][0]
        for shift in (0, 8, 1):
            dev = [torch.cat([torch.zeros(shift, dtype=t.dtype), t.reshape(-1)]).cuda()[shift:] for t in ins]
            out = torch.full((dims[0] * dims[1] + 64,), float("nan"), dtype=torch.bfloat16, device="cuda")
            h.launch(dims, dev, [out[shift:]])
            torch.cuda.synchronize()
            n = dims[0] * dims[1]
            assert_close(out[shift : shift + n].reshape(dims).cpu(), want, f"base shifted by {shift}")
            assert bool(out[:shift].isnan().all()) and bool(out[shift + n :].isnan().all())
    finally:
        c.close()


def test_lines_with_bases_on_sixteen_bytes():
    """Slots on whole lines of the tensor where its base lies on 16 bytes but off a line: taken from 128 lanes on; the
    guard elements around the result stay untouched."""
    from paper_2103_05288_amd import Context
    c = Context(0)
    c.test_option("non_temporal", 1)
    try:
        cfg = CONFIGS["C4"]
        pat = cfg.pattern()
        h = c.register(pat)
        for dims in ([600, 1023], [300, 2047], [257, 4098], [260, 5739]):
            ins = cfg.inputs(dims, seed=11)
            dev = [torch.cat([torch.zeros(24, dtype=t.dtype), t.reshape(-1)]).cuda()[24:] if t.numel() == dims[0] * dims[1] else t.cuda() for t in ins]
            dev = [torch.cat([torch.zeros(16, dtype=t.dtype), t.reshape(-1)]).cuda()[16:] if t.dtype == torch.bool else d for t, d in zip(ins, dev)]
            n = dims[0] * dims[1]
            out = torch.full((n + 64,), float("nan"), dtype=torch.bfloat16, device="cuda")
            h.launch(dims, dev, [out[8:]])
            torch.cuda.synchronize()
            want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0][0]
            assert_close(out[8 : 8 + n].reshape(dims).cpu(), want, f"{dims}")
            assert bool(out[:8].isnan().all()) and bool(out[8 + n :].isnan().all())
    finally:
        c.close()


@pytest.mark.parametrize("dims,kernel", [([34001, 248], "vec_nts"), ([9001, 1000], "vec_nts"), ([33001, 256], "vec_nts"), ([16501, 512], "vec_nt")])
def test_column_epilogue_versions_of_large_tensors(ctx, dims, kernel):
    """Large column reduces: non-temporal stores alone (row pieces of 64 bytes, rows that end inside a line), and with the
    loads (whole lines)."""
    plan = check(ctx, "C3", dims, seed=21)
    assert plan["kernels"][-1].endswith("k_col_epi2_" + kernel), plan["kernels"]
