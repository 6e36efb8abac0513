"""Row vectors in LDS under vector slots that start on boundaries of the tensor: every lane group, or every shift, has a
copy of its own."""
import re

import pytest
import torch

from oracle import run as oracle_run
from tests.util import assert_close, device_code, run_gpu, to_oracle_input
from workloads import PatternBuilder
from workloads.configs import CONFIGS


def _context(device):
    from paper_2103_05288_amd import Context
    c = Context(device)
    c.test_option("non_temporal", 1)          # the schedules of large launches
    return c


def test_space_for_the_copies():
    """fp32 vectors: as many copies as the block has lane groups, at most four; two-byte ones: where one is enough."""
    c = _context(-1)
    chain, norm = c.register(CONFIGS["C4"].pattern()), c.register(CONFIGS["C2"].pattern())
    for H, copies in ((131, 1), (385, 4), (415, 4), (1501, 4), (2047, 2), (5739, 1), (8191, 1)):
        p = chain.plan([200000, H])
        assert p["kernels"][0].endswith("_s_t") and p["lds_bytes"][0] == copies * ((4 * (H + 16) + 15) // 16 * 16), H
        p = norm.plan([200000, H])
        assert p["kernels"][0].endswith("_s_t") and p["lds_bytes"][0] == 3 * ((2 * (H + 16) + 15) // 16 * 16), H
    c.close()


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["C2", "C4"])
@pytest.mark.parametrize("H", [131, 385, 415, 769, 1023, 1501, 2047, 2501, 3071, 4097, 4099, 5739, 6143, 7801, 8191])
def test_results(name, H):
    c = _context(0)
    cfg = CONFIGS[name]
    h = c.register(cfg.pattern())
    for T in (1, 67, 1030):                   # (with 1030 rows of 4 lane groups and more, blocks past the last row)
        ins = cfg.inputs([T, H], seed=H + T)
        want = oracle_run(cfg.pattern(), [T, H], [to_oracle_input(t) for t in ins])[0]
        for k, (g, w) in enumerate(zip(run_gpu(h, cfg.pattern(), [T, H], ins), want)):
            assert_close(g, w, f"{name} {[T, H]} out{k}")
    c.close()


def _norm(vectors, dtype, loss=False, residual=False):
    """Rows (and a residual) scaled by their norm and by row vectors; with the sum of all squares beside it."""
    pb = PatternBuilder("norm")
    T, H = pb.dims(2)
    x = pb.cast(pb.param("bf16", [T, H]), "f32")
    if residual:
        x = pb.op("add", x, pb.cast(pb.param("bf16", [T, H]), "f32"))
    m = pb.reduce("sum", pb.op("mul", x, x), 1)
    y = pb.op("mul", x, pb.broadcast(pb.op("rsqrt", m), [T, H], [0]))
    for _ in range(vectors):
        v = pb.param(dtype, [H])
        y = pb.op("mul", y, pb.broadcast(v if dtype == "f32" else pb.cast(v, "f32"), [T, H], [1]))
    pb.output(pb.cast(y, "bf16"))
    if loss:
        pb.output(pb.reduce("sum", m, 0))
    return pb.build()


def test_reads_of_the_copies_are_lds_reads(tmp_path):
    """A pointer that is LDS on one path and null on another makes flat loads, which the row loads in flight wait with."""
    c = _context(-1)
    code = device_code(c.register(CONFIGS["C4"].pattern()).source, tmp_path / "pattern.co")
    staged = [k for k in code if k.startswith("row_vec_nv") and "_s" in k]
    assert len(staged) >= 9
    assert not [k for k in staged if "flat_load" in code[k] or "ds_read" not in code[k]]
    c.close()


def _plan(h, dims):
    """(kernel without its prefix, LDS, whether the grid was cut for shifted slots: unshifted ones run on an odd grid)"""
    p = h.plan(dims)
    return p["kernels"][0].split("_k_row_vec_")[1], p["lds_bytes"][0], p["grid"][0][0] % 2 == 0


def test_rows_whose_copies_do_not_fit():
    """fp32 vectors: shifted slots that read them from memory.  Two-byte ones: unshifted, and three slots a lane from eight rows a
    CU of a wide block on, which has the software pipeline; with copies that fit, two slots."""
    from paper_2103_05288_amd import Context
    c = Context(-1)
    two, three = c.register(_norm(2, "f32")), c.register(_norm(3, "f32"))
    for h, H in ((two, 8191), (two, 12289), (three, 5739), (three, 7001), (three, 12289)):
        assert _plan(h, [(1 << 27) // H, H]) == ("nv2w_t" if H > 6144 else "nv3_t", 0, True), H
    # where they do: wide blocks of large launches up to 64 KiB, others up to 48
    assert _plan(two, [9585, 7001]) == ("nv2w_s_t", 2 * 4 * 7020, True) and _plan(two, [599, 7001])[:2] == ("nv2w_t", 0)
    assert _plan(three, [30000, 4097])[:2] == ("nv2_t", 0) and _plan(c.register(_norm(1, "f32")), [30000, 4097])[1] == 4 * 4116
    # no more copies than 3.5 times a row: one vector four, two vectors none
    assert _plan(c.register(_norm(1, "bf16")), [300000, 1023])[1] == 2 * 1040 and _plan(two, [300000, 1023]) == ("nv2_s_t", 2 * 4 * 1040, False)
    norm = c.register(CONFIGS["C2"].pattern())
    for H in (12289, 13001, 15001, 16383):
        assert _plan(norm, [9000, H]) == ("nv3w", 0, False), H
        assert _plan(norm, [2047, H])[0] == "nv2w_t", H
    one = c.register(_norm(1, "bf16"))
    for H in (12289, 15001):
        assert _plan(one, [9000, H])[0] == "nv2w_s_t" and _plan(one, [9000, H + 1])[0] == "nv3w_s", H
    # rows on dword boundaries: shifted while the vectors are a small part of a row
    small = c.register(_norm(1, "bf16", residual=True))
    for h, shifted in ((small, True), (one, False), (norm, False)):
        assert _plan(h, [30000, 4098])[2] == shifted and _plan(h, [30000, 4097])[2]
    assert _plan(small, [30000, 7002])[2] and not _plan(small, [30000, 12290])[2]
    assert not _plan(one, [4500, 4097])[2] and _plan(one, [5500, 4097])[2]      # from 80 MiB on
    c.close()


def test_single_shape_modules_hold_the_kernel_of_misaligned_operands():
    """The one kernel of a module is the one that its plan takes, wherever the operands lie."""
    from paper_2103_05288_amd import Context
    c = Context(-1)
    for pat, dims in ((_norm(2, "f32"), [9585, 7001]), (_norm(2, "f32"), [9585, 8191]), (_norm(1, "bf16"), [9000, 12289]), (CONFIGS["C2"].pattern(), [9000, 7001]),
                      (CONFIGS["C2"].pattern(), [256, 8191]), (CONFIGS["C4"].pattern(), [100000, 1023])):
        h = c.register_static(pat, dims)
        for off in (0, 2, 16):
            p = h.plan(dims, inputs=[(1 << 20) + off] * len(pat.params), outputs=[(1 << 20) + off] * len(pat.outputs))
            assert re.search(r"\b" + p["kernels"][0] + r"\(", h.source), (dims, off, p["kernels"])
    c.close()


@pytest.mark.gpu
@pytest.mark.parametrize("vectors,dtype,H", [(2, "f32", 7001), (2, "f32", 8191), (3, "f32", 5739), (1, "f32", 8191), (2, "f32", 1023), (3, "bf16", 12289)])
def test_rows_off_the_limits(vectors, dtype, H):
    """Shifted slots and row vectors from memory, copies at the limits, and the pipelined wide version; operands on boundaries
    of slots and two bytes off, with the workspace that was asked for without them."""
    from paper_2103_05288_amd import Context
    c = Context(0)
    c.test_option("non_temporal", 1)
    pat = _norm(vectors, dtype, loss=vectors < 3)
    h = c.register(pat)
    T = 2100 if H > 12000 else 6000 if H == 1023 else 517      # (1023: more row groups than blocks, on either kind of operands)
    g = torch.Generator().manual_seed(H)
    ins = [torch.randn([T, H], generator=g).to(torch.bfloat16)] + [torch.randn([H], generator=g).to(torch.float32 if dtype == "f32" else torch.bfloat16) for _ in range(vectors)]
    want = oracle_run(pat, [T, H], [to_oracle_input(t) for t in ins])[0]
    single = c.register_static(pat, [T, H])
    ws = torch.empty(c.workspace_bytes(h.id, [T, H]) + 256, dtype=torch.uint8, device="cuda")
    for off in (0, 1):
        dev = []
        for t in ins:
            b = torch.zeros(t.numel() + 8, dtype=t.dtype, device="cuda")
            dev.append(b[off:off + t.numel()].view(t.shape).copy_(t))
        outs = [torch.full([T, H], float("nan"), dtype=torch.bfloat16, device="cuda")] + [torch.zeros([], device="cuda")] * (vectors < 3)
        print(f"[off the limits] {vectors} {dtype} {H} off={off}", flush=True)
        for handle in (h, single):
            handle.launch([T, H], dev, outs, workspace=ws, workspace_bytes=ws.numel() - 256)
            torch.cuda.synchronize()
            for k, (o, w) in enumerate(zip(outs, want)):
                assert_close(o.cpu(), w, f"{vectors} {dtype} {H} off={off} out{k} single={handle is single}")
                o.fill_(float("nan"))
    c.close()


def test_blocks_of_1024_threads_stage_from_six_rows_on():
    """One vector of 48 to 64 KiB; the launches are beyond 64 MiB on either side of the line."""
    from paper_2103_05288_amd import Context
    c = Context(-1)
    h = c.register(CONFIGS["C4"].pattern())
    line = 6 * 256                            # a block to a CU
    for H in (12289, 16001):
        assert [h.plan([T, H])["kernels"][0].endswith("_s_t") for T in (50, line - 1, line, 4 * line)] == [False, False, True, True], H
    c.close()


@pytest.mark.gpu
@pytest.mark.parametrize("vectors,dtype,H", [(1, "f32", 12289), (2, "bf16", 15001), (2, "f32", 7001)])
def test_workspace_of_the_most_rows_serves_fewer(vectors, dtype, H):
    """Fewer rows that do not stage have more blocks on a CU, and a partial result for each (plans only)."""
    from paper_2103_05288_amd import Context
    c = Context(0)
    h = c.register(_norm(vectors, dtype, loss=True))
    need = [c.workspace_bytes(h.id, [T, H]) for T in (100, 300, 512, 900, 1100, 1366, 1535, 1536, 2047, 2048, 3000, 9000, 60000)]
    assert need == sorted(need), need
    c.close()
