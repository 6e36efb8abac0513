"""Row vectors in LDS under vector slots that start on boundaries of the tensor: every lane group, or every shift, has a
copy of its own."""
import pytest

from oracle import run as oracle_run
from tests.util import assert_close, device_code, run_gpu, to_oracle_input
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


def test_reads_of_the_copies_are_lds_reads(tmp_path):
    """A pointer that is LDS on one path and null on another makes flat loads, which the row loads in flight wait with."""
    c = _context(-1)
    code = device_code(c.register(CONFIGS["C4"].pattern()).source, tmp_path / "pattern.co")
    staged = [k for k in code if k.startswith("row_vec_nv") and "_s" in k]
    assert len(staged) >= 9
    assert not [k for k in staged if "flat_load" in code[k] or "ds_read" not in code[k]]
    c.close()
