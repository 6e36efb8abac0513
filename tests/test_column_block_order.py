"""Column reduces in two and three launches whose blocks come in lists of neighbouring tiles (rows that do not end on cache
lines, or pieces of a row shorter than one) or one by one."""
import ctypes

import pytest

from oracle import run as oracle_run
from tests.util import assert_close, device_header, host_build, run_gpu, to_oracle_input
from workloads import PatternBuilder
from workloads.configs import CONFIGS


@pytest.fixture(scope="module")
def place(tmp_path_factory):
    """col_place of the device header, built for the CPU: the (tile, row range) of every block, in the order of the blocks"""
    lib = host_build(device_header("template <bool BACK>", "col_place") + """
extern "C" void place(int back, int lists, unsigned tiles, unsigned ranges, i64* out) {
  gridDim.x = tiles;
  gridDim.y = ranges;
  for (blockIdx.y = 0; blockIdx.y < ranges; ++blockIdx.y)
    for (blockIdx.x = 0; blockIdx.x < tiles; ++blockIdx.x, out += 2)
      if (back) col_place<true>(lists != 0, out[0], out[1]);
      else col_place<false>(lists != 0, out[0], out[1]);
}
""", tmp_path_factory.mktemp("place") / "columns")

    def call(back, lists, tiles, ranges):
        out = (ctypes.c_int64 * (2 * tiles * ranges))()
        lib.place(back, lists, tiles, ranges, out)
        return list(zip(out[0::2], out[1::2]))
    return call


@pytest.mark.parametrize("lists", [0, 1])
def test_every_block_once(place, lists):
    for tiles, ranges in [(1, 1), (1, 9), (3, 5), (11, 32), (64, 8), (7, 1), (5, 13), (1000, 33)]:
        forward, back = place(0, lists, tiles, ranges), place(1, lists, tiles, ranges)
        every = [(t, r) for t in range(tiles) for r in range(ranges)]
        assert sorted(forward) == every and sorted(back) == every
        if lists:                 # an XCD (blocks i mod 8): neighbours one after the other, and the same ones backwards in the second launch
            for x in range(8):
                at = [r * tiles + t for t, r in forward[x::8]]
                assert at == list(range(at[0], at[0] + len(at))) if at else True
                assert back[x::8] == forward[x::8][::-1]
        else:
            assert back == [(t, ranges - 1 - r) for t, r in forward]


@pytest.mark.gpu
def test_results():
    """Every remainder of the blocks mod 8, a last tile of one column, whole lines beside it; three launches (long, narrow)."""
    from paper_2103_05288_amd import Context
    ctx = Context(0)
    try:
        pat = CONFIGS["C3"].pattern()
        h = ctx.register(pat)
        launches = set()
        for dims in ([6000, 321], [9000, 193], [5000, 256], [2600, 449], [1601, 700], [4100, 513], [2000, 577], [3300, 1000], [2049, 1024],
                     [300, 4001], [40000, 65], [65536, 70], [70001, 33], [2000000, 3]):
            ins = CONFIGS["C3"].inputs(dims, seed=sum(dims))
            launches.add(h.plan(dims)["n_launches"])
            want = oracle_run(pat, dims, [to_oracle_input(t) for t in ins])[0]
            for k, (g, w) in enumerate(zip(run_gpu(h, pat, dims, ins), want)):
                assert_close(g, w, f"{dims} out{k}")
        assert launches >= {2, 3}
        # batches: two-byte elements, a maximum over the middle axis
        pb = PatternBuilder("batched")
        B, T, C = pb.dims(3)
        x = pb.cast(pb.param("bf16", [B, T, C]), "f32")
        m = pb.reduce("max", x, 1)
        pb.output(m)
        pb.output(pb.op("sub", x, pb.broadcast(m, [B, T, C], [0, 2])))
        pat = pb.build()
        h = ctx.register(pat)
        import torch
        gen = torch.Generator().manual_seed(3)
        for dims in ([3, 1500, 515], [7, 2100, 131], [2, 4000, 1001]):
            t = torch.randn(dims, generator=gen).to(torch.bfloat16)
            want = oracle_run(pat, dims, [to_oracle_input(t)])[0]
            for k, (g, w) in enumerate(zip(run_gpu(h, pat, dims, [t]), want)):
                assert_close(g, w, f"{dims} out{k}")
    finally:
        ctx.close()
