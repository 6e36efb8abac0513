"""A predicate of sums of products: every kernel that evaluates it, and every copy in the one-pass kernel, decides alike."""
import re

import numpy as np
import pytest
import torch

from tests.util import device_code, run_gpu
from workloads import PatternBuilder

SCALE = (1.3, 3.7)


def _sums():
    """keep = 1.3 a + 3.7 b > thr; the kept 1.3 a, the slots, the count.  The first product is stored and the second is not,
    which is what a compiler that may fuse one of them goes by."""
    pb = PatternBuilder("sums")
    n = pb.dim()
    a, b, thr = pb.param("f32", [n]), pb.param("f32", [n]), pb.param("f32", [])
    p = pb.op("mul", a, pb.const(SCALE[0]), dims=[n])
    s = pb.op("add", p, pb.op("mul", b, pb.const(SCALE[1]), dims=[n]), dims=[n])
    keep = pb.op("gt", s, thr, dims=[n])
    pb.output(pb.compact(p, keep))
    pb.output(pb.compact_rank(keep, "i32"))
    pb.output(pb.compact_count(keep, "i64"))
    return pb.build()


def _difference():
    """keep = (a - 1.3 b) a - a b > thr, and an output of a sum that decides nothing."""
    pb = PatternBuilder("difference")
    n = pb.dim()
    a, b, thr = pb.param("f32", [n]), pb.param("f32", [n]), pb.param("f32", [])
    d = pb.op("sub", a, pb.op("mul", b, pb.const(SCALE[0]), dims=[n]), dims=[n])
    s = pb.op("sub", pb.op("mul", d, a, dims=[n]), pb.op("mul", a, b, dims=[n]), dims=[n])
    keep = pb.op("gt", s, thr, dims=[n])
    pb.output(pb.compact(d, keep))
    pb.output(pb.compact_count(keep, "i64"))
    return pb.build()


@pytest.mark.parametrize("make", [_sums, _difference])
def test_no_product_is_fused_into_a_sum(make, tmp_path):
    from paper_2103_05288_amd import Context
    ctx = Context(-1)
    code = device_code(ctx.register(make()).source, tmp_path / "pattern.co")
    ctx.close()
    kernels = [k for k in code if k.startswith("compact_") and k not in ("compact_clear", "compact_scan")]      # (these evaluate nothing)
    assert len(kernels) == 6                            # count and scatter of both widths, non-temporal stores, one pass
    for k in kernels:
        assert "v_mul_f32" in code[k] and not re.findall(r"v_(?:pk_)?(?:fma|mac|mad)\w*_f32", code[k]), k


@pytest.mark.gpu
def test_ties():
    """Thresholds that are sums themselves, at which the rounded products give another answer than either fused form: one
    element in 2304 lies on them.  Every version keeps the elements that the op list, one rounding an op, keeps."""
    from paper_2103_05288_amd import Context
    f = np.float32
    rng = np.random.RandomState(11)
    av, bv = rng.randn(48).astype(f), rng.randn(48).astype(f)
    A, B = np.meshgrid(av, bv)
    p, q = f(SCALE[0]) * A, f(SCALE[1]) * B
    s = p + q
    # (in 64 bits a product of two floats is exact, and only the sum is rounded before it is rounded to 32)
    fused = [(np.float64(f(SCALE[0])) * A + np.float64(q)).astype(f), (np.float64(p) + np.float64(f(SCALE[1])) * B).astype(f)]
    above = [np.sort(s[x > s]) for x in fused]
    assert min(len(t) for t in above) > 20
    thrs = [t[k * len(t) // 3] for t in above for k in range(3)]
    ctx = Context(0)
    pat = _sums()
    h = ctx.register(pat)
    kernels = set()
    for n in (20007, 40 * 4096 + 77):
        a, b = av[rng.randint(48, size=n)], bv[rng.randint(48, size=n)]
        first = f(SCALE[0]) * a
        for thr in thrs:
            keep = first + f(SCALE[1]) * b > thr
            rank = np.cumsum(keep) - 1
            for looks in (-1, 0, 500):
                ctx.test_option("compact_looks", looks)
                kernels.add(tuple(k.split("_k_compact_")[1] for k in h.plan([n])["kernels"]))
                got = run_gpu(h, pat, [n], [torch.from_numpy(a), torch.from_numpy(b), torch.tensor(thr)])
                assert int(got[2]) == keep.sum(), (n, thr, looks)
                assert np.array_equal(got[1].numpy(), rank) and np.array_equal(got[0].numpy()[:keep.sum()], first[keep]), (n, thr, looks)
    assert kernels == {("count_vec", "scan", "scatter_vec"), ("count_vec", "scatter_vec"), ("clear", "chain_vec")}
    ctx.close()
