"""Helpers shared by the tests: comparator bars and the GPU / oracle drivers."""
import ctypes
import os
import re
import subprocess

import numpy as np
import torch

from workloads.configs import TORCH_DTYPE

# Parity bars, element-wise.
#  fp32 outputs:        |gpu - oracle| <= 1e-5 |oracle| + 1e-6
#  f16 / bf16 outputs:  the value is computed in fp32 (same 1e-5 / 1e-6 bar on the arithmetic) and then
#                       rounded ONCE to the storage type, which alone costs up to half a unit in the last
#                       place of that type:  |gpu - oracle| <= 0.5 ulp_T(x) + 1e-5 |oracle| + 1e-6.
#                       For f16 (half ulp <= 2^-11 |x|) this is inside the "rel 2e-3" bar; for bf16 the
#                       rounding alone reaches 2^-8 |x| = 3.9e-3 |x|, so no correctly rounded bf16 result can
#                       meet a blanket 2e-3: the bar keeps the arithmetic at the fp32 tolerance and adds
#                       exactly the unavoidable storage rounding, element by element.
#  integer outputs:     bit-exact
RTOL, ATOL = 1e-5, 1e-6
MANT_BITS = {"f16": (10, -14), "bf16": (7, -126)}    # explicit mantissa bits, minimum normal exponent


def ulp(x: np.ndarray, kind: str) -> np.ndarray:
    bits, emin = MANT_BITS[kind]
    ax = np.abs(x)
    e = np.floor(np.log2(np.where(ax > 0, ax, 1.0)))
    e = np.maximum(e, emin)
    return np.exp2(e - bits)


def to_oracle_input(t: torch.Tensor) -> np.ndarray:
    """Storage tensor -> numpy array the oracle takes (every f16/bf16 value is exact in float64)."""
    t = t.detach().cpu()
    if t.dtype in (torch.float16, torch.bfloat16, torch.float32):
        return t.to(torch.float64).numpy()
    return t.numpy()


def alloc_outputs(pattern, dims, device):
    outs = []
    for i in pattern.outputs:
        op = pattern.ops[i]
        outs.append(torch.empty(pattern.shape_of(i, dims), dtype=TORCH_DTYPE[op.dtype], device=device))
    return outs


def run_gpu(handle, pattern, dims, inputs, device="cuda", poison=True, workspace=None):
    # an empty operand still needs an address (the ABI refuses null pointers): any allocation will do
    dev_in = [t.to(device).contiguous() if t.numel() else torch.zeros(16, dtype=t.dtype, device=device) for t in inputs]
    outs = alloc_outputs(pattern, dims, device)
    if poison:
        for o in outs:
            if o.dtype.is_floating_point:
                o.fill_(float("nan"))
            else:
                o.fill_(-7 if o.dtype != torch.uint8 else 255)
    if workspace is None:
        need = handle.ctx.workspace_bytes(handle.id, dims)
        workspace = torch.empty(max(need, 16), dtype=torch.uint8, device=device)
    handle.launch(dims, dev_in, outs, workspace=workspace)
    torch.cuda.synchronize()
    return [o.cpu() for o in outs]


def assert_close(got: torch.Tensor, want: np.ndarray, what: str = ""):
    if not got.dtype.is_floating_point:
        g = got.numpy().astype(np.int64)
        w = np.asarray(want).astype(np.int64)
        assert g.shape == w.shape, (what, g.shape, w.shape)
        bad = np.nonzero(g != w)
        assert bad[0].size == 0, f"{what}: {bad[0].size} index mismatches, first at {[b[0] for b in bad]}"
        return
    g = got.to(torch.float64).numpy()
    w = np.asarray(want, dtype=np.float64)
    assert g.shape == w.shape, (what, g.shape, w.shape)
    err = np.abs(g - w)
    lim = RTOL * np.abs(w) + ATOL
    if got.dtype in (torch.float16, torch.bfloat16):
        kind = "f16" if got.dtype == torch.float16 else "bf16"
        lim = lim + 0.5 * ulp(np.maximum(np.abs(g), np.abs(w)), kind)
    bad = ~(err <= lim)          # NaN-safe: a NaN on either side fails
    if bad.any():
        idx = np.unravel_index(np.argmax(np.where(bad, err - lim, -np.inf)), g.shape)
        raise AssertionError(f"{what}: {int(bad.sum())} of {g.size} elements outside the {got.dtype} bar; "
                             f"worst at {tuple(int(i) for i in idx)}: gpu={g[idx]!r} oracle={w[idx]!r} "
                             f"err={err[idx]:.3e} limit={lim[idx]:.3e}")


def device_code(source: str, path) -> dict:
    """Kernel name (without the pattern's prefix) -> its instructions, as the library's own compiler call builds them."""
    rtc = ctypes.CDLL("libhiprtc.so")
    flags = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-value",
             "-fno-slp-vectorize", "-fno-vectorize"]
    prog, size = ctypes.c_void_p(), ctypes.c_size_t()
    assert rtc.hiprtcCreateProgram(ctypes.byref(prog), source.encode(), b"pattern.hip", 0, None, None) == 0
    assert rtc.hiprtcCompileProgram(prog, len(flags), (ctypes.c_char_p * len(flags))(*[f.encode() for f in flags])) == 0
    assert rtc.hiprtcGetCodeSize(prog, ctypes.byref(size)) == 0
    code = ctypes.create_string_buffer(size.value)
    assert rtc.hiprtcGetCode(prog, code) == 0
    rtc.hiprtcDestroyProgram(ctypes.byref(prog))
    path = str(path)
    with open(path, "wb") as f:
        f.write(code.raw)
    text = subprocess.run([os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump"), "-d", path], check=True,
                          capture_output=True, text=True).stdout
    return {m[1]: m[2] for m in re.finditer(r"^[0-9a-f]+ <\w+?_k_(\w+)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", text, re.M | re.S)}


def host_build(body: str, path):
    """A shared library, for the CPU, of index arithmetic cut out of the device header."""
    head = """typedef long long i64; typedef unsigned u32; typedef unsigned long long u64;
#define DISC_DEV static inline
#define __builtin_amdgcn_readfirstlane(x) (x)
static struct { unsigned x, y, z; } blockIdx, gridDim;
"""
    src, lib = str(path) + ".cpp", str(path) + ".so"
    with open(src, "w") as f:
        f.write(head + body)
    subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-shared", "-fPIC", "-o", lib, src], check=True)
    return ctypes.CDLL(lib)


def device_header(first: str, last: str) -> str:
    """The text of the device header from the line that starts with `first` to the closing brace of the function `last`."""
    import paper_2103_05288_amd
    with open(os.path.join(os.path.dirname(paper_2103_05288_amd.__file__), "csrc", "disc_device.h")) as f:
        text = f.read()
    return re.search("^" + re.escape(first) + r".*?\b" + last + r"\(.*?^}$", text, re.M | re.S)[0]
