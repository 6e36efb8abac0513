"""Performance cases: the fused patterns a program runs through this library, at the sizes it meets.

A program registers each pattern once, keeps the handle, and then launches it at whatever shape
the next batch has; that launch -- `launch(dims, inputs, outputs, workspace=...)` of a pattern or of
an op graph -- is what one pass is.  Tensors, results and the workspace are the caller's and are
allocated beforehand (the library allocates nothing).  Forward: bias + GELU, masked attention
softmax, residual + LayerNorm, a mixed chain, the normaliser of a cross-entropy loss; backward:
LayerNorm with its weight gradients, GELU with its bias gradient; and centring of columns, Unique of
sorted keys, a softmax over a transposed operand as an op graph of two patterns.
"""
import math

import torch

import paper_2103_05288_amd as pkg
from workloads import PatternBuilder
from workloads import configs, extras

MAX_ELEMENTS = 1 << 28          # of one full-size operand, the largest that draw() gives


def _transposed_softmax():
    """Row softmax of a transposed operand: not one pattern, but a tile transpose and a row reduce."""
    pb = PatternBuilder("transposed_softmax")
    P, Q = pb.dims(2)
    x = pb.cast(pb.transpose(pb.param("bf16", [P, Q]), (1, 0)), "f32")
    e = pb.op("exp", pb.op("sub", x, pb.broadcast(pb.reduce("max", x, 1), [Q, P], [0])))
    pb.output(pb.cast(pb.op("div", e, pb.broadcast(pb.reduce("sum", e, 1), [Q, P], [0])), "bf16"))
    return pb.build()


# kind -> (op list, registered as an op graph)
_KINDS = {
    "bias_gelu": (configs.c0_pattern, False),
    "attention_softmax": (configs.c1_pattern, False),
    "residual_layernorm": (configs.c2_pattern, False),
    "center_columns": (configs.c3_pattern, False),
    "mixed_chain": (configs.c4_pattern, False),
    "layernorm_backward": (extras.layernorm_backward_graph, False),
    "gelu_backward": (extras.gelu_backward_bias_gradient, False),
    "logsumexp": (extras.logsumexp_with_total_and_amax, False),
    "unique": (extras.unique_of_sorted, False),
    "transposed_softmax": (_transposed_softmax, True),
}

_context = None
_handles = {}


def _pattern(case):
    make = _KINDS[case["kind"]][0]
    return make(case["dtype"]) if case["kind"] == "unique" else make()


def _handle(case):
    """The registered pattern: compiled once in a program's life, whatever shapes follow."""
    global _context
    key = (case["kind"], case.get("dtype"))
    if key not in _handles:
        if _context is None:
            _context = pkg.Context(torch.cuda.current_device())
        p = _pattern(case)
        _handles[key] = (p, (_context.register_graph if _KINDS[case["kind"]][1] else _context.register)(p))
    return _handles[key]


def listed():
    return [
        # One decoding step or a short sentence through the activation of a feed-forward layer: the
        # time of a call, not of its memory traffic.
        {"name": "bias_gelu_37x768", "kind": "bias_gelu", "T": 37, "H": 768},
        # Attention probabilities of a short batch, sequence length off every power of two.
        {"name": "attention_softmax_s197", "kind": "attention_softmax", "B": 8, "NH": 12, "S": 197},
        # Residual + LayerNorm over the tokens of a batch of variable-length sentences.
        {"name": "layernorm_16007x768", "kind": "residual_layernorm", "T": 16007, "H": 768},
        # Per-feature centring of one small batch and of a whole data set.
        {"name": "center_700x1024", "kind": "center_columns", "T": 700, "C": 1024},
        {"name": "center_65536x1024", "kind": "center_columns", "T": 65536, "C": 1024},
        # The long chain: many short odd rows (features of an embedding), and long odd rows.
        {"name": "chain_300007x93", "kind": "mixed_chain", "T": 300007, "H": 93},
        {"name": "chain_46773x5739", "kind": "mixed_chain", "T": 46773, "H": 5739},
        # Training: input and weight gradients of LayerNorm at a transformer's hidden size.
        {"name": "layernorm_backward_32768x1024", "kind": "layernorm_backward", "T": 32768, "H": 1024},
        # Training: GELU backward with the bias gradient at a wide feed-forward layer (4 x 4096).
        {"name": "gelu_backward_8192x16384", "kind": "gelu_backward", "T": 8192, "H": 16384},
        # Cross-entropy normaliser over a vocabulary: rows too long to stay in one block's registers.
        {"name": "logsumexp_4096x32000", "kind": "logsumexp", "T": 4096, "H": 32000},
        # Distinct keys of a sorted column with the index of every row's key (ids of a sparse batch).
        {"name": "unique_i32_33555445", "kind": "unique", "N": 33555445, "dtype": "i32"},
        # Softmax along the other axis of a score matrix: transpose kernel + row kernel.
        {"name": "transposed_softmax_6000x4097", "kind": "transposed_softmax", "P": 6000, "Q": 4097},
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(2.0 ** rng.uniform(math.log2(lo), math.log2(hi))))))


def draw(rng):
    kind = rng.choice(sorted(_KINDS))
    if kind == "attention_softmax":
        return {"kind": kind, "B": rng.randint(1, 16), "NH": rng.choice((8, 12, 16)), "S": rng.randint(16, 512)}
    if kind == "unique":
        return {"kind": kind, "N": _log(rng, 1 << 10, 1 << 25), "dtype": rng.choice(("i32", "i32", "i64", "f32"))}
    if kind == "transposed_softmax":
        return {"kind": kind, "P": _log(rng, 64, 8192), "Q": _log(rng, 64, 8192)}
    # (name of the long dimension's partner, its range, range of the rows, most elements)
    inner, h_lo, h_hi, t_lo, t_hi, most = {
        "bias_gelu": ("H", 256, 4096, 1, 4096, 1 << 24),
        "residual_layernorm": ("H", 256, 8192, 32, 32768, 1 << 26),
        "center_columns": ("C", 64, 4096, 1, 65536, 1 << 26),
        "mixed_chain": ("H", 64, 8192, 1, 1 << 20, MAX_ELEMENTS),
        "layernorm_backward": ("H", 128, 8192, 64, 65536, 1 << 26),
        "gelu_backward": ("H", 512, 16384, 64, 32768, 1 << 27),
        "logsumexp": ("H", 1000, 64000, 64, 16384, 1 << 27),
    }[kind]
    h = _log(rng, h_lo, h_hi)
    return {"kind": kind, "T": _log(rng, t_lo, min(t_hi, most // h)), inner: h}


def _dims(case):
    return [int(case[k]) for k in ("B", "NH", "T", "N", "P", "Q", "C", "H", "S") if k in case]


def _normal(shape, dtype, g, mean=0.0, std=1.0):
    return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(mean, std, generator=g).to(dtype)


def _inputs(case, seed):
    kind, dims = case["kind"], _dims(case)
    for name, config in zip(("bias_gelu", "attention_softmax", "residual_layernorm", "center_columns", "mixed_chain"),
                            ("C0", "C1", "C2", "C3", "C4")):
        if kind == name:
            return configs.CONFIGS[config].inputs(dims, seed, "cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    bf = torch.bfloat16
    if kind == "layernorm_backward":        # activations, incoming gradient, gamma
        return [_normal(dims, bf, g), _normal(dims, bf, g, 0.0, 0.1), _normal(dims[1:], torch.float32, g, 1.0, 0.1)]
    if kind == "gelu_backward":             # incoming gradient, pre-activations, bias
        return [_normal(dims, bf, g, 0.0, 0.1), _normal(dims, bf, g), _normal(dims[1:], torch.float32, g, 0.0, 0.02)]
    if kind == "logsumexp":                 # logits
        return [_normal(dims, bf, g, 0.0, 2.0)]
    if kind == "transposed_softmax":
        return [_normal(dims, bf, g)]
    # unique: sorted keys, four equal ones in a row on average
    n = dims[0]
    keys = torch.randint(0, max(1, n // 4), (n,), generator=g, device="cuda", dtype=torch.int32)
    return [torch.sort(keys)[0].to(configs.TORCH_DTYPE[case["dtype"]])]


def prepare(case, seed):
    pattern, handle = _handle(case)
    dims = _dims(case)
    inputs = _inputs(case, seed)
    # (zeros: of Unique's first result only the elements in front of the count are written)
    outputs = [torch.zeros(pattern.shape_of(i, dims), dtype=configs.TORCH_DTYPE[pattern.ops[i].dtype], device="cuda")
               for i in pattern.outputs]
    if _KINDS[case["kind"]][1]:
        need = handle.workspace_bytes(dims)
    else:
        need = handle.ctx.workspace_bytes(handle.id, dims)
    return {"handle": handle, "dims": dims, "inputs": inputs, "outputs": outputs,
            "workspace": torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")}


def run(state):
    state["handle"].launch(state["dims"], state["inputs"], state["outputs"], workspace=state["workspace"])
    return state["outputs"]


#: arithmetic operations per element of the iteration space, counted from the op lists
_FLOPS = {"bias_gelu": 11, "attention_softmax": 6, "residual_layernorm": 8, "center_columns": 2, "mixed_chain": 9,
          "layernorm_backward": 17, "gelu_backward": 9, "logsumexp": 5, "unique": 2, "transposed_softmax": 4}


def work(case):
    pattern = _pattern(case)
    dims = _dims(case)
    total = configs.algorithmic_bytes(pattern, dims)
    elements = math.prod(dims)
    if case["kind"] == "attention_softmax":
        elements *= dims[-1]
    if case["kind"] == "unique":            # the distinct keys, not the buffer that could hold as many as there are rows
        size = configs.DTYPE_BYTES[case["dtype"]]
        m = max(1, dims[0] // 4)
        total -= int(size * (dims[0] - m * (1.0 - math.exp(-dims[0] / m))))
    return {"bytes": total, "flops": _FLOPS[case["kind"]] * elements}


def tolerance(case):
    return {
        "bias_gelu": {"rel": 1e-6, "max": 1e-5},
        "attention_softmax": {"rel": 1e-3, "max": 5e-3},
        "residual_layernorm": {"rel": 7e-3, "max": 2e-2},
        "center_columns": {"rel": 1e-6, "max": 1e-5},
        "mixed_chain": {"rel": 7e-3, "max": 2e-2},
        "layernorm_backward": {"rel": 7e-3, "max": 2e-2},
        "gelu_backward": {"rel": 7e-3, "max": 2e-2},
        "logsumexp": {"rel": 1e-6, "max": 1e-5},
        "unique": "exact",
        "transposed_softmax": {"rel": 7e-3, "max": 2e-2},
    }[case["kind"]]


def exact(case, seed):
    kind, dims = case["kind"], _dims(case)
    inputs = _inputs(case, seed)
    if kind == "unique":
        values, rank = torch.unique_consecutive(inputs[0], return_inverse=True)
        padded = torch.zeros_like(inputs[0])
        padded[: values.numel()] = values
        return [padded, rank.to(torch.int32), torch.tensor(values.numel(), dtype=torch.int64, device="cuda")]
    d = [t.double() if t.is_floating_point() else t for t in inputs]
    if kind == "bias_gelu":
        x, b, r = d
        u = x + b
        return [0.5 * u * (1.0 + torch.tanh(0.7978845608028654 * (u + 0.044715 * u ** 3))) + r]
    if kind == "attention_softmax":
        return [torch.softmax(d[0] * 0.125 + d[1], -1)]
    if kind == "residual_layernorm":
        x, r, b, gamma, beta = d
        v = x + r + b
        c = v - v.mean(1, keepdim=True)
        return [c * torch.rsqrt((c * c).mean(1, keepdim=True) + 1e-5) * gamma + beta]
    if kind == "center_columns":
        s = d[0].sum(0)
        return [s, s / dims[0], d[0] - s / dims[0]]
    if kind == "mixed_chain":
        x, mask, bH, cT = d
        b = x + bH + cT
        e = torch.exp(b - b.amax(1, keepdim=True))
        s = e.sum(1, keepdim=True)
        return [torch.where(mask != 0, 0.0, e / s) + x * torch.rsqrt(s)]
    if kind == "layernorm_backward":
        x, dy, gamma = d
        c = x - x.mean(1, keepdim=True)
        rstd = torch.rsqrt((c * c).mean(1, keepdim=True) + 1e-5)
        xhat = c * rstd
        g = dy * gamma
        dx = (g - g.mean(1, keepdim=True) - xhat * (g * xhat).mean(1, keepdim=True)) * rstd
        return [dx, (dy * xhat).sum(0), dy.sum(0)]
    if kind == "gelu_backward":
        dy, x, b = d
        a = 1.702 * (x + b)
        s = torch.sigmoid(a)
        dx = dy * s * (1.0 + a * (1.0 - s))
        return [dx, dx.sum(0)]
    if kind == "logsumexp":
        lse = torch.logsumexp(d[0], 1)
        return [lse, lse.sum(), d[0].abs().amax()]
    return [torch.softmax(d[0].T, 1)]
