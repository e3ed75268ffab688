"""The work that a user of this package has it do, as cases whose time can be measured.

A decoding model calls vq_gemv and vq_gemv_multi for every linear layer and token, a prompt goes through vq_gemm (or
vq_dequant and a product of the caller's own), and a quantizer calls vq_assign and vq_quantize_columns for every layer of
the model that it encodes.  The listed cases are these calls on the layers of the benchmark configurations
(vq_synth.CONFIGS) and on the parameter settings that the benchmark and the tests use; draw() gives the same kinds of calls
over the sizes and options in between and around them, ragged ones included.
"""
import math

import numpy as np
import torch

import paper_2409_17066_amd as vq
from vq_synth import VQLayer, index_bits, row_stride_bytes

# (v, k, k_res, percentage of outlier columns, k_out, codebook groups): what layers are stored with.  Outlier vectors have
# four elements throughout.
SETTINGS = {
    "v6": (6, 4096, 0, 0, 0, 1),                # 2 bits a weight
    "v6 k256": (6, 256, 0, 0, 0, 1),
    "v6 + 4096": (6, 4096, 4096, 0, 0, 1),      # 4 bits a weight
    "v6 + 256, outliers": (6, 4096, 256, 1, 4096, 1),
    "v6, 4 groups": (6, 4096, 0, 0, 0, 4),
    "v8": (8, 65536, 0, 0, 0, 1),               # 2 bits a weight, a table larger than LDS
    "v12 + 4096": (12, 4096, 4096, 0, 0, 1),
    "v12 + 4096, outliers, 4 groups": (12, 4096, 4096, 1, 8192, 4),    # 2.26 bits a weight
    "v4 k256": (4, 256, 0, 0, 0, 1),
    "v2 k16": (2, 16, 0, 0, 0, 1),
}


def layer_of(setting, out_features, in_features, orientation=0, permute=False):
    """The fields of a case that say how a layer is stored."""
    v, k, k_res, percent, k_out, groups = SETTINGS[setting]
    n_out = int(in_features * percent / 100 / 4 + 0.5) * 4
    positions = in_features - n_out if orientation else -(-(in_features - n_out) // v)
    group_vectors = -(-positions // (8 * groups)) * 8 if groups > 1 else 0
    return {"out": out_features, "in": in_features, "v": v, "k": k, "k_res": k_res, "outliers": n_out, "k_out": k_out if n_out else 0,
            "group_vectors": group_vectors, "orientation": orientation, "permute": permute}


def listed():
    return [
        # The smallest call: configuration 0, one activation row.  Launch and host time are all of it.
        dict(name="decode tiny", op="gemv", batch=1, workspace=False, **layer_of("v6 k256", 256, 384)),
        # One projection of a 2-bit 7B-shaped model, one activation row: configuration 1, what the benchmark quotes.
        dict(name="decode up projection", op="gemv", batch=1, workspace=False, **layer_of("v6", 11008, 4096)),
        # A whole 7B-shaped decoder layer with residual tables (configuration 2): q, k, v in one call, o, gate and up in one
        # call, down.  One row: a single user's decoding; sixteen: a batch of users or drafted tokens.
        dict(name="decoder layer, 1 row", op="decoder", hidden=4096, inter=11008, k_res=4096, orientation=0, batch=1),
        dict(name="decoder layer, 16 rows", op="decoder", hidden=4096, inter=11008, k_res=4096, orientation=0, batch=16),
        # The largest decode call: the 70B-shaped down projection with outlier columns (configuration 3).
        dict(name="decode 70B down projection", op="gemv", batch=1, workspace=True, **layer_of("v6 + 256, outliers", 8192, 28672)),
        # The 2.26-bit 7B setting: two tables of 12-element vectors, four codebook groups, outlier columns wherever the
        # Hessian put them (a column permutation), with the workspace that a serving loop keeps.
        dict(name="decode 2.26 bit", op="gemv", batch=1, workspace=True, **layer_of("v12 + 4096, outliers, 4 groups", 11008, 4096, permute=True)),
        # Vectors down the output dimension, as the quantizer below writes them; a few rows.
        dict(name="decode orientation 1", op="gemv", batch=4, workspace=True, **layer_of("v6", 11008, 4096, orientation=1)),
        # Prompts.  Configuration 4 at its largest token count, with the workspace; and a prompt of ragged length on the
        # 7B-shaped projection without one.
        dict(name="prefill 2048 tokens", op="gemm", tokens=2048, workspace=True, **layer_of("v8", 8192, 8192)),
        dict(name="prefill 509 tokens", op="gemm", tokens=509, workspace=False, **layer_of("v6", 11008, 4096)),
        # Restoring a layer's weights for a product of the caller's own.
        dict(name="dequant", op="dequant", **layer_of("v6 + 4096", 11008, 4096)),
        # Encoding: nearest centroids of a whole matrix, and Algorithm 1's column loop on a square projection.
        dict(name="assign", op="assign", rows=11008, cols=4096, v=6, k=4096, base=False, orientation=0),
        dict(name="quantize columns", op="quantize", rows=4096, cols=4096, v=6, k=4096, k_res=0, block=128),
    ]


def _size(rng, low, high, multiple=1):
    """A size between low and high, even over its logarithm, rounded to a multiple."""
    return max(low, int(math.exp(rng.uniform(math.log(low), math.log(high))) / multiple + 0.5) * multiple)


def _columns(rng, low, high):
    """Input widths: models' are multiples of 64; slices and tests have any."""
    return _size(rng, low, high, rng.choice((64, 64, 64, 8, 1)))


def draw(rng):
    op = rng.choice(("gemv", "gemv", "gemv", "decoder", "gemm", "gemm", "dequant", "assign", "quantize"))
    orientation = rng.choice((0, 0, 1))
    if op == "decoder":
        hidden = _size(rng, 512, 5120, 64)
        return {"op": op, "hidden": hidden, "inter": int(hidden * rng.uniform(2.5, 4.0) / 64) * 64, "k_res": rng.choice((0, 256, 4096)),
                "orientation": orientation, "batch": _size(rng, 1, 16)}
    if op == "assign":
        v, k = rng.choice(((6, 4096), (6, 4096), (6, 256), (8, 65536), (12, 4096), (4, 256), (2, 16)))
        cols = _columns(rng, 256, 8192)
        most = min(11008, 11008 * 4096 * 4096 // (k * cols))
        return {"op": op, "rows": _size(rng, min(64, most // 2), most), "cols": cols, "v": v, "k": k, "base": rng.choice((False, True)),
                "orientation": orientation}
    if op == "quantize":
        v, k, k_res = rng.choice(((6, 4096, 0), (6, 4096, 0), (6, 4096, 256), (8, 256, 256), (12, 4096, 0), (4, 256, 0)))
        return {"op": op, "rows": _size(rng, 128, 3072), "cols": _size(rng, 128, 3072, rng.choice((64, 1))), "v": v, "k": k, "k_res": k_res,
                "block": 128}
    setting = rng.choice(sorted(SETTINGS))
    permute = bool(SETTINGS[setting][3]) and rng.random() < 0.5
    if op == "gemm":
        in_features = _size(rng, 512, 11008, rng.choice((256, 256, 256, 8)))
        layer = layer_of(setting, _size(rng, 256, 11008, rng.choice((64, 1))), in_features, orientation, permute)
        workspace = rng.choice((True, True, False))
        # (long prompts are served with a workspace, which takes widths in multiples of 256)
        return {"op": op, "tokens": _size(rng, 17, 2048 if workspace and in_features % 256 == 0 else 512), "workspace": workspace, **layer}
    in_features = _columns(rng, 256, 28672)
    layer = layer_of(setting, _size(rng, 256, min(14336, 8192 * 28672 // in_features), rng.choice((64, 1))), in_features, orientation, permute)
    if op == "dequant":
        return {"op": op, **layer}
    return {"op": op, "batch": _size(rng, 1, 16), "workspace": rng.choice((False, True)), **layer}


# ---- inputs -----------------------------------------------------------------------------------------------------------
def _normal(rng, shape, sigma):
    return (rng.standard_normal(shape, dtype=np.float32) * sigma).astype(np.float16)


def _stream(rng, streams, per_stream, k):
    """A packed index stream.  Every table has a power of two of entries, so uniform indices are uniform bits."""
    stride = row_stride_bytes(per_stream, index_bits(k))
    return np.frombuffer(rng.bytes(streams * stride), dtype=np.uint8).reshape(streams, stride).copy()


def _fields(case):
    return VQLayer("layer", case["out"], case["in"], case["v"], case["k"], case["k_res"], case["outliers"], 4 if case["outliers"] else 0,
                   case["k_out"], case["group_vectors"], case["orientation"])


def _layer(case, rng):
    """One layer on the GPU: Gaussian tables, uniform indices, scale and bias, as vq_synth makes them."""
    L = _fields(case)
    L.codebook = _normal(rng, (L.n_groups * L.k, L.v), 0.02)
    L.idx = _stream(rng, L.streams, L.vectors_per_row, L.k)
    if L.k_res:
        L.codebook_res = _normal(rng, (L.n_groups * L.k_res, L.v), 0.005)
        L.idx_res = _stream(rng, L.streams, L.vectors_per_row, L.k_res)
    if L.n_outlier_cols:
        L.codebook_out = _normal(rng, (L.k_out, L.v_out), 0.1)
        L.idx_out = _stream(rng, L.outlier_streams, L.outlier_vectors_per_row, L.k_out)
    if case["permute"]:
        L.col_perm = rng.permutation(L.in_features).astype(np.int32)
    L.scale = rng.uniform(0.5, 1.5, L.out_features).astype(np.float16)
    L.bias = _normal(rng, L.out_features, 0.01)
    return vq.DeviceLayer(L)


def _activations(layer, rows, generator, pitch=None):
    """fp16 N(0, 1), the outlier columns ten times larger."""
    n = layer.in_features
    x = torch.randn((rows, pitch or n), dtype=torch.float32, device="cuda", generator=generator)
    if layer.n_outlier_cols:
        cols = torch.arange(layer.n_outlier_cols) if layer.col_perm is None else torch.from_numpy(layer.col_perm[: layer.n_outlier_cols].astype(np.int64))
        x[:, cols.cuda()] *= 10.0
    return x.half()[:, :n]


def _inverse_factor(n, generator):
    """The upper Cholesky factor of the inverse of a layer's Hessian, fp32: activations whose neighbouring channels are
    correlated and of which 3 % are ten times larger, 1 % of the mean diagonal as damping (as vq_synth.make_hessian)."""
    at = torch.arange(n, device="cuda")
    lag = (at[None, :] - at[:, None]).clamp(min=0)
    mix = torch.where(at[None, :] >= at[:, None], 0.6 ** lag.float(), torch.zeros((), device="cuda"))
    X = torch.randn((2 * n, n), device="cuda", generator=generator) @ mix
    X *= 1.0 + 9.0 * (torch.rand(n, device="cuda", generator=generator) > 0.97)
    H = (X.T.contiguous() @ X / (2 * n)).double()
    H.diagonal().add_(0.01 * H.diagonal().mean())
    # H = R R^T with R upper triangular, from the Cholesky factor of H in reversed order; the factor asked for is R^-1
    R = torch.linalg.cholesky(H.flip(0, 1)).flip(0, 1)
    return torch.linalg.solve_triangular(R, torch.eye(n, dtype=torch.float64, device="cuda"), upper=True).float().contiguous()


def prepare(case, seed):
    rng, generator = np.random.default_rng(seed), torch.Generator(device="cuda").manual_seed(seed)
    op = case["op"]
    if op == "assign":
        W = torch.randn((case["rows"], case["cols"]), device="cuda", generator=generator) * 0.02
        B = None
        if case["base"]:                       # the second stage: what the first one restored, and a table for what it left
            B = (W + 0.005 * torch.randn(W.shape, device="cuda", generator=generator)).half()
        C = torch.from_numpy(_normal(rng, (case["k"], case["v"]), 0.005 if case["base"] else 0.02)).cuda()
        return {"op": op, "W": W.half(), "B": B, "C": C, "orientation": case["orientation"]}
    if op == "quantize":
        W = (torch.randn((case["rows"], case["cols"]), device="cuda", generator=generator) * 0.02).half().float()
        C = torch.from_numpy(_normal(rng, (case["k"], case["v"]), 0.02)).cuda()
        R = torch.from_numpy(_normal(rng, (case["k_res"], case["v"]), 0.005)).cuda() if case["k_res"] else None
        return {"op": op, "W": W, "Hinv": _inverse_factor(case["cols"], generator), "C": C, "R": R, "block": case["block"]}
    if op == "decoder":
        h, i = case["hidden"], case["inter"]
        shapes = {"q": (h, h), "k": (h, h), "v": (h, h), "o": (h, h), "gate": (i, h), "up": (i, h), "down": (h, i)}
        state = {"op": op}
        for name, (m, n) in shapes.items():
            state[name] = _layer({"out": m, "in": n, "v": 6, "k": 4096, "k_res": case["k_res"], "outliers": 0, "k_out": 0, "group_vectors": 0,
                                  "orientation": case["orientation"], "permute": False}, rng)
        for name, of in (("x", "q"), ("attention", "o"), ("x_mlp", "up"), ("hidden", "down")):
            state[name] = _activations(state[of].layer, case["batch"], generator)
        for name in ("o", "down"):
            state["ws_" + name] = _gemv_workspace(state[name], case["batch"])
        return state
    layer = _layer(case, rng)
    state = {"op": op, "layer": layer}
    if op == "gemv":
        state["x"] = _activations(layer.layer, case["batch"], generator)
        state["workspace"] = _gemv_workspace(layer, case["batch"]) if case["workspace"] else None
    elif op == "gemm":
        state["x"] = _activations(layer.layer, case["tokens"], generator, pitch=-(-case["in"] // 8) * 8)
        size = vq.vq_gemm_fast_workspace_bytes(layer.desc, case["tokens"]) if case["workspace"] else 0
        state["workspace"] = torch.empty(size, dtype=torch.uint8, device="cuda") if size else None
    return state


def _gemv_workspace(layer, batch):
    size = vq.vq_gemv_workspace_bytes(layer.desc, batch)
    return torch.empty(size, dtype=torch.uint8, device="cuda") if size else None


# ---- one pass ---------------------------------------------------------------------------------------------------------
def run(state):
    op = state["op"]
    if op == "gemv":
        return vq.gemv(state["layer"], state["x"], workspace=state["workspace"])
    if op == "decoder":
        qkv = vq.gemv_multi([state["q"], state["k"], state["v"]], state["x"])
        o = vq.gemv(state["o"], state["attention"], workspace=state["ws_o"])
        gate_up = vq.gemv_multi([state["gate"], state["up"]], state["x_mlp"])
        return qkv + [o] + gate_up + [vq.gemv(state["down"], state["hidden"], workspace=state["ws_down"])]
    if op == "gemm":
        return vq.gemm(state["layer"], state["x"], workspace=state["workspace"])
    if op == "dequant":
        return vq.dequant(state["layer"])
    if op == "assign":
        return vq.assign(state["W"], state["C"], base=state["B"], orientation=state["orientation"])
    W = state["W"].clone()                     # the call overwrites the weights with the quantized ones
    idx, idx_res, T = vq.quantize_columns(W, state["Hinv"], state["C"], state["R"], block=state["block"])
    return {"W": W, "idx": idx, "idx_res": idx_res, "T": T}


# ---- what a pass cannot do without, and how close two correct results are ----------------------------------------------
def work(case):
    op = case["op"]
    if op == "assign":
        m, n = case["rows"], case["cols"]
        vectors = (m * n) // case["v"]
        # a subtraction and a multiply-add per element of a (vector, centroid) pair
        return {"bytes": 2 * m * n * (2 if case["base"] else 1) + 2 * case["k"] * case["v"] + vectors * index_bits(case["k"]) // 8,
                "flops": 3 * m * n * case["k"]}
    if op == "quantize":
        m, n = case["rows"], case["cols"]
        bits = index_bits(case["k"]) + (index_bits(case["k_res"]) if case["k_res"] else 0)
        # the searches, and a multiply-add per weight and later column
        return {"bytes": 12 * m * n + 2 * n * n + m * n // case["v"] * bits // 8, "flops": 3 * m * n * (case["k"] + case["k_res"]) + m * n * n}
    if op == "decoder":
        h, i, total = case["hidden"], case["inter"], {"bytes": 0, "flops": 0}
        for m, n, count in ((h, h, 4), (i, h, 2), (h, i, 1)):
            one = work({"op": "gemv", "out": m, "in": n, "v": 6, "k": 4096, "k_res": case["k_res"], "outliers": 0, "k_out": 0, "group_vectors": 0,
                        "orientation": case["orientation"], "permute": False, "batch": case["batch"]})
            for key in total:
                total[key] += count * one[key]
        return total
    L = _fields(case)
    L.scale = L.bias = True                    # both are there
    fixed = L.algorithmic_bytes(0) + (4 * L.in_features if case["permute"] else 0)
    m, n = L.out_features, L.in_features
    if op == "dequant":
        return {"bytes": fixed + 2 * m * n, "flops": 3 * m * n}
    rows = case["batch"] if op == "gemv" else case["tokens"]
    return {"bytes": fixed + 2 * rows * (m + n), "flops": 2 * rows * m * n}


def tolerance(case):
    if case["op"] in ("dequant", "assign"):
        return "exact"
    if case["op"] == "quantize":
        # binary32 sums in another order move a column by about 1e-6 of its values; where that decides a nearly tied choice
        # the other way, the later columns of that stack position are other ones, and as correct
        return {"rel": 1e-2, "max": 0.99, "differ": 1e-2}
    # fp16 inputs and results, binary32 sums
    return {"rel": 2e-3, "max": 1e-2}
