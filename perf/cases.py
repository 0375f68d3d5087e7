"""Timed cases of the LUT-NN linear operator, through the calls that a user's program makes.

A case is a dict of plain values; `path` names the entry point:

  linear        lut.linear               nearest-centroid encoding, then the table lookup
  conv          lut.conv2d               the same on an NCHW batch
  encoder_layer lut.linear, four times   the linears of one transformer encoder layer
  tree          lut.linear_tree / lut.linear_tree16 (above 8 levels): the hash encoder in front
  train_linear  softpq.SoftPQLinear      forward and backward of one training step of the layer
  train_conv    softpq.SoftPQConv2d      the same for a convolution

Sizes are those of lutnn_workloads.py and bench.py (N rows, D = C*V inputs, K centroids per codebook, M outputs);
`draw` spreads more of them over the same ranges.
"""
import math

import torch

import paper_2302_03213_amd as lut
from paper_2302_03213_amd.softpq import SoftPQConv2d, SoftPQLinear

TABLES = {"i8": lut.TABLE_I8, "i4": lut.TABLE_I4, "f32": lut.TABLE_F32}
ENTRY_BYTES = {"i8": 1.0, "i4": 0.5, "f32": 4.0}

# the linears of an encoder layer of width H and feed-forward width 4H: QKV, attention output, FFN up, FFN down
LAYER_LINEARS = ((1, 3), (1, 1), (1, 4), (4, 1))


def listed():
    return [
        # one token through a BERT-base FFN-up layer: on-device inference, where latency and launches count
        dict(name="row_ffn_up_i8", path="linear", N=1, C=384, K=16, V=2, M=3072, table="i8"),
        # a small fully connected layer with the unquantised table (benchmark configuration 1)
        dict(name="fc_small_f32", path="linear", N=256, C=128, K=16, V=4, M=512, table="f32"),
        # a ResNet-18 3x3 convolution on one image (configuration 2) and on a batch of 32
        dict(name="conv_image_i8", path="conv", B=1, Cin=64, H=56, Wd=56, kernel=3, stride=1, pad=1, K=16, V=9, M=64, table="i8"),
        dict(name="conv_batch_i8", path="conv", B=32, Cin=64, H=56, Wd=56, kernel=3, stride=1, pad=1, K=16, V=9, M=64, table="i8"),
        # the four linears of a BERT-base encoder layer at batch 32 x 128 tokens: with the short sub-vectors of
        # configuration 4, and with the paper's own (K, V) = (16, 32)
        dict(name="bert_layer_v2_i8", path="encoder_layer", N=4096, H=768, K=16, V=2, table="i8"),
        dict(name="bert_layer_v32_i8", path="encoder_layer", N=4096, H=768, K=16, V=32, table="i8"),
        # the large fully connected layer (configuration 5), the benchmark's headline
        dict(name="fc_large_i8", path="linear", N=16384, C=1024, K=16, V=4, M=4096, table="i8"),
        # FFN-up rows at batch size with the unquantised table
        dict(name="ffn_up_f32", path="linear", N=4096, C=192, K=16, V=4, M=3072, table="f32"),
        # sizes that are multiples of nothing, the hash encoder and the smallest table type
        dict(name="ragged_tree_i4", path="tree", N=3001, C=75, V=8, M=1001, levels=4, table="i4"),
        # FFN-down with the paper's 12-level trees: 4096 table rows per codebook
        dict(name="tree12_ffn_down_i8", path="tree", N=4096, C=96, V=32, M=768, levels=12, table="i8"),
        # a training step of one layer: FFN-up in the paper's (16, 16) setting, and the 3x3 convolution
        dict(name="train_ffn_up_i8", path="train_linear", N=4096, C=48, K=16, V=16, M=3072, table="i8"),
        dict(name="train_conv_i8", path="train_conv", B=16, Cin=64, H=56, Wd=56, kernel=3, stride=1, pad=1, K=16, V=9, M=64, table="i8"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sub_vectors(rng, V, lo, hi):
    """A number of codebooks for an input width between lo and hi; every other draw is a power-of-two width."""
    D = _log_int(rng, lo, hi)
    if rng.random() < 0.5:
        D = 1 << max(D.bit_length() - 1, 5)
    return max(1, D // V)


def _width(rng, lo, hi):
    M = _log_int(rng, lo, hi)
    return M if rng.random() < 0.5 else max(64, M // 64 * 64)


def _conv_shape(rng, max_batch):
    HW = rng.choice([7, 14, 28, 32, 56])
    kernel = rng.choice([1, 3, 3])
    Cin = _log_int(rng, 16, 256)
    if kernel == 1 or rng.random() < 0.5:
        Cin = max(16, Cin // 16 * 16)
    return dict(B=_log_int(rng, 1, max_batch), Cin=Cin, H=HW, Wd=HW, kernel=kernel, stride=rng.choice([1, 1, 2]) if HW > 7 else 1,
                pad=kernel // 2, K=rng.choice([8, 16, 16]), V=9 if kernel == 3 else 4, M=_width(rng, 32, 512))


def draw(rng):
    while True:
        path = rng.choice(["linear", "linear", "linear", "conv", "encoder_layer", "tree", "train_linear", "train_conv"])
        table = rng.choice(["i8", "i8", "i8", "i4", "f32"])
        if path == "linear":
            V = rng.choice([2, 4, 8, 16, 32])
            case = dict(path=path, N=_log_int(rng, 1, 16384), C=_sub_vectors(rng, V, 64, 4096), K=rng.choice([8, 16, 16, 16]), V=V,
                        M=_width(rng, 64, 4096), table=table)
        elif path == "conv":
            case = dict(_conv_shape(rng, 32), path=path, table=table)
        elif path == "encoder_layer":
            case = dict(path=path, N=_log_int(rng, 1, 4096), H=rng.choice([256, 384, 512, 768, 1024]), K=16, V=rng.choice([2, 4, 16, 32]), table="i8")
        elif path == "tree":
            V = rng.choice([4, 8, 16, 32])
            levels = rng.choice([3, 4, 4, 6, 8, 10, 12])
            case = dict(path=path, N=_log_int(rng, 16, 16384), C=_sub_vectors(rng, V, 64, 4096), V=V, M=_width(rng, 64, 1024 if levels > 4 else 4096),
                        levels=levels, table=table if levels <= 8 else rng.choice(["i8", "f32"]))
        elif path == "train_linear":
            V = rng.choice([4, 8, 16, 32])
            case = dict(path=path, N=_log_int(rng, 64, 8192), C=_sub_vectors(rng, V, 64, 3072), K=rng.choice([8, 16, 16]), V=V,
                        M=_width(rng, 64, 3072), table=rng.choice(["i8", "i8", "f32"]))
        else:
            case = dict(_conv_shape(rng, 16), path=path, table=rng.choice(["i8", "i8", "f32"]))
        if _costs_no_more_than_the_largest(case):
            return case


def _linears(case):
    """[(N, C, K, V, M)] of the operator calls of one pass."""
    if case["path"] == "encoder_layer":
        return [(case["N"], a * case["H"] // case["V"], case["K"], case["V"], b * case["H"]) for a, b in LAYER_LINEARS]
    if "B" in case:
        return [(case["B"] * _conv_out(case)[0] * _conv_out(case)[1], case["Cin"] * case["kernel"] ** 2 // case["V"], case["K"], case["V"], case["M"])]
    return [(case["N"], case["C"], case["K"] if "K" in case else 1 << case["levels"], case["V"], case["M"])]


def _conv_out(case):
    return [(case[side] + 2 * case["pad"] - case["kernel"]) // case["stride"] + 1 for side in ("H", "Wd")]


def _costs_no_more_than_the_largest(case):
    for N, C, K, V, M in _linears(case):
        adds = N * C * M
        if adds > (2.0e10 if K <= 16 and case["table"] != "f32" else 4.0e9):
            return False
        if C * K * M * ENTRY_BYTES[case["table"]] > 4.0e8 or (K > 16 and C * K * V > 2.0e7):
            return False
    return True


def _gpu_normal(gen, shape, std=1.0):
    return torch.randn(shape, generator=gen, device="cuda") * std


def _drawn_layer(gen, C, K, V, M, table, P=None):
    P = _gpu_normal(gen, (C, K, V)) if P is None else P
    return lut.build_table(P, _gpu_normal(gen, (C * V, M), 0.05), TABLES[table], bias=_gpu_normal(gen, (M,), 0.1))


def _rows(gen, N, D):
    """Activations ~ N(0, 1), one in a hundred of them ten times as large."""
    X = _gpu_normal(gen, (N, D))
    return torch.where(torch.rand((N, D), generator=gen, device="cuda") < 0.01, X * 10.0, X)


def _centroids_of(gen, Xs, K):
    """[C, K, V] for sub-vectors Xs [N, C, V]: for each codebook, K sub-vectors of the data, as a clustering starts."""
    N, C, _ = Xs.shape
    pick = torch.randint(0, N, (C, K), generator=gen, device="cuda")
    return Xs[pick, torch.arange(C, device="cuda")[:, None]].contiguous()


def _error_of_the_layer(Xs, P, W):
    """(Xhat - X) @ W with every sub-vector of Xhat the nearest centroid: the gradient, at the layer's output, of half the
    squared distance to the layer it replaces."""
    out = []
    for part in Xs.split(8192):
        d = torch.cdist(part.transpose(0, 1).contiguous(), P, compute_mode="donot_use_mm_for_euclid_dist")  # [C, n, K]
        near = P.gather(1, d.argmin(dim=2)[:, :, None].expand(-1, -1, P.shape[2]))  # [C, n, V]
        out.append((near.transpose(0, 1) - part).reshape(part.shape[0], -1) @ W)
    return torch.cat(out)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    path = case["path"]
    state = {"case": case}
    if path in ("linear", "encoder_layer"):
        state["calls"] = [(_drawn_layer(gen, C, K, V, M, case["table"]), _rows(gen, N, C * V)) for N, C, K, V, M in _linears(case)]
        return state
    if path == "tree":
        (N, C, K, V, M), = _linears(case)
        nodes = K - 1
        state["layer"] = _drawn_layer(gen, C, K, V, M, case["table"])
        state["tree"] = lut.LutTree(torch.randint(0, V, (C, nodes), generator=gen, device="cuda", dtype=torch.int32),
                                    _gpu_normal(gen, (C, nodes), 0.5), V)
        state["X"] = _rows(gen, N, C * V)
        return state
    (N, C, K, V, M), = _linears(case)
    if path == "conv":
        state["layer"] = _drawn_layer(gen, C, K, V, M, case["table"])
        state["inp"] = _gpu_normal(gen, (case["B"], case["Cin"], case["H"], case["Wd"]))
        return state
    W, bias = _gpu_normal(gen, (C * V, M), 0.05), _gpu_normal(gen, (M,), 0.1)
    if path == "train_linear":
        X = _gpu_normal(gen, (N, C * V))
        rows = X
    else:
        X = _gpu_normal(gen, (case["B"], case["Cin"], case["H"], case["Wd"]))
        rows = torch.nn.functional.unfold(X, case["kernel"], padding=case["pad"], stride=case["stride"]).transpose(1, 2).reshape(N, C * V)
    Xs = rows.reshape(N, C, V)
    P = _centroids_of(gen, Xs, K)
    G = _error_of_the_layer(Xs, P, W)
    if path == "train_linear":
        state["layer"] = SoftPQLinear(P, W, bias=bias, table_dtype=TABLES[case["table"]])
        state["G"] = G
    else:
        state["layer"] = SoftPQConv2d(P, W, case["kernel"], case["stride"], case["pad"], bias=bias, table_dtype=TABLES[case["table"]])
        Ho, Wo = _conv_out(case)
        state["G"] = G.view(case["B"], Ho, Wo, M).permute(0, 3, 1, 2).contiguous()
    state["X"] = X.requires_grad_(True)  # earlier layers want its gradient
    return state


def run(state):
    case = state["case"]
    path = case["path"]
    if path in ("linear", "encoder_layer"):
        return [lut.linear(layer, X) for layer, X in state["calls"]]
    if path == "conv":
        return lut.conv2d(state["layer"], state["inp"], case["kernel"], case["stride"], case["pad"])
    if path == "tree":
        call = lut.linear_tree if case["levels"] <= 8 else lut.linear_tree16
        return call(state["layer"], state["tree"], state["X"])
    layer, X = state["layer"], state["X"]
    Y = layer(X)
    dX, dP, dt, dbias = torch.autograd.grad(Y, (X, layer.centroids, layer.temperature, layer.bias), state["G"])
    return {"Y": Y.detach(), "dX": dX, "dP": dP, "dt": dt, "dbias": dbias}


def work(case):
    """Each input read once and each output written once; of a table, the rows that so many indices can select. One
    multiply-add is two operations: three per centroid and value for the distances (a tree walk: one per level), one
    per output and codebook for the sums."""
    total = {"bytes": 0.0, "flops": 0.0}
    for N, C, K, V, M in _linears(case):
        D = C * V
        inputs = case["B"] * case["Cin"] * case["H"] * case["Wd"] if "B" in case else N * D
        rows = min(N, K)
        encoder = 8 * C * (K - 1) if case["path"] == "tree" else 4 * C * K * V
        search = N * C * case["levels"] if case["path"] == "tree" else 3 * N * C * K * V
        if case["path"].startswith("train"):
            # forward: X, P, W, bias in, Y out; backward: G, X again as W and P are kept on the chip, dX, dP, dbias out
            total["bytes"] += 4.0 * (inputs + 2 * C * K * V + D * M + 2 * M + 2 * N * M + inputs)
            # table, distances, sums; Z = G @ W^T, soft encoding and its gradients
            total["flops"] += 2.0 * C * K * V * M + search + N * C * M + 2.0 * N * D * M + N * C * K * (14.0 * V + 10)
        else:
            total["bytes"] += 4.0 * inputs + encoder + C * rows * M * ENTRY_BYTES[case["table"]] + 4.0 * M + 4.0 * N * M
            total["flops"] += search + N * C * M
    return total


def tolerance(case):
    if case["path"].startswith("train"):
        return {"rel": 1e-5}  # measured against 64-bit gradients: up to 2.5e-6 over these ranges
    if case["table"] == "f32":
        return {"rel": 2e-6}  # measured against 64-bit sums: up to 2.5e-7, growing with the number of codebooks
    return "exact"
