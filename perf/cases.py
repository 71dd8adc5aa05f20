"""Workloads of the tile-wise sparse GEMM library as a user's program runs them.

Every case is a pass through the public entry points on weights that were pruned and packed
beforehand (the exception is `load_weight`, where pruning and packing are the pass), with
activations, outputs and packed weights of its own for every launch.

  op         what a pass calls
  tw         tw_gemm on tile-wise weights, activations K x M (the library's main path)
  tvw        tw_gemm on tile-vector-wise weights (tile-wise, then 2:4 along the kept rows)
  tew        tw_gemm on tile-wise weights with restored single elements
  tw_mk      tw_gemm on row-major activations and outputs (what a torch model holds)
  tw_i8      tw_gemm_i8, tile-wise; int32 sums or requantised int8
  tvw_i8     tw_gemm_i8, tile-vector-wise
  conv       tw_conv_gemm: a stride-1 "same" convolution without a materialised img2col matrix
  conv_i8    tw_conv_gemm_i8
  load       tw_prune_dev, tw_pack_dev and the first tw_gemm with a new weight

`layers` lists the weights K x N of a pass; "KxN*3" are three weights that multiply the same
activations, packed one by one and joined with tw_concat (the Q, K and V projections).
"""
from __future__ import annotations

import math

import torch

import paper_2402_10876_amd as tw

INT8_OPS = ("tw_i8", "tvw_i8", "conv_i8")
CONV_OPS = ("conv", "conv_i8")
BERT_BASE = "768x768*3,768x768,768x3072,3072x768"     # the linear layers of one encoder layer
BERT_BASE_FFN = "768x3072,3072x768"


def listed():
    return [
        # The smallest configured problem: one launch, all latency.
        dict(name="tiny_tw50", op="tw", M=128, layers="256x256", G=64, sparsity=0.5, cols=0.0),
        # One sequence of 128 tokens through an encoder layer: serving without batching.
        dict(name="bert_base_one_sequence_tw75", op="tw", M=128, layers=BERT_BASE, G=128, sparsity=0.75, cols=0.1),
        # The step the benchmark is quoted on: batch 32 x 128 tokens through an encoder layer.
        dict(name="bert_base_layer_tw75", op="tw", M=4096, layers=BERT_BASE, G=128, sparsity=0.75, cols=0.1),
        # The same step with 2:4 inside the kept rows.
        dict(name="bert_base_layer_tvw875", op="tvw", M=4096, layers=BERT_BASE, G=128, sparsity=0.875, cols=0.1),
        # The largest configured problem at the least sparsity that is of use.
        dict(name="bert_large_ffn_tw50", op="tw", M=8192, layers="1024x4096,4096x1024", G=128, sparsity=0.5, cols=0.1),
        # Global pruning of a weight whose column blocks differ in magnitude: tiles of very
        # different height, and sizes that are multiples of nothing.
        dict(name="ragged_uneven_tw75", op="tw", M=1957, layers="1003x2491", G=64, sparsity=0.75, cols=0.1, uneven=True),
        # 1.5 % single elements put back on top of a tile-wise mask.
        dict(name="bert_base_ffn_tew75", op="tew", M=4096, layers=BERT_BASE_FFN, G=128, sparsity=0.75, cols=0.1,
             delta=0.015),
        # A quantised encoder layer: int8 activations in, int8 activations out.
        dict(name="bert_base_layer_i8_tw75", op="tw_i8", M=4096, layers=BERT_BASE, G=128, sparsity=0.75, cols=0.1,
             out_i8=True),
        # Quantised feed-forward layers with int32 sums for a caller that rescales by itself.
        dict(name="bert_base_ffn_i8_tvw875", op="tvw_i8", M=4096, layers=BERT_BASE_FFN, G=128, sparsity=0.875, cols=0.1,
             out_i8=False),
        # A VGG-16 convolution, 256 channels of 56 x 56, batch 8, with the tile width used for CNNs.
        dict(name="vgg16_conv_256_56_tw75", op="conv", C=256, N=256, H=56, W=56, R=3, S=3, batch=8, G=64,
             sparsity=0.75, cols=0.1),
        # The encoder layer on row-major activations, as a torch model holds them.
        dict(name="bert_base_layer_rowmajor_tw75", op="tw_mk", M=4096, layers=BERT_BASE, G=128, sparsity=0.75, cols=0.1),
        # A new weight on the device: prune it, pack it, run one sequence through it.
        dict(name="load_weight_tvw875", op="load", M=128, layers="1024x4096", G=128, sparsity=0.875, cols=0.1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case of these ranges: one launch, no more work than the listed case of its op."""
    ops = ["tw"] * 8 + ["tvw"] * 5 + ["tw_mk"] * 3 + ["tew"] * 2 + ["tw_i8"] * 4 + ["tvw_i8"] * 3 + ["conv"] * 3 + \
          ["conv_i8"] + ["load"] * 2
    op = rng.choice(ops)
    cap_of = {"conv_i8": "conv"}.get(op, op)
    caps = [work(c) for c in listed() if c["op"] == cap_of]
    cap_b, cap_f = max(c["bytes"] for c in caps), max(c["flops"] for c in caps)
    while True:
        pairs24 = op in ("tvw", "tvw_i8") or op == "load"
        case = dict(op=op, G=rng.choice([64, 128, 128]), cols=rng.choice([0.0, 0.1, 0.1, 0.2]),
                    sparsity=round(rng.uniform(0.75 if pairs24 else 0.5, 0.95), 3))
        if op in ("tw", "tw_mk") and rng.random() < 0.1:
            case["G"] = 32
        if op in CONV_OPS:
            case.update(C=_log_int(rng, 16, 512), N=_log_int(rng, 64, 512), batch=_log_int(rng, 1, 16),
                        H=_log_int(rng, 7, 112))
            case["W"] = max(7, case["H"] + rng.choice([-3, 0, 0, 5]))
            case["R"], case["S"] = rng.choice([(3, 3), (3, 3), (3, 3), (1, 1), (5, 5), (1, 3)])
        else:
            case["M"] = _log_int(rng, 1, 8192)
            K, N = _log_int(rng, 64, 4096), _log_int(rng, 64, 4096)
            if rng.random() < 0.6:                                 # most layers are multiples of 64
                K, N = max(64, K // 64 * 64), max(64, N // 64 * 64)
            case["layers"] = f"{K}x{N}"
        if op in INT8_OPS:
            case["out_i8"] = rng.random() < 0.5
        if op == "tew":
            case["delta"] = rng.choice([0.005, 0.01, 0.015, 0.03])
        if op == "tw":
            case["uneven"] = rng.random() < 0.25
        w = work(case)
        if w["bytes"] <= cap_b and w["flops"] <= cap_f:
            return case


# ---- geometry ---------------------------------------------------------------------------------
def _up(x, a):
    return -(-x // a) * a


def _layers(case):
    """(K, N, copies) of every launch of a pass."""
    if case["op"] in CONV_OPS:
        return [(case["C"] * case["R"] * case["S"], case["N"], 1)]
    out = []
    for text in case["layers"].split(","):
        shape, _, copies = text.partition("*")
        k, n = shape.split("x")
        out.append((int(k), int(n), int(copies or 1)))
    return out


class _Geom:
    """Wide input of a stride-1 "same" convolution (see tw_conv_geom): lines of P elements,
    L lines per image, padding stored."""

    def __init__(self, case):
        self.C, self.R, self.S, self.B = case["C"], case["R"], case["S"], case["batch"]
        self.H, self.W = case["H"], case["W"]
        self.P, self.L = self.W + self.S - 1, self.H + self.R - 1
        self.Mp = self.B * self.L * self.P
        chunk = 16 if case["op"] == "conv_i8" else 8
        self.ldx = _up(_up(self.Mp, chunk) + (self.R - 1) * self.P + self.S - 1, chunk)
        self.ldc = _up(self.Mp, chunk)


def _kept(case, K, N):
    """Kept columns and the share of rows that a tile keeps, so that the whole mask reaches the
    case's sparsity (2:4 halves what the tiles keep; restored elements come out of the same share)."""
    n = N - int(math.floor(case["cols"] * N))
    density = 1.0 - case["sparsity"] - case.get("delta", 0.0)
    if case["op"] in ("tvw", "tvw_i8", "load"):
        density *= 2.0
    return n, min(1.0, density * N / n)


def work(case):
    op = case["op"]
    el = 1 if op in INT8_OPS else 2
    c_el = (1 if case["out_i8"] else 4) if op in INT8_OPS else 2
    total_b = total_f = 0.0
    for K, N, copies in _layers(case):
        n, rho = _kept(case, K, N)
        tiles = -(-n // case["G"]) * copies
        kept = rho * K * n * copies                          # elements in the kept rows and columns
        union = K * (1.0 - (1.0 - rho) ** tiles)             # rows of the input that some tile keeps
        pairs24 = op in ("tvw", "tvw_i8", "load")
        used = kept / 2 if pairs24 else kept
        weight = el * used + (kept / 8 if pairs24 else 0) + 4 * rho * K * tiles
        extra = case.get("delta", 0.0) * K * N * copies
        if extra:
            used += extra
            weight += 4 * extra
            union = K
        if op in CONV_OPS:
            pixels = case["batch"] * case["H"] * case["W"]
            g = _Geom(case)
            channels = case["C"] * (1.0 - (1.0 - union / K) ** (case["R"] * case["S"]))
            total_b += el * channels * pixels + c_el * N * g.Mp + weight
            total_f += 2.0 * pixels * used
            continue
        total_b += el * case["M"] * union + c_el * case["M"] * N * copies + weight
        total_f += 2.0 * case["M"] * used
        if op == "load":       # the weight read once, both masks and the packed form written
            total_b += 2 * K * N + 2 * K * N + weight
            total_f += 4.0 * K * N
    return {"bytes": int(total_b), "flops": int(total_f)}


def tolerance(case):
    if case["op"] in INT8_OPS:
        return "exact"
    # fp16 results of fp32 sums: 2.1e-4 from the same product in 64 bits (the rounding to fp16);
    # a rounding that falls the other way is one unit in the last place, 9.8e-4 of the value
    return {"rel": 8e-4, "max": 2e-3}


# ---- inputs -----------------------------------------------------------------------------------
def _tile_mask(W, G, n_kept, rho, uneven):
    """Tile-wise mask by magnitude: the best n_kept columns, then in every tile of G of them the
    best rho*K rows (uneven: one threshold over the rows of all tiles).  Returns the K x N mask,
    the kept columns and the tiles' row masks (tiles x K)."""
    K, N = W.shape
    sq = W.double() ** 2
    cols = sq.sum(0).topk(n_kept).indices.sort().values
    tiles = -(-n_kept // G)
    padded = torch.zeros((K, tiles * G), dtype=torch.float64, device=W.device)
    padded[:, :n_kept] = sq[:, cols]
    score = padded.view(K, tiles, G).sum(2).t()                         # tiles x K
    width = torch.full((tiles, 1), float(G), dtype=torch.float64, device=W.device)
    width[-1] = n_kept - (tiles - 1) * G
    score = (score / width).contiguous()
    keep = torch.zeros(score.shape, dtype=torch.bool, device=W.device)
    rows = max(1, int(math.floor(rho * K + 0.5)))
    if uneven:
        keep.view(-1)[score.view(-1).topk(min(score.numel(), rows * tiles)).indices] = True
    else:
        keep.scatter_(1, score.topk(rows, dim=1).indices, True)
    mask = torch.zeros((K, N), dtype=torch.bool, device=W.device)
    mask[:, cols] = keep.repeat_interleave(G, dim=0)[:n_kept].t()
    return mask, cols, keep


def _two_of_four(W, G, cols, keep):
    """2 of every 4 consecutive kept rows of a tile, per column, by magnitude (equal rows per tile)."""
    K, N = W.shape
    mask = torch.zeros((K, N), dtype=torch.bool, device=W.device)
    for t in range(keep.shape[0]):
        rows, tc = keep[t].nonzero().flatten(), cols[t * G:(t + 1) * G]
        groups = -(-rows.numel() // 4)
        mag = torch.full((groups * 4, tc.numel()), -1.0, dtype=torch.float32, device=W.device)
        mag[:rows.numel()] = W[rows][:, tc].float().abs()
        best = mag.view(groups, 4, -1).topk(2, dim=1).indices
        hit = torch.zeros((groups, 4, tc.numel()), dtype=torch.bool, device=W.device)
        hit.scatter_(1, best, True)
        mask[rows[:, None], tc[None, :]] = hit.view(groups * 4, -1)[:rows.numel()]
    return mask


def _host(x):
    return x.to(torch.uint8).cpu().numpy()


def _weight(case, K, N, gen, dev):
    """One pruned and packed weight, as a program holds it after loading a model."""
    op, G = case["op"], case["G"]
    W = torch.randn((K, N), generator=gen, device=dev, dtype=torch.float32)
    if case.get("uneven"):             # column blocks of different magnitude: tiles of different height
        scale = torch.exp(0.6 * torch.randn((-(-N // 128),), generator=gen, device=dev))
        W *= scale.repeat_interleave(128)[:N]
    if op in INT8_OPS:
        W = (W * 40.0).round().clamp(-127, 127)
        values = W.to(torch.int8)
    else:
        values = (W * 0.02).to(torch.float16)
        W = values.float()
    n, rho = _kept(case, K, N)
    mask, cols, keep = _tile_mask(W, G, n, rho, case.get("uneven", False))
    tile_mask = None
    if op in ("tvw", "tvw_i8"):
        tile_mask, mask = mask, _two_of_four(W, G, cols, keep)
    elif op == "tew":                  # the largest pruned elements come back
        tile_mask, mask = mask, mask.clone()
        score = W.abs().masked_fill(tile_mask, -1.0).view(-1)
        mask.view(-1)[score.topk(int(case["delta"] * K * N)).indices] = True
    pattern = {"tvw": tw.PATTERN_TVW, "tvw_i8": tw.PATTERN_TVW, "tew": tw.PATTERN_TEW}.get(op, tw.PATTERN_TW)
    pack = tw.tw_pack_i8 if op in INT8_OPS else tw.tw_pack
    return pack(values.cpu().numpy(), _host(mask), G, pattern, tile_mask=None if tile_mask is None else _host(tile_mask))


def _activations(shape, op, gen, dev):
    x = torch.randn(shape, generator=gen, device=dev, dtype=torch.float32)
    return (x * 40.0).round().clamp(-127, 127).to(torch.int8) if op in INT8_OPS else x.to(torch.float16)


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    op = case["op"]
    state = {"op": op, "launches": []}
    c_dtype = (torch.int8 if case["out_i8"] else torch.int32) if op in INT8_OPS else torch.float16
    if op in INT8_OPS:
        state["c_dtype"] = 1 if case["out_i8"] else 0
    if op in CONV_OPS:
        g = _Geom(case)
        X = torch.zeros((g.C, g.ldx), dtype=torch.int8 if op == "conv_i8" else torch.float16, device=dev)
        top, left = (g.R - 1) // 2, (g.S - 1) // 2
        X[:, :g.Mp].view(g.C, g.B, g.L, g.P)[:, :, top:top + g.H, left:left + g.W] = \
            _activations((g.C, g.B, g.H, g.W), op, gen, dev)
        packed = _weight(case, g.C * g.R * g.S, case["N"], gen, dev)
        state["launches"].append((X, tw.tw_conv_bind(packed, g, g.ldx), g.ldc,
                                  torch.zeros((case["N"], g.ldc), dtype=c_dtype, device=dev)))
        state["scale"] = 1.0 / (40.0 * math.sqrt(g.C * g.R * g.S))
        return state
    M = state["M"] = case["M"]
    ld = state["ld"] = _up(M, 16)
    for K, N, copies in _layers(case):
        state["scale"] = 1.0 / (40.0 * math.sqrt(K))
        if op == "load":
            n, rho = _kept(case, K, N)
            W = (0.02 * torch.randn((K, N), generator=gen, device=dev)).to(torch.float16)
            mask, tile_mask = (torch.zeros((K, N), dtype=torch.uint8, device=dev) for _ in range(2))
            ws_bytes = tw.tw_prune_workspace_bytes(K, N, case["G"])
            state.update(W=W, K=K, N=N, G=case["G"], drop=N - n, rows=int(math.floor(rho * K + 0.5)), mask=mask,
                         tile_mask=tile_mask, ws=torch.empty((ws_bytes,), dtype=torch.uint8, device=dev),
                         A=_activations((K, ld), op, gen, dev), C=torch.zeros((N, ld), dtype=c_dtype, device=dev))
            return state
        parts = [_weight(case, K, N, gen, dev) for _ in range(copies)]
        packed = parts[0] if copies == 1 else tw.tw_concat(parts)
        if op == "tw_mk":
            lda, ldc = _up(K, 8), _up(N * copies, 8)
            A = _activations((M, lda), op, gen, dev)
            C = torch.zeros((M, ldc), dtype=c_dtype, device=dev)
        else:
            lda = ldc = ld
            A = _activations((K, ld), op, gen, dev)
            C = torch.zeros((N * copies, ld), dtype=c_dtype, device=dev)
        state["launches"].append((A, packed, (lda, ldc), C))
    return state


# ---- one pass ---------------------------------------------------------------------------------
def run(state):
    stream = torch.cuda.current_stream().cuda_stream
    op = state["op"]
    if op == "load":
        K, N, G, M, ld = state["K"], state["N"], state["G"], state["M"], state["ld"]
        W, mask, tile_mask, ws = state["W"], state["mask"], state["tile_mask"], state["ws"]
        tw.tw_prune_dev(W.data_ptr(), K, N, N, G, tw.PATTERN_TVW, state["drop"], state["rows"], mask.data_ptr(),
                        tile_mask.data_ptr(), ws.data_ptr(), ws.numel(), stream)
        state["packed"] = packed = tw.tw_pack_dev(W.data_ptr(), N, mask.data_ptr(), tile_mask.data_ptr(), K, N, G,
                                                  tw.PATTERN_TVW, stream)
        tw.tw_gemm(state["A"].data_ptr(), M, ld, tw.LAYOUT_KM, packed, state["C"].data_ptr(), ld, stream)
        return {"mask": mask, "tile_mask": tile_mask, "C": state["C"]}
    for X, weight, ld, C in state["launches"]:
        if op == "conv":
            tw.tw_conv_gemm(X.data_ptr(), weight, C.data_ptr(), ld, stream)
        elif op == "conv_i8":
            tw.tw_conv_gemm_i8(X.data_ptr(), weight, C.data_ptr(), ld, state["c_dtype"], state["scale"], stream)
        elif op in INT8_OPS:
            tw.tw_gemm_i8(X.data_ptr(), state["M"], ld[0], weight, C.data_ptr(), ld[1], state["c_dtype"],
                          state["scale"], stream)
        else:
            layout = tw.LAYOUT_MK if op == "tw_mk" else tw.LAYOUT_KM
            tw.tw_gemm(X.data_ptr(), state["M"], ld[0], layout, weight, C.data_ptr(), ld[1], stream)
    return [C for _, _, _, C in state["launches"]]
