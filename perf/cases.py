"""The boundary workloads whose speed is measured, and how one pass of each runs.

A pass takes `micro` micro-batches across a pipeline-stage boundary: for each,
the sender's call and the receiver's call of paper_2401_07788_amd.tc (or, for
op "module", the forward and backward pass of boundary.TopkBoundary).  The
error feedback residuals and AQ-SGD buffers carry on from micro-batch to
micro-batch and from pass to pass, as in training.

A case is a dict of plain values:
  op      topk | topk_ef | quant | quant_ef | topk_quant_ef | efmix | aqsgd | module
  dtype   f32 | bf16 | f16: the boundary tensor's (and the wire's) dtype
  n, len  segments (samples, token rows, examples, quantization groups) and
          elements per segment
  num, den  TopK keeps ceil(len * num / den) entries per segment (0: no TopK)
  bits    bits per code of the quantizers (0: none)
  data    relu | grad | hidden | outliers | drift: the values' distribution
  micro   micro-batches per pass
  graph   the pass is one replay of a HIP graph that holds the calls of all its
          micro-batches (a training loop that captures its boundary work, as
          bench.py does); else eager calls, one micro-batch after the other
          out of a few that take turns
"""
import torch

from paper_2401_07788_amd import boundary, tc
from paper_2401_07788_amd import workloads as W

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
DEV = "cuda"
EAGER_TURNS = 4          # micro-batches that take turns in an eager case (2 of the largest)


def case(op, dtype, n, length, num=0, den=1, bits=0, data="relu", micro=1, graph=False, name=None):
    c = {"op": op, "dtype": dtype, "n": n, "len": length, "num": num, "den": den, "bits": bits, "data": data,
         "micro": micro, "graph": graph}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a small transformer boundary (64 token rows of 768): the smallest
        # messages, where launches and the host's calls are what counts
        case("quant_ef", "bf16", 64, 768, bits=4, data="hidden", name="rows64_q4_ef"),
        # the tiny CNN boundary (32 samples of 256x8x8), called eagerly
        case("topk_ef", "f32", 32, 16384, 1, 10, data="relu", name="cnn_topk10_ef"),
        # gradients of ragged, unaligned samples, plain TopK
        case("topk", "f16", 5, 100003, 3, 10, data="grad", name="ragged_topk30"),
        # the autograd module in a transformer (GPT-2 small: 8 x 512 token
        # rows of 768): forward TopK with EF, the gradient at its indices
        case("module", "bf16", 4096, 768, 1, 10, data="hidden", name="gpt2_module"),
        # the same boundary's activations, captured, TopK per token row + EF
        case("topk_ef", "bf16", 4096, 768, 1, 10, data="hidden", micro=4, graph=True, name="gpt2_rows_topk10_ef"),
        # the ResNet-18 boundary (128 samples of 128x16x16): TopK with error
        # feedback, 4-bit quantization with error feedback, EF-mixed
        case("topk_ef", "f32", 128, 32768, 1, 10, data="relu", micro=4, graph=True, name="resnet_topk10_ef"),
        case("quant_ef", "f32", 128, 32768, bits=4, data="relu", micro=4, graph=True, name="resnet_q4_ef"),
        case("efmix", "f32", 128, 32768, 1, 10, data="relu", micro=4, graph=True, name="resnet_efmix10"),
        # AQ-SGD fine-tuning of GPT-2 small: whole examples (512 x 768), and
        # one buffer row per token row
        case("aqsgd", "f16", 8, 393216, 3, 10, data="drift", micro=8, graph=True, name="aqsgd_examples"),
        case("aqsgd", "f16", 4096, 768, 3, 10, data="drift", micro=4, graph=True, name="aqsgd_token_rows"),
        # one selection over a whole transformer micro-batch (8 x 512 x 768)
        case("topk_ef", "bf16", 1, 3145728, 1, 10, data="hidden", name="whole_topk10_ef"),
        # a large language model's micro-batch (16 x 2048 x 4096), TopK with
        # the kept values quantized to 4 bits
        case("topk_quant_ef", "bf16", 1, 1 << 27, 1, 10, 4, data="outliers", name="lm_topk10_q4_ef"),
    ]


def _log_int(rng, lo, hi):
    """an integer spread evenly over the logarithm of [lo, hi]; half of them odd"""
    v = int(round(lo * (hi / lo) ** rng.random()))
    return max(lo, min(hi, v | 1)) if rng.random() < 0.5 else v


def draw(rng):
    """one more case: token rows, per-sample tensors, long examples or whole
    tensors, each with the operations that are run on them"""
    family = rng.choice(("rows", "samples", "long", "whole"))
    dtype = rng.choice(("f32", "bf16", "f16"))
    num, den = rng.choice(((1, 100), (1, 20), (1, 10), (3, 10), (1, 2)))
    bits = rng.choice((2, 3, 4, 6, 8))
    if family == "rows":
        op = rng.choice(("topk", "topk_ef", "quant", "quant_ef", "aqsgd", "module"))
        length = _log_int(rng, 64, 2048)
        n = _log_int(rng, 16, 4096)
    elif family == "samples":
        op = rng.choice(("topk", "topk_ef", "quant", "quant_ef", "efmix", "aqsgd", "module"))
        length = _log_int(rng, 2049, 32768)
        n = _log_int(rng, 4, 128)
    elif family == "long":
        op = rng.choice(("topk", "topk_ef", "quant_ef", "aqsgd"))
        length = _log_int(rng, 32769, 400000)
        n = _log_int(rng, 1, 8)
    else:
        op = rng.choice(("topk", "topk_ef", "topk_quant_ef"))
        length = _log_int(rng, 400000, 1 << 25 if op == "topk_quant_ef" else 1 << 22)
        n = 1
    graph = family != "whole" and op != "module" and rng.random() < 0.5
    micro = rng.choice((2, 4)) if graph else 1
    data = "drift" if op == "aqsgd" else rng.choice(("relu", "grad", "hidden", "outliers"))
    quant = op in ("quant", "quant_ef")
    return case(op, dtype, n, length, 0 if quant else num, 1 if quant else den,
                bits if quant or op == "topk_quant_ef" else 0, data, micro, graph)


# ------------------------------------------------------------------ inputs
def _k(c):
    return -(-c["len"] * c["num"] // c["den"])


def _turns(c):
    if c["graph"]:
        return c["micro"]
    return 2 if c["n"] * c["len"] > 1 << 26 else EAGER_TURNS


def _tensor(c, kind, seed, tid):
    shape, L = (c["n"], c["len"]), c["len"]
    if kind == "relu":
        t = W.relu_activation(shape, seed, tid, DEV)
    elif kind == "grad":
        t = W.normal_gradient(shape, 1e-3, seed, tid, DEV)
    elif kind == "hidden":
        # hidden states of 768 channels with their outlier channels, cut to
        # segments of this length
        total = c["n"] * L
        t = W.transformer_hidden((-(-total // 768), 768), seed, tid, DEV).reshape(-1)[:total].reshape(shape)
    else:
        t = W.sparse_outlier_stream(shape, seed, tid, DEV)
    return t.to(DTYPES[c["dtype"]]).contiguous()


def _inputs(c, seed):
    """the tensors of one state, made from the seed alone"""
    n, L, dt = c["n"], c["len"], DTYPES[c["dtype"]]
    s = {}
    if c["op"] == "aqsgd":
        # each set of ids is visited twice in a turn over the micro-batches,
        # with another drift of its examples' activations each time
        sets = max(1, _turns(c) // 2)
        n_samples = 2 * sets * n
        m = torch.empty((n_samples, L), dtype=dt, device=DEV)
        step = max(1, (1 << 26) // L)
        for r in range(0, n_samples, step):
            m[r:r + step] = W.randn((min(step, n_samples - r), L), seed, 100 + r // step, DEV).to(dt)
        ids = W.epoch_ids(n_samples, n, seed, tensor_id=1)[:sets].to(DEV)
        s["m"], s["m_r"] = m, m.clone()
        s["ids"] = [ids[j % sets].contiguous() for j in range(_turns(c))]
        s["x"] = [W.drifted_activation(m, ids[j % sets], seed, 2 + j) for j in range(_turns(c))]
        return s
    s["x"] = [_tensor(c, c["data"], seed, 2 + j) for j in range(_turns(c))]
    if c["op"] == "module":
        s["gy"] = [_tensor(c, "grad", seed, 50 + j) for j in range(_turns(c))]
    elif c["op"] in ("topk_ef", "quant_ef", "topk_quant_ef", "efmix"):
        s["e"] = torch.zeros(n * L, dtype=torch.float32, device=DEV)
    return s


# ------------------------------------------------------------- one micro-batch
def _micro(c, s, j, ws=None, out=None, y=None):
    """sender and receiver of micro-batch j: {name: tensor} of what they give"""
    op, n, L, k, b = c["op"], c["n"], c["len"], _k(c), c["bits"]
    x = s["x"][j]
    if op in ("topk", "topk_ef"):
        if op == "topk":
            pl = tc.topk_compress(x, k, n, ws=ws, out=out)
        else:
            pl = tc.ef_step_topk(x, s["e"], k, n, ws=ws, out=out)
        y = tc.topk_decompress(pl, L, out=y)
        return {"idx": pl.idx, "val": pl.val, "blk": pl.blk, "y": y}
    if op in ("quant", "quant_ef"):
        if op == "quant":
            codes, meta = tc.quant_pack(x, b, n, ws=ws)
        else:
            codes, meta = tc.ef_step_quant(x, s["e"], b, n, ws=ws, out=out)
        y = tc.quant_unpack(codes, meta, L, b, out_dtype=x.dtype, out=y)
        return {"codes": codes, "meta": meta, "y": y}
    if op == "topk_quant_ef":
        pl = tc.ef_step_topk_quant(x, s["e"], k, b, n, ws=ws, out=out)
        y = tc.topk_quant_decompress(pl, L, out_dtype=x.dtype, out=y)
        return {"idx": pl.idx, "codes": pl.codes, "meta": pl.meta, "blk": pl.blk, "y": y}
    if op == "efmix":
        px, pe = tc.efmix_step(x, s["e"], k, n, out=out)
        y = tc.efmix_reconstruct(px, pe, L, out=y)
        return {"idx": px.idx, "val": px.val, "idx_e": pe.idx, "val_e": pe.val, "y": y}
    if op == "aqsgd":
        pl = tc.aqsgd_step(x, s["m"], s["ids"][j], k, ws=ws, out=out)
        y = tc.aqsgd_reconstruct(pl, s["m_r"], s["ids"][j], out=y)
        return {"idx": pl.idx, "val": pl.val, "blk": pl.blk, "y": y}
    xg = x.requires_grad_()
    y = s["module"](xg)
    gx, = torch.autograd.grad(y, xg, s["gy"][j])
    return {"y": y.detach(), "gx": gx, "e_fwd": s["module"].e_fwd, "e_bwd": s["module"].e_bwd}


def _carried(c, s):
    return {name: s[name] for name in ("e", "m", "m_r") if name in s}


def _buffers(c):
    """what a captured micro-batch writes to: (payload, dense tensor)"""
    op, n, L, k, dt = c["op"], c["n"], c["len"], _k(c), DTYPES[c["dtype"]]
    y = torch.empty((n, L), dtype=dt, device=DEV)
    if op == "efmix":
        kx, ke = tc.efmix_counts(k)
        return (tc.empty_topk_payload(n, L, kx, dt, DEV), tc.empty_topk_payload(n, L, ke, dt, DEV)), y
    if op in ("quant", "quant_ef"):
        return (torch.empty((n, tc.quant_group_bytes(L, c["bits"])), dtype=torch.uint8, device=DEV),
                torch.empty((n, 2), dtype=torch.float32, device=DEV)), y
    return tc.empty_topk_payload(n, L, k, dt, torch.device(DEV, torch.cuda.current_device())), y


def _workspace(c):
    kind = {"quant": tc.TC_QUANT, "quant_ef": tc.TC_QUANT}.get(c["op"], tc.TC_TOPK)
    wire = {"f32": tc.TC_F32, "bf16": tc.TC_BF16, "f16": tc.TC_F16}[c["dtype"]]
    need = tc.workspace_bytes(tc.codec(kind, c["n"], c["len"], _k(c), c["bits"], wire))
    return torch.zeros(max(need, 8), dtype=torch.uint8, device=DEV)


def prepare(c, seed):
    s = _inputs(c, seed)
    s["case"], s["turn"] = c, 0
    if c["op"] == "module":
        s["module"] = boundary.TopkBoundary(c["num"], c["den"], ef=True, reuse_indices=True)
    if not c["graph"]:
        return s
    # the calls of the pass's micro-batches, captured once
    ws = _workspace(c)
    bufs = [_buffers(c) for _ in range(c["micro"])]

    def calls():
        return [_micro(c, s, j, ws, *bufs[j]) for j in range(c["micro"])]

    kept = {name: t.clone() for name, t in _carried(c, s).items()}
    calls()      # the library's first call of a kind, before the capture
    torch.cuda.synchronize()
    for name, t in kept.items():
        s[name].copy_(t)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        outs = calls()
    s["ws"], s["bufs"], s["g"] = ws, bufs, g
    s["outs"] = {"micro": outs, **_carried(c, s)}
    return s


def run(s):
    if "g" in s:
        s["g"].replay()
        return s["outs"]
    c, j = s["case"], s["turn"]
    s["turn"] = (j + 1) % _turns(c)
    return {"micro": [_micro(c, s, j)], **_carried(c, s)}


# -------------------------------------------------------------------- costs
def work(c):
    """bytes of the one-pass minimum of both sides; the path does a few
    operations per element and no contraction"""
    es = 4 if c["dtype"] == "f32" else 2
    N, K, op = c["n"] * c["len"], c["n"] * _k(c), c["op"]
    blk = 4 * c["n"] * (-(-c["len"] // 4096) + 1)
    pay = K * (4 + es) + blk
    codes = c["n"] * (4 * -(-c["len"] * c["bits"] // 32) + 8)
    kept = K * 4 + c["n"] * (4 * -(-_k(c) * c["bits"] // 32) + 8) + blk
    per = {"topk": 2 * N * es + 2 * pay,
           "topk_ef": 2 * N * es + 8 * N + 2 * pay,
           "quant": 2 * N * es + 2 * codes,
           "quant_ef": 2 * N * es + 8 * N + 2 * codes,
           "topk_quant_ef": 2 * N * es + 8 * N + 2 * kept,
           "efmix": 2 * N * es + 8 * N + 2 * (pay + blk),
           "aqsgd": 6 * N * es + 2 * pay,
           # forward and backward; the backward list travels without indices
           "module": 4 * N * es + 16 * N + 2 * pay + 2 * (pay + K * es)}[op]
    return {"bytes": c["micro"] * per, "flops": c["micro"] * 4 * N}


def tolerance(c):
    # every operation is defined in IEEE binary32 with fixed roundings, order
    # and tie rules, and both sides of a boundary rely on it: bits stay equal
    return "exact"


# ------------------------------------------------------------------- 64 bits
def _keep(v, k):
    """0/1 mask of each row's k largest magnitudes, ties to the lower index"""
    order = torch.sort(v.abs(), dim=1, descending=True, stable=True).indices[:, :k]
    return torch.zeros_like(v).scatter_(1, order, 1.0)


def _quantized(v, bits):
    lo, hi = v.amin(1, keepdim=True), v.amax(1, keepdim=True)
    top = 2 ** bits - 1
    rng = hi - lo
    codes = torch.round((v - lo) / torch.where(rng > 0, rng, 1) * top).clamp(max=top)
    codes = torch.where(rng > 0, codes, 0)
    return lo + codes * (rng / top), torch.cat([lo, rng / top], 1)


def exact(c, seed):
    """the same pass in 64 bits; values are rounded where they go through the
    wire or a buffer of the tensor's dtype, which is part of what is computed"""
    op, n, L, k, dt = c["op"], c["n"], c["len"], _k(c), DTYPES[c["dtype"]]
    s = _inputs(c, seed)

    def wire(v):
        return v.to(dt).double()

    micro = []
    e = torch.zeros((n, L), dtype=torch.float64, device=DEV)
    if op == "aqsgd":
        m = s["m"].double()
    for j in range(c["micro"]):
        x = s["x"][j].double()
        if op == "topk":
            micro.append({"idx": None, "val": None, "blk": None, "y": x * _keep(x, k)})
        elif op == "topk_ef":
            X = x + e
            y = wire(X * _keep(X, k))
            e = X - y
            micro.append({"idx": None, "val": None, "blk": None, "y": y})
        elif op in ("quant", "quant_ef"):
            X = x + e
            y, meta = _quantized(X, c["bits"])
            if op == "quant_ef":
                e = X - wire(y)
            micro.append({"codes": None, "meta": meta, "y": wire(y)})
        elif op == "topk_quant_ef":
            X = x + e
            keep = _keep(X, k)
            vals, meta = _quantized(X[keep > 0].reshape(n, k), c["bits"])
            y = torch.zeros_like(X)
            y[keep > 0] = wire(vals).reshape(-1)
            e = X - y
            micro.append({"idx": None, "codes": None, "meta": meta, "blk": None, "y": y})
        elif op == "efmix":
            sx = x * _keep(x, k - k // 2)
            se = wire(e * _keep(e, k // 2)) if k // 2 else torch.zeros_like(e)
            e = x + e - wire(sx + se)
            micro.append({"idx": None, "val": None, "idx_e": None, "val_e": None, "y": wire(sx + se)})
        elif op == "aqsgd":
            ids = s["ids"][j]
            d = x - m[ids]
            m[ids] = wire(m[ids] + wire(d * _keep(d, k)))
            micro.append({"idx": None, "val": None, "blk": None, "y": m[ids]})
        else:
            keep = _keep(x, k)
            y, g = x * keep, s["gy"][j].double()
            micro.append({"y": y, "gx": g * keep, "e_fwd": (x - y).reshape(-1), "e_bwd": (g - g * keep).reshape(-1)})
    carried = {}
    if op in ("topk_ef", "quant_ef", "topk_quant_ef", "efmix"):
        carried["e"] = e.reshape(-1)
    elif op == "aqsgd":
        carried["m"] = carried["m_r"] = m
    return {"micro": micro, **carried}
