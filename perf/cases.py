"""Performance cases of one device's share of an ATP transformer layer.

A case is one call (or the forward and the backward call) of the C ABI's
Python binding on one GPU: the linear block of the layer (QKV, out-proj, fc1
with GeLU, fc2, each with its group's Partial(SUM) reduction), the causal
attention core, the attention block chained from them, and the single
pieces a program can call by themselves (one shard linear forward, backward
or fused with its reduction, and the reduction alone).  Sizes are the GPT
layers of synth_inputs.py's workloads (hidden sizes 512 to 20480, sequences of
2048 tokens) and their neighbours.

Inputs are drawn on the GPU from the seed: activations and upstream gradients
N(0, 1), weights N(0, 0.02^2) (0.01 for h = 20480), biases N(0, 0.02^2), the
other group members' partial sums with the spread of a real partial product.
"""
import math

import torch

import paper_2301_08658_amd as atp

DEV = "cuda"
LIN = ("qkv", "out", "fc1", "fc2")
HEAD = 128                      # head dimension of every configuration
MODES = {"col": atp.ATP_BLOCK_COL, "row": atp.ATP_BLOCK_ROW}
LINMODES = {"col": atp.ATP_COL_FIRST, "row": atp.ATP_ROW_FIRST}
EPIS = {"none": atp.ATP_EPI_NONE, "bias": atp.ATP_EPI_BIAS, "bias_gelu": atp.ATP_EPI_BIAS_GELU,
        "gelu_bwd": atp.ATP_EPI_GELU_BWD}
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
LAYOUTS = {"kn": atp.ATP_W_KN, "nk": atp.ATP_W_NK}
BF = torch.bfloat16
MESHES = ((1, 1), (2, 1), (1, 2), (2, 2), (4, 1), (1, 4), (4, 2), (2, 4), (8, 1), (1, 8))


# ------------------------------------------------------------------ the cases
def listed():
    def layer(name, kind, mode, d1, d2, i1, i2, tokens, h, chunks, bwd_chunks=1, partials="f32",
              layout="kn"):
        return dict(name=name, kind=kind, mode=mode, d1=d1, d2=d2, i1=i1, i2=i2, tokens=tokens,
                    h=h, chunks=chunks, bwd_chunks=bwd_chunks, partials=partials, layout=layout,
                    ws=True)

    def attn(name, kind, d1, d2, i1, i2, batch, seq, h, **kw):
        return dict(name=name, kind=kind, mode="col", d1=d1, d2=d2, i1=i1, i2=i2, batch=batch,
                    seq=seq, h=h, **kw)

    return [
        # a small model's training step: launches and latency
        layer("layer_step_h512_2x2", "layer_step", "col", 2, 2, 1, 0, 256, 512, 2, 2),
        # an ordinary GPT layer's forward, four token chunks overlapping their
        # reductions (Sec. 4.1)
        layer("layer_fwd_h4096_2x4", "layer_fwd", "col", 2, 4, 0, 1, 8192, 4096, 4),
        # the transposed arrangement's backward (Sec. 4.2), dX chunked as well
        layer("layer_bwd_h4096_row_4x2", "layer_bwd", "row", 4, 2, 2, 1, 8192, 4096, 4, 4),
        # a GPT-3 sized layer at micro-batch 1 with 16-bit partials (Sec. 5) and
        # weights in torch.nn.Linear's order
        layer("layer_fwd_h12288_4x2_bf16", "layer_fwd", "col", 4, 2, 3, 0, 2048, 12288, 4,
              partials="bf16", layout="nk"),
        # the benchmark's training step of the widest layer: the largest call
        layer("layer_step_h20480_8x1", "layer_step", "col", 8, 1, 0, 0, 4096, 20480, 8, 1),
        # the attention core of a GPT-3 sized layer at micro-batch 1 (12 heads)
        attn("attn_fwd_h12288_4x2", "attn_fwd", 4, 2, 1, 1, 1, 2048, 12288),
        # the attention core's backward of the widest layer (20 heads)
        attn("attn_bwd_h20480_8x1", "attn_bwd", 8, 1, 0, 0, 2, 2048, 20480),
        # an ordinary attention block, forward and backward
        attn("attn_block_h4096_2x4", "attn_block", 2, 4, 1, 2, 4, 2048, 4096, chunks=4,
             bwd_chunks=1, partials="f32", layout="kn", ws=True),
        # one linear with its bias and GeLU, sizes off every tile (a ragged
        # batch of prompts)
        dict(name="linear_fwd_1003x2056x1608", kind="linear_fwd", mode="row", d1=1, d2=2, i1=0,
             i2=1, tokens=1003, k=1608, n=4112, chunks=1, epi="bias_gelu", y="bf16"),
        # one linear's backward without a workspace
        dict(name="linear_bwd_2048x4096x1024", kind="linear_bwd", mode="col", d1=2, d2=2, i1=1,
             i2=1, tokens=2048, k=2048, n=8192, chunks=2),
        # one linear with its group's reduction fused into the product
        dict(name="linear_fused_2048x6144x12288", kind="linear_fused", mode="row", d1=4, d2=2,
             i1=1, i2=0, tokens=2048, k=49152, n=12288, epi="bias"),
        # the reduction alone, fc1's epilogue, in chunks
        dict(name="reduce_4x8192x8192_gelu", kind="reduce", parts=4, tokens=8192, n=8192, chunks=4,
             partials="f32", epi="bias_gelu", out="bf16"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _tokens(rng, lo, hi):
    """Token counts: often a multiple of 64, as batch x sequence is, else any."""
    t = int(_log(rng, lo, hi))
    return max(lo, t // 64 * 64) if rng.random() < 0.6 else max(lo, t)


def _chunks(rng, tokens):
    return rng.choice([c for c in (1, 2, 4, 8) if tokens % c == 0 and tokens // c >= 16] or [1])


def _hidden(rng, d, lo, hi):
    """A hidden size whose heads divide over the mesh."""
    u = HEAD * d
    return max(1, round(_log(rng, max(lo, u), max(hi, u)) / u)) * u


LARGEST = 24.0 * 4096 * 20480 * 20480 * 3 / 8       # flops of the largest listed case


def draw(rng):
    kind = rng.choice(("layer_fwd", "layer_bwd", "layer_step", "attn_fwd", "attn_bwd",
                       "attn_block", "linear_fwd", "linear_bwd", "linear_fused", "reduce"))
    while True:
        d1, d2 = rng.choice(MESHES)
        c = dict(kind=kind, mode=rng.choice(("col", "row")), d1=d1, d2=d2,
                 i1=rng.randrange(d1), i2=rng.randrange(d2))
        if kind.startswith("layer"):
            tokens = _tokens(rng, 64, 8192)
            c.update(tokens=tokens, h=_hidden(rng, d1 * d2, 512, 16384),
                     chunks=_chunks(rng, tokens), bwd_chunks=1,
                     partials=rng.choice(("f32", "f32", "bf16")),
                     layout=rng.choice(("kn", "nk")), ws=rng.random() < 0.8)
            if rng.random() < 0.3:
                c["bwd_chunks"] = c["chunks"]
        elif kind.startswith("attn"):
            seq = _tokens(rng, 64, 4096)
            c.update(batch=min(int(_log(rng, 1, 8.99)), 16384 // seq), seq=seq,
                     h=_hidden(rng, d1 * d2, 512, 12288))
            if kind == "attn_block":
                c.update(chunks=_chunks(rng, c["batch"] * seq), bwd_chunks=1,
                         partials=rng.choice(("f32", "f32", "bf16")),
                         layout=rng.choice(("kn", "nk")), ws=rng.random() < 0.8)
        elif kind.startswith("linear"):
            tokens = _tokens(rng, 16, 8192)
            k = int(_log(rng, 64, 12288)) // 8 * 8
            n = int(_log(rng, 64, 12288)) // 8 * 8
            row = c["mode"] == "row"
            red = d1 if row else d2
            c.update(tokens=tokens, k=k * red, n=n * (d2 if row else d1))
            if kind == "linear_fwd":
                c.update(chunks=_chunks(rng, tokens), y=rng.choice(("f32", "bf16")),
                         epi=rng.choice(("bias", "bias_gelu")) if red == 1 else "none")
            elif kind == "linear_bwd":
                c["chunks"] = _chunks(rng, tokens)
            else:
                c["epi"] = rng.choice(("bias", "bias_gelu"))
        else:
            tokens = _tokens(rng, 16, 8192)
            c = dict(kind=kind, parts=rng.choice((2, 4, 8)), tokens=tokens,
                     n=int(_log(rng, 64, 20480)) // 8 * 8, chunks=_chunks(rng, tokens),
                     partials=rng.choice(("f32", "f32", "bf16")),
                     epi=rng.choice(("none", "bias", "bias_gelu", "gelu_bwd")),
                     out="bf16")
        if work(c)["flops"] <= LARGEST and work(c)["bytes"] <= 16e9:
            return c


# ------------------------------------------------------------------ inputs
class Draw:
    """Seeded normal draws on the GPU, the same for prepare() and exact()."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def __call__(self, shape, std, dtype=BF):
        t = torch.randn(shape, generator=self.g, dtype=torch.float32, device=DEV)
        return (t if std == 1.0 else t.mul_(std)).to(dtype)


def _sigma(case):
    return 0.01 if case["h"] >= 20480 else 0.02


def _mesh(case):
    return atp.mesh(case["d1"], case["d2"], case["i1"], case["i2"])


def _shape(case, mode, k, n):
    """Local sizes of a shard linear (Sec. 3.2): k_loc, n_loc, the forward
    reduction's group size and the device's place in it, the backward's."""
    row = mode == "row"
    dk, dn = (case["d1"], case["d2"]) if row else (case["d2"], case["d1"])
    ik, jn = (case["i1"], case["i2"]) if row else (case["i2"], case["i1"])
    return dict(k=k // dk, n=n // dn, red=dk, own=ik, bwd=dn, bown=jn)


def _linears(case):
    h = case["h"]
    modes = ("col", "row", "col", "row") if case["mode"] == "col" else ("row", "col", "row", "col")
    return [_shape(case, m, k, n) for m, k, n in
            zip(modes, (h, h, h, 4 * h), (3 * h, h, 4 * h, h))]


def _heads(case, L):
    """Heads of the QKV block, and the device's first and number of heads."""
    blk = L[0]["n"] // (3 * HEAD)
    hd = blk // L[0]["red"]
    return blk, L[0]["own"] * hd, hd


def _group(D, size, own, shape, std, dtype):
    """The group's partial buffers; the device's own is written by the call."""
    if size == 1:
        return None
    return [torch.zeros(shape, dtype=dtype, device=DEV) if j == own else D(shape, std, dtype)
            for j in range(size)]


def _empty(r, c, dtype=BF):
    return torch.empty((r, c), dtype=dtype, device=DEV)


def _layer_inputs(case, seed):
    D, L, sw = Draw(seed), _linears(case), _sigma(case)
    T, pdt = case["tokens"], DTYPES[case["partials"]]
    s = dict(L=L, x=D((T, L[0]["k"]), 1.0), a=D((T, L[1]["k"]), 1.0),
             w=[D((g["k"], g["n"]), sw) for g in L], b=[D((g["n"],), 0.02) for g in L])
    if case["kind"] != "layer_bwd":
        s["parts"] = [_group(D, g["red"], g["own"], (T, g["n"]), math.sqrt(g["k"]) * sw, pdt)
                      for g in L]
    if case["kind"] == "layer_bwd":
        s["pre"] = D((T, L[2]["n"]), math.sqrt(case["h"]) * sw)
        s["hact"] = torch.nn.functional.gelu(s["pre"].float()).to(BF)
    if case["kind"] != "layer_fwd":
        s["dz"], s["dqkv"], s["do"] = (D((T, L[i]["n"]), 1.0) for i in (3, 0, 1))
        s["dparts"] = [_group(D, g["bwd"], g["bown"], (T, g["k"]), math.sqrt(g["n"]) * sw, pdt)
                       for g in L]
    return s


def _store_weights(case, w):
    return w if case["layout"] == "kn" else [t.t().contiguous() for t in w]


def _prepare_layer(case, seed):
    s = _layer_inputs(case, seed)
    L, T = s["L"], case["tokens"]
    s["w"] = _store_weights(case, s["w"])
    s["m"], s["bm"] = _mesh(case), MODES[case["mode"]]
    s["comm"] = torch.cuda.Stream()
    lay = LAYOUTS[case["layout"]]
    s["work"] = None
    if case["ws"]:
        nb = atp.atp_block_workspace_bytes(s["m"], s["bm"], T, case["h"], case["chunks"], lay)
        s["work"] = torch.empty(nb, dtype=torch.uint8, device=DEV)
    if case["kind"] != "layer_bwd":
        s.update(qkv=_empty(T, L[0]["n"]), o=_empty(T, L[1]["n"]), hact=_empty(T, L[2]["n"]),
                 pre=_empty(T, L[2]["n"]), z=_empty(T, L[3]["n"]))
    if case["kind"] != "layer_fwd":
        s.update(dh_pre=_empty(T, L[2]["n"]), dx_qkv=_empty(T, L[0]["k"]),
                 dx_fc1=_empty(T, L[2]["k"]), d_attn=_empty(T, L[1]["k"]),
                 dw=[torch.empty_like(w, dtype=torch.float32) for w in s["w"]],
                 db=[torch.empty(g["n"], device=DEV) for g in L])
    return s


def _attn_cols(case, L):
    blk, first, hd = _heads(case, L)
    return blk, slice(first * 3 * HEAD, (first + hd) * 3 * HEAD), slice(first * HEAD,
                                                                        (first + hd) * HEAD)


def _core(case, L, qkv, dt, dout=None):
    """The device's heads' causal attention of a QKV block in plain torch, a
    few (sequence, head) pairs at a time: output token rows, row log-sum-exps
    [heads, tokens] and, with the output gradient's token rows, d_qkv's
    columns of those heads."""
    _, cq, _ = _attn_cols(case, L)
    B, S = case["batch"], case["seq"]
    H = (cq.stop - cq.start) // (3 * HEAD)
    t = qkv[:, cq].reshape(B, S, H, 3, HEAD).permute(3, 0, 2, 1, 4).reshape(3, B * H, S, HEAD)
    o = torch.empty((B * H, S, HEAD), dtype=dt, device=DEV)
    lse = torch.empty((B * H, S), dtype=dt, device=DEV)
    d = None
    if dout is not None:
        d = torch.empty((3, B * H, S, HEAD), dtype=dt, device=DEV)
        dout = dout.reshape(B, S, H, HEAD).permute(0, 2, 1, 3).reshape(B * H, S, HEAD)
    future = torch.ones(S, S, dtype=torch.bool, device=DEV).triu_(1)
    step = max(1, (1 << 28) // (S * S))
    for i in range(0, B * H, step):
        q, k, v = (t[j, i:i + step].to(dt) for j in range(3))
        p = torch.matmul(q, k.transpose(-1, -2).contiguous()).mul_(1.0 / math.sqrt(HEAD))
        p.masked_fill_(future, -math.inf)
        lse[i:i + step] = torch.logsumexp(p, -1)
        p.sub_(lse[i:i + step, :, None]).exp_()
        o[i:i + step] = torch.matmul(p, v)
        if dout is None:
            continue
        do = dout[i:i + step].to(dt)
        d[2, i:i + step] = torch.matmul(p.transpose(-1, -2).contiguous(), do)
        ds = torch.matmul(do, v.transpose(-1, -2).contiguous())
        ds.sub_((do * o[i:i + step]).sum(-1, keepdim=True)).mul_(p).mul_(1.0 / math.sqrt(HEAD))
        d[0, i:i + step] = torch.matmul(ds, k)
        d[1, i:i + step] = torch.matmul(ds.transpose(-1, -2).contiguous(), q)
    o = o.reshape(B, H, S, HEAD).permute(0, 2, 1, 3).reshape(B * S, H * HEAD)
    lse = lse.reshape(B, H, S).transpose(0, 1).reshape(H, B * S)
    if d is not None:
        d = d.reshape(3, B, H, S, HEAD).permute(1, 3, 2, 0, 4).reshape(B * S, H * 3 * HEAD)
    return o, lse, d


def _attn_inputs(case, seed):
    D, L = Draw(seed), _linears(case)
    T = case["batch"] * case["seq"]
    s = dict(L=L, qkv=D((T, L[0]["n"]), 1.0))
    if case["kind"] == "attn_bwd":
        s["d_out"] = D((T, L[1]["k"]), 1.0)
    return s


def _prepare_attn(case, seed):
    s = _attn_inputs(case, seed)
    L, T = s["L"], case["batch"] * case["seq"]
    hd = _heads(case, L)[2]
    s["m"], s["bm"] = _mesh(case), MODES[case["mode"]]
    s["out"] = torch.zeros((T, L[1]["k"]), dtype=BF, device=DEV)
    s["lse"] = torch.empty((hd, T), device=DEV)
    if case["kind"] == "attn_bwd":
        # the forward's saved output and row log-sum-exps
        o, lse, _ = _core(case, L, s["qkv"], torch.float32)
        s["out"][:, _attn_cols(case, L)[2]] = o.to(BF)
        s["lse"].copy_(lse)
        s["d_qkv"] = torch.zeros_like(s["qkv"])
        s["delta"] = torch.empty((hd, T), device=DEV)
    return s


def _attn_block_inputs(case, seed):
    D, L, sw = Draw(seed), _linears(case), _sigma(case)
    T, pdt = case["batch"] * case["seq"], DTYPES[case["partials"]]
    q, o = L[0], L[1]
    return dict(
        L=L, x=D((T, q["k"]), 1.0), w=[D((g["k"], g["n"]), sw) for g in (q, o)],
        b=[D((g["n"],), 0.02) for g in (q, o)],
        # the QKV block has unit spread, so the scores do
        qparts=_group(D, q["red"], q["own"], (T, q["n"]), math.sqrt(q["k"]) * sw, pdt),
        oparts=_group(D, o["red"], o["own"], (T, o["n"]), math.sqrt(o["k"]) * sw, pdt),
        # the other members' heads of the gathered block and of its gradient
        attn=D((T, o["k"]), 1.0), d_qkv=D((T, q["n"]), 1.0), d_o=D((T, o["n"]), 1.0),
        daparts=_group(D, o["bwd"], o["bown"], (T, o["k"]), math.sqrt(o["n"]) * sw, pdt),
        dxparts=_group(D, q["bwd"], q["bown"], (T, q["k"]), math.sqrt(q["n"]) * sw, pdt))


def _prepare_attn_block(case, seed):
    s = _attn_block_inputs(case, seed)
    L, T = s["L"], case["batch"] * case["seq"]
    hd = _heads(case, L)[2]
    s["w"] = _store_weights(case, s["w"])
    s["m"], s["bm"] = _mesh(case), MODES[case["mode"]]
    s["comm"] = torch.cuda.Stream()
    s["work"] = None
    if case["ws"]:
        nb = atp.atp_block_workspace_bytes(s["m"], s["bm"], T, case["h"], case["chunks"],
                                           LAYOUTS[case["layout"]])
        s["work"] = torch.empty(nb, dtype=torch.uint8, device=DEV)
    s.update(qkv=_empty(T, L[0]["n"]), lse=torch.empty((hd, T), device=DEV),
             o=_empty(T, L[1]["n"]), d_attn=_empty(T, L[1]["k"]),
             delta=torch.empty((hd, T), device=DEV), dx=_empty(T, L[0]["k"]),
             dw=[torch.empty_like(w, dtype=torch.float32) for w in s["w"]],
             db=[torch.empty(g["n"], device=DEV) for g in L[:2]])
    return s


def _linear_inputs(case, seed):
    D, g = Draw(seed), _shape(case, case["mode"], case["k"], case["n"])
    T = case["tokens"]
    s = dict(g=g, x=D((T, g["k"]), 1.0), w=D((g["k"], g["n"]), 0.02), b=D((g["n"],), 0.02))
    if case["kind"] == "linear_bwd":
        s["dy"] = D((T, g["n"]), 1.0)
    if case["kind"] == "linear_fused":
        s["peers"] = [None if j == g["own"] else
                      D((T, g["n"]), math.sqrt(g["k"]) * 0.02, torch.float32)
                      for j in range(g["red"])]
    return s


def _prepare_linear(case, seed):
    s = _linear_inputs(case, seed)
    g, T = s["g"], case["tokens"]
    s["m"] = _mesh(case)
    if case["kind"] == "linear_bwd":
        s.update(dx=_empty(T, g["k"], torch.float32), dw=_empty(g["k"], g["n"], torch.float32),
                 db=torch.empty(g["n"], device=DEV))
    else:
        s["y"] = _empty(T, g["n"], DTYPES[case["y"]] if case["kind"] == "linear_fwd" else BF)
        s["pre"] = _empty(T, g["n"]) if case["epi"] == "bias_gelu" else None
    return s


def _reduce_inputs(case, seed):
    D, T, n = Draw(seed), case["tokens"], case["n"]
    return dict(parts=[D((T, n), 1.0, DTYPES[case["partials"]]) for _ in range(case["parts"])],
                b=D((n,), 0.02) if "bias" in case["epi"] else None,
                pin=D((T, n), 1.0) if case["epi"] == "gelu_bwd" else None)


def _prepare_reduce(case, seed):
    s = _reduce_inputs(case, seed)
    T, n = case["tokens"], case["n"]
    s["y"] = _empty(T, n, DTYPES[case["out"]])
    s["pre"] = _empty(T, n) if case["epi"] == "bias_gelu" else None
    return s


def prepare(case, seed):
    kind = case["kind"]
    if kind.startswith("layer"):
        s = _prepare_layer(case, seed)
    elif kind == "attn_block":
        s = _prepare_attn_block(case, seed)
    elif kind.startswith("attn"):
        s = _prepare_attn(case, seed)
    elif kind.startswith("linear"):
        s = _prepare_linear(case, seed)
    else:
        s = _prepare_reduce(case, seed)
    s["case"] = dict(case)
    return s


# ------------------------------------------------------------------ one pass
def _owns(groups, L, own):
    """The own partials that a call writes beside its reduced outputs."""
    return [p[g[own]] if p is not None else None for p, g in zip(groups, L)]


def _run_layer(c, s):
    out = {}
    lay = LAYOUTS[c["layout"]]
    if c["kind"] != "layer_bwd":
        atp.atp_block_fwd(s["m"], s["bm"], c["tokens"], c["h"], c["chunks"], s["w"], s["b"],
                          s["x"], s["a"], s["parts"], s["qkv"], s["o"], s["hact"], s["pre"],
                          s["z"], workspace=s["work"], comm_stream=s["comm"], weight_layout=lay)
        out.update(qkv=s["qkv"], o=s["o"], h=s["hact"], pre=s["pre"], z=s["z"],
                   own=_owns(s["parts"], s["L"], "own"))
    if c["kind"] != "layer_fwd":
        atp.atp_block_bwd(s["m"], s["bm"], c["tokens"], c["h"], c["bwd_chunks"], s["w"], s["b"],
                          s["x"], s["a"], s["hact"], s["pre"], s["dz"], s["dqkv"], s["do"],
                          s["dparts"], s["dh_pre"], s["dx_qkv"], s["dx_fc1"], s["d_attn"],
                          s["dw"], s["db"], workspace=s["work"], comm_stream=s["comm"],
                          weight_layout=lay)
        out.update(dh_pre=s["dh_pre"], dx_qkv=s["dx_qkv"], dx_fc1=s["dx_fc1"],
                   d_attn=s["d_attn"], dw=s["dw"], db=s["db"],
                   down=_owns(s["dparts"], s["L"], "bown"))
    return out


def _run_attn(c, s):
    if c["kind"] == "attn_fwd":
        atp.atp_attention_fwd(s["m"], s["bm"], c["batch"], c["seq"], c["h"], c["h"] // HEAD,
                              s["qkv"], s["out"], s["lse"])
        return dict(out=s["out"], lse=s["lse"])
    atp.atp_attention_bwd(s["m"], s["bm"], c["batch"], c["seq"], c["h"], c["h"] // HEAD, s["qkv"],
                          s["out"], s["lse"], s["d_out"], s["d_qkv"], s["delta"])
    return dict(d_qkv=s["d_qkv"])


def _run_attn_block(c, s):
    lay = LAYOUTS[c["layout"]]
    heads = c["h"] // HEAD
    atp.atp_attention_block_fwd(s["m"], s["bm"], c["batch"], c["seq"], c["h"], heads, c["chunks"],
                                s["w"], s["b"], s["x"], s["qparts"], s["qkv"], s["attn"],
                                s["lse"], s["oparts"], s["o"], workspace=s["work"],
                                comm_stream=s["comm"], weight_layout=lay)
    atp.atp_attention_block_bwd(s["m"], s["bm"], c["batch"], c["seq"], c["h"], heads,
                                c["bwd_chunks"], s["w"], s["b"], s["x"], s["qkv"], s["attn"],
                                s["lse"], s["d_o"], s["daparts"], s["d_attn"], s["delta"],
                                s["d_qkv"], s["dxparts"], s["dx"], s["dw"], s["db"],
                                workspace=s["work"], comm_stream=s["comm"], weight_layout=lay)
    return dict(qkv=s["qkv"], attn=s["attn"], lse=s["lse"], o=s["o"], d_attn=s["d_attn"],
                d_qkv=s["d_qkv"], dx=s["dx"], dw=s["dw"], db=s["db"],
                own=_owns((s["qparts"], s["oparts"]), s["L"], "own"),
                down=_owns((s["dxparts"], s["daparts"]), s["L"], "bown"))


def _run_linear(c, s):
    mode = LINMODES[c["mode"]]
    if c["kind"] == "linear_bwd":
        atp.atp_shard_linear_bwd(s["m"], mode, c["tokens"], c["k"], c["n"], c["chunks"], s["x"],
                                 s["w"], s["dy"], s["dx"], s["dw"], s["db"])
        return dict(dx=s["dx"], dw=s["dw"], db=s["db"])
    if c["kind"] == "linear_fused":
        atp.atp_shard_linear_fwd_fused(s["m"], mode, c["tokens"], c["k"], c["n"], s["x"], s["w"],
                                       s["peers"], s["b"], EPIS[c["epi"]], s["y"],
                                       preact=s["pre"])
    else:
        atp.atp_shard_linear_fwd(s["m"], mode, c["tokens"], c["k"], c["n"], c["chunks"], s["x"],
                                 s["w"], s["b"] if c["epi"] != "none" else None, EPIS[c["epi"]],
                                 s["y"], preact=s["pre"])
    return dict(y=s["y"], pre=s["pre"])


def _run_reduce(c, s):
    f = atp.atp_chunked_partial_reduce if c["partials"] == "f32" else \
        atp.atp_chunked_partial_reduce_bf16
    f(c["parts"], c["tokens"], c["n"], c["chunks"], s["parts"], s["b"], EPIS[c["epi"]], s["y"],
      preact_in=s["pin"], preact_out=s["pre"])
    return dict(y=s["y"], pre=s["pre"])


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind.startswith("layer"):
        return _run_layer(c, s)
    if kind == "attn_block":
        return _run_attn_block(c, s)
    if kind.startswith("attn"):
        return _run_attn(c, s)
    if kind.startswith("linear"):
        return _run_linear(c, s)
    return _run_reduce(c, s)


# ------------------------------------------------------------------ what it needs
def work(case):
    kind = case["kind"]
    if kind == "reduce":
        el, e = case["tokens"] * case["n"], 4 if case["partials"] == "f32" else 2
        extra = {"none": 0, "bias": 0, "bias_gelu": 2, "gelu_bwd": 2}[case["epi"]]
        return dict(bytes=el * (case["parts"] * e + extra + (2 if case["out"] == "bf16" else 4)),
                    flops=el * case["parts"])
    if kind.startswith("linear"):
        g, T = _shape(case, case["mode"], case["k"], case["n"]), case["tokens"]
        k, n = g["k"], g["n"]
        if kind == "linear_bwd":
            return dict(bytes=2 * (T * k + k * n + T * n) + 4 * (T * k + k * n + n),
                        flops=4 * T * k * n)
        y = 4 if case.get("y") == "f32" else 2
        b = 2 * (T * k + k * n + n) + y * T * n + (2 * T * n if case["epi"] == "bias_gelu" else 0)
        if kind == "linear_fused":
            b += 4 * (g["red"] - 1) * T * n
        return dict(bytes=b, flops=2 * T * k * n)
    L = _linears(case)
    if kind.startswith("layer"):
        T, pe = case["tokens"], 4 if case["partials"] == "f32" else 2
        b = f = 0
        wb = sum(2 * g["k"] * g["n"] for g in L)
        if kind != "layer_bwd":
            f += sum(2 * T * g["k"] * g["n"] for g in L)
            # x, the attention block, weights, every member's partial (the own
            # one written), the outputs and the pre-activation
            b += 2 * T * (L[0]["k"] + L[1]["k"]) + wb
            b += sum(T * g["n"] * (pe * g["red"] * (g["red"] > 1) + 2) for g in L)
            b += 2 * T * L[2]["n"]
        if kind != "layer_fwd":
            f += sum(4 * T * g["k"] * g["n"] for g in L)
            # x, attention block, H, pre; the three upstream gradients; weights
            b += 2 * T * (L[0]["k"] + L[1]["k"] + 2 * L[2]["n"] + L[3]["n"] + L[0]["n"] +
                          L[1]["n"]) + wb
            # dX (dh_pre for fc2) with their groups' partials, dW, db
            b += sum(T * g["k"] * (pe * g["bwd"] * (g["bwd"] > 1) + 2) for g in L)
            b += sum(4 * g["k"] * g["n"] + 4 * g["n"] for g in L)
        return dict(bytes=b, flops=f)
    T, S = case["batch"] * case["seq"], case["seq"]
    hd = _heads(case, L)[2]
    pairs = case["batch"] * hd * S * (S + 1) // 2
    fw = dict(bytes=T * hd * (4 * HEAD * 2 + 4), flops=4 * HEAD * pairs)
    bw = dict(bytes=T * hd * (8 * HEAD * 2 + 4), flops=10 * HEAD * pairs)
    if kind == "attn_fwd":
        return fw
    if kind == "attn_bwd":
        return bw
    pe = 4 if case["partials"] == "f32" else 2
    b, f = fw["bytes"] + bw["bytes"], fw["flops"] + bw["flops"]
    for g in L[:2]:
        f += 6 * T * g["k"] * g["n"]
        b += 2 * (2 * T * g["k"] + 2 * T * g["n"] + 2 * g["k"] * g["n"]) + 4 * g["k"] * g["n"]
        b += T * pe * (g["n"] * g["red"] * (g["red"] > 1) + g["k"] * g["bwd"] * (g["bwd"] > 1))
    return dict(bytes=b, flops=f)


def tolerance(case):
    """Relative 2-norm.  Outputs rounded to bf16 sit 1.7e-3 to 2.6e-3 from the
    64-bit result (measured), the attention block's up to 7e-3 where its scores
    are sharp; what one linear stores in fp32 only (its partial, dX, dW, db)
    4e-7, and differs by the order of fp32 sums."""
    kind = case["kind"]
    if kind == "linear_bwd" or (kind == "linear_fwd" and case["y"] == "f32" and
                                case["epi"] == "none"):
        return dict(rel=5e-6)
    return dict(rel=2e-2 if kind == "attn_block" else 1e-2)


# ------------------------------------------------------------------ 64-bit results
F64 = torch.float64


def _mm(a, b):
    return torch.matmul(a.to(F64), b.to(F64))


def _gelu(x):
    return 0.5 * x * (1.0 + torch.erf(x / math.sqrt(2.0)))


def _gelu_grad(x):
    return 0.5 * (1.0 + torch.erf(x / math.sqrt(2.0))) + \
        x * torch.exp(-0.5 * x * x) / math.sqrt(2.0 * math.pi)


def _sum(p, group, own):
    """The group's sum with the device's exact partial in its place."""
    if group is None:
        return p
    for j, t in enumerate(group):
        if j != own:
            p = p + t.to(F64)
    return p


def _linear64(out, key, p, group, own):
    out[key].append(p if group is not None else None)
    return _sum(p, group, own)


def _exact_layer(case, seed):
    s = _layer_inputs(case, seed)
    L, w, b = s["L"], s["w"], s["b"]
    out, fwd, bwd = {}, case["kind"] != "layer_bwd", case["kind"] != "layer_fwd"
    if fwd:
        out["own"] = []
        ys = []
        for i, g in enumerate(L):
            a = (s["x"], s["a"], s["x"], None)[i] if i < 3 else out["h"]
            y = _linear64(out, "own", _mm(a, w[i]), s["parts"][i], g["own"]) + b[i].to(F64)
            if i == 2:
                out["pre"], out["h"] = y, _gelu(y)
            ys.append(y)
        out.update(qkv=ys[0], o=ys[1], z=ys[3])
    if bwd:
        hact = out["h"] if fwd else s["hact"].to(F64)
        pre = out["pre"] if fwd else s["pre"].to(F64)
        down = {}
        dy = [s["dqkv"].to(F64), s["do"].to(F64), None, s["dz"].to(F64)]
        dx, dw, db = [None] * 4, [None] * 4, [None] * 4
        x_in = (s["x"], s["a"], s["x"], hact)
        for i in (3, 0, 1, 2):
            g = L[i]
            if i == 2:
                dy[2] = dx[3] * _gelu_grad(pre)
            p = _mm(dy[i], w[i].t())
            down[i] = p if s["dparts"][i] is not None else None
            dx[i] = _sum(p, s["dparts"][i], g["bown"])
            dw[i] = _mm(x_in[i].t(), dy[i])
            if case["layout"] == "nk":
                dw[i] = dw[i].t().contiguous()
            db[i] = dy[i].sum(0)
        out.update(dh_pre=dy[2], dx_qkv=dx[0], dx_fc1=dx[2], d_attn=dx[1], dw=dw, db=db,
                   down=[down[i] for i in range(4)])
    return out


def _exact_attn(case, seed):
    s = _attn_inputs(case, seed)
    L = s["L"]
    T = case["batch"] * case["seq"]
    _, cq, co = _attn_cols(case, L)
    if case["kind"] == "attn_fwd":
        out = torch.zeros((T, L[1]["k"]), dtype=F64, device=DEV)
        out[:, co], lse, _ = _core(case, L, s["qkv"], F64)
        return dict(out=out, lse=lse)
    d = torch.zeros((T, L[0]["n"]), dtype=F64, device=DEV)
    d[:, cq] = _core(case, L, s["qkv"], F64, s["d_out"][:, co])[2]
    return dict(d_qkv=d)


def _exact_attn_block(case, seed):
    s = _attn_block_inputs(case, seed)
    L, w, b = s["L"], s["w"], s["b"]
    q, o = L[0], L[1]
    _, cq, co = _attn_cols(case, L)
    out = dict(own=[])
    out["qkv"] = _linear64(out, "own", _mm(s["x"], w[0]), s["qparts"], q["own"]) + b[0].to(F64)
    p = _mm(s["d_o"], w[1].t())
    da_own = p if s["daparts"] is not None else None
    out["d_attn"] = _sum(p, s["daparts"], o["bown"])
    attn, d_qkv = s["attn"].to(F64), s["d_qkv"].to(F64)
    attn[:, co], out["lse"], d_qkv[:, cq] = _core(case, L, out["qkv"], F64, out["d_attn"][:, co])
    out["attn"], out["d_qkv"] = attn, d_qkv
    out["o"] = _linear64(out, "own", _mm(attn, w[1]), s["oparts"], o["own"]) + b[1].to(F64)
    p = _mm(d_qkv, w[0].t())
    out["down"] = [p if s["dxparts"] is not None else None, da_own]
    out["dx"] = _sum(p, s["dxparts"], q["bown"])
    dw = [_mm(s["x"].t(), d_qkv), _mm(attn.t(), s["d_o"])]
    out["dw"] = [t.t().contiguous() for t in dw] if case["layout"] == "nk" else dw
    out["db"] = [d_qkv.sum(0), s["d_o"].to(F64).sum(0)]
    return out


def _exact_linear(case, seed):
    s = _linear_inputs(case, seed)
    if case["kind"] == "linear_bwd":
        return dict(dx=_mm(s["dy"], s["w"].t()), dw=_mm(s["x"].t(), s["dy"]),
                    db=s["dy"].to(F64).sum(0))
    y = _mm(s["x"], s["w"])
    if case["kind"] == "linear_fused":
        y = _sum(y, s["peers"], s["g"]["own"])
    if case["epi"] != "none":
        y = y + s["b"].to(F64)
    if case["epi"] == "bias_gelu":
        return dict(y=_gelu(y), pre=y)
    return dict(y=y, pre=None)


def _exact_reduce(case, seed):
    s = _reduce_inputs(case, seed)
    y = sum(t.to(F64) for t in s["parts"])
    if s["b"] is not None:
        y = y + s["b"].to(F64)
    if case["epi"] == "bias_gelu":
        return dict(y=_gelu(y), pre=y)
    if case["epi"] == "gelu_bwd":
        y = y * _gelu_grad(s["pin"].to(F64))
    return dict(y=y, pre=None)


def exact(case, seed):
    kind = case["kind"]
    if kind.startswith("layer"):
        return _exact_layer(case, seed)
    if kind == "attn_block":
        return _exact_attn_block(case, seed)
    if kind.startswith("attn"):
        return _exact_attn(case, seed)
    if kind.startswith("linear"):
        return _exact_linear(case, seed)
    return _exact_reduce(case, seed)
