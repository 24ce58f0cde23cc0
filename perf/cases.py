"""The work that performance is judged on: one quantised linear layer per case, as a model server calls it.

A pass is what the server does for one layer and one batch of tokens: quantise the activations (or the gated
product that feeds a down projection) and run the layer on the codes, through the functions of
`paper_2603_08185_amd.binding`.  Weights, packed once, the workspace and the output buffers are what such a
program keeps.  Three forms of the layer are covered: the integer layer (W4A8 / W4A4, 16-bit or 4-bit
compensation matrix), the MXFP4 layer, and the layer with group-128 weight scales and asymmetric activations.

A case:
  form      "int", "mx" or "g128"
  abits     4 or 8 (4 for "mx")
  M, K, N   tokens, input channels, output channels
  r, rform  rank of the compensation matrix (0: none) and its form: "bf16", "fp16", "i4" (mx: always MXFP4)
  inp, out  storage types of the activations and of Y
  glu       the input is silu(G) * U of two buffers (the down projection of a gated MLP)
  flat      the flattening multiply is done by the quantiser (False: folded into the previous layer)
"""
import math

import torch

from paper_2603_08185_amd import binding as B

DT = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}


def _case(name, form, abits, M, K, N, r, rform="bf16", inp="bf16", out="bf16", glu=False, flat=True):
    return {"name": name, "form": form, "abits": abits, "M": M, "K": K, "N": N, "r": r, "rform": rform, "inp": inp,
            "out": out, "glu": glu, "flat": flat}


def listed():
    return [
        # one token of one user: latency and launches; the up projection of a 7B-class model
        _case("decode_w4a8_m1", "int", 8, 1, 4096, 11008, 128),
        # a decode batch on the widest layer: the weight stream
        _case("decode_w4a4_m24", "int", 4, 24, 8192, 28672, 128),
        # a decode batch in the accuracy setting
        _case("decode_g128_w4a8_m16", "g128", 8, 16, 4096, 11008, 128),
        # a large decode batch or a short prompt: a hundred tokens through the fused q/k/v projection
        _case("batch_w4a8_m100_qkv", "int", 8, 100, 4096, 6144, 128),
        # a chunk of a prompt through a down projection (few channels, long K), gated product quantised where it is made
        _case("chunk_w4a8_m256_down", "int", 8, 256, 11008, 4096, 128, glu=True),
        # a ragged chunk with the all-integer compensation on an attention projection, fp16 model
        _case("chunk_w4a4_i4_m333_o", "int", 4, 333, 4096, 4096, 64, rform="i4", inp="fp16", out="fp16"),
        # a ragged chunk of the MXFP4 model's down projection, flattening folded upstream
        _case("chunk_mx_m200_down", "mx", 4, 200, 14336, 4096, 128, glu=True, flat=False),
        # a ragged chunk in the accuracy setting, fp32 residual stream
        _case("chunk_g128_w4a4_m150_down", "g128", 4, 150, 11008, 4096, 64, out="fp32"),
        # whole prompts: the benchmark layer ...
        _case("prefill_w4a8_m4096_up", "int", 8, 4096, 4096, 11008, 128),
        # ... the widest layer of a W4A4 model (the largest case) ...
        _case("prefill_w4a4_m4096_gateup", "int", 4, 4096, 4096, 28672, 128),
        # ... the MXFP4 model ...
        _case("prefill_mx_m4096_up", "mx", 4, 4096, 4096, 11008, 128),
        # ... and the accuracy setting, prompts that do not fill their last tile
        _case("prefill_g128_w4a8_m3000_qkv", "g128", 8, 3000, 4096, 6144, 128),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    form, abits = rng.choice([("int", 8), ("int", 8), ("int", 4), ("int", 4), ("mx", 4), ("g128", 8), ("g128", 4)])
    unit = 128 if form == "g128" else 64
    most = 4096 * 4096 * 28672 * (0.4 if form == "g128" else 0.8)
    while True:
        M = max(1, min(4096, round(_log(rng, 1, 4096))))
        K = unit * max(1024 // unit, round(_log(rng, 1024, 14336) / unit))
        N = 32 * max(32, round(_log(rng, 1024, 28672) / 32))
        if M * K * N <= most:
            break
    r = rng.choice([0, 32, 64, 96, 128, 256])
    inp = rng.choice(["bf16", "bf16", "fp16"])
    rform = "i4" if form == "int" and rng.random() < 0.3 else inp
    case = _case("", form, abits, M, K, N, r, rform, inp, rng.choice([inp, inp, inp, "fp32"]),
                 form != "g128" and rng.random() < 0.3, rng.random() < 0.7)
    del case["name"]
    return case


def _inputs(case, seed):
    """The tensors of the case: activations with outlier channels, flattening vector, weights (original channel order)."""
    M, K, N, dt = case["M"], case["K"], case["N"], DT[case["inp"]]
    dev = "cuda"
    gen = torch.Generator(device=dev).manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev, dtype=torch.float32)

    def uniform(n, lo, hi):
        return torch.rand(n, generator=gen, device=dev, dtype=torch.float32) * (hi - lo) + lo

    n_out = max(1, K // 100)                             # one channel in a hundred is 30 to 100 times larger
    where = torch.randperm(K, generator=gen, device=dev)[:n_out]
    mult = torch.ones(K, device=dev)
    mult[where] = uniform(n_out, 30.0, 100.0)
    s = uniform(K, 0.5, 2.0) * mult.sqrt()
    W = normal(N, K).mul_(0.02).to(dt)
    if not case["flat"]:                                 # the previous layer has divided by s already
        mult = mult / s
    if case["glu"]:
        G = normal(M, K).mul_(2.0).to(dt)
        X = (normal(M, K) * mult).to(dt)
    else:
        G, X = None, (normal(M, K) * mult).to(dt)
    return G, X, s, W


def _permuted(T, perm):
    return None if T is None else T.index_select(1, perm).contiguous()


def prepare(case, seed):
    """What a server holds for a layer and a batch: the packed layer, the activations, the buffers it reuses."""
    form, abits, M, K, N, r = (case[k] for k in ("form", "abits", "M", "K", "N", "r"))
    dev = "cuda"
    G, X, s, W = _inputs(case, seed)
    st = {"case": case, "Y": torch.empty((M, N), dtype=DT[case["out"]], device=dev)}
    if form == "mx":
        layer = B.mx_pack_weights(W, s, r)
        st["ws"] = B.mx_workspace(M, N, K, dev)
        st["xsc"] = torch.empty(B.lib().serq_mx_act_scale_bytes(M, K), dtype=torch.uint8, device=dev)
    else:
        rdt = DT[case["inp"] if case["rform"] == "i4" else case["rform"]]
        pack = B.pack_weights if form == "int" else B.g128_pack_weights
        layer = pack(W, s, r, r_dtype=rdt)
        st["scale"] = torch.empty(M, dtype=torch.float32, device=dev)
        st["rdt"] = rdt
        st["Rp"] = layer.Rp
        if form == "int":
            st["ws"] = B.workspace(M, N, K, r, abits, dev)
            if case["rform"] == "i4" and r > 0:
                st["Rp"], st["rdt"] = B.pack_lowrank_q4(layer.R), B.I4
        else:
            st["zero"] = torch.empty(M, dtype=torch.int32, device=dev)
    st["Xq"] = torch.empty(B.lib().serq_packed_act_bytes(M, K, abits), dtype=torch.uint8, device=dev)
    perm = layer.perm.long()
    st["X"], st["G"] = _permuted(X, perm), _permuted(G, perm)
    st["s_inv"] = layer.s_inv if case["flat"] else None
    st["layer"] = layer
    return st


def run(st):
    c, L, X, G = st["case"], st["layer"], st["X"], st["G"]
    M, K, N, r = c["M"], c["K"], c["N"], c["r"]
    if c["form"] == "mx":
        if G is not None:
            Xq, xsc = B.mx_swiglu_quantize_act(G, X, st["s_inv"], st["Xq"], st["xsc"])
        else:
            Xq, xsc = B.mx_quantize_act(X, st["s_inv"], st["Xq"], st["xsc"])
        return B.mx_linear(Xq, xsc, L.Wq, L.wsc, M, N, K, Rq=L.Rq, rsc=L.rsc, r=r, Y=st["Y"], ws=st["ws"])
    if c["form"] == "g128":
        Xq, scale, zero = B.quantize_act_asym(X, st["s_inv"], c["abits"], st["Xq"], st["scale"], st["zero"])
        Y = B.g128_linear(Xq, scale, zero, c["abits"], L.Wq, L.gscale, L.wsum, M, N, K, Rp=st["Rp"], r=r,
                          r_dtype=st["rdt"], Y=st["Y"])
        return {"Y": Y, "scale": scale, "zero": zero}
    if G is not None:
        Xq, scale = B.swiglu_quantize_act(G, X, st["s_inv"], c["abits"], st["Xq"], st["scale"])
    else:
        Xq, scale = B.quantize_act(X, st["s_inv"], c["abits"], st["Xq"], st["scale"])
    Y = B.linear(Xq, scale, c["abits"], L.Wq, L.wscale, M, N, K, Rp=st["Rp"], r=r, r_dtype=st["rdt"], Y=st["Y"],
                 ws=st["ws"])
    return {"Y": Y, "scale": scale}


def work(case):
    M, K, N, r = case["M"], case["K"], case["N"], case["r"]
    byt = M * K * 2 * (2 if case["glu"] else 1) + (4 * K if case["flat"] else 0)       # activations, flattening factors
    byt += N * K // 2                                                                  # weight codes
    byt += {"int": 4 * N, "mx": N * K // 32, "g128": N * K // 64 + 4 * N}[case["form"]]  # and their scales
    byt += {"mx": N * r * 17 // 32}.get(case["form"], N * r // 2 if case["rform"] == "i4" else 2 * N * r)
    byt += M * N * (4 if case["out"] == "fp32" else 2) + 4 * M
    return {"bytes": byt, "flops": 2 * M * N * (K + r)}


def tolerance(case):
    # 16-bit outputs: the rounding itself is 1.7e-3 of the result in bf16 and 2e-4 in fp16 (2-norm), and two correct
    # results may round to neighbouring values.  fp32 outputs show the order of the fp32 sums: 5e-8 measured for the
    # integer form, 3e-7 for the group form (its zero-point term cancels), and MXFP4 sums of these sizes come out exact.
    # The gated product is good to a few ulps, not bit-defined: now and then a code moves by one step.
    rel = {"bf16": 6e-3, "fp16": 8e-4, "fp32": 1.2e-6 if case["form"] == "g128" else 4e-7}[case["out"]]
    most = {"bf16": 0.016, "fp16": 0.002, "fp32": 4e-5}[case["out"]]
    return {"rel": max(rel, 3e-4), "max": 0.05} if case["glu"] else {"rel": rel, "max": most}


# ---- the same layer from its definition, in plain torch ------------------------------------------------------
def _over(v, d):
    """v / d as one IEEE division (a Python number as divisor would become a multiplication by its reciprocal)."""
    return v / torch.full_like(v, d)


def _rne_clip(v, sc, q):
    return torch.clamp(torch.round(v / sc), -q, q)


def _mx(v):
    """MXFP4 in blocks of 32 along the last dimension: the values the codes stand for (fp64)."""
    b = v.reshape(*v.shape[:-1], -1, 32).double()
    amax = b.abs().amax(-1, keepdim=True)
    e = torch.clamp(torch.frexp(amax)[1] - 1 - 2, min=-127)           # floor(log2(amax)) - 2
    sc = torch.where(amax > 0, torch.ldexp(torch.ones_like(amax), e), torch.ones_like(amax))
    t = b / sc
    a = t.abs()
    grid = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)
    out = torch.zeros_like(a)
    for i in range(1, 8):                                             # midpoints; ties go to the even code
        mid = 0.5 * (grid[i - 1] + grid[i])
        out = torch.where((a > mid) if i % 2 == 1 else (a >= mid), torch.full_like(a, grid[i]), out)
    return (torch.sign(t) * out * sc).reshape(v.shape)


def exact(case, seed):
    form, abits, M, K, N, r = (case[k] for k in ("form", "abits", "M", "K", "N", "r"))
    G, X, s, W = _inputs(case, seed)
    W = W.float() * s
    perm = torch.sort(W.abs().amax(0), descending=True, stable=True)[1]
    W = W.index_select(1, perm)
    v = X.index_select(1, perm).float()
    if G is not None:
        g = G.index_select(1, perm).double()
        v = (g / (1.0 + torch.exp(-g)) * v.double()).float()
        del g
    if case["flat"]:
        v = v * (torch.ones_like(s) / s).index_select(0, perm)
    if form == "mx":
        x = _mx(v)
        w = _mx(W)
        Y = x @ w.t()
        if r > 0:
            pad = torch.zeros(N, -r % 64, device=W.device)
            R = _mx(torch.cat([W[:, :r] - w[:, :r].float(), pad], 1))[:, :r]
            Y += x[:, :r] @ R.t()
        return Y
    if form == "int":
        ws = W.abs().amax(1, keepdim=True)
        ws = torch.where(ws > 0, _over(ws, 7.0), torch.ones_like(ws))
    else:
        gm = W.reshape(N, K // 128, 128).abs().amax(2)
        gs = torch.where(gm > 0, _over(gm, 7.0).half().float().clamp(2.0 ** -24, 65504.0), torch.ones_like(gm))
        ws = gs.repeat_interleave(128, 1)
    w = _rne_clip(W, ws, 7.0).double() * ws.double()
    R = (W[:, :r].double() - w[:, :r]).float()
    if case["rform"] == "i4":
        R = R.to(DT[case["inp"]]).float()
        rs = R.abs().amax(1, keepdim=True) if r > 0 else torch.zeros(N, 1, device=W.device)
        rs = torch.where(rs > 0, _over(rs, 7.0), torch.ones_like(rs))
        R = _rne_clip(R, rs, 7.0).double() * rs.double()
    else:
        R = R.to(DT[case["rform"]]).double()
    del W, ws
    if form == "int":
        q = float(2 ** (abits - 1) - 1)
        amax = v.abs().amax(1, keepdim=True)
        sc = torch.where(amax > 0, _over(amax, q), torch.ones_like(amax))
        x, zero = _rne_clip(v, sc, q).double(), None
    else:
        top = float(2 ** abits - 1)
        lo, hi = v.amin(1, keepdim=True).clamp(max=0.0), v.amax(1, keepdim=True).clamp(min=0.0)
        sc = torch.where(hi > lo, _over(hi - lo, top), torch.ones_like(hi))
        z = torch.round(-lo / sc)
        x = (torch.clamp(torch.round(v / sc) + z, 0.0, top) - z).double()
        zero = (z.reshape(-1) - 2 ** (abits - 1)).to(torch.int32)
    Y = x @ w.t()
    if r > 0:
        Y += x[:, :r] @ R.t()
    Y *= sc.double()
    out = {"Y": Y, "scale": sc.reshape(-1).double()}
    if zero is not None:
        out["zero"] = zero
    return out
