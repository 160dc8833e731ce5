"""The work by which the speed of this package is followed, as cases that a timing program can prepare and run.

A case is a dict of plain values.  Its "kind" says which part of the framework it exercises, through the public entry
points only (TrainHandle for whole steps, the kernel-level C ABI for the parts of a block at sizes whose host state
would take too long to set up):

  step   one training step of a whole model through TrainHandle (with or without the overlapped host optimizer)
  mlp    the MLP half of a block: norm, gate|up with SwiGLU, down with residual; with train also every gradient
  proj   the projections around attention: norm, q|k|v with the rotary embedding, output with residual; with train
         also every gradient
  attn   causal attention, forward; with train also its backward with the rotary backward folded in
  head   the loss: logits of a token chunk, cross-entropy, the gradients of input and head weights
  norm   RMSNorm forward, backward with the residual add
  embed  embedding lookup, and the gradient of the table

Sizes are those of the five workloads in mt_inputs (tiny, 1.3B, 7B, 14B, 7B at long context), of the tests, or generic
ones between them.  Token ids follow a Zipf-like law, as words in text do.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2604_05091_amd as mt

UNSUPPORTED = -2  # MT_ERR_UNSUPPORTED: the fused form does not take this size, the separate kernels do


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest model anyone trains here: launches, events and host threads decide (the "tiny" workload)
        _step("step-tiny", 2, 256, 4, 4, 64, 688, 1024, 2, 128, adam=True),
        # a small grouped-query model with biases and tied embeddings on sequences that fill no tile (3 x 1000 tokens)
        _step("step-gqa-ragged", 4, 1024, 16, 4, 64, 2816, 8000, 3, 1000, bias=True, tied=True),
        # two layers at the width, vocabulary and batch of the 1.3B workload, optimizer overlapped: the ordinary step
        _step("step-1.3B-2-layers", 2, 2048, 16, 16, 128, 5504, 32000, 8, 2048, adam=True),
        # the MLP of a 7B block, four sequences: two thirds of the FLOPs of the headline workload
        {"name": "mlp-7B", "kind": "mlp", "tokens": 16384, "d": 4096, "ffn": 11008, "train": True},
        # the MLP at 1.3B width on one short sequence of a length that is no multiple of a tile
        {"name": "mlp-1.3B-1000-tokens", "kind": "mlp", "tokens": 1000, "d": 2048, "ffn": 5504, "train": True},
        # the attention projections of a 14B block (grouped KV heads), one sequence
        {"name": "proj-14B", "kind": "proj", "batch": 1, "seq": 4096, "d": 5120, "hq": 40, "hkv": 8, "hd": 128,
         "bias": False, "train": True},
        # attention of a 7B block, four sequences of the headline length
        {"name": "attn-7B", "kind": "attn", "batch": 4, "seq": 4096, "hq": 32, "hkv": 32, "hd": 128, "train": True},
        # long context with grouped KV heads (14B head layout)
        {"name": "attn-14B-32k", "kind": "attn", "batch": 1, "seq": 32768, "hq": 40, "hkv": 8, "hd": 128, "train": True},
        # small heads, few of them, a length that is no multiple of any tile
        {"name": "attn-small-520", "kind": "attn", "batch": 3, "seq": 520, "hq": 8, "hkv": 2, "hd": 64, "train": True},
        # one chunk of the loss at 7B width
        {"name": "head-7B", "kind": "head", "tokens": 8192, "d": 4096, "vocab": 32000},
        # RMSNorm of a 14B block at the full batch
        {"name": "norm-14B", "kind": "norm", "tokens": 65536, "d": 5120},
        # the embedding of the 7B workload at the full batch
        {"name": "embed-7B", "kind": "embed", "tokens": 65536, "d": 4096, "vocab": 32000},
    ]


def _step(name, layers, d, hq, hkv, hd, ffn, vocab, batch, seq, adam=False, bias=False, tied=False, ckpt=1, mlp_chunk=0):
    c = {"kind": "step", "layers": layers, "d": d, "hq": hq, "hkv": hkv, "hd": hd, "ffn": ffn, "vocab": vocab, "batch": batch,
         "seq": seq, "adam": adam, "bias": bias, "tied": tied, "ckpt": ckpt, "mlp_chunk": mlp_chunk}
    return dict(c, name=name) if name else c


def _log(rng, lo, hi, mult):
    """A multiple of mult between lo and hi, spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / mult)) * mult))


def _seq(rng, lo, hi):
    """A sequence length: half of the time whole tiles of 128, otherwise any multiple of 8."""
    return _log(rng, max(lo, 128), hi, 128) if rng.random() < 0.5 else _log(rng, lo, hi, 8)


def _heads(rng, hd, d):
    """Query and KV head counts for a model of width d."""
    hq = max(1, d // hd)
    group = rng.choice([g for g in (1, 1, 2, 4, 5, 8) if hq % g == 0])
    return hq, hq // group


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["mlp"] * 4 + ["proj"] * 3 + ["attn"] * 4 + ["head"] * 2 + ["norm", "embed"])
    if kind == "step":
        hd = rng.choice([64, 128])
        d = _log(rng, 128, 2048, hd)
        hq, hkv = _heads(rng, hd, d)
        ffn = int(round(d * rng.uniform(2.5, 3.0) / 16)) * 16
        vocab = _log(rng, 512, 32000, 8)
        adam = rng.random() < 0.5
        layers = rng.randint(1, 3 if adam else 4)
        seq = _seq(rng, 64, 2048)
        batch = max(1, min(rng.randint(1, 8), 16384 // seq))
        mlp_chunk = rng.choice([0, 0, 0, 512])
        return _step("", layers, d, hq, hkv, hd, ffn, vocab, batch, seq, adam=adam, bias=(not adam and rng.random() < 0.4),
                     tied=rng.random() < 0.3, ckpt=rng.choice([1, 1, 1, 2]), mlp_chunk=mlp_chunk)
    if kind == "mlp":
        d = _log(rng, 256, 5120, 64)
        return {"kind": "mlp", "tokens": _log(rng, 128, 16384, rng.choice([8, 64])), "d": d,
                "ffn": int(round(d * rng.uniform(2.5, 3.0) / 16)) * 16, "train": rng.random() < 0.75}
    if kind == "proj":
        hd = rng.choice([64, 128, 128])
        d = _log(rng, 256, 5120, hd)
        hq, hkv = _heads(rng, hd, d)
        seq = _seq(rng, 128, 4096)
        batch = max(1, min(rng.randint(1, 8), 16384 // seq))
        return {"kind": "proj", "batch": batch, "seq": seq, "d": d, "hq": hq, "hkv": hkv, "hd": hd,
                "bias": rng.random() < 0.3, "train": rng.random() < 0.75}
    if kind == "attn":
        hd = rng.choice([64, 128, 128])
        hkv = rng.choice([1, 2, 4, 8, 16, 32])
        hq = hkv * rng.choice([g for g in (1, 2, 4, 5, 8) if hkv * g <= 40])
        seq = _seq(rng, 128, 32768)
        batch = max(1, min(rng.randint(1, 8), int(2.0e10 / (float(seq) * seq * hq))))
        return {"kind": "attn", "batch": batch, "seq": seq, "hq": hq, "hkv": hkv, "hd": hd, "train": rng.random() < 0.75}
    if kind == "head":
        return {"kind": "head", "tokens": _log(rng, 128, 8192, rng.choice([8, 64])), "d": _log(rng, 256, 5120, 64),
                "vocab": _log(rng, 1024, 32000, 8)}
    if kind == "norm":
        return {"kind": "norm", "tokens": _log(rng, 64, 65536, 8), "d": _log(rng, 256, 8192, 64)}
    return {"kind": "embed", "tokens": _log(rng, 256, 65536, 8), "d": _log(rng, 256, 5120, 64), "vocab": _log(rng, 1024, 32000, 8)}


# ------------------------------------------------------------------ inputs
class _Gen:
    """Tensors on the GPU from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(int(seed))

    def bf16(self, rows, cols, std=1.0):
        return (torch.randn((rows, cols), device="cuda", generator=self.g) * std).to(torch.bfloat16)

    def gain(self, d):
        return (1.0 + 0.1 * torch.randn((d,), device="cuda", generator=self.g)).to(torch.bfloat16)

    def tokens(self, n, vocab):
        """n ids with probability falling like 1 / (rank + 2.7), ranks scattered over the vocabulary."""
        u = torch.rand((n,), device="cuda", generator=self.g, dtype=torch.float64)
        rank = (2.7 * ((vocab + 2.7) / 2.7) ** u - 2.7).to(torch.int64).clamp_(0, vocab - 1)
        return torch.randperm(vocab, device="cuda", generator=self.g)[rank].to(torch.int32)


def _empty(rows, cols, dtype=torch.bfloat16):
    return torch.empty((rows, cols), device="cuda", dtype=dtype)


def _f32(*shape):
    return torch.empty(shape, device="cuda", dtype=torch.float32)


def _rope_tables(T, hd, base=10000.0):
    cs, sn = np.empty((T, hd // 2), np.float32), np.empty((T, hd // 2), np.float32)
    mt.binding.check(mt.lib().mt_k_rope_table(cs.ctypes.data, sn.ctypes.data, T, hd, base))
    return torch.from_numpy(cs).cuda(), torch.from_numpy(sn).cuda()


def _check(status):
    if status != 0:
        mt.binding.check(status)


class _WeightGrad:
    """dW[out, in] = dY^T X with its scratch memory: token-major where the token count allows it, else transposed copies."""

    def __init__(self, n, out, inn):
        self.n, self.out, self.inn = n, out, inn
        self.dw = _f32(out, inn)
        self.direct = n % 64 == 0
        if self.direct:
            cu = torch.cuda.get_device_properties(0).multi_processor_count
            self.split = mt.lib().mt_k_gemm_tn_pick_split(out, inn, n, cu)
            self.ws = _f32(max(1, (self.split - 1) * out * inn))
        else:
            self.ty, self.tx = _empty(out, n), _empty(inn, n)

    def __call__(self, dy, ldy, x, ldx):
        L, n, out, inn = mt.lib(), self.n, self.out, self.inn
        if self.direct:
            _check(L.mt_k_gemm_tn_split(dy, ldy, x, ldx, self.dw.data_ptr(), inn, out, inn, n, 0, self.split, self.ws.data_ptr(), None))
        else:
            ty, tx = self.ty.data_ptr(), self.tx.data_ptr()
            _check(L.mt_k_transpose(dy, ty, n, out, ldy, n, 1, 1, 0, 0, 0, 0, None))
            _check(L.mt_k_transpose(x, tx, n, inn, ldx, n, 1, 1, 0, 0, 0, 0, None))
            _check(L.mt_k_gemm_nt(ty, n, tx, n, self.dw.data_ptr(), inn, None, 0, out, inn, n, 1, 0, None))
        return self.dw


# ------------------------------------------------------------------ whole steps
class _Held(np.ndarray):
    """A view of host memory that belongs to a handle, which it keeps alive."""


def _held(a, owner):
    v = a.view(_Held)
    v.owner = owner
    return v


def _n_params(c):
    nq, nkv = c["hq"] * c["hd"], c["hkv"] * c["hd"]
    layer = (2 * nq + 2 * nkv + 3 * c["ffn"] + 2) * c["d"] + (nq + 2 * nkv if c["bias"] else 0)
    return c["layers"] * layer + (1 if c["tied"] else 2) * c["vocab"] * c["d"] + c["d"]


def _prepare_step(c, g):
    nq, nkv, d = c["hq"] * c["hd"], c["hkv"] * c["hd"], c["d"]
    shapes = [(c["vocab"], d)]
    for _ in range(c["layers"]):
        shapes += [(d,), (nq, d), (nkv, d), (nkv, d), (d, nq), (d,), (c["ffn"], d), (c["ffn"], d), (d, c["ffn"])]
        if c["bias"]:
            shapes += [(nq, 1), (nkv, 1), (nkv, 1)]
    shapes += [(d,)] + ([] if c["tied"] else [(c["vocab"], d)])
    params = []
    for s in shapes:
        if s == (d,):
            params.append(np.ones(s, np.float32))
        else:
            t = torch.randn(s, device="cuda", generator=g.g) * 0.02
            params.append((t.flatten() if s[1] == 1 else t).cpu().numpy())
    ids = g.tokens(c["batch"] * (c["seq"] + 1), c["vocab"]).reshape(c["batch"], c["seq"] + 1).cpu().numpy()
    cfg = mt.ModelCfg.make(c["layers"], d, c["hq"], c["hkv"], c["hd"], c["ffn"], c["vocab"], c["batch"], c["seq"],
                           ckpt_interval=c["ckpt"], qkv_bias=c["bias"], tie_embeddings=c["tied"], mlp_chunk=c["mlp_chunk"])
    h = mt.TrainHandle(cfg, params)
    s = {"h": h, "tokens": np.ascontiguousarray(ids[:, :-1]), "labels": np.ascontiguousarray(ids[:, 1:]), "adam": c["adam"], "n": 0}
    s["out"] = [_held(a, h) for a in h.grads()] + ([_held(p, h) for p in params] if c["adam"] else [])
    return s


def _run_step(s):
    if s["adam"]:
        s["n"] += 1
        loss = s["h"].train_step_adam(s["tokens"], s["labels"], 1e-4, step=s["n"])
    else:
        loss = s["h"].train_step(s["tokens"], s["labels"])
    return {"loss": loss, "state": s["out"]}


# ------------------------------------------------------------------ the MLP of a block
def _prepare_mlp(c, g):
    n, d, F = c["tokens"], c["d"], c["ffn"]
    s = {"n": n, "d": d, "F": F, "train": c["train"], "h1": g.bf16(n, d), "g2": g.gain(d), "wgu": g.bf16(2 * F, d, 0.02),
         "wd": g.bf16(d, F, 0.02), "yn": _empty(n, d), "s": _empty(n, F), "gu": _empty(n, 2 * F), "y": _empty(n, d)}
    if c["train"]:
        s.update(gy=g.bf16(n, d, 1e-3), wdT=_empty(F, d), wguT=_empty(d, 2 * F), ds=_empty(n, F), dgu=_empty(n, 2 * F), dyn=_empty(n, d),
                 dh1=_empty(n, d), dg2=_f32(d), dwd=_WeightGrad(n, d, F), dwgu=_WeightGrad(n, 2 * F, d),
                 ws=torch.empty(mt.lib().mt_k_rmsnorm_bwd_ws_bytes(d), device="cuda", dtype=torch.uint8))
    s["p"] = {k: v.data_ptr() for k, v in s.items() if isinstance(v, torch.Tensor)}
    return s


def _run_mlp(s):
    L, p, n, d, F, train = mt.lib(), s["p"], s["n"], s["d"], s["F"], s["train"]
    _check(L.mt_k_rmsnorm_fwd(p["yn"], p["h1"], p["g2"], n, d, 1e-5, None))
    st = L.mt_k_gemm_nt_swiglu(p["yn"], d, p["wgu"], d, p["gu"] if train else None, 2 * F, p["s"], F, n, F, d, None)
    if st == UNSUPPORTED:
        _check(L.mt_k_gemm_nt(p["yn"], d, p["wgu"], d, p["gu"], 2 * F, None, 0, n, 2 * F, d, 0, 0, None))
        st = L.mt_k_swiglu_fwd(p["s"], p["gu"], n, F, None)
    _check(st)
    _check(L.mt_k_gemm_nt(p["s"], F, p["wd"], F, p["y"], d, p["h1"], d, n, d, F, 0, 0, None))
    if not train:
        return [s["y"], s["s"]]
    _check(L.mt_k_transpose(p["wd"], p["wdT"], d, F, F, d, 1, 1, 0, 0, 0, 0, None))
    _check(L.mt_k_transpose(p["wgu"], p["wguT"], 2 * F, d, d, 2 * F, 1, 1, 0, 0, 0, 0, None))
    dwd = s["dwd"](p["gy"], d, p["s"], F)
    st = L.mt_k_gemm_nt_swiglu_bwd(p["gy"], d, p["wdT"], d, p["dgu"], 2 * F, p["gu"], 2 * F, n, F, d, None)
    if st == UNSUPPORTED:
        _check(L.mt_k_gemm_nt(p["gy"], d, p["wdT"], d, p["ds"], F, None, 0, n, F, d, 0, 0, None))
        st = L.mt_k_swiglu_bwd(p["dgu"], p["ds"], p["gu"], n, F, None)
    _check(st)
    dwgu = s["dwgu"](p["dgu"], 2 * F, p["yn"], d)
    _check(L.mt_k_gemm_nt(p["dgu"], 2 * F, p["wguT"], 2 * F, p["dyn"], d, None, 0, n, d, 2 * F, 0, 0, None))
    _check(L.mt_k_rmsnorm_bwd(p["dh1"], p["dg2"], p["dyn"], p["h1"], p["g2"], p["gy"], p["ws"], n, d, 1e-5, None))
    return [s["y"], s["dh1"], s["dg2"], dwd, dwgu]


# ------------------------------------------------------------------ the projections around attention
def _prepare_proj(c, g):
    n, d, hd = c["batch"] * c["seq"], c["d"], c["hd"]
    nq, nkv = c["hq"] * hd, c["hkv"] * hd
    N = nq + 2 * nkv
    cs, sn = _rope_tables(c["seq"], hd)
    s = {"n": n, "d": d, "T": c["seq"], "hd": hd, "nq": nq, "rot": nq + nkv, "N": N, "train": c["train"], "x": g.bf16(n, d), "g1": g.gain(d),
         "wqkv": g.bf16(N, d, 0.02), "wo": g.bf16(d, nq, 0.02), "att": g.bf16(n, nq, 0.5), "cos": cs, "sin": sn,
         "xn": _empty(n, d), "qkv": _empty(n, N), "h1": _empty(n, d)}
    if c["bias"]:
        s["b"] = g.bf16(1, N, 0.1)
    if c["train"]:
        s.update(dh1=g.bf16(n, d, 1e-3), dqkv=g.bf16(n, N, 1e-3), woT=_empty(nq, d), wqkvT=_empty(d, N), datt=_empty(n, nq), dxn=_empty(n, d),
                 dx=_empty(n, d), dg1=_f32(d), dwo=_WeightGrad(n, d, nq), dwqkv=_WeightGrad(n, N, d),
                 ws=torch.empty(mt.lib().mt_k_rmsnorm_bwd_ws_bytes(d), device="cuda", dtype=torch.uint8))
        if c["bias"]:
            s.update(db=_f32(N), bws=torch.empty(mt.lib().mt_k_bias_grad_ws_bytes(N), device="cuda", dtype=torch.uint8))
    s["p"] = {k: v.data_ptr() for k, v in s.items() if isinstance(v, torch.Tensor)}
    return s


def _run_proj(s):
    L, p, n, d, N, nq = mt.lib(), s["p"], s["n"], s["d"], s["N"], s["nq"]
    b = p.get("b")
    _check(L.mt_k_rmsnorm_fwd(p["xn"], p["x"], p["g1"], n, d, 1e-5, None))
    st = UNSUPPORTED
    if s["hd"] == 128:
        st = L.mt_k_gemm_nt_rope(p["xn"], d, p["wqkv"], d, p["qkv"], N, b, p["cos"], p["sin"], s["T"], s["rot"], n, N, d, None)
    if st == UNSUPPORTED:
        if b:
            _check(L.mt_k_gemm_nt_bias(p["xn"], d, p["wqkv"], d, p["qkv"], N, b, n, N, d, None))
        else:
            _check(L.mt_k_gemm_nt(p["xn"], d, p["wqkv"], d, p["qkv"], N, None, 0, n, N, d, 0, 0, None))
        st = L.mt_k_rope(p["qkv"], N, n, s["T"], s["rot"] // s["hd"], s["hd"], p["cos"], p["sin"], 1, None)
    _check(st)
    _check(L.mt_k_gemm_nt(p["att"], nq, p["wo"], nq, p["h1"], d, p["x"], d, n, d, nq, 0, 0, None))
    if not s["train"]:
        return [s["qkv"], s["h1"]]
    dwo = s["dwo"](p["dh1"], d, p["att"], nq)
    _check(L.mt_k_transpose(p["wo"], p["woT"], d, nq, nq, d, 1, 1, 0, 0, 0, 0, None))
    _check(L.mt_k_gemm_nt(p["dh1"], d, p["woT"], d, p["datt"], nq, None, 0, n, nq, d, 0, 0, None))
    out = [s["qkv"], s["h1"], dwo, s["datt"], s["dx"], s["dg1"]]
    if b:
        _check(L.mt_k_bias_grad(p["db"], p["dqkv"], N, n, N, p["bws"], None))
        out.append(s["db"])
    out.append(s["dwqkv"](p["dqkv"], N, p["xn"], d))
    _check(L.mt_k_transpose(p["wqkv"], p["wqkvT"], N, d, d, N, 1, 1, 0, 0, 0, 0, None))
    _check(L.mt_k_gemm_nt(p["dqkv"], N, p["wqkvT"], N, p["dxn"], d, None, 0, n, d, N, 0, 0, None))
    _check(L.mt_k_rmsnorm_bwd(p["dx"], p["dg1"], p["dxn"], p["x"], p["g1"], p["dh1"], p["ws"], n, d, 1e-5, None))
    return out


# ------------------------------------------------------------------ attention
def _prepare_attn(c, g):
    B, T, hd = c["batch"], c["seq"], c["hd"]
    nq, nkv = c["hq"] * hd, c["hkv"] * hd
    n, ld = B * T, nq + 2 * nkv
    s = {"B": B, "T": T, "hq": c["hq"], "hkv": c["hkv"], "hd": hd, "nq": nq, "nkv": nkv, "ld": ld, "train": c["train"], "qkv": g.bf16(n, ld),
         "o": _empty(n, nq), "lse": _f32(B, c["hq"], T)}
    if c["train"]:
        cs, sn = _rope_tables(T, hd)
        s.update(dout=g.bf16(n, nq, 1e-3), delta=_f32(B, c["hq"], T), dqkv=_empty(n, ld), cos=cs, sin=sn)
    s["p"] = {k: v.data_ptr() for k, v in s.items() if isinstance(v, torch.Tensor)}
    return s


def _run_attn(s):
    L, p, nq, nkv, ld = mt.lib(), s["p"], s["nq"], s["nkv"], s["ld"]
    shape = (s["B"], s["T"], s["hq"], s["hkv"], s["hd"], 1.0 / math.sqrt(s["hd"]), None)
    q, k, v = p["qkv"], p["qkv"] + 2 * nq, p["qkv"] + 2 * (nq + nkv)
    _check(L.mt_k_flash_fwd(p["o"], nq, p["lse"], q, ld, k, ld, v, ld, *shape))
    if not s["train"]:
        return [s["o"], s["lse"]]
    dq, dk, dv = p["dqkv"], p["dqkv"] + 2 * nq, p["dqkv"] + 2 * (nq + nkv)
    _check(L.mt_k_flash_bwd_rope(dq, ld, dk, ld, dv, ld, p["dout"], nq, q, ld, k, ld, v, ld, p["o"], nq, p["lse"], p["delta"],
                                 p["cos"], p["sin"], *shape))
    return [s["o"], s["lse"], s["dqkv"]]


# ------------------------------------------------------------------ the loss
def _prepare_head(c, g):
    n, d, V = c["tokens"], c["d"], c["vocab"]
    s = {"n": n, "d": d, "V": V, "zn": g.bf16(n, d), "w": g.bf16(V, d, 0.02), "labels": g.tokens(n, V), "wT": _empty(d, V),
         "logits": _f32(n, V), "dlogits": _empty(n, V), "rows": _f32(n), "loss": _f32(1), "dzn": _empty(n, d), "dw": _WeightGrad(n, V, d)}
    s["p"] = {k: v.data_ptr() for k, v in s.items() if isinstance(v, torch.Tensor)}
    return s


def _run_head(s):
    L, p, n, d, V = mt.lib(), s["p"], s["n"], s["d"], s["V"]
    _check(L.mt_k_transpose(p["w"], p["wT"], V, d, d, V, 1, 1, 0, 0, 0, 0, None))
    _check(L.mt_k_gemm_nt(p["zn"], d, p["w"], d, p["logits"], V, None, 0, n, V, d, 1, 0, None))
    _check(L.mt_k_cross_entropy(p["rows"], p["dlogits"], p["logits"], p["labels"], n, V, 1.0 / n, None))
    _check(L.mt_k_reduce_sum(p["loss"], p["rows"], n, 1.0 / n, 0, None))
    _check(L.mt_k_gemm_nt(p["dlogits"], V, p["wT"], V, p["dzn"], d, None, 0, n, d, V, 0, 0, None))
    dw = s["dw"](p["dlogits"], V, p["zn"], d)
    return [s["loss"], s["rows"], s["dzn"], dw]


# ------------------------------------------------------------------ norm and embedding
def _prepare_norm(c, g):
    n, d = c["tokens"], c["d"]
    s = {"n": n, "d": d, "x": g.bf16(n, d), "g": g.gain(d), "dy": g.bf16(n, d, 1e-3), "dres": g.bf16(n, d, 1e-3), "y": _empty(n, d),
         "dx": _empty(n, d), "dg": _f32(d), "ws": torch.empty(mt.lib().mt_k_rmsnorm_bwd_ws_bytes(d), device="cuda", dtype=torch.uint8)}
    s["p"] = {k: v.data_ptr() for k, v in s.items() if isinstance(v, torch.Tensor)}
    return s


def _run_norm(s):
    L, p, n, d = mt.lib(), s["p"], s["n"], s["d"]
    _check(L.mt_k_rmsnorm_fwd(p["y"], p["x"], p["g"], n, d, 1e-5, None))
    _check(L.mt_k_rmsnorm_bwd(p["dx"], p["dg"], p["dy"], p["x"], p["g"], p["dres"], p["ws"], n, d, 1e-5, None))
    return [s["y"], s["dx"], s["dg"]]


def _prepare_embed(c, g):
    n, d, V = c["tokens"], c["d"], c["vocab"]
    tok = g.tokens(n, V)
    start = torch.zeros(V + 1, device="cuda", dtype=torch.int32)
    start[1:] = torch.cumsum(torch.bincount(tok.long(), minlength=V), 0).to(torch.int32)
    s = {"n": n, "d": d, "V": V, "tok": tok, "start": start, "order": torch.argsort(tok, stable=True).to(torch.int32), "table": g.bf16(V, d, 0.02),
         "dh": g.bf16(n, d, 1e-3), "h": _empty(n, d), "dtable": _f32(V, d)}
    s["p"] = {k: v.data_ptr() for k, v in s.items() if isinstance(v, torch.Tensor)}
    return s


def _run_embed(s):
    L, p, n, d, V = mt.lib(), s["p"], s["n"], s["d"], s["V"]
    _check(L.mt_k_embed_gather(p["h"], p["table"], p["tok"], n, d, None))
    _check(L.mt_k_embed_scatter(p["dtable"], p["dh"], p["start"], p["order"], V, d, None))
    return [s["h"], s["dtable"]]


# ------------------------------------------------------------------ the interface
_PREPARE = {"step": _prepare_step, "mlp": _prepare_mlp, "proj": _prepare_proj, "attn": _prepare_attn, "head": _prepare_head,
            "norm": _prepare_norm, "embed": _prepare_embed}
_RUN = {"step": _run_step, "mlp": _run_mlp, "proj": _run_proj, "attn": _run_attn, "head": _run_head, "norm": _run_norm,
        "embed": _run_embed}


def prepare(case, seed):
    s = _PREPARE[case["kind"]](case, _Gen(seed))
    s["kind"] = case["kind"]
    return s


def run(state):
    return _RUN[state["kind"]](state)


def work(case):
    """Bytes and floating-point operations one pass cannot do without: every input read once, every result written once."""
    c = case
    if c["kind"] == "step":
        n, P = c["batch"] * c["seq"], _n_params(c)
        mat = P - (0 if c["tied"] else c["vocab"] * c["d"])         # the embedding table is looked up, not multiplied
        attn = 9.0 * c["batch"] * c["hq"] * c["hd"] * float(c["seq"]) * (c["seq"] + 1.0) * c["layers"]
        # bf16 weights in, fp32 gradients out; the optimizer reads p, g, m, v and writes p, m, v and the bf16 copy
        return {"bytes": 6.0 * P + 8.0 * n + (30.0 * P if c["adam"] else 0.0), "flops": 6.0 * mat * n + attn}
    if c["kind"] == "mlp":
        n, d, F, W = c["tokens"], c["d"], c["ffn"], 3.0 * c["ffn"] * c["d"]
        if not c["train"]:
            return {"bytes": 2.0 * (2 * n * d + W), "flops": 2.0 * n * W}
        return {"bytes": 2.0 * (4 * n * d + W) + 4.0 * (W + d), "flops": 6.0 * n * W}
    if c["kind"] == "proj":
        n, d, nq, nkv = c["batch"] * c["seq"], c["d"], c["hq"] * c["hd"], c["hkv"] * c["hd"]
        N, W = nq + 2 * nkv, (2.0 * nq + 2 * nkv) * d
        fwd = 2.0 * (2 * n * d + n * nq + n * N + W)
        if not c["train"]:
            return {"bytes": fwd, "flops": 2.0 * n * W}
        return {"bytes": fwd + 2.0 * (2 * n * d + n * nq + n * N) + 4.0 * W, "flops": 6.0 * n * W}
    if c["kind"] == "attn":
        n, nq, nkv, T = c["batch"] * c["seq"], c["hq"] * c["hd"], c["hkv"] * c["hd"], float(c["seq"])
        pair = c["batch"] * c["hq"] * c["hd"] * T * (T + 1.0)        # one product over the causal half
        fwd = 2.0 * n * (2 * nq + 2 * nkv) + 4.0 * n * c["hq"]
        if not c["train"]:
            return {"bytes": fwd, "flops": 2.0 * pair}
        return {"bytes": fwd + 2.0 * n * (2 * nq + 2 * nkv), "flops": 7.0 * pair}
    if c["kind"] == "head":
        n, d, V = c["tokens"], c["d"], c["vocab"]
        return {"bytes": 2.0 * (2 * n * d + V * d) + 4.0 * V * d + 8.0 * n, "flops": 6.0 * n * d * V}
    if c["kind"] == "norm":
        n, d = c["tokens"], c["d"]
        return {"bytes": 2.0 * 5 * n * d + 6.0 * d, "flops": 12.0 * n * d}
    n, d, V = c["tokens"], c["d"], c["vocab"]
    return {"bytes": 2.0 * (2 * n * d + min(n, V) * d) + 4.0 * V * d + 8.0 * n, "flops": float(n * d)}


# Largest relative error against the same path in 64 bits, measured at sizes like 2 x 520 .. 2 x 1000 tokens and widths of
# 512 .. 5120 (2-norm / largest single difference), and about four times that allowed:
#   mlp    3.9e-3 / 2.3e-2 (weight gradients: four bf16 roundings deep)   proj   2.8e-3 / 1.5e-2 (the projection, rounded, rotated)
#   attn   2.4e-3 / 8.8e-2 (dq, dk, dv: P, dS and O pass through bf16)   head   1.7e-3 / 4.7e-3     norm   1.7e-3 / 3.9e-3
#   embed  7.8e-9 / 7.1e-7 (fp32 sums of bf16 rows; rows that occur thousands of times differ more)
#   step   1.4e-2 / 2.7e-1 (worst of all gradient tensors, weights rounded to bf16 included)
_TOLERANCE = {"mlp": (1.5e-2, 0.1), "proj": (1.1e-2, 0.06), "attn": (1e-2, 0.35), "head": (7e-3, 2e-2), "norm": (7e-3, 1.6e-2),
              "embed": (1e-6, 1e-5), "step": (2.5e-2, 0.8)}


def tolerance(case):
    rel, largest = _TOLERANCE[case["kind"]]
    return {"rel": rel, "max": largest}
