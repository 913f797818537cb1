"""The work that users of this library have it do, as cases that can be timed and compared.

Every case goes through the public Python entry points with tensors that are already on the GPU.  A case is a dict of
plain values:

  kind     "train"    la2_fwd, then la2_bwd (or, "saved", the backward that takes over the forward call's workspace);
                      with "norm" the normalised operator (la2_fwd_norm, la2_bwd_norm)
           "packed"   the same over packed sequences of different lengths (la2_fwd_varlen, la2_bwd_varlen, with "norm"
                      their normalised forms)
           "prefill"  la2_fwd_state: one segment of a prompt with its final state, "init": continued from a state
           "decode"   "tokens" positions on a kept state: la2_decode_step for one, la2_decode_multi for several, with
                      "norm" their normalised forms
  dtype    "bf16", "f16" or "f32";  b, h, n, d: batch, heads, sequence length, head_dim
  packed:  "total" positions, the "longest" sequence and "mix", the number that the lengths are drawn from

Decays follow the per-head schedule exp(-2^(-8 (h + 1) / H)); q, k, v and the output gradient are N(0, 1) / sqrt(d),
states N(0, 0.1^2).
"""
import math
import random

import torch

import paper_2401_04658_amd as la2
from paper_2401_04658_amd import binding

_DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
_EPS = 1e-6


def _train(name, b, h, n, d, dtype="bf16", norm=False, saved=False):
    return {"name": name, "kind": "train", "dtype": dtype, "b": b, "h": h, "n": n, "d": d, "norm": norm, "saved": saved}


def _decode(name, b, h, d, tokens, dtype="bf16", norm=False):
    return {"name": name, "kind": "decode", "dtype": dtype, "b": b, "h": h, "d": d, "tokens": tokens, "norm": norm}


def listed():
    return [
        # one user's next token: latency and launch cost only
        _decode("decode_b1_h16_d128", 1, 16, 128, 1),
        # a serving batch of a 3B-like model, one token each: the state's bytes
        _decode("decode_b128_h32_d128", 128, 32, 128, 1),
        # a few proposed tokens at once on a middle batch
        _decode("decode_5_tokens_b32_h32_d128", 32, 32, 128, 5),
        # a short prompt of odd length, state handed to decoding
        {"name": "prefill_b1_h16_n777_d128", "kind": "prefill", "dtype": "bf16", "b": 1, "h": 16, "n": 777, "d": 128,
         "init": False},
        # training step of one layer of a 400M-like model: few chains, several dependent launches
        _train("train_b4_h16_n2048_d64", 4, 16, 2048, 64),
        # the ordinary training step: one chain for every compute unit (second point of the benchmark's sweep)
        _train("train_b16_h16_n4096_d128", 16, 16, 4096, 128),
        # one very long sequence, backward from the forward call's states (last point of the sweep)
        _train("train_saved_b1_h16_n65536_d128", 1, 16, 65536, 128, saved=True),
        # normalised operator, half precision, a length that is no multiple of any tile
        _train("train_norm_b8_h16_n3001_d64_f16", 8, 16, 3001, 64, dtype="f16", norm=True),
        # a packed batch of documents from 64 to 8192 positions
        {"name": "packed_65536_longest_8192_h16_d128", "kind": "packed", "dtype": "bf16", "h": 16, "d": 128, "total": 65536,
         "longest": 8192, "mix": 1, "norm": False},
        # single precision: reference runs and small models
        _train("train_b4_h16_n2048_d128_f32", 4, 16, 2048, 128, dtype="f32"),
        # the other two head dimensions
        _train("train_b16_h8_n2048_d256", 16, 8, 2048, 256),
        _train("train_b8_h12_n4099_d96", 8, 12, 4099, 96),
    ]


# No drawn case has more elements per tensor than the largest listed case of its kind of arithmetic.
_MOST_16BIT = 16 * 16 * 4096 * 128
_MOST_F32 = 4 * 16 * 2048 * 128


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.99)))))))


def draw(rng):
    kind = rng.choice(("train", "train", "train", "train", "packed", "prefill", "decode", "decode"))
    dtype = rng.choice(("bf16", "bf16", "bf16", "f16", "f32"))
    if kind == "packed" and dtype == "f32":
        dtype = "bf16"
    most = _MOST_F32 if dtype == "f32" else _MOST_16BIT
    d = rng.choice((64, 128)) if dtype == "f32" else rng.choice((64, 64, 96, 128, 128, 128, 256))
    h = rng.choice((1, 2, 4, 6, 8, 12, 16, 20, 32))
    if kind == "decode":
        tokens = rng.choice((1, 1, 1, 2, 3, 5, 8, 16))
        states = 128 * 32 * 128 * 128 // (8 if dtype == "f32" and tokens > 1 else 1)
        b = _log_int(rng, 1, max(1, min(512, states // (h * d * d))))
        return {"kind": "decode", "dtype": dtype, "b": b, "h": h, "d": d, "tokens": tokens, "norm": rng.random() < 0.25}
    norm = rng.random() < 0.25
    if kind == "packed":
        longest = _log_int(rng, 128, 16384)
        total = longest + _log_int(rng, longest, max(longest + 1, min(131072, most // (h * d) - longest)))
        return {"kind": "packed", "dtype": dtype, "h": h, "d": d, "total": min(total, most // (h * d)), "longest": longest,
                "mix": rng.randrange(1 << 30), "norm": norm}
    n = _log_int(rng, 32, min(65536, most // (h * d)))
    b = _log_int(rng, 1, max(1, min(512, most // (h * d * n))))
    if kind == "prefill":
        return {"kind": "prefill", "dtype": dtype, "b": b, "h": h, "n": n, "d": d, "init": rng.random() < 0.5}
    return {"kind": "train", "dtype": dtype, "b": b, "h": h, "n": n, "d": d, "norm": norm,
            "saved": not norm and rng.random() < 0.5}


def _lengths(case):
    """The packed batch's sequence lengths: the longest first, the others spread over the logarithm."""
    rng = random.Random(case["mix"])
    out, left = [min(case["longest"], case["total"])], case["total"] - min(case["longest"], case["total"])
    lo = min(64, case["longest"])
    while left > 0:
        out.append(min(left, _log_int(rng, lo, case["longest"])))
        left -= out[-1]
    return out


def _decay(heads, device):
    i = torch.arange(1, heads + 1, dtype=torch.float64, device=device)
    return torch.exp(-torch.pow(torch.tensor(2.0, dtype=torch.float64, device=device), -8.0 * i / heads)).float()


def _inputs(case, seed):
    """Everything that is drawn from the seed: the tensors of a case by name."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    dt, h, d = _DTYPES[case["dtype"]], case["h"], case["d"]

    def normal(shape, scale, dtype):
        return (torch.randn(shape, generator=gen, device=dev, dtype=torch.float32) * scale).to(dtype)

    if case["kind"] == "packed":
        shape = (case["total"], h, d)
    elif case["kind"] == "decode":
        shape = (case["b"], h, d) if case["tokens"] == 1 else (case["b"], h, case["tokens"], d)
    else:
        shape = (case["b"], h, case["n"], d)
    t = {x: normal(shape, d ** -0.5, dt) for x in ("q", "k", "v")}
    if case["kind"] in ("train", "packed"):
        t["d_o"] = normal(shape, d ** -0.5, dt)
    if case["kind"] == "decode" or case.get("init"):
        t["kv"] = normal((case["b"], h, d, d), 0.1, torch.float32)
    t["lam"] = _decay(h, dev)
    return t


def prepare(case, seed):
    """Inputs and what a program keeps across calls: the workspaces and a packed batch's offsets."""
    st = dict(_inputs(case, seed), case=case)
    q = st["q"]
    if case["kind"] == "packed":
        ends = [0]
        for x in _lengths(case):
            ends.append(ends[-1] + x)
        st["cu"] = torch.tensor(ends, dtype=torch.int32, device=q.device)
        st["longest"] = max(_lengths(case))
    elif case["kind"] == "train":
        for name, op in (("ws_f", binding.LA2_OP_FWD),
                         ("ws_b", binding.LA2_OP_BWD_STATE if case["saved"] else binding.LA2_OP_BWD)):
            st[name] = torch.empty(max(1, la2.la2_workspace_bytes(q, op)), dtype=torch.uint8, device=q.device)
    elif case["kind"] == "prefill":
        need = la2.la2_workspace_bytes(q, binding.LA2_OP_FWD_STATE)
        st["ws_f"] = torch.empty(max(1, need), dtype=torch.uint8, device=q.device)
    return st


def run(state):
    s, case = state, state["case"]
    q, k, v, lam = s["q"], s["k"], s["v"], s["lam"]
    if case["kind"] == "decode":
        if case["tokens"] == 1:
            if case["norm"]:
                return la2.la2_decode_step_norm(q, k, v, lam, s["kv"], _EPS), s["kv"]
            return la2.la2_decode_step(q, k, v, lam, s["kv"]), s["kv"]
        if case["norm"]:
            return la2.la2_decode_multi_norm(q, k, v, lam, s["kv"], _EPS) + (s["kv"],)
        return la2.la2_decode_multi(q, k, v, lam, s["kv"]), s["kv"]
    if case["kind"] == "prefill":
        return la2.la2_fwd_state(q, k, v, lam, kv_init=s.get("kv"), workspace=s["ws_f"])
    if case["kind"] == "packed":
        at = (lam, s["cu"], s["longest"])
        if case["norm"]:
            o, rstd = la2.la2_fwd_varlen_norm(q, k, v, *at, _EPS)
            return (o, rstd) + tuple(la2.la2_bwd_varlen_norm(q, k, v, o, rstd, s["d_o"], *at))
        return (la2.la2_fwd_varlen(q, k, v, *at),) + tuple(la2.la2_bwd_varlen(q, k, v, s["d_o"], *at))
    if case["norm"]:
        o, rstd = la2.la2_fwd_norm(q, k, v, lam, _EPS, workspace=s["ws_f"])
        return (o, rstd) + tuple(la2.la2_bwd_norm(q, k, v, o, rstd, s["d_o"], lam, workspace=s["ws_b"]))
    o = la2.la2_fwd(q, k, v, lam, workspace=s["ws_f"])
    if case["saved"]:
        grads = la2.la2_bwd_state(q, k, v, s["d_o"], lam, want_d_kv_init=False, workspace=s["ws_b"],
                                  fwd_workspace=s["ws_f"])[:3]
    else:
        grads = la2.la2_bwd(q, k, v, s["d_o"], lam, workspace=s["ws_b"])
    return (o,) + tuple(grads)


def work(case):
    """Bytes: inputs once, outputs once, per call.  Operations: the recurrence (2 d^2 multiply-adds per position and
    head for one output, 5 d^2 for the three gradients), which any evaluation needs."""
    size = 4 if case["dtype"] == "f32" else 2
    h, d = case["h"], case["d"]
    if case["kind"] == "decode":
        rows = case["b"] * h * case["tokens"]
        extra = 4 * rows if case["norm"] and case["tokens"] > 1 else 0
        return {"bytes": 2 * 4 * case["b"] * h * d * d + 4 * rows * d * size + extra, "flops": 4 * rows * d * d}
    rows = h * (case["total"] if case["kind"] == "packed" else case["b"] * case["n"])
    unit = rows * d * size
    if case["kind"] == "prefill":
        return {"bytes": 4 * unit + 4 * case["b"] * h * d * d * (2 if case["init"] else 1), "flops": 4 * rows * d * d}
    # forward 3 in, 1 out; backward 4 in, 3 out; the normalised backward also reads the outputs, both sides the row scales
    return {"bytes": (12 * unit + 8 * rows) if case["norm"] else 11 * unit, "flops": 14 * rows * d * d}


def tolerance(case):
    return {"rel": {"bf16": 1.5e-2, "f16": 2e-3, "f32": 3e-6}[case["dtype"]]}


# ---- the same in 64 bits, plain torch -----------------------------------------------------------------------------

_BLOCK = 128


def _scan(x, y, z, lam, state, reverse=False):
    """w_t = sum over s <= t (reverse: s >= t) of lam^|t - s| (x_t . y_s) z_s, plus the state's share; [c, n, d] float64,
    lam [c], state [c, d, d] = sum of lam^(age) y^T z up to the position before the first one (None: zero).  Returns w
    and the state after the last position."""
    c, n, d = x.shape
    if reverse:
        x, y, z = x.flip(1), y.flip(1), z.flip(1)
    w = torch.empty_like(x)
    s = torch.zeros(c, d, d, dtype=x.dtype, device=x.device) if state is None else state.clone()
    at = torch.arange(_BLOCK, device=x.device, dtype=x.dtype)
    gap = at[:, None] - at[None, :]
    mask = torch.where(gap >= 0, lam[:, None, None] ** gap.clamp(min=0), torch.zeros((), dtype=x.dtype, device=x.device))
    for i in range(0, n, _BLOCK):
        xb, yb, zb = (t[:, i:i + _BLOCK].contiguous() for t in (x, y, z))
        m = xb.shape[1]
        p = torch.matmul(xb, yb.transpose(1, 2).contiguous()) * mask[:, :m, :m]
        row = lam[:, None] ** (at[:m] + 1)
        w[:, i:i + m] = torch.matmul(p, zb) + row[:, :, None] * torch.matmul(xb, s)
        left = lam[:, None] ** (m - 1 - at[:m])
        s = (lam ** m)[:, None, None] * s + torch.matmul(yb.transpose(1, 2).contiguous(), left[:, :, None] * zb)
    return (w.flip(1) if reverse else w), s


def _exact_chains(q, k, v, d_o, lam, norm):
    """Forward and backward of chains [c, n, d] in float64."""
    o, _ = _scan(q, k, v, lam, None)
    out = [o]
    if norm:
        r = (o.pow(2).mean(-1) + _EPS).rsqrt()
        o = o * r[..., None]
        d_o = r[..., None] * (d_o - o * (d_o * o).mean(-1, keepdim=True))
        out = [o, r]
    out.append(_scan(d_o, v, k, lam, None)[0])
    out.append(_scan(v, d_o, q, lam, None, reverse=True)[0])
    out.append(_scan(k, q, d_o, lam, None, reverse=True)[0])
    return out


def exact(case, seed):
    t = {x: y.double() for x, y in _inputs(case, seed).items()}
    h, d = case["h"], case["d"]
    if case["kind"] == "packed":
        outs, at = None, 0
        for n in _lengths(case):
            part = [t[x][at:at + n].permute(1, 0, 2).contiguous() for x in ("q", "k", "v", "d_o")]
            got = _exact_chains(*part, t["lam"], case["norm"])
            got = [g if g.dim() == 2 else g.permute(1, 0, 2) for g in got]
            if outs is None:
                outs = [torch.empty((h, case["total"]) if g.dim() == 2 else (case["total"], h, d), dtype=g.dtype,
                                    device=g.device) for g in got]
            for o, g in zip(outs, got):
                if g.dim() == 2:
                    o[:, at:at + n] = g
                else:
                    o[at:at + n] = g
            at += n
        return tuple(outs)
    b = case["b"]
    lam = t["lam"].repeat(b)
    chains = {x: t[x].reshape(b * h, -1, d) for x in ("q", "k", "v", "d_o") if x in t}
    shape = t["q"].shape
    if case["kind"] == "train":
        got = _exact_chains(chains["q"], chains["k"], chains["v"], chains["d_o"], lam, case["norm"])
        return tuple(g.reshape(b, h, -1) if g.dim() == 2 else g.reshape(shape) for g in got)
    o, s = _scan(chains["q"], chains["k"], chains["v"], lam, t["kv"].reshape(b * h, d, d) if "kv" in t else None)
    s = s.reshape(b, h, d, d)
    if case["kind"] == "decode" and case["norm"]:
        r = (o.pow(2).mean(-1) + _EPS).rsqrt()
        o = o * r[..., None]
        if case["tokens"] > 1:
            return o.reshape(shape), r.reshape(b, h, -1), s
    return o.reshape(shape), s
