"""GPU parity of la2_fwd_state_norm / la2_bwd_state_norm (the normalised operator on a segment with state
hand-over) against the fp64 oracle: all dtypes and head dimensions, ragged lengths (block kernels + short-run
kernels), sequence chunks, with and without the final state and its gradient, two segments against the whole."""
import numpy as np
import pytest
import torch

import oracle
from paper_2401_04658_amd import binding, workloads
from parity import assert_close, to64

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
EPS = 1e-3


@pytest.fixture(autouse=True)
def _defaults():
    binding.la2_set_chunk_tokens(0)
    binding.la2_set_scan_variant(0)
    yield
    binding.la2_set_chunk_tokens(0)
    binding.la2_set_scan_variant(0)


def inputs(b, H, n, d, dtype, seed, lam=None):
    t = workloads.Workload("norm_state", b, H, n, d, dtype, seed=seed, backward=True).tensors()
    if lam is not None:
        t["lam"] = torch.as_tensor(lam, dtype=torch.float32).reshape(-1).expand(H).contiguous()
    gen = torch.Generator(device="cpu")
    gen.manual_seed(seed + 1)
    t["kv_init"] = torch.randn((b, H, d, d), generator=gen, dtype=torch.float32) * 0.3
    t["d_kv_final"] = torch.randn((b, H, d, d), generator=gen, dtype=torch.float32) * 0.3
    return t, {k: v.to(DEV) for k, v in t.items()}


def check(t, g, dtype, tag, final=True, init=True):
    kv0 = g["kv_init"] if init else None
    o, rstd, kvf = binding.la2_fwd_state_norm(g["q"], g["k"], g["v"], g["lam"], EPS, kv_init=kv0, want_final=final)
    dq, dk, dv, dkv0 = binding.la2_bwd_state_norm(g["q"], g["k"], g["v"], o, rstd, g["d_o"], g["lam"], kv_init=kv0,
                                                  d_kv_final=g["d_kv_final"] if final else None)
    torch.cuda.synchronize()
    q, k, v, do, lam = (to64(t[x]) for x in ("q", "k", "v", "d_o", "lam"))
    init64 = to64(t["kv_init"]) if init else None
    ro, rr, rkvf = oracle.fwd_norm_state(q, k, v, lam, EPS, init64)
    refs = oracle.bwd_norm_state(q, k, v, do, lam, EPS, init64, to64(t["d_kv_final"]) if final else None)
    assert_close(tag + " o", o, ro, dtype)
    assert_close(tag + " rstd", rstd, rr, dtype)
    if final:
        assert_close(tag + " kv_final", kvf, rkvf, dtype)
    if q.shape[2] > 1 or init:   # one position from a zero state leaves dq, dk as pure cancellation
        for name, got, ref in zip(("dq", "dk", "dv", "d_kv_init"), (dq, dk, dv, dkv0), refs):
            assert_close(tag + " " + name, got, ref, dtype)


@pytest.mark.parametrize("final", [True, False])
@pytest.mark.parametrize("n", [1, 31, 32, 45, 64, 100, 300])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("d", [64, 96, 128, 256])
def test_segment(d, dtype, n, final):
    if dtype == torch.float32 and d in (96, 256) and n > 100:
        n = 100    # fp32 at these head dimensions is the token recurrence
    t, g = inputs(2, 2, n, d, dtype, seed=3000 + d + n, lam=[0.7, 0.98])
    check(t, g, dtype, "d%d %s n%d final %s" % (d, dtype, n, final), final)


@pytest.mark.parametrize("chunk", [64, 192])
@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.bfloat16, 64), (torch.float32, 128),
                                     (torch.float16, 128), (torch.bfloat16, 256), (torch.bfloat16, 96)])
def test_segment_chunked(dtype, d, chunk):
    binding.la2_set_chunk_tokens(chunk)
    t, g = inputs(1, 2, 700, d, dtype, seed=3100 + d + chunk, lam=[0.8, 0.99])
    check(t, g, dtype, "d%d %s chunk %d" % (d, dtype, chunk))
    check(t, g, dtype, "d%d %s chunk %d, zero start" % (d, dtype, chunk), init=False)


@pytest.mark.usefixtures("both_paths")
@pytest.mark.parametrize("d", [64, 128, 256])
def test_two_segments_against_the_whole_sequence(d):
    t, g = inputs(1, 2, 150, d, torch.bfloat16, seed=3200 + d, lam=[0.9, 0.97])
    cut = 77
    first = [g[x][:, :, :cut].contiguous() for x in ("q", "k", "v")]
    second = [g[x][:, :, cut:].contiguous() for x in ("q", "k", "v")]
    o1, r1, s1 = binding.la2_fwd_state_norm(*first, g["lam"], EPS)
    o2, r2, s2 = binding.la2_fwd_state_norm(*second, g["lam"], EPS, kv_init=s1)
    ow, rw = binding.la2_fwd_norm(g["q"], g["k"], g["v"], g["lam"], EPS)
    torch.cuda.synchronize()
    q, k, v, lam = (to64(t[x]) for x in ("q", "k", "v", "lam"))
    ro, rr, rs = oracle.fwd_norm_state(q, k, v, lam, EPS)
    assert_close("segments o", torch.cat([o1, o2], dim=2), ro, torch.bfloat16)
    assert_close("segments rstd", torch.cat([r1, r2], dim=2), rr, torch.bfloat16)
    assert_close("segments state", s2, rs, torch.bfloat16)
    assert_close("whole o", ow, ro, torch.bfloat16)


@pytest.mark.usefixtures("both_paths")
def test_strided_layout_and_given_buffers():
    t, g = inputs(2, 3, 90, 128, torch.bfloat16, seed=3300)
    for name in ("q", "k", "v", "d_o"):
        g[name] = t[name].permute(0, 2, 1, 3).contiguous().to(DEV).permute(0, 2, 1, 3)
    check(t, g, torch.bfloat16, "bnhd")


def test_empty_sequence_passes_the_state_through():
    d = 64
    t, g = inputs(2, 2, 0, d, torch.bfloat16, seed=3400)
    o, rstd, kvf = binding.la2_fwd_state_norm(g["q"], g["k"], g["v"], g["lam"], EPS, kv_init=g["kv_init"])
    dq, dk, dv, dkv0 = binding.la2_bwd_state_norm(g["q"], g["k"], g["v"], o, rstd, g["d_o"], g["lam"],
                                                  kv_init=g["kv_init"], d_kv_final=g["d_kv_final"])
    torch.cuda.synchronize()
    assert torch.equal(kvf, g["kv_init"]) and torch.equal(dkv0, g["d_kv_final"])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("d", [64, 96, 128, 256])
def test_normalised_decode_steps_follow_the_segment(d, dtype):
    """Prefill a segment with la2_fwd_state_norm, then decode token by token with la2_decode_step_norm: the
    outputs are those of the normalised operator on the whole sequence."""
    b, H, n, steps = 2, 3, 40, 6
    t, g = inputs(b, H, n + steps, d, dtype, seed=3500 + d, lam=[0.5, 0.9, 1.0])
    pre = [g[x][:, :, :n].contiguous() for x in ("q", "k", "v")]
    o_pre, _, state = binding.la2_fwd_state_norm(*pre, g["lam"], EPS, kv_init=g["kv_init"])
    outs = [o_pre]
    for i in range(n, n + steps):
        outs.append(binding.la2_decode_step_norm(g["q"][:, :, i].contiguous(), g["k"][:, :, i].contiguous(),
                                                 g["v"][:, :, i].contiguous(), g["lam"], state, EPS)[:, :, None])
    torch.cuda.synchronize()
    q, k, v, lam = (to64(t[x]) for x in ("q", "k", "v", "lam"))
    ro, _, rs = oracle.fwd_norm_state(q, k, v, lam, EPS, to64(t["kv_init"]))
    assert_close("d%d %s prefill + decode o" % (d, dtype), torch.cat(outs, dim=2), ro, dtype)
    assert_close("d%d %s prefill + decode state" % (d, dtype), state, rs, dtype)


# ---- the normalised operator over packed sequences and in multi-token decode ---------------------------------------
def _packed(lengths, H, d, dtype, seed, lead=0, trail=0):
    import numpy as np
    total = lead + int(sum(lengths)) + trail
    t = workloads.Workload("packed", 1, H, total, d, dtype, seed=seed, backward=True).tensors()
    out = {name: t[name][0].permute(1, 0, 2).contiguous() for name in ("q", "k", "v", "d_o")}
    out["lam"] = t["lam"]
    cu = np.concatenate([[lead], lead + np.cumsum(lengths)]).astype(np.int32)
    return out, cu


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.bfloat16, 64), (torch.float16, 128), (torch.float32, 64),
                                     (torch.bfloat16, 96)])
@pytest.mark.parametrize("chunk", [0, 128])
def test_norm_over_packed_sequences(dtype, d, chunk):
    check_norm_packed([70, 0, 1, 31, 300, 517, 64], 2, d, dtype, chunk, seed=900 + d)


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.bfloat16, 64)])
@pytest.mark.parametrize("kind", ["sorted", "even", "quarters", "few", "four"])
def test_norm_over_packed_sequences_by_every_plan(kind, dtype, d):
    """The automatic plans of a packed batch (workloads.packed_plan_lengths), normalised.  (bf16: fp16's tolerance of
    2.5e-3, five roundings of 2^-11, is for tensors of up to a million elements; the largest of ten million here is six
    standard deviations of about 5e-4 out, 3.0e-3.)"""
    lengths, H = workloads.packed_plan_lengths(kind)
    check_norm_packed(lengths, H, d, dtype, 0, seed=940 + d, lam=[0.7, 0.97, 0.995, 1.0][:H] * max(1, H // 4))


def check_norm_packed(lengths, H, d, dtype, chunk, seed, lam=None):
    import numpy as np
    t, cu = _packed(lengths, H, d, dtype, seed=seed, lead=3, trail=5)
    if lam is not None:
        t["lam"] = torch.as_tensor(lam, dtype=torch.float32)
    g = {k_: v_.to(DEV) for k_, v_ in t.items()}
    cu_g = torch.from_numpy(cu).to(DEV)
    eps = 1e-5
    binding.la2_set_chunk_tokens(chunk)
    try:
        o = torch.full_like(g["q"], float("nan"))
        rstd = torch.full((H, g["q"].shape[0]), float("nan"), dtype=torch.float32, device=DEV)
        binding.la2_fwd_varlen_norm(g["q"], g["k"], g["v"], g["lam"], cu_g, max(lengths), eps, out=o, rstd=rstd)
        grads = tuple(torch.full_like(g["q"], float("nan")) for _ in range(3))
        d_u = torch.full_like(g["q"], float("nan"))
        binding.la2_bwd_varlen_norm(g["q"], g["k"], g["v"], o, rstd, g["d_o"], g["lam"], cu_g, max(lengths), out=grads, d_u=d_u)
        torch.cuda.synchronize()
    finally:
        binding.la2_set_chunk_tokens(0)
    q, k, v, do, lam = (to64(t[x]) for x in ("q", "k", "v", "d_o", "lam"))
    ro, rr = oracle.fwd_norm_packed(q, k, v, lam, cu, eps)
    lo, hi = int(cu[0]), int(cu[-1])
    tag = "packed norm %s d%d chunk%d" % (dtype, d, chunk)
    assert_close(tag + " o", o[lo:hi], ro[lo:hi], dtype)
    assert_close(tag + " rstd", rstd[:, lo:hi], rr[:, lo:hi], dtype)
    # the backward pass from the GPU's own (rounded) o and rstd, as a training step has them
    du_ref = oracle.norm_backward_rows(to64(o)[lo:hi], to64(rstd)[:, lo:hi].T, do[lo:hi])
    assert_close(tag + " d_u", d_u[lo:hi], du_ref, dtype)
    for b in range(len(lengths)):
        s0, s1 = int(cu[b]), int(cu[b + 1])
        if s1 == s0:
            continue
        seq = [np.ascontiguousarray(x[s0:s1].transpose(1, 0, 2))[None] for x in (q, k, v)]
        du_seq = np.ascontiguousarray(to64(d_u)[s0:s1].transpose(1, 0, 2))[None]
        for name, got, ref in zip(("dq", "dk", "dv"), grads, oracle.bwd_direct(seq[0], seq[1], seq[2], du_seq, lam)):
            assert_close("%s seq %d %s" % (tag, b, name), got[s0:s1].permute(1, 0, 2)[None], ref, dtype)
    # nothing outside the sequences is written
    for x in (o, d_u) + grads:
        assert torch.isnan(x[:lo].float()).all() and torch.isnan(x[hi:].float()).all()
    assert torch.isnan(rstd[:, :lo]).all() and torch.isnan(rstd[:, hi:]).all()


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.bfloat16, 64), (torch.float32, 128), (torch.float16, 256),
                                     (torch.float32, 96)])
@pytest.mark.parametrize("T", [1, 8, 33, 70])
def test_multi_token_decode_with_norm(dtype, d, T):
    b, H = 3, 2
    t = workloads.Workload("dm", b, H, T, d, dtype, seed=950 + d + T, backward=False).tensors()
    gen = torch.Generator(device="cpu")
    gen.manual_seed(7)
    kv0 = torch.randn((b, H, d, d), generator=gen, dtype=torch.float32) * 0.2
    g = {k_: v_.to(DEV) for k_, v_ in t.items()}
    state = kv0.to(DEV)
    eps = 1e-5
    o, rstd = binding.la2_decode_multi_norm(g["q"], g["k"], g["v"], g["lam"], state, eps)
    torch.cuda.synchronize()
    ro, rr, rs = oracle.fwd_norm_state(to64(t["q"]), to64(t["k"]), to64(t["v"]), to64(t["lam"]), eps, kv_init=to64(kv0))
    tag = "decode multi norm %s d%d T%d" % (dtype, d, T)
    assert_close(tag + " o", o, ro, dtype)
    assert_close(tag + " rstd", rstd, rr, dtype)
    assert_close(tag + " state", state, rs, dtype)


@pytest.mark.parametrize("d,H,lengths", [(96, 3, [300, 20, 1, 40, 64, 0, 33]), (256, 2, [257, 20, 1, 40, 64, 0, 33]),
                                         (96, 16, [3000] + [130] * 430), (256, 8, [1500] + [130] * 320)])
def test_norm_over_packed_sequences_of_unequal_lengths_at_96_and_256(d, H, lengths):
    """Such batches store through the caches, with their tiles kept (small) or not (above 160 MiB): rows of the longest, of a
    middle and of the last sequence against the oracle, and the middle one bit for bit against a dense call on it."""
    dtype = torch.bfloat16
    total = sum(lengths)
    assert len(lengths) * max(lengths) > 2 * total and (total * H * d * 2 > 160 << 20) == (len(lengths) > 100)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d + total)
    q, k, v = ((torch.randn((total, H, d), generator=gen, device=DEV) * d ** -0.5).to(dtype) for _ in range(3))
    lam = torch.exp(-torch.pow(2.0, -8.0 * torch.arange(1, H + 1) / H)).to(DEV)
    ends = np.concatenate([[0], np.cumsum(lengths)])
    cu = torch.tensor(ends, dtype=torch.int32, device=DEV)
    o, rstd = binding.la2_fwd_varlen_norm(q, k, v, lam, cu, max(lengths), EPS)
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all() and torch.isfinite(rstd).all()
    for s in (0, len(lengths) // 2, len(lengths) - 1):
        lo, hi = int(ends[s]), int(ends[s + 1])
        if s:
            part = [x[lo:hi].permute(1, 0, 2)[None].contiguous() for x in (q, k, v)]
            on, rn = binding.la2_fwd_norm(*part, lam, EPS)
            torch.cuda.synchronize()
            assert torch.equal(on[0].permute(1, 0, 2), o[lo:hi]) and torch.equal(rn[0], rstd[:, lo:hi])
        for h in (0, H - 1):
            x = [to64(t[lo:hi, h])[None, None] for t in (q, k, v)]
            ro, rr = oracle.fwd_norm(*x, to64(lam[h:h + 1]), EPS)
            assert_close("seq %d o" % s, o[lo:hi, h][None, None], ro, dtype)
            assert_close("seq %d rstd" % s, rstd[h, lo:hi][None, None], rr, dtype)
