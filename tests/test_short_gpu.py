"""Short sequences on few chains (16-bit data, head_dim 64 / 128): the launch that looks back over all positions, against the
fp64 oracle and against the block recurrence (scan variant 2 asks for the latter's kernels)."""
import numpy as np
import pytest
import torch

import oracle
from oracle import norm as oracle_norm
from paper_2401_04658_amd import binding, workloads
from parity import RMS_TOL, TOL, assert_close, rms_rel, to64

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
EPS = 1e-6


@pytest.fixture(autouse=True)
def _defaults():
    binding.la2_set_chunk_tokens(0)
    binding.la2_set_scan_variant(0)
    yield
    binding.la2_set_chunk_tokens(0)
    binding.la2_set_scan_variant(0)


def inputs(b, H, n, d, dtype, seed):
    t = workloads.Workload("short", b, H, n, d, dtype, seed=seed, backward=True).tensors()
    t["lam"] = torch.tensor([0.43, 0.9, 0.99, 1.0], dtype=torch.float32)[torch.arange(H) % 4].contiguous()
    g = torch.Generator(device="cpu")
    g.manual_seed(seed + 1000)
    t["kv_init"] = torch.randn((b, H, d, d), generator=g, dtype=torch.float32) * 0.3
    t["d_kv_final"] = torch.randn((b, H, d, d), generator=g, dtype=torch.float32) * 0.3
    return t


def padded(x):
    """The same values with rows 16 elements further apart and positions outside heads: [b, n, H, d + 16] viewed back."""
    store = torch.zeros((x.shape[0], x.shape[2], x.shape[1], x.shape[3] + 16), dtype=x.dtype, device=DEV)
    view = store[..., : x.shape[3]].permute(0, 2, 1, 3)
    view.copy_(x)
    return view


# a lone row; one block of 32 and of 64, one position less and more; one step of the loop and a remainder; several steps
@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 200, 449])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_short_passes_with_and_without_states(dtype, d, n):
    for strided in (False, True):
        t = inputs(1, 4, n, d, dtype, seed=7000 + n + d)
        g = {k: padded(v) if strided and v.dtype == dtype else v.to(DEV) for k, v in t.items()}
        q, k, v, do, lam = (to64(t[x]) for x in ("q", "k", "v", "d_o", "lam"))
        for states in (False, True):
            i64, f64 = (to64(t["kv_init"]), to64(t["d_kv_final"])) if states else (None, None)
            init, fin = (g["kv_init"], g["d_kv_final"]) if states else (None, None)
            o, kvf = binding.la2_fwd_state(g["q"], g["k"], g["v"], g["lam"], kv_init=init)
            grads = binding.la2_bwd_state(g["q"], g["k"], g["v"], g["d_o"], g["lam"], kv_init=init, d_kv_final=fin)
            torch.cuda.synchronize()
            ro, rkvf = oracle.fwd_recurrent(q, k, v, lam, kv_init=i64, return_state=True)
            refs = oracle.bwd_recurrent_state(q, k, v, do, lam, kv_init=i64, d_kv_final=f64)
            tag = "n%d d%d %s strided %s states %s " % (n, d, dtype, strided, states)
            for name, got, ref in zip(("o", "kv_final", "dq", "dk", "dv", "d_kv_init"), (o, kvf) + tuple(grads), (ro, rkvf) + tuple(refs)):
                assert_close(tag + name, got, ref, dtype)
        o, rstd = binding.la2_fwd_norm(g["q"], g["k"], g["v"], g["lam"], EPS)
        ro, rr = oracle_norm.fwd_norm(q, k, v, lam, EPS)
        assert_close(tag + "norm o", o, ro, dtype)
        assert_close(tag + "rstd", rstd, rr, dtype)


# (chains, n) on both sides of every border of the rule: blocks of work, lengths, chains
BORDERS = [(4, 1536), (4, 1537), (4, 3072), (4, 3073), (64, 768), (64, 769), (65, 200), (96, 256), (128, 256), (128, 257),
           (128, 512), (129, 64), (129, 65), (256, 128), (256, 129), (512, 64), (513, 64), (16, 32), (16, 33),
           # ... and of what states change: lengths, blocks of work with the states' share
           (4, 640), (4, 641), (4, 1024), (4, 1025), (4, 1280), (4, 1281), (4, 2048), (4, 2049), (4, 2560), (4, 2561),
           (4, 96), (4, 97), (4, 160), (4, 161), (4, 700), (16, 1100), (16, 1152), (16, 1153),
           (32, 1024), (33, 640), (48, 512), (64, 384), (64, 640), (96, 128), (128, 128), (128, 200), (129, 33), (192, 128)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("chains,n", BORDERS)
def test_short_against_the_block_recurrence(chains, n, d):
    """Both paths round the same operands to 16 bits in different places: their errors against fp64 are of one size (bound on
    the rms difference: both paths' rms bounds together).  The backward that is handed the forward call's workspace gives the
    same bits as the one that is not, whatever was in that workspace, unless it read chunk states there: on a cut sequence,
    where the forward call has written its workspace and the backward call uses its own."""
    H = next(h for h in (16, 8, 4, 3, 1) if chains % h == 0)
    dtype = torch.bfloat16
    gen = torch.Generator(device=DEV)
    gen.manual_seed(chains + n + d)
    q, k, v, do = ((torch.randn((chains // H, H, n, d), generator=gen, device=DEV) * d ** -0.5).to(dtype) for _ in range(4))
    kv0, dkvf = (torch.randn((chains // H, H, d, d), generator=gen, device=DEV) * 0.1 for _ in range(2))
    lam = torch.exp(-torch.pow(2.0, -8.0 * torch.arange(1, H + 1) / H)).to(DEV)
    runs = []
    for variant in (0, 2):
        binding.la2_set_scan_variant(variant)
        ws, ws_b = (torch.full((max(1, binding.la2_workspace_bytes(q, op)),), 0xFF, dtype=torch.uint8, device=DEV)
                    for op in (binding.LA2_OP_FWD_STATE, binding.LA2_OP_BWD_STATE))
        o, kvf = binding.la2_fwd_state(q, k, v, lam, kv_init=kv0, workspace=ws)
        grads = binding.la2_bwd_state(q, k, v, do, lam, kv_init=kv0, d_kv_final=dkvf)
        saved = binding.la2_bwd_state(q, k, v, do, lam, kv_init=kv0, d_kv_final=dkvf, workspace=ws_b, fwd_workspace=ws,
                                      fwd_wrote_kv_final=True)
        torch.cuda.synchronize()
        read_states = not (ws == 0xFF).all() and not (ws_b == 0xFF).all()
        if variant == 2:
            assert read_states == (binding.la2_chunk_plan(q)[0] > 1)
        for x, y in zip(grads, saved):
            # (the saved states are the forward's, the recomputed ones the dQ scan's own transposes)
            assert torch.equal(x, y) or (read_states and rms_rel(to64(x), to64(y)) <= RMS_TOL[dtype])
        runs.append((o, kvf) + tuple(grads))
    for name, a, b in zip(("o", "kv_final", "dq", "dk", "dv", "d_kv_init"), *runs):
        assert torch.isfinite(a).all(), name
        assert rms_rel(to64(a), to64(b)) <= 2 * RMS_TOL[dtype], name


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.float16, 64)])
def test_short_packed_batch_with_empty_sequences(dtype, d):
    lengths, H = [70, 0, 1, 200, 64, 33], 2
    total = sum(lengths)
    t = workloads.Workload("packed", 1, H, total, d, dtype, seed=7400, backward=True).tensors()
    g = {x: t[x][0].permute(1, 0, 2).contiguous().to(DEV) for x in ("q", "k", "v", "d_o")}
    lam = torch.tensor([0.6, 0.98])
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32, device=DEV)
    gen = torch.Generator(device="cpu")
    gen.manual_seed(7401)
    init, dfin = (torch.randn((len(lengths), H, d, d), generator=gen) * 0.3 for _ in range(2))
    o, kvf = binding.la2_fwd_varlen_state(g["q"], g["k"], g["v"], lam.to(DEV), cu, 200, kv_init=init.to(DEV))
    grads = binding.la2_bwd_varlen_state(g["q"], g["k"], g["v"], g["d_o"], lam.to(DEV), cu, 200, kv_init=init.to(DEV),
                                         d_kv_final=dfin.to(DEV))
    on, rstd = binding.la2_fwd_varlen_norm(g["q"], g["k"], g["v"], lam.to(DEV), cu, 200, EPS)
    torch.cuda.synchronize()
    at = 0
    for s, n in enumerate(lengths):
        if n == 0:
            assert torch.equal(kvf[s].cpu(), init[s]) and torch.equal(grads[3][s].cpu(), dfin[s])
            continue
        x = [to64(t[name][:, :, at:at + n]) for name in ("q", "k", "v", "d_o")]
        ro, rkvf = oracle.fwd_recurrent(*x[:3], to64(lam), kv_init=to64(init[s:s + 1]), return_state=True)
        refs = oracle.bwd_recurrent_state(*x, to64(lam), kv_init=to64(init[s:s + 1]), d_kv_final=to64(dfin[s:s + 1]))
        tag = "seq %d n %d " % (s, n)
        assert_close(tag + "o", o[at:at + n].permute(1, 0, 2)[None], ro, dtype)
        assert_close(tag + "kv_final", kvf[s:s + 1], rkvf, dtype)
        for name, got, ref in zip(("dq", "dk", "dv"), grads[:3], refs[:3]):
            assert_close(tag + name, got[at:at + n].permute(1, 0, 2)[None], ref, dtype)
        assert_close(tag + "d_kv_init", grads[3][s:s + 1], refs[3], dtype)
        rn, rr = oracle_norm.fwd_norm(*x[:3], to64(lam), EPS)
        assert_close(tag + "norm o", on[at:at + n].permute(1, 0, 2)[None], rn, dtype)
        assert_close(tag + "rstd", rstd[:, at:at + n][None], rr, dtype)
        at += n


def test_short_pass_hands_its_state_out_in_the_place_of_the_one_it_starts_from():
    """kv_final in kv_init's place (what multi-token decoding does inside the library) and d_kv_init in d_kv_final's."""
    t = inputs(1, 4, 100, 128, torch.bfloat16, seed=7500)
    g = {k: v.to(DEV) for k, v in t.items()}
    o, kvf = binding.la2_fwd_state(g["q"], g["k"], g["v"], g["lam"], kv_init=g["kv_init"])
    grads = binding.la2_bwd_state(g["q"], g["k"], g["v"], g["d_o"], g["lam"], kv_init=g["kv_init"], d_kv_final=g["d_kv_final"])
    kv, dkv = g["kv_init"].clone(), g["d_kv_final"].clone()
    o2, _ = binding.la2_fwd_state(g["q"], g["k"], g["v"], g["lam"], kv_init=kv, kv_final=kv)
    grads2 = binding.la2_bwd_state(g["q"], g["k"], g["v"], g["d_o"], g["lam"], kv_init=g["kv_init"], d_kv_final=dkv, d_kv_init=dkv)
    torch.cuda.synchronize()
    for a, b in zip((o, kvf) + tuple(grads), (o2, kv) + tuple(grads2[:3]) + (dkv,)):
        assert rms_rel(to64(b), to64(a)) <= 2 * RMS_TOL[torch.bfloat16]


@pytest.mark.parametrize("d", [64, 128])
def test_short_backward_of_the_norm_and_graph_replay(d):
    """The normalised backward on the short path against fp64, and a captured pass replayed after the inputs changed."""
    t = inputs(1, 4, 150, d, torch.bfloat16, seed=7600 + d)
    g = {k: v.to(DEV) for k, v in t.items()}
    x = [to64(t[name]) for name in ("q", "k", "v", "d_o", "lam")]
    o, rstd = binding.la2_fwd_norm(g["q"], g["k"], g["v"], g["lam"], EPS)
    grads = binding.la2_bwd_norm(g["q"], g["k"], g["v"], o, rstd, g["d_o"], g["lam"])
    for name, got, ref in zip(("dq", "dk", "dv"), grads, oracle_norm.bwd_norm(*x, EPS)):
        assert rms_rel(to64(got), ref) <= 2 * RMS_TOL[torch.bfloat16], name
    outs = [torch.empty_like(g["q"]) for _ in range(4)]

    def both():
        binding.la2_fwd(g["q"], g["k"], g["v"], g["lam"], out=outs[0])
        binding.la2_bwd(g["q"], g["k"], g["v"], g["d_o"], g["lam"], out=tuple(outs[1:]))

    both()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        both()
    for replay in range(3):
        g["q"].mul_(-1.5)
        both()
        torch.cuda.synchronize()
        ref = [y.clone() for y in outs]
        for y in outs:
            y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, ref)), replay


@pytest.mark.parametrize("padding", ["none", "last", "first"])
@pytest.mark.parametrize("grad", [1.0, 1e-3, 1e-4])
@pytest.mark.parametrize("d,n", [(64, 777), (128, 1500)])
def test_fp16_short_passes_lose_no_range(d, n, grad, padding):
    """fp16 starts at 2^-14 and ends, subnormal, at 2^-24.  The recurrence rounds operands that carry the decay of one block at most
    and sums the rest in fp32; the short path may not round anything smaller: not a state's operands by the decay of the whole
    sequence (padding: a third of the positions is zero, what is left has decayed when the state is handed out), not the scores
    of small gradients (gradients without loss scaling) one by one.  Every head's error against 64 bits, on the short path and
    on the recurrence's kernels; they round different operands, so the bound has a quarter of slack (the fp16 arithmetic of both,
    followed on the CPU over 60 shapes, decays and scales: at most 1.02 times)."""
    lams = [0.9, 0.98, 0.99, 0.9999]
    gen = torch.Generator(device="cpu")
    gen.manual_seed(n + d)
    q, k, v, do = (torch.randn((1, 4, n, d), generator=gen) * d ** -0.5 for _ in range(4))
    do = do * grad
    cut = n // 3
    for x in (k, v, do):
        if padding != "none":
            x[:, :, slice(n - cut, n) if padding == "last" else slice(0, cut)] = 0
    q, k, v, do = (x.to(torch.float16) for x in (q, k, v, do))
    lam = torch.tensor(lams)
    g = [x.to(DEV) for x in (q, k, v, do, lam)]
    outs = []
    for variant in (0, 2):
        binding.la2_set_scan_variant(variant)
        outs.append(tuple(binding.la2_fwd_state(*g[:3], g[4])) + tuple(binding.la2_bwd_state(*g)))
    torch.cuda.synchronize()
    q64, k64, v64, do64, lam64 = (to64(x) for x in (q, k, v, do, lam))
    refs = tuple(oracle.fwd_recurrent(q64, k64, v64, lam64, return_state=True)) + tuple(oracle.bwd_recurrent_state(q64, k64, v64, do64, lam64))
    assert all(np.all(np.isfinite(to64(x))) for x in outs[0])
    for name, short, blocks, ref in zip(("o", "kv_final", "dq", "dk", "dv", "d_kv_init"), *outs, refs):
        for h in range(4):
            a, b = (rms_rel(to64(x[0, h]), ref[0, h]) for x in (short, blocks))
            assert a <= 1.25 * b, "%s lambda %g: %.2e on the short path, %.2e in blocks" % (name, lams[h], a, b)


@pytest.mark.parametrize("dtype,d,chains,n", [(torch.bfloat16, 128, 64, 640), (torch.bfloat16, 128, 16, 1536), (torch.float16, 64, 32, 1024)])
def test_backward_in_blocks_after_a_short_forward(dtype, d, chains, n):
    """A forward pass without states on the short path (its workspace stays as it was) and a backward with all of them that the
    recurrence is faster at: it forms its own chunk states, or, given only the room for the other half of them, takes the short
    path as well.  Either way nothing is read from the forward call's workspace."""
    H = 16
    gen = torch.Generator(device=DEV)
    gen.manual_seed(chains + n + d)
    q, k, v, do = ((torch.randn((chains // H, H, n, d), generator=gen, device=DEV) * d ** -0.5).to(dtype) for _ in range(4))
    dkvf = torch.randn((chains // H, H, d, d), generator=gen, device=DEV) * 0.1
    lam = torch.exp(-torch.pow(2.0, -8.0 * torch.arange(1, H + 1) / H)).to(DEV)
    nchunks, _ = binding.la2_chunk_plan(q)
    states = chains * nchunks * d * d * 4
    assert nchunks > 1
    ws = torch.full((states,), 0xFF, dtype=torch.uint8, device=DEV)   # (as fp32: NaN)
    binding.la2_fwd(q, k, v, lam, workspace=ws)
    fresh = binding.la2_bwd_state(q, k, v, do, lam, d_kv_final=dkvf)
    outs = []
    for size in (2 * states, states):
        ws_b = torch.full((size,), 0xFF, dtype=torch.uint8, device=DEV)
        outs.append(binding.la2_bwd_state(q, k, v, do, lam, d_kv_final=dkvf, workspace=ws_b, fwd_workspace=ws))
        torch.cuda.synchronize()
        assert bool((ws_b == 0xFF).all()) == (size == states)
    assert bool((ws == 0xFF).all())
    for x, y, z in zip(fresh, *outs):
        assert torch.isfinite(x).all() and torch.equal(x, y) and rms_rel(to64(z), to64(x)) <= 2 * RMS_TOL[dtype]
