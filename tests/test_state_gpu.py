"""GPU parity of la2_fwd_state / la2_bwd_state (segments with state hand-over) against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2401_04658_amd import binding, workloads
from parity import TOL, assert_close, max_rel, to64

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(autouse=True)
def _defaults():
    binding.la2_set_chunk_tokens(0)
    binding.la2_set_scan_variant(0)
    yield
    binding.la2_set_chunk_tokens(0)
    binding.la2_set_scan_variant(0)


def inputs(b, H, n, d, dtype, seed, lam=None):
    t = workloads.Workload("case", b, H, n, d, dtype, seed=seed, backward=True).tensors()
    if lam is not None:
        t["lam"] = torch.as_tensor(lam, dtype=torch.float32).reshape(-1).expand(H).contiguous()
    g = torch.Generator(device="cpu")
    g.manual_seed(seed + 1000)
    # states of the size a few hundred tokens of such inputs build up; gradients of the same order
    t["kv_init"] = torch.randn((b, H, d, d), generator=g, dtype=torch.float32) * 0.3
    t["d_kv_final"] = torch.randn((b, H, d, d), generator=g, dtype=torch.float32) * 0.3
    return t


def state_tol(dtype):
    # states are fp32 sums of products of the (bf16 or fp32) inputs
    return TOL[dtype]


def check_segment(t, dtype, tag, use_init=True, use_final=True):
    g = {k: v.to(DEV) for k, v in t.items()}
    kv_init = g["kv_init"] if use_init else None
    d_fin = g["d_kv_final"] if use_final else None
    o, kvf = binding.la2_fwd_state(g["q"], g["k"], g["v"], g["lam"], kv_init=kv_init, want_final=use_final)
    dq, dk, dv, dkv0 = binding.la2_bwd_state(g["q"], g["k"], g["v"], g["d_o"], g["lam"], kv_init=kv_init,
                                             d_kv_final=d_fin)
    torch.cuda.synchronize()
    q, k, v, do, lam = (to64(t[x]) for x in ("q", "k", "v", "d_o", "lam"))
    init64 = to64(t["kv_init"]) if use_init else None
    fin64 = to64(t["d_kv_final"]) if use_final else None
    ro, rkvf = oracle.fwd_recurrent(q, k, v, lam, kv_init=init64, return_state=True)
    rdq, rdk, rdv, rdkv0 = oracle.bwd_recurrent_state(q, k, v, do, lam, kv_init=init64, d_kv_final=fin64)
    assert_close(tag + " o", o, ro, dtype)
    if use_final:
        assert_close(tag + " kv_final", kvf, rkvf, dtype)
    assert_close(tag + " dq", dq, rdq, dtype)
    assert_close(tag + " dk", dk, rdk, dtype)
    assert_close(tag + " dv", dv, rdv, dtype)
    assert_close(tag + " d_kv_init", dkv0, rdkv0, dtype)


@pytest.mark.usefixtures("both_paths")
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [64, 128, 320])
def test_segment_with_all_states(dtype, d, n):
    t = inputs(2, 3, n, d, dtype, seed=500 + n + d, lam=[0.5, 0.93, 1.0])
    check_segment(t, dtype, "n%d d%d %s" % (n, d, dtype))


@pytest.mark.usefixtures("both_paths")
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [1, 31, 64, 100, 129, 300])
def test_ragged_segments(dtype, d, n):
    """Lengths that do not end on a block boundary: the block kernels do the whole blocks, a token-by-token
    tail the rest (both directions), with and without the states at the far end."""
    t = inputs(1, 3, n, d, dtype, seed=600 + n + d, lam=[0.43, 0.9, 0.99])
    check_segment(t, dtype, "ragged n%d d%d %s start state only" % (n, d, dtype), use_final=False)
    check_segment(t, dtype, "ragged n%d d%d %s all states" % (n, d, dtype))
    check_segment(t, dtype, "ragged n%d d%d %s final states only" % (n, d, dtype), use_init=False)


@pytest.mark.parametrize("variant", [1, 2])
@pytest.mark.parametrize("chunk", [0, 128])
@pytest.mark.parametrize("d", [64, 128])
def test_segment_chunked_and_variants(variant, chunk, d):
    binding.la2_set_scan_variant(variant)
    binding.la2_set_chunk_tokens(chunk)
    t = inputs(1, 4, 512, d, torch.bfloat16, seed=700 + d + chunk)
    if chunk:
        assert binding.la2_workspace_bytes(t["q"].to(DEV)) > 0
    check_segment(t, torch.bfloat16, "variant%d chunk%d d%d" % (variant, chunk, d))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("nchunks", [2, 3, 4, 5])
def test_plans_of_few_chunks_form_their_start_states_in_the_scan(nchunks, d, dtype):
    """Up to four chunks the scan over the chunk states has no launch of its own: every scan workgroup combines the
    local states of the chunks before it (with the caller's start state in front, also where it is read transposed
    or enters behind a ragged last block); five chunks take the launch.  Same results either way, with all four
    states, with none, and for a last chunk that is shorter than the others and ends inside a block."""
    chunk = 128
    for n in (nchunks * chunk, nchunks * chunk - 45):
        binding.la2_set_chunk_tokens(chunk)
        t = inputs(2, 3, n, d, dtype, seed=900 + 10 * nchunks + d + n, lam=[0.6, 0.95, 1.0])
        whole = {k: (v[:, :, : n - n % 32] if k in ("q", "k", "v", "d_o") else v) for k, v in t.items()}
        plan = binding.la2_chunk_plan(whole["q"].contiguous().to(DEV))
        assert plan == (nchunks, chunk), plan
        tag = "%d chunks n%d d%d %s" % (nchunks, n, d, dtype)
        check_segment(t, dtype, tag + " all states")
        check_segment(t, dtype, tag + " no states", use_init=False, use_final=False)
        check_segment(t, dtype, tag + " start state only", use_final=False)


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 64), (torch.float16, 128), (torch.float32, 64), (torch.bfloat16, 96),
                                     (torch.bfloat16, 256)])
@pytest.mark.parametrize("nchunks", [32, 33, 64, 65, 71])
def test_scan_over_more_chunks_than_it_holds_at_once(nchunks, dtype, d):
    """The scan over the chunk states takes 32 of them at a time: counts on both sides of one and two such runs, a last
    chunk that is whole and one that ends inside a block, with all states and with none."""
    chunk = 64
    for n in (nchunks * chunk, nchunks * chunk - 45):
        binding.la2_set_chunk_tokens(chunk)
        t = inputs(1, 2, n, d, dtype, seed=700 + nchunks + d + n, lam=[0.99, 0.9995])
        assert binding.la2_chunk_plan(t["q"]) == (nchunks, chunk)
        check_segment(t, dtype, "%d chunks n%d d%d %s" % (nchunks, n, d, dtype))
        check_segment(t, dtype, "%d chunks n%d d%d %s, no states" % (nchunks, n, d, dtype), use_init=False, use_final=False)


def test_fp32_chunked_segment():
    binding.la2_set_chunk_tokens(128)
    t = inputs(1, 2, 384, 128, torch.float32, seed=777)
    check_segment(t, torch.float32, "fp32 chunked")


@pytest.mark.usefixtures("both_paths")
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
def test_two_segments_equal_the_whole_sequence(dtype):
    """Forward left to right, backward right to left through the hand-over states, against the oracle's
    DIRECT form of the whole sequence (which has no notion of a state)."""
    b, H, n, d, cut = 2, 4, 448, 128, 192
    t = inputs(b, H, n, d, dtype, seed=800)
    g = {k: v.to(DEV) for k, v in t.items()}
    seg = [slice(0, cut), slice(cut, n)]
    part = lambda name, s: g[name][:, :, s].contiguous()
    o1, s1 = binding.la2_fwd_state(part("q", seg[0]), part("k", seg[0]), part("v", seg[0]), g["lam"])
    o2, _ = binding.la2_fwd_state(part("q", seg[1]), part("k", seg[1]), part("v", seg[1]), g["lam"], kv_init=s1,
                                  want_final=False)
    dq2, dk2, dv2, gs = binding.la2_bwd_state(part("q", seg[1]), part("k", seg[1]), part("v", seg[1]),
                                              part("d_o", seg[1]), g["lam"], kv_init=s1)
    dq1, dk1, dv1, g0 = binding.la2_bwd_state(part("q", seg[0]), part("k", seg[0]), part("v", seg[0]),
                                              part("d_o", seg[0]), g["lam"], d_kv_final=gs)
    torch.cuda.synchronize()
    q, k, v, do, lam = (to64(t[x]) for x in ("q", "k", "v", "d_o", "lam"))
    assert_close("two segments o", torch.cat([o1, o2], 2), oracle.fwd_direct(q, k, v, lam), dtype)
    rq, rk, rv = oracle.bwd_direct(q, k, v, do, lam)
    assert_close("two segments dq", torch.cat([dq1, dq2], 2), rq, dtype)
    assert_close("two segments dk", torch.cat([dk1, dk2], 2), rk, dtype)
    assert_close("two segments dv", torch.cat([dv1, dv2], 2), rv, dtype)


@pytest.mark.usefixtures("both_paths")
def test_prefill_then_decode():
    """The final state of a prefill continues with la2_decode_step (same state layout)."""
    b, H, n, d = 2, 4, 256, 128
    t = inputs(b, H, n + 3, d, torch.bfloat16, seed=900)
    g = {k: v.to(DEV) for k, v in t.items()}
    head = lambda name: g[name][:, :, :n].contiguous()
    _, state = binding.la2_fwd_state(head("q"), head("k"), head("v"), g["lam"])
    outs = []
    for i in range(n, n + 3):
        outs.append(binding.la2_decode_step(g["q"][:, :, i].contiguous(), g["k"][:, :, i].contiguous(),
                                            g["v"][:, :, i].contiguous(), g["lam"], state))
    torch.cuda.synchronize()
    ref = oracle.fwd_direct(to64(t["q"]), to64(t["k"]), to64(t["v"]), to64(t["lam"]))
    for j, o in enumerate(outs):
        assert max_rel(to64(o), ref[:, :, n + j]) <= TOL[torch.bfloat16]


def test_empty_segment_passes_the_state_through():
    t = inputs(2, 2, 0, 64, torch.bfloat16, seed=1)
    g = {k: v.to(DEV) for k, v in t.items()}
    _, kvf = binding.la2_fwd_state(g["q"], g["k"], g["v"], g["lam"], kv_init=g["kv_init"])
    *_, g0 = binding.la2_bwd_state(g["q"], g["k"], g["v"], g["d_o"], g["lam"], d_kv_final=g["d_kv_final"])
    _, kvz = binding.la2_fwd_state(g["q"], g["k"], g["v"], g["lam"])
    torch.cuda.synchronize()
    assert torch.equal(kvf, g["kv_init"]) and torch.equal(g0, g["d_kv_final"])
    assert torch.count_nonzero(kvz) == 0


@pytest.mark.parametrize("point", [1, 2])
def test_sweep_points_with_states(point):
    """Configuration-3 sweep points ((16, 4K) un-chunked, (4, 16K) sequence-chunked) in the launch
    configuration bench.py times, with a start state and both state gradients; full tensors against the
    oracle's recurrent form."""
    wl = workloads.CONFIG3[point]
    t = wl.tensors()
    g = torch.Generator(device="cpu")
    g.manual_seed(4242 + point)
    shape = (wl.batch, wl.heads, wl.head_dim, wl.head_dim)
    t["kv_init"] = torch.randn(shape, generator=g, dtype=torch.float32) * 0.3
    t["d_kv_final"] = torch.randn(shape, generator=g, dtype=torch.float32) * 0.3
    check_segment(t, wl.dtype, wl.name + " with states")


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T", [1, 2, 7, 32, 33, 64, 100])
def test_decode_multi(dtype, d, T):
    b, H = 3, 4
    t = inputs(b, H, T, d, dtype, seed=1100 + T + d, lam=[0.5, 0.9, 0.99, 1.0])
    g = {k: v.to(DEV) for k, v in t.items()}
    state = g["kv_init"].clone()
    o = binding.la2_decode_multi(g["q"], g["k"], g["v"], g["lam"], state)
    # the same tokens one step at a time
    state1 = g["kv_init"].clone()
    o1 = [binding.la2_decode_step(g["q"][:, :, i].contiguous(), g["k"][:, :, i].contiguous(),
                                  g["v"][:, :, i].contiguous(), g["lam"], state1) for i in range(T)]
    torch.cuda.synchronize()
    ro, rs = oracle.fwd_recurrent(to64(t["q"]), to64(t["k"]), to64(t["v"]), to64(t["lam"]),
                                  kv_init=to64(t["kv_init"]), return_state=True)
    assert_close("decode_multi o", o, ro, dtype)
    assert_close("decode_multi state", state, rs, dtype)
    assert max_rel(to64(torch.stack(o1, 2)), ro) <= TOL[dtype]
    assert max_rel(to64(state1), rs) <= TOL[dtype]


def test_decode_multi_config5_shape():
    """Configuration 5's batch and heads, 8 tokens per launch, one batch row against the oracle."""
    dw = workloads.CONFIG5
    gen = dw.generator()
    kv0 = dw.initial_state(gen)
    toks = [dw.token(gen) for _ in range(8)]
    q, k, v = (torch.stack([tk[i] for tk in toks], 2).contiguous() for i in range(3))
    lam = dw.decay()
    state = kv0.to(DEV)
    o = binding.la2_decode_multi(q.to(DEV), k.to(DEV), v.to(DEV), lam.to(DEV), state)
    torch.cuda.synchronize()
    rows = slice(5, 7)
    ro, rs = oracle.fwd_recurrent(to64(q[rows]), to64(k[rows]), to64(v[rows]), to64(lam), kv_init=to64(kv0[rows]),
                                  return_state=True)
    assert_close("config5 multi o", o[rows], ro, torch.bfloat16)
    assert_close("config5 multi state", state[rows], rs, torch.bfloat16)


@pytest.mark.parametrize("b,H,n,d,dtype", [(20, 16, 2048, 128, torch.bfloat16), (18, 16, 2100, 64, torch.float16),
                                           (18, 16, 1100, 128, torch.float32), (34, 8, 2048, 256, torch.bfloat16),
                                           # 12 heads do not divide 256 units: the first part has 252 chains, which the
                                           # fp32 head_dim 64 plan cuts in three, so both parts use the workspace
                                           (22, 12, 2048, 64, torch.float32)])
def test_states_of_batches_a_little_above_the_compute_unit_count(b, H, n, d, dtype):
    """Such a batch runs as two calls (the rows that give every compute unit one chain, then the others in chunks):
    each part takes its own rows of kv_init / d_kv_final and writes its own rows of kv_final / d_kv_init.  Whole
    lengths and ragged ones, full tensors against the oracle's recurrent form; then the training-step pair, the
    backward reading the chunk states the forward call left in its workspace."""
    t = inputs(b, H, n, d, dtype, seed=1700 + n + d)
    check_segment(t, dtype, "two calls %s b%d n%d d%d" % (dtype, b, n, d))
    g = {k: v.to(DEV) for k, v in t.items()}
    need = binding.la2_workspace_bytes(g["q"], binding.LA2_OP_BWD_STATE)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert need > 0 and binding.la2_chunk_plan(g["q"])[0] == 1      # one call would need none
    ws_f = torch.empty(max(256, need), dtype=torch.uint8, device=DEV)
    ws_b = torch.empty(max(256, need), dtype=torch.uint8, device=DEV)
    binding.la2_fwd_state(g["q"], g["k"], g["v"], g["lam"], kv_init=g["kv_init"], want_final=False, workspace=ws_f)
    dq, dk, dv, g0 = binding.la2_bwd_state(g["q"], g["k"], g["v"], g["d_o"], g["lam"], kv_init=g["kv_init"],
                                           workspace=ws_b, fwd_workspace=ws_f)
    torch.cuda.synchronize()
    q, k, v, do, lam = (to64(t[x]) for x in ("q", "k", "v", "d_o", "lam"))
    rdq, rdk, rdv, rg0 = oracle.bwd_recurrent_state(q, k, v, do, lam, kv_init=to64(t["kv_init"]))
    for name, got, ref in (("dq", dq, rdq), ("dk", dk, rdk), ("dv", dv, rdv), ("d_kv_init", g0, rg0)):
        assert_close("two calls, saved states " + name, got, ref, dtype)


@pytest.mark.parametrize("dtype,d,n,chunk", [(torch.bfloat16, 128, 1024, 256), (torch.bfloat16, 64, 1000, 128),
                                             (torch.float32, 128, 640, 128), (torch.bfloat16, 128, 900, 0)])
def test_backward_reuses_the_forward_chunk_states(dtype, d, n, chunk):
    """A training step: the forward call's workspace (chunk start states of the K, V scan) is handed to the
    backward call, which then skips its own pre-pass for dQ.  Same results within tolerance, with and
    without a start state; no effect when the launch is not chunked (chunk = 0 with enough chains)."""
    binding.la2_set_chunk_tokens(chunk)
    b, H = (1, 4) if chunk else (16, 16)
    t = inputs(b, H, n, d, dtype, seed=1300 + n + d)
    g = {k: v.to(DEV) for k, v in t.items()}
    need = binding.la2_workspace_bytes(g["q"], binding.LA2_OP_BWD_STATE)
    assert (need > 0) == bool(chunk) or n % 64 != 0
    ws_f = torch.empty(max(256, need), dtype=torch.uint8, device=DEV)
    ws_b = torch.empty(max(256, need), dtype=torch.uint8, device=DEV)
    for use_init in (False, True):
        kv_init = g["kv_init"] if use_init else None
        binding.la2_fwd_state(g["q"], g["k"], g["v"], g["lam"], kv_init=kv_init, want_final=False, workspace=ws_f)
        dq, dk, dv, g0 = binding.la2_bwd_state(g["q"], g["k"], g["v"], g["d_o"], g["lam"], kv_init=kv_init,
                                               workspace=ws_b, fwd_workspace=ws_f)
        torch.cuda.synchronize()
        q, k, v, do, lam = (to64(t[x]) for x in ("q", "k", "v", "d_o", "lam"))
        rdq, rdk, rdv, rg0 = oracle.bwd_recurrent_state(q, k, v, do, lam,
                                                        kv_init=to64(t["kv_init"]) if use_init else None)
        tag = "saved states %s d%d n%d init=%s" % (dtype, d, n, use_init)
        assert_close(tag + " dq", dq, rdq, dtype)
        assert_close(tag + " dk", dk, rdk, dtype)
        assert_close(tag + " dv", dv, rdv, dtype)
        assert_close(tag + " d_kv_init", g0, rg0, dtype)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("nchunks", [3, 4, 5])
def test_fp32_ignores_the_scan_variant_between_forward_and_backward(nchunks, d):
    """The scan variant is a knob of the 16-bit kernels: an fp32 forward call and a backward call that reads its chunk
    states agree on what the workspace holds whatever the knob says in between."""
    b, H, chunk = 2, 3, 64
    n = chunk * nchunks - 7
    t = inputs(b, H, n, d, torch.float32, seed=31 * nchunks + d, lam=0.99)
    g = {k: v.to(DEV) for k, v in t.items()}
    binding.la2_set_chunk_tokens(chunk)
    results = []
    for first, second in ((0, 0), (0, 1), (1, 0)):
        binding.la2_set_scan_variant(first)
        ws_f = torch.empty(binding.la2_workspace_bytes(g["q"], binding.LA2_OP_FWD), dtype=torch.uint8, device=DEV)
        o = binding.la2_fwd(g["q"], g["k"], g["v"], g["lam"], workspace=ws_f)
        binding.la2_set_scan_variant(second)
        grads = binding.la2_bwd_state(g["q"], g["k"], g["v"], g["d_o"], g["lam"], fwd_workspace=ws_f)
        torch.cuda.synchronize()
        results.append((o,) + grads)
    q, k, v, do, lam = (to64(t[x]) for x in ("q", "k", "v", "d_o", "lam"))
    for name, got, ref in zip(("dq", "dk", "dv"), results[0][1:], oracle.bwd_direct(q, k, v, do, lam)):
        assert_close(name, got, ref, torch.float32)
    for other in results[1:]:
        assert all(torch.equal(x, y) for x, y in zip(results[0], other))


@pytest.mark.parametrize("d,n,chunk", [(64, 1000, 128), (128, 1025, 256), (128, 1000, 256)])
def test_backward_after_a_forward_that_wrote_kv_final_at_a_ragged_length(d, n, chunk):
    """The forward call that hands out kv_final for a ragged length plans its chunks for the whole blocks only.
    Told so, the backward call uses the saved chunk states when the two plans agree ((64, 1000, 128) and
    (128, 1000, 256)) and recomputes them when they do not ((128, 1025, 256): 5 chunks against 4)."""
    dtype = torch.bfloat16
    binding.la2_set_chunk_tokens(chunk)
    try:
        t = inputs(1, 4, n, d, dtype, seed=1400 + n + d)
        g = {k: v.to(DEV) for k, v in t.items()}
        need_f = binding.la2_workspace_bytes(g["q"], binding.LA2_OP_FWD_STATE)
        need_b = binding.la2_workspace_bytes(g["q"], binding.LA2_OP_BWD_STATE)
        ws_f = torch.full((need_f,), 0xFF, dtype=torch.uint8, device=DEV)      # NaN patterns where nothing is written
        ws_b = torch.empty(need_b, dtype=torch.uint8, device=DEV)
        o, kvn = binding.la2_fwd_state(g["q"], g["k"], g["v"], g["lam"], kv_init=g["kv_init"], workspace=ws_f)
        dq, dk, dv, g0 = binding.la2_bwd_state(g["q"], g["k"], g["v"], g["d_o"], g["lam"], kv_init=g["kv_init"],
                                               workspace=ws_b, fwd_workspace=ws_f, fwd_wrote_kv_final=True)
        torch.cuda.synchronize()
    finally:
        binding.la2_set_chunk_tokens(0)
    q, k, v, do, lam = (to64(t[x]) for x in ("q", "k", "v", "d_o", "lam"))
    rdq, rdk, rdv, rg0 = oracle.bwd_recurrent_state(q, k, v, do, lam, kv_init=to64(t["kv_init"]))
    tag = "saved after kv_final d%d n%d" % (d, n)
    assert_close(tag + " dq", dq, rdq, dtype)
    assert_close(tag + " dk", dk, rdk, dtype)
    assert_close(tag + " dv", dv, rdv, dtype)
    assert_close(tag + " d_kv_init", g0, rg0, dtype)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n,chunk", [(1024, 256), (1000, 128), (777, 64), (4096, 512)])
def test_dq_launch_forms_the_reverse_chunk_states(dtype, d, n, chunk):
    """Sequence chunks at head_dim 64 / 128: the dQ scan's launch also accumulates the local dKV states of the chunks
    (second wave group), the dK / dV scan starts from them.  Against the oracle, with start state and incoming
    state gradient, whole and ragged lengths, single-block chunks (64) included; and against the path that does
    not fuse (full-block kernel forced: separate pre-pass over Q and dO)."""
    t = inputs(2, 3, n, d, dtype, seed=1500 + n + d, lam=[0.37, 0.9, 0.999])
    g = {k: v.to(DEV) for k, v in t.items()}
    binding.la2_set_chunk_tokens(chunk)
    assert binding.la2_chunk_plan(g["q"])[0] > 1
    use_final = n % 32 == 0   # an incoming gradient at a ragged end splits the reverse pass: not the fused path
    d_fin = g["d_kv_final"] if use_final else None
    dq, dk, dv, g0 = binding.la2_bwd_state(g["q"], g["k"], g["v"], g["d_o"], g["lam"], kv_init=g["kv_init"],
                                           d_kv_final=d_fin)
    binding.la2_set_scan_variant(1)
    uq, uk, uv, u0 = binding.la2_bwd_state(g["q"], g["k"], g["v"], g["d_o"], g["lam"], kv_init=g["kv_init"],
                                           d_kv_final=d_fin)
    torch.cuda.synchronize()
    q, k, v, do, lam = (to64(t[x]) for x in ("q", "k", "v", "d_o", "lam"))
    rdq, rdk, rdv, rg0 = oracle.bwd_recurrent_state(q, k, v, do, lam, kv_init=to64(t["kv_init"]),
                                                    d_kv_final=to64(t["d_kv_final"]) if use_final else None)
    tag = "fused reverse states %s d%d n%d chunk%d" % (dtype, d, n, chunk)
    for name, got, other, ref in (("dq", dq, uq, rdq), ("dk", dk, uk, rdk), ("dv", dv, uv, rdv), ("d_kv_init", g0, u0, rg0)):
        assert_close(tag + " " + name, got, ref, dtype)
        assert_close(tag + " unfused " + name, other, ref, dtype)


@pytest.mark.parametrize("d,chains,n", [(128, 224, 128), (128, 224, 150), (128, 223, 150), (64, 448, 160), (64, 448, 129), (64, 447, 129),
                                        (128, 256, 1152), (128, 256, 1153)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_prefill_of_a_full_round_stores_through_the_caches(dtype, d, chains, n):
    """A forward pass that hands out its state, from as many chains as fill the units on, up to tensors of 72 MiB: four chains
    against the oracle, with the Norm as well, and over whole blocks the bits of the pass without states, whose outputs go past
    the caches.  (A ragged length with a state has an instantiation of its own, which forms its update weights as one exponential
    each and not as a product of two: other roundings.)"""
    H = next(h for h in (16, 7, 3, 1) if chains % h == 0)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d + n + chains)
    q, k, v = ((torch.randn((chains // H, H, n, d), generator=gen, device=DEV) * d ** -0.5).to(dtype) for _ in range(3))
    lam = torch.exp(-torch.pow(2.0, -8.0 * torch.arange(1, H + 1) / H)).to(DEV)
    assert binding.la2_workspace_bytes(q, binding.LA2_OP_FWD_STATE) == 0   # not cut
    o, kvf = binding.la2_fwd_state(q, k, v, lam)
    on, rstd, kvn = binding.la2_fwd_state_norm(q, k, v, lam, 1e-4)
    plain = binding.la2_fwd(q, k, v, lam)
    plain_n, plain_r = binding.la2_fwd_norm(q, k, v, lam, 1e-4)
    torch.cuda.synchronize()
    if n % 32 == 0:
        assert torch.equal(o, plain) and torch.equal(on, plain_n) and torch.equal(rstd, plain_r)
    assert torch.equal(kvf, kvn)
    for b, h in ((0, 0), (chains // H - 1, H - 1), (chains // H // 2, H // 2), (0, H - 1)):
        x = [to64(t[b:b + 1, h:h + 1]) for t in (q, k, v)]
        ro, rkv = oracle.fwd_recurrent(*x, to64(lam[h:h + 1]), return_state=True)
        assert_close("prefill o", o[b:b + 1, h:h + 1], ro, dtype)
        assert_close("prefill state", kvf[b:b + 1, h:h + 1], rkv, dtype)
        rn, rr, _ = oracle.fwd_norm_state(*x, to64(lam[h:h + 1]), 1e-4, None)
        assert_close("prefill norm o", on[b:b + 1, h:h + 1], rn, dtype)
        assert_close("prefill rstd", rstd[b:b + 1, h:h + 1], rr, dtype)
