"""GPU parity: la2_fwd / la2_bwd / la2_decode_step (through the C ABI) against the fp64 oracle,
element by element on the same seeded inputs."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2401_04658_amd import binding, workloads
from parity import TOL, assert_close, max_rel, to64

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(autouse=True)
def _auto_chunking():
    binding.la2_set_chunk_tokens(0)
    binding.la2_set_scan_variant(0)
    yield
    binding.la2_set_chunk_tokens(0)
    binding.la2_set_scan_variant(0)


def make_inputs(b, H, n, d, dtype, seed, lam=None, backward=True):
    wl = workloads.Workload("case", b, H, n, d, dtype, seed=seed, backward=backward)
    t = wl.tensors()
    if lam is not None:
        t["lam"] = torch.as_tensor(lam, dtype=torch.float32).reshape(-1).expand(H).contiguous()
    return t


def gpu(t):
    return {k: v.to(DEV) for k, v in t.items()}


def check_fwd_bwd(t, dtype, tag, backward=True):
    g = gpu(t)
    o = binding.la2_fwd(g["q"], g["k"], g["v"], g["lam"])
    torch.cuda.synchronize()
    q, k, v, lam = to64(t["q"]), to64(t["k"]), to64(t["v"]), to64(t["lam"])
    res = {"o": assert_close(tag + " o", o, oracle.fwd_direct(q, k, v, lam), dtype)}
    if backward:
        dq, dk, dv = binding.la2_bwd(g["q"], g["k"], g["v"], g["d_o"], g["lam"])
        torch.cuda.synchronize()
        rq, rk, rv = oracle.bwd_direct(q, k, v, to64(t["d_o"]), lam)
        res["dq"] = assert_close(tag + " dq", dq, rq, dtype)
        res["dk"] = assert_close(tag + " dk", dk, rk, dtype)
        res["dv"] = assert_close(tag + " dv", dv, rv, dtype)
    return res


# ---- configuration 1: forward, fp32 -------------------------------------------------------------------------
def test_config1_fwd_fp32():
    wl = workloads.CONFIG1
    check_fwd_bwd(wl.tensors(), wl.dtype, wl.name, backward=False)


# ---- configuration 2: 400M-model layer, bf16, full tensors against the O(n^2) oracle -----------------------------
def test_config2_fwd_bwd_bf16_full():
    wl = workloads.CONFIG2
    check_fwd_bwd(wl.tensors(), wl.dtype, wl.name)


# ---- small shapes spanning several tiles and ragged tails, both dtypes, both head dims ------------------------------
@pytest.mark.usefixtures("both_paths")
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [1, 31, 128, 129, 200, 384, 517])
def test_small_shapes(dtype, d, n):
    t = make_inputs(2, 3, n, d, dtype, seed=100 + n + d, lam=[0.5, 0.93, 1.0])
    check_fwd_bwd(t, dtype, "n%d d%d %s" % (n, d, dtype))


# ---- both bf16 head_dim-128 scan kernels (full-block B = 64, half-block B = 32), forced explicitly: the
# automatic choice depends on the launch size and would pick the full-block kernel for all small cases
@pytest.mark.parametrize("variant", [1, 2])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 64, 95, 129, 200, 517])
def test_scan_variants_small_shapes(variant, n):
    binding.la2_set_scan_variant(variant)
    t = make_inputs(2, 3, n, 128, torch.bfloat16, seed=300 + n, lam=[0.5, 0.93, 1.0])
    check_fwd_bwd(t, torch.bfloat16, "variant%d n%d" % (variant, n))


@pytest.mark.parametrize("variant", [1, 2])
@pytest.mark.parametrize("chunk,n", [(128, 1000), (192, 1024), (256, 700)])
def test_scan_variants_chunked(variant, chunk, n):
    binding.la2_set_scan_variant(variant)
    binding.la2_set_chunk_tokens(chunk)
    t = make_inputs(1, 4, n, 128, torch.bfloat16, seed=17 * n + chunk)
    assert binding.la2_workspace_bytes(t["q"].to(DEV)) > 0
    check_fwd_bwd(t, torch.bfloat16, "variant%d chunk%d n%d" % (variant, chunk, n))


@pytest.mark.parametrize("variant", [1, 2])
def test_scan_variants_extreme_decays_and_strides(variant):
    binding.la2_set_scan_variant(variant)
    t = make_inputs(1, 3, 300, 128, torch.bfloat16, seed=23, lam=[1.0, 1e-6, 0.43])
    check_fwd_bwd(t, torch.bfloat16, "variant%d extreme decays" % variant)
    b, H, n, d = 2, 4, 260, 128
    t = make_inputs(b, H, n, d, torch.bfloat16, seed=33)
    g = {}
    for name in ("q", "k", "v", "d_o"):
        g[name] = t[name].permute(0, 2, 1, 3).contiguous().to(DEV).permute(0, 2, 1, 3)   # [b, n, H, d] storage
    lam = t["lam"].to(DEV)
    o = binding.la2_fwd(g["q"], g["k"], g["v"], lam)
    dq, dk, dv = binding.la2_bwd(g["q"], g["k"], g["v"], g["d_o"], lam)
    torch.cuda.synchronize()
    q, k, v, do, lam64 = (to64(t[x]) for x in ("q", "k", "v", "d_o", "lam"))
    assert_close("variant%d strided o" % variant, o, oracle.fwd_direct(q, k, v, lam64), torch.bfloat16)
    for name, got, ref in zip(("dq", "dk", "dv"), (dq, dk, dv), oracle.bwd_direct(q, k, v, do, lam64)):
        assert_close("variant%d strided %s" % (variant, name), got, ref, torch.bfloat16)


def test_scan_variants_agree():
    """The two kernels compute the same function: outputs differ by bf16 rounding only."""
    t = gpu(make_inputs(2, 4, 1500, 128, torch.bfloat16, seed=55))
    out = {}
    for variant in (1, 2):
        binding.la2_set_scan_variant(variant)
        out[variant] = (binding.la2_fwd(t["q"], t["k"], t["v"], t["lam"]),) + tuple(
            binding.la2_bwd(t["q"], t["k"], t["v"], t["d_o"], t["lam"]))
    torch.cuda.synchronize()
    for a, b in zip(out[1], out[2]):
        assert max_rel(to64(a), to64(b)) <= 1e-2


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("chunk", [128, 256, 384])
@pytest.mark.parametrize("d,n", [(64, 1000), (128, 1000), (128, 1024), (64, 257)])
def test_chunked_path(dtype, chunk, d, n):
    """Forces the sequence-chunk path (state pre-pass + scan) incl. a ragged last chunk."""
    binding.la2_set_chunk_tokens(chunk)
    t = make_inputs(1, 4, n, d, dtype, seed=7 * n + d + chunk)
    if chunk < n - 128:
        assert binding.la2_workspace_bytes(t["q"].to(DEV)) > 0
    check_fwd_bwd(t, dtype, "chunk%d n%d d%d %s" % (chunk, n, d, dtype))


def test_chunking_changes_results_only_by_rounding():
    t = gpu(make_inputs(1, 2, 2048, 128, torch.bfloat16, seed=11))
    base = binding.la2_fwd(t["q"], t["k"], t["v"], t["lam"])
    binding.la2_set_chunk_tokens(512)
    chunked = binding.la2_fwd(t["q"], t["k"], t["v"], t["lam"])
    torch.cuda.synchronize()
    assert max_rel(to64(chunked), to64(base)) <= 1e-2


def test_empty_and_degenerate():
    for n in (0,):
        t = gpu(make_inputs(2, 2, n, 64, torch.bfloat16, seed=1))
        o = binding.la2_fwd(t["q"], t["k"], t["v"], t["lam"])
        g = binding.la2_bwd(t["q"], t["k"], t["v"], t["d_o"], t["lam"])
        torch.cuda.synchronize()
        assert o.shape == (2, 2, 0, 64) and all(x.shape == (2, 2, 0, 64) for x in g)
    # batch of zero
    t = gpu(make_inputs(0, 2, 64, 64, torch.bfloat16, seed=1))
    assert binding.la2_fwd(t["q"], t["k"], t["v"], t["lam"]).numel() == 0


def test_longest_sequence_one_chain_spans_4_gib():
    """Close to the longest sequence the descriptor allows for head_dim 128 in bf16: one chain of 16,777,087
    positions, just short of 4 GiB (the kernels address a chain with 32-bit byte offsets), cut into about 256
    chunks, ragged at the end.  Constant inputs and lambda = 1/2: contributions from more than 160 positions away are
    below 2^-160, so every row equals a row of the oracle's result on a 160-position window."""
    n, d, win = (1 << 24) - 129, 128, 160
    c = 0.25
    x = torch.full((1, 1, n, d), c, dtype=torch.bfloat16, device=DEV)
    lam = torch.tensor([0.5], dtype=torch.float32, device=DEV)
    w64 = np.full((1, 1, win, d), c)
    ref_o = oracle.fwd_direct(w64, w64, w64, 0.5)[0, 0]
    ref_dq, ref_dk, ref_dv = (r[0, 0] for r in oracle.bwd_direct(w64, w64, w64, w64, 0.5))
    tol = TOL[torch.bfloat16]

    def check(name, got, ref, forward):
        got = got[0, 0]
        scale = float(np.max(np.abs(ref)))
        if forward:   # the first rows, then the steady state
            head, steady, rest = got[:win], ref[win - 1], got[win - 1:]
            edge_ref = ref
        else:         # the last rows (aligned at the end), and the steady state before them
            head, steady, rest = got[n - win:], ref[0], got[:n - win + 1]
            edge_ref = ref
        assert np.max(np.abs(to64(head) - edge_ref)) <= tol * scale, name + " edge rows"
        steady_t = torch.as_tensor(steady, dtype=torch.float32, device=DEV)
        err = (rest.float() - steady_t).abs().max().item()
        assert err <= tol * scale, "%s steady state: %.3e" % (name, err / scale)

    o = binding.la2_fwd(x, x, x, lam)
    torch.cuda.synchronize()
    check("o", o, ref_o, True)
    del o
    dq, dk, dv = binding.la2_bwd(x, x, x, x, lam)
    torch.cuda.synchronize()
    check("dq", dq, ref_dq, True)
    check("dk", dk, ref_dk, False)
    check("dv", dv, ref_dv, False)
    # two more positions do not fit the 32-bit chain offsets: refused on the host
    y = torch.empty((1, 1, n + 2, d), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(binding.LA2Error):
        binding.la2_fwd(y, y, y, lam)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_unscaled_values_and_slow_decay(dtype):
    """V and dO of unit variance (configuration 4's value scale) with decays close to 1 over a long sequence: the
    running state grows to its largest, which is what the 16-bit state operand (fp16: range 65504) has to hold."""
    wl = workloads.Workload("unscaled", 1, 3, 3000, 128, dtype, seed=71, v_scale=1.0)
    t = wl.tensors()
    t["lam"] = torch.tensor([1.0, 0.9999, 0.99], dtype=torch.float32)
    check_fwd_bwd(t, dtype, "unscaled %s" % dtype)


@pytest.mark.usefixtures("both_paths")
def test_extreme_decays():
    """lambda = 1 (pure causal prefix sum) and a very small lambda (only the diagonal survives)."""
    for dtype in (torch.bfloat16, torch.float16, torch.float32):
        t = make_inputs(1, 3, 300, 64, dtype, seed=21, lam=[1.0, 1e-6, 0.43])
        check_fwd_bwd(t, dtype, "extreme decays %s" % dtype)


@pytest.mark.usefixtures("both_paths")
def test_strided_layout():
    """[b, n, H, d] storage viewed as [b, H, n, d]: strides go through the descriptor."""
    b, H, n, d = 2, 4, 260, 128
    for dtype in (torch.bfloat16, torch.float16, torch.float32):
        t = make_inputs(b, H, n, d, dtype, seed=31)
        g = {}
        for name in ("q", "k", "v", "d_o"):
            store = t[name].permute(0, 2, 1, 3).contiguous().to(DEV)  # [b, n, H, d]
            g[name] = store.permute(0, 2, 1, 3)                       # view [b, H, n, d]
            assert not g[name].is_contiguous()
        lam = t["lam"].to(DEV)
        o = binding.la2_fwd(g["q"], g["k"], g["v"], lam)
        dq, dk, dv = binding.la2_bwd(g["q"], g["k"], g["v"], g["d_o"], lam)
        torch.cuda.synchronize()
        q, k, v, do, lam64 = (to64(t[x]) for x in ("q", "k", "v", "d_o", "lam"))
        assert_close("strided o", o, oracle.fwd_direct(q, k, v, lam64), dtype)
        for name, got, ref in zip(("dq", "dk", "dv"), (dq, dk, dv), oracle.bwd_direct(q, k, v, do, lam64)):
            assert_close("strided " + name, got, ref, dtype)


SPLIT_CASES = [(b, H, n, d, st, dt) for dt in (torch.bfloat16, torch.float16)
               for b, H, n, d, st in ((20, 16, 2048, 128, False), (18, 16, 2100, 64, True), (11, 32, 4096, 128, False))]
SPLIT_CASES += [(36, 16, 4096, 128, False, torch.float16), (34, 16, 4100, 64, True, torch.bfloat16),   # two rounds
                (50, 16, 4096, 64, False, torch.bfloat16),                                           # three
                (34, 8, 2048, 256, False, torch.bfloat16), (36, 8, 2100, 256, True, torch.float16),
                (18, 16, 2048, 96, False, torch.float16), (34, 16, 4096, 96, False, torch.bfloat16),
                (18, 16, 2048, 64, False, torch.float32), (18, 16, 1100, 128, True, torch.float32),
                (34, 16, 2048, 128, False, torch.float32)]


@pytest.mark.parametrize("b,H,n,d,strided,dtype", SPLIT_CASES)
def test_batches_a_little_above_the_compute_unit_count(b, H, n, d, strided, dtype):
    """A few more chains than one (or two) per compute unit: la2_fwd / la2_bwd run the rows that make whole rounds
    un-chunked and the remaining rows in chunks, as two calls on the same stream.  Chains on both sides of that cut,
    at sampled positions (block and chunk borders among them) against the O(n^2) oracle, and the Euler identity over
    everything."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    t = make_inputs(b, H, n, d, dtype, seed=53)
    g = {}
    for name in ("q", "k", "v", "d_o"):
        if strided:
            g[name] = t[name].permute(0, 2, 1, 3).contiguous().to(DEV).permute(0, 2, 1, 3)
        else:
            g[name] = t[name].to(DEV)
    lam = t["lam"].to(DEV)
    cut = min(max((b * H // cus) * cus // H, 1), b - 1)
    nch, chunk = binding.la2_chunk_plan(g["q"][cut:])
    if cus == 256:     # the split is what runs: its workspace is that of the remaining rows' plan
        assert nch > 1
        assert binding.la2_workspace_bytes(g["q"]) == binding.la2_workspace_bytes(g["q"][cut:]) > 0
    o = binding.la2_fwd(g["q"], g["k"], g["v"], lam)
    dq, dk, dv = binding.la2_bwd(g["q"], g["k"], g["v"], g["d_o"], lam)
    torch.cuda.synchronize()
    rng = np.random.default_rng(53)
    tol = TOL[dtype]
    borders = [c * chunk + e for c in range(1, nch) for e in (-1, 0, 1)]
    for row in sorted({0, cut - 1, cut, b - 1}):
        for h in (0, H // 2, H - 1):
            rows = np.array(sorted(set(sampled_rows(n, rng).tolist() + [r for r in borders if 0 <= r < n])), dtype=np.int64)
            q, k, v, do = (to64(t[x][row, h]) for x in ("q", "k", "v", "d_o"))
            lam_h = float(t["lam"][h].double())
            ref_o = oracle.fwd_rows(q, k, v, lam_h, rows)
            ref_dq, ref_dk, ref_dv = oracle.bwd_rows(q, k, v, do, lam_h, rows)
            for name, got, ref in (("o", o, ref_o), ("dq", dq, ref_dq), ("dk", dk, ref_dk), ("dv", dv, ref_dv)):
                x = to64(got[row, h])[rows]
                assert np.all(np.isfinite(x))
                err = float(np.max(np.abs(x - ref))) / float(np.max(np.abs(ref)))
                assert err <= tol, "%s (b%d h%d): %.3e" % (name, row, h, err)
    f64 = lambda x: x.to(torch.float64)
    L = torch.sum(f64(o) * f64(g["d_o"])).item()
    scale = torch.sum(torch.abs(f64(o) * f64(g["d_o"]))).item()
    for name, grad, x in (("dq", dq, g["q"]), ("dk", dk, g["k"]), ("dv", dv, g["v"])):
        assert abs(torch.sum(f64(grad) * f64(x)).item() - L) <= 2e-3 * scale, name
    for x in (o, dq, dk, dv):
        assert torch.isfinite(x.float()).all()


@pytest.mark.parametrize("d,n", [(128, 700), (64, 1300)])
def test_deterministic_and_causal(both_paths, d, n):
    t = gpu(make_inputs(2, 2, n, d, torch.bfloat16, seed=41))
    assert binding.la2_chunk_plan(t["q"])[0] > 1   # (blocks: pre-pass, accumulating dQ launch and twin launch)
    o1 = binding.la2_fwd(t["q"], t["k"], t["v"], t["lam"])
    o2 = binding.la2_fwd(t["q"], t["k"], t["v"], t["lam"])
    g1 = binding.la2_bwd(t["q"], t["k"], t["v"], t["d_o"], t["lam"])
    g2 = binding.la2_bwd(t["q"], t["k"], t["v"], t["d_o"], t["lam"])
    torch.cuda.synchronize()
    assert torch.equal(o1, o2)
    assert all(torch.equal(a, b) for a, b in zip(g1, g2))
    # changing tokens after position `cut` must leave earlier outputs bit-identical
    cut = 300
    q2, k2, v2 = t["q"].clone(), t["k"].clone(), t["v"].clone()
    for x in (q2, k2, v2):
        x[:, :, cut:] += 1.0
    o3 = binding.la2_fwd(q2, k2, v2, t["lam"])
    torch.cuda.synchronize()
    assert torch.equal(o1[:, :, :cut], o3[:, :, :cut])
    # changing dO before `cut` must leave dK, dV from `cut` on bit-identical
    do2 = t["d_o"].clone()
    do2[:, :, :cut] -= 2.0
    g3 = binding.la2_bwd(t["q"], t["k"], t["v"], do2, t["lam"])
    torch.cuda.synchronize()
    assert torch.equal(g1[1][:, :, cut:], g3[1][:, :, cut:])
    assert torch.equal(g1[2][:, :, cut:], g3[2][:, :, cut:])


# ---- full-size configurations 3 and 4: sampled rows against the O(n^2) oracle + Euler identity ----------------------
def sampled_rows(n, rng, count=24):
    fixed = [0, 1, 127, 128, 129, n // 2 - 1, n // 2, n - 129, n - 128, n - 2, n - 1]
    rnd = rng.integers(0, n, size=count - len(fixed)).tolist()
    return np.array(sorted(set(int(r) for r in fixed + rnd if 0 <= r < n)), dtype=np.int64)


def check_sampled(wl):
    t = wl.tensors()
    g = gpu(t)
    o = binding.la2_fwd(g["q"], g["k"], g["v"], g["lam"])
    dq, dk, dv = binding.la2_bwd(g["q"], g["k"], g["v"], g["d_o"], g["lam"])
    torch.cuda.synchronize()
    rng = np.random.default_rng(wl.seed)
    H = wl.heads
    tol = TOL[wl.dtype]
    for b, h in ((0, 0), (wl.batch - 1, H // 2), (0, H - 1)):
        rows = sampled_rows(wl.seqlen, rng)
        q, k, v, do = (to64(t[x][b, h]) for x in ("q", "k", "v", "d_o"))
        lam = float(t["lam"][h].double())
        ref_o = oracle.fwd_rows(q, k, v, lam, rows)
        ref_dq, ref_dk, ref_dv = oracle.bwd_rows(q, k, v, do, lam, rows)
        for name, got, ref in (("o", o, ref_o), ("dq", dq, ref_dq), ("dk", dk, ref_dk), ("dv", dv, ref_dv)):
            x = to64(got[b, h])[rows]
            # normalise by the largest magnitude of the sampled oracle rows of this chain
            err = float(np.max(np.abs(x - ref))) / float(np.max(np.abs(ref)))
            assert np.all(np.isfinite(x))
            assert err <= tol, "%s %s (b%d h%d): %.3e" % (wl.name, name, b, h, err)
    # Euler identity on the full GPU outputs: <dQ,Q> = <dK,K> = <dV,V> = <dO,O>
    f64 = lambda x: x.to(torch.float64)
    L = torch.sum(f64(o) * f64(g["d_o"])).item()
    scale = torch.sum(torch.abs(f64(o) * f64(g["d_o"]))).item()
    for name, grad, x in (("dq", dq, g["q"]), ("dk", dk, g["k"]), ("dv", dv, g["v"])):
        val = torch.sum(f64(grad) * f64(x)).item()
        assert abs(val - L) <= 2e-3 * scale, "%s Euler identity: %g vs %g" % (name, val, L)
    for x in (o, dq, dk, dv):
        assert torch.isfinite(x.float()).all()


@pytest.mark.parametrize("idx", range(4))
def test_config3_sweep_sampled(idx):
    check_sampled(workloads.CONFIG3[idx])


def test_config4_3b_layer_sampled():
    check_sampled(workloads.CONFIG4)


# ---- configuration 5: decode ------------------------------------------------------------------------------------
def run_decode(wl, batch, steps):
    g = wl.generator()
    H, d = wl.heads, wl.head_dim
    state0 = wl.initial_state(g)[:batch].contiguous()
    lam = wl.decay()
    kv_gpu = state0.to(DEV)
    kv_ref = state0.double().numpy().copy()
    lam_gpu, lam64 = lam.to(DEV), lam.double().numpy()
    worst = 0.0
    for step in range(steps):
        q, k, v = (x[:batch].contiguous() for x in wl.token(g))
        o = binding.la2_decode_step(q.to(DEV), k.to(DEV), v.to(DEV), lam_gpu, kv_gpu)
        ref = oracle.decode_step(to64(q), to64(k), to64(v), lam64, kv_ref)
        if step < 4 or step % 97 == 0 or step == steps - 1:
            worst = max(worst, max_rel(to64(o), ref))
            assert worst <= TOL[torch.bfloat16], "decode o at step %d: %.3e" % (step, worst)
    torch.cuda.synchronize()
    m = max_rel(to64(kv_gpu), kv_ref)
    assert m <= 1e-5, "decode state after %d steps: %.3e" % (steps, m)


def test_config5_decode_full_batch_few_steps():
    run_decode(workloads.CONFIG5, workloads.CONFIG5.batch, 3)


def test_config5_decode_1024_steps_one_batch_row():
    run_decode(workloads.CONFIG5, 1, workloads.CONFIG5.steps)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
def test_decode_matches_forward(d, dtype):
    """n decode steps from a zero state reproduce the forward output row by row."""
    b, H, n = 2, 3, 40
    t = make_inputs(b, H, n, d, dtype, seed=51, backward=False)
    g = gpu(t)
    kv = torch.zeros(b, H, d, d, dtype=torch.float32, device=DEV)
    rows = []
    for s in range(n):
        rows.append(binding.la2_decode_step(g["q"][:, :, s].contiguous(), g["k"][:, :, s].contiguous(),
                                            g["v"][:, :, s].contiguous(), g["lam"], kv))
    torch.cuda.synchronize()
    o = torch.stack(rows, dim=2)
    q, k, v, lam = (to64(t[x]) for x in ("q", "k", "v", "lam"))
    assert_close("decode-as-forward", o, oracle.fwd_direct(q, k, v, lam), dtype)
    _, kvf = oracle.fwd_recurrent(q, k, v, lam, return_state=True)
    assert max_rel(to64(kv), kvf) <= 1e-5


@pytest.mark.usefixtures("both_paths")
def test_hip_graph_capture_and_replay():
    """The library allocates nothing and never synchronises, so a forward + backward (incl. the chunked
    path with its workspace) can be captured into a HIP graph.  Replays, with eager work and
    synchronisations between them, must reproduce the eager results bit for bit."""
    # the last shape runs as two calls (288 chains on 256 units): an un-chunked part and a chunked one per pass
    for (b, H, n, d) in ((2, 4, 700, 128), (1, 2, 2048, 128), (1, 4, 900, 64), (18, 16, 2048, 64)):
        t = gpu(make_inputs(b, H, n, d, torch.bfloat16, seed=61 + n))
        ws = torch.empty(max(256, binding.la2_workspace_bytes(t["q"], binding.LA2_OP_BWD)), dtype=torch.uint8,
                         device=DEV)
        o = torch.empty_like(t["q"])
        grads = tuple(torch.empty_like(t["q"]) for _ in range(3))
        eager_o = binding.la2_fwd(t["q"], t["k"], t["v"], t["lam"], workspace=ws).clone()
        eager_g = [x.clone() for x in binding.la2_bwd(t["q"], t["k"], t["v"], t["d_o"], t["lam"], workspace=ws)]
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            # warm-up on the capture stream, then capture
            binding.la2_fwd(t["q"], t["k"], t["v"], t["lam"], out=o, workspace=ws)
            side.synchronize()
            with torch.cuda.graph(graph, stream=side):
                binding.la2_fwd(t["q"], t["k"], t["v"], t["lam"], out=o, workspace=ws)
                binding.la2_bwd(t["q"], t["k"], t["v"], t["d_o"], t["lam"], out=grads, workspace=ws)
        torch.cuda.current_stream().wait_stream(side)
        for replay in range(3):
            o.fill_(float("nan"))
            for x in grads:
                x.fill_(float("nan"))
            ws.random_(0, 255)                      # the workspace carries nothing between calls
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(o, eager_o), (n, d, replay)
            for got, ref in zip(grads, eager_g):
                assert torch.equal(got, ref), (n, d, replay)
            # eager work between replays
            assert torch.equal(binding.la2_fwd(t["q"], t["k"], t["v"], t["lam"], workspace=ws), eager_o)
            torch.cuda.synchronize()


@pytest.mark.usefixtures("both_paths")
def test_hip_graph_capture_of_the_other_entry_points():
    """Segments with state hand-over (ragged: block kernels + short-run kernels), the normalised operator,
    multi-token decode and a decode step in one captured graph; replays reproduce the eager results bit for bit."""
    b, H, n, d = 2, 3, 300, 128
    t = gpu(make_inputs(b, H, n, d, torch.bfloat16, seed=77))
    gen = torch.Generator(device="cpu")
    gen.manual_seed(78)
    kv0 = (torch.randn((b, H, d, d), generator=gen) * 0.3).to(DEV)
    dkvn = (torch.randn((b, H, d, d), generator=gen) * 0.3).to(DEV)
    ws = torch.empty(max(256, binding.la2_workspace_bytes(t["q"], binding.LA2_OP_BWD_STATE)), dtype=torch.uint8, device=DEV)
    T = 8
    qm, km, vm = (t[x][:, :, :T].contiguous() for x in ("q", "k", "v"))

    def run(out):
        o, kvf = binding.la2_fwd_state(t["q"], t["k"], t["v"], t["lam"], kv_init=kv0, out=out["o"], kv_final=out["kvf"],
                                       workspace=ws)
        binding.la2_bwd_state(t["q"], t["k"], t["v"], t["d_o"], t["lam"], kv_init=kv0, d_kv_final=dkvn,
                              out=out["grads"], d_kv_init=out["dkv0"], workspace=ws)
        binding.la2_fwd_norm(t["q"], t["k"], t["v"], t["lam"], 1e-5, out=out["on"], rstd=out["rstd"], workspace=ws)
        binding.la2_bwd_norm(t["q"], t["k"], t["v"], out["on"], out["rstd"], t["d_o"], t["lam"], out=out["gn"],
                             d_u=out["du"], workspace=ws)
        out["state"].copy_(kv0)
        binding.la2_decode_multi(qm, km, vm, t["lam"], out["state"], out=out["om"])
        binding.la2_decode_step(qm[:, :, 0].contiguous(), km[:, :, 0].contiguous(), vm[:, :, 0].contiguous(), t["lam"],
                                out["state"], out=out["o1"])

    def buffers():
        like = lambda: torch.empty_like(t["q"])
        return {"o": like(), "kvf": torch.empty_like(kv0), "grads": (like(), like(), like()), "dkv0": torch.empty_like(kv0),
                "on": like(), "rstd": torch.empty((b, H, n), device=DEV), "gn": (like(), like(), like()), "du": like(),
                "state": torch.empty_like(kv0), "om": torch.empty_like(qm), "o1": torch.empty_like(qm[:, :, 0])}

    def flat(out):
        return [out["o"], out["kvf"], *out["grads"], out["dkv0"], out["on"], out["rstd"], *out["gn"], out["du"],
                out["state"], out["om"], out["o1"]]

    # .contiguous() inside run() allocates: do those once outside the capture by warming up first
    eager = buffers()
    run(eager)
    torch.cuda.synchronize()
    captured = buffers()
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run(captured)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            run(captured)
    torch.cuda.current_stream().wait_stream(side)
    for replay in range(3):
        for x in flat(captured):
            x.fill_(float("nan"))
        ws.random_(0, 255)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for i, (got, ref) in enumerate(zip(flat(captured), flat(eager))):
            assert torch.equal(got, ref), (replay, i)
        scratch = buffers()            # eager work between the replays
        run(scratch)
        torch.cuda.synchronize()


# ---- the O(n^2 d) left-product comparison kernel computes the same forward pass ---------------------------------------
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [1, 31, 64, 128, 129, 200, 517, 1000])
def test_left_product_kernel_small_shapes(d, n):
    t = make_inputs(2, 3, n, d, torch.bfloat16, seed=400 + n + d, lam=[0.5, 0.93, 1.0])
    g = gpu(t)
    o = binding.la2_left_product_fwd(g["q"], g["k"], g["v"], g["lam"])
    torch.cuda.synchronize()
    ref = oracle.fwd_direct(to64(t["q"]), to64(t["k"]), to64(t["v"]), to64(t["lam"]))
    assert_close("left product n%d d%d" % (n, d), o, ref, torch.bfloat16)


def test_left_product_kernel_config2_and_extreme_decays():
    wl = workloads.CONFIG2
    t = wl.tensors()
    g = gpu(t)
    o = binding.la2_left_product_fwd(g["q"], g["k"], g["v"], g["lam"])
    torch.cuda.synchronize()
    assert_close("left product config2", o, oracle.fwd_direct(to64(t["q"]), to64(t["k"]), to64(t["v"]), to64(t["lam"])),
                 torch.bfloat16)
    t = make_inputs(1, 3, 300, 128, torch.bfloat16, seed=24, lam=[1.0, 1e-6, 0.43])
    g = gpu(t)
    o = binding.la2_left_product_fwd(g["q"], g["k"], g["v"], g["lam"])
    torch.cuda.synchronize()
    assert_close("left product extreme decays", o,
                 oracle.fwd_direct(to64(t["q"]), to64(t["k"]), to64(t["v"]), to64(t["lam"])), torch.bfloat16)
    with pytest.raises(binding.LA2Error):
        f = gpu(make_inputs(1, 1, 64, 64, torch.float32, seed=1))
        binding.la2_left_product_fwd(f["q"], f["k"], f["v"], f["lam"])


# ---- ... and its backward form the same gradients ------------------------------------------------------------------
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [1, 31, 64, 128, 129, 200, 517, 1000])
def test_left_product_backward_small_shapes(d, n):
    t = make_inputs(2, 3, n, d, torch.bfloat16, seed=450 + n + d, lam=[0.5, 0.93, 1.0])
    g = gpu(t)
    dq, dk, dv = binding.la2_left_product_bwd(g["q"], g["k"], g["v"], g["d_o"], g["lam"])
    torch.cuda.synchronize()
    refs = oracle.bwd_direct(to64(t["q"]), to64(t["k"]), to64(t["v"]), to64(t["d_o"]), to64(t["lam"]))
    for name, got, ref in zip(("dq", "dk", "dv"), (dq, dk, dv), refs):
        assert_close("left product %s n%d d%d" % (name, n, d), got, ref, torch.bfloat16)


def test_left_product_backward_config2_and_extreme_decays():
    for t in (workloads.CONFIG2.tensors(), make_inputs(1, 3, 300, 128, torch.bfloat16, seed=25, lam=[1.0, 1e-6, 0.43])):
        g = gpu(t)
        got = binding.la2_left_product_bwd(g["q"], g["k"], g["v"], g["d_o"], g["lam"])
        torch.cuda.synchronize()
        refs = oracle.bwd_direct(to64(t["q"]), to64(t["k"]), to64(t["v"]), to64(t["d_o"]), to64(t["lam"]))
        for name, x, ref in zip(("dq", "dk", "dv"), got, refs):
            assert_close("left product bwd " + name, x, ref, torch.bfloat16)
    # strided layout ([b, n, H, d] storage)
    t = make_inputs(2, 3, 333, 128, torch.bfloat16, seed=26)
    g = {}
    for name in ("q", "k", "v", "d_o"):
        g[name] = t[name].permute(0, 2, 1, 3).contiguous().to(DEV).permute(0, 2, 1, 3)
    lam = t["lam"].to(DEV)
    got = binding.la2_left_product_bwd(g["q"], g["k"], g["v"], g["d_o"], lam)
    torch.cuda.synchronize()
    refs = oracle.bwd_direct(to64(t["q"]), to64(t["k"]), to64(t["v"]), to64(t["d_o"]), to64(t["lam"]))
    for name, x, ref in zip(("dq", "dk", "dv"), got, refs):
        assert_close("left product bwd strided " + name, x, ref, torch.bfloat16)
    with pytest.raises(binding.LA2Error):
        f = gpu(make_inputs(1, 1, 64, 64, torch.float16, seed=1))
        binding.la2_left_product_bwd(f["q"], f["k"], f["v"], f["d_o"], f["lam"])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n,chunk", [(33, 0), (95, 0), (290, 64), (290, 96)])
def test_fp32_products_keep_fp32_accuracy_whatever_the_scale_of_a_feature(n, chunk, d):
    """The fp32 kernels multiply on the bf16 matrix instructions, every float split into three bf16 parts.  Features
    scaled by powers of two from 2^-20 to 2^20 (key-like and query-like inversely, so that every term counts; value-like
    each its own): every output column stays within 1e-6 of its own size, which one part less (2^-17) would miss by a
    factor of ten and a shared exponent by far more.  Bound: products within 2^-24 (rms 2^-27), fp32 sums of at most
    290 + 128 terms and decay weights good to a few 2^-24."""
    g = torch.Generator(device="cpu")
    g.manual_seed(n + d)
    b, H = 1, 3
    draw = lambda: torch.randn((b, H, n, d), generator=g, dtype=torch.float32)
    qk = torch.pow(2.0, torch.randint(-20, 21, (d,), generator=g).float())
    vv = torch.pow(2.0, torch.randint(-20, 21, (d,), generator=g).float())
    q, k, v, do = draw() * qk, draw() / qk, draw() * vv, draw() / vv
    lam = torch.tensor([0.3, 0.95, 1.0])
    binding.la2_set_chunk_tokens(chunk)
    try:
        gq, gk, gv, gdo, gl = (x.to(DEV) for x in (q, k, v, do, lam))
        got = (binding.la2_fwd(gq, gk, gv, gl),) + tuple(binding.la2_bwd(gq, gk, gv, gdo, gl))
        torch.cuda.synchronize()
    finally:
        binding.la2_set_chunk_tokens(0)
    q, k, v, do, lam = (to64(x) for x in (q, k, v, do, lam))
    ref = (oracle.fwd_direct(q, k, v, lam),) + tuple(oracle.bwd_direct(q, k, v, do, lam))
    for name, x, r in zip(("o", "dq", "dk", "dv"), got, ref):
        err = np.sqrt(((to64(x) - r) ** 2).mean(axis=2)) / np.sqrt((r ** 2).mean(axis=2))
        assert err.max() <= 1e-6, (name, err.max())


def fp32_case(n, d, exps=(0, 0, 0, 0), seed=11):
    """q, k, v, d_o of N(0, 1) times 2^e each, three heads."""
    g = torch.Generator(device="cpu")
    g.manual_seed(seed + n + d)
    return [torch.randn((1, 3, n, d), generator=g) * 2.0 ** e for e in exps] + [torch.tensor([0.3, 0.95, 1.0])]


def fp32_run(x):
    q, k, v, do, lam = (t.to(DEV) for t in x)
    out = (binding.la2_fwd(q, k, v, lam),) + tuple(binding.la2_bwd(q, k, v, do, lam))
    torch.cuda.synchronize()
    return out


def fp32_refs(x):
    q, k, v, do, lam = (to64(t) for t in x)
    return (oracle.fwd_direct(q, k, v, lam),) + tuple(oracle.bwd_direct(q, k, v, do, lam))


@pytest.mark.parametrize("exps", [(0, -116, 0, 0), (116, -116, 0, 0), (0, 0, -116, 100), (-130, 20, 0, 116), (0, -58, -58, 0),
                                  (-60, -60, 90, 0), (60, 60, -60, 0), (116, 0, -50, -50), (0, 115, 4, -115), (118, -120, 0, 0),
                                  (40, 40, 40, 0)])
@pytest.mark.parametrize("d,chunk", [(64, 0), (128, 0), (64, 64), (128, 96)])
def test_fp32_accuracy_over_the_range_of_the_type(d, chunk, exps):
    """Inputs, scores and states from 2^-130 to 2^122: every output is as accurate as on ordinary data.  (The bf16 parts of
    a value below 2^-110 would leave bf16's range, those of one above 3.39e38 as well.  No combination has scores or states
    that fp32 itself rounds to its subnormals.)"""
    n = 200
    x = fp32_case(n, d, exps)
    binding.la2_set_chunk_tokens(chunk)
    got, refs = fp32_run(x), fp32_refs(x)
    for name, y, r in zip(("o", "dq", "dk", "dv"), got, refs):
        big = np.abs(r).max()
        if big > 3e38 or big < 1e-36:     # beyond the type, or rounded to its subnormals
            continue
        assert np.isfinite(to64(y)).all(), (name, big)
        err = np.sqrt(((to64(y) - r) ** 2).sum() / (r ** 2).sum())
        assert err <= 1e-6, (name, err, big)


@pytest.mark.parametrize("d,chunk", [(64, 0), (128, 0), (64, 64), (128, 96)])
@pytest.mark.parametrize("which", [0, 1, 2, 3])
def test_fp32_one_largest_value_is_a_finite_number(which, d, chunk):
    """A value next to fp32's largest (rounded to bf16 it is Inf) among ordinary ones: every result is finite and within
    264 roundings (d + n products and sums) of the sum of the magnitudes it is made of."""
    n, at, bound = 200, 70, 264 * 2.0 ** -24
    x = fp32_case(n, d, (-6, -6, -6, -6), seed=which)
    for value in (3.4028234e38, -3.4e38):
        x[which][0, 1, at, 5] = value
        binding.la2_set_chunk_tokens(chunk)
        got, refs, sizes = fp32_run(x), fp32_refs(x), fp32_refs([t.abs() for t in x])
        for name, y, r, size in zip(("o", "dq", "dk", "dv"), got, refs, sizes):
            assert size.max() < 3e38
            assert np.isfinite(to64(y)).all(), name
            assert (np.abs(to64(y) - r) <= bound * size).all(), (name, (np.abs(to64(y) - r) / size).max())


@pytest.mark.parametrize("d,n", [(64, 200), (128, 200), (64, 192), (128, 193)])
def test_fp32_chunks_that_are_walked_again_keep_states_and_norm(d, n):
    """A query value that overflows the split operands sends its chunk through the fp32 matrix instructions: start and
    final states (in place too), their gradients, the Norm epilogue and every other row as without it."""
    x = fp32_case(n, d, seed=5)
    gen = torch.Generator(device="cpu")
    gen.manual_seed(d + n)
    kv0, dkv = (torch.randn((1, 3, d, d), generator=gen) for _ in range(2))
    q, k, v, do, lam = (t.to(DEV) for t in x)
    odd = q.clone()
    odd[0, 1, 70, 5] = 1e36
    for chunk in (0, 64):
        binding.la2_set_chunk_tokens(chunk)
        outs = []
        for y in (q, odd):
            o, kvf = binding.la2_fwd_state(y, k, v, lam, kv_init=kv0.to(DEV))
            grads = binding.la2_bwd_state(q, k, v, torch.where(y == 1e36, y, do), lam, kv_init=kv0.to(DEV), d_kv_final=dkv.to(DEV))
            on, rstd = binding.la2_fwd_norm(y, k, v, lam, 1e-6)
            kept = kv0.to(DEV)
            om = binding.la2_decode_multi(y, k, v, lam, kept)
            torch.cuda.synchronize()
            outs.append([to64(z) for z in (o, grads[0], on, rstd, om, kvf, kept)])
        for i, (a, b) in enumerate(zip(*outs)):
            assert np.abs(a).max() < 1e6
            if i < 5:      # all rows but the one that the value belongs to
                rows = np.delete(np.arange(n), 70)
                assert np.abs(b[0, 1, 70]).max() > 1e30 or i == 3 or i == 2
                a, b = a[:, :, rows], b[:, :, rows]
            # (Norm: a row's r takes the relative error of its norm, up to 264 roundings where its terms cancel)
            assert np.abs(a - b).max() <= (264 * 2.0 ** -24 if i in (2, 3) else 2e-6) * np.abs(a).max(), (chunk, i)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("chunk", [0, 64])
def test_fp32_infinite_values_stay_infinite(chunk, d):
    """One infinite key feature: the state row it enters is infinite, and every later block's output is the infinity of
    the sign of q_t[i] v_s[j], not NaN; dv's infinities towards earlier positions come from an infinite query."""
    n, at = 200, 70
    x = fp32_case(n, d, (-3, -3, -3, -3))
    binding.la2_set_chunk_tokens(chunk)
    q, k, v, do, lam = x
    bad = [q, k.clone(), v, do, lam]
    bad[1][0, 1, at, 5] = float("inf")
    o = fp32_run(bad)[0].cpu()
    assert torch.equal(o[0, 1, 96:], torch.sign(q[0, 1, 96:, 5, None] * v[0, 1, at]) * float("inf"))
    bad = [q.clone(), k, v, do, lam]
    bad[0][0, 1, at, 5] = float("-inf")
    dv = fp32_run(bad)[3].cpu()
    assert torch.equal(dv[0, 1, :64], torch.sign(k[0, 1, :64, 5, None] * do[0, 1, at]) * float("-inf"))


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_a_non_finite_value_reaches_its_block_and_later_positions_only(d):
    """(Positions 64 .. 69 share the block of 32 with it: their masked products are 0 times it, which is NaN.)"""
    n, at = 130, 70   # block 64 .. 95 holds it
    g = torch.Generator(device="cpu")
    g.manual_seed(d)
    q, k, v = (torch.randn((1, 2, n, d), generator=g).to(DEV) for _ in range(3))
    lam = torch.tensor([0.9, 0.99], device=DEV)
    ref = binding.la2_fwd(q, k, v, lam)
    for bad in (float("nan"), float("inf")):
        w = v.clone()
        w[0, 1, at, 5] = bad
        o = binding.la2_fwd(q, k, w, lam)
        torch.cuda.synchronize()
        assert torch.equal(o[0, 0], ref[0, 0]) and torch.equal(o[0, 1, :64], ref[0, 1, :64])
        assert not torch.isfinite(o[0, 1, at:, 5]).any()
