"""Backward passes whose three scans run in one launch (16-bit data), against the fp64 oracle and against the
launches one after the other (scan variant 2)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2401_04658_amd import binding, workloads
from parity import assert_close, rms_rel, to64

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(autouse=True)
def _defaults():
    binding.la2_set_chunk_tokens(0)
    binding.la2_set_scan_variant(0)
    yield
    binding.la2_set_chunk_tokens(0)
    binding.la2_set_scan_variant(0)


# head_dim, batch, heads, length: in the plan's chunks with a scan over their states and without one, uncut instead of them, uncut as
# before; up to half the units, about all of them, a partial second round, and one that else runs as two calls
@pytest.mark.parametrize("d,b,h,n", [(64, 1, 4, 2113), (64, 1, 16, 2048), (64, 3, 16, 1000), (64, 6, 16, 1100), (64, 8, 16, 1031),
                                     (64, 10, 16, 200), (64, 16, 16, 257), (64, 18, 16, 130), (128, 5, 16, 416), (128, 3, 16, 1000),
                                     (96, 3, 2, 300), (96, 3, 16, 1000), (96, 5, 16, 1100), (96, 17, 16, 97), (96, 1, 16, 2050), (96, 1, 4, 2050),
                                     (128, 6, 16, 1056), (128, 10, 16, 100), (128, 16, 16, 65), (128, 13, 16, 225), (128, 18, 16, 127),
                                     (128, 19, 16, 2049), (96, 17, 16, 2053), (64, 19, 16, 2055)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_all_scans_in_one_launch(dtype, d, b, h, n):
    """Batch rows are copies of one, so every row has the same bits; with states and without, the forward call's states and none,
    and d_kv_init in kv_init's place (which the dQ scan has to have read by then)."""
    t = workloads.Workload("joint", 1, h, n, d, dtype, seed=8300 + n + d, backward=True).tensors()
    gen = torch.Generator(device="cpu")
    gen.manual_seed(8300 + n)
    init, dfin = (torch.randn((1, h, d, d), generator=gen) * 0.3 for _ in range(2))
    lam = t["lam"].to(DEV)
    q, k, v, do = (t[x].to(DEV).expand(b, -1, -1, -1).contiguous() for x in ("q", "k", "v", "d_o"))
    q64, k64, v64, do64, lam64 = (to64(t[x]) for x in ("q", "k", "v", "d_o", "lam"))
    for given in (False, True):
        kv0, dkv = (x.to(DEV).expand(b, -1, -1, -1).contiguous() if given else None for x in (init, dfin))
        i64, f64 = (to64(init), to64(dfin)) if given else (None, None)
        refs = oracle.bwd_recurrent_state(q64, k64, v64, do64, lam64, kv_init=i64, d_kv_final=f64)
        binding.la2_set_scan_variant(2)
        apart = binding.la2_bwd_state(q, k, v, do, lam, kv_init=kv0, d_kv_final=dkv)
        binding.la2_set_scan_variant(0)
        ws = torch.empty(max(256, binding.la2_workspace_bytes(q, binding.LA2_OP_FWD_STATE)), dtype=torch.uint8, device=DEV)
        binding.la2_fwd_state(q, k, v, lam, kv_init=kv0, want_final=False, workspace=ws)
        runs = {"": binding.la2_bwd_state(q, k, v, do, lam, kv_init=kv0, d_kv_final=dkv),
                "saved": binding.la2_bwd_state(q, k, v, do, lam, kv_init=kv0, d_kv_final=dkv, fwd_workspace=ws)}
        if given:
            place = kv0.clone()
            runs["in place"] = binding.la2_bwd_state(q, k, v, do, lam, kv_init=place, d_kv_final=dkv, d_kv_init=place)
        torch.cuda.synchronize()
        for kind, outs in runs.items():
            for name, x, ref, other in zip(("dq", "dk", "dv", "d_kv_init"), outs, refs, apart):
                label = "%s d%d b%d h%d n%d states %s %s" % (name, d, b, h, n, given, kind)
                if kind == "in place":   # (one after the other again, where that is two calls with chunks of their own)
                    assert_close(label, x[-1:], ref, dtype)
                else:
                    assert torch.equal(x, x[:1].expand_as(x)), label
                assert_close(label, x[:1], ref, dtype)
                # no further from the truth than the launches apart (the same sums, or those of other chunks: up to their order)
                assert rms_rel(to64(x[:1]), ref) <= 1.05 * rms_rel(to64(other[:1]), ref) + 1e-7, label


# packed: in the plan's chunks through the pair map (a scan over the chunk states, none), uncut, few chains of head_dim 128, head_dim 96
# (no states there); sequences of no position, of one, off the block boundaries
PACKED = [(64, 2, [2500, 700, 33, 0, 1, 400]), (64, 16, [1, 33, 700, 0, 257, 64, 900, 31, 500, 450, 300, 222]), (64, 16, [1100, 1000, 1050, 0, 1200, 1]),
          (128, 16, [416, 33, 0, 257, 400]), (96, 4, [300, 33, 1, 257, 0, 400, 31]), (96, 16, [97] * 40 + [96, 1, 130])]


@pytest.mark.parametrize("d,h,lengths", PACKED)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_all_scans_of_a_packed_batch_in_one_launch(dtype, d, h, lengths):
    """With states and without (head_dim 96: without), and with d_kv_init in kv_init's place, against the launches apart and the oracle."""
    total, nseq = sum(lengths), len(lengths)
    t = workloads.Workload("joint", 1, h, total, d, dtype, seed=8700 + total + d, backward=True).tensors()
    gen = torch.Generator(device="cpu")
    gen.manual_seed(8700 + total)
    init, dfin = (torch.randn((nseq, h, d, d), generator=gen) * 0.3 for _ in range(2))
    q, k, v, do = (t[x][0].permute(1, 0, 2).contiguous().to(DEV) for x in ("q", "k", "v", "d_o"))
    lam, ends = t["lam"].to(DEV), [0]
    for n in lengths:
        ends.append(ends[-1] + n)
    cu, longest = torch.tensor(ends, dtype=torch.int32, device=DEV), max(lengths)
    for given in (False, True) if d != 96 else (False,):
        kv0, dkv = (init.to(DEV), dfin.to(DEV)) if given else (None, None)
        call = dict(kv_init=kv0, d_kv_final=dkv, want_d_kv_init=given)
        binding.la2_set_scan_variant(2)
        apart = binding.la2_bwd_varlen_state(q, k, v, do, lam, cu, longest, **call)
        binding.la2_set_scan_variant(0)
        runs = {"": binding.la2_bwd_varlen_state(q, k, v, do, lam, cu, longest, **call)}
        if given:
            place = kv0.clone()
            runs["in place"] = binding.la2_bwd_varlen_state(q, k, v, do, lam, cu, longest, kv_init=place, d_kv_final=dkv, d_kv_init=place)
        torch.cuda.synchronize()
        refs = [[], [], []]
        for i, n in enumerate(lengths):
            if n == 0:
                continue
            seq = {x: to64(t[x][:, :, ends[i]:ends[i + 1]].contiguous()) for x in ("q", "k", "v", "d_o")}
            grads = oracle.bwd_recurrent_state(seq["q"], seq["k"], seq["v"], seq["d_o"], to64(t["lam"]),
                                               kv_init=to64(init[i:i + 1]) if given else None, d_kv_final=to64(dfin[i:i + 1]) if given else None)
            for ref, x in zip(refs, grads):
                ref.append(x[0].transpose(1, 0, 2))
            for kind, outs in runs.items():
                if given:
                    assert_close("d_kv_init seq %d %s" % (i, kind), outs[3][i:i + 1], grads[3], dtype)
        for kind, outs in runs.items():
            for name, x, ref, other in zip(("dq", "dk", "dv"), outs, refs, apart):
                label = "%s d%d h%d %s states %s %s" % (name, d, h, lengths[:8], given, kind)
                ref = np.concatenate(ref)
                assert_close(label, x, ref, dtype)
                # no further from the truth than the launches apart
                assert rms_rel(to64(x), ref) <= 1.05 * rms_rel(to64(other), ref) + 1e-7, label
            if given:   # a sequence of no positions passes its state's gradient on
                for i, n in enumerate(lengths):
                    assert n > 0 or torch.equal(outs[3][i].cpu(), dfin[i])


@pytest.mark.parametrize("d,h,n", [(64, 4, 1000), (64, 16, 2050), (128, 16, 1500), (128, 8, 3001)])
def test_fp32_chunk_states_in_one_launch(d, h, n):
    """fp32 in chunks: on dense tensors the KV states wait in dV's place; with rows further apart nothing between them is touched."""
    t = workloads.Workload("pair", 2, h, n, d, torch.float32, seed=8600 + n + d, backward=True).tensors()
    assert binding.la2_chunk_plan(t["q"])[0] > 1
    g = {x: y.to(DEV) for x, y in t.items()}
    dense = binding.la2_bwd(g["q"], g["k"], g["v"], g["d_o"], g["lam"])

    def apart(x):   # rows 16 floats further apart, 7.0 between them
        store = torch.full(x.shape[:3] + (d + 16,), 7.0, device=DEV)
        store[..., :d] = x
        return store[..., :d], store

    q, k, v, do = (apart(g[x])[0] for x in ("q", "k", "v", "d_o"))
    outs, stores = zip(*(apart(torch.zeros_like(g["q"])) for _ in range(3)))
    binding.la2_bwd(q, k, v, do, g["lam"], out=outs)
    torch.cuda.synchronize()
    refs = oracle.bwd_recurrent_state(*(to64(t[x][:1]) for x in ("q", "k", "v", "d_o")), to64(t["lam"]))
    for name, x, y, store, ref in zip(("dq", "dk", "dv"), dense, outs, stores, refs):
        assert torch.equal(x, y), name
        assert bool((store[..., d:] == 7.0).all()), name
        assert_close("%s d%d h%d n%d" % (name, d, h, n), x[:1], ref, torch.float32)
