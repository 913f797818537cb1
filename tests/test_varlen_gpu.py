"""GPU parity of la2_fwd_varlen / la2_bwd_varlen (packed sequences of different lengths) against the fp64 oracle:
every sequence is a chain of its own, so the reference is the oracle applied sequence by sequence."""
import numpy as np
import pytest
import torch

import oracle
from paper_2401_04658_amd import binding, workloads
from parity import assert_close, to64

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(autouse=True)
def _defaults():
    binding.la2_set_chunk_tokens(0)
    binding.la2_set_scan_variant(0)
    yield
    binding.la2_set_chunk_tokens(0)
    binding.la2_set_scan_variant(0)


def packed_inputs(lengths, H, d, dtype, seed, lead=0, trail=0):
    """q, k, v, d_o as [lead + sum(lengths) + trail, H, d] (rows outside the sequences belong to nobody)."""
    total = lead + int(sum(lengths)) + trail
    wl = workloads.Workload("packed", 1, H, max(total, 1), d, dtype, seed=seed, backward=True)
    t = wl.tensors()
    out = {name: t[name][0, :, :total].permute(1, 0, 2).contiguous() for name in ("q", "k", "v", "d_o")}
    out["lam"] = t["lam"]
    cu = np.concatenate([[lead], lead + np.cumsum(lengths)]).astype(np.int32)
    return out, torch.from_numpy(cu)


def check_packed(lengths, H, d, dtype, seed, lead=0, trail=0, lam=None):
    t, cu = packed_inputs(lengths, H, d, dtype, seed, lead, trail)
    if lam is not None:
        t["lam"] = torch.as_tensor(lam, dtype=torch.float32).reshape(-1).expand(H).contiguous()
    g = {k: v.to(DEV) for k, v in t.items()}
    cu_g = cu.to(DEV)
    max_len = int(max(lengths)) if len(lengths) else 0
    o = torch.full_like(g["q"], float("nan"))
    grads = tuple(torch.full_like(g["q"], float("nan")) for _ in range(3))
    binding.la2_fwd_varlen(g["q"], g["k"], g["v"], g["lam"], cu_g, max_len, out=o)
    binding.la2_bwd_varlen(g["q"], g["k"], g["v"], g["d_o"], g["lam"], cu_g, max_len, out=grads)
    torch.cuda.synchronize()
    lam64 = to64(t["lam"])
    for b, n in enumerate(lengths):
        lo, hi = int(cu[b]), int(cu[b + 1])
        if n == 0:
            continue
        seq = {name: to64(t[name][lo:hi]).transpose(1, 0, 2)[None] for name in ("q", "k", "v", "d_o")}   # [1, H, n, d]
        tag = "lengths %s seq %d (n %d) d%d %s" % (list(lengths), b, n, d, dtype)
        ref_o = oracle.fwd_direct(seq["q"], seq["k"], seq["v"], lam64)
        assert_close(tag + " o", o[lo:hi].permute(1, 0, 2)[None], ref_o, dtype)
        for name, got, ref in zip(("dq", "dk", "dv"), grads,
                                  oracle.bwd_direct(seq["q"], seq["k"], seq["v"], seq["d_o"], lam64)):
            assert_close(tag + " " + name, got[lo:hi].permute(1, 0, 2)[None], ref, dtype)
    # rows that belong to no sequence are not written
    for x in (o,) + grads:
        assert torch.isnan(x[: int(cu[0])].float()).all() and torch.isnan(x[int(cu[-1]):].float()).all()
        assert torch.isfinite(x[int(cu[0]): int(cu[-1])].float()).all()


@pytest.mark.usefixtures("both_paths")
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("d", [64, 128])
def test_mixed_lengths(dtype, d):
    check_packed([70, 0, 1, 31, 32, 100, 517, 64, 3], 3, d, dtype, seed=800 + d, lam=[0.5, 0.93, 1.0])


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.bfloat16, 64), (torch.float32, 128), (torch.float16, 128)])
@pytest.mark.parametrize("chunk", [64, 192])
def test_mixed_lengths_chunked(dtype, d, chunk):
    """Few sequences, long ones among them: the launch is cut into sequence chunks planned for the longest;
    shorter sequences use fewer of them (16-bit data: one workgroup per chunk that exists; fp32: a dense grid)."""
    binding.la2_set_chunk_tokens(chunk)
    check_packed([700, 130, 64, 1000, 5, 0, 383], 2, d, dtype, seed=810 + d + chunk, lam=[0.8, 0.99])


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.bfloat16, 64), (torch.float16, 128)])
def test_skewed_lengths_with_many_chains_are_chunked(dtype, d):
    """Chains enough to fill the device, but one sequence 32 times longer than the others: told the total number
    of positions the library cuts the sequences into chunks of a quarter of the longest (the short ones are
    single chunks, interleaved here with the long one); same results."""
    import ctypes
    lengths = [64] * 150 + [2048] + [37] * 120 + [300, 0, 1]
    H = 2
    desc = binding.la2_desc(len(lengths), H, 2048, d, binding._dtype_code(torch.empty(0, dtype=dtype)), 0, 0, d, H * d)
    total, C = int(sum(lengths)), 512
    pairs, slots, nlong = total // C + len(lengths), 2 * total // C, total // C
    assert binding.load().la2_varlen_workspace_bytes(ctypes.byref(desc), total, binding.LA2_OP_FWD) == \
        ((pairs * 16 + nlong * 4 + 255) // 256) * 256 + slots * H * d * d * 4
    assert binding.load().la2_varlen_workspace_bytes(ctypes.byref(desc), 0, binding.LA2_OP_FWD) == 0
    check_packed(lengths, H, d, dtype, seed=850 + d, lam=[0.7, 0.995])


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.bfloat16, 64), (torch.float16, 128)])
@pytest.mark.parametrize("kind", ["sorted", "even", "few"])
def test_unequal_lengths_sorted_and_cut_evenly(kind, dtype, d):
    """The three plans of a batch of unequal lengths (256 compute units): chains that fill the device, the longest
    about the average load of a unit (uncut, the map only sorts); the longest well above it (even pieces); too few
    chains (even pieces, one per 256 positions).  Lengths on and off the 64-position granule, empty ones included."""
    if kind == "few":
        lengths, H = [1500, 40, 0, 333, 64, 257, 256], 2
    else:
        longest, total, H = (600, 16500, 16) if kind == "sorted" else (1300, 9500, 16)
        lengths = [longest - 23, 1, longest, 0, 449, 385, 384, 64, 65]
        while sum(lengths) < total:
            lengths.append(37 + 13 * (len(lengths) % 19))
    check_packed(lengths, H, d, dtype, seed=880 + d, lam=[0.6, 0.9, 0.99, 0.997] * (H // 4) if H >= 4 else [0.8, 0.997])


@pytest.mark.parametrize("batch", [255, 256, 257, 1023, 1024, 1025, 2070])
@pytest.mark.parametrize("even", [False, True])
def test_pair_map_over_its_rounds_of_sequences(even, batch):
    """The pair map takes 256 sequences at once, or 1024 at a time: long ones at the ends of such a round, empty ones,
    pieces of one size (the test knob) and even pieces (the automatic cut)."""
    lengths = [(7 * i) % 61 for i in range(batch)]
    for i in (0, 200, 255, 256, 1000, 1023, 1024, 2047, batch - 1):
        if i < batch:
            lengths[i] = 700 + i % 90
    if not even:
        binding.la2_set_chunk_tokens(128)
    check_packed(lengths, 1, 64, torch.bfloat16, seed=898 + batch, lam=[0.99])


def test_a_sequence_of_more_chunks_than_the_state_scan_holds_at_once():
    """Few chains, pieces of 256 positions: 36, 33 and 32 chunks in one batch, the scan over their states takes 32 at a
    time."""
    check_packed([9000, 300, 0, 8200, 8192], 1, 64, torch.bfloat16, seed=897, lam=[0.9995])


def test_an_uncut_batch_needs_no_workspace():
    """The map that sorts an uncut batch lives in the workspace; without one the batch runs in the order of the
    sequences, same results bit for bit."""
    import ctypes
    lengths, H, d = [600, 100, 577] + [170, 230] * 26, 16, 128
    t, cu = packed_inputs(lengths, H, d, torch.bfloat16, seed=890)
    g = {k: v.to(DEV) for k, v in t.items()}
    cu_g = cu.to(DEV)
    desc = binding._varlen_desc(g["q"], cu_g, max(lengths))
    lib, stream = binding.load(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    need = int(lib.la2_varlen_workspace_bytes(ctypes.byref(desc), sum(lengths), binding.LA2_OP_FWD))
    assert 0 < need < 4096
    o = binding.la2_fwd_varlen(g["q"], g["k"], g["v"], g["lam"], cu_g, max(lengths))
    o2 = torch.empty_like(o)
    assert lib.la2_fwd_varlen(ctypes.byref(desc), cu_g.data_ptr(), sum(lengths), g["q"].data_ptr(), g["k"].data_ptr(),
                              g["v"].data_ptr(), g["lam"].data_ptr(), o2.data_ptr(), None, 0, stream) == 0
    grads = binding.la2_bwd_varlen(g["q"], g["k"], g["v"], g["d_o"], g["lam"], cu_g, max(lengths))
    grads2 = [torch.empty_like(o) for _ in range(3)]
    assert lib.la2_bwd_varlen(ctypes.byref(desc), cu_g.data_ptr(), sum(lengths), g["q"].data_ptr(), g["k"].data_ptr(),
                              g["v"].data_ptr(), g["d_o"].data_ptr(), g["lam"].data_ptr(), grads2[0].data_ptr(),
                              grads2[1].data_ptr(), grads2[2].data_ptr(), None, 0, stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(o, o2) and all(torch.equal(a, b) for a, b in zip(grads, grads2))


@pytest.mark.usefixtures("both_paths")
def test_offset_first_sequence_and_unused_tail():
    check_packed([200, 45], 2, 128, torch.bfloat16, seed=820, lead=7, trail=9)


@pytest.mark.parametrize("variant", [1, 2])
def test_scan_variants(variant):
    binding.la2_set_scan_variant(variant)
    check_packed([129, 64, 300], 2, 128, torch.bfloat16, seed=830 + variant)


@pytest.mark.usefixtures("both_paths")
def test_equal_lengths_reproduce_the_dense_batch_bit_for_bit():
    b, H, n, d = 3, 4, 260, 128
    t = workloads.Workload("dense", b, H, n, d, torch.bfloat16, seed=840).tensors()
    g = {k: v.to(DEV) for k, v in t.items()}
    o = binding.la2_fwd(g["q"], g["k"], g["v"], g["lam"])
    grads = binding.la2_bwd(g["q"], g["k"], g["v"], g["d_o"], g["lam"])
    pk = {name: g[name].permute(0, 2, 1, 3).reshape(b * n, H, d).contiguous() for name in ("q", "k", "v", "d_o")}
    cu = torch.arange(0, (b + 1) * n, n, dtype=torch.int32, device=DEV)
    o2 = binding.la2_fwd_varlen(pk["q"], pk["k"], pk["v"], g["lam"], cu, n)
    grads2 = binding.la2_bwd_varlen(pk["q"], pk["k"], pk["v"], pk["d_o"], g["lam"], cu, n)
    torch.cuda.synchronize()
    unpack = lambda x: x.reshape(b, n, H, d).permute(0, 2, 1, 3)
    assert torch.equal(unpack(o2), o)
    for a, ref in zip(grads2, grads):
        assert torch.equal(unpack(a), ref)


def test_a_total_below_the_real_one_drops_sequences_and_stays_inside_the_workspace():
    """total_positions sizes the pair map and the state slots.  Told less than the lengths add up to, the library
    computes the sequences that fit its map and slots, leaves the others untouched and writes nothing past the
    workspace it asked for (the bytes behind it keep their pattern)."""
    import ctypes
    binding.la2_set_chunk_tokens(64)
    lengths, H, d, dtype = [700, 130, 64, 1000, 5, 383], 2, 128, torch.bfloat16
    t, cu = packed_inputs(lengths, H, d, dtype, seed=870)
    g = {k: v.to(DEV) for k, v in t.items()}
    cu_g = cu.to(DEV)
    lib, told, guard = binding.load(), 600, 4096
    desc = binding._varlen_desc(g["q"], cu_g, max(lengths))
    # 600 / 64 + 6 = 15 pairs, 2 * 600 / 64 = 18 slots: sequences 0 (11 chunks), 1 (3 chunks) and 2 (1 chunk) fit
    fits = [True, True, True, False, False, False]
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    o = torch.full_like(g["q"], float("nan"))
    grads = tuple(torch.full_like(g["q"], float("nan")) for _ in range(3))
    for op in (binding.LA2_OP_FWD, binding.LA2_OP_BWD):
        need = int(lib.la2_varlen_workspace_bytes(ctypes.byref(desc), told, op))
        assert 0 < need < int(lib.la2_varlen_workspace_bytes(ctypes.byref(desc), g["q"].shape[0], op))
        ws = torch.full((need + guard,), 0xAB, dtype=torch.uint8, device=DEV)
        if op == binding.LA2_OP_FWD:
            st = lib.la2_fwd_varlen(ctypes.byref(desc), cu_g.data_ptr(), told, g["q"].data_ptr(), g["k"].data_ptr(),
                                    g["v"].data_ptr(), g["lam"].data_ptr(), o.data_ptr(), ws.data_ptr(), need, stream)
        else:
            st = lib.la2_bwd_varlen(ctypes.byref(desc), cu_g.data_ptr(), told, g["q"].data_ptr(), g["k"].data_ptr(),
                                    g["v"].data_ptr(), g["d_o"].data_ptr(), g["lam"].data_ptr(), grads[0].data_ptr(),
                                    grads[1].data_ptr(), grads[2].data_ptr(), ws.data_ptr(), need, stream)
        assert st == 0
        torch.cuda.synchronize()
        assert bool((ws[need:] == 0xAB).all())
    lam64 = to64(t["lam"])
    for b, n in enumerate(lengths):
        lo, hi = int(cu[b]), int(cu[b + 1])
        if not fits[b]:
            for x in (o,) + grads:
                assert torch.isnan(x[lo:hi].float()).all(), b
            continue
        seq = {name: to64(t[name][lo:hi]).transpose(1, 0, 2)[None] for name in ("q", "k", "v", "d_o")}
        assert_close("seq %d o" % b, o[lo:hi].permute(1, 0, 2)[None], oracle.fwd_direct(seq["q"], seq["k"], seq["v"], lam64), dtype)
        for name, got, ref in zip(("dq", "dk", "dv"), grads,
                                  oracle.bwd_direct(seq["q"], seq["k"], seq["v"], seq["d_o"], lam64)):
            assert_close("seq %d %s" % (b, name), got[lo:hi].permute(1, 0, 2)[None], ref, dtype)


def test_a_total_below_the_real_one_with_even_pieces():
    """The same with the automatic even cut: what fits the map and the slots planned from the told total is computed, the
    other sequences stay untouched, nothing is written past the workspace."""
    import ctypes
    lengths, H, d, dtype, told, guard = [900, 64, 1500, 33, 700, 300], 2, 128, torch.bfloat16, 1500, 4096
    t, cu = packed_inputs(lengths, H, d, dtype, seed=895)
    g = {k: v.to(DEV) for k, v in t.items()}
    cu_g = cu.to(DEV)
    lib = binding.load()
    desc = binding._varlen_desc(g["q"], cu_g, max(lengths))
    need = int(lib.la2_varlen_workspace_bytes(ctypes.byref(desc), told, binding.LA2_OP_FWD))
    ws = torch.full((need + guard,), 0xAB, dtype=torch.uint8, device=DEV)
    o = torch.full_like(g["q"], float("nan"))
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert lib.la2_fwd_varlen(ctypes.byref(desc), cu_g.data_ptr(), told, g["q"].data_ptr(), g["k"].data_ptr(),
                              g["v"].data_ptr(), g["lam"].data_ptr(), o.data_ptr(), ws.data_ptr(), need, stream) == 0
    torch.cuda.synchronize()
    assert bool((ws[need:] == 0xAB).all())
    # pieces of at most 256: 1500 / 256 + 6 = 11 pairs and 2 * 1500 / 256 = 11 slots; 900 takes 4 of each, 64 a pair,
    # 1500 would take 6 pairs and slots (11 and 10 in all: fits), everything behind it finds the map full
    lam64 = to64(t["lam"])
    for b, n in enumerate(lengths):
        lo, hi = int(cu[b]), int(cu[b + 1])
        if b > 2:
            assert torch.isnan(o[lo:hi].float()).all(), b
            continue
        seq = {name: to64(t[name][lo:hi]).transpose(1, 0, 2)[None] for name in ("q", "k", "v")}
        assert_close("seq %d o" % b, o[lo:hi].permute(1, 0, 2)[None], oracle.fwd_direct(seq["q"], seq["k"], seq["v"], lam64), dtype)


def test_empty_cases_and_validation():
    lam = torch.ones(2, device=DEV)
    x = torch.zeros((0, 2, 64), dtype=torch.bfloat16, device=DEV)
    cu = torch.zeros(1, dtype=torch.int32, device=DEV)          # no sequences
    assert binding.la2_fwd_varlen(x, x, x, lam, cu, 0).shape == x.shape
    cu = torch.zeros(4, dtype=torch.int32, device=DEV)          # three empty sequences
    assert binding.la2_fwd_varlen(x, x, x, lam, cu, 0).shape == x.shape
    y = torch.zeros((10, 2, 64), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(ValueError):
        binding.la2_fwd_varlen(y, y, y, lam, cu.long(), 10)     # cu_seqlens must be int32
    with pytest.raises(ValueError):
        binding.la2_fwd_varlen(y[None], y[None], y[None], lam, cu, 10)   # packed tensors are 3-dimensional
