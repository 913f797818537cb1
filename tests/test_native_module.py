"""The binding's native module: what its checks take and refuse, and how a Python value becomes an entry point's argument (CPU; no
call gets as far as a launch)."""
import threading

import pytest
import torch

from paper_2401_04658_amd import binding

lib = binding._module()


def q4(b=1, h=2, n=5, d=64, dtype=torch.bfloat16):
    return torch.zeros(b, h, n, d, dtype=dtype)


def test_same_layout():
    q = q4()
    assert lib.same_layout(q, q.clone(), torch.empty_like(q)) is None
    view = torch.zeros(1, 5, 2, 64, dtype=torch.bfloat16).permute(0, 2, 1, 3)
    for other in (q4(n=6), q4(dtype=torch.float16), view, torch.zeros(2, 5, 64, dtype=torch.bfloat16), q.to("meta")):
        with pytest.raises(ValueError):
            lib.same_layout(q, other)
    with pytest.raises(TypeError):
        lib.same_layout(q, None)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
def test_new_tensors(dtype):
    x = torch.zeros(3, 7, 2, 80, dtype=dtype)[..., :64].permute(0, 2, 1, 3)
    y = lib.like(x)
    assert y.shape == x.shape and y.stride() == x.stride() and y.dtype == dtype and not y.requires_grad
    assert lib.like(x.float().requires_grad_()).requires_grad is False
    z = lib.f32(x, 3, 2, 64, 64)
    assert z.shape == (3, 2, 64, 64) and z.dtype == torch.float32 and z.is_contiguous()
    assert lib.f32(x, 0, 4).numel() == 0
    with pytest.raises(RuntimeError):
        lib.f32(x, -1)
    with pytest.raises(TypeError):
        lib.f32(x, 1.5)


def test_workspace_is_what_the_query_says():
    for n, op in ((100, 0), (4096, 0), (4096, 1), (4100, 2), (4100, 3)):
        for dtype in (torch.bfloat16, torch.float32):
            q = q4(1, 4, n, 128, dtype)
            need = binding.la2_workspace_bytes(q, op)
            ws = lib.workspace(q, op)
            assert (ws is None and need == 0) or (ws.dtype == torch.uint8 and ws.numel() == need)
    for bad, error in ((torch.zeros(2, 3, 64), ValueError), (q4().transpose(2, 3), ValueError), (q4(dtype=torch.int32), TypeError)):
        with pytest.raises(error):
            lib.workspace(bad, 0)


def test_states():
    q, s = q4(2, 3), torch.zeros(2, 3, 64, 64)
    assert lib.state(None, q, "kv_init") is None and lib.state(s, q, "kv_init") is s
    assert lib.state(torch.zeros(0, 3, 64, 64), q4(0, 3), "kv_init") is None
    packed = torch.zeros(50, 3, 64, dtype=torch.bfloat16)
    assert lib.state(s, packed, "kv_init", 2) is s
    for bad in (s.double(), s[:, :2], s.transpose(2, 3), s.view(2, 3, 4096), s.to("meta"), torch.zeros(2, 3, 32, 64)):
        with pytest.raises(ValueError, match="kv_init"):
            lib.state(bad, q, "kv_init")
    with pytest.raises(ValueError, match="sequences"):
        lib.state(s, packed, "kv_init", 3)


def test_decode_shapes():
    q, kv = torch.zeros(2, 3, 64, dtype=torch.float16), torch.zeros(2, 3, 64, 64)
    assert lib.decode_shape("f", 3, q, q, q, kv) == (2, 3, 64, binding.LA2_F16)
    t = torch.zeros(2, 3, 5, 64)
    assert lib.decode_shape("f", 4, t, t, t, kv) == (2, 3, 5, 64, binding.LA2_F32)
    for args in ((3, q, q, q.float(), kv), (3, q, q[:, :2], q, kv), (3, q, q, q, kv.transpose(2, 3)), (3, q, q, q, kv.half()),
                 (3, t, t, t, kv), (4, q, q, q, kv), (3, q, q, q, kv[:1])):
        with pytest.raises(ValueError, match="f: "):
            lib.decode_shape("f", *args)
    with pytest.raises(TypeError):
        lib.decode_shape("f", 3, q.int(), q.int(), q.int(), kv)


def test_arguments_and_statuses():
    """Statuses of refused calls come back as numbers; a descriptor is a tensor or a la2_desc; a pointer a tensor, None or a number."""
    q = q4(n=64)
    assert lib.la2_fwd(q, None, q, q, q, q, None, None, 0) == 1                      # LA2_ERR_NULL
    assert lib.la2_fwd(binding.make_desc(q), None, q, q, q, q, None, 0, 0) == 1
    assert lib.la2_fwd(q, 1 << 40, (1 << 40) + 8, 1 << 40, 1 << 40, 1 << 40, None, 0, 0) == 4   # alignment, nothing is read
    assert lib.la2_fwd(q4(n=0), None, None, None, None, None, None, None, None) == 0           # nothing to do
    assert lib.la2_decode_step(1, 2, 65, binding.LA2_BF16, q, q, q, q, q, q, 0) == 2   # LA2_ERR_SHAPE
    for args, error in (((q,), TypeError), ((q, "x", q, q, q, q, None, 0, 0), TypeError), ((b"short", q, q, q, q, q, None, 0, 0), ValueError),
                        ((q, q, q, q, q, q, None, -1, 0), OverflowError), ((3, q, q, q, q, q, None, 0, 0), TypeError)):
        with pytest.raises(error):
            lib.la2_fwd(*args)
    with pytest.raises(OverflowError):
        lib.la2_decode_step(1 << 33, 2, 64, 1, q, q, q, q, q, q, 0)
    with pytest.raises(RuntimeError):   # a tensor without storage of its own: torch's error, not a null pointer
        torch.vmap(lambda x: lib.la2_fwd(q, x, q, q, q, q, None, 0, 0) or x)(torch.zeros(2, 1, 2, 64, 64))
    with pytest.raises(ValueError):
        binding.la2_fwd(q, q, q, torch.ones(2))   # not on the GPU


def test_calls_from_several_threads():
    q, bad = q4(n=64), []

    def work():
        for _ in range(2000):
            if lib.la2_fwd(q, None, q, q, q, q, None, None, 0) != 1 or lib.like(q).shape != q.shape:
                bad.append(1)

    threads = [threading.Thread(target=work) for _ in range(4)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not bad


PUBLIC = {   # name: (sequence tensors in front of lam or kv_state, arguments that the caller may give as a tensor or leave out)
    "la2_fwd": ("q k v lam", ("workspace",)), "la2_fwd_noalloc": ("q k v lam out", ()), "la2_bwd": ("q k v o lam", ("workspace",)),
    "la2_fwd_norm": ("q k v lam", ("workspace",)), "la2_bwd_norm": ("q k v o rstd o lam", ("workspace",)),
    "la2_fwd_state": ("q k v lam", ("workspace",)), "la2_bwd_state": ("q k v o lam", ("workspace", "fwd_workspace")),
    "la2_fwd_state_norm": ("q k v lam", ("workspace",)), "la2_bwd_state_norm": ("q k v o rstd o lam", ("workspace",)),
    "la2_decode_step": ("dq dq dq lam kv", ("out",)), "la2_decode_step_norm": ("dq dq dq lam kv", ("out",)),
    "la2_decode_multi": ("q q q lam kv", ("out",)), "la2_decode_multi_norm": ("q q q lam kv", ("out", "rstd")),
    "la2_left_product_fwd": ("q k v lam", ()), "la2_left_product_bwd": ("q k v o lam", ()),
}


@pytest.mark.parametrize("name", sorted(PUBLIC))
def test_a_number_never_becomes_an_address(name, monkeypatch):
    """Every pointer that a caller of the Python functions hands over has to be a tensor: a number (or a truth value) is refused before
    the call."""
    reached = []
    monkeypatch.setattr(binding, "_on_gpu", lambda t, what: None)
    monkeypatch.setattr(binding, "_run", lambda entry, t, *args: reached.append(args))
    have = {x: q4(2, 3) for x in ("q", "k", "v", "o", "out")}
    have.update(lam=torch.ones(3), rstd=torch.ones(2, 3, 5), dq=torch.zeros(2, 3, 64), kv=torch.zeros(2, 3, 64, 64))
    front, optional = PUBLIC[name]
    args = [have[x] for x in front.split()]
    fn = getattr(binding, name)
    fn(*args)
    assert len(reached) == 1
    for x in optional:   # a tensor is taken
        fn(*args, **{x: torch.empty(64, dtype=torch.uint8)})
    assert len(reached) == 1 + len(optional)
    del reached[:]
    at = front.split().index("lam")
    for bad in (4096, True, 1.0, "x"):
        with pytest.raises(TypeError):
            fn(*args[:at], bad, *args[at + 1:])
        for x in optional:
            with pytest.raises(TypeError):
                fn(*args, **{x: bad})
    with pytest.raises(TypeError):
        fn(*args[:at], None, *args[at + 1:])
    assert not reached


def test_a_packed_call_takes_no_number_either(monkeypatch):
    reached = []
    monkeypatch.setattr(binding, "_on_gpu", lambda t, what: None)
    monkeypatch.setattr(binding, "_run", lambda entry, t, *args: reached.append(args))
    monkeypatch.setattr(binding, "_varlen_desc", lambda q, cu, longest: binding.la2_desc(2, 3, 30, 64, binding.LA2_BF16, 0, 0, 64, 192))
    x, cu, rstd = torch.zeros(50, 3, 64, dtype=torch.bfloat16), torch.tensor([0, 20, 50], dtype=torch.int32), torch.ones(3, 50)
    for name, front in (("la2_fwd_varlen", (x,) * 3), ("la2_bwd_varlen", (x,) * 4), ("la2_fwd_varlen_state", (x,) * 3),
                        ("la2_bwd_varlen_state", (x,) * 4), ("la2_fwd_varlen_norm", (x,) * 3),
                        ("la2_bwd_varlen_norm", (x, x, x, x, rstd, x))):
        fn = getattr(binding, name)
        fn(*front, torch.ones(3), cu, 30)
        assert len(reached) == 1, name
        del reached[:]
        for bad in (4096, True, None):
            with pytest.raises(TypeError):
                fn(*front, bad, cu, 30)
        with pytest.raises(TypeError):
            fn(*front, torch.ones(3), cu, 30, workspace=4096)
        assert not reached, name


def test_eps_is_what_float_takes():
    q = q4(n=64)
    for eps in (1e-6, 0, "1e-6", torch.tensor(1e-6)):
        assert lib.la2_fwd_norm(q, None, q, q, q, eps, q, q, None, 0, 0) == 1   # LA2_ERR_NULL: eps was taken
    assert lib.la2_fwd_norm(q, q, q, q, q, -1, q, q, None, 0, 0) == 7            # LA2_ERR_VALUE
    for eps, error in ((None, TypeError), ("x", ValueError), ([], TypeError)):
        with pytest.raises(error):
            lib.la2_fwd_norm(q, None, q, q, q, eps, q, q, None, 0, 0)


def test_the_module_is_refused_by_a_torch_that_it_was_not_built_for(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_native", None)
    assert binding._module().built_for[2] == torch.__version__
    monkeypatch.setattr(binding, "_native", None)
    monkeypatch.setattr(torch, "__version__", "1.0.0")
    with pytest.raises(ImportError, match="built for .* not for .* torch 1.0.0; build it again"):
        binding._module()
    assert binding._native is None
    monkeypatch.undo()
    monkeypatch.setattr(binding, "_native", None)
    broken = tmp_path / "_la2_native.so"
    broken.write_bytes(b"not a library")
    monkeypatch.setattr(binding, "_NATIVE_PATH", str(broken))
    with pytest.raises(ImportError, match="does not load with .* build it with them"):
        binding._module()
