"""Decode steps at the sizes where the kernel changes: a chain's state shared by several workgroups on few chains, updated past the
caches from 160 MiB on."""
import pytest
import torch

from paper_2401_04658_amd import binding

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

SIZES = [(64, 10239), (64, 10240), (96, 4551), (96, 4552), (128, 128), (128, 129), (128, 2559), (128, 2560),
         (256, 64), (256, 65), (256, 128), (256, 129), (256, 512), (256, 513), (256, 640)]


@pytest.mark.parametrize("d,chains", SIZES)
@pytest.mark.parametrize("tokens", [1, 5])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
def test_decode_against_the_recurrence_in_64_bits(d, chains, tokens, dtype):
    """First, last and middle chains.  States: a few fp32 roundings per step (16-bit operands of five tokens in one launch: 2^-8
    (fp16: 2^-11) of each product, against the largest state element).  Outputs: one rounding to the type and d fp32 additions;
    with five tokens the operands' roundings as well."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d + chains + tokens)
    shape = (chains, 1, d) if tokens == 1 else (chains, 1, tokens, d)
    q, k, v = ((torch.randn(shape, generator=gen, device=DEV) * d ** -0.5).to(dtype) for _ in range(3))
    kv = torch.randn((chains, 1, d, d), generator=gen, device=DEV) * 0.1
    lam = torch.tensor([0.97], device=DEV)
    rows = torch.tensor([0, 1, chains // 2, chains - 2, chains - 1], device=DEV)
    state = kv[rows, 0].double()
    x = [t[rows, 0].double().reshape(5, tokens, d) for t in (q, k, v)]
    outs = []
    for t in range(tokens):
        state = lam.double() * state + x[1][:, t, :, None] * x[2][:, t, None, :]
        outs.append((x[0][:, t, :, None] * state).sum(1))
    o = (binding.la2_decode_step if tokens == 1 else binding.la2_decode_multi)(q, k, v, lam, kv)
    torch.cuda.synchronize()
    got = o[rows].reshape(5, tokens, d).double()
    ref = torch.stack(outs, 1)
    unit = {torch.bfloat16: 2.0 ** -8, torch.float16: 2.0 ** -11, torch.float32: d * 2.0 ** -23}[dtype]
    blocks = tokens > 1 and dtype != torch.float32
    o_tol = 2 * unit if blocks else unit
    s_tol = unit if blocks else tokens * 2.0 ** -22
    assert (got - ref).abs().max() <= o_tol * ref.abs().max()
    assert (kv[rows, 0].double() - state).abs().max() <= s_tol * state.abs().max()
    assert torch.isfinite(kv).all()


@pytest.mark.parametrize("d,chains", [(64, 10239), (64, 10240), (96, 4551), (96, 4552), (128, 128), (128, 2559), (128, 2560), (256, 128)])
@pytest.mark.parametrize("tokens", [1, 5])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_normalised_decode_against_the_recurrence_in_64_bits(d, chains, tokens, dtype):
    """The same with the Norm (whose columns are never shared).  Its row scale is the root of a mean of squares: no more relative
    error than an output row has in the 2-norm, and an output has its own rounding and the scale's."""
    eps = 1e-4
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d + chains + tokens + 7)
    shape = (chains, 1, d) if tokens == 1 else (chains, 1, tokens, d)
    q, k, v = ((torch.randn(shape, generator=gen, device=DEV) * d ** -0.5).to(dtype) for _ in range(3))
    kv = torch.randn((chains, 1, d, d), generator=gen, device=DEV) * 0.1
    lam = torch.tensor([0.97], device=DEV)
    rows = torch.tensor([0, 1, chains // 2, chains - 2, chains - 1], device=DEV)
    state = kv[rows, 0].double()
    x = [t[rows, 0].double().reshape(5, tokens, d) for t in (q, k, v)]
    outs = []
    for t in range(tokens):
        state = lam.double() * state + x[1][:, t, :, None] * x[2][:, t, None, :]
        outs.append((x[0][:, t, :, None] * state).sum(1))
    u = torch.stack(outs, 1)
    r = (u.pow(2).mean(-1) + eps).rsqrt()
    if tokens == 1:
        o = binding.la2_decode_step_norm(q, k, v, lam, kv, eps)
    else:
        o, rstd = binding.la2_decode_multi_norm(q, k, v, lam, kv, eps)
    torch.cuda.synchronize()
    unit = {torch.bfloat16: 2.0 ** -8, torch.float16: 2.0 ** -11}[dtype]
    ref = u * r[..., None]
    got = o[rows].reshape(5, tokens, d).double()
    assert (got - ref).abs().max() <= (2 if tokens == 1 else 3) * unit * ref.abs().max()
    if tokens > 1:
        assert (rstd[rows].reshape(5, tokens).double() / r - 1).abs().max() <= unit
        assert torch.isfinite(rstd).all()
    assert (kv[rows, 0].double() - state).abs().max() <= (unit if tokens > 1 else 2.0 ** -22) * state.abs().max()
    assert torch.isfinite(kv).all() and torch.isfinite(o.float()).all()
