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
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_decode_against_the_recurrence_in_64_bits(d, chains, tokens, dtype):
    """First, last and middle chains.  States: a few fp32 roundings per step (16-bit operands of five tokens in one launch: 2^-8 of
    each product, against the largest state element).  Outputs: one rounding to the type and d fp32 additions; with five tokens
    the operands' roundings as well."""
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
    blocks = tokens > 1 and dtype == torch.bfloat16
    o_tol = 2.0 ** -7 if blocks else 2.0 ** -8 if dtype == torch.bfloat16 else d * 2.0 ** -23
    s_tol = 2.0 ** -8 if blocks else tokens * 2.0 ** -22
    assert (got - ref).abs().max() <= o_tol * ref.abs().max()
    assert (kv[rows, 0].double() - state).abs().max() <= s_tol * state.abs().max()
    assert torch.isfinite(kv).all()
