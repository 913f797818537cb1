"""Decode steps on states around the size from which they are updated past the caches (160 MiB): the step on many chains gives
the same bits as the step on a few of them."""
import pytest
import torch

from paper_2401_04658_amd import binding

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("d,chains", [(64, 10239), (64, 10240), (96, 4552), (128, 2559), (128, 2560), (256, 640)])
@pytest.mark.parametrize("tokens", [1, 5])
def test_decode_of_large_states_equals_the_decode_of_a_part(d, chains, tokens):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d + chains + tokens)
    shape = (chains, 1, d) if tokens == 1 else (chains, 1, tokens, d)
    q, k, v = ((torch.randn(shape, generator=gen, device=DEV) * d ** -0.5).bfloat16() for _ in range(3))
    kv = torch.randn((chains, 1, d, d), generator=gen, device=DEV) * 0.1
    lam = torch.tensor([0.97], device=DEV)
    rows = torch.tensor([0, 1, chains // 2, chains - 2, chains - 1], device=DEV)
    few = kv[rows].contiguous()
    step = binding.la2_decode_step if tokens == 1 else binding.la2_decode_multi
    o = step(q, k, v, lam, kv)
    o_few = step(q[rows].contiguous(), k[rows].contiguous(), v[rows].contiguous(), lam, few)
    torch.cuda.synchronize()
    assert torch.equal(o[rows], o_few) and torch.equal(kv[rows], few)
    assert torch.isfinite(kv).all()
