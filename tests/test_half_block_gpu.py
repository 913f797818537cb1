"""Half-block scans (16-bit data, head_dim 64 / 128) at the ends of chains and chunks.

The waves of a scan share one output tile in LDS: each writes its columns of a block and reads whole rows.  The last block of a
chunk is written into it behind a barrier as every other block is; without one a wave that is still to read the rows of the
block before would store the last block's values in their place."""
import pytest
import torch

import oracle
from paper_2401_04658_amd import binding, workloads
from parity import assert_close, to64

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(autouse=True)
def _defaults():
    yield
    binding.la2_set_chunk_tokens(0)
    binding.la2_set_scan_variant(0)


# chunks of one to four blocks of 32, whole and ragged, and the same as whole chains; states and none
@pytest.mark.parametrize("n,chunk", [(33, 0), (64, 0), (90, 0), (128, 0), (129, 64), (192, 64), (250, 128), (320, 192)])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_last_two_blocks_of_every_chunk(dtype, d, n, chunk):
    """Against the fp64 oracle on four chains among 300 equal ones (more workgroups than compute units, in different places of
    the launch), which all have to give the same bits, three times over: forward, the dQ launch (with a chunk also its accumulating
    wave group), the dK / dV launch, and the forms that take a state at a ragged end."""
    copies = 75
    t = workloads.Workload("ends", 1, 4, n, d, dtype, seed=8100 + n + d, backward=True).tensors()
    gen = torch.Generator(device="cpu")
    gen.manual_seed(8100 + n)
    init, dfin = (torch.randn((1, 4, d, d), generator=gen) * 0.3 for _ in range(2))
    g = {x: y.to(DEV) for x, y in t.items()}
    big = {x: g[x].expand(copies, -1, -1, -1).contiguous() for x in ("q", "k", "v", "d_o")}
    states = {None: (None, None), "given": tuple(x.to(DEV).expand(copies, -1, -1, -1).contiguous() for x in (init, dfin))}
    binding.la2_set_scan_variant(2)
    binding.la2_set_chunk_tokens(chunk)
    q, k, v, do, lam = (to64(t[x]) for x in ("q", "k", "v", "d_o", "lam"))
    for given, (kv0, dkv) in states.items():
        first = None
        for _ in range(3):
            o, kvf = binding.la2_fwd_state(big["q"], big["k"], big["v"], g["lam"], kv_init=kv0, want_final=given is not None)
            grads = binding.la2_bwd_state(big["q"], big["k"], big["v"], big["d_o"], g["lam"], kv_init=kv0, d_kv_final=dkv)
            torch.cuda.synchronize()
            outs = (o,) + tuple(grads) + (() if kvf is None else (kvf,))
            for x in outs:
                assert torch.equal(x, x[:1].expand_as(x))
            first = first or outs
            assert all(torch.equal(x, y) for x, y in zip(outs, first))
        i64, f64 = (None, None) if given is None else (to64(init), to64(dfin))
        refs = (oracle.fwd_recurrent(q, k, v, lam, kv_init=i64),) + tuple(
            oracle.bwd_recurrent_state(q, k, v, do, lam, kv_init=i64, d_kv_final=f64))
        for name, x, ref in zip(("o", "dq", "dk", "dv", "d_kv_init"), first, refs):
            assert_close("%s n%d d%d chunk %d states %s" % (name, n, d, chunk, given), x[:1], ref, dtype)
