"""Which kernels the calls take (CPU: launchers that only write down what they are asked for)."""
import pytest

import routes
from paper_2401_04658_amd import binding

DTYPES = [binding.LA2_BF16, binding.LA2_F16]


def work_items(x):
    """Work-items of the launch of all three scans: two workgroups of 4 d threads per chain (or pair) and chunk."""
    units = x["pairs"] * x["heads"] if x["pairs"] else x["batch"] * x["heads"] * x["nchunks"]
    return 2 * units * 4 * x["d"]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("d", [64, 96, 128])
def test_one_launch_stays_below_the_largest_grid(d, dtype):
    """A grid has at most 2^32 - 1 work-items; the launch of all three scans has twice the workgroups of the widest launch otherwise.
    Batches up to the largest that is accepted (2^24 chains), dense and packed, the packed ones almost all of empty sequences."""
    taken = 0
    for chains in (384, 1 << 12, 1 << 20, 5 << 20, 5600000, (1 << 23) - 16, 1 << 23, 11000000, 1 << 24):
        for n in (1, 8, 64, 200):
            x = routes.one_launch(routes.backward(routes.desc(chains // 16, 16, n, d, dtype)))
            taken += x is not None
            assert x is None or work_items(x) < 1 << 32, (chains, n)
            for total in (0, 1000, chains // 16 * n):
                x = routes.one_launch(routes.backward(routes.desc(chains // 16, 16, n, d, dtype, packed=True), total=total))
                taken += x is not None
                assert x is None or work_items(x) < 1 << 32, (chains, n, total)
    assert taken > 0 or d == 128


@pytest.mark.parametrize("dtype", DTYPES)
def test_a_forward_pass_keeps_its_tiles_only_where_it_gains_itself(dtype):
    """Above 96 MiB a tensor a forward pass alone is 2 to 5 % slower with its tiles kept in the caches, at head_dim 64 as at 128."""
    for d, b, n in ((64, 16, 4096), (64, 16, 3300), (64, 64, 1024), (64, 24, 2500), (128, 16, 2048)):
        for x in routes.forward(routes.desc(b, 16, n, d, dtype)):
            assert x["keep"] == 0, (d, b, n)
    for d, b, n in ((64, 16, 3000), (64, 16, 100), (128, 16, 1500)):
        for x in routes.forward(routes.desc(b, 16, n, d, dtype)):
            assert x["launcher"] == "short" or x["keep"] == 1, (d, b, n)


@pytest.mark.parametrize("d,b,h,n", [(96, 16, 16, 900), (96, 7, 32, 855), (128, 16, 16, 900), (256, 8, 16, 189), (64, 16, 16, 8192)])
def test_the_order_of_a_backward_pass_that_is_not_cut(d, b, h, n):
    """dK and dV first where no state is given or wanted, the dQ scan first with any state (measured: la2_api.hip)."""
    A = routes.ADDRESS
    x = routes.desc(b, h, n, d)
    reverse = [y["rev"] for y in routes.backward(x)]
    assert reverse == [1, 0]
    for states in (dict(init=A["kv_init"]), dict(d_final=A["d_kv_final"]), dict(d_init=A["d_kv_init"]),
                   dict(init=A["kv_init"], d_final=A["d_kv_final"], d_init=A["d_kv_init"]), dict(init=A["kv_init"], d_init=A["kv_init"])):
        launches = routes.backward(x, **states)
        assert [y["rev"] for y in launches] == [0, 1], states
        assert launches[0]["w"] == "0x%x" % A["dq"] and launches[0]["nscan"] == 1 and launches[1]["nscan"] == 2
