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


@pytest.mark.parametrize("d,b,h,n", [(96, 16, 16, 900), (96, 7, 32, 855), (128, 16, 16, 900), (256, 8, 16, 289), (64, 16, 16, 8192)])
def test_the_order_of_a_backward_pass_that_is_not_cut(d, b, h, n):
    """dK and dV first on at most one chain per unit and above 16 MiB a tensor where no state is given or wanted, else the dQ scan first
    (measured: la2_api.hip)."""
    A = routes.ADDRESS
    x = routes.desc(b, h, n, d)
    reverse = [y["rev"] for y in routes.backward(x)]
    assert reverse == [1, 0]
    for states in (dict(init=A["kv_init"]), dict(d_final=A["d_kv_final"]), dict(d_init=A["d_kv_init"]),
                   dict(init=A["kv_init"], d_final=A["d_kv_final"], d_init=A["d_kv_init"]), dict(init=A["kv_init"], d_init=A["kv_init"])):
        launches = routes.backward(x, **states)
        assert [y["rev"] for y in launches] == [0, 1], states
        assert launches[0]["w"] == "0x%x" % A["dq"] and launches[0]["nscan"] == 1 and launches[1]["nscan"] == 2
    few = routes.backward(routes.desc(b, h, (16 << 20) // (2 * b * h * d), d))   # (at head_dim 64 one launch)
    assert routes.one_launch(few) is not None or [y["rev"] for y in few] == [0, 1]
    more = routes.backward(routes.desc(4096 // h, h, 160, d))   # (at head_dim 96 one launch)
    assert routes.one_launch(more) is not None or [y["rev"] for y in more] == [0, 1]


# chains, positions, one launch; either side of every line for many chains
LINES = {64: [(768, 32, True), (784, 32, False), (784, 33, True), (896, 64, True), (912, 64, False), (912, 191, False), (912, 192, True),
              (1024, 128, False), (1024, 300, True), (1040, 63, False), (1040, 64, True), (1792, 64, True), (1808, 300, False), (2048, 32, False),
              (8192, 64, False), (16384, 32, False), (272, 32, True), (512, 400, True)],
         96: [(272, 8, True), (640, 8, True), (656, 159, False), (656, 160, True), (1024, 64, False), (1040, 64, True), (1152, 64, True), (1168, 127, False), (1168, 128, True),
              (4096, 64, False), (4096, 128, True), (16384, 32, False), (16384, 128, True), (160, 8, True), (176, 8, False), (256, 300, False)],
         128: [(160, 2300, True), (160, 2500, False), (128, 5000, True), (176, 300, False), (192, 300, True), (192, 199, False), (256, 134, False),
               (272, 33, True), (336, 90, True), (640, 64, False), (640, 65, True), (448, 300, False), (768, 300, False)]}


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("d,chains,n,one", [(d, *x) for d in LINES for x in LINES[d]])
def test_one_launch_of_many_short_chains(d, chains, n, one, dtype):
    launchers = [x["launcher"] for x in routes.backward(routes.desc(chains // 16, 16, n, d, dtype))]
    if launchers != ["short"]:   # (up to two chains per unit the short path comes first)
        assert any(x in ("bwd_scans_bf16", "bwd_scans_wide") for x in launchers) == one, launchers


@pytest.mark.parametrize("d,sequences,average,longest,one", [(64, 48, 100, 160, True), (64, 230, 47, 90, False), (64, 64, 80, 120, False), (64, 70, 80, 120, True),
                                                             (64, 110, 80, 120, True), (64, 128, 80, 120, False), (64, 700, 51, 90, False), (96, 96, 30, 60, True),
                                                             (96, 98, 95, 180, False), (96, 98, 96, 180, True), (96, 700, 46, 90, False)])
def test_one_launch_of_many_packed_sequences(d, sequences, average, longest, one):
    """As for dense batches, by the average length."""
    x = routes.desc(sequences, 16, longest, d, packed=True)
    assert (routes.one_launch(routes.backward(x, total=sequences * average)) is not None) == one


def test_the_one_launch_starts_where_the_short_path_ends():
    """head_dim 128, 64 chains without states: the one launch's line (704 positions) is where the short path's own line lies."""
    for n in (300, 640, 704):
        assert [x["launcher"] for x in routes.backward(routes.desc(4, 16, n, 128))] == ["short"], n
    for n in (705, 768, 1152):
        assert routes.one_launch(routes.backward(routes.desc(4, 16, n, 128))) is not None, n


# what test_joint_backward_gpu.py runs: chunks of the one launch (None: another path) without states, with all of them, and both again from
# the forward call's workspace
JOINT = {(64, 1, 4, 2113): (None, 9, None, 9), (64, 1, 16, 2048): (8, 8, 8, 8), (64, 3, 16, 1000): (4, 4, 4, 4), (64, 6, 16, 1100): (1, 1, 1, 1),
         (64, 8, 16, 1031): (1, 1, 1, 1), (64, 10, 16, 200): (1, 1, 1, 1), (64, 16, 16, 257): (1, 1, 1, 1), (64, 18, 16, 130): (1, 1, 1, 1),
         (128, 5, 16, 416): (1, 1, 1, 1), (128, 3, 16, 1000): (1, 1, None, None), (96, 3, 2, 300): (1, 1, 1, 1), (96, 3, 16, 1000): (1, 1, None, None),
         (96, 5, 16, 1100): (1, 1, None, None), (96, 17, 16, 97): (1, 1, 1, 1), (96, 1, 16, 2050): (None,) * 4, (96, 1, 4, 2050): (None, None, 9, 9),
         (128, 6, 16, 1056): (1, 1, None, None), (128, 10, 16, 100): (1, 1, 1, 1), (128, 16, 16, 65): (None,) * 4, (128, 13, 16, 225): (1, 1, 1, 1), (128, 18, 16, 127): (1, 1, 1, 1),
         (128, 19, 16, 2049): (1, 1, 1, 1), (96, 17, 16, 2053): (1, 1, 1, 1), (64, 19, 16, 2055): (1, 1, 1, 1)}
# (chunks, pairs of the map: 0 none) of its packed batches
PACKED = [(10, 20), (4, 25), (1, 0), (1, 0), (1, 0), (1, 0)]


@pytest.mark.parametrize("dtype", DTYPES)
def test_the_gpu_test_of_the_one_launch_reaches_it(dtype):
    import test_joint_backward_gpu as gpu
    A = routes.ADDRESS
    states = dict(init=A["kv_init"], d_final=A["d_kv_final"], d_init=A["d_kv_init"])
    shapes = [m.args[1] for m in gpu.test_all_scans_in_one_launch.pytestmark if m.args and m.args[0] == "d,b,h,n"][0]
    assert set(shapes) == set(JOINT)
    for (d, b, h, n), want in JOINT.items():
        x = routes.desc(b, h, n, d, dtype)
        got = [routes.one_launch(routes.backward(x, saved=saved, **st)) for saved in (False, True) for st in ({}, states)]
        assert tuple(y and y["nchunks"] for y in got) == want, (d, b, h, n)
        # d_kv_init in kv_init's place: the dQ scan has read it by then, in a launch of its own
        in_place = routes.backward(x, init=A["kv_init"], d_final=A["d_kv_final"], d_init=A["kv_init"])
        assert routes.one_launch(in_place) is None
    for (d, h, lengths), want in zip(gpu.PACKED, PACKED):
        x = routes.desc(len(lengths), h, max(lengths), d, dtype, packed=True)
        for st in ({}, states) if d != 96 else ({},):
            y = routes.one_launch(routes.backward(x, total=sum(lengths), **st))
            assert (y["nchunks"], y["pairs"]) == want, (d, h, lengths)
        if d != 96:
            assert routes.one_launch(routes.backward(x, total=sum(lengths), init=A["kv_init"], d_final=A["d_kv_final"], d_init=A["kv_init"])) is None


@pytest.mark.parametrize("d,b,h,n,pair", [(64, 1, 4, 1000, True), (64, 2, 8, 6000, True), (64, 3, 1, 39661, False), (64, 3, 8, 12000, False), (64, 1, 6, 40000, False),
                                          (128, 4, 16, 2048, True), (128, 3, 8, 6000, True)])
def test_fp32_chunk_states_in_one_launch(d, b, h, n, pair):
    """Up to 24 MiB a tensor at head_dim 64 (measured: la2_api.hip); never with rows apart, from saved states, or behind a ragged end."""
    x = routes.desc(b, h, n, d, binding.LA2_F32)
    assert any(y["launcher"] == "chunk_state_pair_f32" for y in routes.backward(x)) == pair
    assert not any(y["launcher"] == "chunk_state_pair_f32" for y in routes.backward(x, saved=True))
    apart = binding.la2_desc(b, h, n, d, binding.LA2_F32, 0, h * n * (d + 16), n * (d + 16), d + 16)
    assert not any(y["launcher"] == "chunk_state_pair_f32" for y in routes.backward(apart))
    if pair:
        first, second = [y for y in routes.backward(x) if y["launcher"] in ("chunk_state_pair_f32", "+rev")]
        assert first["states"] == "0x%x" % routes.ADDRESS["dv"] and second["states"] == "0x%x" % routes.ADDRESS["ws"]


@pytest.mark.parametrize("dtype", DTYPES)
def test_one_launch_in_chunks_at_head_dim_64(dtype):
    """By the bytes of a tensor: up to 22 MiB, from saved states 16 (48 chains and more) or 8."""
    for b, h, n, fresh, saved in ((3, 20, 2900, True, False), (3, 20, 3100, False, False), (1, 16, 8001, True, False), (2, 12, 8161, False, False),
                                  (3, 20, 31455, False, False), (2, 2, 53997, False, False), (4, 16, 2048, True, True), (3, 16, 1300, True, True),
                                  (1, 12, 5000, True, True), (1, 12, 6000, True, False)):
        x = routes.desc(b, h, n, 64, dtype)
        assert (routes.one_launch(routes.backward(x)) is not None) == fresh, (b, h, n)
        assert (routes.one_launch(routes.backward(x, saved=True)) is not None) == saved, (b, h, n)
