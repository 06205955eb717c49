"""Which tile height the Actor step takes, asked of the library without a GPU."""
import ctypes as C

import pytest

from paper_2307_12983_amd import binding as B
from paper_2307_12983_amd import workloads as W


def tile_rows(hidden, o, a, num, sac=False):
    fn = B.load_library().pql_internal_act_tile_rows
    fn.restype, fn.argtypes = C.c_int32, [C.POINTER(B.PqlConfig), C.c_int32]
    w = W.WORKLOADS["tiny"].replace(obs_dim=o, act_dim=a, num_envs=37, capacity=37 * 9, hidden=hidden, sac=sac)
    cfg = B.make_config(o, a, w.num_envs, w.capacity, w.nstep, w.gamma, hidden, num, w.rng_seed, stochastic_policy=int(sac))
    return fn(C.byref(cfg), num)


@pytest.mark.parametrize("num,rows", [(8192, 32), (8193, 64), (16384, 64), (16385, 32), (24576, 32), (24577, 64), (32768, 64), (65537, 64)])
def test_wide_policies_count_rounds(num, rows):
    for hidden, o, a in (((512, 256, 128), 108, 21), ((256, 256), 60, 8), ((64, 64), 24, 6)):
        assert tile_rows(hidden, o, a, num) == rows
        if hidden[0] <= 256:
            assert tile_rows(hidden, o, a, num, sac=True) == rows


SMALL = [(8193, 32), (9216, 32), (9217, 64), (16384, 64), (24577, 32), (32768, 64), (40961, 32), (57344, 32)]


@pytest.mark.parametrize("num,rows", SMALL + [(49153, 64), (65537, 64)])
def test_few_actions_keep_32_rows_where_64_are_slower(num, rows):
    for hidden, o, a, sac in (((64, 32), 20, 4, False), ((128, 128), 60, 3, False), ((256, 256), 60, 4, False), ((64, 32), 20, 4, True)):
        assert tile_rows(hidden, o, a, num, sac) == rows


@pytest.mark.parametrize("num,rows", SMALL + [(49153, 32), (65537, 32)])
def test_one_narrow_layer_keeps_32_rows_where_64_are_slower(num, rows):
    for hidden, o, a, sac in (((64,), 20, 4, False), ((64,), 250, 4, False), ((32,), 200, 20, False), ((64,), 250, 4, True)):
        assert tile_rows(hidden, o, a, num, sac) == rows


@pytest.mark.parametrize("hidden,o,rows", [((512, 64, 256), 256, 64), ((512, 64, 256), 224, 64), ((512, 64, 256), 257, 32), ((256, 256), 256, 64),
                                           ((512, 512, 512, 256), 225, 64), ((256, 256), 1024, 32)])
def test_states_alone_decide_not_the_actions_beside_them(hidden, o, rows):
    for a in (5, 16, 32):
        assert tile_rows(hidden, o, a, 8193) == rows
