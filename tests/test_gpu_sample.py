"""pql_sample_nstep where a sample's rows take several passes or divide into no 16-byte granules: rows of one value per lane
and of many passes, 16-byte states with odd actions and the reverse, windows around the four rewards that are read at once,
with and without standardisation, against the CPU oracle (indices and returns' inputs exactly, values to fp32 rounding)."""
import numpy as np
import pytest

from paper_2307_12983_amd import workloads as W

from parity_util import assert_batch_matches, batch_to_numpy, fill_both, oracle_batch, oracle_normalizer, oracle_ring

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("norm", [False, True])
@pytest.mark.parametrize("o,a,nstep", [(1, 1, 1), (13, 17, 4), (64, 31, 5), (211, 20, 8), (257, 32, 9), (603, 3, 3), (1036, 5, 2)])
def test_rows_of_several_passes(o, a, nstep, norm):
    import torch
    from paper_2307_12983_amd.session import LearnerSession
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the gpu-marked tests need a real MI355X")
    w = W.WORKLOADS["tiny"].replace(name="passes", obs_dim=o, act_dim=a, num_envs=37, capacity=37 * 12, batch=129, nstep=nstep,
                                    hidden=(8,), obs_norm=norm, index=91)
    print(o, a, nstep, norm, flush=True)
    s, ring, nz = LearnerSession(w), oracle_ring(w), oracle_normalizer(w) if norm else None
    fill_both(s, ring, w, 15, normalizer=nz)
    for i in range(2):
        s.sample(w.batch)
        assert_batch_matches(batch_to_numpy(s.batch, w.batch), oracle_batch(ring, w, w.batch, i, nz), normalized=norm, ring=ring,
                             normalizer=nz)
