"""The row-tile kernels on fp16 pairs (pql_split.hip) at the sizes where they can go wrong: widths that fill no tile, inputs
of more than 256 columns (brought in twice), an input tile that shares its place with the activations, layers above 512
(critics one after the other), one hidden layer, last row tiles of one row, and values far from 1, against the CPU oracle.

Tolerances: a product of fp16 pairs is off by at most 3 * 2^-22 of |x| |w|, so a layer by 7e-7 of its largest term sum, and
the fp32 sums behind it are those of the other kernels: gradients and losses within 1e-5 of a tensor's largest value
(measured below 4e-6) instead of the 1e-4 that holds everywhere."""
import numpy as np
import pytest

from oracle import pql_oracle as O
from paper_2307_12983_amd import workloads as W

from parity_util import assert_params_close, fill_both, oracle_batch, oracle_learner, oracle_ring, rel_err

pytestmark = pytest.mark.gpu
TOL = 1e-5


def session(w):
    import torch
    from paper_2307_12983_amd.session import LearnerSession
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the gpu-marked tests need a real MI355X")
    return LearnerSession(w)


def workload(hidden, o, a, batch, **kw):
    return W.WORKLOADS["tiny"].replace(name="split", obs_dim=o, act_dim=a, num_envs=37, capacity=37 * 9, batch=batch,
                                       hidden=hidden, index=90, **kw)


CASES = {
    "single_two_pass_input": workload((1024, 40), 230, 32, 2049),
    "widest_input": workload((200, 40), 1024, 32, 65),                  # 1056 columns: 33 k-steps
    "pair_shared_input_tile": workload((512, 512), 250, 10, 2050),
    "pair_two_tiles_odd": workload((300, 136, 24), 33, 1, 65),
    "odd_widths_sac": workload((100, 200), 45, 11, 31, sac=True),
    "one_layer_sac": workload((40,), 7, 3, 33, sac=True),
    "one_layer_single": workload((1024,), 20, 4, 97),                   # no barrier but the heads' own between the two critics
    "one_layer_single_sac": workload((640,), 20, 4, 2049, sac=True),
    "one_layer_atoms": workload((24,), 7, 3, 33, num_atoms=51),
    "few_atoms_wide": workload((512, 72), 19, 5, 97, num_atoms=11, v_min=-2.0, v_max=3.0),
    "deep": workload((40, 72, 100, 24, 200, 8, 64, 33), 5, 2, 64),
}


@pytest.mark.parametrize("case", list(CASES))
def test_gradients_at_the_edges(case):
    w = CASES[case]
    print(case, w.hidden, "B", w.batch, flush=True)
    s, ring = session(w), oracle_ring(w)
    fill_both(s, ring, w, w.nstep + 3)
    L = oracle_learner(w, s.actor_init, s.critic_init)
    s.sample(w.batch)
    batch = oracle_batch(ring, w, w.batch, 0, None)
    s.ctx.pql_profile_begin(64)
    s.critic_update(w.batch)
    losses, g = L.critic_update(batch)
    s.actor_update(None, w.batch)
    names = {k["name"] for k in s.ctx.pql_profile_end()}
    assert {"split_weights_kernel", "split_critic_kernel", "split_policy_kernel"} <= names
    _, ga = L.actor_update(batch["obs"])
    assert rel_err(s.critic_loss.cpu().numpy(), losses) <= TOL
    e = assert_params_close(s.c_g.cpu().numpy(), g, w.critic_dims(), 2, TOL, "critic grad")
    ea = assert_params_close(s.a_g.cpu().numpy(), ga, w.actor_dims(), 1, TOL, "actor grad")
    print(case, "critic grad", e, "actor grad", ea, flush=True)


LAYERS = {          # what the layer kernel's tiles and loads depend on: 64 / 32 rows, rows of more than 1024 columns, segments
    "tiles_of_64_and_32_rows": workload((640, 150), 30, 5, 8225),
    "rows_brought_in_twice": workload((1156, 204, 130), 33, 4, 4161),
    "wide_odd_input": workload((136, 128), 603, 17, 8193),
    "scales_of_65_tiles": workload((2080, 64), 20, 3, 8192),          # one column tile more than 64
    "scales_of_128_tiles": workload((128, 4096, 128), 20, 3, 4100),   # both directions: the second layer's transpose has 4096 rows
    "matrix_on_the_tiled_kernel": workload((1312, 128), 20, 3, 8192),
}


@pytest.mark.parametrize("case", list(LAYERS))
def test_layers_at_the_edges(case):
    w = LAYERS[case]
    print(case, w.hidden, "B", w.batch, flush=True)
    s, ring = session(w), oracle_ring(w)
    fill_both(s, ring, w, w.nstep + 3)
    L = oracle_learner(w, s.actor_init, s.critic_init)
    s.sample(w.batch)
    batch = oracle_batch(ring, w, w.batch, 0, None)
    s.ctx.pql_profile_begin(200)
    s.critic_update(w.batch)
    losses, g = L.critic_update(batch)
    s.actor_update(None, w.batch)
    names = {k["name"] for k in s.ctx.pql_profile_end()}
    assert "layer_rowtile_kernel" in names and not {n for n in names if n.startswith(("split_critic", "split_policy"))}
    _, ga = L.actor_update(batch["obs"])
    assert rel_err(s.critic_loss.cpu().numpy(), losses) <= TOL
    e = assert_params_close(s.c_g.cpu().numpy(), g, w.critic_dims(), 2, TOL, "critic grad")
    ea = assert_params_close(s.a_g.cpu().numpy(), ga, w.actor_dims(), 1, TOL, "actor grad")
    print(case, "critic grad", e, "actor grad", ea, flush=True)


@pytest.mark.parametrize("hidden", [(256, 256), (512, 96), (40, 100)])
def test_rows_and_weights_of_very_different_size(hidden):
    """Every row of a batch has its own scale, every 32 columns of a matrix theirs: states between 1e-2 and 1e6 in one batch,
    layers scaled by 1e3 and 1e-4, Q row by row to 1e-5 of the row's own value; a row of NaN and one of infinity stay alone."""
    import torch
    from test_gpu_parity import workspace_rows
    w = workload(hidden, 20, 4, 96)
    s = session(w)
    rng = np.random.default_rng(3)
    c = s.critic_init.astype(np.float64)
    dims = w.critic_dims()
    half, off = c.size // 2, 0
    for l, (i, o) in enumerate(dims):
        for h in (0, half):
            c[h + off:h + off + i * o] *= (1e3, 1e-4, 1.0)[l % 3]
        off += i * o + o
    c = c.astype(np.float32)
    B = w.batch
    scale = 10.0 ** (np.arange(B) % 9 - 2)
    obs = (rng.standard_normal((B, w.obs_dim)) * scale[:, None]).astype(np.float32)
    act = rng.uniform(-1, 1, (B, w.act_dim)).astype(np.float32)

    def run(obs):
        s.critic.copy_(torch.from_numpy(c))
        s.critic_target.copy_(torch.from_numpy(c))
        s.batch.obs[:B].copy_(torch.from_numpy(obs))
        s.batch.next_obs[:B].copy_(torch.from_numpy(obs))
        s.batch.act[:B].copy_(torch.from_numpy(act))
        s.batch.ret[:B].zero_()
        s.batch.boot[:B].zero_()
        s.critic_update(B)
        return [workspace_rows(s, 1 + i, B) for i in (0, 1)]

    q = run(obs)
    for i, p in enumerate(O.split_twin(c)):
        ref = O.critic_forward(p, dims, obs, act)
        err = np.abs(q[i] - ref) / np.maximum(np.abs(ref), np.abs(ref).min())
        print(hidden, "critic", i, "worst row", int(err.argmax()), "%.2e" % err.max(), flush=True)
        assert err.max() <= 10 * TOL         # (a row's Q can cancel to a tenth of its terms)
    bad = obs.copy()
    bad[5], bad[40] = np.nan, np.inf
    others = np.setdiff1d(np.arange(B), [5, 40])
    for x, y in zip(run(bad), q):
        assert np.isnan(x[5]) and not np.isfinite(x[40])
        assert np.array_equal(x[others], y[others])


@pytest.mark.parametrize("batch,hidden", [(40, (64, 64)), (333, (96, 40)), (8192, (256, 256))])
def test_weight_gradients_of_columns_that_grow_and_differ(batch, hidden):
    """The weight-gradient kernel's column scales come from a column's first rows: states that grow by 1e7 over the batch
    (the sums are rescaled on the way), columns in units from 1e-3 to 1e4, a column of zeros, one that starts with zeros.
    Every row of dW_1 (one state column) to 1e-5 of its own largest entry, against float64 on the deltas of the oracle."""
    import torch
    w = workload(hidden, 21, 3, batch)
    s, ring = session(w), oracle_ring(w)
    fill_both(s, ring, w, w.nstep + 3)
    s.sample(batch)
    rng = np.random.default_rng(5)
    b = {k: getattr(s.batch, k)[:batch].cpu().numpy().copy() for k in ("obs", "act", "ret", "next_obs", "boot")}
    b["obs"] = (rng.standard_normal((batch, w.obs_dim)) * 10.0 ** (7.0 * np.arange(batch) / batch - 5)[:, None]
                * 10.0 ** (np.arange(w.obs_dim) % 8 - 3)).astype(np.float32)
    b["obs"][:, 4] = 0.0
    b["obs"][:batch // 2, 8] = 0.0
    b["boot"][:] = 0.0
    for k in ("obs", "boot"):
        getattr(s.batch, k)[:batch].copy_(torch.from_numpy(b[k]))
    # small first-layer weights: the hidden layers stay of order 1
    c = s.critic_init.copy()
    for h in (0, c.size // 2):
        c[h:h + w.obs_dim * hidden[0]] *= (1e-3 / np.repeat(10.0 ** (np.arange(w.obs_dim) % 8 - 3), hidden[0])).astype(np.float32)
    s.critic.copy_(torch.from_numpy(c))
    s.critic_update(batch)
    y = b["ret"].astype(np.float64)
    _, g = O.critic_loss_and_grads(c, w.critic_dims(), b, y)
    got, n = s.c_g.cpu().numpy().astype(np.float64), w.obs_dim * hidden[0]
    for h in (0, c.size // 2):
        ref, x = g[h:h + n].reshape(w.obs_dim, -1), got[h:h + n].reshape(w.obs_dim, -1)
        assert np.all(x[4] == 0.0)
        err = np.abs(x - ref).max(1) / np.maximum(np.abs(ref).max(1), 1e-300)
        err[4] = 0.0
        print(batch, hidden, "worst column", int(err.argmax()), "%.2e" % err.max(), flush=True)
        assert err.max() <= TOL


@pytest.mark.parametrize("hidden", [(24,), (512, 512)])
def test_clipped_step_inside_the_ball_is_the_plain_step(hidden):
    """adam_clip_kernel with one workgroup per 256 parameters and with several elements per thread (above 2^18 parameters):
    a bound that no gradient reaches changes nothing, and the norm is the gradient's."""
    import torch
    w = workload(hidden, 20, 4, 64)
    got = []
    for bound in (0.0, 1e6):
        s = session(w.replace(max_grad_norm=bound))
        fill_both(s, oracle_ring(w), w, w.nstep + 3)
        s.sample(w.batch)
        s.critic_update(w.batch)
        got.append([x.cpu().numpy() for x in (s.critic, s.c_m, s.c_v, s.c_g)] + [float(s.critic_grad_norm.cpu()[0])])
    for a, b in zip(got[0][:4], got[1][:4]):
        assert np.abs(a - b).max() <= 2e-7 * np.abs(a).max()
    norm = np.sqrt((got[1][3].astype(np.float64) ** 2).sum())
    assert abs(got[1][4] - norm) <= 1e-6 * norm
    print(hidden, "parameters", got[0][0].size, "norm", norm, flush=True)


@pytest.mark.parametrize("batch,hidden", [(40, (64, 64)), (333, (96, 40)), (8192, (256, 256))])
def test_weight_gradients_of_tiny_columns(batch, hidden):
    """State columns far below 1 beside deltas far below 1: the powers of two by which the sums are rescaled multiply to more
    than fp32 holds (1e-29 and deltas of 1e-7: 2^(7 + 96) times 2^(7 + 23)) while the sums are zero or ordinary.  A column of
    1e-29 throughout, one of subnormals, one that is tiny in the first half and ordinary after it: finite everywhere, every row
    of dW_1 to 1e-5 of its own largest entry (subnormals: to the spacing of fp32 results near zero, 2^-149 a term)."""
    import torch
    w = workload(hidden, 21, 3, batch)
    s, ring = session(w), oracle_ring(w)
    fill_both(s, ring, w, w.nstep + 3)
    s.sample(batch)
    rng = np.random.default_rng(6)
    b = {k: getattr(s.batch, k)[:batch].cpu().numpy().copy() for k in ("obs", "act", "ret", "next_obs", "boot")}
    b["obs"] = rng.standard_normal((batch, w.obs_dim)).astype(np.float32)
    b["obs"][:, 4] *= np.float32(1e-29)
    b["obs"][:, 8] = (b["obs"][:, 8].astype(np.float64) * 1e-40).astype(np.float32)
    b["obs"][:batch // 2, 9] *= np.float32(1e-33)
    b["boot"][:] = 0.0
    b["ret"] = (b["ret"] * np.float32(1e-3)).astype(np.float32)
    for k in ("obs", "ret", "boot"):
        getattr(s.batch, k)[:batch].copy_(torch.from_numpy(b[k]))
    c = s.critic_init.copy()
    dims = w.critic_dims()
    out = sum(i * o + o for i, o in dims[:-1])
    for h in (0, c.size // 2):
        c[h + out:h + c.size // 2] *= np.float32(0.1)             # small output weights: small deltas
    s.critic.copy_(torch.from_numpy(c))
    s.critic_update(batch)
    _, g = O.critic_loss_and_grads(c, dims, b, b["ret"].astype(np.float64))
    got, n = s.c_g.cpu().numpy().astype(np.float64), w.obs_dim * hidden[0]
    assert np.isfinite(got).all()
    for h in (0, c.size // 2):
        ref, x = g[h:h + n].reshape(w.obs_dim, -1), got[h:h + n].reshape(w.obs_dim, -1)
        assert np.abs(x[8] - ref[8]).max() <= batch * 2.0 ** -149
        err = np.abs(x - ref).max(1) / np.abs(ref).max(1)
        err[8] = 0.0
        print(batch, hidden, "worst column", int(err.argmax()), "%.2e" % err.max(), flush=True)
        assert err.max() <= TOL


INFINITE = {        # widths, batch: one launch per update (two classes, critics one after the other), one launch per layer
    "fused": ((64, 64), 65),
    "pair": ((300, 136, 24), 97),
    "single": ((640, 40), 65),
    "layers": ((640, 150), 8225),
}


@pytest.mark.parametrize("case", list(INFINITE))
def test_infinite_weight_stays_in_its_column(case):
    """A weight of -inf on a state column that is positive throughout: its hidden unit is ELU(-inf) = -1 with slope 0 in every
    row, as in any arithmetic, and the other 31 columns that share a scale with it are what they are without it."""
    import torch
    hidden, batch = INFINITE[case]
    w = workload(hidden, 20, 4, batch)
    s, ring = session(w), oracle_ring(w)
    fill_both(s, ring, w, w.nstep + 3)
    s.sample(batch)
    s.batch.obs[:batch, 3].abs_().add_(0.1)
    b = {k: getattr(s.batch, k)[:batch].cpu().numpy().copy() for k in ("obs", "act", "ret", "next_obs", "boot")}
    c = s.critic_init.copy()
    for h, unit in ((0, 5), (c.size // 2, hidden[0] - 1)):
        c[h + 3 * hidden[0] + unit] = -np.inf
    s.critic.copy_(torch.from_numpy(c))
    # the targets stay finite
    L = oracle_learner(w, s.actor_init, s.critic_init)
    L.critic = c.astype(np.float64)
    s.critic_update(batch)
    losses, g = L.critic_update(b)
    s.critic.copy_(torch.from_numpy(c))
    L.critic = c.astype(np.float64)
    s.actor_update(s.batch.obs, batch)
    _, ga = L.actor_update(b["obs"])
    assert np.isfinite(g).all() and np.isfinite(ga).all()
    assert rel_err(s.critic_loss.cpu().numpy(), losses) <= TOL
    e = assert_params_close(s.c_g.cpu().numpy(), g, w.critic_dims(), 2, TOL, "critic grad")
    ea = assert_params_close(s.a_g.cpu().numpy(), ga, w.actor_dims(), 1, TOL, "actor grad")
    print(case, "critic grad", e, "actor grad", ea, flush=True)


@pytest.mark.parametrize("hidden", [(64, 64), (512, 256)])
def test_infinite_output_weights_give_saturated_actions(hidden):
    """The Actor step above 4096 environments: an action with an infinite output weight is +1 or -1 by the sign of its hidden
    unit, the others are the oracle's."""
    import torch
    w = workload(hidden, 20, 4, 4128).replace(num_envs=4128, capacity=4128 * 4, sigma_min=0.0, sigma_max=0.0)
    s = session(w)
    p = s.actor_init.copy()
    dims = w.actor_dims()
    out = sum(i * o + o for i, o in dims[:-1])
    p[out + 7 * 4 + 2] = np.inf
    s.actor.copy_(torch.from_numpy(p))
    obs = np.random.default_rng(8).standard_normal((4128, 20)).astype(np.float32)
    got = s.act(torch.from_numpy(obs).cuda()).cpu().numpy()
    finite = s.actor_init.astype(np.float64)
    ref = O.actor_forward(finite, dims, obs.astype(np.float64))
    others = [0, 1, 3]
    assert np.abs(got[:, others] - ref[:, others]).max() <= TOL
    x = obs.astype(np.float64)
    for l, (i, o) in enumerate(dims[:-1]):
        at = sum(a * b + b for a, b in dims[:l])
        z = x @ finite[at:at + i * o].reshape(i, o) + finite[at + i * o:at + i * o + o]
        x = np.where(z > 0, z, np.expm1(np.minimum(z, 0)))
    clear = np.abs(x[:, 7]) > 1e-4
    assert np.array_equal(got[clear, 2], np.sign(x[clear, 7]).astype(np.float32))


@pytest.mark.parametrize("batch,hidden", [(40, (64, 64)), (333, (96, 40)), (8192, (256, 256))])
def test_weight_gradients_of_columns_with_outliers(batch, hidden):
    """A column's scale is that of its largest value: states of 2^20 in some rows (the first a wavefront sees) and of order 1 in
    the others, where the large ones meet a delta of exactly zero (the TD target of those rows is the critic's own Q value).
    The small ones have to keep 32-bit precision: every row of critic 1's dW_1 to 1e-5 of its own largest entry."""
    import torch
    from test_gpu_parity import workspace_rows
    w = workload(hidden, 21, 3, batch)
    s, ring = session(w), oracle_ring(w)
    fill_both(s, ring, w, w.nstep + 3)
    s.sample(batch)
    rng = np.random.default_rng(9)
    b = {k: getattr(s.batch, k)[:batch].cpu().numpy().copy() for k in ("obs", "act", "ret", "next_obs", "boot")}
    b["obs"] = rng.standard_normal((batch, w.obs_dim)).astype(np.float32)
    large = np.arange(batch) % 64 == 0
    cols = [2, 7, 20]
    b["obs"][np.ix_(large, cols)] *= np.float32(2.0 ** 20)
    b["boot"][:] = 0.0
    c = s.critic_init.copy()
    for h in (0, c.size // 2):
        c[h:h + w.obs_dim * hidden[0]].reshape(w.obs_dim, -1)[cols] = 0.0       # the hidden layers do not see these columns
    for _ in range(2):
        for k in ("obs", "ret", "boot"):
            getattr(s.batch, k)[:batch].copy_(torch.from_numpy(b[k]))
        s.critic.copy_(torch.from_numpy(c))
        s.critic_update(batch)
        b["ret"][large] = workspace_rows(s, 1, batch)[large]
    rest = {k: v[~large] for k, v in b.items()}
    n, half = w.obs_dim * hidden[0], c.size // 2
    _, g = O.critic_loss_and_grads(c, w.critic_dims(), rest, rest["ret"].astype(np.float64))
    ref = g[:n].reshape(w.obs_dim, -1) * ((~large).sum() / batch)
    x = s.c_g.cpu().numpy().astype(np.float64)[:n].reshape(w.obs_dim, -1)
    err = np.abs(x - ref).max(1) / np.abs(ref).max(1)
    print(batch, hidden, "columns with outliers %.2e" % err[cols].max(), "others %.2e" % np.delete(err, cols).max(), flush=True)
    assert err.max() <= TOL


def test_policy_gradient_no_further_from_float64_than_fp32_products():
    """Weights as fp16 pairs miss the last bit of a quarter of them; rounded one way for the whole batch, those errors add up
    in the gradients.  2-norm error of the policy gradient over four batches of 4096 rows: at most 9e-8 (fp32 matrix
    instructions leave 9.8e-8 here, one set of pairs 1.06e-7, two that alternate from row tile to row tile 7.6e-8)."""
    import torch
    w = workload((512, 256, 128), 108, 21, 4096)
    errs = []
    for seed in range(4):
        s = session(w)
        rng = np.random.default_rng(100 + seed)
        nets = []
        for dims, twins in ((w.actor_dims(), 1), (w.critic_dims(), 2)):
            nets.append(np.concatenate([(rng.uniform(-1, 1, i * o + o) / np.sqrt(i)) for _ in range(twins) for i, o in dims])
                        .astype(np.float32))
        obs = rng.standard_normal((w.batch, w.obs_dim)).astype(np.float32)
        s.actor.copy_(torch.from_numpy(nets[0]))
        s.critic.copy_(torch.from_numpy(nets[1]))
        s.actor_update(torch.from_numpy(obs).cuda(), w.batch)
        L = oracle_learner(w, nets[0], nets[1])
        _, g = L.actor_update(obs)
        errs.append(np.linalg.norm(s.a_g.cpu().numpy() - g) / np.linalg.norm(g))
    print("policy gradient 2-norm errors", errs, flush=True)
    assert np.mean(errs) <= 9e-8


@pytest.mark.parametrize("case,num", [("narrow", 8193), ("narrow", 16384), ("one_step_inputs", 16321), ("widest", 8193), ("widest", 24577),
                                      ("wide", 8193), ("stochastic", 8200)])
def test_actor_step_on_tiles_of_64_rows(case, num):
    """The Actor step on tiles of 64 rows: a last tile of one row, full tiles, inputs of one step and of eight (in the place of the
    activations where a layer is 512 wide), standardised observations on both kernels.  To 1e-5 of the actions' scale of 1
    (products to 1e-7, tanh and noise as on the other tiles)."""
    import torch
    from test_actor_tiles_host import tile_rows
    w = {"narrow": workload((96, 64), 60, 8, num), "one_step_inputs": workload((64, 256, 32), 7, 3, num, obs_norm=True),
         "widest": workload((512, 64, 256), 256, 32, num, obs_norm=True), "wide": workload((512, 96), 20, 6, num, obs_norm=True),
         "stochastic": workload((128, 96), 45, 11, num, sac=True)}[case]
    print(case, w.hidden, "N", num, flush=True)
    assert tile_rows(w.hidden, w.obs_dim, w.act_dim, num, w.sac) == 64
    s = session(w)
    rng = np.random.default_rng(17)
    obs = (1.0 + 2.0 * rng.standard_normal((num, w.obs_dim))).astype(np.float32)
    seen = obs
    if w.obs_norm:
        from parity_util import oracle_normalizer
        nz = oracle_normalizer(w)
        row = W.transition_rows(w, W.data_rng(w), 1)[0]
        s.push(row)
        nz.update(row["obs"])
        seen = nz.normalize(obs)
    lo, hi = float(np.float32(0.05)), float(np.float32(0.8))
    got = s.act(torch.from_numpy(obs).cuda(), lo, hi).cpu().numpy().astype(np.float64)
    ref = (O.sac_actor_act(s.actor_init, w.actor_dims(), seen, w.rng_seed, 0) if w.sac else
           O.actor_act(s.actor_init, w.actor_dims(), seen, lo, hi, w.rng_seed, 0))
    err = np.abs(got - ref).max()
    print("max abs err %.2e" % err, flush=True)
    assert err <= TOL


RARE = {            # the kernels that keep what the others leave out: widths that are no multiples of four, inputs of more than eight steps
    "odd_fused": workload((63, 30), 9, 3, 65),
    "odd_pair": workload((301, 62), 33, 5, 97),
    "odd_pair_sac": workload((301, 62), 33, 5, 97, sac=True),
    "odd_pair_atoms": workload((301, 62), 33, 5, 97, num_atoms=21),
    "odd_single_sac": workload((514, 31), 20, 4, 65, sac=True),
    "nine_steps": workload((64, 32), 250, 7, 33),
    "eight_steps": workload((512, 512), 248, 8, 2050),             # 256 columns: the widest regular input, in the place of the activations
}


@pytest.mark.parametrize("case", list(RARE))
def test_gradients_of_rare_shapes(case):
    w = RARE[case]
    print(case, w.hidden, "B", w.batch, flush=True)
    s, ring = session(w), oracle_ring(w)
    fill_both(s, ring, w, w.nstep + 3)
    L = oracle_learner(w, s.actor_init, s.critic_init)
    s.sample(w.batch)
    batch = oracle_batch(ring, w, w.batch, 0, None)
    s.critic_update(w.batch)
    losses, g = L.critic_update(batch)
    s.actor_update(None, w.batch)
    _, ga = L.actor_update(batch["obs"])
    assert rel_err(s.critic_loss.cpu().numpy(), losses) <= TOL
    assert_params_close(s.c_g.cpu().numpy(), g, w.critic_dims(), 2, TOL, "critic grad")
    assert_params_close(s.a_g.cpu().numpy(), ga, w.actor_dims(), 1, TOL, "actor grad")
