"""Step-granular calls (msrl_observe / msrl_act / msrl_env_step) through the C ABI.

The fused rollout is checked against the oracle in test_gpu_parity.py; here the split calls are
checked (a) to reproduce the fused call bit for bit, and (b) directly against the oracle's
environment step for actions the test chooses itself.
"""
import numpy as np
import pytest

from helpers import GpuRollout, TOL_F32, assert_close, oracle_setup
from oracle import ref
from paper_2210_00882_amd import synth

pytestmark = pytest.mark.gpu


def setup_any(cfg):
    """oracle_setup for every env kind (the pursuit env has no entry there)."""
    if cfg.kind == synth.TAG:
        from test_gpu_tag import tag_env
        pol = ref.Policy(cfg.obs_dim, cfg.hidden, 5, bf16=cfg.dtype == synth.BF16)
        return tag_env(cfg), pol, synth.make_params(cfg, bias_std=0.1).astype(np.float64), None
    return oracle_setup(cfg)


def expected_outputs(cfg, pol, params, rows_env):
    """Oracle networks on the N rows of one env -> (logits [N, out], values [N]); handles the role routing of
    the pursuit env and the centralised critic."""
    N = cfg.num_agents
    lg, v = [], []
    central = getattr(cfg, "central_critic", False)
    for i in range(N):
        prm = params
        if cfg.kind == synth.TAG:
            n = pol.param_count
            prm = params[:n] if i < cfg.num_chasers else params[n:]
        if central:
            lg.append(ref.mlp(pol.in_dim, pol.hidden, pol.out_dim, prm[:pol.policy_param_count], rows_env[i],
                              bf16=cfg.dtype == synth.BF16))
            v.append(ref.central_value(pol, prm, rows_env))
        else:
            a, b = ref.policy_value(pol, prm, rows_env[i])
            lg.append(a)
            v.append(b)
    return np.array(lg), np.array(v)


def split_rollout(gpu, T, logits=True):
    """T x { observe / act / env_step } -> the arrays msrl_rollout_step would fill."""
    import torch
    B, cfg = gpu.B, gpu.cfg
    M, D = cfg.M, cfg.obs_dim
    tr = B.alloc_traj(cfg, T, logits=logits, gae=False)
    for v in tr.values():
        if v is not None:
            v.fill_(-77 if v.dtype != torch.uint8 else 77)
    B.msrl_observe(gpu.state, tr["obs"][0])
    for t in range(T):
        B.msrl_act(gpu.state, gpu.params, tr["obs"][t], tr["actions"][t], tr["logp"][t], tr["values"][t],
                   tr["logits"][t] if logits else None)
        B.msrl_env_step(gpu.state, tr["actions"][t], tr["rewards"][t], tr["dones"][t], tr["obs"][t + 1])
    # values[T]: one more evaluation whose sampled outputs are dropped
    scratch_a = torch.empty_like(tr["actions"][0])
    scratch_l = torch.empty(M, dtype=torch.float32, device="cuda")
    B.msrl_act(gpu.state, gpu.params, tr["obs"][T], scratch_a, scratch_l, tr["values"][T], None)
    torch.cuda.synchronize()
    return {k: (None if v is None else v.cpu().numpy()) for k, v in tr.items()}


ACT_CASES = {
    "n3_f32_ragged": lambda: synth.CONFIGS[1].with_(num_envs=53, episode_len=4),
    "n1_f32": lambda: synth.particle("p1", 70, 1, 64, 6, 3, synth.F32, 11),
    "n2_f32": lambda: synth.particle("p2", 37, 2, 64, 6, 3, synth.F32, 13),
    "n6_f32": lambda: synth.CONFIGS[3].with_(num_envs=77, episode_len=5),
    "n3_bf16": lambda: synth.particle("p3b", 45, 3, 64, 6, 3, synth.BF16, 12),
    "n10_bf16": lambda: synth.CONFIGS[5].with_(num_envs=100, episode_len=3),
    "lingauss": lambda: synth.CONFIGS[4].with_(num_envs=150, episode_len=3),
    # shapes off the benchmark table (every agent count 1 .. 10 is compiled for every width and type)
    "n4_h128_bf16": lambda: synth.particle("p4", 45, 4, 128, 6, 3, synth.BF16, 17),
    "n7_h256_f32": lambda: synth.particle("p7", 33, 7, 256, 6, 3, synth.F32, 18),
    "n8_h128_f32_3_layers": lambda: synth.particle("p8", 29, 8, 128, 6, 3, synth.F32, 19).with_(hidden_layers=3),
    "n9_h64_bf16": lambda: synth.particle("p9", 31, 9, 64, 6, 3, synth.BF16, 20),
    # networks with more than two hidden layers (the evaluated networks of section 7.1 have seven layers)
    "n3_f32_4_layers": lambda: synth.particle("p3d", 45, 3, 64, 6, 3, synth.F32, 14).with_(hidden_layers=4),
    "n3_bf16_3_layers": lambda: synth.particle("p3d", 45, 3, 64, 6, 3, synth.BF16, 15).with_(hidden_layers=3),
    "n10_bf16_6_layers": lambda: synth.CONFIGS[5].with_(num_envs=50, episode_len=3, hidden_layers=6),
    "lingauss_3_layers": lambda: synth.CONFIGS[4].with_(num_envs=70, episode_len=3, hidden_layers=3),
    # centralised critic (section 2.1): the value network on the joint observation of the env's agents
    "n3_bf16_central": lambda: synth.particle("p3c", 45, 3, 64, 6, 3, synth.BF16, 16).with_(central_critic=True),
    "n10_bf16_central": lambda: synth.CONFIGS[5].with_(num_envs=50, episode_len=3, central_critic=True),
    "n3_f32_central": lambda: synth.CONFIGS[1].with_(num_envs=45, episode_len=3, central_critic=True),
    # pursuit env (the task of the GPU-only experiment, section 7.3): one parameter set per role
    "tag_3_1": lambda: synth.tag("tag", 70, 3, 1, 2, 64, 6, 3, idx=50).with_(radius_c=0.3, radius_r=0.25),
    "tag_2_2": lambda: synth.tag("tag", 41, 2, 2, 1, 64, 6, 3, idx=51).with_(radius_c=0.3, radius_r=0.25),
    "tag_2_3_f32": lambda: synth.tag("tag", 37, 2, 3, 2, 64, 6, 3, dtype=synth.F32, idx=52).with_(radius_c=0.3, radius_r=0.25),
}


@pytest.mark.parametrize("which", sorted(ACT_CASES))
def test_split_calls_reproduce_the_fused_rollout(which):
    cfg = ACT_CASES[which]()
    T = 7
    _, _, params, dyn = setup_any(cfg)
    with GpuRollout(cfg, params.astype(np.float32), 31, dyn=dyn) as gpu:
        fused = gpu.run(T, gae=False, logits=True)
        es_f, g_f = gpu.get_state()
    with GpuRollout(cfg, params.astype(np.float32), 31, dyn=dyn) as gpu:
        split = split_rollout(gpu, T)
        es_s, g_s = gpu.get_state()
    for k in ("obs", "actions", "logp", "rewards", "dones", "values", "logits"):
        np.testing.assert_array_equal(fused[k], split[k], err_msg=k)
    np.testing.assert_array_equal(es_f, es_s)
    np.testing.assert_array_equal(g_f, g_s)
    assert (g_s == T).all()


@pytest.mark.parametrize("N", range(1, 11))
@pytest.mark.parametrize("H,dtype", [(64, synth.F32), (128, synth.BF16), (256, synth.BF16)])
def test_env_step_rows_are_those_of_the_fused_rollout(N, H, dtype):
    # (the env step's kernel deals a row's features out to the two lanes of the row in a way that depends on N)
    import torch
    cfg = synth.particle("rows", 37, N, H, 3, 2, dtype)
    params = synth.make_params(cfg, bias_std=0.1)
    with GpuRollout(cfg, params, 9) as fused, GpuRollout(cfg, params, 9) as steps:
        want = fused.run(cfg.T)
        obs = torch.full((cfg.M, cfg.obs_dim), -77.0, device="cuda")
        rewards, dones = torch.empty(cfg.M, device="cuda"), torch.empty(cfg.M, dtype=torch.uint8, device="cuda")
        steps.B.msrl_observe(steps.state, obs)
        np.testing.assert_array_equal(obs.cpu().numpy(), want["obs"][0])
        for t in range(cfg.T):
            obs.fill_(-77.0)
            steps.B.msrl_env_step(steps.state, fused.dev["actions"][t], rewards, dones, obs)
            np.testing.assert_array_equal(obs.cpu().numpy(), want["obs"][t + 1], err_msg=f"t {t}")
            np.testing.assert_array_equal(rewards.cpu().numpy(), want["rewards"][t])
            np.testing.assert_array_equal(dones.cpu().numpy(), want["dones"][t])


@pytest.mark.parametrize("which", ["n1_h64_f32", "n10_h256_bf16"])
def test_actor_fragment_over_more_row_blocks_than_compute_units(which):
    # the plain actor kernel is persistent: with more row blocks than the device has compute units a workgroup
    # walks over several of them (a ragged last one included).  T x {act, env_step} must still be the fused
    # rollout bit for bit, for every row.
    cfg = (synth.particle("walk1", 40001, 1, 64, 2, 3, synth.F32, 21) if which == "n1_h64_f32"
           else synth.CONFIGS[5].with_(num_envs=7001, episode_len=3))
    T = 2
    _, _, params, dyn = setup_any(cfg)
    with GpuRollout(cfg, params.astype(np.float32), 33, dyn=dyn) as gpu:
        fused = gpu.run(T, gae=False, logits=True)
        es_f, g_f = gpu.get_state()
    with GpuRollout(cfg, params.astype(np.float32), 33, dyn=dyn) as gpu:
        split = split_rollout(gpu, T)
        es_s, g_s = gpu.get_state()
    for k in ("obs", "actions", "logp", "rewards", "dones", "values", "logits"):
        np.testing.assert_array_equal(fused[k], split[k], err_msg=k)
    np.testing.assert_array_equal(es_f, es_s)
    np.testing.assert_array_equal(g_f, g_s)


@pytest.mark.parametrize("which", ["n3_f32", "tag_3_1", "tag_2_2"])
def test_env_step_against_the_oracle_for_chosen_actions(which):
    import torch
    cfg = synth.CONFIGS[1].with_(num_envs=41, episode_len=3) if which == "n3_f32" else ACT_CASES[which]()
    env, _, params, _ = setup_any(cfg)
    N, M, D = cfg.num_agents, cfg.M, cfg.obs_dim
    rng = np.random.default_rng(5)
    seed = 77
    contacts = 0
    with GpuRollout(cfg, params.astype(np.float32), seed) as gpu:
        B = gpu.B
        obs = torch.empty((M, D), dtype=torch.float32, device="cuda")
        rew = torch.empty(M, dtype=torch.float32, device="cuda")
        done = torch.empty(M, dtype=torch.uint8, device="cuda")
        for step in range(7):                       # crosses episode ends (reset draws)
            es, g = gpu.get_state()
            acts = rng.integers(0, 5, size=M).astype(np.int32)
            B.msrl_env_step(gpu.state, torch.from_numpy(acts).cuda(), rew, done, obs)
            torch.cuda.synchronize()
            r_gpu, d_gpu, o_gpu = rew.cpu().numpy(), done.cpu().numpy(), obs.cpu().numpy()
            es1, g1 = gpu.get_state()
            assert (g1 == g + 1).all()
            for e in range(cfg.num_envs):
                s = es[e].astype(np.float64)
                s2, r, d, margin = ref.env_step(env, seed, e, int(g[e]), s, acts[e * N:(e + 1) * N])
                if margin > 1e-5:   # no pair distance within 1e-5 of the collision / contact threshold
                    assert_close(r_gpu[e * N:(e + 1) * N], np.broadcast_to(r, (N,)), TOL_F32, f"reward env {e} step {step}")
                contacts += int(np.any(np.asarray(r) > 0))
                assert (d_gpu[e * N:(e + 1) * N] == d).all()
                assert_close(es1[e], s2, TOL_F32, f"state env {e} step {step}")
                assert_close(o_gpu[e * N:(e + 1) * N], ref.env_obs(env, es1[e].astype(np.float64)), TOL_F32,
                             f"next obs env {e} step {step}")
    if cfg.kind == synth.TAG:
        assert contacts > 10       # contact forces and contact rewards were exercised


def test_observe_and_act_leave_the_state_alone_and_argument_errors():
    import torch
    cfg = synth.CONFIGS[1].with_(num_envs=9)
    _, _, params, _ = oracle_setup(cfg)
    M, D = cfg.M, cfg.obs_dim
    with GpuRollout(cfg, params.astype(np.float32), 3) as gpu:
        B = gpu.B
        es0, g0 = gpu.get_state()
        obs = torch.empty((M, D), dtype=torch.float32, device="cuda")
        a = torch.empty(M, dtype=torch.int32, device="cuda")
        lp = torch.empty(M, dtype=torch.float32, device="cuda")
        v = torch.empty(M, dtype=torch.float32, device="cuda")
        B.msrl_observe(gpu.state, obs)
        with pytest.raises(B.MsrlError) as e:      # no parameters have been passed to this state yet
            B.msrl_act(gpu.state, None, obs, a, lp, v)
        assert e.value.code == B.MSRL_EINVAL
        B.msrl_act(gpu.state, gpu.params, obs, a, lp, v)
        B.msrl_act(gpu.state, gpu.params, obs, a, lp, v)
        # params = NULL: the image of the last parameters is used again
        a2, lp2, v2 = torch.full_like(a, -1), torch.full_like(lp, -1.0), torch.full_like(v, -1.0)
        B.msrl_act(gpu.state, None, obs, a2, lp2, v2)
        torch.cuda.synchronize()
        assert torch.equal(a, a2) and torch.equal(lp, lp2) and torch.equal(v, v2)
        es1, g1 = gpu.get_state()
        np.testing.assert_array_equal(es0, es1)
        np.testing.assert_array_equal(g0, g1)
        with pytest.raises(B.MsrlError) as e:
            B.msrl_act(gpu.state, gpu.params, obs, a, lp, None)
        assert e.value.code == B.MSRL_EINVAL
        with pytest.raises(B.MsrlError) as e:
            B.msrl_env_step(gpu.state, a, None, None, obs)
        assert e.value.code == B.MSRL_EINVAL



def _caller_rows(cfg, rng, kind):
    """Observation rows [M, D] that no state of the library produced."""
    M, D, N = cfg.M, cfg.obs_dim, cfg.num_agents
    if kind == "random":
        rows = rng.standard_normal((M, D)).astype(np.float32) * np.float32(0.7)
    else:                                          # large and tiny magnitudes: tanh saturation, bf16 rounding
        rows = (rng.standard_normal((M, D)) * rng.choice([1e-3, 0.3, 4.0], size=(M, 1))).astype(np.float32)
    if cfg.kind == synth.PARTICLE and N > 1:       # the trailing 2 (N - 1) slots of the particle layout are zero
        rows[:, D - 2 * (N - 1):] = 0.0
    return rows


@pytest.mark.parametrize("which", sorted(ACT_CASES))
def test_act_on_caller_chosen_rows_against_the_oracle(which):
    """The actor fragment of DP-A / DP-B (section 6, Table 2) acts on observations that come from outside the
    device fragment: rows the test draws itself, and rows of a different env batch.  Networks against
    the oracle row by row; the sampler against the oracle's, fed the GPU's logits and the Philox
    counters (env, agent, step counter of the state)."""
    import torch
    cfg = ACT_CASES[which]()
    env, pol, params, dyn = setup_any(cfg)
    bf16 = cfg.dtype == synth.BF16
    net_tol = 2e-2 if bf16 else TOL_F32
    N, M, D = cfg.num_agents, cfg.M, cfg.obs_dim
    rng = np.random.default_rng(17)
    seed = 901
    # rows of another env batch (other seed, a few steps in)
    with GpuRollout(cfg, params.astype(np.float32), 555, dyn=dyn) as other:
        other.run(3, gae=False, logits=False)
        foreign = torch.empty((M, D), dtype=torch.float32, device="cuda")
        other.B.msrl_observe(other.state, foreign)
        torch.cuda.synchronize()
        foreign = foreign.cpu().numpy()
    with GpuRollout(cfg, params.astype(np.float32), seed, dyn=dyn) as gpu:
        B = gpu.B
        # distinct, non-zero step counters: the noise must be the one of (env, agent, g[env])
        g = (rng.integers(1, 1000, size=cfg.num_envs)).astype(np.int64)
        gpu.set_state(None, g)
        for label, rows in (("random", _caller_rows(cfg, rng, "random")),
                            ("scaled", _caller_rows(cfg, rng, "scaled")),
                            ("foreign", foreign)):
            obs = torch.from_numpy(rows).cuda()
            a = torch.full((M,) if cfg.dist == synth.CATEGORICAL else (M, cfg.act_dim), -7,
                           dtype=torch.int32 if cfg.dist == synth.CATEGORICAL else torch.float32, device="cuda")
            lp = torch.full((M,), -77.0, device="cuda")
            v = torch.full((M,), -77.0, device="cuda")
            lg = torch.full((M, cfg.out_dim), -77.0, device="cuda")
            B.msrl_act(gpu.state, gpu.params, obs, a, lp, v, lg)
            torch.cuda.synchronize()
            a, lp, v, lg = a.cpu().numpy(), lp.cpu().numpy(), v.cpu().numpy(), lg.cpu().numpy()
            edges = 0
            for e in range(cfg.num_envs):
                lg_o, v_o = expected_outputs(cfg, pol, params, rows[e * N:(e + 1) * N])
                for i in range(N):
                    m = e * N + i
                    assert_close(lg[m], lg_o[i], net_tol, f"{label}: logits row {m}")
                    assert_close(v[m], v_o[i], net_tol, f"{label}: value row {m}")
                    a_o, lp_o, mg = ref.sample(pol, seed, e, i, int(g[e]), lg[m])
                    if cfg.dist == synth.CATEGORICAL:
                        if int(a[m]) != a_o:
                            assert mg < 1e-5, f"{label}: action row {m}: gpu {a[m]} oracle {a_o} margin {mg}"
                            edges += 1
                            z = lg[m].astype(np.float64) - lg[m].max()
                            lp_o = float(z[int(a[m])] - np.log(np.exp(z).sum()))
                    else:
                        assert_close(a[m], a_o, TOL_F32, f"{label}: action row {m}")
                    assert_close(lp[m], lp_o, TOL_F32, f"{label}: logp row {m}")
            assert edges <= 2
        es1, g1 = gpu.get_state()
        np.testing.assert_array_equal(g1, g)      # acting does not advance the state


@pytest.mark.parametrize("hidden,gauss", [(64, False), (128, False), (256, False), (256, True)])
def test_infinite_and_nan_observations_in_fp32(hidden, gauss):
    # an infinite input saturates the first layer's units, as in fp32 arithmetic; a NaN spreads within its row only
    import torch
    cfg = synth.lingauss("inf", 8, 17, 6, 256, 4, 1000) if gauss else synth.particle("inf", 4, 3, hidden, 4, 25, synth.F32)
    _, _, params, dyn = oracle_setup(cfg)
    rng = np.random.default_rng(3)
    rows = rng.uniform(-1, 1, (cfg.M, cfg.obs_dim)).astype(np.float32)
    rows[0, 0], rows[1, 3], rows[2, 1], rows[3, 2] = np.inf, -np.inf, np.nan, 3.4e38
    with GpuRollout(cfg, params.astype(np.float32), 11, dyn=dyn) as gpu:
        B = gpu.B
        a = torch.empty((cfg.M, cfg.act_dim) if gauss else (cfg.M,), dtype=torch.float32 if gauss else torch.int32, device="cuda")
        lp, v = torch.empty(cfg.M, device="cuda"), torch.empty(cfg.M, device="cuda")
        B.msrl_act(gpu.state, gpu.params, torch.from_numpy(rows).cuda(), a, lp, v)
        torch.cuda.synchronize()
        v = v.cpu().numpy()
    if not gauss and cfg.num_agents > 1:
        rows[:, -2 * (cfg.num_agents - 1):] = 0.0     # the silent slots are not read
    at = params.size - sum(i * o + o for i, o in ((cfg.obs_dim, cfg.hidden), (cfg.hidden, cfg.hidden), (cfg.hidden, 1)))
    x = rows.astype(np.float64)
    for k, (i, o) in enumerate(((cfg.obs_dim, cfg.hidden), (cfg.hidden, cfg.hidden), (cfg.hidden, 1))):
        x = x @ params[at:at + i * o].reshape(i, o) + params[at + i * o:at + i * o + o]
        at += i * o + o
        x = np.tanh(x) if k < 2 else x
    assert np.isnan(v[2]) and np.isnan(x[2])
    keep = np.arange(cfg.M) != 2
    assert_close(v[keep], x[keep, 0], TOL_F32, "values")


def ieee_net(params, dims, at, x):
    """A network in float64 with the products written out: infinities and NaN as IEEE arithmetic has them."""
    with np.errstate(all="ignore"):
        for k, (i, o) in enumerate(zip(dims[:-1], dims[1:])):
            w = params[at:at + i * o].reshape(i, o)
            y = np.empty((x.shape[0], o))
            for r in range(x.shape[0]):
                y[r] = (x[r][:, None] * w).sum(0)
            x = y + params[at + i * o:at + i * o + o]
            at += i * o + o
            x = np.tanh(x) if k < len(dims) - 2 else x
    return x, at


@pytest.mark.parametrize("where", ["inputs", "hidden weight", "opposed hidden weights", "hidden bias", "first layer",
                                   "output layer"])
@pytest.mark.parametrize("hidden,gauss,layers", [(64, False, 2), (128, False, 2), (128, False, 3), (256, False, 2),
                                                 (256, True, 2), (256, True, 3)])
def test_infinities_behave_as_in_fp32_arithmetic(hidden, gauss, layers, where):
    # products with an infinity, infinities that meet, and values whose products overflow: finite, infinite and NaN where
    # IEEE arithmetic has them
    import torch
    cfg = synth.lingauss("inf", 64, 17, 6, 256, 4, 1000) if gauss else synth.particle("inf", 16, 4, hidden, 4, 25, synth.F32)
    cfg = cfg.with_(hidden_layers=layers)
    _, _, params, dyn = oracle_setup(cfg)
    params = params.astype(np.float32)
    D, H = cfg.obs_dim, cfg.hidden
    dims = [D] + [H] * layers
    value_at = params.size - sum(i * o + o for i, o in zip(dims, dims[1:] + [1]))
    rng = np.random.default_rng(3)
    rows = rng.uniform(-1, 1, (cfg.M, D)).astype(np.float32)
    if not gauss:
        rows[:, -2 * (cfg.num_agents - 1):] = 0.0     # the silent slots are not read
    for at in (0, value_at):                          # both networks
        w1, w2 = params[at:at + D * H].reshape(D, H), params[at + D * H + H:at + D * H + H + H * H].reshape(H, H)
        if where == "inputs":
            w1[2] = np.sign(w1[2]) * np.geomspace(1.0, 3e6, H)  # (times any huge input: saturated, never NaN)
            w1[5, 7] = 0.0
        elif where == "hidden weight":
            w2[3, 4] = np.inf
        elif where == "opposed hidden weights":       # NaN in the rows whose two units agree in sign
            w2[3, 4], w2[5, 4] = np.inf, -np.inf
        elif where == "hidden bias":
            params[at + D * H + H + H * H + 1] = -np.inf
        elif where == "first layer":
            w1[0, 1], w1[1, 2], w1[3, 3] = -np.inf, 1e38, np.inf
        else:
            n = 1 if at else cfg.out_dim
            end = params.size if at else value_at
            w3 = params[end - n - H * n:end - n].reshape(H, n)
            w3[7, 0] = np.inf
            if not at:
                w3[9, 3] = -np.inf
    if where == "inputs":
        rows[:, 2] = 0.0
        rows[0, 0], rows[1, 3], rows[2, 1] = np.inf, -np.inf, np.nan
        for k, v in enumerate((3.4e38, -3.3895e38, 1e38, -7e4, 65536.0, 1e20, np.inf, -np.inf)):
            rows[3 + k, 2] = v
        rows[11, 0], rows[11, 1] = np.inf, np.inf     # meet with both signs
        rows[12, 5] = np.inf                          # times a weight of 0
        rows[13, 0], rows[13, 2] = -np.inf, np.nan
    if where == "first layer":
        rows[0, 0], rows[1, 0], rows[2, 3] = 0.0, np.inf, -np.inf   # inf * 0, inf * inf
    with GpuRollout(cfg, params, 11, dyn=dyn) as gpu:
        B = gpu.B
        a = torch.empty((cfg.M, cfg.act_dim) if gauss else (cfg.M,), dtype=torch.float32 if gauss else torch.int32, device="cuda")
        lp, v = torch.empty(cfg.M, device="cuda"), torch.empty(cfg.M, device="cuda")
        lg = torch.empty((cfg.M, cfg.out_dim), device="cuda")
        B.msrl_act(gpu.state, gpu.params, torch.from_numpy(rows).cuda(), a, lp, v, lg)
        torch.cuda.synchronize()
        got = np.concatenate([lg.cpu().numpy(), v.cpu().numpy()[:, None]], 1).astype(np.float64)
    x = rows.astype(np.float64)
    if not gauss:
        x[:, -2 * (cfg.num_agents - 1):] = 0.0
    pol, at = ieee_net(params.astype(np.float64), dims + [cfg.out_dim], 0, x)
    val, end = ieee_net(params.astype(np.float64), dims + [1], value_at, x)
    assert at == value_at and end == params.size
    want = np.concatenate([pol, val], 1)
    np.testing.assert_array_equal(np.isnan(got), np.isnan(want), err_msg="NaN")
    inf = np.isinf(want)
    np.testing.assert_array_equal(np.isinf(got), inf, err_msg="infinite")
    np.testing.assert_array_equal(got[inf], want[inf])
    fin = np.isfinite(want)
    assert fin.any()
    if where in ("opposed hidden weights", "inputs"):
        assert np.isnan(want).any(1).any() and not np.isnan(want).any(1).all()
    assert_close(got[fin], want[fin], TOL_F32, "finite outputs")


@pytest.mark.parametrize("hidden,gauss,layers,central,roles", [
    (64, False, 2, False, 1), (64, False, 2, False, 2), (64, False, 2, True, 0), (64, False, 3, False, 0),
    (128, False, 2, False, 0), (128, False, 2, True, 0), (256, False, 2, False, 0), (256, False, 3, False, 0),
    (256, True, 2, False, 0), (256, True, 3, False, 0)])
def test_rollouts_of_large_and_infinite_states_in_fp32(hidden, gauss, layers, central, roles):
    # every fp32 rollout kernel on states beyond the ordinary: its own observations through IEEE arithmetic
    cfg = synth.lingauss("big", 40, 17, 6, 256, 4, 1000) if gauss else synth.particle("big", 40, 4, hidden, 4, 25, synth.F32)
    cfg = cfg.with_(hidden_layers=layers, central_critic=central)
    params, dyn = synth.make_params(cfg, bias_std=0.1).astype(np.float32), synth.make_dynamics(cfg) if gauss else None
    D, H = cfg.obs_dim, cfg.hidden
    with GpuRollout(cfg, params, 11, dyn=dyn, wave_roles=roles) as gpu:
        es, _ = gpu.get_state()
        for k, v in enumerate((7e4, 65536.0, -1e6, 1e20, -3.4e38, np.inf, -np.inf, np.nan)):
            es[3 * k, 3] = v                 # (particle env: a velocity, which enters one agent's row alone)
        if not gauss:
            es[30, 0] = 1e10                 # a position, which enters every row of its env
        gpu.set_state(es)
        tr = gpu.run(1, gae=False)
    rows = tr["obs"][0].astype(np.float64)
    pol, at = ieee_net(params.astype(np.float64), [D] + [H] * layers + [cfg.out_dim], 0, rows)
    val, _ = ieee_net(params.astype(np.float64), [cfg.value_in_dim] + [H] * layers + [1], at,
                      rows.reshape(cfg.num_envs, -1) if central else rows)
    val = np.repeat(val[:, 0], cfg.num_agents) if central else val[:, 0]
    assert np.isinf(rows).any() and np.isnan(pol).any()
    for what, got, want in (("logits", tr["logits"][0].astype(np.float64), pol), ("values", tr["values"][0].astype(np.float64), val)):
        np.testing.assert_array_equal(np.isnan(got), np.isnan(want), err_msg=what)
        ok = ~np.isnan(want)
        assert_close(got[ok], want[ok], TOL_F32, what)


@pytest.mark.parametrize("which", sorted(ACT_CASES))
def test_observe_against_the_oracle(which):
    """msrl_observe == the oracle's observation of the state msrl_state_get returns, at the initial
    state, after a rollout (mid-episode, moving agents) and for a state the test injects."""
    import torch
    cfg = ACT_CASES[which]()
    env, _, params, dyn = setup_any(cfg)
    N, M, D = cfg.num_agents, cfg.M, cfg.obs_dim
    rng = np.random.default_rng(23)
    with GpuRollout(cfg, params.astype(np.float32), 77, dyn=dyn) as gpu:
        obs = torch.empty((M, D), dtype=torch.float32, device="cuda")

        def check(label):
            obs.fill_(-77.0)
            gpu.B.msrl_observe(gpu.state, obs)
            torch.cuda.synchronize()
            o = obs.cpu().numpy()
            es, _ = gpu.get_state()
            for e in range(cfg.num_envs):
                assert_close(o[e * N:(e + 1) * N], ref.env_obs(env, es[e].astype(np.float64)), TOL_F32,
                             f"{label}: env {e}")
        check("initial")
        gpu.run(5, gae=False, logits=False)
        check("after 5 steps")
        gpu.set_state(rng.standard_normal((cfg.num_envs, cfg.env_state_size)).astype(np.float32), None)
        check("injected")
