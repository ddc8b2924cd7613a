"""Learner entry points (msrl_ppo_grad / msrl_adam_step / msrl_ppo_update) against the CPU oracle.

Tolerances.  A gradient entry is a sum over the rows of products, which may cancel to anything, so
its error is measured per output unit: for unit j of a layer (column j of W and entry j of b, which
are sums over the rows of the same dL/dz_j times inputs of magnitude <= 1)
    |gpu - oracle| <= tol * max(|oracle| over column j of W and b[j]),
tol = 1e-4 (fp32 networks) or 2e-2 (bf16 networks; the oracle rounds the backward operands to
bf16 at the same points as the kernels, see oracle/msrl_learn_ref.c).  The per-tensor form
(relative to the tensor's largest entry) is implied by it.  Adam is elementwise fp32
arithmetic: 1e-5 relative.
"""
import numpy as np
import pytest

from oracle import ref
from paper_2210_00882_amd import synth

pytestmark = pytest.mark.gpu


def tensors_of(vec, i, h, o, layers=2):
    """(name, slice) of the tensors of one network inside the flat vector, and its length."""
    out, s = [], 0
    names = [("W1", i * h), ("b1", h)]
    for l in range(2, layers + 1):
        names += [(f"W{l}", h * h), (f"b{l}", h)]
    names += [("Wout", h * o), ("bout", o)]
    for name, n in names:
        out.append((name, slice(s, s + n)))
        s += n
    return out, s


def make_batch(cfg, R, seed, params):
    """Rows with the shapes of a stored trajectory; ratios spread around the clip range."""
    rng = np.random.default_rng(seed)
    central = getattr(cfg, "central_critic", False)
    pol = ref.Policy(cfg.obs_dim, cfg.hidden, cfg.out_dim, bf16=cfg.dtype == synth.BF16, dist=cfg.dist,
                     hidden_layers=cfg.hidden_layers, value_in_dim=cfg.value_in_dim if central else 0)
    # single-row calls (the log-probabilities below): the policy network with a per-row value net of zeros
    own = ref.Policy(cfg.obs_dim, cfg.hidden, cfg.out_dim, bf16=cfg.dtype == synth.BF16, dist=cfg.dist,
                     hidden_layers=cfg.hidden_layers)
    p_own = np.concatenate([params[:pol.policy_param_count], np.zeros(own.param_count - own.policy_param_count)])
    obs = rng.uniform(-1, 1, (R, cfg.obs_dim)).astype(np.float32)
    if cfg.kind == synth.PARTICLE:
        obs[:, 4 * cfg.num_agents + 2:] = 0.0      # the zero slots of the particle observation
        actions = rng.integers(0, 5, R).astype(np.int32)
    else:
        actions = rng.normal(0, 1, (R, cfg.act_dim)).astype(np.float32)
    adv = rng.normal(0, 1, R).astype(np.float32)
    ret = rng.normal(0, 1, R).astype(np.float32)
    pc = ref.ppo_cfg()
    logp_new = np.array([-ref.ppo_loss(own, pc, p_own, obs[n:n + 1], actions[n:n + 1], np.zeros(1), adv[n:n + 1],
                                       ret[n:n + 1], want_grad=False)[2][4] for n in range(R)])
    logp_old = (logp_new - rng.choice([-0.5, -0.1, 0.0, 0.1, 0.5], R)).astype(np.float32)
    return pol, obs, actions, logp_old, adv, ret


CASES = {
    "cfg1_f32": (synth.CONFIGS[1], 333),
    "cfg3_f32_ragged": (synth.CONFIGS[3], 517),
    "cfg4_gauss_f32": (synth.CONFIGS[4], 200),
    "p3_bf16": (synth.particle("p3b", 8, 3, 64, 4, 4, synth.BF16, 12), 300),
    "cfg5_bf16": (synth.CONFIGS[5], 259),
    # more than two hidden layers (the kernels that keep the activations in device memory)
    "cfg1_f32_4_layers": (synth.CONFIGS[1].with_(hidden_layers=4), 333),
    "cfg4_gauss_f32_3_layers": (synth.CONFIGS[4].with_(hidden_layers=3), 200),
    "p3_bf16_5_layers": (synth.particle("p3b", 8, 3, 64, 4, 4, synth.BF16, 12).with_(hidden_layers=5), 300),
    "cfg5_bf16_7_layers": (synth.CONFIGS[5].with_(hidden_layers=7), 131),
    "cfg5_bf16_many_tiles": (synth.CONFIGS[5], 32 * 4 * 5 + 17),
    "p6_bf16_h128": (synth.particle("p6b", 8, 6, 128, 4, 4, synth.BF16, 12), 150),
    # 64 units with more than 30 inputs: the on-chip weight gradients with two tiles of observation inputs
    "p6_bf16_h64": (synth.particle("p6c", 8, 6, 64, 4, 4, synth.BF16, 14), 32 * 9 + 5),
    "p10_bf16_h64": (synth.particle("p10c", 8, 10, 64, 4, 4, synth.BF16, 15), 217),
    # the pursuit task's learner with 32 inputs (5 chasers, 3 runners, no landmark): the two parts of the bias need a second
    # tile of inputs
    "tag_5_3_bf16": (synth.tag("t8", 8, 5, 3, 0, 64, 4, 4, synth.BF16, 16).with_(kind=synth.PARTICLE), 32 * 7 + 9),
    # the same bf16 networks through the kernels that keep the activations in device memory
    "p3_bf16_unfused": (synth.particle("p3b", 8, 3, 64, 4, 4, synth.BF16, 12), 300),
    "cfg5_bf16_unfused": (synth.CONFIGS[5], 259),
    # centralised critic: the value network on groups of num_agents consecutive rows (54 inputs: the row
    # kernel's weight panel; 600 inputs: the general kernels for layer 1 and its weight gradient)
    "p3_f32_central": (synth.particle("p3c", 8, 3, 64, 4, 4, synth.F32, 13).with_(central_critic=True), 3 * 111),
    "p3_bf16_central": (synth.particle("p3c", 8, 3, 64, 4, 4, synth.BF16, 13).with_(central_critic=True), 3 * 100),
    "cfg5_f32_central": (synth.CONFIGS[5].with_(dtype=synth.F32, central_critic=True), 10 * 17),
    "cfg5_bf16_central": (synth.CONFIGS[5].with_(central_critic=True), 10 * 26),
    "cfg5_bf16_central_4_layers": (synth.CONFIGS[5].with_(central_critic=True, hidden_layers=4), 10 * 60),
    # (bf16, two hidden layers: the policy network takes the on-chip path, the critic the one through device
    # memory; the same with both networks through device memory)
    "p3_bf16_central_unfused": (synth.particle("p3c", 8, 3, 64, 4, 4, synth.BF16, 13).with_(central_critic=True), 3 * 100),
    "cfg5_bf16_central_unfused": (synth.CONFIGS[5].with_(central_critic=True), 10 * 26),
    "cfg5_bf16_central_many_tiles": (synth.CONFIGS[5].with_(central_critic=True), 10 * 67),
}


@pytest.mark.parametrize("which", list(CASES))
def test_gradient_and_statistics_match_the_oracle(which):
    import torch
    from paper_2210_00882_amd import binding as B
    cfg, R = CASES[which]
    path = B.MSRL_LEARNER_PATH_DEVICE_MEMORY if which.endswith("_unfused") else B.MSRL_LEARNER_PATH_AUTO
    params = synth.make_params(cfg, bias_std=0.1).astype(np.float64)
    pol, obs, actions, logp_old, adv, ret = make_batch(cfg, R, 7, params)
    hp = dict(clip=0.2, vf_coef=0.7, ent_coef=0.03)
    loss, g_ref, st_ref = ref.ppo_loss(pol, ref.ppo_cfg(**hp), params, obs, actions, logp_old, adv, ret)
    L = B.msrl_learner_init_path(B.make_policy_cfg(cfg), R + 5, path)
    try:
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
        grad = torch.full((params.size,), 7.0, dtype=torch.float32, device="cuda")
        stats = torch.zeros(5, dtype=torch.float32, device="cuda")
        d = [dev(x) for x in (params.astype(np.float32), obs, actions, logp_old, adv, ret)]
        for _ in range(2):   # a second call must not see anything of the first
            B.msrl_ppo_grad(L, d[0], d[1], d[2], d[3], d[4], d[5], B.make_ppo_cfg(**hp), grad, stats)
        torch.cuda.synchronize()
        g, st = grad.cpu().numpy().astype(np.float64), stats.cpu().numpy().astype(np.float64) / R
        if cfg.central_critic:
            st[1] *= cfg.num_agents       # the value term is a sum over the R / num_agents groups
            with pytest.raises(B.MsrlError) as e:     # rows that are no whole groups
                B.msrl_ppo_grad(L, d[0], d[1][:R - 1], d[2][:R - 1], d[3][:R - 1], d[4][:R - 1], d[5][:R - 1],
                                B.make_ppo_cfg(**hp), grad, stats)
            assert e.value.code == B.MSRL_EINVAL
    finally:
        B.msrl_learner_destroy(L)
    tol = 2e-2 if cfg.dtype == synth.BF16 else 1e-4
    np.testing.assert_allclose(st[[0, 1, 2, 4]], st_ref[[0, 1, 2, 4]], rtol=tol, atol=tol)
    # make_batch puts every ratio at exp(+-0.5), exp(+-0.1) or 1, far from the clip edges 0.8 and 1.2:
    # the count of clipped rows is exact
    assert abs(st[3] - st_ref[3]) < 0.5 / R
    assert 0.1 < st_ref[3] < 0.9
    check_gradient_per_unit(which, cfg, pol, g, g_ref, tol)


def check_gradient_per_unit(which, cfg, pol, g, g_ref, tol):
    """Every entry of the gradient against the oracle, scaled by the largest entry of its output unit."""
    off = 0
    for o, width in ((cfg.out_dim, cfg.obs_dim), (1, pol.value_in_dim)):
        names, n = tensors_of(g_ref, width, cfg.hidden, o, cfg.hidden_layers)
        for (wname, wsl), (bname, bsl) in zip(names[0::2], names[1::2]):
            units = g_ref[off:off + n][bsl].size
            Wg, Wo = g[off:off + n][wsl].reshape(-1, units), g_ref[off:off + n][wsl].reshape(-1, units)
            bg, bo = g[off:off + n][bsl], g_ref[off:off + n][bsl]
            scale = np.maximum(np.abs(Wo).max(axis=0), np.abs(bo))
            assert np.abs(Wo).max() > 0
            errW = np.abs(Wg - Wo) / np.maximum(scale, 1e-30)[None, :]
            errb = np.abs(bg - bo) / np.maximum(scale, 1e-30)
            # a unit the oracle gives no gradient at all (scale 0) must be exactly zero on the GPU too
            assert (Wg[:, scale == 0] == 0).all() and (bg[scale == 0] == 0).all(), f"{which} {wname}: dead unit"
            live = scale > 0
            worst = max(errW[:, live].max(initial=0.0), errb[live].max(initial=0.0))
            assert worst <= tol, (f"{which} net out={o} {wname}/{bname}: worst per-unit error {worst:.3e} "
                                  f"(unit {int(np.argmax(np.maximum(errW.max(axis=0), errb) * live))})")
        off += n


def test_adam_step_and_update_loop():
    import torch
    from paper_2210_00882_amd import binding as B
    rng = np.random.default_rng(3)
    n = 1000
    p0, g = rng.normal(0, 1, n), rng.normal(0, 1e-2, n)
    m0, v0 = rng.normal(0, 1e-2, n), rng.uniform(0, 1e-4, n)
    hp = dict(lr=1e-2, beta1=0.9, beta2=0.999, adam_eps=1e-8)
    pr, mr, vr = p0.copy(), m0.copy(), v0.copy()
    ref.adam_step(ref.ppo_cfg(**hp), pr, mr, vr, g, 7)
    dev = lambda a: torch.from_numpy(a.astype(np.float32)).cuda()
    p, m, v = dev(p0), dev(m0), dev(v0)
    B.msrl_adam_step(p, m, v, dev(g), 7, B.make_ppo_cfg(**hp))
    torch.cuda.synchronize()
    np.testing.assert_allclose(p.cpu().numpy(), pr, rtol=1e-5, atol=1e-7)
    np.testing.assert_allclose(m.cpu().numpy(), mr, rtol=1e-5, atol=1e-9)
    np.testing.assert_allclose(v.cpu().numpy(), vr, rtol=1e-5, atol=1e-12)

    # the update loop = msrl_ppo_grad + msrl_adam_step per minibatch, in the oracle's order of blocks
    cfg, R = synth.CONFIGS[1], 3 * 97 + 5
    params = synth.make_params(cfg, bias_std=0.1).astype(np.float64)
    pol, obs, actions, logp_old, adv, ret = make_batch(cfg, R, 11, params)
    c = B.make_ppo_cfg(lr=1e-3)
    d = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (obs, actions, logp_old, adv, ret)]
    L = B.msrl_learner_init(B.make_policy_cfg(cfg), 97 + 5)
    try:
        pa = dev(params); ma = torch.zeros_like(pa); va = torch.zeros_like(pa)
        k = B.msrl_ppo_update(L, pa, ma, va, 0, 2, 3, d[0], d[1], d[2], d[3], d[4], c)
        pb = dev(params); mb = torch.zeros_like(pb); vb = torch.zeros_like(pb)
        gr = torch.empty_like(pb)
        kk = 0
        for it in range(2):
            for b in range(3):
                blk = R // 3
                sl = slice(blk * b, R if b == 2 else blk * b + blk)
                B.msrl_ppo_grad(L, pb, d[0][sl], d[1][sl], d[2][sl], d[3][sl], d[4][sl], c, gr)
                kk += 1
                B.msrl_adam_step(pb, mb, vb, gr, kk, c)
        torch.cuda.synchronize()
        assert k == 6
        # Same kernels on the same data, and the slices of every gradient are added in a fixed order: the same bits
        np.testing.assert_array_equal(pa.cpu().numpy(), pb.cpu().numpy())
        np.testing.assert_array_equal(ma.cpu().numpy(), mb.cpu().numpy())
        np.testing.assert_array_equal(va.cpu().numpy(), vb.cpu().numpy())
        # and the loop follows the oracle's loop: the loss of the updated parameters went down as the oracle's does
        po, mo, vo = params.copy(), np.zeros_like(params), np.zeros_like(params)
        ref.ppo_update(pol, ref.ppo_cfg(lr=1e-3), po, mo, vo, 0, 2, 3, obs, actions, logp_old, adv, ret)
        l0 = ref.ppo_loss(pol, ref.ppo_cfg(), params, obs, actions, logp_old, adv, ret, want_grad=False)[0]
        l_gpu = ref.ppo_loss(pol, ref.ppo_cfg(), pa.cpu().numpy().astype(np.float64), obs, actions, logp_old, adv, ret,
                             want_grad=False)[0]
        l_ref = ref.ppo_loss(pol, ref.ppo_cfg(), po, obs, actions, logp_old, adv, ret, want_grad=False)[0]
        assert l_ref < l0 and abs(l_gpu - l_ref) <= 0.02 * abs(l0 - l_ref) + 1e-6
        with pytest.raises(B.MsrlError) as e:   # a minibatch larger than the workspace
            B.msrl_ppo_update(L, pa, ma, va, k, 1, 1, d[0], d[1], d[2], d[3], d[4], c)
        assert e.value.code == B.MSRL_EINVAL
    finally:
        B.msrl_learner_destroy(L)


@pytest.mark.parametrize("which,path", [("cfg5_bf16", "auto"), ("cfg5_bf16", "device_memory"), ("cfg1_f32", "auto"),
                                        ("cfg5_bf16_central", "auto"), ("cfg5_bf16_7_layers", "auto")])
def test_gradient_is_the_same_bits_on_every_call(which, path):
    # The contractions over the rows are split over many workgroups; their shares are added in a fixed order
    # (no float atomics), so neither the order the workgroups finish in nor an earlier call changes a bit.
    import torch
    from paper_2210_00882_amd import binding as B
    cfg, _ = CASES[which]
    R = 3 * 12345 if not getattr(cfg, "central_critic", False) else 3 * 12345 // cfg.num_agents * cfg.num_agents
    rng = np.random.default_rng(17)
    params = torch.from_numpy(synth.make_params(cfg, bias_std=0.1).astype(np.float32)).cuda()
    obs = torch.from_numpy(rng.uniform(-1, 1, (R, cfg.obs_dim)).astype(np.float32)).cuda()
    actions = torch.from_numpy(rng.integers(0, 5, R).astype(np.int32)).cuda()
    f = lambda: torch.from_numpy(rng.normal(0, 1, R).astype(np.float32)).cuda()
    logp_old, adv, ret = f() * 0.1 - 1.6, f(), f()
    which_path = B.MSRL_LEARNER_PATH_AUTO if path == "auto" else B.MSRL_LEARNER_PATH_DEVICE_MEMORY
    got = []
    for learner in range(2):
        L = B.msrl_learner_init_path(B.make_policy_cfg(cfg), R, which_path)
        try:
            for call in range(3):
                grad = torch.full((params.numel(),), float("nan"), dtype=torch.float32, device="cuda")
                stats = torch.zeros(5, dtype=torch.float32, device="cuda")
                if call == 1:   # a smaller call in between leaves other shares in the workspace
                    r = R // 30 * 10
                    B.msrl_ppo_grad(L, params, obs[:r], actions[:r], logp_old[:r], adv[:r], ret[:r], B.make_ppo_cfg(),
                                    grad, stats)
                    continue
                B.msrl_ppo_grad(L, params, obs, actions, logp_old, adv, ret, B.make_ppo_cfg(), grad, stats)
                torch.cuda.synchronize()
                got.append(grad.cpu().numpy())
        finally:
            B.msrl_learner_destroy(L)
    assert np.isfinite(got[0]).all() and np.abs(got[0]).max() > 0
    for g in got[1:]:
        np.testing.assert_array_equal(g, got[0])


EDGE_CFGS = {
    "f32": synth.CONFIGS[1],
    # bf16: the path with the activations on chip (32-row tiles, 8 tiles per workgroup step)
    "bf16_h64": synth.particle("p3b", 8, 3, 64, 4, 4, synth.BF16, 12),
    "bf16_h256": synth.CONFIGS[5],
}


@pytest.mark.parametrize("which,R", [("f32", 1), ("f32", 17), ("f32", 256), ("bf16_h64", 1), ("bf16_h64", 31),
                                     ("bf16_h64", 32), ("bf16_h64", 33), ("bf16_h64", 256), ("bf16_h64", 257),
                                     ("bf16_h256", 1), ("bf16_h256", 64)])
def test_gradient_for_tiny_and_exactly_full_workspaces(which, R):
    import torch
    from paper_2210_00882_amd import binding as B
    cfg = EDGE_CFGS[which]
    params = synth.make_params(cfg, bias_std=0.1).astype(np.float64)
    pol, obs, actions, logp_old, adv, ret = make_batch(cfg, R, 21 + R, params)
    _, g_ref, st_ref = ref.ppo_loss(pol, ref.ppo_cfg(), params, obs, actions, logp_old, adv, ret)
    L = B.msrl_learner_init(B.make_policy_cfg(cfg), R)      # workspace of exactly R rows
    try:
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
        grad = torch.empty(params.size, dtype=torch.float32, device="cuda")
        stats = torch.zeros(5, dtype=torch.float32, device="cuda")
        B.msrl_ppo_grad(L, dev(params.astype(np.float32)), dev(obs), dev(actions), dev(logp_old), dev(adv), dev(ret),
                        B.make_ppo_cfg(), grad, stats)
        torch.cuda.synchronize()
        with pytest.raises(B.MsrlError) as e:     # one row more than the workspace holds
            B.msrl_ppo_grad(L, dev(params.astype(np.float32)), dev(np.zeros((R + 1, cfg.obs_dim), np.float32)),
                            dev(np.zeros(R + 1, np.int32)), dev(np.zeros(R + 1, np.float32)),
                            dev(np.zeros(R + 1, np.float32)), dev(np.zeros(R + 1, np.float32)), B.make_ppo_cfg(), grad)
        assert e.value.code == B.MSRL_EINVAL
    finally:
        B.msrl_learner_destroy(L)
    g = grad.cpu().numpy().astype(np.float64)
    tol = 2e-2 if cfg.dtype == synth.BF16 else 1e-4
    np.testing.assert_allclose(stats.cpu().numpy()[[0, 1, 2]] / R, st_ref[[0, 1, 2]], rtol=tol, atol=tol)
    check_gradient_per_unit(f"{which} R={R}", cfg, pol, g, g_ref, tol)


def test_observation_rows_at_an_address_that_is_not_16_byte_aligned():
    # the on-chip path reads observation rows in 16-byte pieces only when the buffer allows it
    import torch
    from paper_2210_00882_amd import binding as B
    cfg, R = synth.CONFIGS[5], 70
    params = synth.make_params(cfg, bias_std=0.1).astype(np.float64)
    pol, obs, actions, logp_old, adv, ret = make_batch(cfg, R, 5, params)
    _, g_ref, _ = ref.ppo_loss(pol, ref.ppo_cfg(), params, obs, actions, logp_old, adv, ret)
    L = B.msrl_learner_init(B.make_policy_cfg(cfg), R)
    try:
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
        flat = torch.zeros(R * cfg.obs_dim + 4, dtype=torch.float32, device="cuda")
        flat[1:1 + R * cfg.obs_dim] = dev(obs).reshape(-1)
        shifted = flat[1:1 + R * cfg.obs_dim].view(R, cfg.obs_dim)
        assert shifted.data_ptr() % 16 == 4
        grad = torch.empty(params.size, dtype=torch.float32, device="cuda")
        B.msrl_ppo_grad(L, dev(params.astype(np.float32)), shifted, dev(actions), dev(logp_old), dev(adv), dev(ret),
                        B.make_ppo_cfg(), grad)
        torch.cuda.synchronize()
    finally:
        B.msrl_learner_destroy(L)
    g = grad.cpu().numpy().astype(np.float64)
    check_gradient_per_unit("unaligned rows", cfg, pol, g, g_ref, 2e-2)


@pytest.mark.parametrize("layers", [2, 4])
def test_training_loop_improves_the_linear_gaussian_task(layers):
    # Trainer.train of Listing 1 end to end on the device: rollout + GAE, then the learner's update,
    # repeated.  The reward -(|s|^2 + 0.01 |a|^2) punishes the large actions of the initial policy;
    # eighty iterations must at least halve the cost per step (typically it falls 10x or more).
    from paper_2210_00882_amd import train
    cfg = synth.CONFIGS[4].with_(num_envs=2048, T=64, episode_len=64, hidden_layers=layers)
    params = synth.make_params(cfg, bias_std=0.0, seed=5)
    _, hist = train.ppo_train(cfg, params, 80, 123, lr=1e-3, gamma=0.95, lam=0.95, dyn=synth.make_dynamics(cfg))
    first, last = np.mean(hist[:5]), np.mean(hist[-5:])
    assert np.isfinite(hist).all()
    assert first < 0 and last < 0 and last > first / 2.0, (first, last)


def test_params_cast_rounds_to_nearest_even():
    import torch
    from paper_2210_00882_amd import binding as B
    x = np.random.default_rng(0).normal(0, 1, 4099).astype(np.float32)
    d = torch.from_numpy(x).cuda()
    o16 = torch.empty(x.size, dtype=torch.bfloat16, device="cuda")
    o32 = torch.empty(x.size, dtype=torch.float32, device="cuda")
    B.msrl_params_cast(d, o16, B.MSRL_BF16)
    B.msrl_params_cast(d, o32, B.MSRL_F32)
    torch.cuda.synchronize()
    want = np.array([ref.bf16_round(float(t)) for t in x])
    np.testing.assert_array_equal(o16.float().cpu().numpy().astype(np.float64), want)
    np.testing.assert_array_equal(o32.cpu().numpy(), x)
