"""The learner's layer kernels (activations in device memory) where their launches split: many row tiles to a workgroup, more
contractions of a network than one launch takes."""
import numpy as np
import pytest

from oracle import ref
from paper_2210_00882_amd import synth
from test_gpu_learner import check_gradient_per_unit

pytestmark = pytest.mark.gpu


def gradient(pol, params, batch, path):
    import torch
    from paper_2210_00882_amd import binding as B
    L = B.msrl_learner_init_path(pol, len(batch[0]), path)
    try:
        d = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (params.astype(np.float32),) + batch]
        grad = torch.full((params.size,), 7.0, dtype=torch.float32, device="cuda")
        B.msrl_ppo_grad(L, *d, B.make_ppo_cfg(), grad, torch.zeros(5, dtype=torch.float32, device="cuda"))
        torch.cuda.synchronize()
        return grad.cpu().numpy().astype(np.float64)
    finally:
        B.msrl_learner_destroy(L)


def rows(rng, R, width):
    return (rng.uniform(-1, 1, (R, width)).astype(np.float32), rng.integers(0, 5, R).astype(np.int32),
            rng.normal(-1.6, 0.1, R).astype(np.float32), rng.normal(0, 1, R).astype(np.float32), rng.normal(0, 1, R).astype(np.float32))


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("groups,times", [(520, 32), (257, 256)])
def test_repeated_rows_leave_the_gradient(dtype, groups, times):
    # 65 and 257 tiles of 256 rows of the value network (600 inputs; 64 columns to a workgroup in bf16), 650 and 2570 of
    # the policy network: several tiles to a workgroup, the last one ragged.  The rows `times` over have the gradient of
    # the rows themselves; the scale of a row's share is 1 / times exactly (a power of two), so only the order of the
    # fp32 sums differs: at most some 600 roundings of 2^-24 in a chain (a slice's products, the slices), 4e-5 of the
    # sum of the shares' magnitudes, which for independent rows is sqrt(rows) = 23 times their sum: 1e-3.  A tile left
    # out or taken twice is some 1/65 or 1/257 of the gradient: 1.5e-2, 4e-3.
    from paper_2210_00882_amd import binding as B
    cfg = synth.CONFIGS[5].with_(dtype=dtype, central_critic=True)
    params = synth.make_params(cfg, bias_std=0.1)
    batch = rows(np.random.default_rng(5), 10 * groups, cfg.obs_dim)
    once, many = (gradient(B.make_policy_cfg(cfg), params, tuple(np.concatenate([a] * n) for a in batch),
                           B.MSRL_LEARNER_PATH_DEVICE_MEMORY) for n in (1, times))
    pol = ref.Policy(cfg.obs_dim, cfg.hidden, cfg.out_dim, bf16=dtype == synth.BF16, value_in_dim=cfg.value_in_dim)
    check_gradient_per_unit("repeated", cfg, pol, many, once, 1e-3)


@pytest.mark.parametrize("dtype,tol", [(synth.F32, 1e-4), (synth.BF16, 2e-2)])
@pytest.mark.parametrize("agents", [102, 103, 112])
def test_critics_with_more_contractions_than_a_launch(dtype, tol, agents):
    # 24, 25 and 27 panels of 256 inputs, where a launch takes 24 contractions (tolerances of test_gpu_learner.py)
    from paper_2210_00882_amd import binding as B
    cfg = synth.particle("wide", 8, 10, 64, 4, 4, dtype, 12)
    pol = ref.Policy(cfg.obs_dim, cfg.hidden, cfg.out_dim, bf16=dtype == synth.BF16, value_in_dim=agents * cfg.obs_dim)
    rng = np.random.default_rng(agents)
    params = rng.normal(0, 0.05, pol.param_count)
    params = params.astype(np.float32).astype(np.float64)
    batch = rows(rng, 33 * agents, cfg.obs_dim)
    _, g_ref, _ = ref.ppo_loss(pol, ref.ppo_cfg(), params, *batch)
    mine = B.make_policy_cfg(cfg)
    mine.value_in_dim = agents * cfg.obs_dim
    check_gradient_per_unit("wide", cfg, pol, gradient(mine, params, batch, B.MSRL_LEARNER_PATH_AUTO), g_ref, tol)
