"""The gradient in one kernel (learn_block.h, learn_block_bf16.h) against the layer-by-layer kernels, which test_gpu_learner.py checks
against the oracle: sizes at the edges of its row tiles (32 and 64 rows), slices and operand tiles."""
import numpy as np
import pytest
import torch

from paper_2210_00882_amd import binding as B, synth

pytestmark = pytest.mark.gpu


def policy(d, h, o, gauss, dtype=synth.F32):
    p = B.make_policy_cfg(synth.CONFIGS[1])
    p.in_dim, p.hidden, p.out_dim, p.dist, p.dtype = d, h, o, synth.DIAG_GAUSSIAN if gauss else synth.CATEGORICAL, dtype
    p.hidden_layers, p.value_in_dim, p.roles = 0, 0, 1
    return p


def weights(n_in, h, o, g):
    t = lambda i, k: torch.randn((i, k), device="cuda", generator=g) / i ** 0.5
    b = lambda k: 0.1 * torch.randn(k, device="cuda", generator=g)
    return torch.cat([x.reshape(-1) for x in (t(n_in, h), b(h), t(h, h), b(h), t(h, o), b(o))])


def gradients(pol, R, path, rows=None, seed=3):
    """Gradient and statistics of R rows (of a larger array, if `rows` selects them); the same inputs for both paths."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    d, h, o = pol.in_dim, pol.hidden, pol.out_dim
    params = torch.cat([weights(d, h, o, g), weights(d, h, 1, g)])
    assert params.numel() == B.msrl_param_count(pol)
    M = R if rows is None else R // rows.count * rows.group
    f = lambda *s: torch.randn(s, device="cuda", generator=g)
    actions = f(M, o // 2) if pol.dist == synth.DIAG_GAUSSIAN else torch.randint(0, o, (M,), device="cuda", generator=g, dtype=torch.int32)
    # (logp_old near the policy's own values: ratios around 1, clipped and unclipped rows)
    logp = -float(np.log(o)) + 0.3 * f(M) if pol.dist != synth.DIAG_GAUSSIAN else -0.5 * (actions ** 2).sum(1) - 0.9189 * (o // 2) + 0.3 * f(M)
    batch = [f(M, d), actions, logp, f(M), f(M)]
    L = B.msrl_learner_init_path(pol, R, path)
    grad, stats = torch.full_like(params, float("nan")), torch.empty(5, device="cuda")
    try:
        B.msrl_ppo_grad(L, params, *batch, B.make_ppo_cfg(), grad, stats, rows=rows)
        torch.cuda.synchronize()
    finally:
        B.msrl_learner_destroy(L)
    return grad, stats


# in_dim, hidden, out_dim: one and two 32-input tiles, full and ragged; one and two 16-output tiles
SHAPES = [(17, 256, 12, True), (64, 256, 32, True), (33, 128, 18, True), (8, 64, 2, True),
          (18, 64, 5, False), (60, 64, 32, False), (32, 128, 16, False), (33, 256, 17, False), (1, 256, 1, False)]


@pytest.mark.parametrize("d,h,o,gauss", SHAPES)
@pytest.mark.parametrize("R", [1, 31, 33, 64, 65, 513, 9001])
def test_block_kernel_equals_the_layer_kernels(d, h, o, gauss, R):
    pol = policy(d, h, o, gauss)
    g, st = gradients(pol, R, 0)
    g_ref, st_ref = gradients(pol, R, 1)
    assert torch.isfinite(g).all()
    if gauss:
        assert torch.equal(g, g_ref)  # the same slices, every sum in the same order
    else:
        # other slices: sums of up to 9001 products in another order, each 2^-24 off at most, at random: 2^-24 sqrt(R)
        # of the terms' size; that is a few times the sum's own where the terms cancel
        assert (g - g_ref).double().norm() <= 4e-6 * g_ref.double().norm()
    assert torch.allclose(st, st_ref, rtol=1e-4, atol=1e-4 * R ** 0.5)


@pytest.mark.parametrize("d,h,o", [(60, 256, 5), (17, 256, 16), (33, 128, 3), (1, 128, 1), (18, 64, 5), (63, 64, 16), (64, 64, 2)])
@pytest.mark.parametrize("R", [1, 63, 65, 513, 9001])
def test_bf16_block_kernel_equals_the_layer_kernels(d, h, o, R):
    pol = policy(d, h, o, False, synth.BF16)
    g, st = gradients(pol, R, 0)
    g_ref, st_ref = gradients(pol, R, 1)
    assert torch.isfinite(g).all()
    # the same rounding points; where two sums differ by an fp32 rounding next to a bf16 boundary, one activation in
    # about 2^15 (16 bits between the two) is off by 2^-8: 2^-8 / sqrt(2^15) = 2e-5 of the sum, and a few bytes of
    # cancelling terms on top of that
    assert (g - g_ref).double().norm() <= 5e-3 * g_ref.double().norm()
    assert torch.allclose(st, st_ref, rtol=1e-2, atol=1e-2 * R ** 0.5)


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("first,count", [(0, 3), (3, 1), (1, 2)])
def test_block_kernel_reads_selected_rows(first, count, dtype):
    pol = policy(18, 64, 5, False, dtype)
    sel = B.msrl_row_select(4, first, count)
    g, st = gradients(pol, 1000 * count, 0, rows=sel)
    g_ref, st_ref = gradients(pol, 1000 * count, 1, rows=sel)
    assert (g - g_ref).double().norm() <= (4e-6 if dtype == synth.F32 else 5e-3) * g_ref.double().norm()
    assert torch.allclose(st, st_ref, rtol=1e-4 if dtype == synth.F32 else 1e-2, atol=1e-2 if dtype == synth.F32 else 0.5)


def test_bf16_block_kernel_reads_observations_at_an_odd_address():
    pol = policy(18, 64, 5, False, synth.BF16)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    R = 200
    params = torch.cat([weights(18, 64, 5, g), weights(18, 64, 1, g)])
    obs = torch.randn(R * 18 + 1, device="cuda", generator=g)
    rest = [torch.randint(0, 5, (R,), device="cuda", dtype=torch.int32, generator=g)] + [torch.randn(R, device="cuda", generator=g) for _ in range(3)]
    out = []
    for x in (obs[1:].view(R, 18), obs[1:].clone().view(R, 18)):  # 4 bytes off, and 8-byte aligned
        L = B.msrl_learner_init(pol, R)
        out.append(torch.empty_like(params))
        B.msrl_ppo_grad(L, params, x, *rest, B.make_ppo_cfg(), out[-1])
        torch.cuda.synchronize()
        B.msrl_learner_destroy(L)
    assert torch.equal(*out)
