"""Waves of a rollout workgroup that own no rows skip the networks: few envs for the chip, or a last round of smaller
workgroups behind full ones.  An env's trajectory
depends on the seed, its index and the parameters only, so it is the same bits whether the other waves of its workgroup
have rows or not; the reference is a run of full workgroups, where every wave has rows (checked against the oracle in
test_gpu_parity.py, like the shapes here at 50 envs)."""
import numpy as np
import pytest

from paper_2210_00882_amd import synth
from helpers import GpuRollout, oracle_setup

pytestmark = pytest.mark.gpu

CUS = 256  # workgroups of one round


def _run(cfg, T):
    _, _, params, _ = oracle_setup(cfg)
    import torch
    with GpuRollout(cfg, params.astype(np.float32), 77, wave_roles=1) as gpu:
        out = [gpu.run(T, gae=False), gpu.run(T, gae=False)]
        B = gpu.B
        one = B.alloc_traj(cfg, 1, gae=False)
        step = {k: one[k][0] for k in ("obs", "actions", "logp", "values")}
        B.msrl_observe(gpu.state, step["obs"])
        B.msrl_act(gpu.state, gpu.params, step["obs"], step["actions"], step["logp"], step["values"])
        torch.cuda.synchronize()
        out.append({k: v.cpu().numpy()[None] for k, v in step.items()})
        es, g = gpu.get_state()
    return out, es, g


@pytest.mark.parametrize("N,H,dtype,layers,central", [
    (10, 256, synth.BF16, 2, False), (3, 256, synth.BF16, 2, False), (6, 128, synth.BF16, 2, False),
    (6, 128, synth.F32, 2, False), (8, 256, synth.BF16, 3, False), (5, 128, synth.BF16, 6, False),
    (10, 256, synth.BF16, 2, True), (7, 256, synth.BF16, 2, True)])
def test_waves_without_rows_leave_the_others_bits(N, H, dtype, layers, central):
    epw = 32 // N
    T = 4

    def cfg(E):
        c = synth.particle("few", E, N, H, T, 3, dtype=dtype, idx=33)
        return c.with_(hidden_layers=layers, central_critic=central)

    full, es, g = _run(cfg(CUS * 24 * epw), T)  # three rounds of full workgroups, of up to eight waves
    # one env in all; one per workgroup; one full wave and one env; three waves, the last workgroup with fewer envs;
    # seven waves and one env in the eighth; one full round and five envs; two and one of three waves
    for E in (1, CUS + 1, CUS * (epw + 1), CUS * (2 * epw + 1) - 3, CUS * (7 * epw + 1), CUS * 8 * epw + 5, CUS * (18 * epw + 1) - 3):
        got, es1, g1 = _run(cfg(E), T)
        for a, b in zip(got, full):
            for k in a:
                if a[k] is not None:
                    np.testing.assert_array_equal(a[k], b[k][:, :E * N], err_msg=f"{k}, {E} envs")
        np.testing.assert_array_equal(es1, es[:E])
        np.testing.assert_array_equal(g1, g[:E])
