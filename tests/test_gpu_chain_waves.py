"""Actor chains of 32 rows run on eight wavefronts where every workgroup has a CU to itself (32 agents at most), on four
beyond: the sums are in the same order, so an agent's trajectory is the same bit for bit in either population."""
import numpy as np
import pytest

import paper_2206_08888_amd as pp
from gpu_common import ensure_built

pytestmark = pytest.mark.gpu


def _states(algo, P, O, A, agents):
    sac = algo == pp.POP_ALGO_SAC
    hps = [dict(seed=3 + i, lr_actor=3e-4, lr_critic=3e-4, gamma=0.99, tau=0.005, policy_noise=0.2, noise_clip=0.5,
                policy_delay=1, adam_b1=0.9, adam_b2=0.999, adam_eps=1e-8, lr_alpha=3e-4,
                target_entropy=-1.0 if sac else 0.0, init_log_alpha=0.0) for i in range(P)]
    cfg = pp.make_config(P, O, A, (256, 256), 256, 300, algo=algo, launch=pp.POP_LAUNCH_PER_PART, rows=32, half_tiles=1)
    pop = pp.Population(cfg, hps)
    for i in range(P):
        rng = np.random.default_rng(100 + i)
        f = lambda *s: rng.standard_normal(s).astype(np.float32)
        pop.insert(i, obs=f(300, O), act=np.tanh(f(300, A)), rew=f(300), done=(f(300) > 2).astype(np.float32), next_obs=f(300, O))
    pop.update(3)
    out = [[pop.get_params(i, code) for code in range(12)] for i in agents]
    pop.close()
    return out


# first layers narrow and wide, heads of one block of columns, of several (SAC: 2 A), up to the widest
@pytest.mark.parametrize("algo,O,A", [(pp.POP_ALGO_TD3, 17, 6), (pp.POP_ALGO_TD3, 3, 1), (pp.POP_ALGO_TD3, 64, 8),
                                      (pp.POP_ALGO_TD3, 20, 24), (pp.POP_ALGO_TD3, 111, 8), (pp.POP_ALGO_SAC, 17, 6),
                                      (pp.POP_ALGO_SAC, 20, 9), (pp.POP_ALGO_SAC, 20, 24), (pp.POP_ALGO_SAC, 111, 17)])
def test_actor_chains_of_four_and_eight_wavefronts(algo, O, A):
    ensure_built()
    agents = (0, 16)
    eight, four = _states(algo, 17, O, A, agents), _states(algo, 33, O, A, agents)
    for a, b in zip(eight, four):
        for code in range(12):
            assert np.isfinite(a[code]).all()
            assert np.array_equal(a[code], b[code]), code
