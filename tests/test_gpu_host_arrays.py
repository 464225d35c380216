"""Host arrays of a whole population: inserts and actions in one copy per array or piecewise, and the exploit / explore
calls, against the same calls with device arrays or agent by agent."""
import numpy as np
import pytest

import paper_2206_08888_amd as pp
from gpu_common import ensure_built

pytestmark = pytest.mark.gpu
STAGING = 16 << 20


def _population(algo, P, O, A, capacity):
    ensure_built()
    sac = algo == pp.POP_ALGO_SAC
    hps = [dict(seed=7 + i, lr_actor=3e-4, lr_critic=3e-4, gamma=0.99, tau=0.005, policy_noise=0.2, noise_clip=0.5,
                policy_delay=1 if sac else 2, adam_b1=0.9, adam_b2=0.999, adam_eps=1e-8, lr_alpha=3e-4,
                target_entropy=-float(A) if sac else 0.0, init_log_alpha=0.1 * i) for i in range(P)]
    return pp.Population(pp.make_config(P, O, A, (256, 256), 256, capacity, algo=algo), hps), hps


# rows that just fit the staging area with all agents, one more, and more rows than the ring holds
@pytest.mark.parametrize("P,O,A,n,capacity", [(1, 3, 1, 1, 1000), (3, 17, 6, 50, 1000), (2, 11, 3, 1500, 1000),
                                              (2, 376, 17, STAGING // (771 * 4) // 2, 3000), (2, 376, 17, STAGING // (771 * 4) // 2 + 1, 3000)])
def test_host_arrays_like_device_arrays(P, O, A, n, capacity):
    import torch
    g = np.random.default_rng(n)
    tr = dict(obs=g.standard_normal((P, n, O)), act=g.uniform(-1, 1, (P, n, A)), rew=g.standard_normal((P, n)), done=np.zeros((P, n)),
              next_obs=g.standard_normal((P, n, O)))
    tr = {k: v.astype(np.float32) for k, v in tr.items()}
    sigma = np.linspace(0.1, 0.2, P).astype(np.float32)
    got = []
    for host in (True, False):
        pop, _ = _population(pp.POP_ALGO_TD3, P, O, A, capacity)
        for _ in range(2):
            pop.insert(-1, **(tr if host else {k: torch.from_numpy(v).cuda() for k, v in tr.items()}))
        a = pop.act(tr["obs"] if host else torch.from_numpy(tr["obs"]).cuda(), sigma, step=5)
        pop.update(3)
        got.append((a if host else a.cpu().numpy(), [pop.get_params(i, net) for i in range(P) for net in ("actor", "critic1", "t_critic2")]))
        pop.close()
    assert np.array_equal(got[0][0], got[1][0])
    assert all(np.array_equal(x, y) for x, y in zip(got[0][1], got[1][1]))


@pytest.mark.parametrize("algo", [pp.POP_ALGO_TD3, pp.POP_ALGO_SAC, pp.POP_ALGO_TD3_SHARED])
def test_copy_agent_copies_all_an_agent_owns(algo):
    """Right behind update calls, without a synchronisation of the caller's."""
    O, A, P, n = 17, 6, 3, 64
    pop, hps = _population(algo, P, O, A, 200)
    g = np.random.default_rng(1)
    pop.insert(-1, obs=g.standard_normal((P, n, O)).astype(np.float32), act=g.uniform(-1, 1, (P, n, A)).astype(np.float32),
               rew=g.standard_normal((P, n)).astype(np.float32), done=np.zeros((P, n), np.float32), next_obs=g.standard_normal((P, n, O)).astype(np.float32))
    pop.update(4)
    nets = ("actor",) if algo == pp.POP_ALGO_TD3_SHARED else ("actor", "critic1", "critic2")
    codes = [pre + net for pre in ("", "t_", "m_", "v_") for net in nets if not (algo == pp.POP_ALGO_SAC and pre + net == "t_actor")]
    codes += ["log_alpha", "m_log_alpha", "v_log_alpha"] if algo == pp.POP_ALGO_SAC else []
    others = [pop.get_params(0, c) for c in codes]
    pop.copy_agent(2, 1, False)
    pop.set_hparams(2, dict(hps[2], lr_actor=1e-3))
    for c, o in zip(codes, others):
        assert np.array_equal(pop.get_params(2, c), pop.get_params(1, c)), c
        assert np.array_equal(pop.get_params(0, c), o), c
    pop.update(2)
    assert not np.array_equal(pop.get_params(2, "actor"), pop.get_params(1, "actor"))
    pop.close()
