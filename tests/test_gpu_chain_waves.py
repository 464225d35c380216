"""Chains of 32 rows exist on four wavefronts and on eight: eight where a workgroup has a CU to itself, because the launch has
no more workgroups than the chip has CUs (target and actor chains up to 32 agents, critic chains up to 16) or because LDS or
registers leave no other choice.  The sums are in the same order, so an agent's trajectory is the same bit for bit on either.
Each case names two launches that differ in the wavefronts of the chains it lists; chains that only ever run on eight (actor chains
of wide inputs, of wide actions and of SAC, SAC's target chains of wide inputs) have no counterpart to be compared with here and are held
to the oracle by the tests of their shapes.  (64 rows: test_sixty_four_row_chains_match_oracle_and_each_other.)"""
import numpy as np
import pytest

import paper_2206_08888_amd as pp
from gpu_common import ensure_built

pytestmark = pytest.mark.gpu

CRITICS = (1, 2, 4, 5, 7, 8, 10, 11)                   # parameters, targets and moments of both critics


def _states(algo, P, O, A, codes, launch=pp.POP_LAUNCH_PER_PART, gamma=0.99):
    sac = algo == pp.POP_ALGO_SAC
    hps = [dict(seed=3 + i, lr_actor=3e-4, lr_critic=3e-4, gamma=gamma, tau=0.005, policy_noise=0.2, noise_clip=0.5,
                policy_delay=1, adam_b1=0.9, adam_b2=0.999, adam_eps=1e-8, lr_alpha=3e-4,
                target_entropy=-1.0 if sac else 0.0, init_log_alpha=0.0) for i in range(P)]
    cfg = pp.make_config(P, O, A, (256, 256), 256, 300, algo=algo, launch=launch, rows=32, half_tiles=1)
    pop = pp.Population(cfg, hps)
    for i in range(P):
        rng = np.random.default_rng(100 + i)
        f = lambda *s: rng.standard_normal(s).astype(np.float32)
        pop.insert(i, obs=f(300, O), act=np.tanh(f(300, A)), rew=f(300), done=(f(300) > 2).astype(np.float32), next_obs=f(300, O))
    pop.update(3)
    out = [[pop.get_params(i, code) for code in codes] for i in (0, min(P, 16) - 1)]
    pop.close()
    return out


def _same(a, b, codes):
    for x, y in zip(a, b):
        for code, u, v in zip(codes, x, y):
            assert np.isfinite(u).all() and np.array_equal(u, v), code


@pytest.mark.parametrize("O,A", [(17, 6), (3, 1), (56, 8)])
def test_narrow_chains(O, A):
    """16 agents: target, critic and actor chains on eight wavefronts; 17: the critic chains on four; 33: all on four."""
    ensure_built()
    codes = range(12)
    eight = _states(pp.POP_ALGO_TD3, 16, O, A, codes)
    _same(eight, _states(pp.POP_ALGO_TD3, 17, O, A, codes), codes)
    _same(eight, _states(pp.POP_ALGO_TD3, 33, O, A, codes), codes)


@pytest.mark.parametrize("O,A", [(59, 6), (104, 8), (20, 24)])
def test_wide_target_chains(O, A):
    """17 agents: target chains of wide inputs (65, and 112: the last whose LDS lets two workgroups share a CU) and of wide actions on
    eight wavefronts; 33: on four."""
    ensure_built()
    codes = range(12)
    _same(_states(pp.POP_ALGO_TD3, 17, O, A, codes), _states(pp.POP_ALGO_TD3, 33, O, A, codes), codes)


@pytest.mark.parametrize("O,A", [(59, 6), (111, 8), (319, 17)])
def test_wide_critic_chains(O, A):
    """16 agents: critic chains of wide inputs (up to 336, the last whose LDS lets two workgroups share a CU) on eight wavefronts, slabs beside
    the input tile; 17: on four, slabs over it.  The target and actor chains take other rows there, so with a discount of zero, where
    the critics depend on neither."""
    ensure_built()
    _same(_states(pp.POP_ALGO_TD3, 16, O, A, CRITICS, gamma=0.0), _states(pp.POP_ALGO_TD3, 17, O, A, CRITICS, gamma=0.0), CRITICS)


@pytest.mark.parametrize("O,A", [(17, 6), (20, 9), (20, 24)])
def test_sac_target_and_critic_chains(O, A):
    """Launches of their own: on eight wavefronts; in one launch: on four."""
    ensure_built()
    codes = (*range(12), 15)
    eight = _states(pp.POP_ALGO_SAC, 4, O, A, codes)
    _same(eight, _states(pp.POP_ALGO_SAC, 4, O, A, codes, launch=pp.POP_LAUNCH_TARGET_CRITIC), codes)
