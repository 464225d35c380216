"""The target / critic launch of a few agents (target critics in workgroups of their own up to 5 agents, the actor's forward
pass beside them up to 4) and of wide inputs or actions -- all bit for bit what one launch per part computes."""
import numpy as np
import pytest
import torch

import paper_2206_08888_amd as pp
import workloads
from gpu_common import STATE12, ensure_built

pytestmark = pytest.mark.gpu


def _states(algo, P, O, A, **kw):
    hps = workloads.hparams(2, P)
    for i, h in enumerate(hps):
        h["policy_delay"] = 2 if algo == pp.POP_ALGO_TD3_SHARED else 1 + (i + 1) % 3
    kw.setdefault("launch", pp.POP_LAUNCH_TARGET_CRITIC)
    pop = pp.Population(pp.make_config(P, O, A, (256, 256), 256, 300, algo=algo, **kw), hps)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(O)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda")
    pop.insert(-1, obs=rnd(P, 300, O), act=rnd(P, 300, A).clamp(-1, 1), rew=rnd(P, 300), done=(rnd(P, 300) > 2).float(), next_obs=rnd(P, 300, O))
    pop.update(2)
    ms, cnt = pop.update_timed(5)
    sac = algo == pp.POP_ALGO_SAC
    codes = [w for w in STATE12 if not (sac and w == "t_actor")] + (["log_alpha"] if sac else [])
    out = {(i, w): pop.get_params(i, w) for i in range(P) for w in codes}
    out.update({w: pop.debug(w) for w in ("target_y", "target_action", "losses")})
    pop.sync()
    pop.close()
    return out, cnt


@pytest.mark.parametrize("algo, P, O, A", [
    ("td3", 17, 376, 17), ("td3", 20, 111, 8), ("td3", 33, 30, 20), ("td3_shared", 18, 336, 1), ("td3", 24, 424, 24),  # 32-row chains
    ("sac", 1, 17, 6), ("sac", 5, 40, 24), ("sac", 6, 9, 9), ("sac", 3, 424, 24), ("sac", 5, 64, 1), ("sac", 8, 447, 1),
    ("sac", 17, 376, 17), ("sac", 33, 65, 8),
    ("td3", 1, 17, 6), ("td3", 4, 60, 4), ("td3", 5, 1, 1), ("td3_shared", 3, 17, 6),          # narrow: both, both, targets only
    ("td3", 1, 64, 1), ("td3", 4, 424, 24), ("td3", 5, 40, 9), ("td3_shared", 2, 9, 24),       # wide inputs, wide actions, both
    ("td3", 6, 447, 1), ("td3", 8, 65, 8), ("td3", 8, 30, 20), ("td3_shared", 8, 111, 8)])     # fused only
def test_against_one_launch_per_part(algo, P, O, A):
    ensure_built()
    code = {"td3": pp.POP_ALGO_TD3, "td3_shared": pp.POP_ALGO_TD3_SHARED, "sac": pp.POP_ALGO_SAC}[algo]
    want, apart = _states(code, P, O, A, launch=pp.POP_LAUNCH_PER_PART)
    assert apart["target"] == apart["critic"] == 5 and apart["target_critic"] == 0
    for ahead in (0, 1):
        got, cnt = _states(code, P, O, A, actor_ahead=ahead)
        assert cnt["target_critic"] == 5 and cnt["target"] == cnt["critic"] == 0
        assert all(np.array_equal(got[k], want[k]) for k in want), [k for k in want if not np.array_equal(got[k], want[k])][:4]


@pytest.mark.parametrize("algo, P, O, A, apart", [("td3", 1, 17, 6, True), ("td3", 5, 17, 6, True), ("td3", 6, 17, 6, False), ("td3", 5, 111, 8, True), ("td3", 6, 111, 8, False),
                                                  ("sac", 5, 17, 6, True), ("sac", 6, 17, 6, False), ("sac", 2, 376, 17, True), ("td3_shared", 5, 40, 9, True)])
def test_what_the_target_workgroups_publish(algo, P, O, A, apart):
    """One value of each target critic where they have workgroups of their own, y where one workgroup runs both: of all words of the workspace, those with the
    step's tag over the bits of y are there in the second case only."""
    ensure_built()
    code = {"td3": pp.POP_ALGO_TD3, "td3_shared": pp.POP_ALGO_TD3_SHARED, "sac": pp.POP_ALGO_SAC}[algo]
    pop = pp.Population(pp.make_config(P, O, A, (256, 256), 256, 300, algo=code), workloads.hparams(2, P))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(O)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda")
    pop.insert(-1, obs=rnd(P, 300, O), act=rnd(P, 300, A).clamp(-1, 1), rew=rnd(P, 300), done=(rnd(P, 300) > 2).float(), next_obs=rnd(P, 300, O))
    pop.update(400)
    y = pop.debug("target_y")
    words = (400 << 32) | torch.from_numpy(np.ascontiguousarray(y).view(np.uint32).astype(np.int64)).flatten()
    ws = pop.workspace[:pop.workspace.numel() // 8 * 8].view(torch.int64)
    found = int(torch.isin(words.cuda(), ws).sum())
    assert (found <= 4) if apart else found == P * 256, found      # (a y that happens to be some critic's value)
    pop.close()


def test_the_first_population_whose_wide_chains_have_launches_of_their_own():
    fused, apart = pp.POP_LAUNCH_TARGET_CRITIC, pp.POP_LAUNCH_PER_PART
    sac = pp.Population(pp.make_config(20, 111, 8, (256, 256), 256, 64, algo=pp.POP_ALGO_SAC), workloads.hparams(5, 20))
    assert sac.tuning()["launch"] == fused
    sac.close()
    for P, O, launch in ((8, 111, fused), (9, 111, apart), (16, 376, apart), (20, 111, fused), (21, 111, apart), (32, 111, apart), (33, 111, fused),
                         (52, 111, fused), (53, 111, apart), (80, 111, fused), (81, 111, apart), (32, 328, apart), (32, 329, fused), (17, 376, fused)):
        pop = pp.Population(pp.make_config(P, O, 8, (256, 256), 256, 64), workloads.hparams(2, P))
        assert pop.tuning()["launch"] == launch, (P, O)
        pop.close()


@pytest.mark.parametrize("P, launch, rows", [
    (3, "POP_LAUNCH_SINGLE", None), (3, "POP_LAUNCH_TAIL", None), (20, "POP_LAUNCH_SINGLE", None), (3, "POP_LAUNCH_TARGET_CRITIC", (64, 64, 64)),
    (3, "POP_LAUNCH_TARGET_CRITIC", (32, 64, 32)), (3, "POP_LAUNCH_TARGET_CRITIC", (64, 32, 16)), (20, "POP_LAUNCH_TARGET_CRITIC", None),
    (3, "POP_LAUNCH_TARGET_CRITIC", (16, 64, 16)), (34, "POP_LAUNCH_TARGET_CRITIC", None)])
def test_sac_with_more_than_eight_actions_takes_every_launch_and_rows(P, launch, rows):
    """Structures or rows without a fused kernel run one launch per part."""
    ensure_built()
    states = []
    for tuning in (dict(launch=pp.POP_LAUNCH_PER_PART), dict(launch=getattr(pp, launch))):
        pop = pp.Population(pp.make_config(P, 30, 12, (256, 256), 256, 300, algo=pp.POP_ALGO_SAC, rows=rows, half_tiles=1, **tuning), workloads.hparams(5, P))
        gen = torch.Generator(device="cuda")
        gen.manual_seed(3)
        rnd = lambda *s: torch.randn(s, generator=gen, device="cuda")
        pop.insert(-1, obs=rnd(P, 300, 30), act=rnd(P, 300, 12).clamp(-1, 1), rew=rnd(P, 300), done=(rnd(P, 300) > 2).float(), next_obs=rnd(P, 300, 30))
        if tuning["launch"] != pp.POP_LAUNCH_PER_PART:
            assert pop.tuning()["launch"] in (pp.POP_LAUNCH_PER_PART, pp.POP_LAUNCH_TARGET_CRITIC)
        pop.update(3)
        states.append([pop.get_params(i, w) for i in range(P) for w in ("actor", "critic1", "critic2", "t_critic1", "log_alpha")])
        pop.close()
    if rows is not None or P != 20:                       # (20 agents: one launch per part has 32-row target chains, a fused launch 16)
        assert all(np.array_equal(a, b) for a, b in zip(*states))


@pytest.mark.parametrize("bias1, bias2", [(-np.inf, 0.0), (0.0, -np.inf), (np.inf, 0.0), (-np.inf, np.nan), (np.nan, 0.0), (np.inf, np.inf)])
def test_sac_targets_of_a_diverged_population(bias1, bias2):
    """An infinite temperature and infinite or NaN target critics: the two critics' values, handed over apart, give the y of min(Q1', Q2') - alpha log pi."""
    ensure_built()
    hps = workloads.hparams(5, 1)
    hps[0]["init_log_alpha"] = 100.0                      # alpha = inf, alpha log pi = +-inf
    got = []
    for launch in (pp.POP_LAUNCH_PER_PART, pp.POP_LAUNCH_TARGET_CRITIC):
        pop = pp.Population(pp.make_config(1, 17, 6, (256, 256), 256, 300, algo=pp.POP_ALGO_SAC, launch=launch), hps)
        for net, bias in (("t_critic1", bias1), ("t_critic2", bias2)):
            th = pop.get_params(0, net).copy()
            th[-1] = bias
            pop.set_params(0, net, th)
        g = np.random.default_rng(5)
        rows = lambda *s: g.standard_normal((1, 300) + s).astype(np.float32)
        pop.insert(-1, obs=rows(17), act=np.clip(rows(6), -1, 1), rew=rows(), done=np.zeros((1, 300), np.float32), next_obs=rows(17))
        pop.update(1)
        got.append(pop.debug("target_y"))
        pop.close()
    assert not np.isfinite(got[0]).all() and np.array_equal(got[0], got[1], equal_nan=True), (got[0][0, :8], got[1][0, :8])
