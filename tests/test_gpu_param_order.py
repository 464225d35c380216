"""Networks cross the boundary in canonical order (row-major matrices) whatever order the library keeps them in, and the
order changes no result beyond the order of fp32 sums."""
import numpy as np
import pytest

import paper_2206_08888_amd as pp
import workloads
from gpu_common import NETS, STATE12, ensure_built, make_pair, many_rows, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("algo,P,O,A", [(pp.POP_ALGO_TD3, 2, 17, 6), (pp.POP_ALGO_TD3, 9, 17, 6), (pp.POP_ALGO_SAC, 2, 376, 17), (pp.POP_ALGO_TD3_SHARED, 2, 3, 1)])
def test_networks_come_back_as_they_were_set(algo, P, O, A):
    """Every tensor code, from and to host and device memory; device arrays aligned to floats only."""
    import torch
    ensure_built()
    sac = algo == pp.POP_ALGO_SAC
    hps = [dict(seed=3 + i, lr_actor=3e-4, lr_critic=3e-4, gamma=0.99, tau=0.005, policy_noise=0.2, noise_clip=0.5,
                policy_delay=1 if sac else 2, adam_b1=0.9, adam_b2=0.999, adam_eps=1e-8, lr_alpha=3e-4,
                target_entropy=-1.0, init_log_alpha=0.0) for i in range(P)]
    cfg = pp.make_config(P, O, A, (256, 256), 256, 100, algo=algo)
    pop = pp.Population(cfg, hps)
    rng = np.random.default_rng(5)
    for code in range(12):
        n = pp.pop_net_size(cfg, code)
        agents = [0] if algo == pp.POP_ALGO_TD3_SHARED and code % 3 else range(P)
        for agent in agents:
            a = rng.standard_normal(n).astype(np.float32)
            for src_dev in (False, True):
                buf = torch.zeros(n + 1, device="cuda")
                buf[1:] = torch.from_numpy(a).cuda()
                pp.pop_set_params(pop.ctx, agent, code, buf[1:] if src_dev else a)
                out = torch.full((n + 2,), 7.0, device="cuda")
                pp.pop_get_params(pop.ctx, agent, code, out[1:n + 1])
                host = np.empty(n, dtype=np.float32)
                pp.pop_get_params(pop.ctx, agent, code, host)
                got = out.cpu().numpy()
                assert np.array_equal(host, a) and np.array_equal(got[1:-1], a), (code, agent, src_dev)
                assert got[0] == 7.0 and got[-1] == 7.0
    pop.close()


@pytest.mark.parametrize("rows_critic,ahead", [(32, 2), (32, 1), (64, 1)])
def test_row_major_matrices_change_rounding_only(rows_critic, ahead):
    """With critic 1 in the target workgroups hidden matrices lie row-major, as long as the actor chains have 16 rows too: the same
    initial networks and actions bit for bit as with 32-row actor chains, where they do not, and steps that differ in the order of
    fp32 sums only (the bound of the comparison between the row classes)."""
    import torch
    obs = [torch.randn((10, n, 17), generator=torch.Generator().manual_seed(3)).cuda() for n in (40, many_rows(10))]   # both acting kernels
    out = []
    for rows_actor in (16, 32):
        gpu, _, _ = make_pair(2, P=10, capacity=600, hps=workloads.hparams(2, 10), oracle=False, rows=(16, rows_critic, rows_actor),
                              rows_critic1=16, launch=pp.POP_LAUNCH_TARGET_CRITIC, half_tiles=1, actor_ahead=ahead if rows_actor == 16 else 1)
        first = [gpu.get_params(i, w) for i in range(10) for w in NETS] + [gpu.act(o).cpu().numpy() for o in obs]
        gpu.update(3)
        out.append((first, {(i, w): gpu.get_params(i, w) for i in range(10) for w in STATE12}))
        gpu.close()
    assert all(np.array_equal(a, b) for a, b in zip(out[0][0], out[1][0]))
    worst = max(rel_l2(out[0][1][k], out[1][1][k]) for k in out[0][1] if out[1][1][k].any())
    assert worst <= 2e-5, worst


@pytest.mark.parametrize("P", [2, 9])
def test_networks_from_and_to_host_arrays_of_every_kind(P):
    """Pageable and pinned, at the start of an allocation and inside it; each read back into the other kind and from the device."""
    import torch
    ensure_built()
    cfg = pp.make_config(P, 17, 6, (256, 256), 256, 100)
    pop = pp.Population(cfg, workloads.hparams(2, P))
    rng = np.random.default_rng(7)

    def arrays(n):
        return {"pageable": torch.zeros(n), "pageable, inside": torch.zeros(n + 3)[3:], "pinned": torch.zeros(n, pin_memory=True),
                "pinned, inside": torch.zeros(n + 3, pin_memory=True)[3:], "device": torch.zeros(n + 3, device="cuda")[3:]}
    for code in (pp.PARAM_CODES["actor"], pp.PARAM_CODES["v_critic2"]):
        n = pp.pop_net_size(cfg, code)
        src, dst = arrays(n), arrays(n)
        for kind in src:
            a = torch.from_numpy(rng.standard_normal(n).astype(np.float32))
            src[kind].copy_(a)
            torch.cuda.synchronize()
            pp.pop_set_params(pop.ctx, 1, code, src[kind])
            for other in dst:
                dst[other].zero_()
                torch.cuda.synchronize()
                pp.pop_get_params(pop.ctx, 1, code, dst[other])
                pop.sync()
                assert torch.equal(dst[other].cpu(), a), (code, kind, other)
    pop.close()
