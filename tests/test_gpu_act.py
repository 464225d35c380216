"""Acting on a few rows per agent (k_act_few): against the actor's forward pass in 64 bits, at the ends of its range, and the same rows among
many (k_act)."""
import numpy as np
import pytest
import torch

import paper_2206_08888_amd as pp
import workloads
from gpu_common import ensure_built, many_rows

pytestmark = pytest.mark.gpu
H = 256


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


def _actor64(pop, agent, O, out):
    th, off, parts = pop.get_params(agent, "actor").astype(np.float64), 0, []
    for shape in ((O, H), (H,), (H, H), (H,), (H, out), (out,)):
        n = int(np.prod(shape))
        parts.append(th[off:off + n].reshape(shape))
        off += n
    return parts


def _forward64(net, x, chain=64):
    """Head sums, and a bound on what 32-bit sums may be off: u per operation, at most `chain` operations one after the other in a
    sum (k_act_few 64: 28 + 16 for the widest first layer, 32 for the others, and the dot product over lanes; k_act 448: the widest
    first layer; six partial products of 16 instructions for the others), errors of a layer carried through the next."""
    u = chain * 2.0 ** -24
    h, e = x, np.zeros_like(x)
    for k in (0, 2, 4):
        W, b = net[k], net[k + 1]
        e = (e + u * np.abs(h)) @ np.abs(W) + u * np.abs(b)
        h = h @ W + b
        if k < 4:
            h = np.maximum(h, 0.0)
    return h, e


@pytest.mark.parametrize("algo, P, O, A", [("td3", 1, 1, 1), ("td3", 3, 17, 6), ("td3", 10, 64, 8), ("td3", 2, 65, 24),
                                           ("sac", 2, 128, 3), ("sac", 5, 424, 24), ("td3_shared", 3, 447, 1), ("td3", 70, 33, 5),
                                           # heads past 16 columns: even and odd rows in LDS, or two columns of a wavefront (many agents, 17 .. 19)
                                           ("sac", 2, 17, 10), ("td3", 2, 9, 23), ("td3", 3, 40, 17), ("td3", 130, 70, 17), ("td3", 129, 66, 19)])
def test_a_few_rows_per_agent(algo, P, O, A):
    code = {"td3": pp.POP_ALGO_TD3, "sac": pp.POP_ALGO_SAC, "td3_shared": pp.POP_ALGO_TD3_SHARED}[algo]
    pop = pp.Population(pp.make_config(P, O, A, (H, H), 256, 64, algo=code), workloads.hparams(0, P))
    rng = np.random.default_rng(100 * O + A)
    for i in range(P):                                   # biases too
        pop.set_params(i, "actor", pop.get_params(i, "actor") + 0.02 * rng.standard_normal(pop.actor_size).astype(np.float32))
    nets = [_actor64(pop, i, O, 2 * A if algo == "sac" else A) for i in range(P)]
    most = (256 // P) * 4                                # rows per agent up to which the kernel is taken whatever P is
    first = None
    for n in sorted({1, 2, 3, 4, 5, min(7, most), min(most, 41), many_rows(P)}):
        obs = rng.standard_normal((P, n, O)).astype(np.float32)
        if first is not None:
            obs[:, :1] = first
        first = obs[:, :1]
        got = pop.act(torch.from_numpy(obs).cuda()).cpu().numpy()
        for i in range(P):
            z, e = _forward64(nets[i], obs[i].astype(np.float64), 64 if n <= most else 448)
            assert np.all(np.abs(got[i] - np.tanh(z[:, :A])) <= e[:, :A] + 2.0 ** -21), (n, i)
        if n <= 4 or P * ((n + 3) // 4) <= 256:          # a row does not depend on how many there are
            if n > 1:
                assert np.array_equal(got[:, :1], alone)
            alone = got[:, :1]
        assert np.array_equal(got, pop.act(obs))         # host arrays
        if n > most:                                     # the same row among many: both sums are within their bounds
            z, few = _forward64(nets[0], obs[0, :1].astype(np.float64))
            many = _forward64(nets[0], obs[0, :1].astype(np.float64), 448)[1]
            assert np.all(np.abs(got[0, :1] - alone[0]) <= (few + many)[:, :A] + 2.0 ** -20)
        sigma = np.linspace(0.0, 0.3, P).astype(np.float32)
        noisy = pop.act(torch.from_numpy(obs).cuda(), sigma, step=9).cpu().numpy()
        assert np.array_equal(noisy[0], got[0]) and (P == 1 or not np.array_equal(noisy[-1], got[-1]))
    pop.close()


def test_more_rows_than_one_grid_dimension_holds():
    """537 million rows of two agents: their row blocks, 256 threads each, are more than the 2^32 - 1 threads of a grid dimension, past which a launch
    loses workgroups without an error.  Rows at the ends and on both sides of the line between the pieces as in calls of their own."""
    n, few = (1 << 28) + 33, 70_000
    pop = pp.Population(pp.make_config(2, 1, 1, (H, H), 256, 64), workloads.hparams(0, 2))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    obs = torch.randn((2, n, 1), generator=gen, device="cuda")
    sigma = np.array([0.0, 0.1], np.float32)
    got = pop.act(obs, sigma, step=4)
    line = 32 * (((1 << 24) - 1) // 2)                    # rows per agent in the first piece
    for at in (0, line - few // 2, n - few):
        want = pop.act(obs[:, at:at + few].contiguous(), sigma, step=4)
        assert torch.equal(got[0, at:at + few], want[0]), at
        assert (at == 0) == torch.equal(got[1, at:at + few], want[1]), at       # noise is numbered by the row of the call
    still = pop.act(obs[:, line - few // 2:line + few // 2].contiguous())[1]
    noise = got[1, line - few // 2:line + few // 2] - still
    assert 0.05 < float(noise.std()) < 0.15
    pop.close()


@pytest.mark.parametrize("P, O, n", [(300, 100, 151), (30, 376, 370), (257, 376, 45)])
def test_the_last_piece_of_host_arrays_rounds_as_the_others(P, O, n):
    """Host arrays go through a 16 MB staging area piece by piece; the rows of a short last piece come out as in a device call with all rows."""
    A = 6
    piece = (16 << 20) // (P * (O + A) * 4)
    assert n > piece and 0 < n % piece <= 32
    pop = pp.Population(pp.make_config(P, O, A, (H, H), 256, 64), workloads.hparams(0, P))
    obs = np.random.default_rng(n).standard_normal((P, n, O)).astype(np.float32)
    assert np.array_equal(pop.act(obs), pop.act(torch.from_numpy(obs).cuda()).cpu().numpy())
    pop.close()
