"""The 256-deep products on the bf16 pipe (three-way split operands): acting against 64-bit arithmetic at the edges of
the row and contraction tiles and over a wide range of magnitudes (with few rows on the vector ALU, with many on the bf16 pipe), and the row geometries that split their operands
differently against each other."""
import numpy as np
import pytest

import paper_2206_08888_amd as pp
from gpu_common import ensure_built, many_rows, rel_l2
from oracle import sac as oracle_sac, td3 as oracle_td3, td3_shared as oracle_shared

pytestmark = pytest.mark.gpu
H = 256


def _population(algo, P, O, A, capacity=64, **tuning):
    ensure_built()
    cfg = pp.make_config(P, O, A, (H, H), 256, capacity, algo=algo, **tuning)
    return pp.Population(cfg, _hparams(algo, P, A))


def _hparams(algo, P, A):
    sac = algo == pp.POP_ALGO_SAC
    return [dict(seed=7 + i, lr_actor=3e-4, lr_critic=3e-4, gamma=0.99, tau=0.005, policy_noise=0.2, noise_clip=0.5,
                policy_delay=1 if sac else 2, adam_b1=0.9, adam_b2=0.999, adam_eps=1e-8, lr_alpha=3e-4,
                target_entropy=-float(A) if sac else 0.0, init_log_alpha=0.0) for i in range(P)]


def _act64(theta, obs, O, A, out):
    t = theta.astype(np.float64)
    w1, t = t[:O * H].reshape(O, H), t[O * H:]
    b1, t = t[:H], t[H:]
    w2, t = t[:H * H].reshape(H, H), t[H * H:]
    b2, t = t[:H], t[H:]
    w3, b3 = t[:H * out].reshape(H, out), t[H * out:]
    h = np.maximum(obs.astype(np.float64) @ w1 + b1, 0.0)
    h = np.maximum(h @ w2 + b2, 0.0)
    # and the size of the head's terms: rounding is relative to those, also where they cancel in the sum
    return np.tanh(h @ w3 + b3)[:, :A], np.sqrt((h * h) @ (w3 * w3))[:, :A]


def _apart(a, ref, terms):
    return np.linalg.norm(a - ref) / np.linalg.norm(np.maximum(np.abs(ref), np.minimum(terms, 1.0)))


@pytest.mark.parametrize("algo", [pp.POP_ALGO_TD3, pp.POP_ALGO_SAC])
@pytest.mark.parametrize("O,A", [(1, 1), (8, 3), (9, 24), (33, 6), (376, 17), (424, 24), (64, 16), (65, 8), (17, 9)])
@pytest.mark.parametrize("n", [1, 33, many_rows(2), 17 * 32])
def test_acting_against_64_bits(algo, O, A, n):
    pop = _population(algo, 2, O, A)
    obs = np.random.default_rng(O + n).standard_normal((2, n, O)).astype(np.float32)
    a = pop.act(obs)
    for i in range(2):
        ref, terms = _act64(pop.get_params(i, "actor"), obs[i], O, A, 2 * A if algo == pp.POP_ALGO_SAC else A)
        # a product's relative error is 1e-7 (hidden layers) to 2e-7 (fp32 head and first layer), tanh's 1.2e-7
        assert _apart(a[i], ref, terms) < 6e-7
    pop.close()


@pytest.mark.parametrize("scale", [1e-28, 1e-15, 1e15, 1e28])
@pytest.mark.parametrize("n", [64, many_rows(1)])
def test_acting_over_magnitudes(scale, n):
    """Hidden activations of very different sizes: the layers are scaled against each other."""
    O, A = 17, 6
    pop = _population(pp.POP_ALGO_TD3, 1, O, A)
    th = pop.get_params(0, "actor").copy()
    th[:O * H + H] *= np.float32(scale)
    th[O * H + H:O * H + H + H * H] *= np.float32(1.0 / scale)
    pop.set_params(0, "actor", th)
    obs = np.random.default_rng(3).standard_normal((1, n, O)).astype(np.float32)
    assert _apart(pop.act(obs)[0], *_act64(th, obs[0], O, A, A)) < 6e-7
    pop.close()


def _views(th, fan_in, out):
    """W1, b1, W2, b2, W3, b3 of a flat network, as views."""
    at, got = 0, []
    for shape in ((fan_in, H), (H,), (H, H), (H,), (H, out), (out,)):
        n = int(np.prod(shape))
        got.append(th[at:at + n].reshape(shape))
        at += n
    return got


MOST = np.finfo(np.float32).max
PLANTS = {                     # what is put into a network's W1, b1, W2, b2, W3, b3
    "weights": lambda w1, b1, w2, b2, w3, b3: (w2.__setitem__((5, 9), np.inf), w2.__setitem__((7, 20), -np.inf), w2.__setitem__((8, 33), np.nan)),
    "one activation": lambda w1, b1, w2, b2, w3, b3: (b1.__setitem__(3, np.inf), np.abs(w3, out=w3)),
    "opposite infinities": lambda w1, b1, w2, b2, w3, b3: (b1.__setitem__(3, np.inf), w2.__setitem__((40, slice(0, 128)), np.inf), np.abs(w3, out=w3)),
    "largest finite": lambda w1, b1, w2, b2, w3, b3: (b1.__setitem__(3, MOST), np.multiply(w2[3], np.float32(1e-32), out=w2[3]),
                                                     w1.__setitem__((slice(None), 6), 0), b1.__setitem__(6, 1e-33), w2.__setitem__((6, 11), -MOST),
                                                     np.multiply(w3, np.float32(1e-6), out=w3)),
}


@pytest.mark.parametrize("plant", sorted(PLANTS))
@pytest.mark.parametrize("algo", [pp.POP_ALGO_TD3, pp.POP_ALGO_SAC])
@pytest.mark.parametrize("times", [1, 17])                # the same 64 rows over again: 1,088 go to the 32-row kernel
def test_acting_with_infinities(algo, plant, times):
    """Infinite, NaN and the largest finite operands of a hidden product give what fp32 arithmetic gives."""
    O, A, n = 17, 6, 64
    assert times == 1 or times * n >= many_rows(1)
    pop = _population(algo, 1, O, A)
    out = 2 * A if algo == pp.POP_ALGO_SAC else A
    th = pop.get_params(0, "actor").copy()
    PLANTS[plant](*_views(th, O, out))
    pop.set_params(0, "actor", th)
    obs = np.random.default_rng(4).standard_normal((1, n, O)).astype(np.float32)
    got = pop.act(np.tile(obs, (1, times, 1)))[0].astype(np.float64)
    pop.close()
    assert all(np.array_equal(got[:n], got[k * n:(k + 1) * n], equal_nan=True) for k in range(1, times))
    got = got[:n]
    w1, b1, w2, b2, w3, b3 = (v.astype(np.float64) for v in _views(th, O, out))
    with np.errstate(all="ignore"):
        h = np.fmax(obs[0].astype(np.float64) @ w1 + b1, 0.0)      # max(NaN, 0) = 0, as the kernels' ReLU has it
        h = np.fmax((h[:, :, None] * w2[None]).sum(1) + b2, 0.0)
        want = np.tanh((h[:, :, None] * w3[None]).sum(1) + b3)[:, :A]
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.allclose(got, want, rtol=0, atol=2e-6, equal_nan=True)
    if plant == "one activation":
        assert (want == 1.0).all()                                # and not the head's bias


@pytest.mark.parametrize("algo", [pp.POP_ALGO_TD3, pp.POP_ALGO_SAC, pp.POP_ALGO_TD3_SHARED])
@pytest.mark.parametrize("rows", [32, 64])
def test_update_with_infinities(algo, rows):
    """One step of a diverged population: infinite Bellman targets and gradients come out of 32- and 64-row chains as out of
    16-row chains, whose products run on the fp32 instructions."""
    O, A, P = 17, 6, 2
    sac = algo == pp.POP_ALGO_SAC
    got = []
    # critic chains have 16 rows where they follow the target chains of TD3; elsewhere only the targets are compared
    small = dict(rows=(16, 32, 16)) if algo != pp.POP_ALGO_TD3 else dict(rows=(16, 32, 16), rows_critic1=16, launch=pp.POP_LAUNCH_TARGET_CRITIC)
    for tuning in (small, dict(rows=rows)):
        pop = _population(algo, P, O, A, **tuning)
        for agent in range(P):
            for net in ("critic1", "critic2", "t_critic1", "t_critic2"):
                th = pop.get_params(agent, net).copy()
                w1, b1, w2, b2, w3, b3 = _views(th, O + A, 1)
                np.abs(w2, out=w2)
                np.abs(w3, out=w3)
                if net[0] == "t" and agent == 0:
                    b1[3] = np.inf
                pop.set_params(agent, net, th)
        g = np.random.default_rng(6)
        rew = g.standard_normal((P, 64)).astype(np.float32)
        rew[1, 5] = np.inf
        done = np.zeros((P, 64), np.float32)
        pop.insert(-1, obs=g.standard_normal((P, 64, O)).astype(np.float32), act=g.uniform(-1, 1, (P, 64, A)).astype(np.float32),
                   rew=rew, done=done, next_obs=g.standard_normal((P, 64, O)).astype(np.float32))
        pop.set_debug(True)
        pop.update(1)
        got.append((pop.debug("target_y"), [pop.get_params(a, "g_critic1") for a in range(P)]))
        pop.close()
    (y0, g0), (y1, g1) = got
    assert np.array_equal(np.isnan(y0), np.isnan(y1)) and np.array_equal(np.isinf(y0), np.isinf(y1))
    assert np.allclose(y0, y1, rtol=1e-5, atol=1e-5, equal_nan=True)
    if algo != pp.POP_ALGO_TD3_SHARED:
        assert (y0[0] == np.inf).all() and np.isinf(y0[1]).any() and np.isfinite(y0[1]).any()
    if algo == pp.POP_ALGO_TD3:
        for a, b in zip(g0, g1):
            assert np.isinf(a).any()
            assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isinf(a), np.isinf(b))


ORACLES = {pp.POP_ALGO_TD3: oracle_td3, pp.POP_ALGO_SAC: oracle_sac, pp.POP_ALGO_TD3_SHARED: oracle_shared}


def fix_masks(orc, rng):
    """Biases that keep every hidden unit of every network of an oracle population away from its kink: +-4 in the first
    layer (its sums are about 0.5), in the second what brings a unit's mean to +-2.5 (six times what a row changes) -- so the hidden
    sums still cancel to a tenth of their terms, and an error of the terms shows.  Small heads for the policies."""
    seen = set()
    for ag in orc.agents:
        nets = [(ag.actor, True), (ag.critic[0], False), (ag.critic[1], False), (ag.t_critic[0], False), (ag.t_critic[1], False)]
        if hasattr(ag, "t_actor"):
            nets.append((ag.t_actor, True))
        for net, policy in nets:
            if id(net) in seen:
                continue
            seen.add(id(net))
            (w1, b1), (w2, b2), (w3, b3) = net
            b1[:] = rng.choice([-4.0, 4.0], H)
            b2[:] = np.round(8 * (rng.choice([-2.5, 2.5], H) - np.maximum(b1, 0.0) @ w2)) / 8
            if policy:
                w3 *= 1 / 16


@pytest.mark.parametrize("algo,O,A", [(pp.POP_ALGO_TD3, 17, 6), (pp.POP_ALGO_TD3, 56, 8), (pp.POP_ALGO_SAC, 17, 6),
                                      (pp.POP_ALGO_SAC, 40, 24), (pp.POP_ALGO_TD3_SHARED, 17, 6)])
@pytest.mark.parametrize("rows", [(16, 32, 16), 32, 64])
def test_gradients_against_64_bits(algo, O, A, rows):
    """One update step of every network, no hidden unit near its kink: the gradients against 64-bit arithmetic."""
    P, n = 3, 64
    pop = _population(algo, P, O, A, rows=rows)
    orc = ORACLES[algo].Population([dict(h, lr_critic=1e-12) for h in _hparams(algo, P, A)], O, A, [H, H], 256, n)
    for i in range(P):
        pop.set_hparams(i, dict(_hparams(algo, P, A)[i], lr_critic=1e-12))     # the policy step meets the critics as they were
    g = np.random.default_rng(5)
    fix_masks(orc, g)
    for i in range(P):
        tr = dict(obs=g.standard_normal((n, O)).astype(np.float32), act=g.uniform(-1, 1, (n, A)).astype(np.float32),
                  rew=g.standard_normal(n).astype(np.float32), done=(g.random(n) < 0.1).astype(np.float32),
                  next_obs=g.standard_normal((n, O)).astype(np.float32))
        pop.insert(i, **tr)
        orc.insert(i, **tr)
        for net in ("actor", "critic1", "critic2", "t_actor", "t_critic1", "t_critic2"):
            if not (algo == pp.POP_ALGO_SAC and net == "t_actor"):
                pop.set_params(i, net, orc.get_params(i, net))
    pop.set_debug(True)
    pop.update(1)
    orc.update(1)
    errors = {}
    for i in range(P):
        for net in ("critic1", "critic2", "actor"):
            fan_in, out = (O, 2 * A if algo == pp.POP_ALGO_SAC else A) if net == "actor" else (O + A, 1)
            got, want = pop.get_params(i, "g_" + net), orc.get_params(i, "g_" + net)
            for name, x, y in zip(("W1", "b1", "W2", "b2", "W3", "b3"), _views(got, fan_in, out), _views(want, fan_in, out)):
                errors[net, name] = max(errors.get((net, name), 0.0), rel_l2(x, y))
    pop.close()
    print("algo %d, obs %d, act %d, rows %s: %s" % (algo, O, A, rows, {k: "%.1e" % v for k, v in errors.items()}))
    # four products in sequence, 2e-7 each on the fp32 instructions, and the batch sum's 1.4e-7: 4.3e-7, and twice that.
    # (Measured 1.6e-7 .. 4.7e-7 with 16 rows, 1.6e-7 .. 4.3e-7 with 32 and 64; without the low parts of one operand the
    # W3 gradients of a forward product are 3.7e-6 off, the W1 gradients of a backward one 3.2e-6.)
    assert max(errors.values()) < 1e-6, errors


@pytest.mark.parametrize("algo,O,A", [(pp.POP_ALGO_TD3, 17, 6), (pp.POP_ALGO_TD3, 56, 8), (pp.POP_ALGO_SAC, 17, 6),
                                      (pp.POP_ALGO_SAC, 40, 24), (pp.POP_ALGO_TD3_SHARED, 17, 6)])
@pytest.mark.parametrize("rows", [32, 64])
def test_rows_of_a_chain_agree(algo, O, A, rows):
    """One update step: parameters and first moments with every chain at `rows` rows against 16-row target and actor
    chains, whose products run on the fp32 instructions."""
    got = []
    for r in ((16, 32, 16), (rows, rows, rows)):
        pop = _population(algo, 3, O, A, rows=r)
        g = np.random.default_rng(5)
        pop.insert(-1, obs=g.standard_normal((3, 64, O)).astype(np.float32), act=g.uniform(-1, 1, (3, 64, A)).astype(np.float32),
                   rew=g.standard_normal((3, 64)).astype(np.float32), done=np.zeros((3, 64), np.float32),
                   next_obs=g.standard_normal((3, 64, O)).astype(np.float32))
        pop.update(1)
        nets = [(0, net) for net in ("actor", "critic1", "critic2")]
        got.append([pop.get_params(a, "m_" + net) for a, net in nets])     # first Adam moments: (1 - b1) gradient
        pop.close()
    for x, y in zip(*got):
        # a gradient is a sum over 256 rows through four products, each 2e-7 apart, and a ReLU unit within rounding
        # of zero may switch: one of 65,536 is 4e-6 of the gradient's square
        assert rel_l2(y, x) < 2e-3 and np.isfinite(y).all()


@pytest.mark.parametrize("algo", [pp.POP_ALGO_TD3, pp.POP_ALGO_SAC])
@pytest.mark.parametrize("O,A", [(64, 1), (5, 9), (71, 9), (71, 10), (400, 24), (423, 24), (424, 24)])
def test_wide_first_layers_against_64_bits(algo, O, A):
    """First layers on the bf16 pipe (32 rows: 17 agents or more), fan-ins around the ends of its 16-deep blocks and groups of
    blocks: the gradients of one update step against 64-bit arithmetic, no hidden unit near its kink."""
    P, n = 17, 48
    hps = [dict(h, lr_critic=1e-12) for h in _hparams(algo, P, A)]
    ensure_built()
    pop = pp.Population(pp.make_config(P, O, A, (H, H), 256, n, algo=algo), hps)
    orc = ORACLES[algo].Population(hps[:2], O, A, [H, H], 256, n)
    g = np.random.default_rng(O + A)
    fix_masks(orc, g)
    for i in range(P):
        tr = dict(obs=g.standard_normal((n, O)).astype(np.float32), act=g.uniform(-1, 1, (n, A)).astype(np.float32),
                  rew=g.standard_normal(n).astype(np.float32), done=(g.random(n) < 0.1).astype(np.float32),
                  next_obs=g.standard_normal((n, O)).astype(np.float32))
        pop.insert(i, **tr)
        if i < 2:
            orc.insert(i, **tr)
            for net in ("actor", "critic1", "critic2", "t_actor", "t_critic1", "t_critic2"):
                if not (algo == pp.POP_ALGO_SAC and net == "t_actor"):
                    pop.set_params(i, net, orc.get_params(i, net))
    pop.set_debug(True)
    pop.update(1)
    orc.update(1)
    worst = max(rel_l2(pop.get_params(i, "g_" + net), orc.get_params(i, "g_" + net)) for i in range(2) for net in ("critic1", "critic2", "actor"))
    pop.close()
    assert worst < 1e-6                                # as in test_gradients_against_64_bits


@pytest.mark.parametrize("algo", [pp.POP_ALGO_TD3, pp.POP_ALGO_SAC])
@pytest.mark.parametrize("scale", [1e-28, 1e-9, 1e-4, 1.0, 1e3, 1e28])
def test_16_row_chains_over_magnitudes(algo, scale):
    """One step with hidden weights `scale` times as large and first layers scaled the other way: 16-row chains, whose products
    run on the fp32 instructions, against 32-row chains (three-part bf16)."""
    O, A, P = 17, 6, 2
    got = []
    for rows in ((16, 32, 16), 32):
        pop = _population(algo, P, O, A, rows=rows)
        for i in range(P):
            for net, fan_in, out in [(n, O, 2 * A if algo == pp.POP_ALGO_SAC else A) for n in ("actor", "t_actor")] + \
                                    [(n, O + A, 1) for n in ("critic1", "critic2", "t_critic1", "t_critic2")]:
                if algo == pp.POP_ALGO_SAC and net == "t_actor":
                    continue
                th = pop.get_params(i, net).copy()
                w1, b1, w2, b2, w3, b3 = _views(th, fan_in, out)
                w1 /= np.float32(scale)
                w2 *= np.float32(scale)
                w2[:, 5] *= np.float32(1e-6)               # a unit whose weights are small beside the others'
                pop.set_params(i, net, th)
        g = np.random.default_rng(8)
        pop.insert(-1, obs=g.standard_normal((P, 64, O)).astype(np.float32), act=g.uniform(-1, 1, (P, 64, A)).astype(np.float32),
                   rew=g.standard_normal((P, 64)).astype(np.float32), done=np.zeros((P, 64), np.float32),
                   next_obs=g.standard_normal((P, 64, O)).astype(np.float32))
        pop.set_debug(True)
        pop.update(1)
        got.append((pop.debug("target_y"), [pop.get_params(a, "g_actor") for a in range(P)]))
        pop.close()
    (y16, g16), (y32, g32) = got
    # a Q value is a sum of 256 products through two layers, each sum within 3e-7 of its terms on either side
    assert np.linalg.norm(y16 - y32) / np.linalg.norm(y32) < 3e-6
    for x, y in zip(g16, g32):
        assert np.isfinite(y).all() and rel_l2(x, y) < 2e-3    # as in test_rows_of_a_chain_agree
        # the small unit by itself, which the norms of y and of the gradients cannot show: its head weights' gradient
        u16, u32 = (_views(v, O, 2 * A if algo == pp.POP_ALGO_SAC else A)[4][5] for v in (x, y))
        assert np.linalg.norm(u32.astype(np.float64)) > 0 and rel_l2(u16, u32) < 2e-3


def _forward64(net, x):
    """Q of every row in 64 bits, and the size of the head's terms."""
    w1, b1, w2, b2, w3, b3 = (v.astype(np.float64) for v in net)
    h = np.maximum(x @ w1 + b1, 0.0)
    h = np.maximum(h @ w2 + b2, 0.0)
    return (h @ w3 + b3)[:, 0], np.sqrt((h * h) @ (w3 * w3))[:, 0]


# name: (factor of the hidden weights behind half of the units, factor of one unit's activation)
SPREADS = {"alike": (1.0, 1.0), "1e-5": (1e-5, 1.0), "1e-7": (1e-7, 1.0), "1e-9": (1e-9, 1.0), "1e-20": (1e-20, 1.0),
           "one activation 1e8": (1.0, 1e8)}


@pytest.mark.parametrize("spread", sorted(SPREADS))
@pytest.mark.parametrize("rows", [(16, 32, 16), 32, 64])
def test_forward_products_with_mixed_magnitudes(rows, spread):
    """Small and ordinary weights in one column, small and large activations in one row: batch rows that meet only the small
    ones get the Bellman target that their own terms give, and not one that the other rows' sizes spoil."""
    O, A, P, n = 17, 6, 2, 64
    small, large = SPREADS[spread]
    quiet, big = slice(0, H, 2), 1                       # units that are active in the quiet rows; one that is not `quiet`
    pop = _population(pp.POP_ALGO_TD3, P, O, A, rows=rows)
    nets = []
    for i in range(P):
        for net in ("t_critic1", "t_critic2"):
            th = pop.get_params(i, net).copy()
            w1, b1, w2, b2, w3, b3 = _views(th, O + A, 1)
            w1[0] = -4.0                                 # obs 0 is 1 in quiet rows and -1 in the others
            w1[0, quiet] = 4.0
            w1[O:] = 0.0                                 # whatever the target action
            w2[quiet] *= np.float32(small)
            w1[:, big], b1[big], w2[big] = w1[:, big] * np.float32(large), 0.0, 0.0 if large != 1.0 else w2[big]
            if large != 1.0:
                w1[0, big] = 4 * large                   # large in the quiet rows, and every weight it meets is zero
            pop.set_params(i, net, th)
            nets.append(_views(th, O + A, 1))
    g = np.random.default_rng(12)
    obs = g.standard_normal((P, n, O)).astype(np.float32)
    nxt = g.standard_normal((P, n, O)).astype(np.float32)
    nxt[:, :, 0] = np.where(np.arange(n) % 2 == 0, 1.0, -1.0)
    zero = np.zeros((P, n), np.float32)
    pop.insert(-1, obs=obs, act=g.uniform(-1, 1, (P, n, A)).astype(np.float32), rew=zero, done=zero, next_obs=nxt)
    pop.set_debug(True)
    pop.update(1)
    y, batch = pop.debug("target_y").astype(np.float64), pop.debug("batch").astype(np.float64)
    pop.close()
    gamma = float(np.float32(0.99))
    for i in range(P):
        x = np.concatenate([batch[i][:, O + A + 2:], np.zeros((256, A))], axis=1)
        (q0, s0), (q1, s1) = _forward64(nets[2 * i], x), _forward64(nets[2 * i + 1], x)
        want, size = gamma * np.minimum(q0, q1), gamma * np.maximum(s0, s1)
        for rest in (x[:, 0] > 0, x[:, 0] < 0):
            assert rest.any()
            # a hidden unit is 2.9e-7 off at most (its product) and 2e-7 (the first layer's), each independently of the others, so
            # a Q value is 3.5e-7 of the root of its squared head terms off, also where those cancel; and twice that
            apart = np.linalg.norm(y[i][rest] - want[rest]) / np.linalg.norm(np.maximum(np.abs(want[rest]), size[rest]))
            assert apart < 7e-7, (i, rest[0])


@pytest.mark.parametrize("small", [1.0, 1e-5, 1e-7, 1e-9, 1e-20])
@pytest.mark.parametrize("rows", [(16, 32, 16), 32, 64])
def test_backward_products_with_mixed_magnitudes(rows, small):
    """The same for the products with the transposed weights: the policy gradient that comes from batch rows whose active
    units all have small weights behind them."""
    O, A, P, n = 17, 6, 2, 64
    orc = oracle_td3.Population(_hparams(pp.POP_ALGO_TD3, P, A), O, A, [H, H], 256, n)
    hps = [dict(h, lr_critic=1e-12) for h in _hparams(pp.POP_ALGO_TD3, P, A)]      # the policy step meets the critics as they were
    pop = _population(pp.POP_ALGO_TD3, P, O, A, rows=rows)
    g = np.random.default_rng(13)
    fix_masks(orc, g)
    always, gate = slice(0, H, 2), 7                      # units active in every row; the unit that is active in the quiet ones
    for i in range(P):
        ag = orc.agents[i]
        pop.set_hparams(i, hps[i])
        orc.set_hparams(i, hps[i])
        (w1, b1), (w2, b2), (w3, b3) = ag.actor
        w2[:, always] *= small
        w1[:, gate], w1[1, gate], b1[gate] = 0.0, 8.0, -4.0
        mean = np.maximum(b1, 0.0) @ w2
        b2[:] = np.round(8 * (g.choice([-2.5, 2.5], H) - mean)) / 8
        b2[always] = np.round(8 * (2.5 - mean[always])) / 8
        w2[gate, 1::2] = -2.5                            # switches the other half off in the quiet rows (the gate adds 4 times this)
        for net in ("actor", "critic1", "critic2", "t_actor", "t_critic1", "t_critic2"):
            pop.set_params(i, net, orc.get_params(i, net))
        # both sides start from the same 32-bit values
        for layer, got in zip(ag.actor, (_views(pop.get_params(i, "actor"), O, A)[k:k + 2] for k in (0, 2, 4))):
            layer[0][:], layer[1][:] = got
        tr = dict(obs=g.standard_normal((n, O)).astype(np.float32), act=g.uniform(-1, 1, (n, A)).astype(np.float32),
                  rew=g.standard_normal(n).astype(np.float32), done=np.zeros(n, np.float32), next_obs=g.standard_normal((n, O)).astype(np.float32))
        tr["obs"][:, 1] = np.arange(n) % 2               # obs 1: 1 in the quiet rows, 0 in the others
        pop.insert(i, **tr)
        orc.insert(i, **tr)
    pop.set_debug(True)
    pop.update(1)
    orc.update(1)
    for i in range(P):
        got, want = (_views(p.get_params(i, "g_actor"), O, A)[0] for p in (pop, orc))
        assert np.linalg.norm(want[1]) > 0
        # row 1 of dW1 is summed over the quiet rows alone; the bound is test_gradients_against_64_bits'
        assert rel_l2(got[1], want[1]) < 1e-6 and rel_l2(got, want) < 1e-6, i
    pop.close()


@pytest.mark.parametrize("plant", ["bias", "hidden weight"])
def test_wide_first_layer_ends_with_its_fan_in(plant):
    """Fan-in 71: the last block of 16 inputs reaches eight rows past the weights, to the bias and the hidden weights that lie
    behind them; an infinity there stays out of the first layer's sums."""
    O, A, P, n = 65, 6, 17, 64
    pop = _population(pp.POP_ALGO_TD3, P, O, A)
    assert pop.tuning()["rows_target"] == 32
    nets = []
    for net in ("t_critic1", "t_critic2"):
        th = pop.get_params(0, net).copy()
        w1, b1, w2, b2, w3, b3 = _views(th, O + A, 1)
        np.abs(w3, out=w3)
        w1[O:] = 0.0                                     # whatever the target action
        if plant == "bias":
            b1[5] = np.inf
            np.abs(w2[5], out=w2[5])
        else:
            w2[0:6, 9] = -np.inf                         # unit 9 of the second layer is off wherever one of six units is on
        pop.set_params(0, net, th)
        nets.append([v.astype(np.float64) for v in _views(th, O + A, 1)])
    g = np.random.default_rng(14)
    zero = np.zeros((P, n), np.float32)
    pop.insert(-1, obs=g.standard_normal((P, n, O)).astype(np.float32), act=g.uniform(-1, 1, (P, n, A)).astype(np.float32),
               rew=zero, done=zero, next_obs=g.standard_normal((P, n, O)).astype(np.float32))
    pop.set_debug(True)
    pop.update(1)
    y, batch = pop.debug("target_y")[0].astype(np.float64), pop.debug("batch")[0].astype(np.float64)
    pop.close()
    x = np.concatenate([batch[:, O + A + 2:], np.zeros((256, A))], axis=1)
    q = []
    with np.errstate(all="ignore"):
        for w1, b1, w2, b2, w3, b3 in nets:
            h = np.fmax(x @ w1 + b1, 0.0)                # max(NaN, 0) = 0, as the kernels' ReLU has it
            h = np.fmax((h[:, :, None] * w2[None]).sum(1) + b2, 0.0)
            q.append((h * w3[:, 0]).sum(1) + b3[0])
    want = float(np.float32(0.99)) * np.minimum(*q)
    if plant == "bias":
        assert np.isinf(want).all() and np.array_equal(y, want)
    else:
        assert np.isfinite(want).all() and np.allclose(y, want, rtol=0, atol=4e-6)
