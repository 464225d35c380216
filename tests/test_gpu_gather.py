"""The gather of a step's replay rows: each number of floats per thread (4, 8, 16, 32) against the rows the host inserted, and the
kernel's division by the row length."""
import numpy as np
import pytest
import torch

import paper_2206_08888_amd as pp
import workloads
from gpu_common import ensure_built
from oracle import philox


def test_rows_of_flat_elements_by_a_float_product():
    """gather_run takes element e of a stacked batch of rows of n floats to row (int)((e + 0.5f) * (1.0f / n)): exact for all n and e < 256 n."""
    for n in range(5, 922):                               # 2 obs + act + 2: at most 447 + 1 and 424 + 24 inputs
        e = np.arange(256 * n, dtype=np.int32)
        got = ((e.astype(np.float32) + np.float32(0.5)) * (np.float32(1.0) / np.float32(n))).astype(np.int32)
        assert np.array_equal(got, e // n), n


@pytest.mark.gpu
@pytest.mark.parametrize("algo, P, O, A, floats", [("td3", 3, 1, 1, 4), ("td3", 23, 17, 6, 4), ("td3", 24, 17, 6, 8), ("sac", 50, 17, 6, 16),
                                                   ("td3", 250, 25, 6, 32), ("td3", 20, 376, 17, 32), ("td3_shared", 90, 3, 1, 8), ("td3", 1, 447, 1, 4)])       # 20 agents of 376 / 17 fill more than the 32 MB of the L2s
def test_batches_of_every_width(algo, P, O, A, floats):
    ensure_built()
    code = {"td3": pp.POP_ALGO_TD3, "sac": pp.POP_ALGO_SAC, "td3_shared": pp.POP_ALGO_TD3_SHARED}[algo]
    n, row = 700, 2 * O + A + 2
    e = 4                                                 # the rule of gather_floats_per_thread
    while e < 32 and P * -(-256 * row // (256 * e)) > 256:
        e *= 2
    assert e == floats
    hps = workloads.hparams(2, P)
    pop = pp.Population(pp.make_config(P, O, A, (256, 256), 256, n, algo=code), hps)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(P)
    parts = [torch.randn((P, n, k), generator=gen, device="cuda") for k in (O, A, 1, 1, O)]
    pop.insert(-1, obs=parts[0], act=parts[1], rew=parts[2][..., 0].contiguous(), done=parts[3][..., 0].contiguous(), next_obs=parts[4])
    rows = torch.cat(parts, 2).cpu().numpy()
    for t in range(3):                                    # the first batch comes from the stand-alone gather, the others rode along with a step
        pop.update(1)
        idx, batch = pop.debug("indices"), pop.debug("batch")
        for i in {0, P // 2, P - 1}:
            assert np.array_equal(idx[i].astype(np.int64), philox.sample_indices(hps[i]["seed"], t, 256, n))
        for i in range(P):
            assert np.array_equal(batch[i], rows[i][idx[i]]), (t, i)
    pop.close()


@pytest.mark.gpu
def test_batches_on_both_sides_of_the_line_between_loads_through_and_past_the_caches():
    """33 agents of 42 floats: 6,052 rows fill 32 MB but for a few floats, 6,053 more; rows inserted behind a gather go into the next one."""
    ensure_built()
    P, O, A, row = 33, 17, 6, 42
    under = (8 << 20) // (P * row)
    assert P * under * row <= 8 << 20 < P * (under + 1) * row
    hps = workloads.hparams(2, P)
    pop = pp.Population(pp.make_config(P, O, A, (256, 256), 256, under + 8), hps)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(P)
    rows = np.zeros((P, 0, row), np.float32)
    for n in (under, 1, 7):
        parts = [torch.randn((P, n, k), generator=gen, device="cuda") for k in (O, A, 1, 1, O)]
        pop.insert(-1, obs=parts[0], act=parts[1], rew=parts[2][..., 0].contiguous(), done=parts[3][..., 0].contiguous(), next_obs=parts[4])
        rows = np.concatenate([rows, torch.cat(parts, 2).cpu().numpy()], 1)
        for _ in range(2):
            pop.update(1)
            idx, batch = pop.debug("indices"), pop.debug("batch")
            assert idx.max() < rows.shape[1] and all(np.array_equal(batch[i], rows[i][idx[i]]) for i in range(P)), n
    pop.close()
