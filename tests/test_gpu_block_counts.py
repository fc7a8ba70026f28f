"""The blocks that last_timing reports: those that were run, in whole rounds between two looks at the states,
whichever form the iterations take and whichever entry point is called."""

import numpy as np
import pytest

import paper_0802_0748_amd as S
from workloads import simple_cubic

pytestmark = pytest.mark.gpu


# 512 rows: one launch a block; 4,913: three an iteration
@pytest.mark.parametrize("L", [8, 17])
@pytest.mark.parametrize("block,opts", [(48, dict(fixed_iter=48)), (48, dict(fixed_iter=230)), (24, dict(fixed_iter=60)),
                                        (8, dict(fixed_iter=9)), (48, dict(tol=1e-8, max_iter=3000)),
                                        (32, dict(tol=1e-8, max_iter=3000))])
def test_both_entry_points_count_the_same_blocks(L, block, opts):
    H = S.Hamiltonian.from_csr(simple_cubic(L, np.random.default_rng(L).uniform(-1, 1, L ** 3)))
    z = np.linspace(-4, 4, 5) + 0.3j
    blocks = []
    for entry in (S.greens_diag, S.greens_diag_noalloc):
        entry(H, z, [0, 100], block=block, **opts)
        blocks.append(S.last_timing()["blocks"])
    assert blocks[0] == blocks[1]
    if "fixed_iter" in opts:
        looks = max(1, 64 // block)
        done = -(-opts["fixed_iter"] // block)
        assert blocks[0] == -(-done // looks) * looks


@pytest.mark.parametrize("schedule", ["serial", "overlap"])
@pytest.mark.parametrize("L,block", [(8, 48), (8, 8), (17, 48)])
def test_profiling_times_one_update_per_block(L, block, schedule):
    H = S.Hamiltonian.from_csr(simple_cubic(L, np.random.default_rng(L).uniform(-1, 1, L ** 3)))
    z = np.linspace(-4, 4, 5) + 0.3j
    S.set_profiling(True)
    try:
        G = S.greens_diag(H, z, [0, 100], block=block, schedule=schedule, tol=1e-8, max_iter=3000)[0]
        t = S.last_timing()
    finally:
        S.set_profiling(False)
    assert t["update_launches"] == t["blocks"] > 0
    G2 = S.greens_diag(H, z, [0, 100], block=block, schedule=schedule, tol=1e-8, max_iter=3000)[0]
    assert S.last_timing()["blocks"] == t["blocks"] and np.array_equal(G.cpu().numpy(), G2.cpu().numpy())


@pytest.mark.parametrize("K,M", [(40, 3), (30, 16), (20, 50), (300, 70)])
def test_update_counts_of_many_right_hand_sides_are_those_of_each(K, M):
    H = S.Hamiltonian.from_csr(simple_cubic(6, np.random.default_rng(M).uniform(-1, 1, 216)))
    z = np.linspace(-4, 4, M) + 0.3j
    idx = [(7 * j) % 216 for j in range(K)]

    def counts(rhs, entry=S.greens_diag):
        entry(H, z, rhs, block=8, tol=1e-8, max_iter=300)
        return [S.last_timing()[k] for k in ("update_bytes", "update_flops")]

    want = np.sum([counts([j]) for j in sorted(set(idx)) for _ in range(idx.count(j))], axis=0)
    for entry in (S.greens_diag, S.greens_diag_noalloc):
        assert np.array_equal(counts(idx, entry), want)
