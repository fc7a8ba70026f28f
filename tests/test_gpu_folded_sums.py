"""Seed iterations whose reductions are folded into the vector kernels (stored matrices of 4,097 to 65,536
rows) against those with launches of their own: a right-hand side gives the same bits alone (folded) and in
one solve with a lattice of 65,537 rows (not folded), for blocks of one iteration, two and more, one
right-hand side and odd counts, at the first and the last number of tiles; and the projection partials
against the projections of full solutions (1e-10, the bar of the fixed-iteration comparisons)."""

import numpy as np
import pytest
import torch

import paper_0802_0748_amd as S
from workloads.csr import coo_to_csr

pytestmark = pytest.mark.gpu


def _ring(n):
    rng = np.random.default_rng(n)
    i = np.arange(n)
    r, c, v = [i], [i], [rng.normal(size=n)]
    for d in (1, 7):
        t = 0.5 * rng.normal(size=n)
        r += [i, (i + d) % n]
        c += [(i + d) % n, i]
        v += [t, t]
    return S.Hamiltonian.from_csr(coo_to_csr(n, np.concatenate(r), np.concatenate(c), np.concatenate(v)))


@pytest.fixture(scope="module")
def big():
    return _ring(65537)


@pytest.mark.parametrize("n", [4097, 65536])
@pytest.mark.parametrize("rhs", [1, 3, 4])
@pytest.mark.parametrize("block,opts", [(1, dict()), (2, dict()), (8, dict(tol=1e-6)), (0, dict(tol=1e-6)), (4, dict(fixed_iter=13)),
                                        (8, dict(max_iter=20))])
def test_folded_and_separate_sums_give_the_same_bits(big, n, rhs, block, opts):
    H = _ring(n)
    z = np.linspace(-1.5, 1.5, 6) + 0.3j
    idx = [(k * 977 + 3) % n for k in range(rhs)]
    o = dict(dict(tol=1e-4, block=block), **opts)
    G1, rep1, _ = S.greens_diag(H, z, idx, **o)[:3]
    G2, rep2, _ = S.greens_diag_batched([H, big], z, [idx, [0]], **o)[:3]
    assert torch.equal(G1, G2[0])
    for key in ("iters", "status"):
        assert np.array_equal(rep1[key], rep2[0][key])


@pytest.mark.parametrize("n,rhs", [(4097, 1), (5000, 3)])
def test_folded_projection_partials(n, rhs):
    H = _ring(n)
    rng = np.random.default_rng(rhs)
    B, W = (torch.from_numpy(rng.normal(size=(rhs, n)) + 1j * rng.normal(size=(rhs, n))).cuda() for _ in range(2))
    z = np.linspace(-1.5, 1.5, 6) + 0.3j
    X = S.shifted_cocg_solve(H, z, B, fixed_iter=11, seed_index=3)[0]
    G = S.greens_proj(H, z, B, W, fixed_iter=11, seed_index=3)[0]
    want = (X.cpu().numpy() * W.cpu().numpy()[:, None, :]).sum(-1).T
    assert np.max(np.abs(G.cpu().numpy() - want) / np.abs(want).max()) < 1e-10
