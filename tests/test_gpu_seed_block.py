"""The one-launch seed iterations of a block (up to 4096 rows, one workgroup per right-hand side)
against the per-iteration kernels: batched with a matrix too large for one workgroup, a small
matrix goes through the per-iteration kernels, alone through the one-launch form; the results
must be the same bits.  Sizes lie at the edges of the instances (256 ... 4096 rows) and of the
64-row slices, row widths below and above what a lane keeps in registers (7, 12, 17)."""

import numpy as np
import pytest

import paper_0802_0748_amd as S
from workloads import random_sparse_symmetric, simple_cubic
from workloads.csr import coo_to_csr

pytestmark = pytest.mark.gpu


def _banded(n, width, rng):
    """Symmetric band matrix with at most `width` entries per row (odd), the band wrapped around."""
    h = min((width - 1) // 2, (n - 1) // 2)
    i = np.repeat(np.arange(n), h)
    j = (i + np.tile(np.arange(1, h + 1), n)) % n
    v = rng.uniform(-1.0, 1.0, size=len(i))
    d = np.arange(n)
    return coo_to_csr(n, np.concatenate([i, j, d]), np.concatenate([j, i, d]),
                      np.concatenate([v, v, rng.uniform(-2.0, 2.0, size=n)]))


@pytest.fixture(scope="module")
def large():
    return S.Hamiltonian.from_csr(simple_cubic(21, np.random.default_rng(3).uniform(-1, 1, 21 ** 3)))


@pytest.mark.parametrize("n,width", [(1, 1), (63, 7), (65, 17), (256, 7), (257, 17), (300, 11), (512, 17), (513, 11),
                                     (700, 25), (1024, 17), (1024, 7), (1025, 7), (2047, 7), (1500, 17), (2048, 25),
                                     (2049, 7), (4095, 17), (4096, 7)])
def test_one_launch_iterations_match_the_per_iteration_kernels(large, n, width):
    rng = np.random.default_rng(n + width)
    H = S.Hamiltonian.from_csr(_banded(n, width, rng))
    z = np.linspace(-2.5, 2.5, 7) + 1j * np.array([0.2, 0.1, 0.15, 0.1, 0.3, 0.1, 0.2])
    idx = [0, n // 2, n - 1] if n > 2 else [0]
    opts = dict(tol=1e-9, max_iter=400)
    G1, rep1, _, _ = S.greens_diag(H, z, idx, **opts)
    Gb, repb, _ = S.greens_diag_batched([H, large], z, [idx, [5]], **opts)
    assert np.array_equal(G1.cpu().numpy(), Gb[0].cpu().numpy())
    assert np.array_equal(rep1["iters"], repb[0]["iters"])
    assert np.array_equal(rep1["res"], repb[0]["res"])


def test_rows_without_entries_and_uneven_slices(large):
    """Slices of different widths, some of them empty."""
    rng = np.random.default_rng(11)
    n = 700
    i = rng.integers(64, 200, 300)
    j = rng.integers(300, 500, 300)
    key = np.unique(i * n + j)
    i, j = key // n, key % n
    v = rng.uniform(-1, 1, len(i))
    H = S.Hamiltonian.from_csr(coo_to_csr(n, np.concatenate([i, j]), np.concatenate([j, i]), np.concatenate([v, v])))
    z = np.linspace(-1, 1, 5) + 0.2j
    G1, rep1, _, _ = S.greens_diag(H, z, [70, 320, 650], tol=1e-9, max_iter=300)
    Gb, repb, _ = S.greens_diag_batched([H, large], z, [[70, 320, 650], [5]], tol=1e-9, max_iter=300)
    assert np.array_equal(G1.cpu().numpy(), Gb[0].cpu().numpy())
    assert np.array_equal(rep1["iters"], repb[0]["iters"])


def test_up_to_8192_rows_with_many_right_hand_sides(large):
    """4097 to 8192 rows take the one-launch form from 128 right-hand sides on."""
    rng = np.random.default_rng(2)
    for Hc in (simple_cubic(17, rng.uniform(-1, 1, 17 ** 3)), random_sparse_symmetric(4500, 0.004, rng, 2.0)):
        H = S.Hamiltonian.from_csr(Hc)
        z = np.linspace(-3, 3, 4) + 0.3j
        many = list(range(0, 128 * 30, 30))
        G1, rep1, _, _ = S.greens_diag(H, z, many, tol=1e-9, max_iter=300)
        G2, rep2, _, _ = S.greens_diag(H, z, many[:9], tol=1e-9, max_iter=300)
        assert np.array_equal(G1.cpu().numpy()[:, :9], G2.cpu().numpy())
        assert np.array_equal(rep1["iters"][:9], rep2["iters"])
