"""The recurrence of many unit vectors around the lines of its launches: 256 and 257 tiles (sums folded
into the next kernel, or kernels of their own), and group counts that fill the XCD-placed rows of the
grid, or leave some over.  A right-hand side gives the same bits alone and in any batch, and one is held
to the reference recurrence (coefficients within 1e-10, the bar of the other comparisons)."""

import numpy as np
import pytest
import torch

import paper_0802_0748_amd as S
from oracle import krylov as K
from workloads.csr import coo_to_csr

pytestmark = pytest.mark.gpu


def _ring(n, rng):
    i = np.arange(n)
    r, c, v = [i], [i], [rng.normal(size=n)]
    for d in (1, 7):
        t = rng.normal(size=n)
        r += [i, (i + d) % n]
        c += [(i + d) % n, i]
        v += [t, t]
    return coo_to_csr(n, np.concatenate(r), np.concatenate(c), np.concatenate(v))


@pytest.mark.parametrize("n,rhs", [(65, 1), (256, 5), (300, 33), (700, 128), (513, 130), (65536, 9), (65537, 9)])
def test_right_hand_sides_alone_and_in_groups(n, rhs):
    Hc = _ring(n, np.random.default_rng(n))
    H = S.Hamiltonian.from_csr(Hc)
    idx = np.random.default_rng(rhs).integers(0, n, rhs)
    z = np.linspace(-1.0, 1.0, 4) + 0.2j
    G, ab, dim = S.krylov_greens_diag(H, z, idx, 12)
    for c in {0, rhs // 2, rhs - 1}:
        G1, ab1, dim1 = S.krylov_greens_diag(H, z, idx[c:c + 1], 12)
        assert torch.equal(G[:, c], G1[:, 0]) and torch.equal(ab[c], ab1[0]) and dim[c] == dim1[0]
    a, b = K.lanczos(Hc, int(idx[-1]), 12)
    assert dim[-1] == len(a)
    assert np.max(np.abs(ab[-1, 0, :len(a)].cpu().numpy() - a)) < 1e-10
    assert np.max(np.abs(ab[-1, 1, :len(b)].cpu().numpy() - b)) < 1e-10
