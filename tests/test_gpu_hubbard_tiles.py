"""The LDS-tiled matrix-free Hubbard product in each of its forms (down-spin blocks of up to 512,
1024, 2048 and 4096 configurations, one to four rows per thread) against the stored sector matrix.
The products of a row are the same; p.q is summed block by block, so solutions agree to rounding:
within 1e-10 relative, the bar of the fixed-iteration comparisons."""

import numpy as np
import pytest
import torch

import paper_0802_0748_amd as S
from workloads import hubbard_ring

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,n_up,n_dn", [(11, 1, 4), (11, 5, 4), (12, 2, 6), (13, 2, 5), (13, 1, 6), (14, 1, 6), (14, 2, 7)])
@pytest.mark.parametrize("n_rhs", [1, 3])
def test_tiled_products_match_the_stored_matrix(L, n_up, n_dn, n_rhs):
    rng = np.random.default_rng(L)
    Hs = S.Hamiltonian.from_csr(hubbard_ring(L, n_up, n_dn), validate=False)
    Hm = S.Hamiltonian.hubbard(L, n_up, n_dn)
    assert Hs.n == Hm.n and Hs.nnz == Hm.nnz
    B = torch.from_numpy(rng.normal(size=(n_rhs, Hs.n)) + 1j * rng.normal(size=(n_rhs, Hs.n))).cuda()
    z = np.linspace(-8, 18, 5) + 2.0j
    Xs = S.shifted_cocg_solve(Hs, z, B, fixed_iter=12)[0]
    Xm = S.shifted_cocg_solve(Hm, z, B, fixed_iter=12)[0]
    diff = torch.linalg.vector_norm(Xs - Xm, dim=-1) / torch.linalg.vector_norm(Xs, dim=-1)
    assert float(diff.max()) < 1e-10
