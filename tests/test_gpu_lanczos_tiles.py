"""The LDS-tiled Lanczos step of the matrix-free Hubbard operator (down-spin blocks of 256 to 3841
configurations, one to four rows per thread; 252 takes the general step) against the stored sector
matrix: rows, their terms' order and the tiles' sums are the same, so the results are equal bit for
bit."""

import numpy as np
import pytest
import torch

import paper_0802_0748_amd as S
from workloads import hubbard_ring

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,n_up,n_dn", [(10, 3, 5), (11, 5, 4), (11, 1, 5), (12, 2, 6), (13, 2, 5), (13, 1, 6), (14, 1, 6), (14, 3, 7)])
@pytest.mark.parametrize("t", [1.0, -0.7])
def test_tiled_lanczos_matches_the_stored_matrix(L, n_up, n_dn, t):
    rng = np.random.default_rng(L)
    Hs = S.Hamiltonian.from_csr(hubbard_ring(L, n_up, n_dn, t=t, U=4.0, V=1.0), validate=False)
    Hm = S.Hamiltonian.hubbard(L, n_up, n_dn, t=t, U=4.0, V=1.0)
    b = torch.from_numpy(rng.normal(size=Hs.n)).cuda()
    z = np.linspace(-8, 18, 5) + 0.5j
    for got, want in zip(S.krylov_greens_vec(Hm, z, b, 25), S.krylov_greens_vec(Hs, z, b, 25)):
        assert torch.equal(torch.as_tensor(got), torch.as_tensor(want))


@pytest.mark.parametrize("L,n_up,n_dn", [(11, 2, 5), (12, 2, 6), (14, 1, 6)])
def test_ground_state_from_tiled_steps(L, n_up, n_dn):
    # the estimate's vector is equal bit for bit; the refinement's solves sum p.q per block (rounding,
    # far below the residual bound of 1e-10 that both meet: E0 within 1e-9)
    Hs = S.Hamiltonian.from_csr(hubbard_ring(L, n_up, n_dn, t=1.0, U=4.0, V=1.0), validate=False)
    Hm = S.Hamiltonian.hubbard(L, n_up, n_dn, t=1.0, U=4.0, V=1.0)
    x0 = np.random.default_rng(L).normal(size=Hs.n)
    s, m = S.ground_state(Hs, x0), S.ground_state(Hm, x0)
    assert abs(s[1] - m[1]) < 1e-9 and s[2] == m[2] and s[4] == m[4]
