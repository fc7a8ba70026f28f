"""The shift scalars of a block: 64 shifts per workgroup (many pairs) against 16 (few), and the
shift counts around those group sizes, must give the same bits pair by pair; a block in which
pairs converge, break off and run to its end at once."""

import numpy as np
import pytest
import torch

import paper_0802_0748_amd as S
from workloads import random_sparse_symmetric

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_shift,precision,window", [(63, "fp64", 0), (65, "fp64", 0), (64, "fp32", 0), (70, "fp64", 5)])
def test_many_pairs_equal_few(n_shift, precision, window):
    rng = np.random.default_rng(n_shift)
    n = 90
    H = S.Hamiltonian.from_csr(random_sparse_symmetric(n, 0.06, rng, 2.0))
    z = np.linspace(-3, 3, n_shift) + 1j * np.linspace(0.05, 0.4, n_shift)
    B = torch.from_numpy(rng.normal(size=(300, n)) + 1j * rng.normal(size=(300, n))).cuda()
    opts = dict(tol=1e-9, max_iter=150, precision=precision)
    assert 300 * ((n_shift + 15) // 16) > 1024  # the wide form; the five alone take the narrow one
    if window:
        many, rep, _, _ = S.greens_proj(H, z, B, window=window, **opts)
        few, rep5, _, _ = S.greens_proj(H, z, B[:5], window=window, **opts)
        many = many[:, :5]
    else:
        many, rep, _, _ = S.shifted_cocg_solve(H, z, B, **opts)
        few, rep5, _, _ = S.shifted_cocg_solve(H, z, B[:5], **opts)
        many = many[:5]
    assert torch.equal(torch.view_as_real(many.contiguous()), torch.view_as_real(few))
    for key in ("iters", "status", "res"):
        assert np.array_equal(rep[key][:5], rep5[key])
