"""The three forms of the seed iteration (one launch a block; sums folded into three launches an iteration;
sums in launches of their own) where they leave the plain path: breakdown at the first step and at a
later one, the partials of a vector projection, and the residuals they report."""

import numpy as np
import pytest
import torch

import paper_0802_0748_amd as S
from workloads.csr import coo_to_csr

pytestmark = pytest.mark.gpu


def _band(n, width):
    """Symmetric band of `width` entries a row (odd), wrapped around."""
    rng = np.random.default_rng(n + width)
    h = (width - 1) // 2
    i = np.repeat(np.arange(n), h)
    j = (i + np.tile(np.arange(1, h + 1), n)) % n
    v = rng.uniform(-1, 1, len(i)) / np.sqrt(width)
    d = np.arange(n)
    return S.Hamiltonian.from_csr(coo_to_csr(n, np.concatenate([i, j, d]), np.concatenate([j, i, d]),
                                             np.concatenate([v, v, rng.uniform(-2, 2, n)])))


def _operators():
    """One operator per form: 300 and 4,500 rows, 65,537 rows, and a matrix-free one (11 sites, 2 + 5)."""
    return [lambda: _band(300, 7), lambda: _band(4500, 7), lambda: _band(65537, 7), lambda: S.Hamiltonian.hubbard(11, 2, 5)]


@pytest.mark.parametrize("form", range(4))
@pytest.mark.parametrize("block", [1, 4, 48])
def test_first_step_breakdown_leaves_the_other_right_hand_sides_alone(form, block):
    H = _operators()[form]()
    rng = np.random.default_rng(form)
    B = np.zeros((4, H.n), dtype=complex)
    B[1, 3], B[1, 270] = 1, 1j  # b.b = 0 (in two tiles where there are two)
    B[2], B[3] = (rng.normal(size=H.n) + 1j * rng.normal(size=H.n) for _ in range(2))
    B = torch.from_numpy(B).cuda()
    z = np.array([0.3 + 0.4j, 1.0 + 0.5j, -2.0 + 0.3j])
    o = dict(fixed_iter=9, block=block)
    X, rep, _, rc = S.shifted_cocg_solve(H, z, B, allow_breakdown=True, **o)
    assert rc == 4
    assert not torch.any(X[:1] != 0) and np.all(rep["status"][0] == 0)
    assert np.all(rep["status"][1] == 4) and np.all(rep["iters"][1] == 0)
    for j in (2, 3):
        Xj, repj, _, _ = S.shifted_cocg_solve(H, z, B[j:j + 1], **o)
        assert torch.equal(torch.view_as_real(X[j]), torch.view_as_real(Xj[0]))
        assert np.array_equal(rep["status"][j], repj["status"][0]) and np.array_equal(rep["res"][j], repj["res"][0])


@pytest.mark.parametrize("n", [300, 4500, 65537])
@pytest.mark.parametrize("block", [1, 4, 48])
def test_breakdown_at_the_second_step(n, block):
    # H = 0 and the seed at 2i: one step solves the seed system exactly (alpha = 1 / 2i), the next finds p.q = 0
    d = np.arange(n)
    H = S.Hamiltonian.from_csr(coo_to_csr(n, d, d, np.zeros(n)))
    B = torch.zeros((3, n), dtype=torch.complex128, device="cuda")
    B[0, 0], B[1, n - 1], B[2, n // 2] = 1, 2j, -1
    z = np.array([2j, 1 + 2j])
    X, rep, _, rc = S.shifted_cocg_solve(H, z, B, fixed_iter=5, seed_index=0, block=block, allow_breakdown=True)
    assert rc == 4 and np.all(rep["status"] == 4) and np.all(rep["iters"] == 1)
    assert np.array_equal(X[:, 0].cpu().numpy(), B.cpu().numpy() / 2j)


@pytest.mark.parametrize("n,width,many,few", [
    # the same right-hand sides in one launch a block (many) and in launches per iteration (few)
    (700, 401, 160, 1), (1024, 257, 160, 1), (2048, 129, 160, 1), (4096, 33, 160, 1), (4500, 7, 128, 9), (8192, 7, 128, 2)])
def test_projection_partials_of_both_forms_are_the_same_bits(n, width, many, few):
    H = _band(n, width)
    rng = np.random.default_rng(n)
    B, W = (torch.from_numpy(rng.normal(size=(many, n)) + 1j * rng.normal(size=(many, n))).cuda() for _ in range(2))
    z = np.linspace(-1.5, 1.5, 5) + 0.3j
    G, rep = S.greens_proj(H, z, B, W, tol=1e-9, max_iter=70)[:2]
    G1, rep1 = S.greens_proj(H, z, B[:few], W[:few], tol=1e-9, max_iter=70)[:2]
    assert torch.equal(torch.view_as_real(G[:, :few].contiguous()), torch.view_as_real(G1))
    for key in ("iters", "status", "res"):
        assert np.array_equal(rep[key][:few], rep1[key])


@pytest.mark.parametrize("n,width", [(200, 17), (256, 7), (257, 11), (512, 17), (700, 11), (1024, 7), (2048, 7)])
def test_projection_partials_with_the_matrix_in_registers(n, width):
    # against the projections of full solutions (1e-10, the bar of the fixed-iteration comparisons)
    H = _band(n, width)
    rng = np.random.default_rng(n)
    B, W = (torch.from_numpy(rng.normal(size=(3, n)) + 1j * rng.normal(size=(3, n))).cuda() for _ in range(2))
    z = np.linspace(-1.5, 1.5, 6) + 0.3j
    X = S.shifted_cocg_solve(H, z, B, fixed_iter=11, seed_index=3)[0]
    G = S.greens_proj(H, z, B, W, fixed_iter=11, seed_index=3)[0]
    want = (X.cpu().numpy() * W.cpu().numpy()[:, None, :]).sum(-1).T
    assert np.max(np.abs(G.cpu().numpy() - want) / np.abs(want).max()) < 1e-10


@pytest.mark.parametrize("n,rhs,block", [(4097, 3, 8), (4097, 1, 0), (65536, 4, 0), (65536, 3, 2)])
def test_residuals_of_folded_and_separate_sums(n, rhs, block):
    H, big = _band(n, 7), _band(65537, 7)
    z = np.linspace(-1.5, 1.5, 6) + 0.3j
    idx = [(k * 977 + 3) % n for k in range(rhs)]
    rep1 = S.greens_diag(H, z, idx, tol=1e-6, block=block)[1]
    rep2 = S.greens_diag_batched([H, big], z, [idx, [0]], tol=1e-6, block=block)[1]
    assert np.array_equal(rep1["res"], rep2[0]["res"])


@pytest.mark.parametrize("rhs,block", [(1, 1), (3, 0), (4, 8)])
@pytest.mark.parametrize("n", [65537, 66000])
def test_one_row_per_thread_in_uneven_batches(n, rhs, block):
    """Batches of uneven right-hand sides beyond the folded sums against the same right-hand sides alone."""
    H, small = _band(n, 7), _band(4500, 7)
    z = np.linspace(-1.5, 1.5, 6) + 0.3j
    idx = [(k * 977 + 3) % n for k in range(rhs)]
    G1, rep1 = S.greens_diag(H, z, idx, tol=1e-6, block=block)[:2]
    G2, rep2 = S.greens_diag_batched([small, H], z, [[0], idx], tol=1e-6, block=block)[:2]
    assert torch.equal(G1, G2[1])
    for key in ("iters", "status", "res"):
        assert np.array_equal(rep1[key], rep2[1][key])
