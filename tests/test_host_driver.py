"""The host's loop over blocks, on the host: every right-hand side reads as stopped at the first look."""

import pytest

from host_library import run


@pytest.mark.parametrize("entry", ["greens_diag", "greens_diag_noalloc"])
@pytest.mark.parametrize("block", [1, 2, 8, 48])
def test_a_round_launched_ahead_does_not_count_against_the_block_limit(entry, block, tmp_path):
    """Short calls in blocks of one or two iterations: the round that was launched before the look is beyond
    what the iterations could need."""
    run(f"""
_, H = upload(*band(300, 7))
for K, M, opts in ((1, 1, dict(max_iter=1)), (1, 1, dict(fixed_iter=9)), (1, 3, dict(max_iter=20)), (2, 5, dict(max_iter=9))):
    assert greens(H, K, M, entry={entry!r}, block={block}, **opts) == C.OK, lib.scocg_last_error()
    assert launched('k_seed_block') > 0
""", tmp_path)
