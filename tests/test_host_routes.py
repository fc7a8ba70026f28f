"""Which kernels a call launches, on the host: the library runs on a runtime that records launches."""

import pytest

from host_library import run

_SEED_BLOCK = """
def one_launch(K, *matrices):
    seen = []
    Hs = [upload(*m)[1] for m in matrices]
    if len(Hs) == 1:
        for entry in ('greens_diag', 'greens_diag_noalloc')[:1 if K * len(matrices[0][0]) > 60000 else 2]:
            fake.fake_forget()
            assert greens(Hs[0], K, entry=entry) == C.OK, lib.scocg_last_error()
            seen.append(launched('k_seed_block') > 0)
            assert seen[-1] != (launched('k_spmv') > 0)
    else:
        fake.fake_set_word(SEED_STOPPED)
        fake.fake_forget()
        h = (ctypes.c_void_p * len(Hs))(*[H.value for H in Hs])
        nr = np.full(len(Hs), K // len(Hs), dtype=np.int64)
        idx = np.zeros(K, dtype=np.int64)
        z, o = np.array([0.5j]), C.Opts()
        lib.scocg_default_opts(ctypes.byref(o))
        assert lib.greens_diag_batched(len(Hs), h, nr.ctypes.data, idx.ctypes.data, 1, z.ctypes.data, ctypes.byref(o),
                                       OUT, None, None) == C.OK
        seen.append(launched('k_seed_block') > 0)
    for H in Hs:
        lib.csr_free(H)
    assert len(set(seen)) == 1, seen
    return seen[0]


def uneven(n, heavy, width):
    # a band of 7 entries whose first `heavy` rows (and the columns of the same numbers) have `width`
    # entries more, spread over the columns
    rp, col, val = band(n, 7)
    rows = [set(col[rp[i]:rp[i + 1]]) for i in range(n)]
    for i in range(heavy):
        for j in (i + np.arange(width) * (n // width)) % n:
            rows[i].add(j)
            rows[j].add(i)
    rows = [sorted(r) for r in rows]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    col = np.concatenate(rows).astype(np.int64)
    return rp, col, np.ones(len(col))

"""


@pytest.mark.parametrize("what,one", [
    # narrow rows, and wide ones of few rows: one workgroup's stream is short
    ("1, band(4096, 9)", True), ("4, band(4096, 17)", True), ("1, band(512, 511)", True), ("1, band(1024, 65)", True),
    ("16, band(1024, 257)", True),
    # wide rows that the launches spread over the chip
    ("1, band(4096, 33)", False), ("1, band(2048, 129)", False), ("16, band(4096, 65)", False),
    ("64, band(4096, 257)", False), ("1, band(1024, 257)", False), ("1, uneven(4096, 1, 4096)", False),
    # uneven rows: a wave's chain of slots is longer than the mean
    ("1, uneven(4096, 64, 200)", True), ("1, uneven(4096, 256, 200)", False), ("1, uneven(2048, 256, 400)", False),
    # until there are enough right-hand sides for the whole chip
    ("256, band(4096, 257)", True), ("128, band(6000, 17)", True), ("128, band(6000, 129)", False),
    ("127, band(6000, 7)", False),
    # ... and not for a few more than one round of workgroups
    ("260, band(4096, 65)", False), ("512, band(4096, 65)", True), ("260, band(6000, 17)", False), ("256, band(6000, 17)", True),
    ("260, band(4096, 7)", True), ("400, band(512, 511)", True),
    # one wide matrix of a batch is enough
    ("2, band(300, 7), band(4000, 129)", False), ("2, band(300, 7), band(4000, 7)", True)])
def test_one_launch_iterations_only_where_one_workgroup_streams_as_fast(what, one, tmp_path):
    run(_SEED_BLOCK + f"assert one_launch({what}) is {one}", tmp_path)


_TILED = """
def tiled(L, n_up, n_dn):
    H = hubbard(L, n_up, n_dn)
    fake.fake_forget()
    assert krylov_vec(H) == C.OK, lib.scocg_last_error()
    assert (launched('k_lz_hub') > 0) != (launched('k_lz_matvec') > 0)
    return launched('k_lz_hub') > 0

"""


@pytest.mark.parametrize("sector,is_tiled", [
    # up to 65,536 rows the general product folds its sums: two launches a step instead of five
    ("11, 0, 5", False), ("11, 1, 5", False), ("14, 1, 7", False), ("12, 2, 6", False), ("13, 2, 6", True), ("11, 5, 5", True),
    ("14, 3, 7", True), ("10, 5, 5", False), ("16, 2, 8", False)])
def test_tiled_lanczos_steps_only_beyond_the_folded_sums(sector, is_tiled, tmp_path):
    run(_TILED + f"assert tiled({sector}) is {is_tiled}", tmp_path)


def test_launches_of_the_tiled_step_stay_below_2_32_threads(tmp_path):
    """25 sites with 11 + 2 electrons: 4.5 million blocks of 1024 threads would be one launch of more than
    2^32 threads along x, which the runtime refuses; the general step takes the sector."""
    run("""
H = hubbard(25, 11, 2)
assert krylov_vec(H, 1) == C.OK
assert launched('k_lz') > 0
assert max(fake.fake_threads_x(i) for i in range(fake.fake_launches())) < 1 << 32
""", tmp_path)


def test_launch_of_the_shift_scalars_does_not_grow_along_x_with_the_right_hand_sides(tmp_path):
    """8 threads of it per pair, counted along x, would pass 2^32 at 5.4e8 pairs (one thread per pair, as the
    other launches have, at 4.3e9)."""
    run("""
_, H = upload(*band(64, 3))
for K, M in ((3, 5), (3000, 64), (65535, 2), (2, 70000)):
    fake.fake_forget()
    greens(H, K, M, block=1)
    x = [fake.fake_threads_x(i) for i in range(fake.fake_launches()) if b'k_pair_scalars' in fake.fake_name(i)]
    assert x and max(x) <= 16 * (M + 63), (K, M, max(x))
""", tmp_path)


@pytest.mark.parametrize("K,M,threads", [(20000, 1, 64), (3000, 4, 64), (3000, 16, 256), (2, 70, 5 * 256), (400, 70, 5 * 256)])
def test_shift_scalars_take_no_more_threads_than_the_shifts_of_a_right_hand_side_need(K, M, threads, tmp_path):
    run(f"""
_, H = upload(*band(64, 3))
greens(H, {K}, {M}, block=4)
x = [fake.fake_threads_x(i) for i in range(fake.fake_launches()) if b'k_pair_scalars' in fake.fake_name(i)]
assert x and set(x) == {{{threads}}}, set(x)
""", tmp_path)


def test_products_of_iterations_that_are_not_folded_take_the_instance_without_the_state(tmp_path):
    """The instance that brings the seed state up to date needs more registers: only the folded iterations
    (from a block's second one on) take it."""
    run("""
for n, K, folded in ((5000, 3, True), (5000, 1, True), (66000, 3, False), (66000, 1, False), (33000, 64, False)):
    _, H = upload(*band(n, 3))
    fake.fake_forget()
    assert greens(H, K, 1, block=4) == C.OK, lib.scocg_last_error()
    rb = 2 if K > 1 else 1
    plain, state = [launched(f'k_spmvILi{rb}ELb0ELb{f}E') for f in (0, 1)]
    assert plain > 0 and state == (3 * plain if folded else 0), (n, K, plain, state)
    lib.csr_free(H)
""", tmp_path)


def test_uneven_batches_beyond_the_folded_sums_keep_one_row_per_thread(tmp_path):
    run(_SEED_BLOCK + """
for matrices, rows in (((band(66000, 3), band(300, 3)), True), ((band(6000, 3), band(300, 3)), False),
                       ((band(66000, 3), band(66000, 3)), False)):
    one_launch(2, *matrices)
    assert (launched('k_pupd_rows') > 0) == rows and (launched('k_rupd_rows') > 0) == rows
    assert (launched('k_pupdI') > 0) != rows and (launched('k_rupdI') > 0) != rows
""", tmp_path)
