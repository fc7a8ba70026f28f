"""Work buffers kept between calls, on the host: the library runs on a runtime whose memory is counted and
can run out."""

from host_library import run


def test_an_upload_that_finds_no_memory_takes_back_the_kept_buffers(tmp_path):
    run("""
_, H = upload(*band(200000, 3))
matrix = fake.fake_live()
assert krylov_vec(H) == C.OK
kept = fake.fake_live() - matrix
assert kept >= 3 * 200000 * 8
# no room for the second matrix but for the kept buffers
fake.fake_set_limit(fake.fake_live() + (2 << 20))
rc, H2 = upload(*band(20000, 9))
assert fake.fake_refused() > 0
assert rc == C.OK, lib.scocg_last_error()
# and the matrix-free operator's tables likewise
fake.fake_set_limit(1 << 40)
assert krylov_vec(H) == C.OK
fake.fake_set_limit(fake.fake_live() + (1 << 20))
refused = fake.fake_refused()
hubbard(18, 9, 2)
assert fake.fake_refused() > refused
""", tmp_path)


def test_keeping_a_buffer_needs_no_host_memory(tmp_path):
    """A call's buffers are handed back in destructors, which may not throw: with operator new failing from
    the first wait on, the call ends as ever."""
    run("""
_, H = upload(*band(200000, 3))
matrix = fake.fake_live()
for again in range(3):
    fake.fake_new_fails_after_sync(1)
    rc = krylov_vec(H)
    fake.fake_new_fails_after_sync(0)
    assert rc == C.OK, lib.scocg_last_error()
    assert fake.fake_live() - matrix >= 3 * 200000 * 8
# more than is kept: the oldest go
for n in range(4 << 20, 14 << 20, 2 << 20):
    _, Hn = upload(*band(n, 1))
    fake.fake_new_fails_after_sync(1)
    assert krylov_vec(Hn) == C.OK
    fake.fake_new_fails_after_sync(0)
    lib.csr_free(Hn)
assert 900 << 20 <= fake.fake_live() - matrix <= (1 << 30) + (1 << 20)
lib.csr_free(H)
assert fake.fake_live() == 0
""", tmp_path)


def test_a_caller_gets_the_kept_buffers_back(tmp_path):
    run("""
_, H = upload(*band(200000, 3))
matrix = fake.fake_live()
assert krylov_vec(H) == C.OK
assert fake.fake_live() > matrix
lib.scocg_release_workspace()
assert fake.fake_live() == matrix
assert krylov_vec(H) == C.OK
""", tmp_path)
