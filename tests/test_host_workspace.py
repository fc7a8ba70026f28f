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
