"""The library's host code without a GPU (host_calls.py): what it asks of the runtime, in which order
and on which stream and device; and the sizes of its launches, which the runtime takes below 2^32
work-items along a dimension."""
import pytest

import host_calls


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_calls.stand_in(tmp_path_factory)


def test_brute_force_launches(lib):
    host_calls.run(lib, r'''
H.stand_in_copy_args(9, 0)
for nq in (1, 16384, 32768, 65536, (1 << 28) + 77, 1 << 29, (1 << 30) + 1, 1 << 31, (1 << 32) + 12345):
    for n, kernel, fp64 in ((n, k, f) for n in (100, 1000) for k in (0, 1, 2) for f in (0, 1)):
        log()
        assert L.sbh_brute(D, D, D, n, D, nq, kernel, None, fp64, S1, D) == 0, (nq, kernel, L.sbh_last_error())
        rows = of(log(False), "launch")
        first = 0
        for i, r in enumerate(rows):
            a = [H.stand_in_arg(9 * i + k) for k in range(9)]
            assert a[4] == D.value + 12 * first and a[8] == D.value + (8 if fp64 else 4) * first, (i, first)
            groups = r[2] // H.stand_in_block(i)
            assert any(groups == -(-a[5] // (64 * u)) for u in (1, 2, 4))   # queries a lane
            first += a[5]
        assert first == nq
''')
