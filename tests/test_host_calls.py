"""The library's host code without a GPU (host_calls.py): what it asks of the runtime, in which order
and on which stream and device; and the sizes of its launches, which the runtime takes below 2^32
work-items along a dimension."""
import pytest

import host_calls


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_calls.stand_in(tmp_path_factory)


HELD = r'''
held = {}
def follow(rows):
    """Bytes that the library holds after these calls (in use and idle)."""
    for r in rows:
        if r[0] == "malloc": held[r[1]] = r[2]
        if r[0] == "free": del held[r[1]]
    return sum(held.values())
'''


def test_release_on_a_stream_under_capture(lib):
    """A tree of before the capture, freed on the capturing stream: a node of the graph releases it, and no
    later call is given its memory (a launch of the graph may still read it)."""
    host_calls.run(lib, r'''
t = build()
slabs = [r[1] for r in of(log(), "malloc")]
H.stand_in_capture(S1)
assert L.sbh_free_async(t, S1) == 0
rows = log()
assert not of(rows, "record", "wait", "eventsync"), rows
freed = [r[1] for r in of(rows, "free")]
assert len(freed) == 3 and set(freed) <= set(slabs) and all(r[3] == S1.value for r in of(rows, "free")), rows
H.stand_in_capture(C.c_void_p(-1))
u = build()
assert len(of(log(), "malloc")) == 3   # (the build's temporaries are idle blocks, its tree's arrays new ones)
''')


def test_release_never_waits(lib):
    """Beyond the limit on idle memory, sbh_free_async returns memory in stream order instead of waiting."""
    host_calls.run(lib, HELD + r'''
levels((1, 1), (1 << 20, 1 << 17), (1 << 23, 0))
trees = [build(1 << 24) for _ in range(8)]          # about 1.1 GB each
follow(log())
H.stand_in_events_done(0)                            # the GPU is busy with them
for i, t in enumerate(trees):
    s = S1 if i % 2 else S2
    assert L.sbh_free_async(t, s) == 0
    rows = log()
    assert not of(rows, "eventsync", "streamsync", "devicesync"), rows
    # what goes back was freed on this stream, or waited for by it
    waits = set()
    for r in of(rows, "wait", "free"):
        assert r[3] == s.value, rows
    total = follow(rows)
assert total <= 2 * GIB, total
''')


def test_one_block_beyond_the_limit_leaves_the_others(lib):
    host_calls.run(lib, HELD + r'''
other = build()
assert L.sbh_free_async(build(200000), S1) == 0
follow(log())
assert L.sbh_mlp_loss_grad(D, D, D, D, 1 << 28, S1, D) == 0   # a workspace of 27 GB
rows = log()
assert max(r[2] for r in of(rows, "malloc")) > 2 * GIB
assert follow(rows) <= 2 * GIB and not of(rows, "eventsync", "streamsync", "devicesync")
u = build(200000)
assert not of(log(), "malloc")                       # the tree's blocks are there still
''')


def test_memory_goes_back_on_its_own_device(lib):
    host_calls.run(lib, HELD + r'''
t, u = build(), build()
follow(log())
H.hipSetDevice(1)
assert L.sbh_free(t) == 0 and L.sbh_free(u) == 0
rows = log()
assert follow(rows) == 0
assert len(of(rows, "devicesync")) >= 2
bad = [r for r in rows if r[0] in ("record", "wait", "free", "devicesync", "streamsync") and r[3] == 0 and r[4] != "dev0"]
assert not bad, bad
d = C.c_int(-1)
H.hipGetDevice(C.byref(d))
assert d.value == 1                                  # the caller's device again
''')


def test_memory_goes_back(lib):
    host_calls.run(lib, HELD + r'''
KEEP = 64 << 20
# a training call without a tree: its workspace of 1.7 GB is not kept
assert L.sbh_mlp_train(D, D, D, D, D, 1 << 24, 1, 1 << 24, 1e-3, 0, S1, None) == 0
rows = log()
assert follow(rows) <= KEEP and not of(rows, "eventsync", "streamsync", "devicesync"), rows
assert L.sbh_mlp_loss_grad(D, D, D, D, 1 << 24, S1, D) == 0
assert follow(log()) <= KEEP
# a small one is: no allocation the second time
assert L.sbh_mlp_train(D, D, D, D, D, 8192, 1, 8192, 1e-3, 0, S1, None) == 0
follow(log())
assert L.sbh_mlp_train(D, D, D, D, D, 8192, 1, 8192, 1e-3, 0, S1, None) == 0
assert not of(log(), "malloc")
# nor what a build that failed had taken
H.stand_in_refuse(1000)
h = C.c_void_p()
assert L.sbh_build(D, D, None, 1 << 22, None, S1, C.byref(h)) == -2
H.stand_in_refuse(0)
assert follow(log()) <= KEEP
raw = struct.pack("8f44I", 0, 0, 0, 1, 1, 1, 0, 0, *[0] * 44)   # not finite
H.stand_in_info(raw, len(raw))
assert L.sbh_build(D, D, None, 1 << 22, None, S1, C.byref(h)) == -1
assert follow(log()) <= KEEP
# a loop of builds allocates once
levels((1, 1), (8, 0))
for i in range(3):
    assert L.sbh_free_async(build(1 << 20), S1) == 0
    rows = log()
    follow(rows)
    assert i == 0 or not of(rows, "malloc"), rows
assert sum(held.values()) > KEEP
# what it leaves goes back when the allocator is set, also to the one it is
assert L.sbh_set_allocator(None, None, None) == 0
assert follow(log()) == 0
# or with the last tree that is freed
t, u = build(1 << 20), build(1 << 20)
follow(log())
assert L.sbh_free_async(t, S1) == 0 and L.sbh_free(u) == 0
assert follow(log()) == 0
''')


def test_idle_memory_is_used_before_an_allocation_fails(lib):
    host_calls.run(lib, HELD + r'''
assert L.sbh_free_async(build(1 << 20), S1) == 0
follow(log())
assert sum(held.values()) > 0
before = set(held)
H.stand_in_events_done(0)
H.stand_in_refuse(1)
t = build(1 << 22, stream=S2)
rows = log()
follow(rows)
assert not before & set(held)                        # all of it went back, and the build went on
assert all(r[3] == S2.value for r in of(rows, "free", "streamsync", "wait")) and not of(rows, "eventsync", "devicesync")
''')


def test_release_leaves_the_last_error(lib):
    """An error that the caller has not read yet is still there after a release; a release's own queries
    leave none."""
    host_calls.run(lib, r'''
trees = [build() for _ in range(3)]
H.stand_in_error(98)
assert L.sbh_free_async(trees[0], S1) == 0
assert H.hipGetLastError() == 98
H.stand_in_events_done(0)
assert L.sbh_free_async(trees[1], S2) == 0
assert H.hipGetLastError() == 0
H.stand_in_events_done(1)
H.stand_in_error(98)
assert L.sbh_free(trees[2]) == 0
assert H.hipGetLastError() == 98
''')


def test_barnes_hut_launches(lib):
    host_calls.run(lib, r'''
for d in (2, 4):
    t = build(5000, branching=d, normals=True)
    for nq in (1, 1 << 16, (1 << 18) + 1, (1 << 30) - 1, 1 << 30, (1 << 31) - 65, (1 << 31) - 1):
        for beta in (0.1, 0.3, 0.5, 2.0, 1e9):
            for kernel in (0, 1, 2):
                log()
                assert L.sbh_eval(t, D, nq, kernel, beta, 0, 0, None, S1, D) == 0, (d, nq, beta, L.sbh_last_error())
                rows = of(log(), "launch")
                assert len(rows) == 1 and (nq + 63) // 64 * 64 <= rows[0][2] < 1 << 32, rows
''')


def test_target_launches(lib):
    host_calls.run(lib, r'''
t = build(5000, normals=True)
H.stand_in_copy_args(7, 0)
for nq, depth in ((5, 3), ((1 << 20) - 1, 1), (1 << 20, 1), (1 << 21, 1), ((1 << 28) - 1, 1), (1 << 20, 20), (3000001, 7)):
    for kernel, eps in ((0, 1e-3), (0, 0.0), (1, 0.0), (2, 0.0)):
        o = P.EvalOpts(); L.sbh_eval_opts_default(C.byref(o)); o.eps = eps
        log()
        assert L.sbh_mlp_pairs(t, D, nq, kernel, 0, depth, C.byref(o), S1, D, D, D, D) == 0, (nq, depth, L.sbh_last_error())
        rows = of(log(False), "launch")
        path = 0
        for i, r in list(enumerate(rows))[1:]:       # (the first one walks the paths)
            a = [H.stand_in_arg(7 * i + k) for k in range(7)]
            assert path % 8 == 0
            assert a[1] == D.value + 12 * (path // 8) and a[3] == D.value + 16 * depth * path
            assert a[6] == D.value + 32 * depth * path
            path += r[2] // H.stand_in_block(i)
        assert path == 8 * nq, (path, nq)
''')


def test_gradient_launches(lib):
    host_calls.run(lib, r'''
H.stand_in_copy_args(8, 256)
for n in (1, 64, 65, (1 << 30) - 64, 1 << 30, (1 << 31) - 1):
    log()
    assert L.sbh_mlp_loss_grad(D, D, D, D, n, S1, D) == 0, (n, L.sbh_last_error())
    rows = of(log(False), "launch")
    first, part = 0, H.stand_in_arg(7)
    for i, r in enumerate(rows[:-1]):          # (the last one adds the partial gradients)
        a = [H.stand_in_arg(8 * i + k) for k in range(8)]
        assert a[4] == n and a[5] == first and a[7] == part + first // 64 * 1616 * 4
        assert r[2] // 256 == (min(a[6], n - first) + 63) // 64
        first += a[6]
        assert first == n or first % 64 == 0
    assert first == n
''')


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
