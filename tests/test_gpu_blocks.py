"""The default allocator's kept blocks: builds from several threads and streams while trees are freed
in stream order give the trees a lone build gives, and the memory goes back with the last tree."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _cloud(n, seed):
    g = torch.Generator().manual_seed(seed)
    return (torch.rand(n, 3, generator=g).cuda(), (torch.rand(n, generator=g) + 0.5).cuda(),
            torch.rand(777, 3, generator=g).cuda())


@pytest.mark.parametrize("threads", [1, 3])
def test_builds_on_several_streams_reuse_blocks_safely(threads):
    import paper_2506_02219_amd as P
    sizes = [1, 9, 5000, 60001, 61007, 200003]
    clouds = [_cloud(n, i) for i, n in enumerate(sizes)]
    want = []
    for s, w, q in clouds:
        t = P.sbh_build(s, w)
        want.append((t.n_nodes, P.sbh_eval(t, q, P.POTENTIAL, seed=1, group=64).cpu().numpy()))
        t.free()
    torch.cuda.synchronize()
    bad = []

    def work(k):
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        got = []
        for r in range(12):
            i = (r * 5 + k) % len(sizes)
            st = streams[r % 2]
            with torch.cuda.stream(st):
                s, w, q = clouds[i]
                t = P.sbh_build(s, w)
                got.append((i, t.n_nodes, P.sbh_eval(t, q, P.POTENTIAL, seed=1, group=64)))
                t.free_async()   # the evaluation may still run
        torch.cuda.synchronize()
        for i, nodes, out in got:
            if nodes != want[i][0] or not np.array_equal(out.cpu().numpy(), want[i][1]):
                bad.append((k, i))

    ts = [threading.Thread(target=work, args=(k,)) for k in range(threads)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not bad


_LAST = """
import torch
import paper_2506_02219_amd as P
s, w = torch.rand(1 << 21, 3, device="cuda"), torch.rand(1 << 21, device="cuda") + 0.5
P.sbh_build(s, w).free()
torch.cuda.synchronize()
before = torch.cuda.mem_get_info()[0]
a, b = P.sbh_build(s, w), P.sbh_build(s, w)
a.free_async()
kept = torch.cuda.mem_get_info()[0]
b.free()
after = torch.cuda.mem_get_info()[0]
print(before, kept, after)
assert before - kept > 64 << 20 and before - after < 64 << 20
"""


def test_idle_memory_goes_back_with_the_last_object():
    """In a process of its own, where no other test's tree is alive."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", _LAST], cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, (r.stdout, r.stderr[-2000:])
