"""Several threads, each on a stream of its own: one builds on rows that need the padded copy, the others search.  Only one
call at a time holds the workspace block, the block for padded rows and the search's counters that the library keeps; the others
work in blocks of their own.  Every result must be what the same call gives alone."""
import threading

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


def test_builds_and_searches_side_by_side():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as rn
    X = torch.from_numpy(wl.custom("unit_f32", 20_000, 100, 5)).cuda()
    Q = torch.from_numpy(wl.custom("unit_f32", 1500, 100, 6)).cuda()
    U = torch.from_numpy(wl.custom("heavy_u8", 9000, 100, 7)).cuda()
    graph, degree = rn.rnnd_build(X, 20, 64, 2, 5, 3)
    jobs = [lambda: rn.rnnd_build(X, 20, 64, 2, 5, 3),
            lambda: rn.rnnd_search(X, graph, degree, Q[:7].contiguous(), 64, 32, 10, 4, want_dist=True),
            lambda: rn.rnnd_search(X, graph, degree, Q, 32, 32, 10, 4, want_dist=True),
            lambda: rn.rnnd_build(U, 20, 96, 2, 4, 3)]
    want = [f() for f in jobs]
    torch.cuda.synchronize()
    bad, start = [], threading.Barrier(len(jobs))

    def work(i):
        try:
            torch.cuda.set_device(0)
            with torch.cuda.stream(torch.cuda.Stream()):
                start.wait(30)
                for r in range(12):
                    for a, b in zip(jobs[i](), want[i]):
                        if not (torch.equal(a, b) if torch.is_tensor(a) else a == b):
                            bad.append("job %d, pass %d differs" % (i, r))
        except Exception as e:      # reported by the main thread
            bad.append("job %d: %r" % (i, e))
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not bad and not any(t.is_alive() for t in threads), bad[:5]
    rn.rnnd_release_workspace()
