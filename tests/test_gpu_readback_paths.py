"""The ways a call's status words reach the host, each forced: through the
pinned page, by the copy, after a refused launch and after failed allocations
of the page; beside another thread's capture; with work still queued."""
import os
import subprocess
import sys
import threading

import pytest
import torch

import paper_2307_00071_amd as gmm
from paper_2307_00071_amd import _lib, synth

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _problem(n=3000, k=8):
    x = torch.from_numpy(synth.gaussian_blobs(3)[0][:n]).to(DEV)
    th = [torch.as_tensor(a, dtype=torch.float32, device=DEV) for a in synth.random_theta(k, 5)]
    bad = th[2].clone()
    bad[k - 1] = -bad[k - 1]
    return x, th, bad


def _good_and_bad(x, th, bad):
    want = float(gmm.loglik(x, *th, check=False))
    assert float(gmm.loglik(x, *th)) == want
    with pytest.raises(_lib.GmmError, match="SPD"):
        gmm.loglik(x, th[0], th[1], bad)


@pytest.mark.parametrize("way", ["page", "copy", "refuse"])
def test_each_way_reports_the_calls_status(way, monkeypatch):
    print("case: readback by %s" % way, flush=True)
    p = _problem()
    _good_and_bad(*p)
    monkeypatch.setenv("GMM_READ_TEST", way)
    for _ in range(20):   # more than there are slots
        _good_and_bad(*p)
    monkeypatch.setenv("GMM_READ_TEST", "page")
    _good_and_bad(*p)


def _in_a_new_process(code):
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]


def test_a_failed_page_is_tried_again():
    print("case: readback page retried", flush=True)
    _in_a_new_process("""
import os
from tests.test_gpu_readback_paths import _good_and_bad, _problem
p = _problem()
os.environ["GMM_READ_TEST"] = "nopage"
for _ in range(3):
    _good_and_bad(*p)
del os.environ["GMM_READ_TEST"]
for _ in range(10):
    _good_and_bad(*p)
os.environ["GMM_READ_TEST"] = "page"
_good_and_bad(*p)
""")


def test_the_first_read_beside_a_capture_of_another_thread():
    """The page is allocated on the first read of a process, here while
    another thread captures a graph in the global mode: the read goes through
    the page and the capture stays whole."""
    print("case: readback beside a capture", flush=True)
    _in_a_new_process("""
import ctypes, os, threading
import torch
import paper_2307_00071_amd as gmm
from paper_2307_00071_amd import _lib
from tests.test_gpu_readback_paths import DEV, _problem
x, th, bad = _problem()
lib = _lib.load()
ws = [torch.empty(lib.gmm_loglik_workspace_size(len(x), 8), dtype=torch.uint8, device=DEV)
      for _ in range(2)]
out = torch.empty((), dtype=torch.float64, device=DEV)
p = lambda t: ctypes.c_void_p(t.data_ptr())
main = torch.cuda.Stream(DEV)
s = ctypes.c_void_p(main.cuda_stream)
for w, cov in zip(ws, (th[2], bad)):
    _lib.check(lib.gmm_loglik(p(x), len(x), None, 8, p(th[0]), p(th[1]), p(cov), p(out), None,
                              p(w), w.numel(), s))
torch.cuda.synchronize()
a = torch.arange(1000.0, device=DEV)
b = torch.empty_like(a)
begun, read = threading.Event(), threading.Event()
graph = torch.cuda.CUDAGraph()
def capture():
    side = torch.cuda.Stream(DEV)
    with torch.cuda.stream(side):
        graph.capture_begin(capture_error_mode="global")
        torch.mul(a, 2.0, out=b)
        begun.set()
        read.wait(30)
        torch.add(b, 1.0, out=b)
        graph.capture_end()
t = threading.Thread(target=capture)
t.start()
assert begun.wait(30)
os.environ["GMM_READ_TEST"] = "page"
try:
    got = [lib.gmm_workspace_status(p(w), s) for w in ws]
finally:
    read.set()
    t.join()
assert got == [0, 2], got
for _ in range(3):
    b.zero_()
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(b, 2.0 * a + 1.0)
""")


def test_status_with_milliseconds_of_work_queued():
    print("case: readback after queued work", flush=True)
    x, th, bad = _problem()
    want = float(gmm.loglik(x, *th))
    for _ in range(3):
        torch.cuda._sleep(20_000_000)   # cycles: some 10 ms
        assert float(gmm.loglik(x, *th)) == want
        torch.cuda._sleep(20_000_000)
        with pytest.raises(_lib.GmmError, match="SPD"):
            gmm.loglik(x, th[0], th[1], bad)


def test_reads_of_several_words_beside_each_other():
    """Mean shift reads its counters, five words at a time, in 20 threads
    beside one-word reads."""
    print("case: readback of several words", flush=True)
    x, th, bad = _problem()
    ref = {h: (m.clone(), w.clone(), i["n_seeds"]) for h in (0.5, 0.8)
           for m, w, i in (gmm.meanshift(x, h),)}
    torch.cuda.synchronize()
    wrong = []

    def work(t):
        try:
            with torch.cuda.stream(torch.cuda.Stream(DEV)):
                for c in range(6):
                    if (t + c) % 2:
                        h = 0.5 if (t + c) % 3 else 0.8
                        m, w, i = gmm.meanshift(x, h)
                        if not (torch.equal(m, ref[h][0]) and torch.equal(w, ref[h][1]) and
                                i["n_seeds"] == ref[h][2]):
                            wrong.append((t, c, i))
                    else:
                        try:
                            gmm.loglik(x, th[0], th[1], bad)
                            wrong.append((t, c, "no error"))
                        except _lib.GmmError as e:
                            if "SPD" not in str(e):
                                wrong.append((t, c, str(e)))
        except Exception as e:            # a thread's failure is the test's
            wrong.append((t, -1, repr(e)))

    pool = [threading.Thread(target=work, args=(t,)) for t in range(20)]
    for p in pool:
        p.start()
    for p in pool:
        p.join()
    assert not wrong, wrong[:5]
