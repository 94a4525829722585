"""The status word of a call reaches the thread that made the call: many
threads (more than the library has read-back slots), each on a stream of its
own, alternate valid mixtures with ones whose covariance is not positive
definite; every call reports its own outcome and the valid ones their
value."""
import threading

import pytest
import torch

import paper_2307_00071_amd as gmm
from paper_2307_00071_amd import _lib, synth

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("threads", [1, 24])
def test_every_call_reads_its_own_status(threads):
    print("case: readback threads=%d" % threads, flush=True)
    n, k, calls = 3000, 8, 12
    x = torch.from_numpy(synth.gaussian_blobs(3)[0][:n]).to(DEV)
    w, mu, cov = (torch.as_tensor(a, dtype=torch.float32, device=DEV)
                  for a in synth.random_theta(k, 5))
    bad = cov.clone()
    bad[k - 1] = -bad[k - 1]
    want = float(gmm.loglik(x, w, mu, cov))
    torch.cuda.synchronize()
    wrong = []

    def work(t):
        try:
            with torch.cuda.stream(torch.cuda.Stream(DEV)):
                for c in range(calls):
                    if (t + c) % 3 == 0:
                        try:
                            gmm.loglik(x, w, mu, bad)
                            wrong.append((t, c, "no error"))
                        except _lib.GmmError as e:
                            if "SPD" not in str(e):
                                wrong.append((t, c, str(e)))
                    else:
                        got = float(gmm.loglik(x, w, mu, cov))
                        if got != want:
                            wrong.append((t, c, got))
        except Exception as e:            # a thread's failure is the test's
            wrong.append((t, -1, repr(e)))

    pool = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
    for p in pool:
        p.start()
    for p in pool:
        p.join()
    assert not wrong, wrong[:5]
