"""A call that synchronises its stream leaves it idle: hipStreamQuery answers
"ready" straight after each synchronous entry point."""
import ctypes

import pytest
import torch

import paper_2307_00071_amd as gmm
from paper_2307_00071_amd import _lib, synth

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("call", ["status", "fit", "noalloc", "seeding"])
def test_the_stream_is_idle_after_a_synchronous_call(call):
    print("case: idle after %s" % call, flush=True)
    n, k = 3000, 8
    x = torch.from_numpy(synth.gaussian_blobs(3)[0][:n]).to(DEV)
    w, mu, cov = (torch.as_tensor(a, dtype=torch.float32, device=DEV)
                  for a in synth.random_theta(k, 5))
    lab = (torch.arange(n, device=DEV) % k).to(torch.int32)
    u = torch.rand(k, dtype=torch.float64, device=DEV)
    lib = _lib.load()
    stream = torch.cuda.Stream(DEV)
    s = ctypes.c_void_p(stream.cuda_stream)
    query = ctypes.CDLL("libamdhip64.so").hipStreamQuery
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    opts = _lib.FitOpts(2, 1e-3, _lib.GMM_MOMENTS_SHIFTED, 0, 0.0)
    o = ctypes.byref(opts)
    size = {"status": lambda: lib.gmm_loglik_workspace_size(n, k),
            "fit": lambda: lib.gmm_fit_workspace_size(n, k, o), "noalloc": lambda: 1,
            "seeding": lambda: lib.gmm_kmeanspp_workspace_size(n, k)}[call]()
    ws = torch.empty(size, dtype=torch.uint8, device=DEV)
    out = torch.empty(8, dtype=torch.float64, device=DEV)
    centres = torch.empty(k, dtype=torch.int64, device=DEV)
    args = {"status": lambda: (lib.gmm_workspace_status, (p(ws), s)),
            "fit": lambda: (lib.gmm_fit, (p(x), n, k, p(lab), p(w), p(mu), p(cov), p(out), o,
                                          p(ws), ws.numel(), s)),
            "noalloc": lambda: (lib.gmm_fit_noalloc, (p(x), n, k, p(lab), p(w), p(mu), p(cov),
                                                      p(out), o, s)),
            "seeding": lambda: (lib.gmm_kmeanspp, (p(x), n, k, p(u), p(centres), p(lab), p(ws),
                                                   ws.numel(), s))}
    fn, a = args[call]()
    torch.cuda.synchronize()
    busy = 0
    for _ in range(300):
        if call == "status":
            _lib.check(lib.gmm_loglik(p(x), n, None, k, p(w), p(mu), p(cov), p(out), None, p(ws),
                                      ws.numel(), s))
        st = fn(*a)
        busy += query(s) != 0
        assert st == 0, st
    assert busy == 0, busy
