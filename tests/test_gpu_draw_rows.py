"""Draws and probabilities (via_sample_rows_static) at the vocabularies where a
thread's share of ids changes: one id, two with a ragged end, past the eight
that are loaded together, and a last chunk of one to eight.  Probabilities
against fp64 softmax, tokens against the fp64 running sum, and the same call
with the probabilities laid over the logits, which must give the same bits.

Tolerance: a probability is expf (2 ulp) of an argument rounded twice, at most
|l - max| / T * 2^-23 relative with |l - max| / T < 32, times a reciprocal: 3e-5
covers 32 * 2^-22 + 4 ulp.  The running weight is a sum of those: the same bound.
"""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2606_12243_amd import via  # noqa: E402


@pytest.mark.parametrize("V", [1, 257, 16385, 131072, 131073, 250007])
def test_draws_and_probabilities(V):
    print(f"[case] draw rows V={V}", flush=True)
    n, T = 5, 0.8
    g = torch.Generator(device="cuda").manual_seed(V)
    o = via.Out(n, 1, 1, V, logits=True)
    lg = torch.randn(n, V, generator=g, device="cuda") * 2.0
    o.logits.copy_(lg.reshape(-1))
    mx = lg.max(dim=1).values
    o.row_max.copy_(mx)
    o.row_sumexp.copy_(torch.exp((lg - mx[:, None]).double() / T).sum(dim=1))
    ref = torch.softmax(lg.double() / T, dim=1).cpu()
    r, rp = via._i32(list(range(n)))
    u = np.array([0.0, 0.1, 0.5, 0.9, 0.999], np.float32)
    sp = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    apart = torch.full((n, V), -1.0, device="cuda")
    got = []
    for p in (apart.data_ptr(), o.logits.data_ptr()):
        tok = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        via.check(via.via_sample_rows_static(C.byref(o.c), n, V, n, rp, T, u.ctypes.data, tok.data_ptr(), p, V, sp))
        torch.cuda.synchronize()
        got.append(tok.cpu())
    assert torch.equal(got[0], got[1])
    assert torch.equal(apart.reshape(-1), o.logits[:n * V])
    assert ((apart.cpu().double() - ref).abs() <= 3e-5 * ref + 1e-30).all()
    c = torch.cumsum(ref, 1)
    for i in range(n):
        t = int(got[0][i])
        assert 0 <= t < V
        assert c[i, t] >= float(u[i]) - 3e-5 and (t == 0 or c[i, t - 1] <= float(u[i]) + 3e-5)
