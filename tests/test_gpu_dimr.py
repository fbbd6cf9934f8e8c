"""DIMR routing cost on the GPU (via_dimr_cost, RoutingCost, MaskSearch)
against the oracle (oracle/dimr.py).

* via_dimr_cost on random fp32 logits (ragged vocabularies past the 256-wide
  thread stride, the 8B vocabulary, large logit scales, several T, alpha,
  beta) against the fp64 cost of the same logits: the GPU accumulates the
  per-token terms in fp64 from fp32 log-probabilities, so the tolerance is a
  few fp32 ulps of the per-token log-ratios times the number of tokens that
  contribute.
* C(z) of routing masks of the micro models (the routed model's logits from
  the library's forwards) against the oracle's C(z) from its own fp64
  forwards: the two differ by the forwards' rounding, bounded through the
  logit tolerance of the lock-step tests.
* a short mask search: its best mask is the minimum it evaluated, and that
  mask's oracle cost matches.
"""
import ctypes as C
import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2606_12243_amd import via  # noqa: E402
from paper_2606_12243_amd.dimr import MaskSearch, RoutingCost  # noqa: E402
from oracle.dimr import mask_cost, rkl_cost  # noqa: E402
from oracle.model import OracleModel  # noqa: E402
from workload import configs, gen  # noqa: E402


def gpu_cost(q, p, T, alpha, beta, ld=None):
    rows, V = q.shape
    ld = ld or V
    qd = torch.zeros(rows, ld, dtype=torch.float32, device="cuda")
    pd = torch.zeros(rows, ld, dtype=torch.float32, device="cuda")
    qd[:, :V] = q.cuda()
    pd[:, :V] = p.cuda()
    out = torch.full((rows,), float("nan"), dtype=torch.float32, device="cuda")
    sp = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    via.check(via.via_dimr_cost(qd.data_ptr(), pd.data_ptr(), rows, V, ld, T, alpha, beta, out.data_ptr(), sp))
    torch.cuda.synchronize()
    return out.cpu().double()


@pytest.mark.parametrize("rows,V,scale,T,alpha,beta,ld", [
    (7, 1000, 3.0, 1.0, 0.0, 1.0, None),
    (5, 257, 8.0, 0.7, 0.3, 1.5, 300),
    (3, 128256, 4.0, 33.97911834716797, 0.1, 1.0, None),
    (4, 3001, 30.0, 1.0, 0.5, 0.8, None),
])
def test_dimr_cost_matches_fp64(rows, V, scale, T, alpha, beta, ld):
    print(f"[case] dimr_cost rows={rows} V={V} scale={scale} T={T} alpha={alpha} beta={beta}", flush=True)
    g = torch.Generator().manual_seed(rows * 131 + V)
    q = (torch.randn(rows, V, generator=g) * scale).float()
    p = (q + torch.randn(rows, V, generator=g) * scale * 0.5).float()
    got = gpu_cost(q, p, T, alpha, beta, ld)
    ref = rkl_cost(q.double(), p.double(), T, alpha, beta)
    # per-token terms: probability x (log-ratio error <~ 8 fp32 ulps of the
    # larger log-probability magnitude); summed over the vocabulary
    lmax = (torch.cat([q, p]).abs().max().item() / T + math.log(V)) * 2
    tol = 1e-5 * ref.abs() + 8 * 2.0 ** -23 * lmax * 2 + 1e-6
    err = (got - ref).abs()
    print(f"[done] max err {err.max().item():.3g}, max ref {ref.abs().max().item():.3g}", flush=True)
    assert torch.isfinite(got).all()
    assert (err <= tol).all(), (got, ref)


@pytest.mark.parametrize("rows,V,ld", [
    (2, 1, None), (2, 2047, None), (2, 2048, None), (2, 2051, 2052),   # no whole round of 2048 ids, one, one and an end
    (2, 40961, 40964), (2, 57344, None), (2, 57345, 57347), (2, 65540, None),  # past the rounds kept in registers and LDS
    (257, 2049, None), (257, 16390, 16392), (258, 24576, None), (257, 28673, 28675),  # the form of more than 256 rows
])
def test_dimr_cost_at_kept_round_edges(rows, V, ld):
    """The sizes where the kernel keeps one more group of ids, re-reads the
    rest, takes its many-row form, or (ld not a multiple of 4) reads unaligned
    rows; bound as in test_dimr_cost_matches_fp64."""
    print(f"[case] dimr_cost edges rows={rows} V={V} ld={ld}", flush=True)
    g = torch.Generator().manual_seed(rows + V)
    q = torch.randn(rows, V, generator=g) * 2.0
    p = q + torch.randn(rows, V, generator=g)
    got = gpu_cost(q, p, 0.8, 0.1, 1.1, ld)
    ref = rkl_cost(q.double(), p.double(), 0.8, 0.1, 1.1)
    lmax = (torch.cat([q, p]).abs().max().item() / 0.8 + math.log(V)) * 2
    assert ((got - ref).abs() <= 1e-5 * ref.abs() + 8 * 2.0 ** -23 * lmax * 2 + 1e-6).all()


def test_dimr_cost_of_an_infinite_logit_is_not_a_number():
    """A row of q that overflowed has no cost: NaN, as in fp64, and not the 0 of a
    perfect mask.  Its neighbours keep theirs, and a token that p alone excludes
    (-inf) costs what it does in fp64; bound as in test_dimr_cost_matches_fp64."""
    print("[case] dimr_cost infinities", flush=True)
    g = torch.Generator().manual_seed(5)
    q = torch.randn(4, 3001, generator=g) * 2.0
    p = q + torch.randn(4, 3001, generator=g)
    lmax = (torch.cat([q, p]).abs().max().item() / 0.8 + math.log(3001)) * 2
    q[1, 700] = float("inf")
    q[2, 3000] = float("inf")  # among the ids past the last whole round
    p[3, [0, 1, 2, 3, 2999]] = float("-inf")
    got = gpu_cost(q, p, 0.8, 0.1, 1.1)
    ref = rkl_cost(q.double(), p.double(), 0.8, 0.1, 1.1)
    assert torch.isnan(ref[1:3]).all() and torch.isnan(got[1:3]).all()
    tol = 1e-5 * ref.abs() + 8 * 2.0 ** -23 * lmax * 2 + 1e-6
    assert ((got - ref).abs() <= tol)[[0, 3]].all(), (got, ref)


def test_dimr_cost_rejects_bad_arguments():
    sp = C.c_void_p(0)
    buf = torch.zeros(64, dtype=torch.float32, device="cuda")
    p = buf.data_ptr()
    assert via.via_dimr_cost(p, p, 1, 8, 8, 1.0, 1.0, 1.0, p, sp) == via.EINVAL    # alpha = 1
    assert via.via_dimr_cost(p, p, 1, 8, 8, 1.0, 0.0, 0.0, p, sp) == via.EINVAL    # beta = 0
    assert via.via_dimr_cost(p, p, 1, 8, 4, 1.0, 0.0, 1.0, p, sp) == via.EINVAL    # ld < vocab
    assert via.via_dimr_cost(p, p, 1, 8, 8, 0.0, 0.0, 1.0, p, sp) == via.EINVAL    # T = 0
    assert via.via_dimr_cost(None, p, 1, 8, 8, 1.0, 0.0, 1.0, p, sp) == via.EINVAL
    assert via.via_dimr_cost(None, None, 0, 8, 8, 1.0, 0.0, 1.0, None, sp) == via.OK  # no rows: no-op


def micro_model(name):
    cfg = configs.get(name)
    cfg["seed_c"] = 9
    W = gen.model_weights(cfg)
    return cfg, W


@pytest.mark.parametrize("name", ["micro_f32", "micro_bf16"])
def test_routing_cost_matches_oracle(name):
    print(f"[case] routing cost {name}", flush=True)
    cfg, W = micro_model(name)
    md = cfg["model"]
    L = md["n_layers"]
    toks = gen.context_tokens(cfg, 0, 24)
    model = via.Model(md, W, list(range(L)))
    om = OracleModel(md, W)
    try:
        for T, alpha, beta in ((1.0, 0.0, 1.0), (2.0, 0.2, 1.3)):
            rc = RoutingCost(model, toks, T, alpha, beta)
            for route in ([0], [1, 2], [0, 2], list(range(L))):
                got = rc(route)
                ref = mask_cost(om, route, toks, T, alpha, beta)
                print(f"[done] route {route} T={T}: gpu {got:.6g} oracle {ref:.6g}", flush=True)
                assert got == pytest.approx(ref, rel=2e-2, abs=2e-2 * len(toks))
    finally:
        model.close()


def test_mask_search_on_micro_model():
    cfg, W = micro_model("small_bf16_hd128")
    md = cfg["model"]
    L = md["n_layers"]
    toks = gen.context_tokens(cfg, 0, 32)
    model = via.Model(md, W, list(range(L)))
    om = OracleModel(md, W)
    try:
        rc = RoutingCost(model, toks, 1.0, 0.0, 1.0)
        s = MaskSearch(L, 2, rc, seed=2, theta=2, max_steps=6, patience=6)
        best, c = s.run()
        print(f"[done] best {best} cost {c:.6g} history {[(h[0], round(h[1], 4), h[2]) for h in s.history]}", flush=True)
        assert len(s.history) == 6  # C(4, 2) = 6 masks: the whole space
        assert c == min(h[1] for h in s.history)
        assert c == pytest.approx(mask_cost(om, best, toks, 1.0, 0.0, 1.0), rel=2e-2, abs=2e-2 * len(toks))
    finally:
        model.close()
