"""Kernels of fp32 models at the sizes where they change form: probe forwards of
a teacher-forced window against the oracle's fp64 logits.

Rows: one and two 16-row blocks (16 | 17), the last row of a 64-row tile and the
first of the next (64 | 65), more than 256 keys (a second chunk of the online
softmax) and enough rows for four column blocks per work-group (520 at the tiny
shape).  Models: head size 64 without and 128 with grouped queries, a ragged
vocabulary.  Tolerance: the fp32 logit bound of the lock-step tests (1e-4).
"""
import ctypes as C
import functools

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from oracle.model import OracleModel  # noqa: E402
from paper_2606_12243_amd import via  # noqa: E402
from workload import configs, gen  # noqa: E402

HD128 = dict(name="f32_hd128", seed_w=31, seed_c=32,
             model=dict(n_layers=2, d_model=320, n_heads=6, n_kv_heads=2, head_dim=128, d_ffn=704, vocab=501,
                        dtype="f32", rms_eps=1e-5, rope_theta=10000.0))


@functools.lru_cache(maxsize=None)
def models(name):
    cfg = HD128 if name == "f32_hd128" else dict(configs.get(name), seed_c=33)
    W = gen.model_weights(cfg)
    return cfg, via.Model(cfg["model"], W, list(range(cfg["model"]["n_layers"]))), OracleModel(cfg["model"], W)


@pytest.mark.parametrize("name,rows", [(n, r) for n in ("tiny_fp32", "f32_hd128") for r in (1, 16, 17, 64, 65, 300, 520)])
def test_window_logits_match_oracle(name, rows):
    print(f"[case] fp32 kernels {name} rows={rows}", flush=True)
    cfg, model, oracle = models(name)
    V = cfg["model"]["vocab"]
    tokens = gen.context_tokens(cfg, 0, rows)
    blocks = (rows + via.BLOCK - 1) // via.BLOCK
    kv = via.KV(model, max_seqs=1, max_blocks_per_seq=blocks, blocks_full=blocks, blocks_slim=blocks, max_rows=rows,
                max_batch=1, max_drafts=1)
    try:
        # pages hold NaN wherever nothing was written: no unseen key may reach a result
        kv.pool_full.fill_(float("nan"))
        via.check(via.via_kv_seq_reserve(kv.h, 0, 0))
        out = via.Out(1, rows, 1, V, logits=True)
        w = via.WindowBuf([0], [tokens], [[]], [[]], max_drafts=1)
        p = via.tier_params(0.9, 0.5, 1.0)
        via.check(via.via_verify_probe(model.h, kv.h, via.CACHE_FULL, C.byref(w.c), C.byref(p), C.byref(out.c),
                                       via.stream_ptr()))
        torch.cuda.synchronize()
        got = out.logits.view(rows, V).cpu().double()
        assert (got - oracle.forward_sequence(tokens)).abs().max().item() < 1e-4
        assert torch.equal(out.row_argmax.cpu().long(), got.argmax(1))
    finally:
        kv.close()
