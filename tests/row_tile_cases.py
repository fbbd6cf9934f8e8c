"""Small one-layer models and row counts that together reach every tile form of
the row-tile GEMM with every epilogue: 64, 96 and 128 rows x 128 columns (two K
groups up to 512 rows, one above), 96 and 128 rows x 256 columns; split partial
products, SwiGLU, head statistics.  tests/test_gemm_plan.py asserts that they
do; tests/test_gpu_row_tile.py runs them against the oracle."""
import gemm_plans


def _model(d, H, KVH, hd, F, V):
    return dict(n_layers=1, d_model=d, n_heads=H, n_kv_heads=KVH, head_dim=hd, d_ffn=F, vocab=V, dtype="bf16",
                rms_eps=1e-5, rope_theta=10000.0)


MODELS = {
    # gate/up and head widths, in tiles of 128 or 256 columns, decide these models' forms
    "cols_3k": _model(256, 4, 2, 64, 1408, 3001),
    "cols_4k": _model(256, 4, 2, 64, 2112, 4200),
    "cols_6k": _model(256, 4, 2, 64, 3008, 6000),
    "cols_28k": _model(256, 4, 2, 64, 14336, 28600),
    "cols_40k": _model(256, 4, 2, 64, 20480, 40000),
    # QKV, O and down of the 8B and the 1B widths
    "width_8b": _model(4096, 32, 8, 128, 512, 700),
    "width_1b": _model(2048, 16, 4, 128, 5632, 700),
}
CASES = [("cols_3k", 64), ("cols_28k", 96), ("cols_28k", 128), ("cols_40k", 95), ("cols_40k", 128), ("cols_3k", 599),
         ("cols_4k", 600), ("cols_6k", 601), ("width_8b", 96), ("width_8b", 128), ("width_8b", 160), ("width_8b", 256),
         ("width_8b", 513), ("width_1b", 600)]
EPILOGUES = {"qkv": "part", "o": "part", "down": "part", "gate_up": "swiglu", "head": "stats"}


def forms(name, rows):
    """(tile rows, tile columns, K groups, epilogue) the case's launches take."""
    m, out = MODELS[name], set()
    for role, epi in EPILOGUES.items():
        if gemm_plans.path(m, role, rows) == "row_tile":
            r, c, _ = gemm_plans.tile(m, role, rows)
            out.add((r, c, 2 if c == 128 and rows <= 512 else 1, epi))
    return out


ALL_FORMS = {(r, c, g, e) for r, c, g in ((64, 128, 2), (96, 128, 2), (128, 128, 2), (64, 128, 1), (96, 128, 1),
                                          (128, 128, 1), (96, 256, 1), (128, 256, 1))
             for e in ("part", "swiglu", "stats")}
