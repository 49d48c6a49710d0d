"""Every shape of the projection kernels against the oracle, with K whole and split.

One-layer models whose widths make the rules (csrc/launch_rule.h) pick, between them, every shape of the panel kernel at
every row-tile count, whole and split, in each of its epilogues.  The CPU test checks that they still do, so that a rule
refitted later cannot silently leave a shape untested.  With an fp32 KV cache the distance to the oracle is that of 16-bit
activations, 1.5e-5 of a row's norm; the gate is four times that."""
import numpy as np
import pytest

from oracle import llama_ref as R
from paper_2403_12900_amd.configs import ModelConfig
from tests._harness import DeviceRun, check_against_oracle, oracle_shape, say
from tests.test_launch_rule import STREAM, gemm_pick, row_tiles, tile_pick

BF16_KV_TOL, FP32_KV_TOL, FP32_TOL = (5e-2, 1e-2), (6e-4, 6e-5), (1e-4, 1e-5)


def _model(d, heads, kv_heads, head_dim, d_ff, vocab=600, **kw):
    return ModelConfig(n_layers=1, d_model=d, n_heads=heads, n_kv_heads=kv_heads, head_dim=head_dim, d_ff=d_ff, vocab=vocab, **kw)


# name: model, (decode rows, prompt rows of one prefill chunk) of each run
CASES = {
    "1024": (_model(1024, 8, 8, 128, 4096), [(24, 66), (33, 97), (56, 66)]),
    "2048": (_model(2048, 16, 16, 128, 5632), [(9, 97), (33, 66), (56, 66)]),
    "2048_gqa4": (_model(2048, 16, 4, 128, 2048), [(24, 66), (33, 66), (56, 66)]),
    "3072": (_model(3072, 24, 24, 128, 8192), [(24, 66), (56, 66)]),
    "3072_wide": (_model(3072, 8, 1, 128, 12288, 2000), [(9, 66), (24, 97), (33, 66), (56, 66)]),
    "4160_gqa13": (_model(4160, 65, 5, 64, 6208), [(24, 97), (33, 66)]),
    "5120": (_model(5120, 40, 40, 128, 13824), [(9, 97), (24, 66), (56, 66)]),
    "6144": (_model(6144, 24, 8, 128, 6144), [(9, 66), (33, 66), (56, 66)]),
    "8192_gqa8": (_model(8192, 64, 8, 128, 2048), [(9, 66), (24, 97), (33, 66), (56, 66)]),
    "8192_mqa": (_model(8192, 16, 1, 128, 8192), [(33, 97), (56, 66)]),
    "2048_fp32": (_model(2048, 16, 16, 128, 5632, bf16=False), [(24, 30), (40, 40), (64, 64)]),
}


def _ceil(a, b):
    return -(-a // b)


def _picks(m, n, prefill):
    """(epilogue, gemm_pick) of every projection of a pass over n rows."""
    kb, parts = (32, 2) if m.bf16 else (16, 1)
    room = (2048 * m.n_heads * (m.head_dim + 4) - 4096, 4096)
    h = m.n_heads * m.head_dim
    mats = [("qkv", m.qkv_rows // 16, _ceil(m.d_model, kb), 3 if m.bf16 else 1, not prefill),
            ("residual", m.d_model // 16, _ceil(h, kb), parts, False), ("norm", _ceil(m.d_ff, 8), _ceil(m.d_model, kb), parts, not prefill),
            ("residual", m.d_model // 16, _ceil(m.d_ff, kb), parts, False)]
    if not prefill:
        mats.append(("norm", _ceil(m.vocab, 16), _ceil(m.d_model, kb), parts, True))
    return [(epi, gemm_pick(m.bf16, n, nt, kb_, p, norm, room)) for epi, nt, kb_, p, norm in mats]


def test_the_cases_reach_every_panel_shape():
    seen = set()
    for m, runs in CASES.values():
        for n, rows in runs:
            for pass_rows, prefill in [(n, False)] + ([(rows, True)] if m.bf16 else []):
                for epi, p in _picks(m, pass_rows, prefill):
                    if p != STREAM:
                        seen.add((m.bf16, row_tiles(pass_rows), p[:3], p[3] > 1))
    shapes = {1: [(4, 1, 4), (6, 1, 2), (4, 2, 2)], 2: [(4, 1, 2), (6, 1, 2), (8, 1, 2), (7, 2, 2)],
              3: [(4, 1, 2), (8, 1, 2), (4, 2, 2), (6, 2, 2), (7, 2, 2)], 4: [(4, 1, 2), (8, 1, 2), (4, 2, 2), (6, 2, 2), (7, 2, 2)],
              6: [(4, 1, 1), (8, 1, 1), (8, 2, 1), (4, 3, 1)], 8: [(4, 1, 1), (8, 1, 1), (8, 2, 1), (4, 3, 1)]}
    for jt, ss in shapes.items():
        for s in ss:
            assert (True, jt, s, True) in seen, (jt, s)  # split K
    # Whole K, where the rule takes it: few tiles per work-group, or long rounds of large ones.
    for jt, s in [(1, (4, 1, 4)), (1, (6, 1, 2)), (1, (4, 2, 2)), (2, (4, 1, 2)), (2, (6, 1, 2)), (3, (4, 1, 2)), (3, (4, 2, 2)),
                  (4, (4, 1, 2)), (4, (4, 2, 2)), (6, (4, 1, 1)), (6, (4, 3, 1)), (8, (4, 1, 1)), (8, (4, 3, 1))]:
        assert (True, jt, s, False) in seen, (jt, s)
    for jt in (2, 3, 4):
        assert (False, jt, (4, 1, 1), True) in seen and (False, jt, (4, 1, 1), False) in seen, jt


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_projection_shapes_against_the_oracle(case):
    base, runs = CASES[case]
    weights = {}
    for k, (n, rows) in enumerate(runs):
        # bf16 KV caches (QKV epilogues of their own) in every second run.
        m = base if not base.bf16 else _model(base.d_model, base.n_heads, base.n_kv_heads, base.head_dim, base.d_ff, base.vocab,
                                              kv_bf16=k % 2 == 1)
        say(f"projection shapes {case}: {n} rows, prompt {rows} rows, kv_bf16={m.kv_is_bf16}")
        rng = np.random.default_rng(n + rows)
        prompts = [rng.integers(0, m.vocab, size=rows // n + (i < rows % n)).astype(np.int32) for i in range(n)]
        run = DeviceRun(m, 29, prompts, [2] * n)
        w = weights.setdefault("w", R.Weights(oracle_shape(m), 29))
        w.shape = oracle_shape(m)
        st = check_against_oracle(run, w, prompts, [2] * n, range(n),
                                  *(FP32_TOL if not m.bf16 else BF16_KV_TOL if m.kv_is_bf16 else FP32_KV_TOL))
        say(st)
        assert st["rows"] == 2 * n
        run.close()


@pytest.mark.gpu
@pytest.mark.parametrize("d_ff", [5632, 5640])
def test_prefill_split_k_partials_in_idle_activations(d_ff):
    """Prefill chunks that split K: QKV's partials in the record that attention writes next, O's and down's in q; with a
    d_ff that ends inside a K-block (5640) QKV's stay out of that record, whose last K-block h does not fill."""
    m = ModelConfig(n_layers=2, d_model=2048, n_heads=16, n_kv_heads=16, head_dim=128, d_ff=d_ff, vocab=600, kv_bf16=False)
    rows = [100, 41, 108]
    padded = 128 * _ceil(sum(rows), 128)
    for nt, kb, parts in [(128, 64, 2), (256, 64, 3), (128, 64, 2), (128, _ceil(d_ff, 32), 2)]:
        assert tile_pick(nt, kb, padded, parts)[3] > 1
    say(f"prefill split-K room: d_ff={d_ff}")
    rng = np.random.default_rng(d_ff)
    prompts = [rng.integers(0, m.vocab, size=s).astype(np.int32) for s in rows]
    run = DeviceRun(m, 30, prompts, [3] * 3)
    st = check_against_oracle(run, R.Weights(oracle_shape(m), 30), prompts, [3] * 3, range(3), *FP32_KV_TOL)
    say(st)
    run.close()
