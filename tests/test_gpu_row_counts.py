"""Projections at the edges of their row ranges, in a model so narrow that passes of up to 64 rows take the streaming
kernel: packed up to 8 rows, then one row tile more at 17, 33 and 49 rows.  Prefill chunks of 65 to 128 rows take the panel
kernel (one tile per wave, K whole) with six and eight row tiles, larger ones and all fp32 ones the tiled kernel.  The
model's widths leave remainders everywhere: 7 and 10 K-blocks (no multiple of a pipeline stage or of four waves), 14, 25
and 21 weight tiles (no multiple of a work-group's)."""
import numpy as np
import pytest

from oracle import llama_ref as R
from paper_2403_12900_amd.configs import ModelConfig
from tests._harness import DeviceRun, check_against_oracle, oracle_shape, say

BF16_TOL, FP32_TOL = (5e-2, 1e-2), (1e-4, 1e-5)  # the gates of the parity tests


def _model(bf16, kv_bf16=None):
    return ModelConfig(n_layers=2, d_model=224, n_heads=5, n_kv_heads=5, head_dim=64, d_ff=200, vocab=333, bf16=bf16,
                       kv_bf16=kv_bf16)


# (requests, rows of the prefill, bf16 weights, bf16 KV cache)
@pytest.mark.gpu
@pytest.mark.parametrize("n,rows,bf16,kv_bf16", [
    (8, 8, True, True), (9, 9, True, True), (16, 33, True, False), (17, 65, True, True), (32, 96, True, True),
    (33, 97, True, False), (48, 128, True, True), (49, 129, True, True), (64, 64, True, True), (9, 17, False, False),
    (64, 70, False, False)])
def test_rows_at_the_edges(n, rows, bf16, kv_bf16):
    m = _model(bf16, kv_bf16)
    say(f"rows at the edges: {n} requests, {rows} prompt rows, bf16={bf16} kv_bf16={kv_bf16}")
    rng = np.random.default_rng(1000 * n + rows)
    lens = [rows // n + (i < rows % n) for i in range(n)]
    prompts = [rng.integers(0, m.vocab, size=s).astype(np.int32) for s in lens]
    stops = [3] * n
    run = DeviceRun(m, 91, prompts, stops)
    st = check_against_oracle(run, R.Weights(oracle_shape(m), 91), prompts, stops, range(n),
                              *(BF16_TOL if bf16 else FP32_TOL))
    say(st)
    assert st["rows"] == 3 * n
    run.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n,rows", [(3, 40), (17, 65), (20, 150)])
def test_model_width_inside_a_k_block(n, rows):
    """d_model = 208 ends 16 elements into a 32-element K-block: the other 16 of the residual's record must not keep
    what another projection's record left there, or the fused norms count it."""
    m = ModelConfig(n_layers=2, d_model=208, n_heads=5, n_kv_heads=5, head_dim=64, d_ff=200, vocab=333)
    say(f"width inside a K-block: {n} requests, {rows} prompt rows")
    rng = np.random.default_rng(rows)
    prompts = [rng.integers(0, m.vocab, size=rows // n + (i < rows % n)).astype(np.int32) for i in range(n)]
    run = DeviceRun(m, 92, prompts, [3] * n)
    st = check_against_oracle(run, R.Weights(oracle_shape(m), 92), prompts, [3] * n, range(n), *BF16_TOL)
    say(st)
    run.close()


@pytest.mark.gpu
@pytest.mark.parametrize("rows,d_ff,bf16", [(700, 200, True), (1100, 4096, False), (330, 200, False)])
def test_prefill_row_tiles_beyond_a_group(rows, d_ff, bf16):
    """Row tiles that are no multiple of the four of a group (6 of 128 rows, 9 of 128 rows, 6 of 64 rows); 4096
    feed-forward features over 1100 rows are fp32's large tile, the others its small one."""
    m = ModelConfig(n_layers=2, d_model=224, n_heads=5, n_kv_heads=5, head_dim=64, d_ff=d_ff, vocab=333, bf16=bf16)
    say(f"row tiles beyond a group: {rows} prompt rows, d_ff={d_ff} bf16={bf16}")
    rng = np.random.default_rng(rows)
    prompts = [rng.integers(0, m.vocab, size=s).astype(np.int32) for s in (rows // 3, rows // 3, rows - 2 * (rows // 3))]
    run = DeviceRun(m, 93, prompts, [3] * 3)
    st = check_against_oracle(run, R.Weights(oracle_shape(m), 93), prompts, [3] * 3, range(3),
                              *(BF16_TOL if bf16 else FP32_TOL))
    say(st)
    run.close()
