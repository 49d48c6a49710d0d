"""RMSNorm scale of prompt chunks: no fewer bits than the fp32 residual gives.

The gate/up input of a bf16 model is a two-part record (hi + lo); a sum of squares without lo.lo is 2.7e-6 low, the scale
1.35e-6 high, in every row alike.  The rounding of the 16-bit activations (about 1.5e-5 of a logit) hides that in any
single logit, but not in all of them together: the device's logits minus the 64-bit ones are regressed on what a larger
scale of that norm would add (and on the logits themselves, which a larger scale of the final norm adds)."""
import numpy as np
import pytest

from oracle import llama_ref as R
from paper_2403_12900_amd.configs import ModelConfig
from tests._harness import DeviceRun, oracle_shape, say


def _logits(w, prompts, scale):
    """Last-position logits of a one-layer model, its second norm's output times `scale`."""
    sh, g, W = w.shape, w.gain(), w.layer(0)
    out = []
    for p in prompts:
        T, pos = len(p), np.arange(len(p))
        x = R.embed_rows(w, p)
        a = R.rmsnorm(x, g, sh.rms_eps)
        q = R.apply_rope((a @ W["wq"].T).reshape(T, sh.n_heads, sh.head_dim), pos, sh.rope_base)
        k = R.apply_rope((a @ W["wk"].T).reshape(T, sh.n_kv_heads, sh.head_dim), pos, sh.rope_base)
        k, v = R.cache_kv(sh, k, (a @ W["wv"].T).reshape(T, sh.n_kv_heads, sh.head_dim))
        x = x + R.causal_attention(q, k, v).reshape(T, -1) @ W["wo"].T
        out.append(x[-1])
    x = np.array(out)
    x = x + R.swiglu(scale * R.rmsnorm(x, g, sh.rms_eps), W["w1"], W["w3"], W["w2"])
    return R.rmsnorm(x, g, sh.rms_eps) @ w.matrix("lm_head").T


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [64, 128, 192])
def test_chunk_norms_keep_the_fp32_scale(rows):
    m = ModelConfig(n_layers=1, d_model=512, n_heads=8, n_kv_heads=8, head_dim=64, d_ff=2048, vocab=1024, kv_bf16=False)
    say(f"norm scale: {rows} prompt rows")
    rng = np.random.default_rng(rows)
    prompts = [rng.integers(0, m.vocab, size=rows // 64).astype(np.int32) for _ in range(64)]
    run = DeviceRun(m, 17, prompts, [1] * 64)
    z = np.array([run.logits[i][0] for i in range(64)], dtype=np.float64)
    run.close()
    w = R.Weights(oracle_shape(m), 17)
    ref = _logits(w, prompts, 1.0)
    more = (_logits(w, prompts, 1.0 + 1e-4) - _logits(w, prompts, 1.0 - 1e-4)) / 2e-4
    A = np.stack([more.ravel(), ref.ravel()], axis=1)
    (norm, final), *_ = np.linalg.lstsq(A, (z - ref).ravel(), rcond=None)
    noise = np.linalg.norm(z - ref) / np.linalg.norm(more) / np.sqrt(64 * m.d_model)
    say(f"gate/up scale {norm:.2e}, final {final:.2e}, standard error about {noise:.1e}")
    # Half of what leaving lo.lo out gives; the standard error is 3e-8.
    assert abs(norm) < 7e-7
