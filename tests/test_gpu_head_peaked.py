"""Log-probs of confident tokens: one logit far above all others.  The hidden
rows are unit vectors, so a logit IS an entry of W and all that is left is the
softmax's own arithmetic."""
import numpy as np
import pytest

from test_gpu_parity import dev, host, tp  # noqa: F401
from paper_2506_15050_amd import synth

pytestmark = pytest.mark.gpu

V = 32000


def peaked(tp, f32, M, H, lo, hi):
    """(logp, lse, the same in 64 bits): token i's sampled logit lies in [lo, hi), the others have rms 1.4."""
    rng = np.random.default_rng(M + H + lo)
    w = (1.4 * rng.normal(size=(V, H))).astype(np.float32)
    hidden = np.eye(H, dtype=np.float32)
    col = np.arange(M) % H
    at = (np.arange(H) * 997 + 5) % V
    w[at, np.arange(H)] = rng.uniform(lo, hi, size=H)
    if not f32:
        hidden, w = synth.f32_to_bf16_bits(hidden), synth.f32_to_bf16_bits(w)
    logp, lse = tp.tppo_token_logprobs(dev(hidden), dev(w), dev(col.astype(np.int32)), dev(at[col].astype(np.int32)))
    z = (w if f32 else synth.bf16_bits_to_f32(w)).astype(np.float64)
    top = z.max(axis=0)
    ref_lse = top + np.log(np.exp(z - top).sum(axis=0))
    ref = -np.log1p((np.exp(z - top).sum(axis=0) - 1.0)) + (z[at, np.arange(H)] - top)
    return host(logp), host(lse), ref[col], ref_lse[col]


@pytest.mark.parametrize("f32,M,H", [(True, 300, 64), (True, 60, 36), (True, 60, 63),        # fp32: whole stages, ragged, copied
                                     (False, 60, 72), (False, 1500, 72),                     # ragged bf16: small and large tiles
                                     (False, 60, 63), (False, 1500, 129), (False, 60, 2056)])
@pytest.mark.parametrize("lo,hi", [(8, 12), (30, 35), (60, 65)])
def test_peaked_rows_fp32_and_ragged(tp, f32, M, H, lo, hi):
    logp, lse, ref, ref_lse = peaked(tp, f32, M, H, lo, hi)
    assert logp.max() <= 0.0                               # the largest term is exactly 1, so the sum is no less
    # From 30 on the other terms add up to less than 2^-24 and the sum is 1 or its neighbour; at 8 to 12 a sum of 1 to
    # 30 goes through up to 40 additions and is a random walk of 2^-24 of it: six times sqrt(40) / 2 of those.
    tol = 2.0 ** -24 if lo >= 30 else 1.2e-6
    assert np.abs(logp - ref).max() <= tol
    assert np.abs(lse - ref_lse).max() <= 2.0 ** -24 * 2 * hi + tol


@pytest.mark.parametrize("M", [60, 1500])                  # small and large tiles
@pytest.mark.parametrize("lo,hi", [(8, 12), (30, 35), (60, 65)])
def test_peaked_rows_whole_stages_bf16(tp, M, lo, hi):
    logp, lse, ref, ref_lse = peaked(tp, False, M, 64, lo, hi)
    # the maximum is rounded in units of log2, so the largest term is 2^(that rounding): one ulp of exp2 and the rounding
    # of the sum, 3 x 2^-24 of 1
    assert np.abs(logp - ref).max() <= (3 * 2.0 ** -24 if lo >= 30 else 1.2e-6)
