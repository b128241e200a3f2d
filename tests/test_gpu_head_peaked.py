"""Log-probs of confident tokens: one logit far above all others.  The hidden
rows are unit vectors, so a logit IS an entry of W and all that is left is the
softmax's own arithmetic."""
import numpy as np
import pytest

from test_gpu_parity import dev, host, tp  # noqa: F401
from paper_2506_15050_amd import synth

pytestmark = pytest.mark.gpu

V = 32000
SHAPES = [(True, 300, 64), (True, 60, 36), (True, 60, 63),          # fp32: whole stages, ragged, copied
          (False, 60, 64), (False, 1500, 64),                       # bf16: small and large tiles
          (False, 60, 72), (False, 1500, 72),                       # ragged
          (False, 60, 63), (False, 1500, 129), (False, 60, 2056)]   # copied; long


def run(tp, f32, M, H, w, at):
    """(logp, lse, the same in 64 bits) of M tokens; token i's logits are column i % H of w, its target at[i % H]."""
    hidden = np.eye(H, dtype=np.float32)
    col = np.arange(M) % H
    if not f32:
        hidden, w = synth.f32_to_bf16_bits(hidden), synth.f32_to_bf16_bits(w)
    logp, lse = tp.tppo_token_logprobs(dev(hidden), dev(w), dev(col.astype(np.int32)), dev(at[col].astype(np.int32)))
    z = (w if f32 else synth.bf16_bits_to_f32(w)).astype(np.float64)
    top = z.max(axis=0)
    rest = np.exp(z - top).sum(axis=0) - 1.0
    return host(logp), host(lse), (z[at, np.arange(H)] - top - np.log1p(rest))[col], (top + np.log1p(rest))[col]


@pytest.mark.parametrize("f32,M,H", SHAPES)
@pytest.mark.parametrize("lo,hi", [(8, 12), (30, 35), (60, 65)])
def test_peaked_rows(tp, f32, M, H, lo, hi):
    """The sampled logit lies in [lo, hi), the others have rms 1.4."""
    rng = np.random.default_rng(M + H + lo)
    w = (1.4 * rng.normal(size=(V, H))).astype(np.float32)
    at = (np.arange(H) * 997 + 5) % V
    w[at, np.arange(H)] = rng.uniform(lo, hi, size=H)
    logp, lse, ref, ref_lse = run(tp, f32, M, H, w, at)
    assert logp.max() <= 0.0                               # the sum is no less than the largest term, which it holds
    # From 30 on the other terms add up to less than 2^-24 of the largest, so the sum is that or its neighbour; at 8 to 12
    # a sum of 1 to 30 goes through up to 40 additions and is a random walk of 2^-24 of it: six times sqrt(40) / 2 of those.
    tol = 2.0 ** -24 if lo >= 30 else 1.2e-6
    assert np.abs(logp - ref).max() <= tol
    # the log-sum-exp is rounded at its own size, in bf16 by way of log2
    assert np.abs(lse - ref_lse).max() <= 2.0 ** -24 * 4 * hi + tol


@pytest.mark.parametrize("f32,M,H", SHAPES)
def test_entries_of_the_lowest_value(tp, f32, M, H):
    """Vocabulary entries masked with the type's lowest value: nothing for the others, finite for whom samples one."""
    rng = np.random.default_rng(M + H)
    w = (1.4 * rng.normal(size=(V, H))).astype(np.float32)
    lowest = np.float32(np.finfo(np.float32).min) if f32 else synth.bf16_bits_to_f32(np.array([0xFF7F], np.uint16))[0]
    w[rng.integers(0, V, size=500)] = lowest
    w[100], at = lowest, rng.integers(0, V, size=H)
    at[3] = 100
    logp, lse, ref, ref_lse = run(tp, f32, M, H, w, at)
    assert np.isfinite(logp).all() and np.isfinite(lse).all()
    # fp32 sums over V, as without masks; a masked log-prob to its own rounding
    assert np.all(np.abs(logp - ref) <= np.maximum(1e-5, 2.0 ** -23 * np.abs(ref)))
    assert np.abs(lse - ref_lse).max() <= 1e-5
