"""Both forms of the large tiles' log-softmax on whole stages, either side of the line between them (kLongStages), and the derivative's
sweep, which has one form, either side of the same line: a ragged last tile of W rows, token tiles cut short by the device's own count."""

import numpy as np
import pytest

from test_head_routes import rule  # noqa: F401
from test_gpu_parity import _bf16_case, check_logprob_grads, dev, host, ofast, tp  # noqa: F401
from paper_2506_15050_amd import synth

LONG = [(1000, 32001, 35 * 64), (1000, 32001, 36 * 64), (2000, 16001, 36 * 64)]
GRADS = [(1500, 9001, 1600), (2048, 12001, 2304)]


def test_shapes_take_large_tiles(rule):  # noqa: F811
    assert [r[0] for r in rule(LONG + GRADS, True, True)] == [0] * 5


@pytest.mark.gpu
@pytest.mark.parametrize("M,V,H", LONG)
def test_logprobs(tp, M, V, H):
    rng = np.random.default_rng(M + V + H)
    hidden = synth.f32_to_bf16_bits(rng.normal(size=(301, H)).astype(np.float32))
    w = synth.f32_to_bf16_bits((rng.normal(size=(V, H)) / np.sqrt(H)).astype(np.float32))
    rows, targets = rng.integers(0, 301, size=M), (np.arange(M) * 7 + V - 1) % V
    args = (dev(hidden), dev(w), dev(rows.astype(np.int32)), dev(targets.astype(np.int32)))
    ref, ref_lse = ofast.token_logprobs(hidden, w, rows, targets)
    for n in (M, M - M // 3 - 1):
        st = tp.new_status("cuda")
        logp, lse = tp.tppo_token_logprobs(*args, m_actual=dev(np.array([n], np.int64)), status=st)
        assert int(host(st)[0]) == 0
        # exact products summed in fp32 over H and V, logits of size about 5: a few times 2^-24 * 8
        assert np.abs(host(logp)[:n] - ref[:n]).max() <= 1e-5 and np.abs(host(lse)[:n] - ref_lse[:n]).max() <= 1e-5


@pytest.mark.gpu
@pytest.mark.parametrize("M,V,H", GRADS)
def test_grads(tp, M, V, H):
    check_logprob_grads(tp, *_bf16_case(M, V, H, seed=M + V))
