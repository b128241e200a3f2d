"""The value head where its work division changes: two or four rows per
wavefront, groups of rows that end inside a wavefront, rows shorter than one
step of a wavefront, weights that start at any 2-byte address."""
import numpy as np
import pytest

from test_gpu_parity import dev, host, ofast, tp  # noqa: F401
from paper_2506_15050_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [2, 3, 6143, 6144, 6145, 6158])
@pytest.mark.parametrize("H", [8, 504, 520, 1032])
def test_value_head_row_groups(tp, M, H):
    import torch
    N = 300
    rng = np.random.default_rng(M + H)
    hidden = synth.f32_to_bf16_bits(rng.normal(size=(N, H)).astype(np.float32))
    w = synth.f32_to_bf16_bits((rng.normal(size=H) / np.sqrt(H)).astype(np.float32))
    rows = rng.integers(0, N, size=M).astype(np.int32)
    ref, bound = ofast.value_head(hidden, w, 0.5, rows, return_abs_bound=True)
    shifted = torch.empty(H + 3, dtype=torch.bfloat16, device="cuda")[3:]
    shifted.copy_(dev(w))
    got = host(tp.tppo_value_head(dev(hidden), shifted, 0.5, dev(rows)))
    # fp32 accumulation of H products: a few sqrt(H) 2^-24 of the sum of the terms' magnitudes
    assert np.all(np.abs(got - ref) <= 1e-5 * (bound + 0.5))
    bad = rows.copy()
    bad[M - 1] = N                                         # the last row of a group that may not be full
    st = tp.new_status("cuda")
    got2 = host(tp.tppo_value_head(dev(hidden), shifted, 0.5, dev(bad), status=st))
    assert int(host(st)[0]) == tp.STATUS_BAD_ROW and np.isnan(got2[M - 1]) and np.array_equal(got2[:M - 1], got[:M - 1])


def test_value_head_several_turns(tp):
    """More rows than one turn of the largest grid takes (2^20 workgroups of 16), the last turn short and with a bad row."""
    import torch
    H, N, M = 8, 300, (1 << 24) + 41
    rng = np.random.default_rng(7)
    hidden = synth.f32_to_bf16_bits(rng.normal(size=(N, H)).astype(np.float32))
    w = synth.f32_to_bf16_bits(rng.normal(size=H).astype(np.float32))
    rows = torch.arange(M, device="cuda", dtype=torch.int32).mul_(7).remainder_(N)
    rows[M - 3] = -1
    ref = dev(ofast.value_head(hidden, w, 0.5, np.arange(N)).astype(np.float32))[rows.clamp(min=0).long()]
    st = tp.new_status("cuda")
    got = tp.tppo_value_head(dev(hidden), dev(w), 0.5, rows, status=st)
    assert int(host(st)[0]) == tp.STATUS_BAD_ROW and bool(torch.isnan(got[M - 3]))
    got[M - 3] = ref[M - 3]
    # eight products and seven additions in fp32, terms of size 10 at most
    assert float((got - ref).abs().max()) <= 8 * 2.0 ** -23 * 16
