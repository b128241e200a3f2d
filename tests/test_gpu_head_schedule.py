"""The LM-head sweeps' schedule where it changes shape: few token tiles cut into
many vocabulary ranges, token tiles left over after whole rounds of workgroups,
and output tiles of the backward products whose contraction is cut into chunks."""
import numpy as np
import pytest

from test_head_routes import FP32_FEW, FP32_MANY, LARGE_RAGGED, LARGE_WHOLE
from test_gpu_parity import _bf16_case, assert_within_term_bound, check_logprob_grads, check_logprobs, dev, host, ofast, tp  # noqa: F401
from paper_2506_15050_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,V,H", [(5, 70000, 64),        # small tiles: one token tile, 183 vocabulary ranges
                                   (1030, 3000, 64),      # small tiles: 17 token tiles, 12 vocabulary ranges
                                   (64, 32000, 1024), (20, 1500, 320),      # small tiles, 16 and 5 K stages
                                   (16500, 600, 64),      # large tiles: 65 token tiles, 3 vocabulary tiles
                                   (33000, 300, 64),      # 129 token tiles, no cut of the vocabulary
                                   (66000, 200, 64)])     # one vocabulary tile: a round of 256 token tiles, 2 left
def test_logprobs_schedule_shapes(tp, M, V, H):
    rng = np.random.default_rng(M + V)
    hidden = synth.f32_to_bf16_bits(rng.normal(size=(999, H)).astype(np.float32))
    w = synth.f32_to_bf16_bits((rng.normal(size=(V, H)) / np.sqrt(H)).astype(np.float32))
    targets = rng.integers(0, V, size=M)
    targets[:3] = 0, V - 1, min(256, V - 1)
    check_logprobs(tp, hidden, w, rng.integers(0, 999, size=M), targets)


@pytest.mark.parametrize("M,V,H", [*LARGE_WHOLE, *LARGE_RAGGED])
def test_logprobs_large_tiles(tp, M, V, H):
    """The 256 x 256 tiles at sizes that test_head_routes.py shows to reach them: whole and ragged rows, one token tile
    and whole rounds with a rest, a vocabulary that ends one entry into a tile."""
    rng = np.random.default_rng(M + V + H)
    hidden = synth.f32_to_bf16_bits(rng.normal(size=(301, H)).astype(np.float32))
    w = synth.f32_to_bf16_bits((rng.normal(size=(V, H)) / np.sqrt(H)).astype(np.float32))
    rows, targets = rng.integers(0, 301, size=M), (np.arange(M) * 7 + V - 1) % V
    args = (_padded(hidden, H + (-H % 8), 0), _padded(w, H + (-H % 8), 8), dev(rows.astype(np.int32)),
            dev(targets.astype(np.int32)))
    ref, ref_lse = ofast.token_logprobs(hidden, w, rows, targets)
    few = M - M // 3 - 1                                   # the device's own count: token tiles cut short and left out
    for n in (M, few):
        st = tp.new_status("cuda")
        logp, lse = tp.tppo_token_logprobs(*args, m_actual=dev(np.array([n], np.int64)), status=st)
        assert int(host(st)[0]) == 0
        # exact products summed in fp32 over H and V, logits of size about 5: a few times 2^-24 * 8
        assert np.abs(host(logp)[:n] - ref[:n]).max() <= 1e-5 and np.abs(host(lse)[:n] - ref_lse[:n]).max() <= 1e-5


@pytest.mark.parametrize("M,V,H", [(300, 20000, 64),      # grad_hidden: 2 output tiles, 313 K steps in chunks
                                   (200, 9001, 320),      # ragged vocabulary and a second, short column of tiles
                                   (4500, 260, 64)])      # grad_w: 2 output tiles over 71 K steps of tokens
def test_logprob_grads_cut_contraction(tp, M, V, H):
    import torch
    hidden, w, rows, targets, g = _bf16_case(M, V, H, seed=M + V)
    dh, dw = check_logprob_grads(tp, hidden, w, rows, targets, g)
    _, lse = ofast.token_logprobs(hidden, w, rows, targets)
    args = (dev(hidden), dev(w), dev(rows.astype(np.int32)), dev(targets.astype(np.int32)),
            dev(lse.astype(np.float32)), dev(g.astype(np.float32)))
    acc = torch.full((V, H), 2.0, device="cuda")           # partial tiles added to what is there
    again, _ = tp.tppo_token_logprobs_backward(*args, grad_w=acc, accumulate_w=True)
    torch.cuda.synchronize()
    assert np.array_equal(host(again), dh)
    # one fp32 rounding of (2 + dw)
    assert np.abs(host(acc) - 2.0 - dw).max() <= 2.0 ** -23 * (2.0 + np.abs(dw).max())


@pytest.mark.parametrize("M,V,H", [(40, 1472, 64),        # grad_hidden: 23 K steps, whole; a quarter of a tile's columns
                                   (40, 1473, 64),        # ... 24 steps, in chunks of one or two
                                   (1473, 300, 320),      # grad_w: 24 K steps of tokens, a short second column of tiles
                                   (1600, 4200, 704)])    # both, 7 x 3 and 17 x 3 output tiles
def test_logprob_grads_short_contractions(tp, M, V, H):
    """Contractions around the shortest that is cut, with all the room for partial tiles that the call wants, with the
    least workspace that holds all tokens, and, in chunks, with the least that the call takes."""
    case = _bf16_case(M, V, H, seed=M + V)
    check_logprob_grads(tp, *case)
    wanted = tp.load().tppo_token_logprobs_backward_workspace_bytes(M, H, V, tp.TPPO_BF16)

    def least(tokens):                                      # dZ, as much again, Hid^T, the sweep's words
        return 2 * tokens * 2 * ((V + 63) // 64 * 64) + 2 * tokens * H + ((max(tokens, V) // 256 + 64) * 16 + 255) // 256 * 256
    assert least((M + 255) // 256 * 256) <= wanted
    for nbytes in {least((M + 255) // 256 * 256), least(256)}:
        check_logprob_grads(tp, *case, workspace=tp._workspace(nbytes, "cuda"))
    with pytest.raises(RuntimeError):
        check_logprob_grads(tp, *case, workspace=tp._workspace(least(256) - 256, "cuda"))


@pytest.mark.parametrize("M,V,H", [(8300, 33000, 2048),    # grad_hidden: 33 x 8 output tiles, a round and eight more, 516 K steps
                                   (32900, 4300, 4096)])   # grad_w: 17 x 16 tiles, 515 K steps of tokens
def test_logprob_grads_aligned_rounds(tp, M, V, H):
    """Products of several rounds whose workgroups wait for each other, at sampled rows of both results: plain torch in
    64 bits from the same log-sum-exps."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(M)
    hidden = torch.randn(M, H, device="cuda", generator=gen).bfloat16()
    w = (torch.randn(V, H, device="cuda", generator=gen) / H ** 0.5).bfloat16()
    rows = torch.arange(M, device="cuda", dtype=torch.int32).flip(0)
    targets, g = rows * 7 % V, torch.randn(M, device="cuda", generator=gen)
    _, lse = tp.tppo_token_logprobs(hidden, w, rows, targets)
    dh, dw = tp.tppo_token_logprobs_backward(hidden, w, rows, targets, lse, g)

    def dz(t, v):                                           # of tokens t and vocabulary entries v
        z = hidden[rows[t].long()].double() @ w[v].double().t()
        hit = targets[t].long().unsqueeze(1) == v.unsqueeze(0)
        return g[t].double().unsqueeze(1) * (hit.double() - torch.exp(z - lse[t].double().unsqueeze(1)))
    every_t, every_v = torch.arange(M, device="cuda"), torch.arange(V, device="cuda")
    t, v = every_t[::M // 60], every_v[::V // 60]
    d = dz(t, every_v)
    assert_within_term_bound(host(dh[t]), host(d @ w.double()), host(d.abs() @ w.double().abs()), "grad_hidden")
    d = dz(every_t, v).t().contiguous()
    h = hidden[rows.long()].double()
    assert_within_term_bound(host(dw[v]), host(d @ h), host(d.abs() @ h.abs()), "grad_w")


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("M,V", [(1, 1), (1, 129), (63, 127), (64, 128), (65, 1000), (130, 5003), (700, 2000)])
@pytest.mark.parametrize("H", [64, 72, 192])
def test_logprobs_small_tiles(tp, f32, M, V, H):
    """Sizes that go to the 128 x 64 tiles: edges of a tile, one task and many."""
    rng = np.random.default_rng(M + V + H)
    hidden = rng.normal(size=(90, H)).astype(np.float32)
    w = (rng.normal(size=(V, H)) / np.sqrt(H)).astype(np.float32)
    if not f32:
        hidden, w = synth.f32_to_bf16_bits(hidden), synth.f32_to_bf16_bits(w)
    rows, targets = rng.integers(0, 90, size=M), (np.arange(M) * 7 + V - 1) % V
    out = dev(rng.permutation(M + 5)[:M].astype(np.int32))
    logp, lse = tp.tppo_token_logprobs(dev(hidden), dev(w), dev(rows.astype(np.int32)), dev(targets.astype(np.int32)),
                                       out_index=out, out_size=M + 5)
    ref_lp, ref_lse = ofast.token_logprobs(hidden, w, rows, targets)
    at = host(out)
    # exact products summed in fp32 over H and V, logits of size about 5: a few times 2^-24 * 8
    assert np.abs(host(logp)[at] - ref_lp).max() <= 1e-5 and np.abs(host(lse)[at] - ref_lse).max() <= 1e-5


@pytest.mark.parametrize("M,V,H", [*FP32_FEW, *FP32_MANY])
def test_logprobs_fp32_tasks(tp, M, V, H):
    """fp32 with up to two workgroups to a CU and with three: whole and ragged rows, tasks of one tile and of several."""
    rng = np.random.default_rng(M + V + H)
    hidden = rng.normal(size=(90, H)).astype(np.float32)
    w = (rng.normal(size=(V, H)) / np.sqrt(H)).astype(np.float32)
    rows, targets = rng.integers(0, 90, size=M), (np.arange(M) * 7 + V - 1) % V
    logp, lse = tp.tppo_token_logprobs(dev(hidden), dev(w), dev(rows.astype(np.int32)), dev(targets.astype(np.int32)))
    ref_lp, ref_lse = ofast.token_logprobs(hidden, w, rows, targets)
    # products and sums in fp32 over H and V, logits of size about 5: a few times 2^-24 * 8
    assert np.abs(host(logp) - ref_lp).max() <= 1e-5 and np.abs(host(lse) - ref_lse).max() <= 1e-5


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("H", [5112, 5100])
def test_logprobs_long_sums(tp, f32, H):
    """fp32 and ragged bf16 rows of thousands of elements, in sums of 128 that are then added up."""
    M, V = 300, 4000
    rng = np.random.default_rng(H)
    hidden = rng.normal(size=(M, H)).astype(np.float32)
    w = (rng.normal(size=(V, H)) * 0.02).astype(np.float32)
    if not f32:
        hidden, w = synth.f32_to_bf16_bits(hidden), synth.f32_to_bf16_bits(w)
    rows, targets = np.arange(M), rng.integers(0, V, size=M)
    logp, lse = tp.tppo_token_logprobs(dev(hidden), dev(w), dev(rows.astype(np.int32)), dev(targets.astype(np.int32)))
    ref_lp, ref_lse = ofast.token_logprobs(hidden, w, rows, targets)
    # a logit of rms 1.43 by 128 and then 40 additions: a random walk of rms 2^-24 * 1.43 * sqrt(64 + 20) = 8e-7, six of
    # those (one sum over all of H: rms 4e-6)
    assert np.abs(host(logp) - ref_lp).max() <= 5e-6 and np.abs(host(lse) - ref_lse).max() <= 5e-6


@pytest.mark.parametrize("H,pad,offset", [(5120, 1, 0), (2112, 8, 3), (5112, 0, 0)])
def test_logprobs_long_sums_no_worse_than_one_token_at_a_time(tp, H, pad, offset):
    """bf16 rows that the one-token kernel takes when the workspace is small: with room for copies of W and the kept rows
    they go to the tiles, and are summed no less exactly there."""
    M, V = 1500, 8000                                      # 6 token tiles x 32: not too few for the large tiles
    rng = np.random.default_rng(H)
    hidden = synth.f32_to_bf16_bits(rng.normal(size=(M, H)).astype(np.float32))
    w = synth.f32_to_bf16_bits((rng.normal(size=(V, H)) * 0.02).astype(np.float32))
    rows, targets = np.arange(M), rng.integers(0, V, size=M)
    args = (_padded(hidden, H + pad, offset), _padded(w, H + pad, offset), dev(rows.astype(np.int32)),
            dev(targets.astype(np.int32)))
    ref, _ = ofast.token_logprobs(hidden, w, rows, targets)
    room = tp.load().tppo_token_logprobs_workspace_bytes(M, H, V, tp.TPPO_BF16) + 2 * (M + V) * (H + 8)
    rms = [np.sqrt(np.mean((host(tp.tppo_token_logprobs(*args, workspace=tp._workspace(n, "cuda"))[0]) - ref) ** 2))
           for n in (256, room)]
    # (an rms over 1500 tokens is good to 2 %; one sum over all of H = 5120 shows 1.3 times the one-token kernel's)
    assert rms[1] <= 1.1 * rms[0]


@pytest.mark.parametrize("M,V", [(1, 64), (65, 129), (200, 1000), (130, 5003)])
def test_logprob_grads_small_tiles(tp, M, V):
    check_logprob_grads(tp, *_bf16_case(M, V, 128, seed=M + V))


def _padded(a, ld, offset):
    """The matrix on the GPU with leading dimension `ld`, starting `offset` elements into its allocation, everything
    around it NaN."""
    import torch
    t = dev(a)
    buf = torch.full((offset + a.shape[0] * ld,), float("nan"), dtype=t.dtype, device="cuda")
    view = torch.as_strided(buf, t.shape, (ld, 1), offset)
    view.copy_(t)
    return view


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("H,pad,offset", [(64, 0, 0),      # whole stages
                                          (72, 8, 0), (100, 4, 8), (1000, 0, 0),   # a ragged last stage
                                          (36, 60, 4),     # less than one bf16 stage
                                          (8, 0, 0), (4, 12, 0),
                                          (1, 0, 0), (63, 1, 0), (129, 0, 0), (333, 3, 5),   # rows copied to whole chunks
                                          (128, 8, 3), (96, 1, 0)])   # whole chunks at addresses that are not
def test_logprobs_any_row_shape(tp, f32, H, pad, offset):
    M, V, N = 300, 777, 41
    rng = np.random.default_rng(H + pad)
    hidden = rng.normal(size=(N, H)).astype(np.float32)
    w = (rng.normal(size=(V, H)) / np.sqrt(H)).astype(np.float32)
    if not f32:
        hidden, w = synth.f32_to_bf16_bits(hidden), synth.f32_to_bf16_bits(w)
    rows, targets = rng.integers(0, N, size=M), (np.arange(M) * 5 + 1) % V
    st = tp.new_status("cuda")
    args = (_padded(hidden, H + pad, offset), _padded(w, H + pad, offset), dev(rows.astype(np.int32)),
            dev(targets.astype(np.int32)))
    logp, lse = tp.tppo_token_logprobs(*args, status=st)
    ref_lp, ref_lse = ofast.token_logprobs(hidden, w, rows, targets)
    assert int(host(st)[0]) == 0
    # exact products summed in fp32 over H and V, logits of size about 5: a few times 2^-24 * 8
    assert np.abs(host(logp) - ref_lp).max() <= 1e-5 and np.abs(host(lse) - ref_lse).max() <= 1e-5
    # the device's token count, and a workspace without room for copies
    m_dev = dev(np.array([M - 50], np.int64))
    small = tp._workspace(tp.load().tppo_token_logprobs_workspace_bytes(M, 64, V, tp.TPPO_F32), "cuda")
    for ws in (None, small):
        part, _ = tp.tppo_token_logprobs(*args, m_actual=m_dev, workspace=ws, status=st)
        assert np.abs(host(part)[:M - 50] - ref_lp[:M - 50]).max() <= 1e-5
    bad = args[2].clone()
    bad[7] = N
    part, _ = tp.tppo_token_logprobs(args[0], args[1], bad, args[3], status=st)
    assert int(host(st)[0]) == tp.STATUS_BAD_ROW and np.isnan(host(part)[7])
    assert np.abs(np.delete(host(part) - ref_lp, 7)).max() <= 1e-5


@pytest.mark.parametrize("M,V,H", [(1, 1, 64), (65, 63, 64), (63, 65, 320), (257, 640, 192), (300, 1001, 256)])
def test_logprob_grads_operands_read_along_their_rows(tp, M, V, H):
    """W and the logits' derivative are contracted over their row index: row and column counts around a stage and a
    tile, rows of a larger matrix with NaN in everything around them, and the derivatives' neighbours untouched."""
    import torch
    hidden, w, rows, targets, g = _bf16_case(M, V, H, seed=M * 7 + V)
    _, lse = ofast.token_logprobs(hidden, w, rows, targets)
    buf = torch.full((V + 2, H), 5.0, device="cuda")
    dh, dw = tp.tppo_token_logprobs_backward(_padded(hidden, H + 8, 16), _padded(w, H + 24, 8), dev(rows.astype(np.int32)),
                                             dev(targets.astype(np.int32)), dev(lse.astype(np.float32)),
                                             dev(g.astype(np.float32)), grad_w=buf[1:V + 1])
    ref_h, ref_w, abs_h, abs_w = ofast.token_logprob_grads(hidden, w, rows, targets, g, return_abs_bounds=True)
    assert_within_term_bound(host(dh), ref_h, abs_h, "grad_hidden")
    assert_within_term_bound(host(dw), ref_w, abs_w, "grad_w")
    assert (host(buf)[0] == 5.0).all() and (host(buf)[V + 1] == 5.0).all()
