"""The token filter on both sides of the batch size where it goes from one
launch to two: indices, counts, capacity and the plan it hands out."""
import numpy as np
import pytest

from test_gpu_parity import dev, host, ofast, tp  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,most", [(1, 1), (1, 9001), (3, 2), (1023, 40), (1024, 1500), (1025, 1500), (2049, 700)])
def test_select_routes(tp, B, most):
    rng = np.random.default_rng(B + most)
    win = rng.integers(0 if B > 1 else 1, most + 1, size=B)
    win[rng.random(B) < 0.2] *= int(B == 1)                 # empty windows, runs of them among 1024 sequences
    ctx = rng.integers(1, 9, size=B).astype(np.int32)
    done = (rng.random(B) < 0.4).astype(np.int32)
    cu = np.concatenate([[0], np.cumsum(win + ctx)]).astype(np.int32)
    n_tok = int(cu[-1])
    ids = rng.integers(0, 50000, size=n_tok).astype(np.int32)
    for drop in (0, 3):
        ref = ofast.select(cu, ctx, done, ids, drop)
        M = ref["M"]
        for cap, with_ids in ((n_tok, True), (max(M - 1, 0), True), (M, False)):
            st = tp.new_status("cuda")
            sel = tp.tppo_select(dev(cu), dev(ctx), dev(done), dev(ids) if with_ids else None, drop, capacity=cap,
                                 n_tok=n_tok, status=st, want_plan=True)
            assert int(host(st)[0]) == (tp.STATUS_CAPACITY if 0 < cap < M else 0)
            assert host(sel["counts"]).tolist() == [M, ref["N_resp"], ref["N_val"]]
            for k in ("resp_off", "sel_off", "keep_len"):
                assert np.array_equal(host(sel[k]), ref[k]), k
            for k in ("sel_rows", "sel_targets", "sel_resp_idx"):
                if sel[k] is not None:
                    assert np.array_equal(host(sel[k])[:min(M, cap)], ref[k][:cap]), k
        # the plan is the one tppo_plan_build makes of the same offsets
        n, cap_s = ref["N_resp"], n_tok // 1024 + B + 1
        built = host(tp.tppo_plan_build(sel["resp_off"], sel["keep_len"], dev(done), n))
        mine, cap_b = host(sel["plan"]), n // 1024 + B + 1
        h_s, h_b = mine[:64].view(np.int32), built[:64].view(np.int32)
        assert np.array_equal(h_s[:8], h_b[:8]) and (h_s[8], h_b[8]) == (cap_s, cap_b)

        def parts(raw, cap):
            at = 256 + (16 * cap + 255) // 256 * 256
            return (raw[256:256 + 16 * int(h_b[0])], raw[at:at + 32 * ((n + 1023) // 1024)],
                    raw[at + (32 * cap + 255) // 256 * 256:])
        (t_s, f_s, w_s), (t_b, f_b, w_b) = parts(mine, cap_s), parts(built, cap_b)
        assert np.array_equal(t_s, t_b) and np.array_equal(f_s, f_b) and not w_s.any() and not w_b.any()
