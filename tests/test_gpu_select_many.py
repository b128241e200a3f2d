"""The token filter on batches of up to 1024 sequences whose kept tokens are more turns of all workers than the line between both ways
of dealing them out, and just fewer: with one workgroup for the plan's list and with eight, and cut by the capacity."""
import numpy as np
import pytest

from test_gpu_parity import check_select, dev, host, ofast, tp  # noqa: F401

pytestmark = pytest.mark.gpu
TURN = 511 * 1024 * 4                                               # up to 128 sequences: all workgroups but one
LISTED_TURN = 504 * 1024 * 4                                        # more, with a plan: all but eight


def batch(B, n):
    """n kept tokens in B sequences, all of them finished."""
    rng = np.random.default_rng(5)
    win = np.diff(np.concatenate([[0], np.sort(rng.integers(0, n, size=B - 1)), [n]]))
    ctx = rng.integers(1, 9, size=B)
    cu = np.concatenate([[0], np.cumsum(win + ctx)]).astype(np.int32)
    return dict(cu_seqlens=cu, ctx_len=ctx.astype(np.int32), done=np.ones(B, np.int32), n_tok=int(cu[-1]),
                input_ids=rng.integers(0, 1000, size=int(cu[-1])).astype(np.int32), tail_drop=0)


@pytest.mark.parametrize("extra", [-3, 0, 1, 4096 * 300 + 2])
def test_many_turns(tp, extra):
    check_select(tp, batch(7, 5 * TURN + extra))


@pytest.mark.parametrize("B,cap,beyond", [(129, 5 * LISTED_TURN, 0), (200, 5 * LISTED_TURN + 1, 0), (1000, 5 * LISTED_TURN + 4096 * 260 + 3, 0),
                                          (1024, 6 * LISTED_TURN, 70001), (7, 5 * TURN + 4099, 1), (300, 5 * LISTED_TURN + 8190, 5000),
                                          (300, 5 * LISTED_TURN - 2, 5000)])
def test_many_turns_with_a_plan_up_to_the_capacity(tp, B, cap, beyond):
    b = batch(B, cap + beyond)
    ref = ofast.select(b["cu_seqlens"], b["ctx_len"], b["done"], b["input_ids"], 0)
    status = tp.new_status("cuda")
    i32 = lambda n: dev(np.full(n, -7, np.int32))
    resp, sel, keep, counts = i32(B + 1), i32(B + 1), i32(B), dev(np.zeros(3, np.int64))
    lists = [i32(cap + 64) for _ in range(3)]
    native = tp._native()
    ws = dev(np.zeros(native.select_workspace_bytes(B, b["n_tok"]), np.uint8))
    plan = dev(np.full(native.plan_bytes(b["n_tok"], B), 255, np.uint8))
    rc = native.select(dev(b["cu_seqlens"]), dev(b["ctx_len"]), dev(b["done"]), dev(b["input_ids"]), B, b["n_tok"], 0, resp, sel, keep,
                       *lists, cap, counts, ws, plan, status, tp._stream())
    assert rc == 0 and int(host(status)[0]) == (tp.STATUS_CAPACITY if beyond else 0)
    assert host(counts).tolist() == [cap + beyond, ref["N_resp"], ref["N_val"]] == [cap + beyond] * 3
    for got, k in ((resp, "resp_off"), (sel, "sel_off"), (keep, "keep_len")):
        assert np.array_equal(host(got), ref[k]), k
    for got, k in zip(lists, ("sel_rows", "sel_targets", "sel_resp_idx")):
        got = host(got)
        assert np.array_equal(got[:cap], ref[k][:cap]) and (got[cap:] == -7).all(), k
    # the list that tppo_plan_build makes of the same offsets
    n, built = ref["N_resp"], host(tp.tppo_plan_build(resp, keep, dev(b["done"]), ref["N_resp"]))
    mine, tiles = host(plan), int(built[:4].view(np.int32)[0])
    assert np.array_equal(mine[:32], built[:32]) and np.array_equal(mine[256:256 + 16 * tiles], built[256:256 + 16 * tiles])
    words = 256 + (16 * (b["n_tok"] // 1024 + B + 1) + 255) // 256 * 256 + (32 * (b["n_tok"] // 1024 + B + 1) + 255) // 256 * 256
    assert not mine[words:].any() and n == cap + beyond
