"""Thin binding of libtppo.so (see include/tppo.h for the contract): ctypes, and for the calls of a training step a native
half (csrc/marshal.cpp), which checks, allocates and calls in half to four fifths of the time (figures there).

Argument marshalling only: every step of the path runs in the HIP kernels.
PyTorch provides device memory and the current HIP stream.  There is no CPU
fallback: if the shared library is missing, every call raises.
"""
import ctypes
import importlib.machinery
import importlib.util
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libtppo.so")
NATIVE_PATH = os.path.join(_HERE, "_marshal.so")

TPPO_F32, TPPO_BF16 = 0, 1
ERRORS = {-1: "TPPO_ERR_NULL", -2: "TPPO_ERR_SIZE", -3: "TPPO_ERR_PARAM", -4: "TPPO_ERR_DTYPE",
          -5: "TPPO_ERR_WORKSPACE", -6: "TPPO_ERR_LAUNCH"}
STATUS_BAD_TARGET, STATUS_BAD_LAYOUT, STATUS_CAPACITY, STATUS_BAD_ROW, STATUS_TIMEOUT = 1, 2, 4, 8, 16

_c_i64, _c_i32, _c_f32, _c_ptr, _c_size = (ctypes.c_int64, ctypes.c_int32, ctypes.c_float,
                                            ctypes.c_void_p, ctypes.c_size_t)
_SIGNATURES = {
    "tppo_version": (ctypes.c_int, []),
    "tppo_select_workspace_bytes": (_c_size, [_c_i64, _c_i64]),
    "tppo_select": (ctypes.c_int, [_c_ptr] * 4 + [_c_i64, _c_i64, _c_i32] + [_c_ptr] * 6 +
                    [_c_i64, _c_ptr, _c_ptr, _c_size, _c_ptr, _c_size, _c_ptr, _c_ptr]),
    "tppo_plan_bytes": (_c_size, [_c_i64, _c_i64]),
    "tppo_plan_build": (ctypes.c_int, [_c_ptr] * 3 + [_c_i64, _c_i64, _c_ptr, _c_size, _c_ptr, _c_ptr]),
    "tppo_token_logprobs_workspace_bytes": (_c_size, [_c_i64, _c_i64, _c_i64, ctypes.c_int]),
    "tppo_token_logprobs": (ctypes.c_int, [_c_ptr, _c_i64, _c_i64, _c_i64, _c_ptr, _c_i64, _c_i64,
                                           ctypes.c_int, _c_ptr, _c_ptr, _c_i64, _c_ptr, _c_ptr,
                                           _c_ptr, _c_ptr, _c_ptr, _c_size, _c_ptr, _c_ptr]),
    "tppo_egae_workspace_bytes": (_c_size, [_c_i64, _c_i64]),
    "tppo_egae": (ctypes.c_int, [_c_ptr] * 5 + [_c_i64, _c_i64, _c_f32, _c_f32, _c_ptr, _c_ptr,
                                                _c_ptr, _c_size, _c_ptr, _c_ptr, _c_ptr]),
    "tppo_egae_terminal": (ctypes.c_int, [_c_ptr] * 5 + [_c_i64, _c_i64, _c_f32, _c_f32, _c_ptr, _c_ptr,
                                                         _c_ptr, _c_size, _c_ptr, _c_ptr, _c_ptr]),
    "tppo_egae_static_max_tiles": (_c_i64, []),
    "tppo_egae_static": (ctypes.c_int, [_c_ptr] * 5 + [_c_i64, _c_i64, _c_f32, _c_f32, _c_ptr, _c_ptr,
                                                       _c_ptr, _c_ptr]),
    "tppo_ppo_losses_workspace_bytes": (_c_size, [_c_i64, _c_i64]),
    "tppo_ppo_losses": (ctypes.c_int, [_c_ptr] * 9 + [_c_i64, _c_i64] + [_c_f32] * 4 +
                        [_c_ptr, _c_ptr, _c_size, _c_ptr, _c_ptr, _c_ptr]),
    "tppo_ppo_losses_backward_workspace_bytes": (_c_size, [_c_i64, _c_i64]),
    "tppo_ppo_losses_backward": (ctypes.c_int, [_c_ptr] * 9 + [_c_i64, _c_i64] + [_c_f32] * 6 +
                                 [_c_i64, _c_i64] + [_c_ptr] * 5 + [_c_size, _c_ptr, _c_ptr, _c_ptr]),
    "tppo_token_logprobs_backward_workspace_bytes": (_c_size, [_c_i64, _c_i64, _c_i64, ctypes.c_int]),
    "tppo_token_logprobs_backward": (ctypes.c_int, [_c_ptr, _c_i64, _c_i64, _c_i64, _c_ptr, _c_i64, _c_i64,
                                                    ctypes.c_int, _c_ptr, _c_ptr, _c_i64, _c_ptr, _c_ptr,
                                                    _c_ptr, _c_ptr, _c_ptr, _c_i32, _c_ptr, _c_size, _c_ptr,
                                                    _c_ptr]),
    "tppo_batcher_create": (_c_ptr, [_c_i64, _c_i32, _c_i32]),
    "tppo_batcher_destroy": (None, [_c_ptr]),
    "tppo_batcher_refill": (ctypes.c_int, [_c_ptr, _c_ptr, _c_i64, ctypes.POINTER(ctypes.c_int64)]),
    "tppo_batcher_advance": (ctypes.c_int, [_c_ptr, _c_ptr, _c_ptr]),
    "tppo_batcher_layout": (ctypes.c_int, [_c_ptr] * 6),
    "tppo_value_head": (ctypes.c_int, [_c_ptr, _c_i64, _c_i64, _c_i64, _c_ptr, _c_f32, ctypes.c_int, _c_ptr,
                                       _c_ptr, _c_i64, _c_ptr, _c_ptr, _c_ptr, _c_ptr]),
    "tppo_diag_streams": (ctypes.c_int, [_c_ptr, _c_ptr, _c_i64, _c_i64, _c_i32, _c_i32, _c_ptr]),
    "tppo_diag_mfma_rate": (ctypes.c_int, [_c_ptr, _c_ptr, _c_i64, ctypes.POINTER(ctypes.c_double), _c_ptr]),
}
EXPORTS = tuple(_SIGNATURES)
_lib = None


def load():
    """Load libtppo.so (built by ``python -m paper_2506_15050_amd.build``)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: build it with "
                               "`python -m paper_2506_15050_amd.build`; there is no fallback path")
        lib = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in _SIGNATURES.items():
            fn = getattr(lib, name)
            fn.restype, fn.argtypes = res, args
        _lib = lib
    return _lib


_native_module = None


def _native():
    """The native half of the binding (built with the library)."""
    global _native_module
    if _native_module is None:
        load()
        if not os.path.exists(NATIVE_PATH):
            raise RuntimeError(f"{NATIVE_PATH} is missing: build it with "
                               "`python -m paper_2506_15050_amd.build`; there is no fallback path")
        loader = importlib.machinery.ExtensionFileLoader("_marshal", NATIVE_PATH)
        _native_module = importlib.util.module_from_spec(importlib.util.spec_from_loader("_marshal", loader))
        loader.exec_module(_native_module)
    return _native_module


def _check(rc, what):
    if rc != 0:
        raise RuntimeError(f"{what} failed: {ERRORS.get(rc, rc)}")


def _ptr(t):
    return None if t is None else t.data_ptr()          # the argument types turn it into a pointer


# The current stream of the current device.  torch's way to the raw handle has private names; a torch without them gets
# the public way, a Stream object that costs 2.8 us to make (the smallest calls are bound by what happens here).
if hasattr(torch._C, "_cuda_getCurrentRawStream") and hasattr(torch._C, "_cuda_getDevice"):
    _raw_stream, _device = torch._C._cuda_getCurrentRawStream, torch._C._cuda_getDevice

    def _stream():
        return _raw_stream(_device())
else:
    def _stream():
        return torch.cuda.current_stream().cuda_stream


def _dev_i32(t):
    assert t.is_cuda and t.dtype == torch.int32 and t.is_contiguous()
    return t


def _dev_f32(t):
    assert t.is_cuda and t.dtype == torch.float32 and t.is_contiguous()
    return t


def _workspace(nbytes, device):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=device)


def new_status(device):
    return torch.zeros(1, dtype=torch.int32, device=device)


def tppo_select(cu_seqlens, ctx_len, done, input_ids, tail_drop, capacity=None, status=None,
                want_indices=True, n_tok=None, workspace=None, want_plan=False, plan=None):
    """Token filter.  Returns a dict of device tensors: resp_off, sel_off, keep_len,
    sel_rows, sel_targets, sel_resp_idx (capacity-sized) and counts (int64[3] =
    M, n_resp, N_val); with ``want_plan`` (or a ``plan`` buffer) also ``plan``, the
    work plan that tppo_egae* and the loss calls take."""
    native = _native()
    B = ctx_len.numel()
    if input_ids is not None:
        n_tok = input_ids.numel()
    assert n_tok is not None, "n_tok is required when input_ids is None"
    cap = n_tok if capacity is None else int(capacity)
    kinds, sizes = "iiil", [B + 1, B + 1, B, 3]
    if want_indices:
        kinds += "iii" if input_ids is not None else "ii"
        sizes += [cap] * (len(kinds) - 4)
    if workspace is None and want_indices:
        kinds += "b"
        sizes.append(max(native.select_workspace_bytes(B, max(cap, n_tok)), 256))
    if plan is None and want_plan:
        kinds += "b"
        sizes.append(max(native.plan_bytes(n_tok, B), 256))
    made = iter(native.empties(cu_seqlens, kinds, *sizes))
    resp_off, sel_off, keep_len, counts = next(made), next(made), next(made), next(made)
    out = dict(resp_off=resp_off, sel_off=sel_off, keep_len=keep_len, counts=counts)
    rows = targets = resp_idx = None
    ws = workspace
    if want_indices:
        rows, resp_idx = next(made), next(made)
        targets = next(made) if input_ids is not None else None
        out.update(sel_rows=rows, sel_targets=targets, sel_resp_idx=resp_idx)
        if ws is None:
            ws = next(made)
    if plan is None and want_plan:
        plan = next(made)
    out["plan"] = plan
    rc = native.select(cu_seqlens, ctx_len, done, input_ids, B, n_tok, int(tail_drop), resp_off, sel_off, keep_len, rows,
                       targets, resp_idx, cap, counts, ws, plan, status, _stream())
    _check(rc, "tppo_select")
    return out


def tppo_plan_build(resp_off, keep_len, done, n_resp, status=None, plan=None):
    """Work plan of a batch layout (keep_len may be None: such a plan serves tppo_egae* only)."""
    lib = load()
    B = done.numel()
    if plan is None:
        plan = _workspace(lib.tppo_plan_bytes(int(n_resp), B), resp_off.device)
    rc = lib.tppo_plan_build(_ptr(_dev_i32(resp_off)), _ptr(keep_len), _ptr(_dev_i32(done)), B, int(n_resp),
                             _ptr(plan), plan.numel(), _ptr(status), _stream())
    _check(rc, "tppo_plan_build")
    return plan


def tppo_token_logprobs(hidden, w_head, sel_rows, sel_targets, M=None, m_actual=None,
                        out_index=None, out_size=None, want_lse=True, status=None, workspace=None):
    """log pi(a_t|s_t) of the kept tokens.  hidden [n_rows, H], w_head [V, H], both
    bf16 or both fp32.  Returns (logp, lse)."""
    lib = load()
    assert hidden.is_cuda and w_head.is_cuda and hidden.dtype == w_head.dtype
    assert hidden.dim() == 2 and w_head.dim() == 2 and hidden.stride(1) == 1 and w_head.stride(1) == 1
    dt = {torch.float32: TPPO_F32, torch.bfloat16: TPPO_BF16}[hidden.dtype]
    n_rows, H = hidden.shape
    V = w_head.shape[0]
    M = sel_rows.numel() if M is None else int(M)
    n_out = M if out_size is None else int(out_size)
    native = _native()
    made = native.empties(hidden, "ff" if want_lse else "f", *([n_out] * (2 if want_lse else 1)))
    logp, lse = made if want_lse else (made[0], None)
    ws = workspace
    if ws is None:
        ws = _workspace(lib.tppo_token_logprobs_workspace_bytes(M, H, V, dt), hidden.device)
    rc = native.token_logprobs(hidden, n_rows, H, hidden.stride(0), w_head, V, w_head.stride(0), dt, sel_rows, sel_targets, M,
                               m_actual, out_index, logp, lse, ws, status, _stream())
    _check(rc, "tppo_token_logprobs")
    return logp, lse


def _scratch(lib_bytes, n_resp, B, workspace, plan, device):
    """The workspace of a call that may have been given a plan instead."""
    if plan is not None or workspace is not None:
        return workspace
    return _workspace(lib_bytes(n_resp, B), device)


def tppo_egae(rewards, values, resp_off, done, gamma, lam, bootstrap=None, status=None,
              workspace=None, out=None, plan=None):
    """Extended GAE advantages and Monte-Carlo returns.  Returns (adv, ret)."""
    lib = load()
    n_resp, B = rewards.numel(), done.numel()
    adv, ret = out if out is not None else (torch.empty_like(rewards), torch.empty_like(rewards))
    ws = _scratch(lib.tppo_egae_workspace_bytes, n_resp, B, workspace, plan, rewards.device)
    rc = _native().egae(rewards, values, resp_off, done, bootstrap, B, n_resp, float(gamma), float(lam), adv, ret, ws, plan,
                        status, _stream())
    _check(rc, "tppo_egae")
    return adv, ret


def tppo_egae_static(rewards, values, resp_off, done, gamma, lam, bootstrap=None, status=None, out=None):
    """``tppo_egae`` without a workspace: the library's own fixed array holds the plan.  The binding
    still allocates the outputs unless ``out=(adv, ret)`` is given.  Returns (adv, ret)."""
    lib = load()
    n_resp, B = rewards.numel(), done.numel()
    adv, ret = out if out is not None else (torch.empty_like(rewards), torch.empty_like(rewards))
    rc = lib.tppo_egae_static(_ptr(_dev_f32(rewards)), _ptr(_dev_f32(values)), _ptr(_dev_i32(resp_off)),
                              _ptr(_dev_i32(done)), _ptr(bootstrap), B, n_resp, float(gamma), float(lam),
                              _ptr(adv), _ptr(ret), _ptr(status), _stream())
    _check(rc, "tppo_egae_static")
    return adv, ret


def tppo_egae_terminal(terminal_reward, values, resp_off, done, gamma, lam, bootstrap=None, status=None,
                       workspace=None, out=None, plan=None):
    """Extended GAE with one terminal reward per finished sequence instead of a
    dense reward array.  Returns (adv, ret)."""
    lib = load()
    n_resp, B = values.numel(), done.numel()
    adv, ret = out if out is not None else (torch.empty_like(values), torch.empty_like(values))
    ws = _scratch(lib.tppo_egae_workspace_bytes, n_resp, B, workspace, plan, values.device)
    rc = _native().egae_terminal(terminal_reward, values, resp_off, done, bootstrap, B, n_resp, float(gamma), float(lam), adv,
                                 ret, ws, plan, status, _stream())
    _check(rc, "tppo_egae_terminal")
    return adv, ret


class LossOut(ctypes.Structure):
    _fields_ = [("policy_loss", ctypes.c_float), ("value_loss", ctypes.c_float),
                ("policy_sum", ctypes.c_float), ("value_sum", ctypes.c_float),
                ("n_policy", ctypes.c_int64), ("n_value", ctypes.c_int64)]


def tppo_ppo_losses(logp_new, logp_old, adv, v_new, v_old, ret, resp_off, keep_len, done,
                    eps_low, eps_high, xi_low, xi_high, status=None, workspace=None, out=None, plan=None):
    """Clipped policy / value losses.  Returns a 32-byte device tensor holding a
    ``tppo_loss_out``; ``read_loss_out`` copies it to the host."""
    lib = load()
    dev = resp_off.device
    B = done.numel()
    n_resp = (logp_new if logp_new is not None else v_new).numel()
    res = torch.empty(ctypes.sizeof(LossOut), dtype=torch.uint8, device=dev) if out is None else out
    ws = _scratch(lib.tppo_ppo_losses_workspace_bytes, n_resp, B, workspace, plan, dev)
    rc = _native().ppo_losses(logp_new, logp_old, adv, v_new, v_old, ret, resp_off, keep_len, done, B, n_resp, float(eps_low),
                              float(eps_high), float(xi_low), float(xi_high), res, ws, plan, status, _stream())
    _check(rc, "tppo_ppo_losses")
    return res


def read_loss_out(res):
    """Device ``tppo_loss_out`` -> dict (synchronises)."""
    raw = bytes(res.cpu().numpy().tobytes())
    s = LossOut.from_buffer_copy(raw)
    return {name: getattr(s, name) for name, _ in LossOut._fields_}


def tppo_token_logprobs_backward(hidden, w_head, sel_rows, sel_targets, lse, grad_logp, M=None,
                                 in_index=None, want_hidden=True, want_w=True, grad_w=None,
                                 accumulate_w=False, status=None, workspace=None):
    """Derivatives of the kept tokens' log-probs with respect to the hidden rows
    ([M, H] fp32, compact order) and the head matrix ([V, H] fp32)."""
    lib = load()
    assert hidden.is_cuda and w_head.is_cuda and hidden.dtype == w_head.dtype == torch.bfloat16
    assert hidden.stride(1) == 1 and w_head.stride(1) == 1
    n_rows, H = hidden.shape
    V = w_head.shape[0]
    M = sel_rows.numel() if M is None else int(M)
    dev = hidden.device
    g_h = torch.empty(M, H, dtype=torch.float32, device=dev) if want_hidden else None
    if want_w and grad_w is None:
        grad_w = torch.empty(V, H, dtype=torch.float32, device=dev)
    if not want_w:
        grad_w = None
    ws = workspace
    if ws is None:
        ws = _workspace(lib.tppo_token_logprobs_backward_workspace_bytes(M, H, V, TPPO_BF16), dev)
    rc = lib.tppo_token_logprobs_backward(_ptr(hidden), n_rows, H, hidden.stride(0), _ptr(w_head), V,
                                          w_head.stride(0), TPPO_BF16, _ptr(_dev_i32(sel_rows)),
                                          _ptr(_dev_i32(sel_targets)), M, _ptr(_dev_f32(lse)),
                                          _ptr(_dev_f32(grad_logp)), _ptr(in_index), _ptr(g_h), _ptr(grad_w),
                                          1 if accumulate_w else 0, _ptr(ws), ws.numel(), _ptr(status),
                                          _stream())
    _check(rc, "tppo_token_logprobs_backward")
    return g_h, grad_w


def tppo_value_head(hidden, w_value, bias=0.0, rows=None, M=None, m_actual=None, out_index=None,
                    out_size=None, status=None, out=None):
    """V(s_t) = w_value . hidden[rows[t]] + bias.  Returns the fp32 values."""
    lib = load()
    assert hidden.is_cuda and hidden.dtype == w_value.dtype == torch.bfloat16 and hidden.stride(1) == 1
    n_rows, H = hidden.shape
    if M is None:
        M = n_rows if rows is None else rows.numel()
    n_out = int(M) if out_size is None else int(out_size)
    v = torch.empty(n_out, dtype=torch.float32, device=hidden.device) if out is None else out
    rc = _native().value_head(hidden, n_rows, H, hidden.stride(0), w_value, float(bias), TPPO_BF16, rows, out_index, int(M),
                              m_actual, v, status, _stream())
    _check(rc, "tppo_value_head")
    return v


class Batcher:
    """Successive-batching slot bookkeeping (host side, numpy int32 arrays in and out)."""

    def __init__(self, slots, window, max_response):
        self._lib = load()
        self.slots = int(slots)
        self._h = self._lib.tppo_batcher_create(self.slots, int(window), int(max_response))
        if not self._h:
            raise ValueError("tppo_batcher_create: bad sizes")

    def close(self):
        if self._h:
            self._lib.tppo_batcher_destroy(self._h)
            self._h = None

    __del__ = close

    @staticmethod
    def _i32(a):
        import numpy as np
        return np.ascontiguousarray(a, dtype=np.int32)

    def refill(self, prompt_len):
        p = self._i32(prompt_len)
        taken = ctypes.c_int64(0)
        _check(self._lib.tppo_batcher_refill(self._h, p.ctypes.data, p.size, ctypes.byref(taken)),
               "tppo_batcher_refill")
        return taken.value

    def advance(self, gen_len, eos):
        g, e = self._i32(gen_len), self._i32(eos)
        assert g.size == self.slots and e.size == self.slots
        _check(self._lib.tppo_batcher_advance(self._h, g.ctypes.data, e.ctypes.data), "tppo_batcher_advance")

    def layout(self):
        import numpy as np
        cu = np.empty(self.slots + 1, np.int32)
        ctx, prompt, done = (np.empty(self.slots, np.int32) for _ in range(3))
        ids = np.empty(self.slots, np.int64)
        _check(self._lib.tppo_batcher_layout(self._h, cu.ctypes.data, ctx.ctypes.data, prompt.ctypes.data,
                                             done.ctypes.data, ids.ctypes.data), "tppo_batcher_layout")
        return cu, ctx, prompt, done, ids


class LossStats(ctypes.Structure):
    _fields_ = [("ratio_mean", ctypes.c_float), ("policy_clip_frac", ctypes.c_float),
                ("value_clip_frac", ctypes.c_float), ("reserved", ctypes.c_float),
                ("n_policy_clipped", ctypes.c_int64), ("n_value_clipped", ctypes.c_int64)]


def tppo_ppo_losses_backward(logp_new, logp_old, adv, v_new, v_old, ret, resp_off, keep_len, done,
                             eps_low, eps_high, xi_low, xi_high, policy_scale=1.0, value_scale=1.0,
                             policy_denominator=0, value_denominator=0, status=None, workspace=None,
                             out=None, stats=None, grads=None, plan=None):
    """Derivatives of the two losses (plus the losses and clip statistics) in one
    pass.  Returns (grad_logp, grad_v, loss_out tensor, stats tensor)."""
    lib = load()
    dev = resp_off.device
    B = done.numel()
    n_resp = (logp_new if logp_new is not None else v_new).numel()
    if grads is None:
        g_lp = torch.empty(n_resp, dtype=torch.float32, device=dev) if logp_new is not None else None
        g_v = torch.empty(n_resp, dtype=torch.float32, device=dev) if v_new is not None else None
    else:
        g_lp, g_v = grads
    res = torch.empty(ctypes.sizeof(LossOut), dtype=torch.uint8, device=dev) if out is None else out
    st = torch.empty(ctypes.sizeof(LossStats), dtype=torch.uint8, device=dev) if stats is None else stats
    ws = _scratch(lib.tppo_ppo_losses_backward_workspace_bytes, n_resp, B, workspace, plan, dev)
    rc = _native().ppo_losses_backward(
        logp_new, logp_old, adv, v_new, v_old, ret, resp_off, keep_len, done, B, n_resp, float(eps_low), float(eps_high),
        float(xi_low), float(xi_high), float(policy_scale), float(value_scale), int(policy_denominator),
        int(value_denominator), g_lp, g_v, res, st, ws, plan, status, _stream())
    _check(rc, "tppo_ppo_losses_backward")
    return g_lp, g_v, res, st


def read_loss_stats(st):
    """Device ``tppo_loss_stats`` -> dict (synchronises)."""
    s = LossStats.from_buffer_copy(bytes(st.cpu().numpy().tobytes()))
    return {name: getattr(s, name) for name, _ in LossStats._fields_ if name != "reserved"}


def tppo_diag_mfma_rate(operands, out, iters):
    """Launch the register-resident MFMA loop; returns the flop count of the launch."""
    lib = load()
    flop = ctypes.c_double(0.0)
    rc = lib.tppo_diag_mfma_rate(_ptr(operands), _ptr(out), int(iters), ctypes.byref(flop), _stream())
    _check(rc, "tppo_diag_mfma_rate")
    return flop.value


def tppo_diag_streams(src, dst, bytes_per_stream, stride_bytes, n_read, n_write):
    """Elementwise pass over n_read input and n_write output streams; returns the bytes moved."""
    lib = load()
    _check(lib.tppo_diag_streams(_ptr(src), _ptr(dst), int(bytes_per_stream), int(stride_bytes), int(n_read),
                                 int(n_write), _stream()), "tppo_diag_streams")
    return int(bytes_per_stream) * (n_read + n_write)
