"""The binding's native half: what it refuses, and the buffers it makes (no GPU work here)."""
import ctypes
import os

import numpy as np
import pytest
import torch


@pytest.fixture(scope="module")
def native():
    from paper_2506_15050_amd import binding, build
    if not (os.path.exists(binding.LIB_PATH) and os.path.exists(binding.NATIVE_PATH)):
        build.build()
    return binding._native()


def test_empties(native):
    made = native.empties(torch.zeros(1), "ilfb", 3, 0, 5, 7)
    assert [t.dtype for t in made] == [torch.int32, torch.int64, torch.float32, torch.uint8]
    assert [tuple(t.shape) for t in made] == [(3,), (0,), (5,), (7,)] and len({t.data_ptr() for t in made if t.numel()}) == 3
    for bad, error in (((torch.zeros(1), "i", -3), RuntimeError), ((torch.zeros(1), "ii", 3), TypeError),
                       ((None, "i", 3), TypeError), ((torch.zeros(1), "i", "3"), TypeError)):
        with pytest.raises(error):
            native.empties(*bad)


@pytest.mark.parametrize("args,error", [
    ([], TypeError),                                                        # count
    ([torch.zeros(3)] * 15, AssertionError),                                # not on the device
    ([None] * 15, AssertionError),                                          # no tensor where one is required
])
def test_refusals(native, args, error):
    with pytest.raises(error):
        native.egae(*args)


def test_codes_and_pointers_reach_the_entry_point(native):
    # all pointers NULL: the entry point's own codes, by what it looks at first
    args = [None, 1, 8, 8, None, 0.0, 1, None, None, 3, None, None, None, 0]
    assert native.value_head(*args) == -1                                   # NULL
    assert native.value_head(*args[:9], -3, *args[10:]) == -2               # size
    assert native.value_head(*args[:9], 0, *args[10:]) == 0                 # nothing to do
    with pytest.raises(AttributeError):
        native.value_head("hidden", *args[1:])
    with pytest.raises(TypeError):
        native.value_head(*args[:13], "stream")


def test_sizes(native):
    from paper_2506_15050_amd import binding
    lib = binding.load()
    for n, B in ((0, 0), (1, 1), (1000, 3), (2_400_000, 512)):
        assert native.plan_bytes(n, B) == lib.tppo_plan_bytes(n, B)
        assert native.select_workspace_bytes(B, n) == lib.tppo_select_workspace_bytes(B, n)


def test_allocations_raise_what_torch_raises(native):
    from torch.utils._python_dispatch import TorchDispatchMode
    like = torch.zeros(1)

    class Mode(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            raise KeyError("a mode's own exception")
    with Mode():
        for make in (lambda: torch.empty(3), lambda: native.empties(like, "i", 3)):
            with pytest.raises(KeyError):
                make()


def test_other_threads_run_during_allocations(native):
    """torch's filling of fresh memory under deterministic algorithms makes an allocation last: the longest time in which
    another thread got nowhere is well below it."""
    import threading
    import time
    like, stop, gaps = torch.zeros(1), threading.Event(), [0.0]

    def watch():
        last = time.perf_counter()
        while not stop.is_set():
            time.sleep(0.001)
            now = time.perf_counter()
            gaps[0], last = max(gaps[0], now - last), now
    was, threads = torch.are_deterministic_algorithms_enabled(), torch.get_num_threads()
    torch.use_deterministic_algorithms(True)
    torch.set_num_threads(1)
    watcher = threading.Thread(target=watch)
    try:
        watcher.start()
        begin = time.perf_counter()
        native.empties(like, "b", 1 << 30)
        took = time.perf_counter() - begin
    finally:
        stop.set()
        watcher.join()
        torch.use_deterministic_algorithms(was)
        torch.set_num_threads(threads)
    assert took > 0.05 and gaps[0] < took / 2, (took, gaps[0])


class Array:
    """Another library's array: what the entry points need of a tensor, and no torch.Tensor."""
    def __init__(self, at=0, n=0, dtype=torch.float32, is_cuda=True, dense=True):
        self.at, self.n, self.dtype, self.is_cuda, self.dense = at, n, dtype, is_cuda, dense

    def data_ptr(self):
        return self.at

    def numel(self):
        return self.n

    def is_contiguous(self):
        return self.dense


def test_arrays_that_are_no_tensors(native):
    def egae(rewards):
        ints = Array(dtype=torch.int32)
        return native.egae(rewards, Array(), ints, ints, None, 1, 1, 1.0, 1.0, None, None, None, None, None, 0)
    assert egae(Array()) == -1                                              # taken, and its pointer is NULL
    for bad in (Array(dtype=torch.int32), Array(is_cuda=False), Array(dense=False)):
        with pytest.raises(AssertionError):
            egae(bad)
    with pytest.raises(AttributeError):
        egae(3.0)


def test_a_subclass_has_its_say(native):
    says = {torch.Tensor.data_ptr: 0, torch.Tensor.is_cuda.__get__: True}

    class Elsewhere(torch.Tensor):
        @classmethod
        def __torch_function__(cls, func, types, args=(), kwargs=None):
            return says[func] if func in says else super().__torch_function__(func, types, args, kwargs or {})
    f32, i32 = (torch.zeros(3, dtype=t).as_subclass(Elsewhere) for t in (torch.float32, torch.int32))
    assert native.egae(f32, f32, i32, i32, None, 1, 1, 1.0, 1.0, None, None, None, None, None, 0) == -1      # NULL, as it says


@pytest.mark.parametrize("make", [lambda: np.int64(5), lambda: torch.tensor(5), lambda: (1 << 64) + 5, lambda: 5.0, lambda: "5"])
def test_numbers(native, make):
    """Whole numbers are taken and refused as by ctypes."""
    from paper_2506_15050_amd import binding
    for plan_bytes in (binding.load().tppo_plan_bytes, native.plan_bytes):
        if isinstance(make(), (float, str)):
            with pytest.raises(ctypes.ArgumentError):
                plan_bytes(make(), 1)
        else:
            assert plan_bytes(make(), 1) == plan_bytes(5, 1)


@pytest.mark.gpu
def test_buffers_that_are_no_tensors(native):
    from paper_2506_15050_amd import binding as tp
    i32 = lambda *x: torch.tensor(x, dtype=torch.int32, device="cuda")
    cu, ctx, done, n_tok = i32(0, 9, 20), i32(2, 3), i32(1, 0), 20
    plain = tp.tppo_select(cu, ctx, done, None, 1, n_tok=n_tok, want_plan=True)
    keep = [torch.zeros(1 << 22, dtype=torch.uint8, device="cuda") for _ in range(2)]
    ws, plan = (Array(t.data_ptr(), t.numel()) for t in keep)
    again = tp.tppo_select(cu, ctx, done, None, 1, n_tok=n_tok, workspace=ws, plan=plan)
    kept = int(plain["counts"][0])
    assert again["counts"].tolist() == plain["counts"].tolist() == [7 + 8 - 1, 15, 7]
    assert again["sel_rows"][:kept].tolist() == plain["sel_rows"][:kept].tolist()
    for short in (dict(workspace=Array(keep[0].data_ptr(), 16)), dict(plan=Array(keep[1].data_ptr(), 16))):
        with pytest.raises(RuntimeError, match="WORKSPACE"):
            tp.tppo_select(cu, ctx, done, None, 1, n_tok=n_tok, **short)


@pytest.mark.gpu
def test_out_of_memory_is_torchs_own(native):
    like = torch.zeros(1, device="cuda")
    for make in (lambda: torch.empty(1 << 46, dtype=torch.uint8, device="cuda"), lambda: native.empties(like, "b", 1 << 46)):
        with pytest.raises(torch.OutOfMemoryError):
            make()
