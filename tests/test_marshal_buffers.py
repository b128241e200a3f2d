"""The buffers that the binding's native half makes (csrc/marshal.cpp): plain tensors that have nothing to do with each other."""
import io

import pytest
import torch

from test_marshal import native  # noqa: F401

KINDS = {"i": torch.int32, "l": torch.int64, "f": torch.float32, "b": torch.uint8}


def made_of(native, kinds, sizes):  # noqa: F811
    made = native.empties(torch.zeros(1), kinds, *sizes)
    assert [t.dtype for t in made] == [KINDS[k] for k in kinds] and [tuple(t.shape) for t in made] == [(n,) for n in sizes]
    assert all(t.is_contiguous() and t.is_leaf and not t.requires_grad and t._base is None for t in made)
    spans = sorted((t.data_ptr(), t.data_ptr() + t.numel() * t.element_size()) for t in made if t.numel())
    assert all(a[1] <= b[0] for a, b in zip(spans, spans[1:]))
    assert all(t.data_ptr() == 0 for t in made if t.numel() == 0)
    for k, t in enumerate(made):
        t.fill_(k)
    assert all(bool((t == k).all()) for k, t in enumerate(made))
    return made


def storages(made):
    return len({t.untyped_storage().data_ptr() for t in made})


def saved_bytes(t):
    file = io.BytesIO()
    torch.save(t, file)
    return file.tell()


@pytest.mark.parametrize("kinds,sizes", [("iiiliiibb", (5, 5, 4, 3, 100, 100, 100, 512, 40000)), ("iiil", (2, 2, 1, 3)),
                                         ("iiilii", (2, 2, 1, 3, 0, 0)), ("bilf", ((1 << 20) - 1536, 128, 64, 128)), ("ff", (0, 100)),
                                         ("iiilb", (0, 5, 4, 0, 0)), ("f", (7,))])
def test_each_is_an_allocation_of_its_own(native, kinds, sizes):  # noqa: F811
    """What a caller does to one of them, growing it and storing it among others, is as with torch.empty's."""
    made = made_of(native, kinds, sizes)
    assert all(t.untyped_storage().nbytes() == t.numel() * t.element_size() and t.storage_offset() == 0 for t in made)
    if "l" in kinds:
        i = kinds.index("l")
        assert saved_bytes(made[i]) == saved_bytes(torch.empty(sizes[i], dtype=torch.int64).copy_(made[i]))
    for i, grown in enumerate(made):
        before = [t.clone() for t in made]
        grown.resize_(sizes[i] + 300).fill_(101)
        assert torch.equal(grown, torch.full_like(grown, 101))
        assert all(torch.equal(t, was) for j, (t, was) in enumerate(zip(made, before)) if j != i)
    made = made_of(native, kinds, sizes)
    for i in (i for i, n in enumerate(sizes) if n == 0):
        before = [t.clone() for t in made]
        torch.full((300,), 102, dtype=made[i].dtype, out=made[i])
        assert made[i].tolist() == [102] * 300
        assert all(torch.equal(t, was) for j, (t, was) in enumerate(zip(made, before)) if j != i)


@pytest.mark.parametrize("size", [-1, 1 << 62, (1 << 63) - 1])
def test_sizes_that_are_refused(native, size):  # noqa: F811
    for sizes in ((size, 3), (3, size)):
        with pytest.raises(RuntimeError):
            native.empties(torch.zeros(1), "lb" if sizes[0] == size else "bl", *sizes)


@pytest.mark.gpu
def test_one_that_is_kept_keeps_itself(native):  # noqa: F811
    like = torch.zeros(1, device="cuda")
    before = torch.cuda.memory_allocated()
    made = native.empties(like, "iiiliiibb", 5, 5, 4, 3, 100, 100, 0, 512, 40000)
    assert [t.device for t in made] == [like.device] * 9 and made[6].data_ptr() == 0
    assert torch.cuda.memory_allocated() - before == 7 * 512 + 40448
    counts = made[3]
    del made
    assert torch.cuda.memory_allocated() - before == 512
    counts.resize_(65).fill_(3)
    assert counts.tolist() == [3] * 65 and torch.cuda.memory_allocated() - before == 1024
    side = torch.cuda.Stream()                                      # the allocator knows it, and holds it back for another stream's use
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        twice = counts * 2
        counts.record_stream(side)
    del counts
    torch.cuda.current_stream().wait_stream(side)
    assert twice.tolist() == [6] * 65


def test_a_dispatch_mode_sees_every_one(native):  # noqa: F811
    from torch.utils._python_dispatch import TorchDispatchMode
    seen = []

    class Mode(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))

    like = torch.zeros(1)
    with Mode():
        made = native.empties(like, "iiil", 2, 2, 1, 3)
    assert len(seen) == 4 and storages(made) == 4


def test_transforms_and_traces_allocate_for_themselves(native):  # noqa: F811
    like, kinds, sizes = torch.zeros(1), "iiflb", (4, 5, 6, 7, 8)
    seen = {}

    def within(name, wrapped):
        made = native.empties(like, kinds, *sizes)
        seen[name] = [wrapped(t) for t in made], [t.dtype for t in made], [tuple(t.shape) for t in made]
        return made

    def graded(x):
        made = within("grad", torch._C._functorch.is_gradtrackingtensor)
        made[2].fill_(2.0)
        return (x * made[2]).sum()

    assert torch.equal(torch.func.grad(graded)(torch.ones(6)), torch.full((6,), 2.0))
    torch.vmap(lambda x: x + within("vmap", lambda t: not torch._C._functorch.is_batchedtensor(t))[2].zero_())(torch.ones(3, 6))
    torch.func.functionalize(lambda x: x + within("functionalize", torch._is_functional_tensor)[2].zero_())(torch.ones(6))
    traced = torch.jit.trace(lambda x: x + within("trace", lambda t: True)[2].zero_(), torch.ones(6), check_trace=False)
    assert str(traced.graph).count("aten::empty") >= 1 and torch.equal(traced(torch.ones(6)), torch.ones(6))
    assert set(seen) == {"grad", "vmap", "functionalize", "trace"}
    for ok, types, shapes in seen.values():
        assert all(ok) and types == [KINDS[k] for k in kinds] and shapes == [(n,) for n in sizes]
    before = torch.are_deterministic_algorithms_enabled()
    try:
        torch.use_deterministic_algorithms(True)
        made = native.empties(like, kinds, *sizes)
    finally:
        torch.use_deterministic_algorithms(before)
    assert storages(made) == 5 and int(made[0][0]) == torch.iinfo(torch.int32).max
    with torch.inference_mode():
        made = made_of(native, kinds, sizes)
        assert storages(made) == 5 and all(t.is_inference() for t in made)
    made = made_of(native, kinds, sizes)
    assert storages(made) == 5 and not any(t.is_inference() for t in made)
