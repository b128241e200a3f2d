"""The buffers of a small token filter, which share one allocation (csrc/marshal.cpp), and those that do not."""
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


def test_small_ones_share(native):  # noqa: F811
    for kinds, sizes in (("iiiliiibb", (5, 5, 4, 3, 100, 100, 100, 512, 40000)), ("iiil", (2, 2, 1, 3)), ("iiilii", (2, 2, 1, 3, 0, 0)),
                         ("bilf", ((1 << 20) - 1536, 128, 64, 128))):
        made = made_of(native, kinds, sizes)
        assert storages(made) == 1
        first = made[0].untyped_storage().data_ptr()
        assert all((t.data_ptr() - first) % 512 == 0 for t in made if t.numel())
        kept, value = made[-1], made[-1].clone()
        del made                                                    # the storage lives as long as the last of them
        torch.empty(1 << 18).fill_(7.0)
        assert torch.equal(kept, value)


def test_others_do_not(native):  # noqa: F811
    from torch.utils._python_dispatch import TorchDispatchMode
    assert storages(made_of(native, "ff", (100, 100))) == 2
    assert storages(made_of(native, "bilf", ((1 << 20) - 1535, 128, 64, 128))) == 4
    assert storages(made_of(native, "iiii", (1 << 18, 1, 1, 1))) == 4

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
        assert storages(made_of(native, kinds, sizes)) == 1
    assert storages(made_of(native, kinds, sizes)) == 1
