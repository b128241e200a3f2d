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
