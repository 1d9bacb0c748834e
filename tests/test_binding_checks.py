"""The one-pass operand test of the binding takes exactly the operands that
its checks one by one take (and results are laid out like a new tensor)."""
import types

import pytest
import torch

from paper_2505_08098_amd import binding

N = 6


class Sub(torch.Tensor):
    pass


def _base(shape, dtype=torch.float16):
    return torch.zeros(shape, dtype=dtype)


FORMS = {
    "one head": lambda: _base((N, 8)),
    "heads": lambda: _base((N, 2, 8)),
    "parameter": lambda: torch.nn.Parameter(_base((N, 8))),
    "view at an offset": lambda: _base((N + 1, 8))[1:],
    "transposed": lambda: _base((8, N)).t(),
    "heads transposed": lambda: _base((2, N, 8)).transpose(0, 1),
    "strided": lambda: _base((N, 16))[:, ::2],
    "expanded": lambda: _base((1, 8)).expand(N, 8),
    "other rows": lambda: _base((N + 1, 8)),
    "other d": lambda: _base((N, 16)),
    "one dimension": lambda: _base((N,)),
    "four dimensions": lambda: _base((N, 1, 2, 4)),
    "float32": lambda: _base((N, 8), torch.float32),
    "bfloat16": lambda: _base((N, 8), torch.bfloat16),
    "other device": lambda: torch.zeros((N, 8), dtype=torch.float16, device="meta"),
    "subclass": lambda: _base((N, 8)).as_subclass(Sub),
    "no tensor": lambda: [[0.0] * 8] * N,
}


def _one_by_one(plan, dtype, *ts):
    if any(not isinstance(t, torch.Tensor) for t in ts):
        return False
    return all(t.dtype == dtype and t.device == plan.device and t.is_contiguous()
               and t.dim() in (2, 3) and t.shape[0] == plan.N and t.shape == ts[0].shape
               for t in ts)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("other", ["one head", "heads"])
@pytest.mark.parametrize("place", [0, 1, 2])
def test_plain_agrees_with_the_checks(form, other, place):
    plan = types.SimpleNamespace(N=N, device=torch.device("cpu"))
    ts = [FORMS[other]() for _ in range(3)]
    ts[place] = FORMS[form]()
    # (a subclass is left to the checks one by one, which take it)
    want = _one_by_one(plan, torch.float16, *ts) and form != "subclass"
    assert binding._plain(plan, torch.float16, *ts) == want


@pytest.mark.parametrize("form", ["one head", "heads", "parameter", "view at an offset",
                                  "subclass"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_results_are_new_contiguous_tensors(form, dtype):
    t = FORMS[form]()
    out = binding._empty_like(t, dtype)
    assert type(out) is torch.Tensor and not out.requires_grad
    assert out.is_contiguous() and out.shape == t.shape and out.dtype == dtype
    assert out.device == t.device


@pytest.mark.parametrize("other_device", [False, True])
@pytest.mark.parametrize("fails", [False, True])
def test_build_leaves_the_current_device_as_it_was(monkeypatch, other_device, fails):
    """A plan build on another device than the current one leaves it current
    again, also when waiting for the current stream raises (a capture, an error
    of earlier work)."""
    current = [0 if other_device else 1]

    class Guard:
        def __init__(self, device):
            self.to = device.index

        def __enter__(self):
            self.back, current[0] = current[0], self.to

        def __exit__(self, *exc):
            current[0] = self.back

    def wait():
        assert current[0] == 1
        if fails:
            raise RuntimeError("stream is capturing")

    monkeypatch.setattr(torch.cuda, "current_device", lambda: current[0])
    monkeypatch.setattr(torch.cuda, "device", Guard)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda *a: types.SimpleNamespace(synchronize=wait))
    monkeypatch.setattr(binding, "_raw_stream", lambda index: 1234)
    before = current[0]
    built = False
    try:
        with binding._BuildOn(torch.device("cuda", 1)):
            built = current[0] == 1
    except RuntimeError:
        assert fails
    assert current[0] == before and built == (not fails)
