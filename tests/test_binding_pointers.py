"""The binding's native argument checks take and refuse what the Python rules do, with the same addresses and errors."""
import pytest
import torch

from paper_2605_16154_amd import binding


class Marked(torch.Tensor):
    pass


def outcome(check, t, dtype):
    try:
        return check(t, dtype)
    except Exception as e:
        return type(e), str(e)


def forms(device):
    x = torch.arange(24, dtype=torch.float32, device=device).view(4, 6)
    return [None, 5, x, x.t(), x[1:], x[:, 1:], x[0], x[:0], x[:1].t(), x.double(), x.to(torch.uint8), torch.nn.Parameter(x),
            x.clone().as_subclass(Marked), x.to_sparse(), x.cpu().numpy(), torch.empty(3, 2, device="meta"), torch.tensor(1.0, device=device)]


def compare(device):
    binding.lib()
    native = lambda t, dtype: binding._ptrs(((dtype, "x"),), t)[0]
    python = lambda t, dtype: binding._ptr(t, dtype, "x")
    assert binding._ptrs.__name__ == "pointers"
    for t in forms(device):
        for dtype in (None, torch.float32, torch.float64, torch.uint8):
            assert outcome(native, t, dtype) == outcome(python, t, dtype)


def test_native_checks_on_host_tensors():
    compare("cpu")
    with pytest.raises(TypeError):
        binding._ptrs(((None, "x"),))                        # a rule without a tensor
    with pytest.raises(TypeError):
        binding._ptrs((None,), None)


@pytest.mark.gpu
def test_native_checks_on_device_tensors():
    compare("cuda")
    x, y = torch.zeros(3, device="cuda"), torch.zeros(2, dtype=torch.int32, device="cuda")
    rules = ((torch.float32, "a"), (None, "b"), (torch.int32, "c"))
    assert binding._ptrs(rules, x, None, y) == (x.data_ptr(), None, y.data_ptr())
    with pytest.raises(binding.PcmError, match="c must be torch.int32, got torch.float32"):
        binding._ptrs(rules, x, y, x)
    seen = []
    torch.func.vmap(lambda row: seen.append(outcome(lambda t, d: binding._ptrs(((d, "x"),), t)[0], row, None)) or row)(torch.zeros(2, 3, device="cuda"))
    assert seen[0][0] is RuntimeError                        # no address inside vmap
