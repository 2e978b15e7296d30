"""check_tensor accepts and refuses the same arguments by its short form (plain
tensors that pass) as by the list of conditions behind it."""
import pytest
import torch

import paper_2402_03074_amd as H


class Sub(torch.Tensor):
    pass


def _wrap(t, kind):
    if kind == "parameter":
        return torch.nn.Parameter(t)
    return t.as_subclass(Sub) if kind == "subclass" else t


@pytest.mark.parametrize("kind", ["plain", "parameter", "subclass"])
def test_same_verdict_for_every_kind_of_tensor(kind):
    t = torch.zeros(4, 6, dtype=torch.float64)
    ok = [(t, "float64", 24), (t, "float64", 0), (t.to(torch.float32), "float32", 24),
          (t[1:], "float64", 18)]
    if kind != "parameter":  # a parameter is a floating-point tensor
        ok.append((t.to(torch.int32), "int32", 24))
    bad = [(t, "float64", 25, "elements"), (t, "float32", 24, "dtype"),
           (t.to(torch.float32), "float64", 24, "dtype"), (t.t(), "float64", 24, "contiguous"),
           (t[:, ::2], "float64", 12, "contiguous"), (t.to(torch.float16), "float64", 1, "dtype")]
    for x, dtype, n in ok:
        H.check_tensor(_wrap(x, kind), "w", "x", dtype, n, 0, require_cuda=False)
    for x, dtype, n, why in bad:
        with pytest.raises(H.HwenouError, match=why) as e:
            H.check_tensor(_wrap(x, kind), "w", "x", dtype, n, 0, require_cuda=False)
        assert e.value.code == H.HWENOU_EINVAL
    # a host tensor where the GPU's is needed, with and without a device index
    for device in (None, 0):
        with pytest.raises(H.HwenouError, match="not a GPU tensor"):
            H.check_tensor(_wrap(t, kind), "w", "x", "float64", 24, device)


def test_what_is_no_tensor_is_refused():
    for x in (None, 3.0, [1.0], "x"):
        with pytest.raises(H.HwenouError, match="not a tensor"):
            H.check_tensor(x, "w", "x", "float64", 1, require_cuda=False)
