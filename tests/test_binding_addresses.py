"""What the binding takes for an address: tensors, arrays and its own Address type, never a plain integer."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2512_19849_amd import binding, runner  # noqa: E402


@pytest.mark.parametrize("x", [0, 4096, np.int64(4096), True, 1.5, "x"])
def test_numbers_are_not_addresses(x):
    with pytest.raises((AttributeError, TypeError)):
        binding._ptr(x)


def test_misplaced_size_is_refused_before_the_library_sees_it(monkeypatch):
    class Untouched:
        def __getattr__(self, name):
            return lambda *a: pytest.fail(f"{name} was called")
    monkeypatch.setattr(binding, "_lib", Untouched())
    t = torch.zeros(8, dtype=torch.int32)
    with pytest.raises((AttributeError, TypeError)):
        binding.ep_combine(1, t, t, 8, t, 8, t, stream=0)  # d_dst_row and T changed places
    with pytest.raises((AttributeError, TypeError)):
        binding.ep_recv_wait(1, 0, -1, 64, stream=0)


def test_tensors_arrays_and_addresses():
    t, a = torch.zeros(8, dtype=torch.int32), np.zeros(8, np.int32)
    assert binding._ptr(None) is None
    assert binding._ptr(t) == t.data_ptr() and binding._ptr(a) == a.ctypes.data
    assert binding._ptr(binding.Address(64)) == 64
    with pytest.raises(ValueError):
        binding._ptr(torch.zeros(4, 4).t())


@pytest.mark.parametrize("src", [0, 2, -1, np.int32(2), np.int64(1), torch.tensor(2)])
def test_row_of_a_table_by_any_index(src):
    for t in (torch.zeros(3, 5, 2, dtype=torch.int32), torch.zeros(3, 7), torch.zeros(5, 3, 4).transpose(0, 1).contiguous()):
        assert binding._ptr(runner._row(t, src)) == t[src].data_ptr()
    wide = torch.zeros(3, 10)[:, :5]  # rows are contiguous, the table is not
    assert binding._ptr(runner._row(wide, src)) == wide[src].data_ptr()


def test_row_out_of_range_or_not_contiguous_is_refused():
    with pytest.raises(IndexError):
        runner._row(torch.zeros(3, 5), 3)
    with pytest.raises(ValueError):
        binding._ptr(runner._row(torch.zeros(3, 5, 2).transpose(1, 2), 1))
