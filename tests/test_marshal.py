"""Addresses of tensor arguments by the native module and by the Python function that serves everything else: same addresses, same refusals."""
import pytest
import torch

from paper_2605_08151_amd import binding


class _OnDevice:
    """What binding asks of a tensor, without a GPU."""
    def __init__(self, t, is_cuda=True):
        self.t, self.is_cuda, self.dtype = t, is_cuda, t.dtype
    is_contiguous = lambda self: self.t.is_contiguous()     # noqa: E731
    data_ptr = lambda self: self.t.data_ptr()               # noqa: E731


def test_refusals_and_none_without_a_gpu():
    t = torch.zeros(4, 6)
    assert binding._ptr(None) is None and binding._ptr(None, torch.int32) is None
    for bad in (t, torch.nn.Parameter(t), _OnDevice(t, False), _OnDevice(t.t())):
        with pytest.raises(AssertionError, match="device-resident contiguous"):
            binding._ptr(bad, torch.float32)
    with pytest.raises(AssertionError):
        binding._ptr(_OnDevice(t), torch.int32)
    assert binding._ptr(_OnDevice(t), torch.float32) == t.data_ptr()
    with pytest.raises(AttributeError):
        binding._ptr(5)
    with pytest.raises(TypeError):
        binding._ptr()


@pytest.mark.gpu
def test_addresses_and_streams():
    t = torch.zeros(4, 6, device="cuda")
    for x in (t, t[2:], t[4:], torch.nn.Parameter(t), t.view(24)[5:]):
        assert binding._ptr(x) == binding._ptr(x, torch.float32) == x.data_ptr() == binding._ptr_any(x, torch.float32)
    assert binding._ptr(torch.empty(0, device="cuda"), torch.float32) == 0
    for bad, dtype in ((t.t(), torch.float32), (t[:, 1:], None), (t.cpu(), torch.float32), (t, torch.int32), (t, torch.bfloat16)):
        with pytest.raises(AssertionError):
            binding._ptr(bad, dtype)
    assert binding._stream() == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert binding._stream() == side.cuda_stream
    assert binding._stream() != side.cuda_stream


def test_the_import_says_why_the_module_is_missing(tmp_path):
    """Not built, or built and not loadable (against another torch, say): two errors."""
    import os
    import shutil
    import subprocess
    import sys
    package = tmp_path / "pkg"
    package.mkdir()
    (package / "__init__.py").write_text("")
    shutil.copy(binding.__file__, package / "binding.py")

    def error():
        done = subprocess.run([sys.executable, "-c", "import pkg.binding"], cwd=tmp_path, capture_output=True, text=True, env=dict(os.environ, PYTHONPATH=str(tmp_path)))
        assert done.returncode != 0
        return done.stderr.strip().splitlines()[-1]

    assert "_marshal.so is not built" in error()
    (package / "_marshal.so").write_bytes(b"\x7fELF, but no library")
    last = error()
    assert "does not load" in last and torch.__version__ in last and "not built" not in last
