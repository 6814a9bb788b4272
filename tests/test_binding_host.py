"""The Python binding where no GPU is needed: what it imports and when, and the
checks and results of its tensor helpers."""
import os
import subprocess
import sys

import pytest
import torch

import paper_2606_21023_amd as heal

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# (names of the modules, not their files, are refused, so that nothing of an
# installed torch is found)
NO_TORCH = """
import sys
class Refuse:
    def find_spec(self, name, path=None, target=None):
        if name == "torch" or name.startswith("torch."):
            raise ImportError("no torch here")
sys.meta_path.insert(0, Refuse())
"""


def _python(code):
    return subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)


def test_package_and_build_import_without_torch():
    """The C library is built and its host functions are called without PyTorch;
    importing the package does not pull it in either."""
    r = _python(NO_TORCH + "import paper_2606_21023_amd as heal\n"
                "from paper_2606_21023_amd import build\nprint(build.source_hash())\n"
                "import os\n"
                "if os.path.exists(build.LIBRARY): print(heal.heal_packed_size(33, 17, 1))\n")
    assert r.returncode == 0, r.stderr
    r = _python("import sys, paper_2606_21023_amd\nassert 'torch' not in sys.modules\n")
    assert r.returncode == 0, r.stderr


def test_stream_without_raw_stream_accessors():
    """A torch without the raw accessors is asked for its Stream object."""
    r = _python("import torch, types\n"
                "import paper_2606_21023_amd as heal\n"
                "for n in ('_cuda_getCurrentRawStream', '_cuda_getDevice'):\n"
                "    if hasattr(torch._C, n): delattr(torch._C, n)\n"
                "torch.cuda.current_stream = lambda: types.SimpleNamespace(cuda_stream=77)\n"
                "assert heal._stream() == 77 and heal._stream() == 77\n")
    assert r.returncode == 0, r.stderr


class OnDevice(torch.Tensor):
    """A CPU tensor that the checks take for one on the device."""
    is_cuda = True


def _dev(*shape):
    return torch.zeros(shape).as_subclass(OnDevice)


def test_a_tensor_without_dimensions_is_refused():
    """A 0-dimensional tensor has no last dimension to be contiguous in."""
    with pytest.raises(IndexError):
        heal._tensor(_dev(), "x", torch.float32)
    with pytest.raises(heal.HealError):
        heal._tensor(_dev(), "x", torch.float32, 2)
    assert heal._tensor(_dev(0), "x", torch.float32)[0] == (0,)
    assert heal._tensor(_dev(3, 1).t(), "x", torch.float32, 2)[0] == (1, 3)
    with pytest.raises(heal.HealError):
        heal._tensor(_dev(3, 2).t(), "x", torch.float32, 2)


def test_results_are_plain_tensors():
    """A result does not take on the operand's subclass."""
    C, stride = heal._output(None, _dev(2, 3), (2, 5))
    assert type(C) is torch.Tensor and C.dtype is torch.float32 and C.shape == (2, 5)
    assert stride == (5, 1)


def test_a_scale_that_is_no_number_is_a_type_error():
    with pytest.raises(TypeError):
        heal.heal_gemm_f32_strided_batched(_dev(1, 2, 4), _dev(1, 4, 2), alpha="x", out=_dev(1, 2, 2))
    with pytest.raises(TypeError):
        heal.heal_scores_i16(_dev(1, 2, 8).to(torch.int16), _dev(1, 2, 8).to(torch.int16), _dev(1),
                             _dev(1), alpha="x", out=_dev(1, 2, 2))
