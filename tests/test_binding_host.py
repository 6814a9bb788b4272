"""The Python binding where no GPU is needed: what it imports and when, and the
checks and results of its tensor helpers."""
import os
import subprocess
import sys

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
