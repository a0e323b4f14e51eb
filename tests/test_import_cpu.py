"""The package imports on a torch that was built without a GPU runtime."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_import_without_the_raw_stream_call():
    code = ("import torch\n"
            "del torch._C._cuda_getCurrentRawStream\n"
            "import paper_2202_12756_amd.fft as fft\n"
            "assert callable(fft._raw_stream) and fft.Plan\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
