"""CPU: the package imports where torch lacks the functions behind its stream
handle (a torch built without a GPU), and takes the handle from torch.cuda there."""
import subprocess
import sys

CODE = """
import torch
for name in ("_cuda_getDevice", "_cuda_getCurrentRawStream"):
    if hasattr(torch._C, name):
        delattr(torch._C, name)
import paper_2603_15447_amd as bz
class Stream:
    cuda_stream = 1234
torch.cuda.current_stream = Stream
assert bz._stream() == 1234
"""


def test_import_without_raw_streams():
    subprocess.run([sys.executable, "-c", CODE], check=True, timeout=300)
