"""The binding imports, and its host-only calls work, on a torch without GPU support."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_binding_imports_without_gpu_support_in_torch():
    # such a torch has none of the CUDA/HIP entries of torch._C
    code = ("import torch\n"
            "for n in [n for n in dir(torch._C) if n.startswith('_cuda_getCurrent')]: delattr(torch._C, n)\n"
            "from paper_2607_16213_amd import selkv as S\n"
            "p = S.params(seq_len=8192)\n"
            "assert S.budget(p) == (2048, 16, 2032) and S.workspace_bytes(p, S.CALL_SCORE) > 0\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
