"""Allocations of the push model (slab_pieces.cpp): small ones where each of its
arrays is small, one where an array is large by itself."""
import subprocess
from pathlib import Path

from paper_2511_13894_amd import build

HERE = Path(__file__).resolve().parent


def test_allocations_of_the_push_model(tmp_path):
    exe = tmp_path / "slab_pieces"
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", f"-I{build.ROOT / 'include'}", f"-I{build.CSRC}",
                    str(HERE / "slab_pieces.cpp"), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout
