"""Row sums at the last entries a model may hold (fewer than 2^31): the device
functions, built for the host, must not read a position past them or before
them, and kernels whose positions run further ahead must not be chosen
(entry_positions.cpp)."""
import subprocess
from pathlib import Path

from paper_2511_13894_amd import build

HERE = Path(__file__).resolve().parent


def test_row_sums_at_the_last_entries(tmp_path):
    exe = tmp_path / "entry_positions"
    # -fwrapv: a position that leaves the range wraps, as it does on the device
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-fwrapv", "-std=c++17", f"-I{build.ROOT / 'include'}",
                    f"-I{build.CSRC}", str(HERE / "entry_positions.cpp"), "-o", str(exe), "-x", "none", str(build.OUT), f"-Wl,-rpath,{build.PKG}", "-lpthread"], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, (run.returncode, run.stdout[-2000:], run.stderr[-2000:])
