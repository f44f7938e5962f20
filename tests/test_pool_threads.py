"""The device memory cache used by two threads, on the host: pool_two_threads.cpp
compiles the library's pool.cpp against counted stand-ins for the driver's calls."""
from __future__ import annotations

import os
import subprocess

from paper_1506_05083_amd import build


def test_blocks_on_their_way_to_being_available(tmp_path):
    """Giving everything back, running out of memory and releasing, each in a second
    thread while the first waits for the device."""
    src = os.path.join(os.path.dirname(__file__), "pool_two_threads.cpp")
    exe = str(tmp_path / "pool")
    flags = [f for f in build.FLAGS if f != "-O3"]
    subprocess.run([build.HIPCC, *flags, "--offload-host-only", "-O1", "-x", "hip", src, "-o", exe, "-lpthread"],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    print(r.stdout)
    assert r.returncode == 0, r.stdout
