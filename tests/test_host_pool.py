"""The host threads of batched rounds (csrc/host_pool.h) on the CPU, under ThreadSanitizer and under
AddressSanitizer + UndefinedBehaviorSanitizer: phases take every item once while the team shrinks, calls
that run side by side share a bounded number of spinning threads, an exception or a thread that cannot be
started leaves nothing running."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("sanitizer", ["thread", "address,undefined"])
def test_team_phases(sanitizer, tmp_path):
    exe = str(tmp_path / "host_pool")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", f"-fsanitize={sanitizer}", "-fno-sanitize-recover=all",
                        os.path.join(ROOT, "tests", "host_pool_main.cpp"), "-o", exe],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout == "ok\n", f"sanitizer report or crash:\n{r.stderr[-3000:]}"
