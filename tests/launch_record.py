"""Host runtime sources linked with kernel launchers that only record their calls:
which launches a call enqueues, on the CPU (no GPU is touched)."""
import os
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parents[1]
CSRC = ROOT / "paper_2605_17869_amd" / "csrc"

FRAME = r"""
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>
#include "sift_launch.h"
#include "sift_match.h"
#include "sift_verify.h"
static int fails = 0;
#define CHECK(c) do { if (!(c)) { std::printf("FAIL %s line %d\n", #c, __LINE__); ++fails; } } while (0)
// device addresses that nothing dereferences
template <typename T> T* fake(uintptr_t at) { return reinterpret_cast<T*>(at << 20); }
"""


def run(tmp_path, sources, driver):
    """Compile `sources` of the runtime and `driver` (stubs and a main that returns
    the failed checks) for the host and run them."""
    root = os.environ.get("ROCM_PATH", "/opt/rocm")
    hipcc = str(Path(root) / "bin" / "hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    main = tmp_path / "driver.cpp"
    main.write_text(FRAME + driver)
    procs, objs = [], []
    for src in [*(CSRC / s for s in sources), main]:
        obj = tmp_path / (src.name + ".o")
        cmd = [hipcc, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O1",
               "-I", str(CSRC), "-I", str(ROOT / "include"), "-w", "-c", str(src), "-o", str(obj)]
        procs.append(subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT))
        objs.append(obj)
    for p in procs:
        out, _ = p.communicate()
        assert p.returncode == 0, out.decode(errors="replace")[-3000:]
    exe = tmp_path / "driver"
    link = subprocess.run([hipcc, "-o", str(exe), *map(str, objs)], capture_output=True, text=True)
    assert link.returncode == 0, link.stdout[-2000:] + link.stderr[-2000:]
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120,
                         env=dict(os.environ, HIP_VISIBLE_DEVICES=""))
    assert res.returncode == 0, res.stdout[-3000:] + res.stderr[-3000:]
