"""Host build of the host layer (csrc/host.hip) against recording stand-ins for
the runtime and the kernels' launchers: the tile tables of every kind of search
lie inside the workspace and apart from the moments, the grids and the spectra,
over harmonics, curves per wave (half the buffers' capacity among them: there
the next wave is spread on a second stream), grid periods and both strip sizes."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "host", "workspace_test.hip")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC),
                    reason="hipcc not available")
def test_tile_tables_stay_in_their_place(tmp_path):
    exe = str(tmp_path / "workspace_test")
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O2", "-std=c++17", SRC, "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and "ALL OK" in out.stdout, out.stdout + out.stderr
