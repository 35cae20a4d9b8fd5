"""Chunked staging of the LDS tiles (ChunkPlan in tiles.h), on the host: every
dword of a staged plane is copied exactly once, from its own lattice site."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.parametrize("turn", [0, 1, 3])
def test_every_point_is_copied_once(tmp_path, turn):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "tile_chunks")
    subprocess.check_call([HIPCC, "-O1", "-std=c++17", os.path.join(HERE, "hostcheck", "tile_chunks.cpp"), "-o", exe],
                          stderr=subprocess.DEVNULL)
    out = subprocess.run([exe, str(turn)], capture_output=True, text=True, check=True).stdout
    assert out.split("\n")[:-1] == ["0 0"] * 6
