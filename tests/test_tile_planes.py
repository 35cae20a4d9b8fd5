"""LDS planes copied straight from global memory, on the host: every value that
the stencils of a tile read is staged, from its own site and component, for every
tile that the fused stress and LB and the Q update run on (the wide ones too)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("planes") / "tile_planes")
    subprocess.check_call([HIPCC, "-O1", "-std=c++17", os.path.join(HERE, "hostcheck", "tile_planes.cpp"), "-o", exe],
                          stderr=subprocess.DEVNULL)

    def run(drop):
        out = subprocess.run([exe, str(drop)], capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]

    return run


def test_stencils_read_what_was_staged(rows):
    assert rows(0) == [(0, 0)] * 8


def test_a_planted_mistake_shows(rows):
    assert any(wrong > 0 for wrong, _ in rows(1)) and all(wrong > 0 for wrong, _ in rows(2))
