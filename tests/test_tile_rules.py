"""The rules that choose a form of a step by the size of the lattice (tiles.h),
on the host: lattices on which one form was measured the faster by 2% or more on
256 CUs get it."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("rules") / "tile_rules")
    subprocess.check_call([HIPCC, "-O1", "-std=c++17", os.path.join(HERE, "hostcheck", "tile_rules.cpp"), "-o", exe],
                          stderr=subprocess.DEVNULL)

    def run(name, prec, shapes, cus=256):
        out = subprocess.run([exe, name, str(prec), str(cus), *[str(n) for s in shapes for n in s]],
                             capture_output=True, text=True, check=True).stdout
        return [int(v) for v in out.split()]

    return run


FUSED = {32: [(128, 128, 128), (128, 128, 64), (96, 96, 96), (96, 128, 96), (120, 120, 120), (160, 160, 160),
              (192, 192, 192), (200, 200, 200), (64, 64, 256), (61, 159, 127), (175, 149, 62), (170, 90, 111),
              (54, 165, 113), (171, 153, 63)],
         64: [(128, 128, 128), (128, 128, 64), (96, 96, 96), (96, 90, 48), (120, 120, 120), (144, 144, 144),
              (160, 160, 160), (192, 192, 192), (200, 200, 200), (64, 64, 256), (140, 100, 100), (130, 130, 100),
              (300, 50, 120), (64, 40, 160), (512, 4, 512), (81, 58, 91), (165, 122, 160)]}
SWEEPS = {32: [(112, 112, 112), (300, 50, 120), (150, 60, 120), (140, 100, 100), (130, 130, 100), (100, 100, 100),
               (72, 96, 120)],
          64: [(100, 100, 100), (72, 96, 120)]}


@pytest.mark.parametrize("coupling", ["force", "split"])
@pytest.mark.parametrize("prec", [32, 64])
def test_fused_passes_where_they_were_measured_faster(rule, prec, coupling):
    name = "pass_chunk_" + coupling
    for s, tz in zip(FUSED[prec], rule(name, prec, FUSED[prec])):
        assert 6 <= tz <= s[2], s
    assert not any(rule(name, prec, SWEEPS[prec]))
    small = [(4, 4, 4), (32, 8, 5), (4, 4, 4096), (4096, 4, 4), (32, 32, 6), (1024, 1024, 4)]
    assert all(tz == 0 or 6 <= tz <= s[2] for s, tz in zip(small, rule(name, prec, small)))
    assert not any(rule(name, prec, FUSED[prec], cus=0))  # no device to ask


# the fused stress and LB, chunks of 8, 16 and 32 planes
WIDE = {32: {8: [(128, 128, 128), (192, 64, 130), (64, 64, 400), (150, 150, 150), (120, 120, 120), (100, 128, 130),
                 (64, 16, 1700)],
             16: [(128, 128, 128), (176, 176, 176), (192, 192, 64), (120, 120, 120), (150, 150, 150), (200, 200, 200),
                  (100, 200, 200), (61, 159, 180), (58, 200, 200)],
             32: [(176, 176, 176), (192, 192, 64), (150, 150, 150), (200, 200, 200), (120, 116, 160)]},
        64: {tz: [(128, 128, 128), (128, 128, 100), (192, 64, 130), (512, 6, 512)] for tz in (8, 16, 32)}}
NARROW = {32: {8: [(64, 64, 64), (128, 64, 64), (128, 128, 80), (192, 192, 40)],
               16: [(64, 64, 64), (512, 6, 512), (512, 7, 512), (192, 64, 130), (192, 192, 48), (128, 128, 100)],
               32: [(160, 160, 160), (128, 128, 128), (512, 8, 512), (192, 64, 130)]},
          64: {tz: [(64, 64, 64), (512, 11, 256), (100, 200, 200)] for tz in (8, 16, 32)}}


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("tz", [8, 16, 32])
def test_wide_tiles_where_they_were_measured_faster(rule, prec, tz):
    assert all(rule(f"wide_{tz}", prec, WIDE[prec][tz]))
    assert not any(rule(f"wide_{tz}", prec, NARROW[prec][tz]))


TILES = {"update": {32: (16, 12), 64: (16, 12)}, "stress": {32: (32, 8), 64: (16, 12)}, "wide": {32: (64, 5), 64: (32, 4)}}


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("tile", list(TILES))
@pytest.mark.parametrize("per_cu", [1, 2, 4, 8])
def test_chunks_that_fill_the_device(rule, prec, tile, per_cu):
    """The shallowest chunk with which a kernel's own tiles take no more than the slots."""
    tx, ty = TILES[tile][prec]
    shapes = [(128, 64, 128), (128, 128, 128), (192, 192, 192), (130, 130, 100), (96, 96, 96), (512, 6, 512), (61, 159, 180),
              (4, 4, 4), (600, 600, 8)]
    slots = 256 * per_cu
    for (nx, ny, nz), tz in zip(shapes, rule(f"fill_{tile}_{per_cu}", prec, shapes)):
        cols = -(-nx // tx) * -(-ny // ty)
        assert (tz == 0) == (cols > slots)
        if tz:
            assert 1 <= tz <= nz and cols * -(-nz // tz) <= slots
            assert tz == 1 or cols * -(-nz // (tz - 1)) > slots
