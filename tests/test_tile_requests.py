"""Tile sizes past the grid: a request of any size is the whole grid's along its axis
(host-only calls, in a process of their own, since a division by zero would end it)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
from paper_2003_14061_amd import inputs, md
p = md.Params(4000, 0, inputs.box_length(4000, 0.8), 1.0, 1.0, 1.0, 2 ** (1 / 6), 0.3, 0.005,
              0, 1, 0, 0, 1, 256, 0)
ctx = md.md_init(p)
def shape(**kw):
    md.md_set_tuning(ctx, **kw)
    t = md.md_get_tuning(ctx)
    return t["tile_cells"], t["tile_y"], t["tile_z"]
nc = md.md_geometry(ctx).nc
for axis in ("tile_cells", "tile_y", "tile_z"):
    one = dict(tile_cells=1, tile_y=1, tile_z=1)
    assert shape(**{**one, axis: big}) == shape(**{**one, axis: nc}), axis
"""


@pytest.mark.parametrize("big", [12, 13, 1 << 20, (1 << 31) - 12, (1 << 31) - 1])
def test_a_request_past_the_grid(big):
    r = subprocess.run([sys.executable, "-c", f"big = {big}\n" + CODE], cwd=ROOT,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stderr)


def test_at_most_64_home_rows():
    from paper_2003_14061_amd import inputs, md

    # 18 and 70 cells per side
    for n, nc in ((13000, 18), (800000, 70)):
        p = md.Params(n, 0, inputs.box_length(n, 0.8), 1.0, 1.0, 1.0, 2 ** (1 / 6), 0.3, 0.005,
                      0, 1, 0, 0, 1, 256, 0)
        ctx = md.md_init(p)
        got_nc = md.md_geometry(ctx).nc
        assert abs(got_nc - nc) <= 1
        for x in (0, 1, 3):
            for y in (0, 1, 4, 8, 9, 16, 17, 64, 65, 1000):
                for z in (0, 1, 4, 8, 9, 16, 17, 64, 65, 1000):
                    md.md_set_tuning(ctx, tile_cells=x, tile_y=y, tile_z=z)
                    t = md.md_get_tuning(ctx)
                    assert 1 <= t["tile_y"] * t["tile_z"] <= 64, (x, y, z, t)
                    ways = [-(-got_nc // r) for r in (min(y, got_nc), min(z, got_nc)) if r]
                    if y and z and y * z <= 64:  # as requested, evened out
                        assert t["tile_y"] == -(-got_nc // ways[0])
                        assert t["tile_z"] == -(-got_nc // ways[1])
        md.md_destroy(ctx)
