"""The tile shapes a configuration is planned with, seen in the workspace they
need (host only)."""
import pytest

import workloads as W
from helpers import _print_case


def _bytes(nx, ny, nz, q=19):
    import paper_1901_09745_amd.psclbm as P
    lat = W.LatticeSpec(q=q, nx=nx, ny=ny, nz=nz, tau=0.7)
    return P.psclbm_workspace_bytes(P.make_config(lat, "fp64", 5000, 4.0, 64, 16))


@pytest.mark.parametrize("width", [64, 128, 256])
def test_tile_x_forces_row_tiles(width, monkeypatch):
    """PSCLBM_TILE_X gives row tiles of that width also where flat tiles, with
    their longer lists, are the default: one list of 64 ids, two counts and a
    mass partial a tile more or less, to the 256-byte alignment of each array."""
    nx, ny, nz = 80, 40, 30
    _print_case(test="PSCLBM_TILE_X", width=width)
    monkeypatch.delenv("PSCLBM_TILE_X", raising=False)
    flat = _bytes(nx, ny, nz)
    monkeypatch.setenv("PSCLBM_TILE_X", str(width))
    rows = _bytes(nx, ny, nz)
    tiles = -(-nx // width) * -(-ny // (256 // width)) * nz
    full = _bytes(64 * -(-nx // 64), ny, nz)  # whole segments: row tiles in any case
    full_tiles = -(-(64 * -(-nx // 64)) // width) * -(-ny // (256 // width)) * nz
    a_tile = 4 * 64 + 2 * 4 + 8
    cells = (64 * -(-nx // 64) - nx) * ny * nz
    bins = 8 * 8 * 3 * 32 + 4 * 3  # records and counts of a DEM bin
    nbins = lambda x: (x // 9) * (ny // 9) * (nz // 9)  # noqa: E731
    want = full - cells * 19 * 8 - (full_tiles - tiles) * a_tile \
        - (nbins(128) - nbins(nx)) * bins
    assert flat != rows
    assert abs(rows - want) <= 6 * 256


# nx, ny, nz, particles, row tiles chosen: lists that may be longer than LDS holds
# (96 entries of 64) on lattices within the last-level cache, or of 2^18 cells (2D)
@pytest.mark.parametrize("nx, ny, nz, n, rows", [
    (70, 3744, 1, 500, True), (70, 3745, 1, 500, False), (70, 200, 1, 96, False),
    (190, 96, 96, 5000, True), (100, 50, 50, 500, True), (90, 60, 60, 500, True),
    (89, 60, 60, 500, False), (80, 60, 60, 500, False), (10, 50, 50, 500, False),
    (190, 120, 120, 5000, False), (190, 96, 96, 96, False), (128, 60, 60, 500, True)])
def test_row_tiles_of_full_rows_with_long_lists(nx, ny, nz, n, rows, monkeypatch):
    import paper_1901_09745_amd.psclbm as P
    _print_case(test="row tiles of full rows", nx=nx, n=n)
    lat = W.LatticeSpec(q=9 if nz == 1 else 19, nx=nx, ny=ny, nz=nz, tau=0.7)
    cfg = P.make_config(lat, "fp64", n, 4.0, 64, 16)
    monkeypatch.delenv("PSCLBM_TILE_X", raising=False)
    chosen = P.psclbm_workspace_bytes(cfg)
    width = 64 if nz == 1 else min((256, 128, 64), key=lambda t: -(-nx // t) * t)
    monkeypatch.setenv("PSCLBM_TILE_X", str(width))
    assert (chosen == P.psclbm_workspace_bytes(cfg)) == rows
