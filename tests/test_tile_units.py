"""The ragged batch's default tile follows the device's compute units (an
MI355X can be partitioned: 256 units, or 32 in eight parts)."""

import pytest


@pytest.mark.parametrize("units", [32, 128, 256])
def test_tile_gives_every_resident_block_one(monkeypatch, units):
    from paper_2309_04909_amd import batch as bt
    from paper_2309_04909_amd import bicop as B
    monkeypatch.setattr(B, "SCHEDULES", {})
    resident = 8 * units
    for elements, tile in ((1, 256), (resident * 512 - 1, 256), (resident * 512, 512), (resident * 1024 - 1, 512),
                           (resident * 1024, 1024), (1 << 30, 1024)):
        assert bt.default_tile(elements, units) == tile
