"""The gather around the edges of its segments, in grids of one tile, by a wave per
row and by a workgroup, with the tiles of a place shared among workgroups (which
shapes take which: tests/tile_plan_check.cpp), bit for bit against slicing; the blend of a tile tensor past the 320 MB line (four
units a thread) bit for bit against the same field blended in pairs (two units)
and one by one (at the 64 MB line, read through the caches)."""
import pytest
import torch

import oracle
from paper_2609_36757_amd import fastvr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fastvr.load()
    return torch.device("cuda:0")


# Hg, Wg, C, tile, overlap: one row is Wg * C / 8 units of 16 bytes
@pytest.mark.parametrize("Hg,Wg,C,tile,overlap", [(5, 767, 8, 64, 16), (70, 768, 8, 64, 0), (5, 769, 8, 64, 16),
                                                  (9, 11, 560, 64, 16), (33, 97, 64, 32, 31), (1, 1, 8, 1, 0),
                                                  (40, 45, 384, 32, 30), (40, 45, 40, 32, 31), (30, 30, 16, 64, 16),
                                                  (64, 100, 64, 64, 16), (13, 321, 8, 64, 16), (13, 41, 64, 40, 8)])
def test_gather_equals_slices(dev, Hg, Wg, C, tile, overlap):
    B, T = 2, 3
    print(f"\n[gpu case] gather B={B} T={T} {Hg}x{Wg} C={C} tile={tile} overlap={overlap}", flush=True)
    x = torch.randint(-30000, 30000, (B, T, Hg, Wg, C), dtype=torch.int16, device=dev).view(torch.bfloat16)
    got = fastvr.tile_gather(x, tile=tile, overlap=overlap).view(torch.int16)
    torch.cuda.synchronize()
    oy, Ly = oracle.tile_axis(Hg, tile, overlap)
    ox, Lx = oracle.tile_axis(Wg, tile, overlap)
    for ty, y in enumerate(oy):
        for tx, c in enumerate(ox):
            assert torch.equal(got[:, ty * len(ox) + tx], x.view(torch.int16)[:, :, y:y + Ly, c:c + Lx])


@pytest.mark.parametrize("update", [False, True])
def test_blend_paths_agree(dev, update):
    B, T, Hg, Wg, C = 6, 4, 70, 90, 256
    print(f"\n[gpu case] blend B={B} T={T} {Hg}x{Wg} C={C} update={update}", flush=True)
    ny, Ly = fastvr.tile_axis(Hg, 64, 16)
    nx, Lx = fastvr.tile_axis(Wg, 64, 16)
    tiles = torch.randn((B, ny * nx, T, Ly, Lx, C), device=dev)
    assert tiles.numel() * 4 > 320 << 20 > tiles[:2].numel() * 4 > 64 << 20 >= tiles[0].numel() * 4
    z = torch.randn((B, T, Hg, Wg, C), device=dev).to(torch.bfloat16) if update else None
    whole = fastvr.tile_blend(tiles, Hg, Wg, z_lq=z, sigma=0.4)
    for n in (1, 2):
        for b in range(0, B, n):
            part = fastvr.tile_blend(tiles[b:b + n], Hg, Wg, z_lq=z[b:b + n] if update else None, sigma=0.4)
            torch.cuda.synchronize()
            assert torch.equal(part, whole[b:b + n]), (n, b)
