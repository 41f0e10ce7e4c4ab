"""GPU: row gather / scatter and the dense map over the forms of their kernels: rows of 2^k and of other numbers of 16-byte
pieces, ends of a workgroup's share, and sizes whose accesses pass the memory-side cache by.  Bytes, so exact."""
import pytest
import torch

import paper_2301_08739_amd as ff

pytestmark = pytest.mark.gpu
DEV = "cuda"
TORCH = {ff.FF_BF16: torch.bfloat16, ff.FF_F16: torch.float16, ff.FF_F32: torch.float32}


@pytest.mark.parametrize("n, C, dt", [
    (1, 8, ff.FF_BF16), (511, 8, ff.FF_F16), (513, 8, ff.FF_BF16),                    # one piece a row
    (257, 24, ff.FF_BF16), (1000, 96, ff.FF_F16), (171, 12, ff.FF_F32),               # 3 and 12
    (63, 64, ff.FF_BF16), (4097, 128, ff.FF_F16), (3001, 256, ff.FF_F32),             # 8, 16, 64
    ((14 << 20) // 256, 128, ff.FF_F16), ((14 << 20) // 256 + 1, 128, ff.FF_BF16), (50000, 72, ff.FF_F32),  # either side of kRowsShort,
    ((64 << 20) // 512, 256, ff.FF_BF16), ((64 << 20) // 512 + 1, 256, ff.FF_BF16),    # kScatterStreamed
    ((128 << 20) // 512, 256, ff.FF_BF16), ((128 << 20) // 512 + 1, 256, ff.FF_BF16)])  # and kGatherStreamed
def test_rows_there_and_back(n, C, dt):
    gen = torch.Generator(device=DEV).manual_seed(n + C)
    x = torch.randint(-2**31, 2**31 - 1, (n, C * (2 if dt == ff.FF_F32 else 1) // 2), device=DEV, generator=gen,
                      dtype=torch.int32).view(TORCH[dt])
    perm = torch.randperm(n, device=DEV, generator=gen).to(torch.int32)
    bits = torch.int32 if dt == ff.FF_F32 else torch.int16
    g = ff.ff_gather(x, perm, dt)
    assert torch.equal(g.view(bits), x.view(bits)[perm.long()])
    assert torch.equal(ff.ff_scatter(g, perm, dt).view(bits), x.view(bits))


@pytest.mark.parametrize("frames, grid, C, n", [(1, 443, 128, 5000), (1, 444, 128, 5000), (1, 640, 128, 5000), (1, 641, 128, 5000),
                                              (2, 31, 12, 700)])
def test_dense_map_either_side_of_the_streamed_fill(frames, grid, C, n):
    """640 x 640 x 128 floats are 200 MiB, 641 x 641 more; 12 floats are three pieces a row."""
    gen = torch.Generator(device=DEV).manual_seed(grid)
    cells = torch.randperm(frames * grid * grid, device=DEV, generator=gen)[:n]
    coords = torch.stack([cells // (grid * grid), cells // grid % grid, cells % grid], 1).to(torch.int32).contiguous()
    x = torch.randn(n, C, device=DEV, generator=gen)
    out = torch.full((frames, grid, grid, C), 7.0, device=DEV)
    ff.ff_bev_scatter(x, coords, ff.Geometry(frames, grid, grid, 8, 8), ff.FF_F32, out=out)
    want = torch.zeros(frames, grid, grid, C, device=DEV)
    want[coords[:, 0].long(), coords[:, 2].long(), coords[:, 1].long()] = x
    assert torch.equal(out, want)
