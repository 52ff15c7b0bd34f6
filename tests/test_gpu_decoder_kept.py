"""Calls that decode a whole range and read the payloads beyond the pool's beginning past the last-level cache (768 MiB to
4 GiB of pages): the same bytes as the range one page short of it, and as parts of it named by block ids, which are read
plainly -- packed, INT8, raw and refused pages on both sides of the line."""
import pytest
import torch

from paper_2512_11920_amd import kvc
from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d", [(16, 32), (16, 64), (24, 96), (16, 128), (16, 256)])
def test_whole_ranges_beside_the_pools_beginning(N, d):
    n = -(-(768 << 20) // (2 * N * d))
    top = 5 if N == 16 and d in (64, 128, 256) else 4
    g = torch.Generator(device=DEV)
    g.manual_seed(N * d)
    x = torch.randn((n, 1, N, d), generator=g, device=DEV, dtype=torch.float16) * torch.exp(0.5 * torch.randn((n, 1, 1, d), generator=g, device=DEV, dtype=torch.float16))
    x[::17] = 0
    x[3::41, :, 0, 0] = float("nan")  # raw pages
    c = kvc.Codec(N, d, 1, 3)
    c.alloc_pool(n, 2 * x.numel() + 64, DEV)
    print(f"[case] whole ranges N={N} d={d} pages={n}", flush=True)
    c.compress_blocks(x, block_scheme=(torch.arange(n, device=DEV) % (top + 1)).to(torch.uint8))
    assert c.stats()["pool_bytes_used"] > (256 << 20)
    c.desc.view(-1, 16)[7::4099, 14] = 9  # no such mode
    once, short, parts = torch.full_like(x, 7.0), torch.full_like(x, 7.0), torch.full_like(x, 7.0)
    c.decompress_blocks(once)
    c.decompress_blocks(short, n=n - 1)
    ids = torch.arange(n, dtype=torch.int32, device=DEV)
    for part in ids.split(1 << 16):
        c.decompress_blocks(parts, n=part.numel(), pool_ids=part, dst_ids=part)
    assert torch.equal(once[:n - 1].view(torch.int16), short[:n - 1].view(torch.int16))
    assert torch.equal(once.view(torch.int16), parts.view(torch.int16))
    assert not once[7::4099].view(torch.int16).any() and c.stats()["status"] == kvc.ST_CORRUPT


@pytest.mark.parametrize("N,d", [(16, 32), (7, 96), (16, 128), (16, 256)])
@pytest.mark.parametrize("first", [0, (208 << 20) - 16, 208 << 20, 300 << 20])
def test_ranges_that_begin_beside_the_line(N, d, first):
    """A range whose first payload is the pool's, the last unit before the line, the first unit behind it or far behind: the smallest that
    may read past the cache, as the range one page short of it, which may not."""
    n = -(-(608 << 20) // (2 * N * d))
    g = torch.Generator(device=DEV)
    g.manual_seed(N * d + first)
    x = torch.randn((n, 1, N, d), generator=g, device=DEV, dtype=torch.float16)
    x[3::41, :, 0, 0] = float("inf")  # raw pages
    c = kvc.Codec(N, d, 1, 3)
    c.alloc_pool(n, first + 2 * x.numel() + 64, DEV)
    c.restore_pool(first)
    print(f"[case] ranges beside the line N={N} d={d} pages={n} first byte {first}", flush=True)
    c.compress_blocks(x[:1])  # (calls of a stream: page 0 is the first)
    ids = torch.arange(1, n, dtype=torch.int32, device=DEV)
    c.compress_blocks(x, n=n - 1, src_ids=ids, pool_ids=ids)
    assert c.desc_numpy()["off"][0] == first
    once, short = torch.full_like(x, 7.0), torch.full_like(x, 7.0)
    c.decompress_blocks(once)
    c.decompress_blocks(short, n=n - 1)
    assert torch.equal(once[:n - 1].view(torch.int16), short[:n - 1].view(torch.int16)) and c.stats()["status"] == 0
    last = torch.full_like(x[:1], 7.0)
    c.decompress_blocks(last, pool_ids=ids[-1:], dst_ids=torch.zeros(1, dtype=torch.int32, device=DEV))
    assert torch.equal(once[-1:].view(torch.int16), last.view(torch.int16))
