"""Decode calls of 32,768 pages and more, for which pages of 4 KB and more have a limit on the workgroups of a compute
unit: the same bytes as calls that name their blocks, which have none, and as the oracle for pages of every kind."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as o
from paper_2512_11920_amd import kvc
from gpu_util import DEV, fetch_pages

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d", [(16, 128), (32, 64), (15, 128), (16, 96), (16, 160), (32, 96), (11, 256), (16, 224), (13, 256), (16, 256), (15, 256)])
def test_decode_calls_around_the_limit(N, d):
    n, cut = 32768 + 6, 32767
    top = 5 if N == 16 and d == 256 else 4
    g = torch.Generator(device=DEV)
    g.manual_seed(N * d)
    x = (torch.randn((n, 1, N, d), generator=g, device=DEV) * torch.exp(0.5 * torch.randn((n, 1, 1, d), generator=g, device=DEV))).half()
    x[::17] = 0
    x[5::29, :, N // 2:] = 1.0
    x[3::41, :, 0, 0] = float("nan")  # raw pages
    modes = (torch.arange(n, device=DEV) % (top + 1)).to(torch.uint8)
    c = kvc.Codec(N, d, 1, 3)
    c.alloc_pool(n, 2 * x.numel() + 64, DEV)
    c.compress_blocks(x, block_scheme=modes)
    print(f"[case] decode calls around the limit N={N} d={d}", flush=True)
    once, parts = torch.full_like(x, 7.0), torch.full_like(x, 7.0)
    c.decompress_blocks(once)
    ids = torch.arange(n, dtype=torch.int32, device=DEV)
    for part in (ids[:cut], ids[cut:]):
        c.decompress_blocks(parts, n=part.numel(), pool_ids=part, dst_ids=part)
    assert torch.equal(once.view(torch.int16), parts.view(torch.int16))
    some = np.concatenate([np.arange(300), np.arange(n - 60, n)])
    desc, buf = fetch_pages(c, some)
    want, bad = o.decompress_pages(buf, desc, N, d)
    assert bad == 0 and np.array_equal(once[torch.from_numpy(some).to(DEV)].cpu().numpy().view(np.uint16).reshape(want.shape), want)
    assert c.stats()["status"] == 0
