"""Calls below the large launch shapes: the encoder's workgroups on both sides of every line between them, and the
decoder's single-page waves of one- and two-pass pages, against the oracle."""
import numpy as np
import pytest
import torch

import test_gpu_encoder_batches as batches
from oracle import kvc_oracle as o
from paper_2512_11920_amd import kvc
from gpu_util import DEV

pytestmark = pytest.mark.gpu

CASES = [(N, d, scheme, pages) for N, d in ((16, 32), (13, 64), (16, 64), (16, 96), (15, 96), (16, 128), (13, 160), (16, 192), (17, 224), (16, 256)) for scheme, pages in ((3, 7), (3, 509), ("mixed", 516), (3, 1023), ("mixed", 1029))] + \
        [(16, 32, 3, 16380), (16, 32, "mixed", 32764), (7, 32, 3, 16400), (7, 32, 3, 32780), (16, 64, 3, 2046), (16, 64, 5, 2052), (16, 64, 3, 16395), (16, 64, "mixed", 16395), (9, 128, "mixed", 2046), (9, 128, 2, 16383)] + \
        [(16, 96, 3, 8190), (16, 96, "mixed", 8196), (13, 96, 3, 8190), (16, 128, 3, 8190), (16, 128, 3, 8196), (16, 128, 3, 13311), (16, 128, 3, 13317), (16, 128, 3, 16386), (16, 128, 5, 4095), (16, 128, 5, 4101), (16, 128, 5, 13314), (16, 128, 5, 32766)] + \
        [(16, 128, "mixed", 4095), (16, 128, "mixed", 4101), (16, 128, "mixed", 8190), (15, 128, 4, 4095), (15, 128, 4, 4101), (16, 128, 2, 4101), (32, 64, 4, 4095)] + \
        [(16, 128, 1, 2046), (16, 128, 1, 2052), (16, 64, 1, 8190), (16, 64, 0, 8196), (16, 256, 0, 2046), (13, 160, 3, 3069), (16, 192, "mixed", 3075), (16, 192, 3, 3069), (17, 224, 3, 4095), (16, 256, 3, 4095), (16, 256, 5, 4092), (16, 256, "mixed", 4101)]


@pytest.mark.parametrize("N,d,scheme,pages", CASES)
def test_encoder_at_the_lines_between_its_launch_shapes(N, d, scheme, pages):
    batches.test_ids_modes_and_a_full_pool(N, d, scheme, pages, 3)


@pytest.mark.parametrize("N,d,pages", [(16, 32, 5), (16, 32, 4096), (16, 32, 4097), (7, 32, 4095), (16, 64, 8192), (16, 64, 8193), (13, 64, 3), (8, 128, 8190), (5, 192, 100), (3, 256, 8193)])
def test_decoder_of_small_calls(N, d, pages):
    rng = np.random.default_rng(N * d + pages)
    x = batches.make_pages(rng, pages, N, d)
    top = 5 if N == 16 and d in (64, 128, 256) else 4
    modes = np.arange(pages) % (top + 1)
    od, op = batches.oracle_pages(x, N, d, modes)
    od[2::37]["mode"] = 0xFF  # never written: zero-filled
    od[4::53]["n16"] += 1     # a size that is wrong
    want, bad = o.decompress_pages(op, od, N, d, n_threads=8)
    c = kvc.Codec(N, d, 1, 3)
    pool, desc = torch.from_numpy(op).to(DEV), torch.from_numpy(od.view(np.uint8).copy()).to(DEV)
    c.bind_pool(pool, desc)
    dst = rng.permutation(pages + 3)[:pages].astype(np.int32)
    dst[::11] = -1
    out = torch.full((pages + 3, 1, N, d), 7.0, dtype=torch.float16, device=DEV)
    print(f"[case] small decode N={N} d={d} pages={pages}", flush=True)
    c.decompress_blocks(out, n=pages, dst_ids=torch.from_numpy(dst).to(DEV))
    got = out.cpu().numpy().view(np.uint16).reshape(pages + 3, N, d)
    expect = np.full_like(got, np.float16(7.0).view(np.uint16))
    expect[dst[dst >= 0]] = want[dst >= 0]
    assert np.array_equal(got, expect)
