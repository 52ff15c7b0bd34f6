"""The encoder's copy of a wave's payloads to the pool, line by line: from every position of the cursor within a line, with
raw pages among the others, into a pool that ends inside a wave -- the payloads are the oracle's, and not a byte of the
pool outside them changes."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as o
from paper_2512_11920_amd import kvc
from gpu_util import DEV
from launch_shapes import large_encoder_pages
from test_gpu_encoder_batches import check_stored, make_pages

pytestmark = pytest.mark.gpu


# a wave of one page, of several, and of the large shapes; payloads of one round of lanes and of many
@pytest.mark.parametrize("N,d,scheme,pages", [(16, 32, 3, 40), (16, 32, 3, 1030), (16, 32, 3, 0), (7, 32, 4, 0), (16, 64, 5, 0), (24, 96, 2, 0), (16, 128, 3, 600), (16, 128, 3, 0), (16, 128, 1, 0), (16, 256, 3, 0),
                                                (16, 32, 3, 127), (16, 32, 3, 128), (16, 64, 5, 128), (7, 128, 4, 200), (16, 128, 3, 127), (16, 128, 1, 300), (24, 96, 2, 512), (16, 256, 3, 512), (16, 256, 3, 513)])
def test_nothing_beside_the_payloads_changes(N, d, scheme, pages):
    n = pages or large_encoder_pages(N, d, scheme) + 9
    x = make_pages(np.random.default_rng(N * d + n), n, N, d)
    od, op = o.compress_pages(x.view(np.uint16), N, d, scheme, n_threads=8)
    need = int((od["n16"].astype(np.int64) * 16).sum())
    xt = torch.from_numpy(x.reshape(n, 1, N, d)).to(DEV)
    rng = np.random.default_rng(n)
    for first in range(8):
        short = first % 2 == 1  # the pool ends 1 to 40 units early
        room = need - 16 * int(rng.integers(1, 41)) if short else need
        print(f"[case] copy-out N={N} d={d} scheme={scheme} pages={n} first unit {first} room {room} of {need}", flush=True)
        store = torch.full((16 * first + room + 256,), 0xA5, dtype=torch.uint8, device=DEV)
        c = kvc.Codec(N, d, 1, scheme)
        c.bind_pool(store[:16 * first + room], torch.zeros(n * 16, dtype=torch.uint8, device=DEV))
        c.reset_pool()
        c.restore_pool(16 * first)
        c.compress_blocks(xt)
        assert c.stats()["status"] == (kvc.ST_POOL_FULL if short else 0)
        desc, pool = c.desc_numpy(), store.cpu().numpy()
        stored = np.nonzero(desc["mode"] != 0xFF)[0]
        assert short or stored.size == n
        check_stored(desc, pool, stored, od, op, stored)
        end = int((desc["off"][stored].astype(np.int64) + desc["n16"][stored].astype(np.int64) * 16).max())
        assert (pool[:16 * first] == 0xA5).all() and (pool[end:] == 0xA5).all()
