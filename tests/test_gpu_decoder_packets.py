"""The decoder on payloads that no encoder chose: random packet codes (every width, zero runs, runs) and random body
bytes, so that every width begins at every byte offset, differences wrap around 8 bits and a row's sum passes any value,
against the oracle's decoder."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as o
from gpu_util import DEV, make_codec, upload_oracle_pool
from launch_shapes import large_decoder_pages

pytestmark = pytest.mark.gpu


def random_payloads(rng, n, N, d, mode):
    E = N * d
    groups, hdr = E // 32, (E // 32 + 1) // 2
    desc, chunks, off = np.zeros(n, o.DESC_DTYPE), [], 0
    lo, hi = (1, 9) if mode == 2 else (0, 10)
    for i in range(n):
        while True:
            # some pages of one width only, some without runs, the others of any codes
            codes = np.full(groups, rng.integers(1, 9)) if i % 5 == 0 else rng.integers(1, 9, groups) if i % 5 == 1 else rng.integers(lo, hi, groups)
            size = hdr + int(np.where(codes == 9, 1, 4 * codes).sum())
            n16 = (size + 15) // 16
            if n16 < E // 16:
                break
        pay = np.zeros(n16 * 16, np.uint8)
        pay[hdr:size] = rng.integers(0, 256, size - hdr)
        nib = np.zeros(2 * hdr, np.uint8)
        nib[:groups] = codes
        pay[:hdr] = nib[::2] | (nib[1::2] << 4)
        desc[i]["off"], desc[i]["n16"], desc[i]["mode"] = off, n16, mode
        desc[i]["scale"] = np.float32(2.0 ** rng.uniform(-20, 8)) if i % 7 else np.float32(2.0 ** rng.uniform(-31, -24))  # (down to half-precision subnormals)
        chunks.append(pay)
        off += pay.size
    return desc, np.concatenate(chunks)


# rows of 4, 8, 16 and 32 lanes; rows that cross passes; short last passes; mode 5 in its three shapes
@pytest.mark.parametrize("N,d", [(16, 32), (32, 32), (16, 64), (16, 96), (24, 96), (7, 128), (16, 128), (32, 128), (16, 160), (5, 192), (16, 224), (13, 256), (16, 256)])
def test_random_packets_decode_as_the_oracle_decodes_them(N, d):
    rng = np.random.default_rng(N * 1000 + d)
    for mode in (2, 3, 4) + ((5,) if N == 16 and d in (64, 128, 256) else ()):
        n = 420
        desc, pool = random_payloads(rng, n, N, d, mode)
        want, bad = o.decompress_pages(pool, desc, N, d)
        assert bad == 0
        c = make_codec(N, d, 1, 3, 1)
        keep = upload_oracle_pool(c, desc, pool)
        out = torch.empty((n, 1, N, d), dtype=torch.float16, device=DEV)
        print(f"[case] random packets N={N} d={d} mode={mode}", flush=True)
        c.decompress_blocks(out)
        got = out.cpu().numpy().view(np.uint16).reshape(n, N, d)
        wrong = np.nonzero((got != want).any((1, 2)))[0]
        assert wrong.size == 0, f"{wrong.size} of {n} pages differ, first {wrong[:5]}"
        assert c.stats()["status"] == 0
        del keep


# the same payloads many times over, in calls whose waves take four and two pages of one and two passes, which share their header scans
@pytest.mark.parametrize("N,d", [(16, 32), (7, 32), (3, 128), (16, 64), (13, 64), (5, 192)])
def test_random_packets_in_waves_of_several_pages(N, d):
    rng = np.random.default_rng(N * 1000 + d + 1)
    for mode in (2, 3, 4) + ((5,) if N == 16 and d == 64 else ()):
        some, pool = random_payloads(rng, 420, N, d, mode)
        desc = some[rng.integers(0, 420, large_decoder_pages(N, d) + 6)]
        want, bad = o.decompress_pages(pool, desc, N, d, n_threads=8)
        assert bad == 0
        c = make_codec(N, d, 1, 3, 1)
        keep = upload_oracle_pool(c, desc, pool)
        out = torch.empty((desc.size, 1, N, d), dtype=torch.float16, device=DEV)
        print(f"[case] random packets N={N} d={d} mode={mode} pages={desc.size}", flush=True)
        c.decompress_blocks(out)
        wrong = np.nonzero((out.cpu().numpy().view(np.uint16).reshape(-1, N, d) != want).any((1, 2)))[0]
        assert wrong.size == 0, f"{wrong.size} of {desc.size} pages differ, first {wrong[:5]}"
        assert c.stats()["status"] == 0
        del keep
