"""Encoder workgroups that hold several pages: everything that is not the plain case -- block ids that skip or leave
their range inside a wave and over whole waves, a descriptor table that ends inside a block, a last workgroup that is
not full, one mode per block, a pool that fills inside a workgroup -- against the oracle, at call sizes that take the
large-call shapes (large_encoder_pages, which a test on the recorded launches holds to the library) and some below."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as o
from paper_2512_11920_amd import kvc
from launch_shapes import large_encoder_pages

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

def large(N, d, scheme, more=0):
    return N, d, scheme, large_encoder_pages(N, d, scheme) + more


# one to eight passes, whole and short last passes; the middle and the large launch of four-pass pages with the mode fixed;
# both deals of the tasks of whole eight-pass pages (in order up to 32,768 pages)
CASES = [large(N, d, scheme, more) for (N, d) in ((16, 32), (16, 64), (16, 96), (16, 128), (16, 160), (16, 192), (16, 224), (16, 256)) for scheme, more in ((3, 0), ("mixed", 51))] + \
        [(16, 256, 3, 32770), (16, 256, 4, 32770), (32, 128, "mixed", 32770)] + \
        [large(16, 64, 5, 200), large(16, 256, 5), large(16, 128, 5), (16, 64, 5, 2300), (16, 256, 5, 2049), (16, 128, 5, 2049), (16, 128, 3, 16380), (16, 128, 3, 16400), (16, 128, 5, 16400)] + \
        [large(7, 32, 3), large(13, 64, "mixed", 51), large(9, 128, 2, 51), large(15, 96, 4), large(13, 160, 3, 51), large(21, 192, "mixed"), large(17, 224, 1), large(15, 256, 3, 51)] + \
        [(16, 32, 3, 2049), (16, 64, "mixed", 2100), (16, 96, 3, 2049), (16, 128, "mixed", 2100), (16, 224, 3, 2049), (7, 32, 3, 2049), (21, 192, "mixed", 2049)]


def make_pages(rng, n, N, d):
    x = (rng.standard_normal((n, N, d), dtype=np.float32) * np.exp(rng.standard_normal((n, 1, d), dtype=np.float32))).astype(np.float16)
    x[::3] = np.cumsum(rng.integers(-2, 3, (len(x[::3]), N, d), dtype=np.int8), axis=2, dtype=np.float32).astype(np.float16)
    x[5::23] = 0
    x[4::19].view(np.uint16)[:, N // 2, d // 3] = 0x7E00  # raw pages
    x[6::31, :, ::2] = 0
    return x


def oracle_pages(x, N, d, modes):
    """Descriptors and payloads of every page, each in the mode requested for it."""
    od, chunks, off = np.zeros(len(x), o.DESC_DTYPE), [], 0
    for sc in np.unique(modes):
        idx = np.nonzero(modes == sc)[0]
        dd, pp = o.compress_pages(np.ascontiguousarray(x[idx]).view(np.uint16), N, d, int(sc), n_threads=8)
        dd = dd.copy()
        dd["off"] += off
        od[idx] = dd
        chunks.append(pp)
        off += pp.size
    return od, np.concatenate(chunks)


def check_stored(desc, pool, entries, od, op, pages):
    """Descriptor-table entries hold the given pages of the oracle's: fields and payload bytes."""
    got, want = desc[entries], od[pages]
    for f in ("mode", "n16", "rsvd"):
        assert np.array_equal(got[f], want[f]), f
    assert np.array_equal(got["scale"].view(np.uint32), want["scale"].view(np.uint32))
    size = want["n16"].astype(np.int64) * 16
    at = np.arange(size.sum()) - np.repeat(np.cumsum(size) - size, size)
    assert np.array_equal(pool[np.repeat(got["off"].astype(np.int64), size) + at], op[np.repeat(want["off"].astype(np.int64), size) + at]), "payload bytes"


def spans(desc):
    off, size = desc["off"].astype(np.int64), desc["n16"].astype(np.int64) * 16
    order = np.argsort(off, kind="stable")
    return off[order], size[order]


@pytest.mark.parametrize("ppb", [1, 3, 5])
@pytest.mark.parametrize("N,d,scheme,pages", CASES)
def test_ids_modes_and_a_full_pool(N, d, scheme, pages, ppb):
    rng = np.random.default_rng(N * 1000 + d + pages + ppb)
    n = -(-pages // ppb)              # blocks of the call
    n_cache, n_pool = n // 2 + 3, n + 7
    x = make_pages(rng, n_cache * ppb, N, d)
    top = 5 if N == 16 and d in (64, 128, 256) else 4
    if scheme == "mixed":
        block_modes = rng.integers(0, top + 3, n).astype(np.uint8)  # values above the highest are read as the highest
        want_modes = np.minimum(block_modes, top)
    else:
        block_modes, want_modes = None, np.full(n, scheme)
    src = rng.integers(0, n_cache, n).astype(np.int32)
    pool_ids = rng.permutation(n_pool)[:n].astype(np.int32)
    src[rng.random(n) < 0.1] = -1
    pool_ids[rng.random(n) < 0.1] = -3
    src[n // 3: n // 3 + 200 // ppb] = -1        # whole waves, and a whole workgroup, with nothing to do
    src[rng.integers(0, n, 5)] = n_cache
    src[rng.integers(0, n, 3)] = 2**31 - 1
    pool_ids[rng.integers(0, n, 4)] = n_pool
    pool_ids[rng.integers(0, n, 2)] = 2**30
    src[n - 1], pool_ids[n - 1] = 0, n_pool - 1  # the last page of the call, in the block the descriptor table ends in
    pool_ids[:-1][pool_ids[:-1] == n_pool - 1] = -1
    n_desc = n_pool * ppb - (1 if ppb > 1 else 0)

    # what each page task of the call has to do
    page = np.arange(n * ppb)
    b, pg = page // ppb, page % ppb
    wanted = (src[b] >= 0) & (pool_ids[b] >= 0)
    entry = pool_ids[b].astype(np.int64) * ppb + pg
    good = wanted & (src[b] < n_cache) & (entry < n_desc)
    assert (wanted & ~good).any()
    source = src[b].astype(np.int64) * ppb + pg
    # every (source page, mode) the call asks for, through the oracle
    keys, inverse = np.unique(np.stack([source[good], want_modes[b][good]]), axis=1, return_inverse=True)
    inverse = np.ravel(inverse)
    od, op = oracle_pages(x[keys[0]], N, d, keys[1])
    need = int((od["n16"][inverse].astype(np.int64) * 16).sum())

    xt = torch.from_numpy(x.reshape(n_cache, ppb, N, d)).to(DEV)
    args = dict(n=n, src_ids=torch.from_numpy(src).to(DEV), pool_ids=torch.from_numpy(pool_ids).to(DEV),
                block_scheme=None if block_modes is None else torch.from_numpy(block_modes).to(DEV))
    for pool_bytes in (need, need * 3 // 5 // 16 * 16):
        print(f"[case] encoder batches N={N} d={d} scheme={scheme} blocks={n} ppb={ppb} pool={pool_bytes} of {need}", flush=True)
        c = kvc.Codec(N, d, ppb, 3 if scheme == "mixed" else scheme)
        c.bind_pool(torch.zeros(pool_bytes, dtype=torch.uint8, device=DEV), torch.zeros(n_desc * 16, dtype=torch.uint8, device=DEV))
        c.reset_pool()
        c.compress_blocks(xt, **args)
        st = c.stats()
        desc, pool = c.desc_numpy(), c.pool.cpu().numpy()
        full = pool_bytes < need
        assert st["status"] == kvc.ST_BAD_INDEX | (kvc.ST_POOL_FULL if full else 0)
        assert st["pool_bytes_used"] == pool_bytes
        stored = good & (desc["mode"][np.where(good, entry, 0)] != 0xFF)
        assert full or stored[good].all()
        check_stored(desc, pool, entry[stored], od, op, inverse[stored[good]])
        # the stored payloads lie side by side from the pool's beginning, and only what does not fit is missing
        off, size = spans(desc[entry[stored]])
        assert off[0] == 0 and np.array_equal(off[1:], (off + size)[:-1])
        assert pool_bytes - (off[-1] + size[-1]) < (int(od["n16"].max()) * 16 if full else 1)
        # every other descriptor is as the reset left it
        others = np.ones(n_desc, bool)
        others[entry[stored]] = False
        blank = np.zeros(1, desc.dtype)
        blank["mode"] = 0xFF
        assert (desc[others] == blank[0]).all()
