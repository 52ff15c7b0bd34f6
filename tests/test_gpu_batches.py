"""Decoder waves: every kind of page task beside every other, in small calls, whose waves take a page each, and in calls
whose waves take several pages (the last wave not full), and the division the tasks are resolved with."""
import os
import subprocess

import numpy as np
import pytest
import torch

from oracle import kvc_oracle as o
from paper_2512_11920_amd import kvc
from launch_shapes import large_decoder_pages

DEV = "cuda:0"
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_fast_division_is_exact(tmp_path):
    """kvc_fastdiv.h against the machine's own division: every divisor up to 4096 and around every power of two, at the
    numerators where a quotient changes and at the ends of the range (below 2^31)."""
    src = tmp_path / "t.cpp"
    src.write_text("""
#include <stdio.h>
#include <initializer_list>
#include "kvc_fastdiv.h"
int main() {
    unsigned long long bad = 0, n = 0;
    auto one = [&](uint32_t d) {
        const kvc::FastDiv f = kvc::make_fast_div(d);
        const uint32_t last = 0x7FFFFFFFu;
        auto at = [&](uint64_t v) { if (v <= last) { ++n; bad += kvc::fast_div((uint32_t)v, f) != (uint32_t)v / d; } };
        for (uint64_t q : {0ull, 1ull, 2ull, 3ull, 1000ull, (unsigned long long)(last / d), (unsigned long long)(last / d / 2), (unsigned long long)(last / d / 3)})
            for (int e = -2; e <= 2; ++e) at(q * d + (uint64_t)(int64_t)e);
        at(last); at(last - 1); at((1u << 26) - 4); at((1u << 26) - 5);
    };
    for (uint32_t d = 1; d <= 4096; ++d) one(d);
    for (int b = 12; b <= 31; ++b)
        for (int e = -3; e <= 3; ++e)
            if ((1ll << b) + e <= (1ll << 31)) one((uint32_t)((1ll << b) + e));
    printf("%llu of %llu wrong\\n", bad, n);
    return bad != 0;
}
""")
    exe = tmp_path / "t"
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2512_11920_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("0 of "), r.stdout


# one, two, three, four passes, with and without a short last pass, and one of more than 64 groups: a page per wave
@pytest.mark.gpu
@pytest.mark.parametrize("N,d", [(16, 32), (8, 64), (7, 32), (16, 64), (13, 64), (16, 96), (16, 128), (20, 192)])
@pytest.mark.parametrize("ppb,n", [(1, 61), (3, 22)])
def test_every_kind_of_task_in_one_wave(N, d, ppb, n):
    task_kinds(N, d, ppb, n)


# pages of one and two passes in calls whose waves take four and two pages, from several blocks and from one and a part of another
@pytest.mark.gpu
@pytest.mark.parametrize("N,d", [(16, 32), (8, 64), (7, 32), (3, 96), (16, 64), (13, 64), (32, 32), (7, 128)])
@pytest.mark.parametrize("ppb", [1, 3, 5])
def test_every_kind_of_task_in_waves_of_several_pages(N, d, ppb):
    pages = large_decoder_pages(N, d) + 5  # the last wave is not full
    task_kinds(N, d, ppb, -(-pages // ppb), n_hits=pages // 23)


def task_kinds(N, d, ppb, n, n_hits=7):
    rng = np.random.default_rng(1000 * N + d + ppb)
    pages = n * ppb
    x = (rng.standard_normal((pages, N, d)) * np.exp(0.7 * rng.standard_normal((pages, 1, d)))).astype(np.float16)
    x[::2] = np.cumsum(rng.integers(-1, 2, (len(x[::2]), N, d)), axis=2).astype(np.float16)  # narrow packets, zero groups
    x[3::11] = np.float16(2.0)                                                               # zero-run packets
    x[5::13] = 0
    x[4::9].view(np.uint16)[:, N // 2, 3] = 0x7E00                                           # raw pages
    xt = torch.from_numpy(x.reshape(n, ppb, N, d)).to(DEV)
    top = 5 if N == 16 and d in (64, 128, 256) else 4
    modes = torch.from_numpy(rng.integers(0, top + 1, n).astype(np.uint8)).to(DEV)
    c = kvc.Codec(N, d, ppb, 3)
    c.alloc_pool(n, pages * N * d * 2 + 64, DEV)
    c.compress_blocks(xt, block_scheme=modes)
    assert c.stats()["rc"] == 0
    desc = c.desc_numpy().copy()
    pool = c.pool.cpu().numpy()
    # damage: an unknown mode, a wrong size, a span outside the pool, a first packet code no packet has
    packed = np.nonzero((desc["mode"] >= 2) & (desc["mode"] <= 5))[0]
    hit = rng.permutation(packed)[:n_hits]
    desc["mode"][hit[0::7]] = 9
    desc["n16"][hit[1::7]] += 1
    desc["off"][hit[2::7]] = pool.size
    desc["off"][hit[3::7]] += 8
    for h in np.concatenate([hit[4::7], hit[5::7]]):
        pool[int(desc["off"][h])] |= 0x0F
    desc["mode"][hit[6::7]] = 0xFF
    c.desc.copy_(torch.from_numpy(desc.view(np.uint8)).to(DEV))
    c.pool.copy_(torch.from_numpy(pool).to(DEV))
    want, bad = o.decompress_pages(pool, desc, N, d)
    assert bad >= 5
    # blocks out of order, some skipped on either side, some out of range
    src, dst = rng.permutation(n).astype(np.int32), rng.permutation(n).astype(np.int32)
    src[1::6] = -1
    dst[2::8] = -1
    src[9::83], dst[12::97] = n, n
    expect = np.full((n, ppb, N, d), 0x4700, np.uint16)
    for i in range(n):
        if 0 <= dst[i] < n and src[i] >= 0:
            expect[dst[i]] = want.reshape(n, ppb, N, d)[src[i]] if src[i] < n else 0
    out = torch.full((n, ppb, N, d), 7.0, dtype=torch.float16, device=DEV)
    print(f"[case] task kinds N={N} d={d} ppb={ppb} blocks={n}", flush=True)
    c.decompress_blocks(out, n=n, pool_ids=torch.from_numpy(src).to(DEV), dst_ids=torch.from_numpy(dst).to(DEV))
    status = c.stats()["status"]
    assert np.array_equal(out.cpu().numpy().view(np.uint16), expect)
    used = [src[i] for i in range(n) if 0 <= dst[i] < n and 0 <= src[i] < n]
    refused = {int(h) // ppb for h in hit} & {int(u) for u in used}
    assert bool(status & kvc.ST_CORRUPT) == bool(refused) and status & kvc.ST_BAD_INDEX
