"""Prefetch steps of few pages: rows of a part of a workgroup, of one and of many, calls around the pages that the chip holds
waves for, eight predictions and more -- over tags of every kind: blocks of the pool, empty, the largest and smallest of an int32,
blocks of a larger table that was bound before.  A tag that is no block of the step is a slot without one of its blocks, whatever
it is.  Tags, fetch list, places and buffer are the model's at every step."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as o
from oracle import prefetch_model as pm
from paper_2512_11920_amd import kvc
from gpu_util import DEV, gpu_compress

pytestmark = pytest.mark.gpu

STRANGE = [-2, -(1 << 31), (1 << 31) - 1, -(1 << 26) - 1, 1 << 26, (1 << 27) - 1, 0x68000000]  # tags no block of the pool has


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("N,d,ppb,n_seq,k,layers", [
    (16, 128, 1, 5, 1, 1), (16, 128, 7, 3, 1, 2), (16, 32, 8, 4, 1, 1), (8, 96, 9, 4, 1, 2), (16, 128, 2, 9, 4, 3), (13, 160, 5, 10, 7, 3), (16, 256, 3, 8, 8, 2),
    (16, 64, 32, 4, 8, 2), (16, 64, 33, 3, 8, 1), (7, 32, 16, 64, 8, 1), (7, 32, 16, 65, 8, 1), (16, 128, 4, 6, 9, 2)])
def test_steps_match_the_model(N, d, ppb, n_seq, k, layers, policy):
    rng = np.random.default_rng(N * d + ppb * k)
    nb = rng.integers(2, 9, n_seq)
    table = np.full((n_seq, 10), -1, np.int32)
    perm, at = rng.permutation(int(nb.sum())).astype(np.int32), 0
    for s in range(n_seq):
        table[s, :nb[s]] = perm[at:at + nb[s]]
        at += int(nb[s])
    pbl, n_slots = int(nb.sum()), layers * n_seq * k
    x = (rng.standard_normal((layers * pbl, ppb, N, d)) * np.exp(0.5 * rng.standard_normal(d))).astype(np.float16)
    x.reshape(-1, N, d)[3::11, 0, 0] = np.inf  # raw pages
    c, _ = gpu_compress(x, N, d, ppb, 3)
    od, op = o.compress_pages(x.view(np.uint16), N, d, 3, n_threads=8)
    full = o.decompress_pages(op, od, N, d, n_threads=8)[0].reshape(layers * pbl, ppb, N, d)
    c.set_prefetch_policy(policy)
    model_step = pm.prefetch_step_reuse if policy else pm.prefetch_step
    m_tags = rng.choice(np.array([-1, 0, 1, layers * pbl - 1] + STRANGE, np.int64).astype(np.int32), (2, layers, n_seq, k))
    tags = torch.from_numpy(m_tags.reshape(-1).copy()).to(DEV)
    fetch, loc = (torch.full((n_slots,), 7, dtype=torch.int32, device=DEV) for _ in range(2))
    l2 = torch.full((2 * n_slots, ppb, N, d), 5.0, dtype=torch.float16, device=DEV)
    content = np.full((2 * n_slots, ppb, N, d), np.float16(5.0).view(np.uint16), np.uint16)
    dev_table = torch.from_numpy(table).to(DEV)
    any_bad = False
    for step in range(6):
        pred = rng.integers(-1, 10, (n_seq, k)).astype(np.int32)
        if step == 4:
            pred[n_seq // 2, 0] = 10  # beyond the table
        l1 = np.maximum(nb - 1, 1).astype(np.int32) if step % 3 == 2 else None
        print(f"[case] prefetch steps N={N} d={d} ppb={ppb} seqs={n_seq} k={k} layers={layers} policy={policy} step {step}", flush=True)
        for lo, hi in ((0, 1), (1, layers)):  # (the second is a call over no layers where there is one)
            c.prefetch_layers(l2, tags, fetch, loc, dev_table, torch.from_numpy(pred).to(DEV), layers, pbl, step % 2, layer_begin=lo, layer_end=hi,
                              l1_first=None if l1 is None else torch.from_numpy(l1).to(DEV))
        m_fetch, m_loc, bad = model_step(m_tags, step % 2, table, pred, l1, layers, pbl)
        any_bad = any_bad or bad
        assert np.array_equal(tags.cpu().numpy(), m_tags.reshape(-1))
        assert np.array_equal(fetch.cpu().numpy(), m_fetch.reshape(-1)) and np.array_equal(loc.cpu().numpy(), m_loc.reshape(-1))
        got = m_fetch.reshape(-1) >= 0
        content[step % 2 * n_slots + np.nonzero(got)[0]] = full[m_fetch.reshape(-1)[got]]
        assert np.array_equal(l2.cpu().numpy().view(np.uint16), content)
    assert c.stats()["status"] == (kvc.ST_BAD_INDEX if any_bad else 0)
