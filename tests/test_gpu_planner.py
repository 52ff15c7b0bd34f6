"""The prefetch planner at every width of its rows: plan arrays against the plain model over steps with repeated,
missing, unmapped and out-of-range predictions, for k at the edges of the compiled widths (8, 16, 32 lanes per row)
and row counts that do not fill the last workgroup."""
import numpy as np
import pytest
import torch

from oracle import prefetch_model as pm
from paper_2512_11920_amd import kvc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("k,n_seq,n_layers", [(1, 7, 3), (7, 3, 1), (8, 9, 2), (9, 5, 3), (16, 5, 1), (17, 3, 2), (31, 1, 3), (32, 3, 1)])
def test_plans_match_the_model_at_every_row_width(k, n_seq, n_layers, policy):
    rng = np.random.default_rng(100 * k + 10 * n_seq + n_layers + policy)
    N, d, pbl = 16, 32, 40
    c = kvc.Codec(N, d, 1, 3)
    c.alloc_pool(n_layers * pbl, n_layers * pbl * N * d, DEV)
    x = torch.from_numpy(rng.standard_normal((n_layers * pbl, 1, N, d)).astype(np.float16)).to(DEV)
    c.compress_blocks(x)
    c.set_prefetch_policy(policy)
    n_slots = n_layers * n_seq * k
    l2 = torch.zeros((2 * n_slots, 1, N, d), dtype=torch.float16, device=DEV)
    tags = torch.empty(2 * n_slots, dtype=torch.int32, device=DEV)
    fetch, loc = torch.empty(n_slots, dtype=torch.int32, device=DEV), torch.empty(n_slots, dtype=torch.int32, device=DEV)
    c.prefetch_reset(tags, n_seq, k, n_layers)
    m_tags = np.full((2, n_layers, n_seq, k), -1, np.int32)
    max_blocks = 12
    table = rng.integers(0, pbl, (n_seq, max_blocks)).astype(np.int32)  # entries repeat: two logical blocks, one pool block
    table[:, 3] = -1
    step = pm.prefetch_step_reuse if policy else pm.prefetch_step
    any_bad = False
    for t in range(8):
        pred = rng.integers(-1, max_blocks, (n_seq, k)).astype(np.int32)
        if t == 5:
            pred[rng.integers(0, n_seq), rng.integers(0, k)] = max_blocks  # no such logical block
        if t == 6:
            table[rng.integers(0, n_seq), :2] = pbl                        # beyond the layer's pool
        l1 = None if t % 3 else rng.integers(max_blocks // 2, max_blocks + 1, n_seq).astype(np.int32)
        print(f"[case] planner k={k} rows={n_seq * n_layers} policy={policy} step={t}", flush=True)
        c.prefetch_layers(l2, tags, fetch, loc, torch.from_numpy(table).to(DEV), torch.from_numpy(pred).to(DEV), n_layers, pbl, t % 2,
                          l1_first=None if l1 is None else torch.from_numpy(l1).to(DEV))
        m_fetch, m_loc, bad = step(m_tags, t % 2, table, pred, l1, n_layers, pbl)
        any_bad = any_bad or bad
        assert np.array_equal(loc.cpu().numpy(), m_loc.reshape(-1))
        assert np.array_equal(fetch.cpu().numpy(), m_fetch.reshape(-1))
        assert np.array_equal(tags.cpu().numpy(), m_tags.reshape(-1))
        assert bool(c.stats()["status"] & kvc.ST_BAD_INDEX) == any_bad
    assert any_bad
