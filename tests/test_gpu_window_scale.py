"""The prefetch window with every compute unit busy: buffers bit-equal to the unbounded call's, for every kind of payload
and for wide and narrow transfer engines."""
import numpy as np
import pytest
import torch

from paper_2512_11920_amd import kvc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("N,d,ppb,scheme", [(16, 128, 16, 3), (16, 128, 8, 5), (16, 64, 16, 3), (16, 64, 3, 5), (16, 32, 8, 4), (24, 96, 6, 2), (16, 256, 4, 3),
                                            (16, 256, 2, 5), (16, 128, 16, 1), (16, 128, 5, 0), (8, 192, 20, 3)])
def test_window_equals_unbounded_call_on_a_busy_gpu(N, d, ppb, scheme):
    n_layers, n_seq, k, pbl = 4, 64, 8, 600
    g = torch.Generator(device=DEV)
    g.manual_seed(N * d + ppb + scheme)
    x = torch.randn((n_layers * pbl, ppb, N, d), generator=g, device=DEV)
    x = (x * torch.exp(0.5 * torch.randn((ppb, 1, d), generator=g, device=DEV))).half()
    x[::17] = 0
    x[5::29, :, N // 2:] = 0
    c = kvc.Codec(N, d, ppb, scheme)
    c.alloc_pool(n_layers * pbl, x.numel() * 2 + 64, DEV)
    c.compress_blocks(x)
    rng = np.random.default_rng(d + ppb)
    table = torch.from_numpy(rng.integers(0, pbl, (n_seq, 32)).astype(np.int32)).to(DEV)
    preds = [torch.from_numpy(rng.integers(0, 32, (n_seq, k)).astype(np.int32)).to(DEV) for _ in range(2)]
    n_slots = n_layers * n_seq * k

    def run(omega):
        l2 = torch.zeros((2 * n_slots, ppb, N, d), dtype=torch.float16, device=DEV)
        tags = torch.empty(2 * n_slots, dtype=torch.int32, device=DEV)
        fetch, loc = torch.empty(n_slots, dtype=torch.int32, device=DEV), torch.empty(n_slots, dtype=torch.int32, device=DEV)
        notify = torch.zeros(n_layers + 4, dtype=torch.int64, device=DEV)
        work = torch.empty(kvc.window_workspace(n_slots, n_layers), dtype=torch.uint8, device=DEV)
        c.prefetch_reset(tags, n_seq, k, n_layers)
        for half, pred in enumerate(preds):
            if omega:
                c.prefetch_layers_window(l2, tags, fetch, loc, table, pred, n_layers, pbl, half, omega, notify, work)
            else:
                c.prefetch_layers(l2, tags, fetch, loc, table, pred, n_layers, pbl, half)
        torch.cuda.synchronize()
        return l2, tags, notify

    want, tags0, _ = run(0)
    for omega in (64, 256, 4096):
        print(f"[case] busy window N={N} d={d} ppb={ppb} scheme={scheme} omega={omega}", flush=True)
        got, tags, notify = run(omega)
        assert torch.equal(tags, tags0)
        wrong = (got.view(torch.int16) != want.view(torch.int16)).view(2 * n_slots * ppb, -1).any(1)
        assert not wrong.any(), f"omega {omega}: {int(wrong.sum())} of {wrong.numel()} pages differ"
        nt = notify.cpu().numpy()
        assert (nt[:n_layers] >= nt[n_layers]).all() and (nt[:n_layers] <= nt[n_layers + 3]).all()
    assert c.stats()["status"] == 0
