"""The prefetch window's engines where the other window tests do not look: layers read by another stream while later
ones are still in flight, and turns of more page tasks than a wave resolves at once."""
import numpy as np
import pytest
import torch

from paper_2512_11920_amd import kvc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


class Window:
    """A pool with every kind of page in every layer, and one prefetch step over it."""

    def __init__(self, N, d, ppb, n_layers, n_seq, k, pbl):
        self.n_layers, self.n_seq, self.k, self.pbl = n_layers, n_seq, k, pbl
        self.shape = (2, n_layers, n_seq * k, ppb, N, d)
        self.n_slots = n_layers * n_seq * k
        g = torch.Generator(device=DEV)
        g.manual_seed(N * d + ppb + self.n_slots)
        x = torch.randn((n_layers * pbl, ppb, N, d), generator=g, device=DEV)
        x = (x * torch.exp(0.5 * torch.randn((ppb, 1, d), generator=g, device=DEV))).half()
        x[::17] = 0                   # zero-run packets
        x[5::29, :, N // 2:] = 1.0    # run packets
        top = 5 if N == 16 and d in (64, 128, 256) else 4
        modes = (torch.arange(n_layers * pbl, device=DEV) % (top + 1)).to(torch.uint8)
        self.c = kvc.Codec(N, d, ppb, 3)
        self.c.alloc_pool(n_layers * pbl, x.numel() * 2 + 64, DEV)
        self.c.compress_blocks(x, block_scheme=modes)
        assert self.c.stats()["rc"] == 0
        desc = self.c.desc.view(-1, 16)
        desc[3 * ppb::31, 14] = 0xFF  # pages never written: zero-filled
        desc[7 * ppb::37, 12] += 1    # sizes that are wrong: zero-filled too
        self.table = torch.stack([torch.randperm(pbl, generator=g, device=DEV) for _ in range(n_seq)]).int().contiguous()
        self.pred = torch.stack([torch.randperm(pbl, generator=g, device=DEV)[:k] for _ in range(n_seq)]).int().contiguous()
        self.tags = torch.empty(2 * self.n_slots, dtype=torch.int32, device=DEV)
        self.fetch = torch.empty(self.n_slots, dtype=torch.int32, device=DEV)
        self.loc = torch.empty(self.n_slots, dtype=torch.int32, device=DEV)
        self.notify = torch.zeros(n_layers + 4, dtype=torch.int64, device=DEV)
        self.work = torch.empty(kvc.window_workspace(self.n_slots, n_layers), dtype=torch.uint8, device=DEV)

    def buffer(self):
        return torch.full(self.shape, 7.0, dtype=torch.float16, device=DEV)

    def run(self, l2, omega, stream=None):
        flat = l2.view(-1, *self.shape[3:])
        self.c.prefetch_reset(self.tags, self.n_seq, self.k, self.n_layers, stream=stream)
        args = (flat, self.tags, self.fetch, self.loc, self.table, self.pred, self.n_layers, self.pbl, 0)
        if omega:
            self.c.prefetch_layers_window(*args, omega, self.notify, self.work, stream=stream)
        else:
            self.c.prefetch_layers(*args, stream=stream)


# Engines on a queue that keeps them busy for milliseconds: few and many of the wide kind (16 waves, up to 256 or 512 engines by
# page shape), with a clerk and turn by turn; and the narrow kind, which more engines than that take.
@pytest.mark.parametrize("N,d,ppb,omega,layers,n_seq,k", [(16, 128, 4, 2, 8, 16, 8), (16, 64, 16, 4, 8, 16, 8), (16, 256, 3, 3, 8, 16, 8), (24, 96, 5, 2, 8, 16, 8),
                                                          (16, 32, 16, 1, 8, 16, 8), (16, 128, 16, 256, 24, 64, 32), (16, 32, 16, 200, 32, 128, 32), (16, 128, 1, 1024, 16, 1024, 32), (16, 64, 2, 1024, 32, 1024, 32)])
def test_a_layer_stamped_ready_can_be_read_while_the_window_is_open(N, d, ppb, omega, layers, n_seq, k):
    w = Window(N, d, ppb, layers, n_seq, k, 96)
    want = w.buffer()
    w.run(want, 0)
    got = w.buffer()
    snaps = torch.empty_like(got[0])
    seen = torch.zeros(layers + 4, dtype=torch.int64).pin_memory()
    a = torch.cuda.Stream()
    w.run(got, omega, stream=a)
    torch.cuda.synchronize()
    print(f"[case] window read while open N={N} d={d} ppb={ppb} omega={omega}", flush=True)
    # (streams share a few hardware queues: one that shares the window's sees nothing before the call has ended)
    for b in [torch.cuda.Stream() for _ in range(6)]:
        got.fill_(7.0)
        w.notify.zero_()
        with torch.cuda.stream(b):  # once over, so that nothing is loaded or allocated while the window is open
            seen.copy_(w.notify, non_blocking=True)
            snaps.copy_(got[0])
        torch.cuda.synchronize()
        w.run(got, omega, stream=a)
        read, while_open = set(), []
        with torch.cuda.stream(b):
            for _ in range(20000):  # (the whole call is a few milliseconds; a look takes about 20 us)
                seen.copy_(w.notify, non_blocking=True)
                b.synchronize()
                ready = [l for l in range(layers) if seen[l] != 0 and l not in read]
                if seen[layers + 3] != 0:
                    break
                if ready:
                    l = ready[-1]
                    read.add(l)
                    snaps[l].copy_(got[0, l])
                    seen.copy_(w.notify, non_blocking=True)
                    b.synchronize()
                    if seen[layers + 3] == 0:  # the copy was made before the last transfer of the call
                        while_open.append(l)
        torch.cuda.synchronize()
        if while_open:
            break
    engines = int(w.notify[layers + 2])
    print(f"[case] layers read while the window was open: {while_open} ({engines} engines)", flush=True)
    assert engines == omega
    assert while_open, "no layer was ready before the call had ended: the test has seen nothing"
    for l in while_open:
        wrong = (snaps[l].view(torch.int16) != want[0, l].view(torch.int16)).flatten(2).any(2)
        assert not wrong.any(), f"layer {l}: {int(wrong.sum())} of {wrong.numel()} pages are not what was stored"
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    assert w.c.stats()["status"] == kvc.ST_CORRUPT


# wide engines: nine page tasks per wave and block, eight blocks a turn; narrow ones: 36 tasks, two blocks a turn
@pytest.mark.parametrize("N,d,ppb,omega,layers,n_seq,k", [(16, 32, 144, 1, 2, 8, 8), (13, 64, 150, 3, 2, 8, 8), (2, 32, 132, 1024, 3, 32, 24), (3, 96, 140, 1024, 3, 32, 24)])
def test_turns_of_more_page_tasks_than_one_batch_of_descriptors(N, d, ppb, omega, layers, n_seq, k):
    w = Window(N, d, ppb, layers, n_seq, k, 40)
    want, got = w.buffer(), w.buffer()
    w.run(want, 0)
    print(f"[case] long turns N={N} d={d} ppb={ppb} omega={omega}", flush=True)
    w.run(got, omega)
    torch.cuda.synchronize()
    issued, engines = int(w.notify[layers + 1]), int(w.notify[layers + 2])
    waves, side = (16, 1) if omega <= 256 else (4, 4)
    per_block = -(-(-(-ppb // waves)) // side) * side
    assert min(max(issued // (4 * engines), 1), 8) * per_block > 64
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))


# Wide engines: blocks of one page up to more than the clerk looks up (64) and more than a wave resolves at once (1,024
# pages); from one block per engine and fewer than an engine looks ahead, over runs of one, two and more, to runs of eight.
@pytest.mark.parametrize("N,d,ppb,omega,layers,n_seq,k", [(16, 64, 1, 256, 3, 29, 8), (16, 128, 3, 200, 2, 31, 7), (16, 32, 17, 96, 3, 32, 5), (8, 64, 16, 128, 5, 32, 8), (16, 128, 5, 100, 8, 32, 8),
                                                          (5, 96, 64, 60, 2, 16, 8), (5, 96, 65, 33, 2, 16, 8), (1, 32, 1040, 7, 2, 9, 8), (16, 256, 2, 256, 12, 32, 8), (16, 64, 4, 3, 7, 10, 8),
                                                          (16, 32, 1, 256, 3, 29, 8), (16, 32, 16, 96, 12, 32, 5), (7, 32, 16, 30, 4, 32, 8), (3, 128, 9, 200, 2, 31, 7), (5, 96, 2, 256, 12, 32, 8)])  # one-pass pages, few a block: turn by turn
def test_wide_engines_over_every_length_of_run(N, d, ppb, omega, layers, n_seq, k):
    w = Window(N, d, ppb, layers, n_seq, k, 40)
    want = w.buffer()
    w.run(want, 0)
    plan = [t.clone() for t in (w.tags, w.fetch, w.loc)]
    for om in (omega, 1):
        got = w.buffer()
        print(f"[case] wide engines N={N} d={d} ppb={ppb} omega={om}", flush=True)
        w.run(got, om)
        torch.cuda.synchronize()
        nt = w.notify.cpu().numpy()
        assert nt[layers + 1] == int((w.fetch >= 0).sum()) and nt[layers + 2] == min(om, nt[layers + 1])
        assert (nt[:layers] >= nt[layers]).all() and (nt[:layers] <= nt[layers + 3]).all()
        if om == 1:  # one engine completes the layers in order
            assert (np.diff(nt[:layers]) >= 0).all()
        assert all(torch.equal(a, b) for a, b in zip(plan, (w.tags, w.fetch, w.loc)))
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    assert w.c.stats()["status"] == kvc.ST_CORRUPT


# About ten blocks per engine, and two to an engine's run by the call's own measure: the blocks of the first layer are dealt to
# all 256 engines, one each, and no layer waits for an engine's fourth block.
@pytest.mark.parametrize("N,d,ppb,layers,n_seq,k", [(16, 256, 32, 10, 32, 8), (16, 64, 64, 9, 32, 8)])
def test_the_first_layer_is_ready_in_its_turn(N, d, ppb, layers, n_seq, k):
    w = Window(N, d, ppb, layers, n_seq, k, 40)
    got = w.buffer()
    print(f"[case] first layer N={N} d={d} ppb={ppb}", flush=True)
    first = []
    for _ in range(5):
        w.run(got, 256)
        torch.cuda.synchronize()
        nt = w.notify.cpu().numpy()
        issued, engines = int(nt[layers + 1]), int(nt[layers + 2])
        assert engines == 256 and 2 <= issued // (4 * engines) < 4
        first.append((nt[0] - nt[layers]) / (nt[layers + 3] - nt[layers]))
    # one block of an engine's nine or ten, and the way there; with four in a row it is at least 0.4
    assert np.median(first) < 0.3, first
