"""Workloads of the KV page codec for performance measurement: what a serving program does with it, through the
public binding, from one new block to whole caches.

Three kinds of pass:

swap      compress_blocks of a set of cache blocks into the pool and decompress_blocks of the same blocks into
          paged output: a sequence (or a whole batch) is offloaded and comes back.  Both directions in one pass,
          because payload placement in the pool is unspecified: only decoded pages and descriptors compare.
gather    gather_decompress of one decode step: k predicted blocks of every sequence and layer through a block table.
prefetch  two consecutive decode steps of prefetch_layers (or prefetch_layers_window when omega > 0) into the two
          halves of the L2 prefetch buffer, planner and residency filter included.

Inputs have the distribution of LLaMA-shaped K/V caches: per (K|V, head, channel) a scale exp(N(0, 0.5)), for keys
2 % of the channels ten times larger ("llama"); or channels correlated along the channel index ("ar1")."""
import math

import numpy as np
import torch

from paper_2512_11920_amd import kvc

DEV = "cuda:0"


def listed():
    swap = {"kind": "swap", "N": 16, "d": 128, "ppb": 8, "scheme": 3, "data": "llama", "ids": False, "strided": False}
    step = {"kind": "gather", "N": 16, "d": 128, "ppb": 16, "scheme": 3, "data": "llama"}
    pre = {"kind": "prefetch", "N": 16, "d": 128, "ppb": 16, "scheme": 3, "data": "llama", "policy": 0, "omega": 0}
    return [
        # the Tiny configuration (4 heads x 64): the K and V blocks that one sequence filled in a decode step
        dict(swap, name="tiny_new_block", d=64, ppb=4, blocks=2, ids=True),
        # 70B shape (K and V of 8 heads x 128 per block): the blocks a batch filled in one layer, scattered ids
        dict(swap, name="step_offload", ppb=16, blocks=64, ids=True),
        # the 7B single-layer configuration: 32 heads x 128, sequence 2048, batch 8, K and V
        dict(swap, name="layer_7b", ppb=32, blocks=2048),
        # the 70B GQA cache: 16 of its 80 layers (8 heads x 128, sequence 4096, batch 16, K and V), swapped out and in
        dict(swap, name="cache_70b", blocks=131072),
        # the same shape with the channel-pair mode, 8 layers
        dict(swap, name="cache_70b_pairs", scheme=5, blocks=65536),
        # models with 64 channels per head: 2 KB pages, half a million of them
        dict(swap, name="heads_64", d=64, blocks=65536),
        # 16 x 32 pages, the smallest whole-pass page (1 KB)
        dict(swap, name="pages_1kb", d=32, blocks=65536),
        # 24 tokens x 96 channels: a page with a short last pass, plain INT8 + delta, correlated channels
        dict(swap, name="ragged_24x96", N=24, d=96, ppb=6, scheme=2, data="ar1", blocks=16384),
        # 256 channels, a mode of its own for every block, cache in [block][token][head][channel] order
        dict(swap, name="wide_per_block_modes", d=256, scheme=-1, strided=True, blocks=8192),
        # one decode step of the 70B shape: 80 layers x 64 sequences x 8 predicted blocks (655,360 pages)
        dict(step, name="decode_step_70b", layers=80, seqs=64, k=8, tokens=2048),
        # one layer's prefetch as a layer-pipelined decode loop issues it, blocks that stay where they are
        dict(pre, name="prefetch_layer", policy=1, layers=1, seqs=64, k=8, tokens=2048),
        # all layers through the outstanding-request window
        dict(pre, name="prefetch_window", omega=256, layers=20, seqs=32, k=8, tokens=2048),
    ]


def draw(rng):
    """Another call of the same ranges: any page shape the library takes, any mode, from one block to about 2 GB."""
    kind = rng.choice(["swap", "swap", "swap", "gather", "prefetch"])
    d = rng.choice([32, 64, 64, 96, 128, 128, 128, 160, 192, 224, 256])
    most = 4096 // d
    N = rng.choice([16, 16, 16, min(32, most), 8, rng.randint(1, most)])
    pair_modes = N == 16 and d in (64, 128, 256)
    scheme = rng.choice([3, 3, 3, 5 if pair_modes else 4, 4, 2, 1, 0, -1])
    data = rng.choice(["llama", "llama", "ar1"])
    heads = rng.choice([1, 2, 4, 5, 8, 8, 16, 32])
    case = {"kind": kind, "N": N, "d": d, "ppb": heads, "scheme": scheme, "data": data}
    page = 2 * N * d
    if kind == "swap":
        size = math.exp(rng.uniform(math.log(16e3), math.log(2e9)))
        ids = rng.random() < 0.4
        case.update(ids=ids, strided=rng.random() < 0.3, blocks=max(1, min(int(size / (page * heads)), (1 << 19) if ids else (1 << 21))))
        return case
    case["ppb"] = 2 * min(heads, 8)  # K and V of a block's heads together, as one block of the table
    if case["scheme"] < 0:
        case["scheme"] = 3
    case.update(layers=rng.choice([1, 1, 2, 8, 32, 80]), seqs=rng.randint(1, 64), k=rng.choice([4, 5, 6, 7, 8]), tokens=rng.choice([512, 1024, 2048]))
    if kind == "prefetch":
        case.update(policy=rng.choice([0, 1]), omega=rng.choice([0, 0, int(math.exp(rng.uniform(math.log(16), math.log(4096))))]))
    # pool and output both stay below about 8 GB of FP16 pages
    while case["layers"] * case["seqs"] * max(case["tokens"] // N, 1) * case["ppb"] * page > 8e9 and case["layers"] > 1:
        case["layers"] //= 2
    return case


# ------------------------------------------------------------------------------------------------ inputs


def _blocks(case, gen, n):
    """n blocks of pages, FP16 [n][ppb][N][d]; consecutive blocks of one tensor share their channel scales."""
    N, d, ppb = case["N"], case["d"], case["ppb"]
    c = torch.exp(0.5 * torch.randn((ppb, 1, d), generator=gen, device=DEV))
    keys = torch.arange(ppb, device=DEV)[:, None, None] < (ppb + 1) // 2  # the first half of a block's pages are keys
    c = torch.where(keys & (torch.rand((ppb, 1, d), generator=gen, device=DEV) < 0.02), 10.0 * c, c)
    out = torch.empty((n, ppb, N, d), dtype=torch.float16, device=DEV)
    step = max(1, (1 << 26) // (ppb * N * d))
    for b in range(0, n, step):
        z = torch.randn((min(step, n - b), ppb, N, d), generator=gen, device=DEV)
        if case["data"] == "ar1":
            for i in range(1, d):
                z[..., i] = 0.95 * z[..., i - 1] + 0.3122499 * z[..., i]
            z[..., (5 * d) // 8] *= 10.0
        else:
            z *= c
        out[b:b + step] = z.half()
    return out


def _gen(seed, *idx):
    g = torch.Generator(device=DEV)
    s = int(seed)
    for i in idx:
        s = s * 1000003 + int(i) + 1
    g.manual_seed(s % (1 << 62))
    return g


def _block_modes(case, seed):
    top = 5 if case["N"] == 16 and case["d"] in (64, 128, 256) else 4
    # mostly the full scheme and its extensions, some plain INT8 and raw blocks, as a per-layer policy would ask
    r = np.random.default_rng([int(seed), 7]).random(case["blocks"])
    table = np.array([3, 3, 3, top, top, 4, 2, 1, 1, 0], np.uint8)
    return table[np.minimum((r * 10).astype(np.int64), 9)]


def _swap_inputs(case, seed):
    """The cache (dense [blocks][ppb][N][d]), and the block ids of a scattered call or None."""
    n = case["blocks"]
    have = 4 * n if case["ids"] and n <= 4096 else n
    x = _blocks(case, _gen(seed, 1), have)
    ids = None
    if case["ids"]:
        r = np.random.default_rng([int(seed), 5])
        ids = {"src": r.permutation(have)[:n].astype(np.int32), "pool": r.permutation(n).astype(np.int32), "dst": r.permutation(n).astype(np.int32)}
    return x, ids


def _table_inputs(case, seed):
    """Block table, blocks per sequence, and predictions of two consecutive steps (a sequence's own blocks, with
    replacement): the layout of a paged pool whose blocks were handed out in any order."""
    r = np.random.default_rng([int(seed), 6])
    lo = max(1, case["tokens"] // (4 * case["N"]))
    hi = max(lo, case["tokens"] // case["N"])
    nb = r.integers(lo, hi + 1, size=case["seqs"]).astype(np.int32)
    perm = r.permutation(int(nb.sum())).astype(np.int32)
    table = np.full((case["seqs"], int(nb.max())), -1, np.int32)
    o = 0
    for s in range(case["seqs"]):
        table[s, :nb[s]] = perm[o:o + nb[s]]
        o += int(nb[s])
    preds = [np.minimum((r.random((case["seqs"], case["k"])) * nb[:, None]).astype(np.int32), nb[:, None] - 1) for _ in range(2)]
    l1 = np.maximum(nb - max(1, 256 // case["N"] // 4), 1).astype(np.int32)  # the newest blocks are still in the GPU-local cache
    return table, nb, preds, l1, int(nb.sum())


def _layer(case, seed, layer, per_layer):
    return _blocks(case, _gen(seed, 2, layer), per_layer)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


# ------------------------------------------------------------------------------------------------ the pass


def prepare(case, seed):
    page = case["N"] * case["d"]
    if case["kind"] == "swap":
        x, ids = _swap_inputs(case, seed)
        if case["strided"]:
            x = x.permute(0, 2, 1, 3).contiguous()  # [block][token][head][channel]
        c = kvc.Codec(case["N"], case["d"], case["ppb"], max(case["scheme"], 0) if case["scheme"] >= 0 else 3)
        if case["strided"]:
            c.set_cache_layout(case["N"] * case["ppb"] * case["d"], case["d"], case["ppb"] * case["d"])
        n = case["blocks"]
        c.alloc_pool(n, n * case["ppb"] * page * (2 if case["scheme"] <= 0 else 1) + 4096, DEV)
        out = torch.empty((n,) + tuple(x.shape[1:]), dtype=torch.float16, device=DEV)
        return {"kind": "swap", "c": c, "x": x, "out": out, "n": n, "ids": {k: _dev(v) for k, v in ids.items()} if ids else {"src": None, "pool": None, "dst": None},
                "modes": _dev(_block_modes(case, seed)) if case["scheme"] < 0 else None, "sizes": c.desc.view(torch.int32).view(-1, 4)[:, 2:]}
    table, nb, preds, l1, per_layer = _table_inputs(case, seed)
    c = kvc.Codec(case["N"], case["d"], case["ppb"], case["scheme"])
    L = case["layers"]
    c.alloc_pool(L * per_layer, L * per_layer * case["ppb"] * page * (2 if case["scheme"] == 0 else 1) + 4096, DEV)
    for l in range(L):
        x = _layer(case, seed, l, per_layer)
        c.compress_blocks(x, n=per_layer, pool_ids=torch.arange(l * per_layer, (l + 1) * per_layer, dtype=torch.int32, device=DEV))
    slots = L * case["seqs"] * case["k"]
    s = {"kind": case["kind"], "c": c, "table": _dev(table), "preds": [_dev(p) for p in preds], "L": L, "per_layer": per_layer}
    if case["kind"] == "gather":
        s["out"] = torch.empty((slots, case["ppb"], case["N"], case["d"]), dtype=torch.float16, device=DEV)
        return s
    s["l2"] = torch.zeros((2, slots, case["ppb"], case["N"], case["d"]), dtype=torch.float16, device=DEV)
    s["tags"] = torch.empty(2 * slots, dtype=torch.int32, device=DEV)
    s["plan"] = [(torch.empty(slots, dtype=torch.int32, device=DEV), torch.empty(slots, dtype=torch.int32, device=DEV)) for _ in range(2)]
    s["l1"], s["seqs"], s["k"], s["omega"] = _dev(l1), case["seqs"], case["k"], case["omega"]
    c.set_prefetch_policy(case["policy"])
    if case["omega"]:
        s["notify"] = torch.zeros(L + 4, dtype=torch.int64, device=DEV)
        s["work"] = torch.empty(kvc.window_workspace(slots, L), dtype=torch.uint8, device=DEV)
    return s


def run(s):
    c = s["c"]
    if s["kind"] == "swap":
        c.reset_pool()
        c.compress_blocks(s["x"], n=s["n"], src_ids=s["ids"]["src"], pool_ids=s["ids"]["pool"], block_scheme=s["modes"])
        c.decompress_blocks(s["out"], n=s["n"], pool_ids=s["ids"]["pool"], dst_ids=s["ids"]["dst"])
        return {"pages": s["out"], "sizes": s["sizes"]}  # sizes: scale bits, and payload size and mode, of every page
    if s["kind"] == "gather":
        c.gather_decompress(s["out"], s["table"], s["preds"][0], s["L"], s["per_layer"])
        return {"pages": s["out"]}
    c.prefetch_reset(s["tags"], s["seqs"], s["k"], s["L"])
    for half, pred in enumerate(s["preds"]):
        fetch, loc = s["plan"][half]
        if s["omega"]:
            c.prefetch_layers_window(s["l2"], s["tags"], fetch, loc, s["table"], pred, s["L"], s["per_layer"], half, s["omega"], s["notify"], s["work"], l1_first=s["l1"])
        else:
            c.prefetch_layers(s["l2"], s["tags"], fetch, loc, s["table"], pred, s["L"], s["per_layer"], half, l1_first=s["l1"])
    return {"pages": s["l2"], "tags": s["tags"], "plan": s["plan"]}


# ------------------------------------------------------------------------------------------------ what it costs at least

#: payload bytes over FP16 bytes, by requested mode, of the two kinds of input (the page shape moves it by a few percent)
_PAYLOAD = {"llama": {0: 1.0, 1: 0.5, 2: 0.45, 3: 0.45, 4: 0.44, 5: 0.395, -1: 0.5}, "ar1": {0: 1.0, 1: 0.5, 2: 0.3, 3: 0.3, 4: 0.345, 5: 0.345, -1: 0.41}}


def work(case):
    page = 2.0 * case["N"] * case["d"]
    stored = page * _PAYLOAD[case["data"]][case["scheme"]] + 16
    if case["kind"] == "swap":
        pages = case["blocks"] * case["ppb"]
        return {"bytes": 2 * pages * (page + stored), "flops": 4.0 * pages * page / 2}
    pages = case["layers"] * case["seqs"] * case["k"] * case["ppb"]
    if case["kind"] == "prefetch":
        pages *= 2 * 0.85  # two steps; a part of the predictions is resident already
    return {"bytes": pages * (page + stored), "flops": 2.0 * pages * page / 2}


def tolerance(case):
    """Codes, sizes and scales are integers or correctly rounded quotients, and a decoded value is one rounded product
    and one rounded conversion: every correct implementation gives the same bits."""
    return "exact"


# ------------------------------------------------------------------------------------------------ in 64 bits


def _through(x, raw=None):
    """What a page [..., N, d] is after quantization to 127 steps of its largest magnitude and back, in 64 bits."""
    x = x.double()
    s = x.abs().amax(dim=(-2, -1), keepdim=True) / 127.0
    y = torch.where(s > 0, torch.round(x / torch.where(s > 0, s, torch.ones_like(s))) * s, torch.zeros_like(x))
    return y if raw is None else torch.where(raw[:, None, None, None], x, y)


def _through_blocks(x, raw=None):
    out = torch.empty(x.shape, dtype=torch.float64, device=DEV)
    step = max(1, (1 << 27) // x[0].numel())
    for b in range(0, x.shape[0], step):
        out[b:b + step] = _through(x[b:b + step], None if raw is None else raw[b:b + step])
    return out


def _plan(case, table, preds, l1):
    """Per step and sequence: which logical placement (slot -> pool block within a layer) the residency filter leaves,
    starting from an empty buffer.  The same in every layer."""
    S, k = case["seqs"], case["k"]
    held = [[{} for _ in range(S)] for _ in range(2)]  # slot -> block, per half and sequence
    for half in range(2):
        for q in range(S):
            seen, free = set(held[0][q].values()) if half else set(), 0
            for j in range(k):
                lb = int(preds[half][q, j])
                e = int(table[q, lb])
                if lb >= l1[q] or e < 0 or e in seen:
                    continue
                seen.add(e)
                held[half][q][j if case["policy"] == 0 else free] = e
                free += 1
    return held


def exact(case, seed):
    if case["kind"] == "swap":
        x, ids = _swap_inputs(case, seed)
        raw = _dev(_block_modes(case, seed) == 0) if case["scheme"] < 0 else None
        if ids:
            x = x[_dev(ids["src"]).long()]
        y = x.double() if case["scheme"] == 0 else _through_blocks(x, raw)
        del x
        if ids:
            z = torch.empty_like(y)
            z[_dev(ids["dst"]).long()] = y
            y = z
        return {"pages": y.permute(0, 2, 1, 3) if case["strided"] else y, "sizes": None}
    table, nb, preds, l1, per_layer = _table_inputs(case, seed)
    L, S, k = case["layers"], case["seqs"], case["k"]
    halves = 1 if case["kind"] == "gather" else 2
    out = torch.zeros((halves, L, S * k, case["ppb"], case["N"], case["d"]), dtype=torch.float64, device=DEV)
    if halves == 1:
        where = [(torch.arange(S * k, device=DEV), _dev(table[np.arange(S)[:, None], preds[0]].reshape(-1)).long())]
    else:
        where = []
        for held in _plan(case, table, preds, l1):
            pairs = [(q * k + slot, e) for q in range(S) for slot, e in held[q].items()]
            where.append((torch.tensor([p[0] for p in pairs], dtype=torch.long, device=DEV), torch.tensor([p[1] for p in pairs], dtype=torch.long, device=DEV)))
    for l in range(L):
        x = _layer(case, seed, l, per_layer)
        for h, (slots, blocks) in enumerate(where):
            if slots.numel():
                y = x[blocks]
                out[h, l].index_copy_(0, slots, y.double() if case["scheme"] == 0 else _through(y))
    if halves == 1:
        return {"pages": out.view(L * S * k, case["ppb"], case["N"], case["d"])}
    return {"pages": out.view(2, L * S * k, case["ppb"], case["N"], case["d"]), "tags": None, "plan": None}
