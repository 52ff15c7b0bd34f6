"""Rules of the launches, found without a GPU (tests/launch_shapes.py): which kernel a call gets, in which shape."""
from launch_shapes import large_decoder_pages, large_encoder_pages, launches


def decode(N, d, ppb, n, **kw):
    return dict(op="decompress", N=N, d=d, ppb=ppb, n=n, **kw)


def test_only_calls_that_decode_a_whole_range_limit_their_workgroups():
    """Large calls: the limit on a compute unit's decoder workgroups (LDS that nothing uses) slows down lists with blocks left
    out, and holds for calls without lists only.  The milder one of middle calls of large pages is for all."""
    shapes = [(16, 128), (16, 160), (16, 192), (13, 256), (16, 256)]
    whole = launches([decode(N, d, 1, 1 << 17) for N, d in shapes])
    assert all(l[0].kernel == "k_decompress" and l[0].lds > 0 for l in whole)
    # workgroups a compute unit holds: by pages of the call and KB a page
    for n, groups in ((8191, (0, 0, 0, 0, 0)), (8192, (0, 0, 6, 6, 6)), (24575, (0, 0, 6, 6, 6)), (24576, (6, 6, 6, 6, 4)), (1 << 20, (6, 6, 6, 6, 4))):
        calls = [decode(N, d, 1, n) for N, d in shapes] + ([decode(N, d, 1, n, lists=["pool"]) for N, d in shapes] if n < 24576 else [])
        for c, g, l in zip(calls, groups * 2, launches(calls)):
            N, d = c["N"], c["d"]
            own = 4 * (-(-N * d // 512) * 520 + 31) // 16 * 16
            assert (l[0].lds > 0) == (g > 0) and (g == 0 or 160 * 1024 // (own + l[0].lds) == g), (N, d, n, l[0])
    named = [decode(N, d, ppb, (1 << 17) // ppb, lists=lists) for N, d in shapes for ppb in (1, 8) for lists in (["pool"], ["dst"], ["pool", "dst"])]
    named += [dict(op="gather", N=N, d=d, ppb=8, seqs=64, k=8, layers=32) for N, d in shapes]
    named += [dict(op="prefetch", N=N, d=d, ppb=8, seqs=64, k=8, layers=32, omega=0) for N, d in shapes]
    for call, l in zip(named, launches(named)):
        assert l[-1].kernel == "k_decompress" and l[-1].lds == 0, call


def test_the_counting_planner_stays_with_few_sequences():
    """One workgroup per layer plans and counts the transfers of up to two rounds of rows (k <= 8), or one (k <= 32)."""
    few = [(8, 1), (8, 64), (5, 64), (16, 16), (9, 16), (32, 8), (17, 8)]
    many = [(8, 65), (8, 128), (1, 65), (16, 17), (16, 64), (32, 9), (17, 32)]
    calls = [dict(op="prefetch", N=16, d=128, ppb=2, seqs=s, k=k, layers=3, omega=64) for k, s in few + many]
    for (k, s), l in zip(few + many, launches(calls)):
        lanes = 8 if k <= 8 else 16 if k <= 16 else 32
        if (k, s) in few:
            assert [x.kernel for x in l[:2]] == ["k_prefetch_plan_count", "k_window_place"] and l[0].grid == 3, (k, s)
        else:
            assert [x.kernel for x in l[:3]] == ["k_prefetch_plan", "k_window_count", "k_window_place"] and l[0].grid == -(-3 * s // (64 // lanes)), (k, s)
        assert l[0].params == (lanes,)


def test_a_prefetch_step_is_planned_by_rows_and_decoded_by_pages():
    """Whatever the rows: the decoder gets a wave per page, also where a row has one, or one more than fill a workgroup."""
    for k, ppb, seqs, layers in ((1, 1, 1, 1), (1, 1, 8192, 1), (1, 9, 910, 1), (4, 1, 2048, 1), (8, 1, 1024, 1), (8, 16, 64, 1), (8, 16, 4, 2), (8, 33, 3, 1), (9, 4, 6, 2), (32, 2, 5, 1)):
        plan, decoder = launches([dict(op="prefetch", N=16, d=128, ppb=ppb, seqs=seqs, k=k, layers=layers, omega=0, desc=layers * 64 * ppb)])[0]
        lanes = 8 if k <= 8 else 16 if k <= 16 else 32
        assert plan.kernel == "k_prefetch_plan" and plan.params == (lanes,) and plan.grid == -(-layers * seqs // (64 // lanes))
        assert decoder.kernel == "k_decompress" and decoder.grid == -(-layers * seqs * k * ppb // (decoder.block // 64))


def test_wide_engines_of_small_blocks_go_turn_by_turn():
    """Up to 16 one-pass pages a block; blocks of more, and of larger pages, have engines that look ahead."""
    small = [(16, 32, 1), (16, 32, 16), (7, 32, 8), (8, 64, 16), (5, 96, 2), (3, 128, 16), (2, 256, 16)]
    other = [(16, 32, 17), (7, 32, 64), (32, 32, 1), (16, 64, 16), (6, 96, 16), (16, 128, 1), (16, 256, 16)]
    calls = [dict(op="prefetch", N=N, d=d, ppb=ppb, seqs=32, k=8, layers=3, omega=64) for N, d, ppb in small + other]
    for (N, d, ppb), l in zip(small + other, launches(calls)):
        want = "k_decompress_window" if (N, d, ppb) in small else "k_decompress_window_wide"
        assert l[-1].kernel == want and l[-1].block == 1024 and l[-1].grid == 64, (N, d, ppb, l[-1])
    many = launches([dict(c, omega=600) for c in calls])  # more than the device holds of the wide kind
    assert all(l[-1].kernel == "k_decompress_window" and l[-1].block == 256 for l in many)


def test_encoder_workgroups_of_16_waves_end_where_they_stop_being_resident():
    """Four-pass pages with the mode read at run time: 4,096 pages of a wave each fill the chip."""
    calls = [dict(op="compress", N=N, d=d, ppb=1, n=n, **kw) for N, d in ((16, 128), (15, 128), (32, 64), (8, 256)) for n in (4096, 4097) for kw in (dict(mixed=True), dict(scheme=2), dict(scheme=4))]
    for c, l in zip(calls, launches(calls)):
        D, NP, partial, waves, ppw, scheme = l[0].params
        assert scheme < 0 and ((waves, ppw) == (16, 1)) == (c["n"] == 4096), (c, l[0])


def test_where_the_large_launch_shapes_begin():
    """large_encoder_pages and large_decoder_pages, from which tests take their sizes, say what the library does."""
    shapes = [(N, d) for d in range(32, 257, 32) for N in sorted({16, 1, 8, 32, *(512 * p // d + e for p in range(1, 9) for e in (0, 1))}) if 1 <= N <= 4096 // d]
    kinds = [(N, d, sc) for N, d in shapes for sc in (0, 1, 2, 3, 4, "mixed")] + [(16, d, 5) for d in (64, 128, 256)]
    encode = lambda N, d, sc, n: dict(op="compress", N=N, d=d, ppb=1, n=n, scheme=3 if sc == "mixed" else sc, mixed=sc == "mixed")
    calls = [encode(N, d, sc, n) for N, d, sc in kinds for n in (large_encoder_pages(N, d, sc) - 1, large_encoder_pages(N, d, sc), 1 << 20)]
    got = [l[0] for l in launches(calls)]
    for i, kind in enumerate(kinds):
        below, first, large = got[3 * i:3 * i + 3]
        assert first.params == large.params != below.params, (kind, below, first, large)
    several = [(N, d) for N, d in shapes if large_decoder_pages(N, d)]
    for N, d in several:
        below, first = (l[0] for l in launches([decode(N, d, 1, n) for n in (large_decoder_pages(N, d) - 1, large_decoder_pages(N, d))]))
        assert below.params[-1] == 1 and first.params[-1] == (4 if N * d <= 512 else 2), (N, d)


def test_which_calls_read_past_the_last_level_cache():
    """Decoders of a whole range of 608 MiB to 4.25 GiB of pages, whatever their shape, from a pool in the device's own memory; no call that
    names its blocks.  Encoders keep the first 208 MB of such a pool, every call."""
    plain, kept = (1 << 64) - 1, 208 << 20
    calls, want = [], []
    for N, d, ppb in ((16, 128, 8), (16, 128, 1), (16, 32, 8), (24, 96, 6), (7, 32, 3), (16, 256, 16)):
        block = 2 * N * d * ppb
        first, last = -(-(608 << 20) // block), (4352 << 20) // block
        for n, line in ((1, plain), (first - 1, plain), (first, kept), (last, kept), (last + 1, plain)):
            calls.append(decode(N, d, ppb, n))
            want.append(line)
        for lists in (["pool"], ["dst"], ["pool", "dst"]):
            calls.append(decode(N, d, ppb, first, lists=lists))
            want.append(plain)
        calls += [decode(N, d, ppb, first, memory=m) for m in ((1, 0), (2, 1))]  # behind the host link, or the link to another device
        want += [plain] * 2
        for lists in ([], ["pool"], ["src", "pool"]):
            calls += [dict(op="compress", N=N, d=d, ppb=ppb, n=first, lists=lists, scheme=s, memory=m) for s in (0, 3) for m in ((2, 0), (1, 0), (2, 1))]
            want += [kept, 0, 0] * 2
    calls += [dict(op="gather", N=16, d=128, ppb=16, seqs=64, k=8, layers=32), dict(op="prefetch", N=16, d=128, ppb=16, seqs=64, k=8, layers=32, omega=0)]
    want += [plain] * 2
    for call, line, l in zip(calls, want, launches(calls)):
        assert l[-1].kernel == ("k_compress" if call["op"] == "compress" else "k_decompress") and l[-1].line == line, (call, l)
        if l[-1].kernel == "k_decompress":  # the kernel that asks where a payload lies, for these calls alone
            assert l[-1].params[3] == (line == kept), (call, l)


def test_what_waits_in_the_last_level_cache_is_bounded():
    """Payloads wait there until their context fetches or gives them up.  Those of another are stored past it unless both fit: 208 MB, of
    which a block of 128 pages of 16 x 128 is counted as 256 KB."""
    all_of_it = (208 << 20) // (128 * 2048)
    shape = dict(N=16, d=128, ppb=128)

    def compress(context, n, **kw):
        return dict(op="compress", context=context, n=n, **shape, **kw)

    fetches = [decode(16, 128, 128, 1), decode(16, 128, 128, 1, lists=["pool"]), dict(op="gather", seqs=1, k=1, layers=1, **shape), dict(op="prefetch", seqs=1, k=1, layers=1, omega=0, **shape),
               dict(op="prefetch", seqs=1, k=1, layers=1, omega=4, **shape), dict(op="reset", **shape), dict(op="restore", **shape)]
    calls, want = [], []

    def then(call, keeps=None):
        calls.append(call)
        want.append(keeps)

    for f in fetches:
        then(compress("a", 4 * all_of_it), True)  # one context: all calls, whatever their size
        then(compress("a", 1), True)
        then(compress("b", 1), False)
        then(compress("b", 1), False)
        then(dict(f, context="a"))
        then(compress("b", all_of_it - 4), True)  # a and b beside one another
        then(compress("a", 4, lists=["src", "pool"]), True)
        then(compress("a", 1), False)
        then(compress("b", 1), False)
        then(compress("c", 1, memory=(1, 0)), False)  # c is behind the host link: takes no part
        then(dict(f, context="c"))
        then(compress("d", 1), False)
        then(dict(f, context="b"))
        then(compress("d", all_of_it - 4), True)
        then(dict(f, context="a"))
        then(compress("d", 1), True)
        then(compress("a", 4), False)
        then(dict(f, context="d"))
    for call, keeps, l in zip(calls, want, launches(calls)):
        if keeps is not None:
            assert l[-1].line == (208 << 20 if keeps else 0), call
    # a context that ends gives its part back
    ended = [compress("a", 1), dict(compress("", all_of_it)), compress("a", 1), compress("b", 1)]
    del ended[1]["context"]
    assert [l[-1].line for l in launches(ended)] == [208 << 20, 0, 208 << 20, 208 << 20]
    ended = [dict(compress("", all_of_it)), compress("a", all_of_it)]
    del ended[0]["context"]
    assert [l[-1].line for l in launches(ended)] == [208 << 20] * 2
    # and calls of fewer than 128 pages leave none there
    few = [dict(op="compress", N=N, d=d, ppb=1, n=n, lists=lists, scheme=scheme) for N, d in ((16, 32), (16, 128), (7, 96), (16, 256)) for scheme in (1, 3)
           for lists in ([], ["src", "pool"]) for n in (1, 64, 127, 128, 129)]
    for call, l in zip(few, launches(few)):
        assert l[-1].line == (208 << 20 if call["n"] >= 128 else 0), call
