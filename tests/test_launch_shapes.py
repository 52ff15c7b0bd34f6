"""Rules of the launches, found without a GPU (tests/launch_shapes.py): which kernel a call gets, in which shape."""
from launch_shapes import launches


def decode(N, d, ppb, n, **kw):
    return dict(op="decompress", N=N, d=d, ppb=ppb, n=n, **kw)


def test_only_calls_that_decode_a_whole_range_limit_their_workgroups():
    """The limit on a compute unit's decoder workgroups (LDS that nothing uses) slows down lists with blocks left out."""
    shapes = [(16, 128), (16, 160), (16, 192), (13, 256), (16, 256)]
    whole = launches([decode(N, d, 1, 1 << 17) for N, d in shapes])
    assert all(l[0].kernel == "k_decompress" and l[0].lds > 0 for l in whole)
    named = [decode(N, d, ppb, (1 << 17) // ppb, lists=lists) for N, d in shapes for ppb in (1, 8) for lists in (["pool"], ["dst"], ["pool", "dst"])]
    named += [dict(op="gather", N=N, d=d, ppb=8, seqs=64, k=8, layers=32) for N, d in shapes]
    named += [dict(op="prefetch", N=N, d=d, ppb=8, seqs=64, k=8, layers=32, omega=0) for N, d in shapes]
    for call, l in zip(named, launches(named)):
        assert l[-1].kernel == "k_decompress" and l[-1].lds == 0, call
