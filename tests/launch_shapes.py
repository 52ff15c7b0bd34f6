"""What the library launches for a call, found without a GPU: libkvc.so is loaded on top of a HIP runtime that only writes
its launches down (tests/launch_recorder.cpp), in a process of its own, and called with addresses nobody looks at.

    launches([call, ...]) -> [[Launch, ...], ...]

A call is a dict: op ("compress", "decompress", "gather", "prefetch"), N, d, ppb, scheme, n (blocks) and, by op, lists
(names of the id lists it passes), mixed (a mode per block), layers, seqs, k, omega; desc: pages of its descriptor table, where that is not to be a
huge one; memory: (hipMemoryType, device) of its pool; context: a name, where calls share one (the first says what it is; it lives as
long as its process).  "reset" and "restore" are calls too.  Launch.line: kept_units or near_bytes of an encoder or decoder, in bytes of the pool."""
import collections
import ctypes as C
import json
import os
import re
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def large_encoder_pages(N, d, scheme):
    """The smallest call that takes the encoder's large launch shape (scheme: 0..5 for the call, or "mixed": one per block)."""
    passes = -(-N * d // 512)
    if scheme in (0, 1):  # plain: no packets to wait for
        return 8193 if passes <= 2 else 2049
    if passes == 4:
        whole = N * d == 2048 and (N, d) in ((16, 128), (32, 64), (8, 256))  # these have encoders of their own for modes 3 and 5
        return 32769 if whole and scheme == 5 else 16385 if whole and scheme == 3 else 4097
    return {1: 32769, 2: 16385, 3: 8193, 5: 3073, 6: 3073, 7: 4097, 8: 4097}[passes]


def large_decoder_pages(N, d):
    """The smallest call whose decoder waves take several pages (pages of one or two passes; None: there is none)."""
    passes = -(-N * d // 512)
    return 4096 * passes + 1 if passes <= 2 else None


Launch = collections.namedtuple("Launch", "kernel params grid block lds line")  # params: the kernel's template arguments


def _recorder():
    """Build the recorder (once per process)."""
    global _dir
    if "_dir" not in globals():
        _dir = tempfile.TemporaryDirectory()
        versions = os.path.join(_dir.name, "v")
        with open(versions, "w") as f:
            f.write("hip_4.2 { global: *; };\n")
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-Wno-attributes",
                        "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2512_11920_amd", "csrc"),
                        "-Wl,-soname,libamdhip64.so.7", f"-Wl,--version-script={versions}", "-o", os.path.join(_dir.name, "rec.so"),
                        os.path.join(ROOT, "tests", "launch_recorder.cpp")], check=True)
    return os.path.join(_dir.name, "rec.so")


def launches(calls):
    from paper_2512_11920_amd import build

    p = subprocess.run([sys.executable, os.path.abspath(__file__), _recorder(), build.LIB], input=json.dumps(calls), capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stderr[-3000:]
    out = []
    for rows in json.loads(p.stdout):
        out.append([])
        for mangled, grid, block, lds, line in rows:
            name = re.search(r"\d(k_[a-z_]+?)(?:I|E|PK|PN|P[a-z]|N\d|v)", mangled).group(1)
            args = re.search(re.escape(name) + r"I(.*?)EEv", mangled)
            nums = re.findall(r"L[ib](n?)(\d+)E", args.group(1) + "E") if args else []
            out[-1].append(Launch(name, tuple(-int(v) if s else int(v) for s, v in nums), grid, block, lds, line))
    return out


def _main(recorder, lib):
    rec = C.CDLL(recorder, mode=C.RTLD_GLOBAL)
    rec.rec_kernel.restype, rec.rec_line.restype = C.c_char_p, C.c_ulonglong
    L = C.CDLL(lib)
    at, big, i32, i64 = C.c_void_p(1 << 20), C.c_uint64(1 << 40), C.c_int32, C.c_int64
    out, kept = [], {}
    for c in json.load(sys.stdin):
        cfg, ctx = (i32 * 4)(c["N"], c["d"], c["ppb"], c.get("scheme", 3)), C.c_void_p()
        n, lists = c.get("n", 0), c.get("lists", ())
        rec.rec_memory(*c.get("memory", (2, 0)))
        ctx = kept.get(c.get("context"), ctx)
        assert ctx or L.kvc_create(C.byref(ctx), cfg) == 0 and L.kvc_bind_pool(ctx, at, big, at, C.c_uint64(c.get("desc", 1 << 40))) == 0
        if "context" in c:
            kept[c["context"]] = ctx
        rec.rec_clear()
        opt = lambda name: at if name in lists else None
        if c["op"] == "compress" and c.get("mixed"):
            rc = L.kvc_compress_blocks_mixed(ctx, at, i64(n), opt("src"), opt("pool"), at, i32(n), None)
        elif c["op"] == "compress":
            rc = L.kvc_compress_blocks(ctx, at, i64(n), opt("src"), opt("pool"), i32(n), None)
        elif c["op"] == "decompress":
            rc = L.kvc_decompress_blocks(ctx, at, i64(n), opt("pool"), opt("dst"), i32(n), None)
        elif c["op"] == "reset":
            rc = L.kvc_reset_pool(ctx, None)
        elif c["op"] == "restore":
            rc = L.kvc_restore_pool(ctx, C.c_uint64(1 << 20), None)
        elif c["op"] == "gather":
            rc = L.kvc_gather_decompress(ctx, at, at, i32(64), at, i32(c["seqs"]), i32(c["k"]), i32(c["layers"]), i64(64), None)
        else:
            args = [ctx, at, at, at, at, at, i32(64), at, None, i32(c["seqs"]), i32(c["k"]), i32(c["layers"]), i32(0), i32(c["layers"]), i64(64), i32(0)]
            if c["omega"]:
                rc = L.kvc_prefetch_layers_window(*args, i32(c["omega"]), at, at, big, None)
            else:
                rc = L.kvc_prefetch_layers(*args, None)
        assert rc == 0, (rc, c)
        rows = []
        for i in range(rec.rec_count()):
            g, b, l = C.c_uint(), C.c_uint(), C.c_uint()
            rec.rec_shape(i, C.byref(g), C.byref(b), C.byref(l))
            rows.append((rec.rec_kernel(i).decode(), g.value, b.value, l.value, rec.rec_line(i)))
        out.append(rows)
        if "context" not in c:
            L.kvc_destroy(ctx)
    print(json.dumps(out))


if __name__ == "__main__":
    _main(*sys.argv[1:])
