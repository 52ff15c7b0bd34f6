"""Rules for the generated gfx950 code that a GPU run cannot be trusted to catch.

(1) 64-bit shifts by a per-lane amount.  One build of one encoder instantiation wrote wrong payload bytes
for a few pages in a thousand, only when workgroups shared a compute unit, and every recompile that moved
registers made it vanish; the working hypothesis (not established from evidence kept in this tree) is that
v_lshlrev_b64 / v_lshrrev_b64 misread a shift count held in the last VGPR of the wave's allocation.  Which
register holds the count is the compiler's choice, so the kernels contain no 64-bit shift by a register
amount at all (v_ashrrev_i64 is kept out with them): counts that are immediates or scalar registers are fine.

(2) Workgroup barriers of the prefetch window's engines stay out of nested loops (see the test).

(3) Buffer stores of more than 64 bits take no offset from a scalar register.  Such a store reads its data registers
late, one wait state has to pass before they are written again, and the compiler inserts it only for stores without a
scalar offset; without it lanes store what the next instructions compute.

(4) The window's engines write pages through the XCD's L2 (device scope): a block is published by waiting for its
stores, and a store without that scope would leave a consumer that polls the ready stamp with stale bytes.

(5) A block of the window is published by counters that move after all waves of its engine have waited for their stores
and met: the wait stands right before that meeting.

(6) An engine counts itself out of the window only when its layer stamps are in memory: whoever sees the stamp that closes
the window may read the stamps of all layers."""
import concurrent.futures
import os
import re

import pytest

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    """gfx950 assembly of every compilation unit that holds kernels, by unit name."""
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not installed")
    from paper_2512_11920_amd import build

    d = tmp_path_factory.mktemp("asm")
    units = [(src, defs, obj) for src, defs, obj in build.UNITS if src != "kvc_api.hip"]
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        futs = {obj: ex.submit(build.compile_unit, src, defs, str(d / (obj + ".s")), (), True) for src, defs, obj in units}
        texts = {obj: open(f.result()).read() for obj, f in futs.items()}
    for name, text in texts.items():
        assert ".amdgcn_target" in text and "gfx950" in text, name
    return texts


def test_no_64_bit_shift_by_a_vector_register(asm):
    for name, text in asm.items():
        hits = re.findall(r"^\s*v_(?:lshlrev_b64|lshrrev_b64|ashrrev_i64)\s+v\[\d+:\d+\],\s*v\d+,.*$", text, flags=re.M)
        assert not hits, f"{name}: {len(hits)} 64-bit shifts by a VGPR amount, e.g. {hits[0].strip()}"


def test_no_kernel_spills_registers_to_memory(asm):
    """Every kernel keeps its working set in registers: scratch (private memory) use would mean spills,
    which cost HBM traffic the byte accounting does not know about."""
    n = 0
    for name, text in asm.items():
        for m in re.finditer(r"\.name:\s+(\S+).*?\.private_segment_fixed_size:\s*(\d+)", text, flags=re.S):
            n += 1
            assert int(m.group(2)) == 0, f"{name}: {m.group(1)} uses {m.group(2)} bytes of scratch memory"
    assert n > 20


def _kernels(text, name):
    """(label, instructions) of every kernel of a unit whose label contains `name`."""
    for m in re.finditer(rf"^(_Z\w*{name}\w*):[^\n]*\n(.*?)^\.Lfunc_end", text, flags=re.S | re.M):
        yield m.group(1), m.group(2)


WIDE_STORE = r"^\s*((?:buffer|global|flat|scratch)_store_(?:dwordx[34]|b96|b128))\s+([^;\n]*)"


def test_no_wide_buffer_store_with_a_scalar_offset(asm):
    for name, text in asm.items():
        stores = [m.group(2) for m in re.finditer(WIDE_STORE, text, flags=re.M) if m.group(1).startswith("buffer")]
        if name.startswith("kvc_codec"):
            assert len(stores) > 40, f"{name}: the window's decoders of every page shape write with buffer stores"
        for args in stores:  # data, lane offset or off, resource, scalar offset [modifiers]
            soffset = re.fullmatch(r"v\[\d+:\d+\],\s*(?:v\d+|off),\s*s\[\d+:\d+\],\s*(\S+)(?:\s.*)?", args.strip())
            assert soffset and soffset.group(1) == "0", f"{name}: {args}"


def test_window_engines_write_pages_through_to_memory(asm):
    seen = 0
    for name, text in asm.items():
        for kernel, body in _kernels(text, "k_decompress_window"):
            seen += 1
            stores = [(m.group(1), m.group(2).split()) for m in re.finditer(WIDE_STORE, body, flags=re.M)]
            # packed, INT8, raw and zero-filled pages, with the packed ones in several variants
            assert len(stores) >= 5, kernel
            for op, args in stores:
                assert op == "buffer_store_dwordx4" and "sc1" in args, f"{kernel}: {op} {' '.join(args)}"
    assert seen >= 2 * (64 + 16), "wide and narrow engines of every page shape"


def _waits_for_memory(lines, i):
    """Whether the instruction at line i stands behind an s_waitcnt vmcnt(0), with no access to memory and no place that is
    jumped to in between."""
    for l in reversed(lines[:i]):
        if re.search(r"^\s*s_waitcnt\b.*vmcnt\(0\)", l):
            return True
        if re.match(r"\.LBB", l) or re.match(r"\s*(?:global|buffer|flat|scratch)_", l) or "s_barrier" in l:
            return False
    return False


def test_engines_leave_the_window_after_their_stamps(asm):
    seen = 0
    for name, text in asm.items():
        for kernel, body in _kernels(text, "k_decompress_window"):
            lines = body.split("\n")
            counts = [i for i, l in enumerate(lines) if re.match(r"\s*global_atomic_add v\d+, .*offset:128 sc0", l)]  # hdr->done
            assert counts, f"{kernel}: no count of completed blocks"
            stamps = [l for l in lines if re.match(r"\s*global_store_dwordx2 .*sc1", l)]
            assert len(stamps) >= 2, f"{kernel}: a layer's stamp and the closing one"
            assert all(_waits_for_memory(lines, i) for i in counts), f"{kernel}: blocks counted with stores in flight"
            seen += 1
    assert seen >= 2 * (64 + 16)


def test_window_engines_meet_with_their_stores_in_memory(asm):
    seen = {"turn": 0, "ahead": 0}
    for name, text in asm.items():
        for kernel, body in _kernels(text, "k_decompress_window"):
            lines = body.split("\n")
            stores = [i for i, l in enumerate(lines) if re.match(r"\s*buffer_store_dwordx4 ", l)]
            barriers = [i for i, l in enumerate(lines) if "s_barrier" in l]
            counters = [i for i, l in enumerate(lines) if re.match(r"\s*global_atomic_add ", l)]  # ticket, a layer's pending blocks, done
            if "window_wide" in kernel:
                # two meetings (before the loop and in it) of two barriers each, and the second of each is behind the wait
                assert len(barriers) == 4 and sum(_waits_for_memory(lines, i) for i in barriers) == 2, kernel
                seen["ahead"] += 1
            else:
                # the barrier between the page stores and the counters
                first = min(i for i in counters if i > stores[-1])
                between = [i for i in barriers if stores[-1] < i < first]
                assert between and _waits_for_memory(lines, between[0]), kernel
                seen["turn"] += 1
    assert seen["turn"] >= 64 + 16 + 10 and seen["ahead"] >= 64 + 16, seen


def test_window_engines_keep_their_barriers_out_of_nested_loops(asm):
    """The transfer engines of the prefetch window loop over queue entries with workgroup barriers in the
    loop body and single-lane bookkeeping between them.  The compiler must lay that out as one loop whose
    barriers every wave meets with all lanes: a barrier inside a loop nested in the engines' loop means
    the single-lane work was hoisted across the back edge and the other lanes run ahead to the next
    barrier (the workgroup then waits for ever).  Checked on the generated code: in every window kernel
    all s_barrier instructions sit at loop depth 0 or 1."""
    seen = 0
    for name, text in asm.items():
        lines = text.split("\n")
        for st in [i for i, l in enumerate(lines) if re.match(r"^_Z\w*k_decompress_window\w*:", l)]:
            seen += 1
            en = next(i for i in range(st, len(lines)) if "s_endpgm" in lines[i])
            depth, n_barriers = 0, 0
            i = st + 1
            while i <= en:
                l = lines[i]
                if re.match(r"^\.LBB\d+_\d+:", l) or re.match(r"^; %bb\.\d+:", l):
                    # depth of this block: the largest Depth= named in its label comment lines
                    ds = [int(x) for x in re.findall(r"Depth=(\d+)", l)]
                    j = i + 1
                    while j <= en and lines[j].lstrip().startswith(";") and not re.match(r"^; %bb\.", lines[j]):
                        if "This" in lines[j] and "Loop Header" in lines[j]:
                            ds += [int(x) for x in re.findall(r"Depth=(\d+)", lines[j])]
                        j += 1
                    depth = max(ds) if ds else 0
                elif "s_barrier" in l:
                    n_barriers += 1
                    assert depth <= 1, f"{name}: {lines[st][:60]}: s_barrier at loop depth {depth} (line {i - st})"
                i += 1
            assert n_barriers >= 4, "the engine loop should hold two barriers per turn plus two in the prologue"
    assert seen >= 64 + 16, "window kernels of every page shape: 64 with a run-time token count, 16 exact"
