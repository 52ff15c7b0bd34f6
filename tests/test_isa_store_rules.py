"""A rule for the generated gfx950 code: no buffer store of more than 64 bits takes its offset from a scalar register.
Such a store reads its data registers late, one wait state has to pass before they are written again, and the compiler
inserts it only for stores without a scalar offset; without it lanes store what the next instructions compute."""
import os
import re

import pytest

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.parametrize("group", [2, 6])  # page shapes of 64 and 128 channels
def test_no_wide_buffer_store_with_a_scalar_offset(tmp_path, group):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not installed")
    from paper_2512_11920_amd import build

    text = open(build.compile_unit("kvc_codec.hip", (f"-DKVC_SHAPE_GROUP={group}",), str(tmp_path / "k.s"), (), True)).read()
    stores = re.findall(r"^\s*buffer_store_dwordx[34]\s+v\[\d+:\d+\],\s*(?:v\d+|off),\s*s\[\d+:\d+\],\s*(\S+)", text, flags=re.M)
    assert len(stores) > 20, "the window's decoders write their pages with buffer stores"
    assert set(stores) == {"0"}, sorted(set(stores))
