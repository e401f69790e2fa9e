"""The training tile kernel keeps its sums in registers in every shape that is
built: a matrix-instruction kernel that spills vector registers has been
compiled to wrong weight gradients (and the compiler has crashed on it), so a
shape that would spill takes the gathering kernel instead."""
import os
import re

import pytest

from paper_2504_04315_amd import npm as B


def kernel_metadata(blob):
    """{kernel name: spilled vector registers} from the code object's metadata
    (MessagePack maps, one per kernel, whose keys are sorted)."""
    out = {}
    for m in re.finditer(rb"\.name[\xd9\xa0-\xbf]", blob):
        at = m.end() - 1
        first = blob[at]
        n, at = (blob[at + 1], at + 2) if first == 0xd9 else (first & 0x1f, at + 1)
        name = blob[at:at + n]
        key = blob.find(b".vgpr_spill_count", at, at + 2000)
        if not name.startswith(b"_ZN3npm") or key < 0:
            continue
        v = key + len(b".vgpr_spill_count")
        code = blob[v]
        out[name.decode()] = (code if code < 0x80 else blob[v + 1] if code == 0xcc
                              else int.from_bytes(blob[v + 1:v + 3], "big"))
    return out


def test_training_tile_kernel_does_not_spill():
    if not os.path.exists(B.LIB_PATH):
        pytest.fail("libnpm.so is not built")
    with open(B.LIB_PATH, "rb") as f:
        found = kernel_metadata(f.read())
    tiles = {k: v for k, v in found.items() if "k_train_tile" in k}
    assert len(tiles) >= 16, sorted(found)
    assert not {k: v for k, v in tiles.items() if v}
