"""Every kernel of the built library keeps its data in registers and LDS: the compiler's metadata
reports no scratch memory (private segment) for any of them.  Needs the built library; no GPU."""
import os
import re

import pytest

import paper_1112_1805_amd as pkg

pytestmark = pytest.mark.skipif(not os.path.exists(pkg.LIB_PATH), reason="library not built")


def unsigned(b, i):
    """The MessagePack unsigned integer at offset i of b."""
    t = b[i]
    if t < 0x80:
        return t
    size = {0xCC: 1, 0xCD: 2, 0xCE: 4, 0xCF: 8}[t]
    return int.from_bytes(b[i + 1:i + 1 + size], "big")


def kernels():
    """{kernel symbol: private segment bytes per lane} from the code objects' metadata notes (one
    MessagePack map per kernel, keys in alphabetical order)."""
    data = open(pkg.LIB_PATH, "rb").read()
    key, out = b"\xbb.private_segment_fixed_size", {}
    for m in re.finditer(re.escape(key), data):
        sym = re.compile(rb"\xa7\.symbol(?:\xd9.|\xda..|[\xa0-\xbf])([A-Za-z0-9_]+)\.kd", re.S).search(data, m.end(), m.end() + 4096)
        out[sym.group(1).decode()] = unsigned(data, m.end())
    return out


def test_no_kernel_uses_scratch_memory():
    k = kernels()
    assert len(k) > 400
    for name in ("k_row_g", "kg_row_g", "k_colg", "kg_colg", "k_colg_solve", "k_mid_g", "k_row", "k_nl_dual", "k_tv_update"):
        assert any(f"{len(name)}{name}" in s for s in k), name
    assert {s: b for s, b in k.items() if b} == {}
