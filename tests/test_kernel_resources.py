"""The built library's own kernel metadata: no per-coefficient or transform
kernel spills vector registers (k_ks_fused, the measured alternative that is
off by default, does)."""
import os

import msgpack

from paper_2602_24271_amd import build


def kernels():
    data = open(build.LIB, "rb").read()
    out, key = [], b"amdhsa.kernels"
    at = data.find(key)
    while at >= 0:
        # a code object's metadata: a map whose first key this is
        unpacker = msgpack.Unpacker(raw=False, strict_map_key=False,
                                    max_buffer_size=len(data))
        unpacker.feed(data[at - 2:at + (8 << 20)])
        out += unpacker.unpack()["amdhsa.kernels"]
        at = data.find(key, at + 1)
    return out


def test_no_vector_register_spills():
    assert os.path.exists(build.LIB)
    found = kernels()
    assert len(found) > 400
    spills = {k[".name"]: k[".vgpr_spill_count"] for k in found if k[".vgpr_spill_count"]}
    assert all("k_ks_fused" in name for name in spills), spills
