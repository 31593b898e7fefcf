"""Register use of the built kernels, read from the code objects' own metadata (no GPU): a kernel
that keeps part of its state in private memory does so silently and pays a memory access each time."""
import os
import struct

import msgpack
import pytest

import paper_1510_06585_amd as sk


def kernels():
    """{mangled name: metadata} of every gfx950 kernel in libskel.so: the AMDGPU metadata notes
    (name "AMDGPU", type 32, a msgpack map) of the code objects it embeds."""
    sk.lib()
    data = open(os.path.join(os.path.dirname(sk.__file__), "libskel.so"), "rb").read()
    out, i = {}, data.find(b"AMDGPU\0\0")
    while i >= 0:
        namesz, size, kind = struct.unpack("<III", data[i - 12:i])
        if (namesz, kind) == (7, 32):
            meta = msgpack.unpackb(data[i + 8:i + 8 + size], strict_map_key=False)
            out.update({k[".name"]: k for k in meta["amdhsa.kernels"]})
        i = data.find(b"AMDGPU\0\0", i + 8)
    return out


@pytest.mark.parametrize("family", ["mlp_", "img_band_", "img_batch_", "fft_", "vec_", "nbody_", "gray_", "hist_", "while_"])
def test_no_private_memory(family):
    found = {n: k for n, k in kernels().items() if family in n}
    assert found
    bad = {n: k[".private_segment_fixed_size"] for n, k in found.items() if k[".private_segment_fixed_size"]}
    assert not bad, bad
