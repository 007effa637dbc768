"""Resources of the built kernels, from the metadata of the library's code
objects (CPU only): the kernels of the CG loop -- the Green-operator passes and
the regular- and irregular-voxel operator -- keep everything in registers.  A
spill there turns register traffic into memory traffic of every wave, and the
compiler makes it without an error when a launch bound asks for more waves than
the registers allow."""

import os
import re
import struct
import subprocess

import pytest

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
LOOP_KERNELS = r"k_fft_(plane|x|y|z)|k_regular|k_irregular"


def _code_objects(lib):
    """gfx950 code objects in the library's offload bundles."""
    data = open(lib, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(count):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(magic, at + 1)


def _kernels(lib, tmp_path):
    out = {}
    for i, obj in enumerate(_code_objects(lib)):
        path = tmp_path / f"{i}.co"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        # one entry per kernel: ".name:", ".private_segment_fixed_size:", ".vgpr_spill_count:"
        for entry in re.split(r"\n  - (?=\.)", notes):
            name = re.search(r"\n\s+\.name:\s+(_Z\S+)", entry)
            scratch = re.search(r"\.private_segment_fixed_size:\s+(\d+)", entry)
            spills = re.search(r"\.vgpr_spill_count:\s+(\d+)", entry)
            if name and scratch and spills:
                out[name.group(1)] = (int(scratch.group(1)), int(spills.group(1)))
    return out


def test_loop_kernels_do_not_spill(tmp_path):
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf not found")
    from paper_2601_02172_amd import xfft, build
    xfft._lib()
    kernels = _kernels(build.LIB, tmp_path)
    loop = {k: v for k, v in kernels.items() if re.search(LOOP_KERNELS, k)}
    assert len(loop) > 100
    assert not {k: v for k, v in loop.items() if v != (0, 0)}
