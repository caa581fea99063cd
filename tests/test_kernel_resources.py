"""What the compiler made of the kernels, read from the notes of the built library's code objects (this repository's own code): the
kernels of the default paths keep everything in registers.  A private segment means that a value is stored to memory and read back."""
import os
import re
import shutil
import struct
import subprocess

import pytest

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"


def _code_objects(blob):
    """gfx950 code objects of the offload bundles in `blob`: magic, number of entries, then offset, size and name of each."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        n, p = struct.unpack_from("<Q", blob, at + 24)[0], at + 32
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", blob, p)
            name, p = blob[p + 24:p + 24 + ln], p + 24 + ln
            if b"gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(magic, at + 24)


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    import paper_2412_07017_amd as pkg
    if not os.path.exists(pkg.library_path()):
        from paper_2412_07017_amd.build import build_library
        build_library()
    f, out = str(tmp_path_factory.mktemp("co") / "co"), {}
    with open(pkg.library_path(), "rb") as lib:
        blob = lib.read()
    for co in _code_objects(blob):
        with open(f, "wb") as o:
            o.write(co)
        notes = subprocess.run([READELF, "--notes", f], capture_output=True, text=True, check=True).stdout
        names, sizes = re.findall(r"^ +\.name: +(_Z\S+)$", notes, re.M), re.findall(r"^ +\.private_segment_fixed_size: (\d+)", notes, re.M)
        assert len(names) == len(sizes)
        out.update(zip(names, map(int, sizes)))
    return out


def test_kernels_of_the_default_paths_use_no_scratch(scratch):
    # the variants for the step on two streams are bounded to half of the registers (two workgroups per compute unit)
    two_streams = re.compile(r"k_gemvI[ft]Li\dELi\d+ELi1EE|k_attn_decodeI[ft]Li\d+ELi\dELb[01]ELi1EE")
    assert len(scratch) > 100 and any("k_attn_decode" in n for n in scratch)
    used = {n: s for n, s in scratch.items() if s and not two_streams.search(n)}
    assert not used
