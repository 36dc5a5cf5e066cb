"""Registers of the built kernels, from the metadata of the library's own code
objects (no GPU): the persistent step kernel, which runs one workgroup per
compute unit with every register it can have, keeps all of its state in
registers in each of its variants, and so do the one- and two-tile GEMMs of
the balanced path that have splits to add."""
import re
import struct
import subprocess

import pytest

from tests.harness import ensure_built

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """Mangled kernel name -> bytes of scratch per lane, over the gfx950 code objects in libas2d.so."""
    from paper_2609_37617_amd import as2d
    ensure_built()
    data = open(as2d.LIB_PATH, "rb").read()
    folder, out = tmp_path_factory.mktemp("co"), {}
    for at in (m.start() for m in re.finditer(re.escape(MAGIC), data)):
        p = at + len(MAGIC)
        (n,) = struct.unpack_from("<Q", data, p)
        p += 8
        if n > 8:   # the magic's own bytes elsewhere in the file
            continue
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            ident = data[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" not in ident:
                continue
            co = folder / f"{at}.co"
            co.write_bytes(data[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", str(co)], capture_output=True, text=True, check=True).stdout
            for name, seg in re.findall(r"\.name:\s+(_Z\S+)\n(?:.*\n)*?\s+\.private_segment_fixed_size:\s+(\d+)", notes):
                out[name] = int(seg)
    return out


def test_step_kernels_use_no_scratch(scratch):
    steps = {k: v for k, v in scratch.items() if "step_kernel" in k}
    assert len(steps) == 16, sorted(steps)   # bf16 x (two tiles, four slice lengths), float32 x (two tiles, two), two head sizes
    assert not {k: v for k, v in steps.items() if v}


def test_balanced_gemms_with_splits_use_no_scratch(scratch):
    # gemm_range_kernel<bf16, row tiles, 0, A, epilogue>
    gemms = {k: v for k, v in scratch.items() if re.search(r"gemm_range_kernelILb[01]ELi[12]ELi0E", k)}
    assert len(gemms) == 20, sorted(gemms)
    assert not {k: v for k, v in gemms.items() if v}
