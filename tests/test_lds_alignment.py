"""Where a kernel's dynamic LDS holds 16-byte elements, it begins at a multiple of 16: behind the static part, whose size the code
object's metadata gives."""
import os
import re
import struct
import subprocess

import pytest

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
SIXTEEN = ["path_sum_kernel"]                     # kernels with double2 (or wider) in their dynamic LDS


def _static_lds(path, tmp):
    """Static LDS bytes of every kernel in the library's gfx950 code objects."""
    lib, out, at = open(path, "rb").read(), {}, 0
    while (at := lib.find(b"\x7fELF", at + 1)) > 0:
        if struct.unpack_from("<H", lib, at + 18)[0] != 224:          # EM_AMDGPU
            continue
        obj = os.path.join(tmp, "obj")
        open(obj, "wb").write(lib[at:])
        name = None
        for line in subprocess.run([READELF, "--notes", obj], capture_output=True, text=True).stdout.splitlines():
            if m := re.match(r"\s+(?:- )?\.group_segment_fixed_size:\s+(\d+)", line):
                size = int(m[1])
            elif m := re.match(r"\s+\.name:\s+'?(_Z\w+|\w+_kernel)", line):
                out[m[1]] = size
    return out


def test_dynamic_lds_of_wide_elements(tmp_path):
    import paper_2408_00741_amd as dyn
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    lds = _static_lds(dyn.lib_path(), str(tmp_path))
    assert len(lds) > 50
    for kernel in SIXTEEN:
        found = {k: v for k, v in lds.items() if kernel in k}
        assert found and all(v % 16 == 0 for v in found.values()), found
