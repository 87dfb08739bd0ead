"""Static LDS of kernels that have to find room beside a kernel of another stream that fills the device: about 20 KB find it at once, 40
wait for that kernel's end.  From the code objects' metadata, no GPU needed."""
import os
import re
import struct
import subprocess

import pytest

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
# The walk of a path call of some hundred windows; its rows hold 16-byte elements and are static, so that the compiler places them.
AT_MOST = {"path_walk_kernelILi16E": 8192, "path_walk_kernelILi32E": 16384, "path_walk_kernelILi48E": 20480, "path_walk_kernelILi64E": 28672}


def _static_lds(path, tmp):
    """Static LDS bytes of every kernel in the library's gfx950 code objects."""
    lib, out, at = open(path, "rb").read(), {}, 0
    while (at := lib.find(b"\x7fELF", at + 1)) > 0:
        if struct.unpack_from("<H", lib, at + 18)[0] != 224:          # EM_AMDGPU
            continue
        obj = os.path.join(tmp, "obj")
        open(obj, "wb").write(lib[at:])
        for line in subprocess.run([READELF, "--notes", obj], capture_output=True, text=True).stdout.splitlines():
            if m := re.match(r"\s+(?:- )?\.group_segment_fixed_size:\s+(\d+)", line):
                size = int(m[1])
            elif m := re.match(r"\s+\.name:\s+'?(_Z\w+|\w+_kernel)", line):
                out[m[1]] = size
    return out


def test_room_beside_other_streams(tmp_path):
    import paper_2408_00741_amd as dyn
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    lds = _static_lds(dyn.lib_path(), str(tmp_path))
    assert len(lds) > 50
    for kernel, most in AT_MOST.items():
        found = [v for k, v in lds.items() if kernel in k]
        assert len(found) == 1 and found[0] <= most, (kernel, found)
