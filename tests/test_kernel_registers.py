"""CPU-only: what the compiler says of the built kernels.  Those of the main path keep nothing in scratch memory."""
import os
import re
import struct
import subprocess

import pytest

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAIN_PATH = ("k_layer_slice", "k_layer_mfma", "k_direct", "k_split", "k_buckets", "k_vox_", "k_rows")


def _kernels(tmp_path):
    """{mangled name: bytes of scratch memory a lane} of every kernel in the library."""
    import paper_2301_08739_amd as ff
    if not os.path.exists(ff.library_path()):
        pytest.skip("library not built (run __graft_entry__.build())")
    if not os.path.exists(READELF):
        pytest.skip("no " + READELF)
    blob, mark, found = open(ff.library_path(), "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", {}
    at = blob.find(mark)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(mark))
        entry = at + len(mark) + 8
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", blob, entry)
            target = blob[entry + 24:entry + 24 + name].decode()
            entry += 24 + name
            if "gfx950" in target and size:
                code = tmp_path / "code.elf"
                code.write_bytes(blob[at + offset:at + offset + size])
                notes = subprocess.run([READELF, "--notes", str(code)], capture_output=True, text=True, check=True).stdout
                for kernel in re.split(r"\n +- \.agpr_count", notes)[1:]:
                    field = lambda k: re.search(r"\.%s: +(\S+)" % k, kernel).group(1)
                    found[field("name")] = int(field("private_segment_fixed_size"))
        at = blob.find(mark, at + 1)
    return found


def test_main_path_keeps_nothing_in_scratch_memory(tmp_path):
    kernels = _kernels(tmp_path)
    for name in MAIN_PATH:
        of_it = {k: v for k, v in kernels.items() if name in k}
        assert of_it and not any(of_it.values()), {k: v for k, v in of_it.items() if v}
