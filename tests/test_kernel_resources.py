"""What the compiler gave the kernels of the built library, from the metadata of its code objects: no GPU needed."""
import os
import re
import struct
import subprocess

import pytest

from paper_2405_10951_amd import build as B

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> (bytes of scratch memory a lane asks for, spilled vector registers)"""
    lib = B.LIB if os.path.exists(B.LIB) else B.build()
    data, out = open(lib, "rb").read(), {}
    for m in re.finditer(b"\x7fELF", data):
        at = m.start()
        if struct.unpack_from("<H", data, at + 18)[0] != 224:           # a code object for AMD GPUs
            continue
        shoff, = struct.unpack_from("<Q", data, at + 40)
        size, count = struct.unpack_from("<HH", data, at + 58)
        obj = tmp_path_factory.mktemp("co") / "k.co"
        obj.write_bytes(data[at:at + shoff + size * count])
        notes = subprocess.run([READELF, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout
        for block in notes.split("  - .agpr_count")[1:]:
            get = lambda key: re.search(r"\.%s:\s+(\S+)" % key, block).group(1)      # noqa: E731
            out[get("name")] = (int(get("private_segment_fixed_size")), int(get("vgpr_spill_count")))
    return out


def test_no_gradient_kernel_needs_scratch(kernels):
    """A weight gradient only ever leaves as plain fp32: an epilogue with other paths in it cost the joint kernels registers that
    they then spilled around code that never ran."""
    grads = {n: v for n, v in kernels.items() if "gemm_pair_kernel" in n or "gemm_tn_kernel" in n}
    assert len(grads) == 10
    assert {n: v for n, v in grads.items() if v != (0, 0)} == {}
