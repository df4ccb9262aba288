"""No kernel of the built library keeps registers in scratch memory: a reload inside the loop over key blocks waits for
every copy in flight, which the pipeline's partial waits are there to avoid.  Read from the metadata of the library's
own code objects."""
import os
import re
import struct
import subprocess

import pytest

from paper_2512_07011_amd import binding

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def code_objects(path):
    """The AMDGPU ELF images inside a host library, cut out by their section header tables."""
    data = open(path, "rb").read()
    at = data.find(b"\x7fELF", 4)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == 224:                  # EM_AMDGPU
            shoff, = struct.unpack_from("<Q", data, at + 40)
            shentsize, shnum = struct.unpack_from("<HH", data, at + 58)
            yield data[at:at + shoff + shentsize * shnum]
        at = data.find(b"\x7fELF", at + 4)


@pytest.mark.skipif(not os.path.exists(READELF), reason="llvm-readelf is not installed")
def test_no_kernel_uses_scratch_memory(tmp_path):
    if not os.path.exists(binding.LIB_PATH):
        from paper_2512_07011_amd import build
        build.build_lib()
    seen = {}
    for i, image in enumerate(code_objects(binding.LIB_PATH)):
        f = tmp_path / ("%d.elf" % i)
        f.write_bytes(image)
        notes = subprocess.run([READELF, "--notes", str(f)], check=True, capture_output=True, text=True).stdout
        for k in re.split(r"\n {2}- ", notes):
            name, size = re.search(r"\.name: +(_Z\w+)", k), re.search(r"\.private_segment_fixed_size: (\d+)", k)
            if name and size:
                seen[name[1]] = int(size[1])
    assert sum("bsfa_fwd_kernel" in n for n in seen) >= 60 and any("topk_kernel" in n for n in seen)
    assert not {n: s for n, s in seen.items() if s}
