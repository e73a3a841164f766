"""What the compiler made of the attention kernels: facts of the built library that their speed rests on."""
import os
import re
import struct
import subprocess

import pytest

import paper_2512_11529_amd as gr

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code objects of the library, one per source, as files."""
    if not os.path.exists(gr.LIB_PATH):
        from paper_2512_11529_amd import build
        build.build_lib()
    with open(gr.LIB_PATH, "rb") as f:
        lib = f.read()
    out = []
    for bundle in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", lib):
        at = bundle.start()
        count, = struct.unpack_from("<Q", lib, at + 24)
        pos = at + 32
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", lib, pos)
            target = lib[pos + 24:pos + 24 + n]
            pos += 24 + n
            if target.endswith(b"gfx950") and size:
                path = tmp_path_factory.mktemp("co") / "a.elf"
                path.write_bytes(lib[at + offset:at + offset + size])
                out.append(str(path))
    assert out
    return out


def test_attention_kernels_do_not_spill(code_objects):
    seen = 0
    for path in code_objects:
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", path], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
            name = re.search(r"\.name:\s+(\S+)", kernel)[1]
            if "k_beam_attn" not in name and "k_attn_merge" not in name:
                continue
            seen += 1
            spilled = {k: int(v) for k, v in re.findall(r"\.([sv]gpr_spill_count):\s+(\d+)", kernel)}
            assert spilled == {"sgpr_spill_count": 0, "vgpr_spill_count": 0}, name
    assert seen == 27           # 20 decode kernels, 5 causal ones, two of the merge
