"""What has to be in the kernels as they are built and shows in no result: read from the disassembly of the library's own code."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2506_15704_amd import build

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler for gfx950 here")


@pytest.fixture(scope="module")
def device_objects(tmp_path_factory):
    """The gfx950 code objects of the library: one offload bundle per source, one after the other in its image."""
    image, magic = open(build.LIB_PATH, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__"
    where, found = tmp_path_factory.mktemp("code"), []
    for m in re.finditer(magic, image):
        at = m.end()
        (entries,) = struct.unpack_from("<Q", image, at)
        if not 0 < entries < 16:
            continue
        at += 8
        for _ in range(entries):
            offset, size, id_len = struct.unpack_from("<QQQ", image, at)
            at += 24
            name = image[at:at + id_len]
            at += id_len
            if b"gfx950" in name and size:
                path = where / f"{len(found)}.o"
                path.write_bytes(image[m.start() + offset:m.start() + offset + size])
                found.append(str(path))
    assert found
    return found


def _disassembly(objects, kernel):
    """{symbol: instructions} of the kernels whose mangled names begin with that of `kernel`."""
    prefix, out = f"_ZN4lfps{len(kernel)}{kernel}I", {}
    for path in objects:
        table = subprocess.run([OBJDUMP, "-t", path], capture_output=True, text=True, check=True).stdout
        names = sorted({w for w in re.findall(r"\S+", table) if w.startswith(prefix) and not w.endswith(".kd")})
        if not names:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", "--mcpu=gfx950",
                               "--disassemble-symbols=" + ",".join(names), path], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n(?=(?:[0-9a-f]+ )?<)", text):
            m = re.match(r"(?:[0-9a-f]+ )?<([^>]+)>:", part)
            if m and m.group(1) in names:
                out[m.group(1)] = part
    return out


def test_many_queries_can_read_their_keys_past_the_caches(device_objects):
    kernels = _disassembly(device_objects, "k_batch_stats")
    assert len(kernels) >= 36
    for name, text in kernels.items():
        assert re.search(r"global_load_dwordx4 .* nt\b", text), name


def test_the_barriers_of_the_batch_kernels_are_common_to_all_waves(device_objects):
    """The source has one before the first products, one per chunk and one before the last sums.  (The compiler may take an iteration
    out of the loop; two loops, one for the waves that load and one for those that add up, make six.)"""
    kernels = _disassembly(device_objects, "k_batch_apply")
    assert len(kernels) >= 36
    for name, text in kernels.items():
        assert 3 <= len(re.findall(r"\bs_barrier\b", text)) <= 4, name
