"""Registers that the built kernels keep in scratch memory, from the metadata of the code objects in the library.  A mask predictor
that spills more than a few pays for it in its loops: groups of 8, k = 32, N = 32, L = 8192, keep = 82 took 198 us with 103
registers in scratch and takes 146 with 7."""
import re
import struct
import subprocess

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MOST = 16                       # up to 13 are values that live through a kernel and are not used in its loops


def code_objects(blob):
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        place = at + 32
        for _ in range(struct.unpack_from("<Q", blob, at + 24)[0]):
            offset, size, name = struct.unpack_from("<QQQ", blob, place)
            if b"gfx950" in blob[place + 24:place + 24 + name]:
                yield blob[at + offset:at + offset + size]
            place += 24 + name
        at = blob.find(magic, at + 1)


def test_spilled_registers(tmp_path):
    from paper_2110_11299_amd import build
    if not build.LIB.exists():
        build.build_hip()
    seen, worst = 0, {}
    for i, code in enumerate(code_objects(build.LIB.read_bytes())):
        path = tmp_path / f"{i}.elf"
        path.write_bytes(code)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for kernel in notes.split("- .agpr_count")[1:]:
            name = re.search(r"\.symbol:\s+(\S+)", kernel)[1]
            seen += 1
            spilled = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel)[1])
            if spilled > MOST:
                worst[name] = spilled
    assert seen > 100 and not worst, worst
