"""Registers of the built kernels (from the metadata of the library's own
code objects): no instance of the forward or the backward spills, and each
leaves room for the waves per SIMD that the launch rules count with."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TOOLS = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
LIB = os.path.join(ROOT, "paper_2505_08098_amd", "libf3s.so")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: (registers, spilled registers)} of libf3s.so."""
    objcopy, readelf = (os.path.join(TOOLS, t) for t in ("llvm-objcopy", "llvm-readelf"))
    if not (os.path.exists(objcopy) and os.path.exists(readelf) and os.path.exists(LIB)):
        pytest.skip("the library or ROCm's object tools are not there")
    d = tmp_path_factory.mktemp("objects")
    fat = d / "fatbin"
    subprocess.run([objcopy, "--dump-section", f".hip_fatbin={fat}", LIB, str(d / "copy")],
                   check=True)
    data, found, magic = fat.read_bytes(), {}, b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        pos = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, length = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" not in name or not size:
                continue
            obj = d / "object"
            obj.write_bytes(data[at + off:at + off + size])
            notes = subprocess.run([readelf, "--notes", str(obj)], check=True,
                                   capture_output=True, text=True).stdout
            for k in re.split(r"\n  - \.a", notes):
                names = re.findall(r"^    \.name:\s+(_Z\S+)", k, re.M)
                if names:
                    found[names[0]] = tuple(
                        int(re.search(rf"^    \.{f}:\s+(\d+)", k, re.M)[1])
                        for f in ("vgpr_count", "vgpr_spill_count"))
        at = data.find(magic, at + 1)
    return found


def _room(registers):
    return min(8, 512 // (-(-registers // 8) * 8))


FORWARD = {32: 6, 64: 4, 96: 3, 128: 2, 160: 2, 192: 1, 224: 1, 256: 1}
DQ = {32: 6, 64: 4, 96: 2, 128: 2, 160: 1, 192: 1, 224: 1, 256: 1}
DKDV = {32: 5, 64: 3, 96: 2, 128: 2, 160: 1, 192: 1, 224: 1, 256: 1}


@pytest.mark.parametrize("kernel", ["k_fused3s", "k_bwd_dq", "k_bwd_dkdv"])
def test_no_spills_and_room_for_the_counted_waves(kernels, kernel):
    args = (r"Li(\d+)ELb(\d)ELi(\d)ELb(\d)ELb(\d)ELi(\d)ELb(\d)E" if kernel == "k_fused3s"
            else r"Li(\d+)ELb(\d)ELb(\d)ELi(\d)E")
    seen = set()
    for name, (registers, spilled) in kernels.items():
        m = re.search(r"\d%sI%s" % (kernel, args), name)
        if not m:
            continue
        a = [int(x) for x in m.groups()]
        d, wide, waves = a[0], a[1], a[5] if kernel == "k_fused3s" else a[3]
        if kernel == "k_fused3s" and a[4]:
            continue  # the narrow-gather ablation
        room = {"k_fused3s": FORWARD, "k_bwd_dq": DQ, "k_bwd_dkdv": DKDV}[kernel][d]
        if kernel == "k_fused3s" and a[2] == 1 and d == 32:
            room -= 1  # bf16: the second probability term
        if kernel == "k_bwd_dq" and d == 64 and wide and waves > 1:
            room -= 1
        assert spilled == 0, (name, spilled)
        assert _room(registers) >= room, (name, registers)
        seen.add(tuple(a))
    # f16 and bf16 (forward: fp8, both outputs, traced), both addressings
    assert len(seen) == (8 * (3 * 2 * 2 * 3 + 3) if kernel == "k_fused3s" else 8 * 2 * 2 * 3)
