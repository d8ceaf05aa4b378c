"""What the built library's own metadata says of its kernels."""
import os
import re
import struct
import subprocess

import pytest

import paper_2110_09524_amd as pk

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def scratch_bytes(tmp_path):
    """bytes of scratch memory a lane takes, by kernel (mangled)"""
    with open(pk.LIB_PATH, "rb") as f:
        data = f.read()
    sizes, at = {}, data.find(BUNDLE)
    while at >= 0:
        (entries,), p = struct.unpack_from("<Q", data, at + len(BUNDLE)), at + len(BUNDLE) + 8
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in target and size:
                code = tmp_path / "code.o"
                code.write_bytes(data[at + offset:at + offset + size])
                notes = subprocess.run([READELF, "--notes", str(code)], capture_output=True, text=True, check=True).stdout
                sizes.update((n, int(b)) for n, b in re.findall(r"\.name: +(\S+)\n +\.private_segment_fixed_size: (\d+)", notes))
        at = data.find(BUNDLE, at + 1)
    return sizes


@pytest.mark.skipif(not (os.path.exists(READELF) and os.path.exists(pk.LIB_PATH)), reason="needs the built library and llvm-readelf")
@pytest.mark.parametrize("kernel", ["k_gmmp_fwd_nr", "k_gmmp_bwd_nr", "k_gmmp_bwd_dst_nr"])
def test_narrow_monet_walks_keep_their_values_in_registers(kernel, tmp_path):
    """A bound on registers that has the sums of a walk in scratch memory costs more than the wavefronts it makes room for."""
    found = {n: b for n, b in scratch_bytes(tmp_path).items() if re.search(rf"\d{kernel}I", n)}
    assert len(found) >= 24
    # projected, two or three kernels, one coordinate, groups of eight lanes, room for seven wavefronts: for skewed gathers
    repaid = re.compile(r"k_gmmp_fwd_nrILi8ELb1ELi[23]ELi1ELi8ELi7E")
    assert not {n: b for n, b in found.items() if b > (12 if repaid.search(n) else 0)}
