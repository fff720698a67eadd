"""What the compiler made of the kernels: the metadata of the code objects in the built library.

The one-launch stacks keep the next layer's weights in flight across all phases and fill the register file with one to
four batch rows (with RMSNorm one); scratch there means spills between a layer's first loads and their use.
"""
import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")
NT_AMDGPU_METADATA = 32


def code_objects(blob):
    """The gfx950 ELF files inside the host library."""
    at = blob.find(b"\x7fELF", 4)
    while at >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == 224:          # EM_AMDGPU
            yield at
        at = blob.find(b"\x7fELF", at + 4)


def kernels():
    """name -> metadata of every kernel of the library."""
    from paper_2508_18850_amd import lib_path
    with open(lib_path(), "rb") as f:
        blob = f.read()
    found = {}
    for base in code_objects(blob):
        shoff, = struct.unpack_from("<Q", blob, base + 40)
        shentsize, shnum = struct.unpack_from("<HH", blob, base + 58)
        for k in range(shnum):
            kind, _, _, off, size = struct.unpack_from("<IQQQQ", blob, base + shoff + k * shentsize + 4)
            if kind != 7:                                              # SHT_NOTE
                continue
            p, end = base + off, base + off + size
            while p < end:
                namesz, descsz, note = struct.unpack_from("<III", blob, p)
                desc = p + 12 + (namesz + 3) // 4 * 4
                if note == NT_AMDGPU_METADATA:
                    for kern in msgpack.unpackb(blob[desc:desc + descsz])["amdhsa.kernels"]:
                        found[kern[".name"]] = kern
                p = desc + (descsz + 3) // 4 * 4
    return found


def test_one_launch_stack_has_no_scratch_up_to_batch_4():
    from paper_2508_18850_amd import lib_path
    if not os.path.exists(lib_path()):
        from paper_2508_18850_amd import build
        build.build()
    all_kernels = kernels()
    for group in (1, 2, 4, 8):
        for tile in (1, 4):
            mine = [v for k, v in all_kernels.items() if "fused_decode_stackILi128ELi%dELi%dEE" % (group, tile) in k]
            if tile == 1:
                mine += [v for k, v in all_kernels.items() if "fused_layer_stackILi128ELi%dELi1EE" % group in k]
            assert len(mine) == (2 if tile == 1 else 1), (group, tile)
            for kernel in mine:
                assert kernel[".private_segment_fixed_size"] == 0, (group, tile, kernel[".name"])


def test_16_row_tile_has_no_scratch():
    all_kernels = kernels()
    for name in ("block", "layer"):
        for hd in (64, 128):
            for group in (1, 2, 4, 8):
                mine = [v for k, v in all_kernels.items() if "fused_decode_%sILi%dELi%dELi16EE" % (name, hd, group) in k]
                assert len(mine) == 1 and mine[0][".private_segment_fixed_size"] == 0, (name, hd, group)


def test_counters_are_not_read_as_constants(tmp_path):
    """A launch counter is overwritten by the launch that reads it, so it may not be read through the constant address space:
    such a load may be repeated by the compiler at any place, also behind the store.  (The kernel arguments are in that address
    space from the start; nothing is cast to it.)"""
    import re
    import subprocess

    from paper_2508_18850_amd import build
    ir = tmp_path / "cf_ffn.ll"
    subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, "--cuda-device-only", "-S", "-emit-llvm", "-Xclang", "-disable-llvm-passes",
                    "-o", str(ir), os.path.join(build.CSRC, "cf_ffn.hip")], check=True, capture_output=True)
    text = ir.read_text()
    assert "fused_ffn_tiles" in text
    assert not re.findall(r"(?:inttoptr|addrspacecast) .* to ptr addrspace\(4\)", text)
