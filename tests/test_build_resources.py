"""What the built library says about its kernels: the persistent recurrence keeps its weights in registers for a whole
sequence and must not spill (scratch accesses would queue with its polls in the in-order memory counter); the linear layers live
on several workgroups per compute unit."""
import os
import re
import struct

import msgpack

from paper_2206_07882_amd import qrnnt

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2206_07882_amd", "libqrnnt.so")


def kernels():
    """{name: metadata} of every kernel in the code objects inside the library (AMDGPU metadata notes)."""
    blob, out = open(LIB, "rb").read(), {}
    for m in re.finditer(b"\x7fELF\x02\x01", blob):
        base = m.start()
        if base == 0 or struct.unpack_from("<H", blob, base + 18)[0] != 224:   # EM_AMDGPU
            continue
        shoff, = struct.unpack_from("<Q", blob, base + 40)
        shentsize, shnum = struct.unpack_from("<HH", blob, base + 58)
        for i in range(shnum):
            _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", blob, base + shoff + i * shentsize)
            if kind != 7:   # SHT_NOTE
                continue
            at, end = base + off, base + off + size
            while at < end:
                namesz, descsz, note = struct.unpack_from("<III", blob, at)
                desc = at + 12 + (namesz + 3) // 4 * 4
                if note == 32:   # NT_AMDGPU_METADATA
                    for k in msgpack.unpackb(blob[desc:desc + descsz], strict_map_key=False)["amdhsa.kernels"]:
                        out[k[".name"]] = k
                at = desc + (descsz + 3) // 4 * 4
    return out


def test_the_recurrence_does_not_spill():
    qrnnt.load()
    rec = {n: k for n, k in kernels().items() if "lstm_rec_kernel" in n}
    assert len(rec) >= 56
    assert sum(n.endswith("ELi2EEEv10QrRecGroup") for n in rec) == 8   # two groups of utterances in turn: 257 to 640 cells
    spilled = {n: k[".private_segment_fixed_size"] for n, k in rec.items() if k[".private_segment_fixed_size"]}
    assert not spilled
    assert max(k[".group_segment_fixed_size"] for k in rec.values()) <= 160 * 1024


def test_linear_layers_leave_room_for_a_third_workgroup():
    """Four waves a workgroup, 512 registers a lane and SIMD: three fit if a wave takes at most 168."""
    qrnnt.load()
    lin = [k for n, k in kernels().items() if "linear_head_kernel" in n]
    assert lin
    for k in lin:
        assert k[".vgpr_count"] <= 168 and k[".private_segment_fixed_size"] == 0   # (accumulation registers included)
