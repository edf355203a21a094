"""Registers of the station kernels, from the metadata of the built library's code objects: a
SIMD's 512 vector registers hold as many waves as a kernel's count allows, and large batches
need several to hide their memory latency."""
import os
import re
import struct

import pytest

from paper_2503_09203_amd import mgx

msgpack = pytest.importorskip("msgpack")


def _kernels():
    """Metadata of every gfx950 kernel in the library: {mangled name: dict}."""
    if not os.path.exists(mgx.LIB_PATH):
        mgx.lib()
    data = open(mgx.LIB_PATH, "rb").read()
    out = {}
    for at in (m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data)):
        pos, (n,) = at + 32, struct.unpack_from("<Q", data, at + 24)
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" not in name or not size:
                continue
            elf = data[at + off:at + off + size]
            shoff, = struct.unpack_from("<Q", elf, 40)
            shentsize, shnum = struct.unpack_from("<HH", elf, 58)
            for i in range(shnum):
                kind, _, _, o, sz = struct.unpack_from("<IQQQQ", elf, shoff + i * shentsize + 4)
                if kind != 7:       # SHT_NOTE
                    continue
                namesz, descsz, _ = struct.unpack_from("<III", elf, o)
                desc = o + 12 + (namesz + 3) // 4 * 4
                for k in msgpack.unpackb(elf[desc:desc + descsz], strict_map_key=False)["amdhsa.kernels"]:
                    out[k[".name"]] = k
    return out


def test_station_kernels_hold_their_waves():
    """One-step kernels (m thrusters; shaped, fins, payload): the most vector registers at which
    as many waves fit a SIMD as the launches of large batches count on, and no spills."""
    kernels = _kernels()
    # (type, m, shaped, fins, payload): vector registers
    bound = {("f", 6, 0, 0, 0): 128, ("f", 6, 1, 0, 0): 128, ("f", 6, 1, 0, 1): 168, ("f", 8, 0, 0, 0): 192,
             ("f", 5, 1, 1, 0): 256, ("f", 6, 1, 1, 0): 256, ("d", 6, 0, 0, 0): 256, ("d", 6, 1, 0, 0): 256}
    for (t, m, *body), most in bound.items():
        name = f"_ZN3mgx14k_station_stepI{t}Li{m}E" + "".join(f"Lb{x}E" for x in body) + "Lb0E"
        k, = (v for key, v in kernels.items() if key.startswith(name))
        assert k[".vgpr_count"] <= most and k[".vgpr_spill_count"] == 0, (name, k[".vgpr_count"])
    # calls of many steps: two waves for six propellers and a payload, and for eight propellers
    for name in ("fLi6ELb0ELb0ELb0ELb1E", "fLi6ELb1ELb0ELb1ELb1E", "fLi8ELb0ELb0ELb0ELb1E"):
        k, = (v for key, v in kernels.items() if key.startswith("_ZN3mgx14k_station_stepI" + name))
        assert k[".vgpr_count"] <= 256, (name, k[".vgpr_count"])


def test_single_steps_with_payload_and_fins_in_double_spill_no_more():
    """The largest one-step body: its spills are memory traffic of every step."""
    k, = (v for key, v in _kernels().items() if key.startswith("_ZN3mgx6k_stepIdLi8ELb0ELb1ELb1ELb1ELb1E"))
    assert k[".vgpr_spill_count"] <= 96, k[".vgpr_spill_count"]
