"""What kernels rely on of their registers (host-only: reads the metadata of the built library)."""
import random
import re
import struct

import pytest

from paper_2404_19124_amd import binding as B

msgpack = pytest.importorskip("msgpack")


def kernels():
    """(name, metadata) of every kernel of the library: the notes of its code objects."""
    data = open(B.LIB_PATH, "rb").read()
    at = data.find(b"AMDGPU\0\0")
    while at >= 0:
        name_size, size, kind = struct.unpack_from("<III", data, at - 12)
        if (name_size, kind) == (7, 32):
            for k in msgpack.unpackb(data[at + 8:at + 8 + size])["amdhsa.kernels"]:
                yield k[".name"], k
        at = data.find(b"AMDGPU\0\0", at + 8)


def test_tile_kernel_without_scratch():
    """A reload would wait for every copy in flight, and the spills of 256 persistent workgroups are traffic of their own."""
    B.lib()
    found = {name: k[".private_segment_fixed_size"] for name, k in kernels() if "head_tile_kernel" in name}
    assert len(found) == 5 and not any(found.values()), found


def test_one_round_kernel_without_scratch():
    """Its counted waits are for copies: a spill's loads and stores would count with them."""
    B.lib()
    found = {name: k[".private_segment_fixed_size"] for name, k in kernels() if "head_once_kernel" in name}
    assert len(found) == 15 and not any(found.values()), found


def test_stage_kernels_share_a_cu():
    """Rows of up to 4096 elements one chunk per thread, up to 8192 two: of the latter two workgroups of 512 threads fit a CU's 512
    registers per lane (four siblings at a time do not), of the former three."""
    B.lib()
    found = {name: k[".vgpr_count"] for name, k in kernels() if "stage_kernel" in name}
    two = {name: n for name, n in found.items() if "ELi2ELi512EE" in name}
    one = {name: n for name, n in found.items() if "ELi1ELi512EE" in name}
    assert len(two) == 14 and max(two.values()) <= 128, two
    assert len(one) == 14 and max(one.values()) <= 80, one


def test_the_plan_reaches_every_instance():
    """Of the panel kernel and of the one-round kernel, and asks for no other."""
    rnd = random.Random(8)
    asked = set()
    for _ in range(20000):
        n_head = rnd.choice([rnd.randint(1, 3000), rnd.randint(3000, 60000)])
        k = 64 * rnd.randint(4, 70)
        p = B.spec_plan_panel(rnd.randint(17, 330), k, n_head, rnd.randint(1, 8), rnd.choice([0, k]), 256)["kernel"]
        if 400 <= p < 1000:
            asked.add(("head_once_kernel", 4 if p >= 500 else 5, p % 100 // 10, p % 10))
        elif 300 <= p < 400:
            asked.add(("head_panel_kernel", p % 100 // 10, p % 10))
    built = set()
    for name, _ in kernels():
        m = re.search(r"(head_once_kernel|head_panel_kernel)I((?:Li\d+E)+)E", name)
        if m:
            built.add((m.group(1),) + tuple(int(x) for x in re.findall(r"Li(\d+)E", m.group(2))))
    assert built == asked, (built - asked, asked - built)
