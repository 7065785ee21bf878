"""What the compiler made of the searches' registers, read from the metadata of the library that is built here: at most 128 for two
blocks per CU.  k_search_dense holds the row loop's values in them: a variant that keeps one double too many per p_D
value spills 8 to 15, and the shortest launches get a quarter slower.  k_search_batch holds everything with one scalar key other than the
product; with the others it stores, once an item, what only a recovered position reads."""
import os
import re
import struct

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.environ.get("MMEE_LIB") or os.path.join(ROOT, "paper_2604_03446_amd", "libmmee.so")


def kernels(path):
    """The kernels' metadata: the msgpack notes of the AMDGPU code objects inside the library."""
    data, out = open(path, "rb").read(), {}
    for m in re.finditer(rb"AMDGPU\0\0", data):              # a note's name, behind its sizes and its type
        name_size, size, kind = struct.unpack_from("<III", data, m.start() - 12)
        if name_size != 7 or kind != 32 or m.end() + size > len(data):
            continue
        for k in msgpack.unpackb(data[m.end():m.end() + size], raw=False)["amdhsa.kernels"]:
            out[k[".name"]] = k
    return out


@pytest.mark.skipif(not os.path.exists(LIB), reason="the library is not built")
def test_spills_of_the_dense_kernel():
    dense = {n: k for n, k in kernels(LIB).items() if "k_search_dense" in n}
    assert len(dense) >= 40
    for name, k in dense.items():
        # _ZN4mmee14k_search_denseILi<keys>ELb<exact time>ELb<bounded>ELi<kind of sum>ELb<capped>EE...
        keys, fast, bounded, kind, capped = map(int, re.search(r"k_search_denseILi(\d+)ELb(\d)ELb(\d)ELi(\d)ELb(\d)E", name).groups())
        assert k[".vgpr_count"] <= 128, name
        regrouped, both = kind == 1, keys != 2 and keys != 1 or bounded or capped
        # one key that needs the energy or the time alone, or a regrouped one: none; constants in order cost a few
        assert k[".vgpr_spill_count"] <= (0 if regrouped or not both else 5), (name, k[".vgpr_spill_count"])


@pytest.mark.skipif(not os.path.exists(LIB), reason="the library is not built")
def test_spills_of_the_batched_kernel():
    batch = {n: k for n, k in kernels(LIB).items() if "k_search_batch" in n}
    assert len(batch) == 15
    for name, k in batch.items():
        keys = int(re.search(r"k_search_batchILi(\d+)E", name).group(1))
        assert k[".vgpr_count"] <= 128 and 2 * k[".group_segment_fixed_size"] <= 160 << 10, name
        # energy, latency: none; both: the nine combinations' constants, 18 doubles, at most; (latency, energy), product: fewer
        assert k[".vgpr_spill_count"] <= {1: 0, 2: 0, 3: 25, 4: 20, 8: 10}[keys], (name, k[".vgpr_spill_count"])
