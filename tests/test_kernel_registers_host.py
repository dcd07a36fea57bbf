"""CPU test: vector registers of built kernels, read from the code objects in libhisa.so.  Where a kernel's speed hangs on how many
of its waves fit a SIMD (512 registers a lane), a change that costs it a wave or makes it spill shows here."""
import os
import re

import pytest

INT = rb"(\xcd..|\xcc.|[\x00-\x7f])"      # MessagePack: two bytes, one, or the value itself


def value(b):
    return int.from_bytes(b[1:] if len(b) > 1 else b, "big")


@pytest.fixture(scope="module")
def kernels():
    """{mangled name: (vector registers, spilled vector registers)}"""
    import __graft_entry__
    from paper_1810_00845_amd import build
    if not os.path.exists(build.LIB):
        __graft_entry__.build()
    with open(build.LIB, "rb") as f:
        blob = f.read()
    # a kernel's metadata are a map sorted by key: .symbol (its name and ".kd"), ..., .vgpr_count, .vgpr_spill_count
    found = re.findall(rb"\.symbol(?:\xda..|\xd9.|[\xa0-\xbf])(\w+)\.kd.{0,200}?\.vgpr_count" + INT + rb"\xb1\.vgpr_spill_count" + INT, blob, re.S)
    return {name.decode(): (value(a), value(b)) for name, a, b in found}


# (mangled name, how many instantiations, most registers)
FIT = [
    (r"_Z27inner_product_sum_fp_kernelILi[14]ELi0EE.*", 2, 96),     # four to eight digits: five waves
    (r"_Z13ntt_fp_kernelILi[45]ELi[346]ELb1EE.*", 6, 80),           # columns at N = 2^14, 2^15: three workgroups of eight waves
    (r"_Z20ntt_fp_chunks_kernelILi[45]ELi[346]EE.*", 6, 128),       # sixteen waves
    (r"_Z20scalar_mac_fp_kernel.*", 1, 80),                         # six waves
    (r"_Z19encrypt_rows_kernelILi[2345]EE.*", 4, 128),              # four waves
]


@pytest.mark.parametrize("name,count,most", FIT)
def test_registers(kernels, name, count, most):
    which = {k: v for k, v in kernels.items() if re.fullmatch(name, k)}
    assert len(which) == count, sorted(which)
    for k, (used, spilled) in which.items():
        assert used <= most and spilled == 0, (k, used, spilled)
