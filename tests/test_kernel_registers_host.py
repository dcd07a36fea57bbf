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
    (r"_Z\d+inner_product_sum_(fp|once)_kernelILi[14]ELi0EE.*", 4, 96),     # four to eight digits: five waves
    (r"_Z13ntt_fp_kernelILi[45]ELi[346]ELb1EE.*", 6, 80),           # columns at N = 2^14, 2^15: three workgroups of eight waves
    (r"_Z20ntt_fp_chunks_kernelILi[45]ELi[346]EE.*", 6, 128),       # sixteen waves
    (r"_Z14ntt_int_kernelILi[012]ELi2ELb1EE.*", 3, 64),             # integer columns, columns_waves: eight waves at N <= 2^12,
    (r"_Z14ntt_int_kernelILi3ELi2ELb1EE.*", 1, 72),                 # seven at 2^13,
    (r"_Z14ntt_int_kernelILi[45]ELi2ELb1EE.*", 2, 128),             # four at 2^14 and 2^15,
    (r"_Z14ntt_int_kernelILi6ELi2ELb1EE.*", 1, 256),                # two at 2^16
    (r"_Z21plain_mac_half_kernel.*", 2, 168),                       # three waves: 3072 on the chip
    (r"_Z23rotated_mac_mfma_kernelILi(3ELi[567]|5ELi[56])ELi[123]EE.*", 15, 256),   # two waves, nothing spilled
    (r"_Z20scalar_mac_fp_kernel.*", 1, 80),                         # six waves
    (r"_Z19encrypt_rows_kernelILi[2345]EE.*", 4, 128),              # four waves
]


@pytest.mark.parametrize("name,count,most", FIT)
def test_registers(kernels, name, count, most):
    which = {k: v for k, v in kernels.items() if re.fullmatch(name, k)}
    assert len(which) == count, sorted(which)
    for k, (used, spilled) in which.items():
        assert used <= most and spilled == 0, (k, used, spilled)
