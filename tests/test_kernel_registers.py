"""Registers of the Hogwild kernels, from the metadata of the code objects in the built library.

Both orders of bfloat16 with several samples a wavefront spill nothing: a register that the sampling loop
spills costs a scratch load there, and its wait also waits for the acknowledgements of the stores before it.

One order with a wavefront a sample (bfloat16 up to two units a lane, binary32 with four) stays within 80
registers, six wavefronts per SIMD (512 / 80).  The hot set follows the samples in flight, 256 x 4 x 6 here,
and heats are whole powers of two: rows that a sample touches with probability 2^-13 to 2^-14 are hot at the
default threshold with six (6144 / 0.75 = 2^13) and cold with five.  With six to eight negatives a bfloat16
kernel of that shape has five, 81 to 96 registers, and spills none."""
import re
import struct

import msgpack
import pytest

from paper_2604_09419_amd import build as hipbuild


def _code_objects(data):
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + length]
            p += 24 + length
            if triple.endswith(b"gfx950") and size:
                yield data[at + off:at + off + size]
        at = data.find(magic, at + 24)


def _kernels(elf):
    """The kernels' records of an AMDGPU code object's metadata note."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * shentsize)
        if kind != 7:  # SHT_NOTE
            continue
        namesz, descsz, note = struct.unpack_from("<III", elf, off)
        if note == 32:  # NT_AMDGPU_METADATA
            desc = off + 12 + (namesz + 3) // 4 * 4
            yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]


@pytest.fixture(scope="module")
def kernels():
    with open(hipbuild.SO, "rb") as f:
        data = f.read()
    return {k[".name"]: k for c in _code_objects(data) for k in _kernels(c)}


@pytest.mark.parametrize("lanes,units", [(16, 1), (32, 1), (16, 2), (32, 2)])
def test_both_orders_bfloat16_kernels_spill_nothing(kernels, lanes, units):
    found = [k for name, k in kernels.items()
             if re.search(rf"k_hogwildItLi{lanes}ELi{units}ELi5ELi3ELb0ELb[01]E", name)]
    assert len(found) == 2
    assert [k[".vgpr_spill_count"] for k in found] == [0, 0]


@pytest.mark.parametrize("table,lanes,units,order", [("t", 64, 1, 1), ("t", 64, 1, 2), ("t", 64, 2, 1), ("f", 64, 4, 1),
                                                     ("f", 64, 4, 2)])
def test_one_order_kernels_fit_six_wavefronts(kernels, table, lanes, units, order):
    found = [k for name, k in kernels.items()
             if re.search(rf"k_hogwildI{table}Li{lanes}ELi{units}ELi5ELi{order}ELb0ELb1E", name)]
    assert len(found) == 1
    assert found[0][".vgpr_count"] <= 80


@pytest.mark.parametrize("units", [1, 2])
def test_one_order_kernels_for_more_negatives_keep_five_wavefronts(kernels, units):
    found = [k for name, k in kernels.items() if re.search(rf"k_hogwildItLi64ELi{units}ELi8ELi1ELb0ELb0E", name)]
    assert len(found) == 1
    assert found[0][".vgpr_spill_count"] == 0
    assert 80 < found[0][".vgpr_count"] <= 96


@pytest.mark.parametrize("lanes", [16, 32])
@pytest.mark.parametrize("order", [1, 2])
def test_narrow_four_unit_kernels_spill_nothing(kernels, lanes, order):
    found = [k for name, k in kernels.items() if re.search(rf"k_hogwildItLi{lanes}ELi4ELi5ELi{order}ELb0ELb[01]E", name)]
    assert len(found) == 2
    assert [k[".vgpr_spill_count"] for k in found] == [0, 0]
