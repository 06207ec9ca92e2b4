"""Registers, scratch memory and LDS of the kernels as built, read from the code objects inside the library: what decides how
many workgroups a compute unit holds, which the launch rules count on."""
import ctypes
import re
import struct
import subprocess

import msgpack
import pytest

from paper_2605_25716_amd import build as fbuild

LDS_BYTES = 160 * 1024  # of a compute unit
LANE_REGS = 512         # registers of a lane over all waves of a SIMD, handed out eight at a time


def _code_objects(path):
    data, at = open(path, "rb").read(), 0
    while (i := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        at = p = i + 32
        for _ in range(struct.unpack_from("<Q", data, i + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + n] and size:
                yield data[i + off:i + off + size]
            p += 24 + n


def _kernels(elf):
    table, (entry, count) = struct.unpack_from("<Q", elf, 0x28)[0], struct.unpack_from("<HH", elf, 0x3A)
    for k in range(count):
        head = struct.unpack_from("<IIQQQQIIQQ", elf, table + k * entry)
        p, end = head[4], head[4] + head[5]
        while head[1] == 7 and p < end:  # notes; 32: the kernels' metadata
            name, size, kind = struct.unpack_from("<III", elf, p)
            p += 12 + (name + 3) // 4 * 4
            if kind == 32:
                yield from msgpack.unpackb(elf[p:p + size])["amdhsa.kernels"]
            p += (size + 3) // 4 * 4


def _functions(elf):
    """(address, name) of the dynamic symbols that are functions"""
    table, (entry, count) = struct.unpack_from("<Q", elf, 0x28)[0], struct.unpack_from("<HH", elf, 0x3A)
    heads = [struct.unpack_from("<IIQQQQIIQQ", elf, table + k * entry) for k in range(count)]
    for head in heads:
        for at in range(head[4], head[4] + head[5], 24) if head[1] == 11 else ():
            name, info, _, _, value, _ = struct.unpack_from("<IBBHQQ", elf, at)
            if info & 15 == 2:
                start = heads[head[6]][4] + name
                yield value, elf[start:elf.index(b"\0", start)].decode()


@pytest.fixture(scope="module")
def kernels():
    """name<template arguments> -> metadata"""
    fbuild.build_library(force=False)
    meta = [k for elf in _code_objects(fbuild.LIB_PATH) for k in _kernels(elf)]
    assert len(meta) > 50
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in meta), capture_output=True, text=True, check=True).stdout
    short = [re.sub(r"^void |fedrag::", "", n.split("(")[0]) for n in names.splitlines()]
    return dict(zip(short, meta))


def workgroups_per_unit(k):
    waves = k[".max_flat_workgroup_size"] // 64
    by_regs = LANE_REGS // ((k[".vgpr_count"] + 7) // 8 * 8) * 4 // waves
    lds = k[".group_segment_fixed_size"]
    return min(by_regs, LDS_BYTES // lds if lds else by_regs)


def test_scratch_memory(kernels):
    """A reload from scratch waits for the loads in flight.  Only the four-wave form of 64 columns on 8-bit codes has any, three
    registers' worth."""
    for name, k in kernels.items():
        spills = re.match(r"prefill_attn_kernel<\w+, 64, false, 8, 4, false, 1>", name)
        assert k[".private_segment_fixed_size"] <= (16 if spills else 0), name


def test_kernels_start_on_pages():
    """So that the time of one does not hang on the sizes of the others in its code object."""
    fbuild.build_library(force=False)
    at = [f for elf in _code_objects(fbuild.LIB_PATH) for f in _functions(elf)]
    assert len(at) > 50 and not [f for f in at if f[0] % 4096]


def test_few_rows_in_64_bits(kernels):
    """Sums in 64 bits: LDS for the rows that the form takes, no more, so that four workgroups of 64 columns share a compute
    unit (two of them took 9.7 us for 64 x 32 slabs of 5 rows, four 6.9)."""
    for st in ("false", "true"):
        assert workgroups_per_unit(kernels[f"few_rows_kernel<F32, 64, false, {st}, true>"]) >= 4


def test_rows_that_fill_half_a_step(kernels):
    """fp32 rows of 64 columns, 32 at most: workgroups of one row tile's two waves, eight of them to a compute unit (they were
    four of four waves, half of them idle)."""
    for scatter in ("false", "true"):
        k = kernels[f"rows_times_matrix_mfma_f32_kernel<64, {scatter}, false, false, 1>"]
        assert k[".max_flat_workgroup_size"] == 128 and workgroups_per_unit(k) >= 8


def test_nothing_is_built_that_no_call_reaches(kernels):
    """Dec with the aggregation takes a matrix, never a key's factors; Dec by a key's factors is no product."""
    merging = [n for n in kernels if re.match(r"rows_times_matrix_mfma_f32_kernel<\d+, \w+, \w+, true, ", n)]
    assert len(merging) == 3 and not any(re.match(r"rows_times_matrix_mfma_f32_kernel<\d+, \w+, true, true, ", n) for n in merging)
    assert not [n for n in kernels if re.match(r"rows_times_matrix_mfma_f32_kernel<\d+, true, true, ", n)]
    few = [n for n in kernels if n.startswith("few_rows_kernel<")]
    assert few and not [n for n in few if ", true, true, " in n]  # <type, d, Dec, key's factors, ...>


def test_residency_that_the_row_products_are_cut_for(kernels):
    """Workgroups a compute unit holds of the fp32 row products are those that the choice of row steps per workgroup counts."""
    counted = ctypes.CDLL(fbuild.LIB_PATH)._ZN6fedrag18row_steps_residentEibb
    counted.argtypes = [ctypes.c_int, ctypes.c_bool, ctypes.c_bool]
    checked = 0
    for name, k in kernels.items():
        m = re.match(r"rows_times_matrix_mfma_f32_kernel<(\d+), \w+, (\w+), (\w+), (\d)>", name)
        if m and (m[1], m[4]) != ("64", "1"):  # (that form has one step)
            assert workgroups_per_unit(k) == counted(int(m[1]), m[2] == "true", m[3] == "true"), name
            checked += 1
    assert checked == 8
