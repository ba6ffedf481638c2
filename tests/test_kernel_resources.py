"""No kernel of the built library keeps registers in scratch memory: a reload inside a main loop waits
behind the copies in flight and undoes their overlap with the products.  Read from the metadata that
the compiler writes into the code objects of this library."""
import os
import struct

import pytest

from paper_2509_13523_amd import build

msgpack = pytest.importorskip("msgpack")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    """The gfx950 ELF images of every offload bundle in a shared library."""
    at = blob.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", blob, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, name_len = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + name_len]
            pos += 24 + name_len
            if b"gfx950" in name and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(MAGIC, at + 1)


def kernel_metadata(elf):
    (shoff,) = struct.unpack_from("<Q", elf, 0x28)
    entry, number = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(number):
        kind, _, _, offset, size = struct.unpack_from("<IQQQQ", elf, shoff + i * entry + 4)
        pos, end = offset, offset + size
        while kind == 7 and pos < end:                       # SHT_NOTE
            name_size, desc_size, note = struct.unpack_from("<III", elf, pos)
            desc = pos + 12 + (name_size + 3) // 4 * 4
            if elf[pos + 12:pos + 18] == b"AMDGPU" and note == 32:
                yield from msgpack.unpackb(elf[desc:desc + desc_size])["amdhsa.kernels"]
            pos = desc + (desc_size + 3) // 4 * 4


def library_kernels():
    with open(build.LIB, "rb") as f:
        blob = f.read()
    return [k for elf in code_objects(blob) for k in kernel_metadata(elf)]


def test_no_kernel_uses_scratch_memory():
    kernels = library_kernels()
    assert sum("winattn_dkdv" in k[".name"] for k in kernels) == 10   # two at 32, 64, 128, pipelined
    bad = {k[".name"]: (k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for k in kernels
           if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]}
    assert not bad


def test_scalar_registers_are_spilled_outside_of_step_loops_only():
    """Scalar values that do not fit are parked in lanes of a vector register.  The three kernels that do so
    fetch them before the loop over steps, per output tile (projection_gemm_kernel) or in the last steps of
    a row range (linear_wgrad_large_kernel), never in the loop that a workgroup spends its time in: read
    from their assembly with these counts.  More of them, or another kernel, has to be looked at again."""
    looked_at = {"projection_gemm_kernel": 7, "linear_wgrad_large_kernel": 14, "winattn_bwd_short_kernelILi128E": 6}
    spills = {k[".name"]: k[".sgpr_spill_count"] for k in library_kernels() if k[".sgpr_spill_count"]}
    more = {n: c for n, c in spills.items() if c > max((v for k, v in looked_at.items() if k in n), default=0)}
    assert not more


def test_bench_and_profiles_name_kernels_of_the_library():
    """bench.py names the kernels that run, and attaches to a kernel only the traffic that a profile
    recorded of it: both by names that the library has."""
    import bench
    names = [k[".name"] for k in library_kernels()]
    has = lambda kernel: any("%d%s" % (len(kernel), kernel) in n for n in names)     # a mangled name
    assert not has("norm_fold") and has("norm_fold_kernel")
    for plan in ((0, 1), (0, 2), (0, 3), (1, 0), (3, 0), (2, 2)):
        for stage in ("fwd", "bwd", "dq", "dkdv"):
            assert all(has(k) for k in bench.kernel_symbol(stage, plan).split(" + ")), (stage, plan)
    folder = os.path.join(bench.ROOT, "profiles")
    lines = [line.split() for name in sorted(os.listdir(folder)) for line in open(os.path.join(folder, name))]
    traffic = [f for f in lines if f and f[0] == "TRAFFIC"]
    assert traffic
    for f in traffic:
        assert len(f) == 5 and has(f[3]) and float(f[4]) > 0, f
        assert bench.profiled_traffic(f[1], f[2], "another_kernel") == {"traffic": None}
