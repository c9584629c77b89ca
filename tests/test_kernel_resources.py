"""What the built kernels ask of the hardware, read from the code objects inside the library (no GPU): the sizes and registers that the
kernels' speed rests on and that a change of source or compiler can take away without any result being wrong."""
import re
import struct
import subprocess

import pytest

import paper_2310_03841_amd as ab

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Name -> properties, of every kernel of the library."""
    ab.lib()
    with open(ab.lib_path(), "rb") as f:
        data = f.read()
    out, at, n = {}, 0, 0
    work = tmp_path_factory.mktemp("objects")
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        entries, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(entries):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            p += 24
            if b"gfx950" in data[p:p + length] and size:
                path = work / f"{n}.co"
                n += 1
                path.write_bytes(data[at + off:at + off + size])
                notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
                for text in re.split(r"\n  - (?=\.agpr_count)", notes)[1:]:
                    name = re.search(r"\.name:\s+(_Z\S+)", text).group(1)
                    out[name] = {k: int(re.search(rf"\.{k}:\s+(\d+)", text).group(1)) for k in ("agpr_count", "kernarg_segment_size", "sgpr_spill_count", "vgpr_spill_count")}
            p += length
        at += 24
    return out


def of(kernels, kernel):
    """(template arguments, properties) of a kernel's instantiations."""
    found = []
    for name, k in kernels.items():
        m = re.search(rf"{len(kernel)}{kernel}I((?:L[ib]\d+E)+)E", name)
        if m:
            found.append(([int(x) for x in re.findall(r"L[ib](\d+)E", m.group(1))], k))
    assert found, kernel
    return found


def test_unprotected_tiles_take_few_arguments(kernels):
    """A line of 64 bytes of a launch's arguments that is asked for costs the start of a kernel some 100 clocks: unprotected tiles of the general kernel take
    nothing of the passes over A and B."""
    sizes = {bool(t[4]): set() for t, _ in of(kernels, "gemm_tile_kernel")}
    for t, k in of(kernels, "gemm_tile_kernel"):
        sizes[bool(t[4])].add(k["kernarg_segment_size"])
    assert max(sizes[False]) <= 5 * 64, sizes


def test_fast_tiles_keep_their_accumulators_in_vector_registers(kernels):
    """The epilogue reads accumulators where they are; a built-in or an asm that asks for an accumulation register makes the compiler split a lane's
    registers, and each accumulator is moved before it is used.  Only tiles of both heights with stored sums (STO 2) are built that way."""
    for (dt, mode, sto), k in of(kernels, "gemm_fast_kernel"):
        assert (k["agpr_count"] == 0) == (sto != 2), ((dt, mode, sto), k)
        assert k["vgpr_spill_count"] == 0, ((dt, mode, sto), k)


@pytest.mark.parametrize("kernel", ["gemm_fast_kernel", "item_rows_kernel", "item_cols_kernel"])
def test_phases_read_their_own_arguments(kernels, kernel):
    """Arguments taken from the parameter are held across the loop over tiles or items: 60 to 290 scalars more than there are, which live in lanes of vector
    registers.  Read by phase, the most is 15."""
    for t, k in of(kernels, kernel):
        assert k["sgpr_spill_count"] <= 24 and k["vgpr_spill_count"] <= 1, (t, k)
