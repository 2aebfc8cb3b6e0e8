"""LDS reads that are issued in one asm statement and waited for in another: the build looks at the code that came out and
fails where a register is used in between (paper_2407_20496_amd/lds_reads.py).  CPU only; the planted kernel is compiled and
never run."""
import re

import pytest

from paper_2407_20496_amd import build, lds_reads

PLANTED = """#include <hip/hip_runtime.h>
extern "C" __global__ void planted(float* y) {
  __shared__ float s[64];
  s[threadIdx.x] = y[threadIdx.x];
  __syncthreads();
  const unsigned at = threadIdx.x * 4;
  float v, w;
  asm volatile("ds_read_b32 %%0, %%1" : "=&v"(v) : "v"(at));
  %s
  y[threadIdx.x] = w;
}
"""
WAIT = 'asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v));'
COPY = 'asm volatile("v_mov_b32 %0, %1" : "=v"(w) : "v"(v));'


@pytest.mark.timeout(300)
def test_the_build_refuses_a_copy_of_a_register_in_flight(tmp_path):
    good, bad = tmp_path / "good.hip", tmp_path / "bad.hip"
    good.write_text(PLANTED % (WAIT + COPY))
    bad.write_text(PLANTED % (COPY + WAIT))
    build._compile(str(good))
    with pytest.raises(RuntimeError, match="in flight"):
        build._compile(str(bad))


def _text(*lines):
    """Instructions, four bytes each, as `llvm-objdump -d` prints them; "-> n" names the instruction branched to."""
    out = ["0000000000001000 <k>:"]
    for i, line in enumerate(lines):
        ins, _, to = line.partition(" -> ")
        out.append("\t%-58s // %012X: 00000000%s" % (ins, 0x1000 + 4 * i, " <k+0x%x>" % (4 * int(to)) if to else ""))
    return "\n".join(out) + "\n"


READ = "ds_read_b64_tr_b16 v[2:3], v9 offset:16"


@pytest.mark.parametrize("lines,faults", [
    ([READ, "v_mov_b32_e32 v4, v3", "s_waitcnt lgkmcnt(0)", "s_endpgm"], [1]),                     # read of it
    ([READ, "v_accvgpr_write_b32 a0, v2", "s_endpgm"], [1]),
    ([READ, "v_mov_b32_e32 v2, 0", "s_waitcnt lgkmcnt(0)", "s_endpgm"], [1]),                      # write of it
    ([READ, "s_waitcnt vmcnt(0)", "v_add_u32_e32 v1, v2, v1", "s_endpgm"], [2]),                   # another counter
    ([READ, "s_waitcnt vmcnt(3) lgkmcnt(0)", "v_add_u32_e32 v1, v2, v1", "s_endpgm"], []),
    ([READ, "v_mov_b32_e32 v4, v1", "s_waitcnt lgkmcnt(0)", "v_mov_b32_e32 v5, v3", "s_endpgm"], []),
    ([READ, "ds_read_b32 v5, v9", "s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v6, v2", "s_endpgm"], []),   # in order: the first is there
    ([READ, "ds_read_b32 v5, v9", "s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v6, v5", "s_endpgm"], [3]),  # the second is not
    ([READ, "ds_read_b32 v5, v2", "s_waitcnt lgkmcnt(0)", "s_endpgm"], [1]),                        # an address that is in flight
    # round the back edge of a loop; the wait is on the path that leaves it
    (["v_mov_b32_e32 v4, v2", READ, "s_cbranch_scc1 65533 -> 0", "s_waitcnt lgkmcnt(0)", "v_mov_b32_e32 v4, v2", "s_endpgm"], [0, 1]),
    # one of two paths waits
    (["s_cbranch_scc1 2 -> 3", READ, "s_branch 2 -> 5", READ, "s_waitcnt lgkmcnt(0)", "v_mov_b32_e32 v4, v2", "s_endpgm"], [5]),
    (["s_cbranch_scc1 3 -> 4", READ, "s_waitcnt lgkmcnt(0)", "s_branch 2 -> 6", READ, "s_waitcnt lgkmcnt(0)",
      "v_mov_b32_e32 v4, v2", "s_endpgm"], []),
])
def test_what_counts_as_in_flight(lines, faults):
    got = [int(re.search(r": ([0-9a-f]+):", f)[1], 16) for f in lds_reads.violations(_text(*lines))]
    assert got == [0x1000 + 4 * i for i in faults]


@pytest.mark.timeout(300)
def test_built_library(tmp_path):
    """The library that is there: nothing in flight is touched; without their waits the tile kernels' reads would be found, and
    the kernels with private rings are among those whose registers are looked at."""
    rings = planted = 0
    for code in lds_reads.code_objects(build.LIB, str(tmp_path)):
        notes = lds_reads._run(lds_reads.LLVM + "/llvm-readelf", "--notes", code)
        if "RingParams" not in notes:
            continue
        rings += sum("RingParams" in name for name in lds_reads.resources(notes))
        first = lds_reads.disassembly(code).split("\n\n")[2]     # one kernel
        assert not lds_reads.violations(first)
        planted += len(lds_reads.violations(re.sub(r"s_waitcnt lgkmcnt\(0\) ", "s_nop 0 ", first)))
    assert rings >= 60 and planted > 100
    assert lds_reads.check(build.LIB) == []


def test_chains_of_the_assignment_solver_keep_their_registers(tmp_path):
    """One row a column: a link of a path is a dependent chain on one wave, and no form of it spills."""
    forms = 0
    for code in lds_reads.code_objects(build.LIB, str(tmp_path)):
        notes = lds_reads._run(lds_reads.LLVM + "/llvm-readelf", "--notes", code)
        for name, (_, spilled, _) in lds_reads.resources(notes).items():
            if re.search(r"assign_kernelILi\d+ELi\d+ELb[01]ELb0E", name) or re.search(r"assign_tile_kernelILi\dELi\dELi\d+ELb0E", name):
                forms += 1
                assert spilled == 0, (name, spilled)
    assert forms >= 8


def test_sums_of_the_row_search_take_lds_by_the_tile(tmp_path):
    """No room for the tallest tile at every launch: eight workgroups share a unit."""
    sizes = []
    for code in lds_reads.code_objects(build.LIB, str(tmp_path)):
        notes = lds_reads._run(lds_reads.LLVM + "/llvm-readelf", "--notes", code)
        for entry in re.split(r"\n\s*- \.agpr_count:", notes)[1:]:
            if "ocp_sums_kernel" in re.search(r"\n\s*\.name:\s*(\S+)", entry)[1]:
                sizes.append(int(re.search(r"\.group_segment_fixed_size:\s*(\d+)", entry)[1]))
    assert len(sizes) == 2 and max(sizes) == 0, sizes
