"""What kernels leave room for on a compute unit: registers, LDS and waves as the compiler counts them (no GPU)."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

from paper_2302_02390_amd import build as lib_build

GRAD, WEIGHT, CODES = 0, 1, 3
# most registers at which that many waves share a SIMD's 512, in steps of eight
REGISTERS = {7: 72, 6: 80, 5: 96, 4: 128}
# rows of a team of four waves -> mode -> waves to a SIMD
NEEDED = {4: {GRAD: 7, WEIGHT: 7, CODES: 6}, 6: {GRAD: 7, WEIGHT: 7, CODES: 5}, 8: {WEIGHT: 7, CODES: 4}}


def _assembly(source, *defines):
    cmd = [lib_build.HIPCC] + lib_build.FLAGS + list(defines)
    cmd += ["--cuda-device-only", "-S", os.path.join(lib_build.CSRC, source), "-o", "-"]
    return subprocess.run(cmd, capture_output=True, text=True, check=True).stdout


def _registers(rows):
    asm = _assembly("qsdp_tile_inst.hip", "-DQSDP_TILE_W=4", f"-DQSDP_TILE_R={rows}")
    found = re.findall(rf"\.name:\s+_ZN4qsdp11tile_kernelILi(\d+)ELi{rows}ELi4E.*?\.vgpr_count:\s+(\d+)", asm, re.S)
    return {int(mode): int(n) for mode, n in found}


def test_waves_of_the_tile_kernel():
    """Rows side by side took registers and, with them, waves that the encoders and the code-resident step need."""
    with ThreadPoolExecutor(3) as ex:
        counts = dict(zip(NEEDED, ex.map(_registers, NEEDED)))
    for rows, modes in NEEDED.items():
        for mode, waves in modes.items():
            assert counts[rows][mode] <= REGISTERS[waves], (rows, mode, counts)


def test_workgroups_of_the_level_fit():
    """Buckets of up to 256: three workgroups to a compute unit's 160 KB of LDS. Six producers there and for tables of
    up to 8 levels with buckets of up to 512, seven otherwise, and the consumer."""
    with ThreadPoolExecutor(2) as ex:
        assembly = dict(zip((4, 8), ex.map(
            lambda v: _assembly("qsdp_fit_inst.hip", f"-DQSDP_FIT_V={v}", "-DQSDP_FIT_W=1"), (4, 8))))
    for values, asm in assembly.items():
        found = re.findall(rf"\.group_segment_fixed_size:\s+(\d+).*?\.max_flat_workgroup_size:\s+(\d+)"
                           rf".*?\.name:\s+_ZN4qsdp17fit_levels_kernelILi(\d)ELi{values}ELi1E", asm, re.S)
        assert len(found) == 8
        for lds, threads, bits in (map(int, f) for f in found):
            assert values != 4 or lds <= 160 * 1024 // 3, (bits, lds)
            assert threads == 64 * (7 if values == 4 or bits <= 3 else 8), (values, bits, threads)
