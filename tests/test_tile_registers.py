"""Waves that the tile kernel's shapes leave room for: registers as the compiler counts them (no GPU)."""
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


def _registers(rows):
    cmd = [lib_build.HIPCC] + lib_build.FLAGS + ["-DQSDP_TILE_W=4", f"-DQSDP_TILE_R={rows}", "--cuda-device-only", "-S",
                                                 os.path.join(lib_build.CSRC, "qsdp_tile_inst.hip"), "-o", "-"]
    asm = subprocess.run(cmd, capture_output=True, text=True, check=True).stdout
    found = re.findall(rf"\.name:\s+_ZN4qsdp11tile_kernelILi(\d+)ELi{rows}ELi4E.*?\.vgpr_count:\s+(\d+)", asm, re.S)
    return {int(mode): int(n) for mode, n in found}


def test_waves_of_the_tile_kernel():
    """Rows side by side took registers and, with them, waves that the encoders and the code-resident step need."""
    with ThreadPoolExecutor(3) as ex:
        counts = dict(zip(NEEDED, ex.map(_registers, NEEDED)))
    for rows, modes in NEEDED.items():
        for mode, waves in modes.items():
            assert counts[rows][mode] <= REGISTERS[waves], (rows, mode, counts)
