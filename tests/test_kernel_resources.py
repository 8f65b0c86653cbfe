"""What kernels leave room for on a compute unit: registers, LDS and waves as the compiler counts them (no GPU)."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

from paper_2302_02390_amd import build as lib_build

GRAD, WEIGHT, CODES = 0, 1, 3
# most registers at which that many waves share a SIMD's 512, in steps of eight
REGISTERS = {7: 72, 6: 80, 5: 96, 4: 128}
# waves and rows of a team -> mode -> waves to a SIMD
NEEDED = {(4, 4): {GRAD: 7, WEIGHT: 7, CODES: 6}, (4, 6): {GRAD: 7, WEIGHT: 7, CODES: 5}, (4, 8): {WEIGHT: 7, CODES: 4},
          (1, 4): {GRAD: 7, WEIGHT: 7, CODES: 7}, (1, 6): {GRAD: 7, WEIGHT: 7, CODES: 5},
          (1, 8): {GRAD: 5, WEIGHT: 7, CODES: 4}}


def _assembly(source, *defines):
    cmd = [lib_build.HIPCC] + lib_build.FLAGS + list(defines)
    cmd += ["--cuda-device-only", "-S", os.path.join(lib_build.CSRC, source), "-o", "-"]
    return subprocess.run(cmd, capture_output=True, text=True, check=True).stdout


def _registers(team):
    waves, rows = team
    asm = _assembly("qsdp_tile_inst.hip", f"-DQSDP_TILE_W={waves}", f"-DQSDP_TILE_R={rows}")
    found = re.findall(rf"\.name:\s+_ZN4qsdp11tile_kernelILi(\d+)ELi{rows}ELi{waves}E.*?\.vgpr_count:\s+(\d+)", asm, re.S)
    return {int(mode): int(n) for mode, n in found}


def test_waves_of_the_tile_kernel():
    """Rows side by side took registers and, with them, waves that the encoders and the code-resident step need."""
    with ThreadPoolExecutor(len(NEEDED)) as ex:
        counts = dict(zip(NEEDED, ex.map(_registers, NEEDED)))
    for team, modes in NEEDED.items():
        for mode, waves in modes.items():
            assert counts[team][mode] <= REGISTERS[waves], (team, mode, counts)


def _fit(values):
    """{bits: (LDS, threads, registers, spilled registers)} of the fit's kernels with that many values to a lane."""
    asm = _assembly("qsdp_fit_inst.hip", f"-DQSDP_FIT_V={values}", "-DQSDP_FIT_W=1")
    found = re.findall(rf"\.group_segment_fixed_size:\s+(\d+).*?\.max_flat_workgroup_size:\s+(\d+)"
                       rf".*?\.name:\s+_ZN4qsdp17fit_levels_kernelILi(\d)ELi{values}ELi1E"
                       rf".*?\.vgpr_count:\s+(\d+)\s+\.vgpr_spill_count:\s+(\d+)", asm, re.S)
    return {int(bits): tuple(map(int, (lds, threads, registers, spilled)))
            for lds, threads, bits, registers, spilled in found}


def test_workgroups_of_the_level_fit():
    """Buckets of up to 256: three workgroups to a compute unit's 160 KB of LDS. Six producers for buckets of 129-256 and,
    for tables of up to 8 levels, of 257-512, eleven for 513-1024, seven otherwise, and the consumer. One workgroup of the
    larger ones to a compute unit, whose LDS their slots take almost whole; no register spilled. At 8 bits registers leave
    two of the small ones."""
    shapes = (2, 4, 8, 16, 32)
    with ThreadPoolExecutor(len(shapes)) as ex:
        kernels = dict(zip(shapes, ex.map(_fit, shapes)))
    for values, widths in kernels.items():
        assert sorted(widths) == list(range(1, 9)), (values, widths)
        for bits, (lds, threads, registers, spilled) in widths.items():
            producers = 11 if values == 16 else 6 if values == 4 or (values == 8 and bits <= 3) else 7
            assert threads == 64 * (producers + 1), (values, bits, threads)
            assert lds <= 160 * 1024 // (3 if values <= 4 else 1), (values, bits, lds)
            # waves to a SIMD: the workgroup's, or those of all
            waves = -(-(producers + 1) * (1 if values > 4 else 3 if bits < 8 else 2) // 4)
            assert spilled == 0 and registers <= 512 // waves // 8 * 8, (values, bits, registers, spilled)


def test_waves_of_the_receive_side_with_adamw():
    """Buckets of 1024: four waves to a SIMD, which take all of its registers."""
    asm = _assembly("qsdp_wave_inst.hip", "-DQSDP_G=64", "-DQSDP_R=4", "-DQSDP_W=1", "-DQSDP_B=1024")
    found = re.findall(r"\.name:\s+_ZN4qsdp11wave_kernelILi7ELi64ELi4ELi(\d)ELi1E.*?\.vgpr_count:\s+(\d+)\s+"
                       r"\.vgpr_spill_count:\s+(\d+)", asm, re.S)
    assert len(found) == 9  # without codes and with 1-8 bits
    for bits, registers, spilled in found:
        assert int(registers) <= REGISTERS[4] and int(spilled) == 0, (bits, registers, spilled)
