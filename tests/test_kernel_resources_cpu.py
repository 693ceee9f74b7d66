"""Register budget of the kernels, read from the device compiler's resource
report (no GPU needed).

An 8-wave tile of at most 128x128 outputs is sized to run two workgroups per
compute unit: each wave then has at most 128 VGPRs.  A change that pushes
one of these kernels past that budget, or into scratch, halves its
occupancy or adds memory traffic to every step without changing any result,
so the parity tests cannot see it; this test does.  The 256x256 tile runs
one workgroup per compute unit with up to 256 VGPRs per wave; its fp32
one-product kernel in the RC layout (the cube workloads' kernel) must not
spill.
"""
import concurrent.futures as cf
import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_2006_12645_amd import build as B


def _have_hipcc():
    try:
        return shutil.which(B._hipcc()) is not None
    except RuntimeError:
        return False


pytestmark = pytest.mark.skipif(not _have_hipcc(), reason="hipcc not available")

NAME = re.compile(r"Function Name: (\S+)")
FIELD = re.compile(r"remark:\s+(VGPRs|ScratchSize \[bytes/lane\]|Occupancy \[waves/SIMD\]): (\d+)")
SPILL = re.compile(r"remark:\s+VGPRs Spill: (\d+)")
ARGS = r"gemm_bias_act_%s(I.*)EvNS_8GemmArgsE"


def template_args(mangled, kernel="fast16"):
    """Integer and bool template arguments of a mangled kernel name, in order."""
    m = re.search(ARGS % kernel, mangled)
    return [int(v) for v in re.findall(r"L[ib](-?\d+)E", m.group(1))] if m else None


def resources(unit, tmp):
    src, defines, name = unit
    cmd = ([B._hipcc()] + B.HIPCC_FLAGS + defines +
           ["-Rpass-analysis=kernel-resource-usage", "--cuda-device-only", "-c",
            os.path.join(B.CSRC, src), "-o", os.path.join(tmp, name)])
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out, cur = {}, None
    for line in r.stderr.splitlines():
        m = NAME.search(line)
        if m:
            cur = out.setdefault(m.group(1), {})
            continue
        m = SPILL.search(line)
        if m and cur is not None:
            cur["Spill"] = int(m.group(1))
        m = FIELD.search(line)
        if m and cur is not None:
            cur[m.group(1).split()[0]] = int(m.group(2))
    return out


def kernels_of(source, kernel):
    units = [u for u in B.UNITS if u[0] == source]
    with tempfile.TemporaryDirectory() as tmp, cf.ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as ex:
        reports = list(ex.map(lambda u: resources(u, tmp), units))
    kernels = {}
    for rep in reports:
        for name, res in rep.items():
            args = template_args(name, kernel)
            if args is not None:
                kernels[name] = (args, res)
    assert kernels, f"no {kernel} kernel found in the resource report"
    return kernels


@pytest.fixture(scope="module")
def fast16_kernels():
    return kernels_of("gba_gemm_unit.hip", "fast16")


def test_small_eight_wave_tiles_fit_two_workgroups_per_cu(fast16_kernels):
    checked = 0
    for name, (args, res) in fast16_kernels.items():
        bm, bn, wm, wn = args[:4]
        if wm * wn != 8 or bm * bn > 128 * 128:
            continue
        checked += 1
        assert res["ScratchSize"] == 0, (name, res)
        assert res["VGPRs"] <= 128 and res["Occupancy"] >= 4, (name, res)
    assert checked >= 4 * 4 * 3, checked  # three tiles in every layout and variant


def test_four_wave_tiles_do_not_spill(fast16_kernels):
    for name, (args, res) in fast16_kernels.items():
        bm, bn, wm, wn = args[:4]
        if wm * wn < 8:
            assert res["ScratchSize"] == 0, (name, res)


def test_cube_kernel_does_not_spill(fast16_kernels):
    # <256, 256, 2, 4, SK 1, 2 stages, A row-major, B column-major, fp32
    # accumulation, no prologue, one product, not split>
    want = [256, 256, 2, 4, 1, 2, 0, 1, 0, 0, 0, 0]
    hits = [res for args, res in fast16_kernels.values() if args == want]
    assert len(hits) == 1
    assert hits[0]["ScratchSize"] == 0 and hits[0]["Occupancy"] >= 2, hits[0]


# Registers the 256x256 kernels (all 256 VGPRs in use) spill, by (A layout, B
# layout, fp16 accumulation, prologue, second product): every one not listed
# spills none.  CR fp32 at 12 of them instead of 6 took 27.9 us against 25.3
# on 5176 x 4456 x 128.
SPILLS_256 = {(0, 0, 1, 1, 1): 1, (0, 1, 1, 1, 0): 2, (0, 1, 1, 1, 1): 16, (1, 0, 0, 0, 0): 6, (1, 0, 1, 0, 1): 4,
              (1, 0, 1, 1, 0): 17, (1, 0, 1, 1, 1): 40, (1, 1, 0, 0, 0): 4, (1, 1, 1, 0, 1): 2, (1, 1, 1, 1, 0): 22,
              (1, 1, 1, 1, 1): 49}


def test_256x256_tile_spills_no_more_than_measured(fast16_kernels):
    seen = 0
    for args, res in fast16_kernels.values():
        if args[:6] == [256, 256, 2, 4, 1, 2]:
            seen += 1
            assert res["Spill"] <= SPILLS_256.get(tuple(args[6:11]), 0), (args, res)
    assert seen == 32, seen


def test_few_row_kernels_do_not_spill():
    """<A layout, B layout, row blocks, column blocks>: 16 waves of a workgroup
    have 128 registers each (up to three blocks), 8 have 256."""
    kernels = kernels_of("gba_thin_unit.hip", "thin")
    assert len(kernels) == 4 * 3
    for args, res in kernels.values():
        assert res["Spill"] == 0 and res["ScratchSize"] == 0, (args, res)
        assert res["Occupancy"] >= (4 if args[2] + args[3] <= 3 else 2), (args, res)


def test_unaligned_kernels_spill_no_more_than_measured():
    """<BM, BN, WM, WN, A layout, B layout, fp16 accumulation>: the 128x128
    tile runs two workgroups per compute unit.  The 256x256 one (fp32 only)
    spills, in RC outside its loop."""
    spills = {(256, 0, 0, 0): 7, (256, 0, 1, 0): 36, (256, 1, 1, 0): 38, (128, 0, 1, 1): 3}
    kernels = kernels_of("gba_ragged_unit.hip", "ragged")
    assert len(kernels) == 4 * 5
    for args, res in kernels.values():
        assert res["Spill"] <= spills.get((args[0], *args[4:]), 0), (args, res)
        assert res["Occupancy"] >= (4 if args[0] == 128 else 2), (args, res)
