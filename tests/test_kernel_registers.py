"""Registers of the compression kernels, of the small fp32 scan and of the backward kernels, as the compiler reports them (CPU: nothing
is run): vector registers and scratch memory.  Scalar registers a build has too many of lie in lanes of vector ones and are not looked at.
In the two-role kernel a SIMD holds a wave of either role, 256 registers each.  A build that wants more keeps the rest in scratch memory: the
logit waves of width 21 then read addresses back in front of every walk, 1 % of a step of several chains."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2406_05317_amd import build as lib_build

TEXT = """#include "compress_roles.h"
using namespace lococo;
using namespace lococo::compress_detail;
template <int KW, int NORM, int PROT, int MULTI, int SPLIT, int CIN>
__global__ __launch_bounds__(kRoleThreads, 2) void roles_k(ScanArgs sa, const uint16_t* wp, int64_t wp_head_stride) {
  extern __shared__ __align__(16) unsigned char smem[];
  compress_roles<KW, NORM, PROT, MULTI, SPLIT, CIN>(sa, wp, wp_head_stride, smem, blockIdx.x, gridDim.x);
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_builds_without_protected_slots_keep_everything_in_registers(tmp_path):
    # one workgroup per (chain, slot tile); several chains per workgroup; pairs that take the steps in turn, filters over
    # [K | V] and over the keys
    builds = [(kw, 1, 0, *form) for kw in (15, 21) for form in ((0, 0, 1), (1, 0, 1), (0, 2, 1), (0, 2, 0))]
    src = tmp_path / "roles.hip"
    src.write_text(TEXT + "".join(f"template __global__ void roles_k<{', '.join(map(str, b))}>(ScanArgs, const uint16_t*, int64_t);\n"
                                  for b in builds))
    r = subprocess.run(["hipcc", "-x", "hip", *lib_build.FLAGS, *lib_build.COMPRESS, "--cuda-device-only", "-c", str(src), "-o",
                        str(tmp_path / "roles.o"), "-Rpass-analysis=kernel-resource-usage"],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    spilled = [int(n) for n in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    assert len(names) == len(spilled) == len(builds)
    assert not any(spilled), dict(zip(names, spilled))


TILE_TEXT = """#include "compress_tile.h"
using namespace lococo;
using namespace lococo::compress_detail;
template <int BM, int KW, int NORM, int PROT, int MULTI, int SPLIT, int LOG>
__global__ __launch_bounds__(kThreads, 1) void tile_k(ScanArgs sa, const uint16_t* wp, int64_t wp_head_stride) {
  extern __shared__ __align__(16) unsigned char smem[];
  const uint32_t wg_id = blockIdx.x, wg_count = gridDim.x;
#include "compress_tile.inl"
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_scan_builds_of_32_slots_keep_everything_in_registers(tmp_path):
    """One chain a workgroup, nothing protected, steps in turn by pairs or not.  Where the last step's choice of a place had put six
    registers into scratch memory, scans of 132 steps on 512 slots took 1.5 % longer."""
    builds = [(32, kw, norm, 0, 0, split, log) for kw in (15, 21) for norm in (0, 1) for split in (0, 2) for log in (0, 1)]
    src = tmp_path / "tile.hip"
    src.write_text(TILE_TEXT + "".join(f"template __global__ void tile_k<{', '.join(map(str, b))}>(ScanArgs, const uint16_t*, int64_t);\n"
                                       for b in builds))
    r = subprocess.run(["hipcc", "-x", "hip", *lib_build.FLAGS, *lib_build.COMPRESS, "--cuda-device-only", "-c", str(src), "-o",
                        str(tmp_path / "tile.o"), "-Rpass-analysis=kernel-resource-usage"],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    spilled = [int(n) for n in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    assert len(names) == len(spilled) == len(builds)
    assert not any(spilled), dict(zip(names, spilled))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("source", ["bwd_attn_mfma.hip", "bwd_conv_mfma.hip"])
def test_backward_kernels_keep_everything_in_registers(tmp_path, source):
    """A reload from scratch memory inside their loops waits for every load on its way: the tiles, rows and filters requested ahead."""
    r = subprocess.run(["hipcc", "-x", "hip", *lib_build.FLAGS, *lib_build.EXTRA[source], "--cuda-device-only", "-c",
                        os.path.join(lib_build.CSRC, source), "-o", str(tmp_path / "bwd.o"), "-Rpass-analysis=kernel-resource-usage"],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    spilled = [int(n) for n in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    scratch = [int(n) for n in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    assert names and len(names) == len(spilled) == len(scratch)
    assert not any(spilled) and not any(scratch), dict(zip(names, zip(spilled, scratch)))
    # one tile a wave: two workgroups of eight waves to a compute unit, registers and LDS allowing
    waves = dict(zip(names, (int(n) for n in re.findall(r"Occupancy \[waves/SIMD\]: (\d+)", r.stderr))))
    rows = {n: w for n, w in waves.items() if "bwd_rows_kILi1ELb0E" in n}
    assert len(rows) == (4 if source == "bwd_conv_mfma.hip" else 0) and all(w >= 4 for w in rows.values()), rows


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_small_scan_kernels_keep_everything_in_registers(tmp_path):
    """compress64_k: 15 builds of a width and a number of slot tiles, each for either kind of Eq. 6."""
    r = subprocess.run(["hipcc", "-x", "hip", *lib_build.FLAGS, "--cuda-device-only", "-c", os.path.join(lib_build.CSRC, "scan_small.hip"),
                        "-o", str(tmp_path / "small.o"), "-Rpass-analysis=kernel-resource-usage"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    spilled = [int(n) for n in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    scratch = [int(n) for n in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    assert len(names) == len(spilled) == len(scratch) and sum("compress64_k" in n for n in names) == 30
    assert not any(spilled) and not any(scratch), dict(zip(names, zip(spilled, scratch)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_step_kernels_take_nothing_that_only_scans_use(tmp_path):
    """Scan and step kernels share their arguments, and a single step waits for them: where a scan over the keys leaves its last state
    has to share its place with the area of [K | V] filters (with room of its own a step of 77 tokens on 256 slots took 1 % longer)."""
    src = tmp_path / "args.hip"
    src.write_text("""#include "lococo_internal.h"
using lococo::ScanArgs;
static_assert(offsetof(ScanArgs, last_k) == offsetof(ScanArgs, prelogits) && offsetof(ScanArgs, last_v) == offsetof(ScanArgs, pre_stride), "");
static_assert(sizeof(ScanArgs) - sizeof(lococo::StepArgs) == 144, "bytes a step kernel takes beside the step's own");
""")
    r = subprocess.run(["hipcc", "-x", "hip", *lib_build.FLAGS, "--cuda-host-only", "-include", "cstddef", "-c", str(src), "-o",
                        str(tmp_path / "args.o")], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
