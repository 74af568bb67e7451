"""Registers of sweep kernels whose speed hangs on the waves that a SIMD holds: compiled for gfx950
alone, each reaches its number of waves and none spills.  (No GPU needed; hipcc is.)"""
import os
import re
import subprocess

import pytest

from paper_1402_4986_amd import build

HIPCC = build._hipcc() if os.path.exists("/opt/rocm/bin/hipcc") else None


def _kernels(tmp_path, source):
    """[(mangled name, waves per SIMD, spilled registers)] of the kernels that `source` instantiates."""
    src = tmp_path / "k.hip"
    src.write_text(source)
    cmd = [HIPCC] + build.HIPFLAGS + ["-I", build.CSRC, "--cuda-device-only", "-c", str(src), "-o", os.devnull,
                                      "-Rpass-analysis=kernel-resource-usage"]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stdout)
    waves = [int(v) for v in re.findall(r"Occupancy \[waves/SIMD\]: (\d+)", r.stdout)]
    spills = [int(v) for v in re.findall(r"VGPRs Spill: (\d+)", r.stdout)]
    assert names and len(names) == len(waves) == len(spills)
    return list(zip(names, waves, spills))


pytestmark = pytest.mark.skipif(HIPCC is None, reason="no hipcc")


@pytest.mark.parametrize("pm", ["PM_1", "PM_2", "PM_3", "PM_4"])
def test_fp64_query_sweep_3d_has_three_waves(tmp_path, pm):
    ks = _kernels(tmp_path, f"""
#include "idw_bwd.hpp"
using namespace idw;
template hipError_t idw::launch_bwd_query_t<double, 3, L_HYBRID, {pm}>(const BwdArgs&, int, int64_t, double4*,
                                                                      hipStream_t);
""")
    assert len(ks) == 3
    for name, waves, spills in ks:
        assert waves >= 3 and spills == 0, (name, waves, spills)


@pytest.mark.parametrize("dim", [2, 3])
def test_dz_alone_with_relative_weights_has_16_queries_per_wave(tmp_path, dim):
    ks = _kernels(tmp_path, f"""
#include "idw_bwd_fused.hpp"
using namespace idw;
template hipError_t idw::launch_bwd_fused_t<float, {dim}, L_HYBRID, PM_GEN, true>(const BwdArgs&, int, int, int64_t,
                                                                                 hipStream_t);
""")
    # <dim, layout, PM_GEN, no dp, no dq, no dx, relative, leave-one-out or not, queries per wave>
    alone = [k for k in ks if f"k_bwd_fused32ILi{dim}ELi3ELi0ELb0ELb0ELb0ELb1E" in k[0]]
    assert len(alone) == 2
    for name, waves, spills in alone:
        assert "ELi16EEE" in name and waves == 4 and spills == 0, (name, waves, spills)
