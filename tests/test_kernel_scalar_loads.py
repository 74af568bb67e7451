"""The FP64 dz and dx pass over the flagged queries is a serial chain of loads that are the same for every lane:
compiled for gfx950, its loop reads all of them through the scalar cache.  (No GPU needed; hipcc is.)"""
import os
import re
import subprocess

import pytest

from paper_1402_4986_amd import build

HIPCC = build._hipcc() if os.path.exists("/opt/rocm/bin/hipcc") else None
pytestmark = pytest.mark.skipif(HIPCC is None, reason="no hipcc")


@pytest.mark.parametrize("layout", ["L_SOA", "L_AOS", "L_AOAS", "L_HYBRID", "L_SOAOS"])
def test_flagged_queries_are_read_by_scalar_loads(tmp_path, layout):
    src, out = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text("#include \"idw_bwd.hpp\"\nusing namespace idw;\n" + "\n".join(
        f"template hipError_t idw::launch_bwd_fix_t<{t}, {dim}, {layout}, {pm}>(const BwdArgs&, hipStream_t);"
        for t, dim, pm in [("float", 2, "PM_2"), ("float", 3, "PM_GEN"), ("double", 2, "PM_GEN"),
                           ("double", 3, "PM_3")]))
    cmd = [HIPCC] + build.HIPFLAGS + ["-I", build.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(out)]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    kernels = re.findall(r"^(_ZN3idw10k_bwd_fixz\S*):(.*?)^\t\.section", out.read_text(), re.S | re.M)
    assert len(kernels) == 4
    for name, body in kernels:
        blocks = re.split(r"^(?=\.LBB\d+_\d+:)", body, flags=re.M)
        # the loop over the flagged queries is the one that holds scalar loads (dp's hold none)
        heads = [re.match(r"\.L(BB\d+_\d+):", b).group(1) for b in blocks if b.startswith(".LBB")
                 and "Loop Header" in b.split("\n")[0] and re.search(r"^\ts_load_", b, re.M)]
        assert len(heads) == 1, (name, heads)
        loop = [b for b in blocks if b.startswith(f".L{heads[0]}:") or f"Header={heads[0]} " in b]
        vector = re.findall(r"^\t((?:global|flat|buffer)_load.*)", "".join(loop), re.M)
        assert not vector, (name, vector)
