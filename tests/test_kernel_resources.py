"""CPU test of what the compiler gives the dK/dV kernels that run whole key tiles: no
register spilled to memory (a spill in the rotary epilogue cost 1% of the pass), so the
parts of cut tiles stay in kernels of their own."""
import os
import re
import subprocess

from paper_2602_24082_amd import build


def test_whole_tile_dkdv_spills_nothing(tmp_path):
    cmd = [build.hipcc(), *build.COMMON, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-x", "hip", "-c",
           os.path.join(build.CSRC, "pp_attn_bwd.hip"), "-o", str(tmp_path / "bwd.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    seen = {}
    for block in r.stderr.split("Function Name: ")[1:]:
        name = block.split()[0]
        # template arguments: head size, element type, rotary, stored dS, cut
        m = re.search(r"bwd_dkdv_kernelILi(64|128)E(DF16b|f)Lb([01])ELb([01])ELb([01])E", name)
        if m and m.group(5) == "0":
            seen[m.groups()] = [int(re.search(k + r"[^:]*: (\d+)", block).group(1)) for k in ("ScratchSize", "VGPRs Spill")]
    assert len(seen) == 16
    assert all(v == [0, 0] for v in seen.values()), seen
