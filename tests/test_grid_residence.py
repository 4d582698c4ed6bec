"""The blocks of a launch with grid barriers have to be resident together beside
those of the other hardware queues' launches: what the compiler made of those
kernels must leave room for the blocks a CU that the launches count on.  Reads
the compiler's resource report; no GPU."""
import os
import re
import subprocess

from paper_2503_18056_amd import build


def _resources():
    r = subprocess.run([build._hipcc(), *build.FLAGS, "-w", "--cuda-device-only",
                        "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(build.CSRC, "k_eig.hip"),
                        "-o", os.devnull], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out, name = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"remark:\s+(Function Name|Occupancy \[waves/SIMD\]|LDS Size \[bytes/block\]): (\S+)", line)
        if m and m.group(1) == "Function Name":
            name = m.group(2)
        elif m:
            out.setdefault(name, {})[m.group(1)[:3]] = int(m.group(2))
    return out


def test_blocks_a_cu_of_the_grid_barrier_kernels():
    res = _resources()
    # kernel, wavefronts a block, blocks a CU that its launches count on
    for kernel, waves, blocks in [("k_sytrd_gridILb0E", 4, 2), ("k_sytrd_gridILb1E", 4, 1),
                                  ("k_gebrd", 8, 1), ("k_dc_fused", 8, 1)]:
        found = [v for k, v in res.items() if kernel in k]
        assert len(found) == 1, (kernel, sorted(res))
        print(kernel, found[0])
        assert found[0]["Occ"] * 4 >= waves * blocks, (kernel, found[0])
