"""The kernel names bench.py reports are those of the library's kernels as a profiler shows them, so that measured traffic is found
under them."""
import subprocess

import bench
from paper_2011_05630_amd import build


def test_kernel_names_are_the_librarys():
    out = subprocess.run(["nm", "-C", build.LIB], stdout=subprocess.PIPE, text=True, check=True).stdout
    names = set()
    for line in out.splitlines():
        if " k_" in line:
            names.add(bench.kernel_short_name(line[line.index(" k_") + 1:].replace("__device_stub__", "")))
        elif "__device_stub__k_" in line:
            names.add(bench.kernel_short_name(line[line.index("__device_stub__") + 15:]))
    for table in (bench.VARIANT_NAME, bench.PW_NAME, bench.PW2_NAME, bench.SKC_NAME, bench.FC_NAME, bench.DW_NAME, bench.C3_NAME):
        for name in table.values():
            assert name in names, (name, sorted(n for n in names if n.startswith(name.split("<")[0])))
