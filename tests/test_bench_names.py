"""The kernel names bench.py reports are those of the library's kernels as a profiler shows them, so that measured traffic is found
under them."""
import subprocess

import bench
from paper_2011_05630_amd import build


def _library_names():
    out = subprocess.run(["nm", "-C", build.LIB], stdout=subprocess.PIPE, text=True, check=True).stdout
    names = set()
    for line in out.splitlines():
        if " k_" in line:
            names.add(bench.kernel_short_name(line[line.index(" k_") + 1:].replace("__device_stub__", "")))
        elif "__device_stub__k_" in line:
            names.add(bench.kernel_short_name(line[line.index("__device_stub__") + 15:]))
    return names


def test_kernel_names_are_the_librarys():
    names = _library_names()
    for table in (bench.VARIANT_NAME, bench.PW_NAME, bench.PW2_NAME, bench.SKC_NAME, bench.FC_NAME, bench.DW_NAME, bench.C3_NAME):
        for name in table.values():
            assert name in names, (name, sorted(n for n in names if n.startswith(name.split("<")[0])))
    for name in [bench.VARIANT_NAME[16], "k_gap", "k_gap8"]:
        assert name in names, name


def test_split_k_convolutions_are_the_named_ones():
    """The builds of the split-K convolution are those that a layer's filter, or a second operand pair, can ask for: no others."""
    named = {n for n in bench.PW2_NAME.values() if n.startswith("k_skc")}
    for n in bench.SKC_NAME.values():
        named |= {bench.skc_name(n, 1, 1, 0, True), bench.skc_name(n, 3, 3, 1, True), bench.skc_name(n, 5, 5, 2, True)}
        assert bench.skc_name(n, 1, 1, 0, False) == bench.skc_name(n, 1, 1, 1, True) == bench.skc_name(n, 3, 1, 1, True) == n
    assert len(named) == 16 and {n for n in _library_names() if n.startswith("k_skc<")} == named
