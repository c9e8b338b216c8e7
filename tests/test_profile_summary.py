"""The names that profile summaries give kernels, against the symbols of the built library and against the names that
the library gives the kernels it launches."""
import re
import shutil
import subprocess

import pytest

from paper_2502_08145_amd import binding as B
from paper_2502_08145_amd.profile_summary import GEMMS, kernel_key, short


@pytest.fixture(scope="module")
def symbols():
    nm = shutil.which("nm")
    if not nm:
        pytest.skip("nm is missing")
    out = subprocess.run([nm, "-C", B.LIB_PATH], capture_output=True, text=True, check=True).stdout
    found = [m.group(1) for m in re.finditer(r"axonn::__device_stub__(.*)", out)]
    assert len(found) > 50
    return found


def test_every_kernel_of_the_library_has_a_name_of_its_own(symbols):
    names = {s: short("void axonn::" + s) for s in symbols}
    for s, n in names.items():
        assert re.fullmatch(rf"({'|'.join(GEMMS)})[a-z0-9_]*/(NN|NT|TN)|transpose_(tile|window|naive)", n), (s, n)
    gemms = [n for n in names.values() if "/" in n]
    assert len(set(gemms)) == len(gemms)
    # counters are calibrated on the launches of one transpose: no other kernel under its name (the tile kernel has two orders)
    assert sorted(n for n in names.values() if "/" not in n) == ["transpose_naive", "transpose_tile", "transpose_tile", "transpose_window"]


@pytest.mark.parametrize("layout", ["NN", "NT", "TN"])
def test_what_the_library_launches_is_among_them(symbols, layout):
    known = {short(s) for s in symbols}
    shapes = [(640, 640, 2048), (24, 2048, 8192), (1064, 4168, 1608), (2049, 2048, 8192), (4099, 4099, 4099), (2048, 12288, 8192),
              (1024, 1024, 4096), (1024, 3072, 3072), (2048, 4096, 4096), (2048, 1152, 36864), (4096, 16384, 2048), (128, 128, 0)]
    for shape in shapes:
        for kernel in B.kernels(*shape, layout):
            assert kernel_key(kernel, layout) in known, (shape, kernel)
