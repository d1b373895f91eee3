"""The fused sweep's kernels that the library holds (read from the names of its host
stubs): the Jastrow-derivative kernels with the u term spill at more than two waves per SIMD,
so 256-thread ones exist at two only, whatever a tuning asks for (a tuning is
timed without derivatives)."""
import re
import shutil
import subprocess

import pytest

from paper_2507_02888_amd import build as lib_build
from paper_2507_02888_amd import ewald as ew

# k_run<DIM, MIXED, NT, SPT, PPR, JM, PD, ORTHO, XTRA, WV, LAY, QUEUE>
NAME = re.compile(r"__device_stub__k_runI" + "".join(r"L[ib](\d+)E" for _ in range(12)))


@pytest.fixture(scope="module")
def kernels():
    if shutil.which("nm") is None:
        pytest.skip("needs nm")
    ew.load()
    out = subprocess.run(["nm", lib_build.LIB], capture_output=True, text=True, check=True).stdout
    found = {tuple(int(x) for x in m.groups()) for m in NAME.finditer(out)}
    assert found
    return found


def test_derivative_kernels_waves(kernels):
    for dim, mixed, nt, spt, ppr, jm, pd, ortho, xtra, wv, lay, queue in kernels:
        if jm == 4 and nt < 1024:
            assert wv == 2, (dim, mixed, nt, spt)
        if jm == 2 and nt == 256 and dim == 3 and not mixed and spt == 2:
            assert wv <= 3, (dim, mixed, nt, spt)
        if jm == 2 and nt == 512:
            assert wv == 2, (dim, mixed, nt, spt)


def test_shapes_have_kernels(kernels):
    """Every shape that the rules pick exists in each dimension, form and Jastrow mode."""
    for dim in (2, 3):
        for mixed in (0, 1):
            for jm in range(5):
                have = {k[2:5] for k in kernels if k[:2] == (dim, mixed) and k[5] == jm}
                assert have >= {(256, 1, 1), (256, 1, 2), (256, 2, 1), (256, 2, 2), (1024, 1, 1), (512, 2, 2), (512, 4, 2)}
