"""Each marching kernel's strip height comes from its own occupancy: the library
holds one cache entry for every such kernel (with fewer, two kernels would share
one, and which of them is called first in a process would decide the other's
strips and with them the adjoint's order of summation)."""
import shutil
import subprocess

import pytest

from paper_2411_11229_amd import hweno as H


def test_one_cache_entry_per_marching_kernel():
    if not shutil.which('nm'):
        pytest.skip('nm not available')
    out = subprocess.run(['nm', H.LIB_PATH], check=True, capture_output=True, text=True).stdout
    names = set(line.split()[-1] for line in out.splitlines() if line)
    kernels = [n for n in names if '__device_stub__stage2d_kernel' in n or '__device_stub__vjp_y_kernel' in n]
    caches = [n for n in names if 'occupancy' in n and 'per_cu_cache' in n]
    assert kernels and len(caches) == len(kernels)
