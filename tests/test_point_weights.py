"""The interpolation in difference form, which divides by the linear weights
gamma0 and d0, against the direct form over the whole range of weights that a
problem may have, built for and run on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_difference_form_takes_every_accepted_weight(tmp_path):
    hipcc = shutil.which('hipcc') or '/opt/rocm/bin/hipcc'
    if not os.path.exists(hipcc):
        pytest.skip('hipcc not available')
    exe = str(tmp_path / 'point_weights_check')
    subprocess.run([hipcc, '-O1', '-std=c++17', '--offload-arch=gfx950',
                    f'-I{os.path.join(ROOT, "paper_2411_11229_amd", "csrc")}',
                    os.path.join(ROOT, 'tests', 'cpu_math', 'point_weights_check.cpp'), '-o', exe],
                   check=True, capture_output=True, text=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    print(res.stdout)
    assert res.returncode == 0 and 'ALL OK' in res.stdout, res.stdout + res.stderr
