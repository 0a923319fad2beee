"""Set-up of the training state under runtime failures, on the CPU: the built
library with the HIP and rocBLAS entry points of host_train_setup.cpp."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_a_failed_setup_is_done_again(tmp_path):
    from paper_2505_14260_amd import msd
    if not os.path.exists(msd.LIB_PATH):
        pytest.skip("libmsd.so not built")
    exe = str(tmp_path / "host_train_setup")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-rdynamic", "-o", exe,
                           os.path.join(HERE, "host_train_setup.cpp"), msd.LIB_PATH,
                           "-Wl,-rpath," + os.path.dirname(msd.LIB_PATH),
                           "-Wl,--allow-shlib-undefined"])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
    assert ", 0 wrong" in r.stdout
