"""The store of device blocks against a book-keeping runtime (tests/pool_driver.cpp), on the CPU."""
import os
import subprocess

from paper_2008_12336_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))


def test_device_blocks_are_bounded_given_back_and_never_lost(tmp_path):
    exe = str(tmp_path / "pool_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-D__HIP_PLATFORM_AMD__", "-fsanitize=address,undefined",
                    "-I/opt/rocm/include", "-I" + os.path.join(B.ROOT, "include"), "-I" + B.CSRC,
                    os.path.join(B.CSRC, "gosh_device_pool.cpp"), os.path.join(HERE, "pool_driver.cpp"), "-o", exe],
                   check=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0")
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60, env=env)
    assert run.returncode == 0 and run.stdout.strip() == "pool ok", run.stdout + run.stderr
