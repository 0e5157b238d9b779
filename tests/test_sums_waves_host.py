"""CPU check of the rule that lets four wavefronts share a row of several giant-step sums (sums_waves in csrc/kernels.h, __host__
__device__): compiled with hipcc and run on the CPU."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_rows_are_shared_only_by_wavefronts_that_have_a_rotation(tmp_path):
    exe = str(tmp_path / "sums_check")
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O2", "-std=c++17", "-ffp-contract=off", "--offload-arch=gfx950",
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-o", exe,
                           os.path.join(HERE, "host", "sums_check.hip")], stderr=subprocess.DEVNULL)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.startswith("OK"), out.stdout + out.stderr
