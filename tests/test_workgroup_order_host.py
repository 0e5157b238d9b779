"""CPU check of the order of workgroups that hold a limb each (csrc/ntt.h, __host__ __device__): compiled with hipcc and run on
the CPU, it decodes whole grids of 1 to 70 limbs and 1 to 128 instances."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_limbs_come_once_and_the_dies_share_them_evenly(tmp_path):
    exe = str(tmp_path / "order_check")
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O2", "-ffp-contract=off", "--offload-arch=gfx950",
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-o", exe,
                           os.path.join(HERE, "host", "order_check.hip")], stderr=subprocess.DEVNULL)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.startswith("OK"), out.stdout + out.stderr
