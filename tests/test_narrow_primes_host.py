"""CPU check of the forward passes that reduce nothing on their way (narrow primes of csrc/modarith.h): the largest moduli of the class, those of the
workloads and small ones, against 128-bit integers (tests/host/narrow_check.hip)."""
import os
import subprocess

from paper_2310_16530_amd import synth

HERE = os.path.dirname(os.path.abspath(__file__))


def test_eight_stages_and_five_products_without_a_reduction(tmp_path):
    exe = str(tmp_path / "narrow_check")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.check_call([hipcc, "-O2", "-ffp-contract=off", "--offload-arch=gfx950", "-Xclang", "-target-feature",
                           "-Xclang", "-packed-fp32-ops", "-o", exe, os.path.join(HERE, "host", "narrow_check.hip")],
                          stderr=subprocess.DEVNULL)
    limit = 17 << 45
    moduli = [limit, limit - 1, limit - 13, synth.CFG2.q_primes[0], synth.CFG4.q_primes[-1], (1 << 49) - 1, synth.CFG0.q_primes[0], 40961, 8193]
    out = subprocess.run([exe] + [str(m) for m in moduli], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.startswith("OK"), out.stdout + out.stderr
