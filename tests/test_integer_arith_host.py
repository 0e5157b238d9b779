"""CPU check of the integer butterflies and products of csrc/modarith.h, whose differences of products are sums with the negative modulus: the
largest modulus they take, those of the workloads and small ones, against 128-bit integers (tests/host/integer_check.hip)."""
import os
import subprocess

from paper_2310_16530_amd import synth

HERE = os.path.dirname(os.path.abspath(__file__))


def test_butterflies_and_products_at_the_ends_of_their_ranges(tmp_path):
    exe = str(tmp_path / "integer_check")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.check_call([hipcc, "-O2", "-ffp-contract=off", "--offload-arch=gfx950", "-Xclang", "-target-feature",
                           "-Xclang", "-packed-fp32-ops", "-o", exe, os.path.join(HERE, "host", "integer_check.hip")],
                          stderr=subprocess.DEVNULL)
    moduli = [(1 << 61) - 1, (3 << 48) + 1, (1 << 50) - 27, 8193] + list(synth.CFG2.primes[-2:]) + list(synth.CFG4.primes[-1:])
    out = subprocess.run([exe] + [str(m) for m in moduli], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.startswith("OK"), out.stdout + out.stderr
