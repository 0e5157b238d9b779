"""CPU check of the unreduced sums and of the base conversion's recombination (csrc/modarith.h, __host__ __device__).

The checker (tests/host/wide_check.hip) is compiled with hipcc and run on the CPU against 128-bit integer arithmetic:
sums of every allowed number of products, sums of up to 128 products joined from those and multiplied by plaintexts, and
conversions from 1 to 17 sources, with extreme operands, for moduli at the edges of both arithmetics.
"""
import os
import subprocess

from paper_2310_16530_amd import synth

HERE = os.path.dirname(os.path.abspath(__file__))


def test_unreduced_sums_and_recombination_are_exact(tmp_path):
    exe = str(tmp_path / "wide_check")
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O2", "-ffp-contract=off", "--offload-arch=gfx950",
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-o", exe,
                           os.path.join(HERE, "host", "wide_check.hip")], stderr=subprocess.DEVNULL)
    limit = 3 << 48
    moduli = [synth.CFG2.q_primes[0], synth.CFG2.p_primes[0], synth.CFG0.q_primes[0], limit - 1, limit - 7, 844424930123777, 12289, 8191, (1 << 28) - 57,
              limit + 1, limit + 9, (1 << 59) + 55, (1 << 60) - 93, (1 << 61) - 1]
    out = subprocess.run([exe] + [str(m) for m in moduli], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.startswith("OK"), out.stdout + out.stderr
