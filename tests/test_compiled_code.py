"""CPU checks of the compiled code: what a kernel must not carry, which shows in no result."""
import os
import re
import subprocess

import pytest

from paper_2310_16530_amd import build


def _assembly(tmp_path, kernel, args, mangled):
    """lines of the kernel's code, and those of the resource summary that follows it"""
    src, out = tmp_path / "one.hip", tmp_path / "one.s"
    src.write_text('#include "%s"\ntemplate __global__ void %s(%s);\n' % (os.path.join(build.CSRC, "kernels.h"), kernel, args))
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + ["--cuda-device-only", "-S", str(src), "-o", str(out)],
                          stderr=subprocess.DEVNULL)
    lines = out.read_text().split("\n")
    start = next(i for i, l in enumerate(lines) if l.startswith(mangled) and l.split(";")[0].strip().endswith(":"))
    end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
    return lines[start:end], lines[end:]


@pytest.mark.parametrize("arith,logN", [("IntAr", 14), ("IntAr", 16), ("FpAr", 16)])
def test_conversions_with_ordinary_stores_hold_no_inverse_pass(tmp_path, arith, logN):
    """Their sources are coefficients: a barrier for the twiddles and one for the exchange of each target (a second one before every
    exchange but the first).  The inverse pass of a source has barriers of its own."""
    targets = 4 if arith == "FpAr" else 1
    code, _ = _assembly(tmp_path, "conv_one_cached_kernel<%s, %d, %d>" % (arith, logN - 8, targets), "ConvArgs, Tables, LimbRun", "_Z22conv_one_cached_kernel")
    barriers = sum(1 for l in code if re.match(r"\s+s_barrier\b", l))
    assert barriers <= (2 if targets == 1 else 3), barriers


@pytest.mark.parametrize("logN", [12, 16])
def test_joint_inner_product_of_a_merged_rescale_spills_nothing(tmp_path, logN):
    """256 registers, all taken: an address computed before the accumulation loop and used after it goes to scratch memory."""
    _, summary = _assembly(tmp_path, "ks_inner_kernel<AnyAr, %d, OWN_TENSOR, false, false>" % (logN - 8), "InnerArgs, Tables, LimbRun", "_Z15ks_inner_kernel")
    assert int(re.search(r"; ScratchSize: (\d+)", "\n".join(summary)).group(1)) == 0


@pytest.mark.parametrize("own", ["OWN_COPY", "OWN_TENSOR", "OWN_ROT", "OWN_ROT_SUM"])
def test_integer_inner_product_keeps_its_twiddle_addresses_out_of_scratch_memory(tmp_path, own):
    """The transforms that end the two components read the same twiddles: their addresses, computed once for both, filled 348 to 480 bytes."""
    _, summary = _assembly(tmp_path, "ks_inner_kernel<IntAr, 8, %s, false, true>" % own, "InnerArgs, Tables, LimbRun", "_Z15ks_inner_kernel")
    assert int(re.search(r"; ScratchSize: (\d+)", "\n".join(summary)).group(1)) <= 32
