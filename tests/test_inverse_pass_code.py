"""CPU check of the compiled first inverse pass: the twiddles of its last four stages are requested together, before the
exchange that feeds those stages is read back.  Requested stage by stage each stage waits for its own (24 x 8 integer limbs at
N = 2^16: 56.6 us against 53.1), which is what the compiler arranges when nothing holds it back.
"""
import os
import subprocess

import pytest

from paper_2310_16530_amd import build

KERNELS = ["inv_contig_kernel<IntAr, 8, INV_PLAIN>", "inv_contig_kernel<IntAr, 8, INV_TENSOR>", "inv_contig_kernel<IntAr, 6, INV_ROT>",
           "inv_contig_kernel<FpAr, 8, INV_PLAIN>"]


@pytest.mark.parametrize("kernel", KERNELS)
def test_last_twiddles_are_requested_before_the_exchange_is_read(tmp_path, kernel):
    src, out = tmp_path / "one.hip", tmp_path / "one.s"
    src.write_text('#include "%s"\ntemplate __global__ void %s(InvContigArgs, Tables, LimbRun);\n'
                   % (os.path.join(build.CSRC, "kernels.h"), kernel))
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + ["--cuda-device-only", "-S", str(src), "-o", str(out)],
                          stderr=subprocess.DEVNULL)
    lines = out.read_text().split("\n")
    start = next(i for i, l in enumerate(lines) if l.startswith("_Z17inv_contig_kernel") and l.split(";")[0].strip().endswith(":"))
    end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
    ops = [l.split()[0] for l in lines[start:end] if l.startswith("\t") and l.split()]
    last_read = max(i for i, op in enumerate(ops) if op.startswith("ds_read"))
    assert any(op.startswith("global_load") for op in ops[:last_read])
    assert not any(op.startswith("global_load") for op in ops[last_read:])
