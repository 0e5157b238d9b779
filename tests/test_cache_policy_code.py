"""CPU check of the compiled code: accesses that bypass the caches do so.  Of a nontemporal and an ordinary load of the same word behind a
condition the compiler makes a single ordinary one, which shows in no result: the last kernel of small rescales left its
operand in the caches and the conversion of the next call wrote a third more slowly over it.
"""
import os
import subprocess

import pytest

from paper_2310_16530_amd import build

# kernel, argument type, mangled start, load or store, count of nontemporal ones (16 words a lane; eight more loads for c')
KERNELS = [("ks_final_kernel<FpAr, 8, FIN_KS>", "FinalArgs", "_Z15ks_final_kernel", "load", 24), ("ks_final_kernel<IntAr, 6, FIN_KS>", "FinalArgs", "_Z15ks_final_kernel", "load", 24),
           ("ks_final_cached_kernel<FpAr, 8>", "FinalArgs", "_Z22ks_final_cached_kernel", "load", 8),
           ("fwd_strided_kernel<FpAr, 8>", "FwdStridedArgs", "_Z18fwd_strided_kernel", "store", 16), ("fwd_strided_cached_kernel<IntAr, 8>", "FwdStridedArgs", "_Z25fwd_strided_cached_kernel", "store", 0),
           ("conv_fwd_strided_kernel<FpAr, 6, CONV_DN, 1, true>", "ConvArgs", "_Z23conv_fwd_strided_kernel", "store", 16),
           ("conv_one_cached_kernel<IntAr, 6, 1>", "ConvArgs", "_Z22conv_one_cached_kernel", "store", 0)]


@pytest.mark.parametrize("kernel,args,mangled,kind,count", KERNELS, ids=lambda v: v.split("<")[0] if isinstance(v, str) and "<" in v else "")
def test_nontemporal_accesses_are_kept(tmp_path, kernel, args, mangled, kind, count):
    src, out = tmp_path / "one.hip", tmp_path / "one.s"
    src.write_text('#include "%s"\ntemplate __global__ void %s(%s, Tables, LimbRun);\n' % (os.path.join(build.CSRC, "kernels.h"), kernel, args))
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + ["--cuda-device-only", "-S", str(src), "-o", str(out)],
                          stderr=subprocess.DEVNULL)
    lines = out.read_text().split("\n")
    start = next(i for i, l in enumerate(lines) if l.startswith(mangled) and l.split(";")[0].strip().endswith(":"))
    end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
    ops = [l.split(";")[0].split() for l in lines[start:end] if l.startswith("\t")]
    found = [o for o in ops if o and o[0].startswith(("global_" + kind, "buffer_" + kind, "flat_" + kind)) and o[-1] == "nt"]
    assert len(found) == count, (kernel, len(found))
