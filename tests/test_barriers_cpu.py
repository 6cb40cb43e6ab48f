"""The stage barriers of the bf16 filter gradient that streams its operands into LDS, as the compiler leaves them (no device).

Behind a stage barrier loads overwrite a stage that fragments were read from.  Products wait for the fragments they use, but there are
stages without products, so each wavefront has to have its reads behind it when it comes to the barrier."""
import importlib.util
import os
import re
import subprocess

# (by path: the package loads its library, and the HIP runtime with it, which has to come behind torch's for the GPU tests of the same process)
PACKAGE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1404_5997_amd")
spec = importlib.util.spec_from_file_location("_owt_build", os.path.join(PACKAGE, "build.py"))
build = importlib.util.module_from_spec(spec)
spec.loader.exec_module(build)


def test_every_stage_barrier_waits_for_the_reads_before_it(tmp_path):
    out = str(tmp_path / "k.s")
    subprocess.run([build.HIPCC] + build.FLAGS + ["--cuda-device-only", "-S", "-o", out, os.path.join(build.CSRC, "ifilter16b_inst.hip")],
                   check=True, capture_output=True)
    with open(out) as f:
        text = f.read()
    kernels = re.findall(r"^(_ZN3owt17ifilter16b_kernel\w+):(.*?)^\.Lfunc_end", text, re.M | re.S)
    assert len(kernels) == 7
    for name, body in kernels:
        code = [l.strip() for l in body.splitlines() if l.startswith("\t") and not l.strip().startswith((";", "."))]
        # the walk: from the first read of a fragment (the barrier in front of it has no reads before it) to the last load into LDS
        walk = code[next(i for i, l in enumerate(code) if l.startswith("ds_read")):max(i for i, l in enumerate(code) if l.startswith("buffer_load") and l.endswith(" lds"))]
        barriers = [i for i, l in enumerate(walk) if l.startswith("s_barrier")]
        assert len(barriers) >= 4, name
        for b in barriers:
            assert re.fullmatch(r"s_waitcnt vmcnt\(\d+\) lgkmcnt\(0\)", walk[b - 1]), (name, b, walk[b - 1])
        # (where wavefronts wait for different numbers of loads, one of the two waits is a branch away from the barrier)
        assert all("lgkmcnt(0)" in l for l in walk if l.startswith("s_waitcnt vmcnt")), name
