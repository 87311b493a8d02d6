"""What the compiler makes of kernels whose speed hangs on it: loads that would wait for a whole stream in flight, and
values that would pass through scratch memory.  Compiles the kernel file to assembly; needs no GPU."""
import os
import re
import subprocess

import pytest

from paper_2502_01941_amd import build


def _kernels(source):
    """{kernel name: its instructions} of one kernel file, with the flags that the library is built with."""
    cmd = [build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, source), "-o", "-"]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    assert proc.returncode == 0, proc.stderr
    names = set(re.findall(r"^\s*\.amdhsa_kernel\s+(\S+)", proc.stdout, re.M))
    kernels, current = {}, None
    for line in proc.stdout.splitlines():
        label = re.match(r"(_Z\w+):", line)
        if label:
            current = label.group(1) if label.group(1) in names else None
            kernels.setdefault(current, [])
        elif line.startswith("\t.section") or line.startswith(".Lfunc_end"):
            current = None
        elif current and re.match(r"\t[a-z]", line):
            kernels[current].append(line.strip())
    kernels.pop(None, None)
    assert kernels and set(kernels) == names and all(kernels.values())
    return kernels


@pytest.mark.parametrize("source", ["prefill_score_mfma.hip", "prefill_reduce.hip", "decode_mfma.hip"])
def test_no_generic_or_scratch_access(source):
    """A load through a generic pointer (global memory or LDS, decided at run time) waits for all vector memory, the
    blocks in flight included; scratch is memory too."""
    for name, code in _kernels(source).items():
        found = [i for i in code if i.startswith(("flat_load", "flat_store", "scratch_load", "scratch_store"))]
        assert not found, (name, found)


@pytest.mark.parametrize("D", [64, 128])
def test_shared_fp32_parts_are_made_once(D):
    """fp32 scores: where the four or eight waves of a workgroup split a block of keys into bf16 parts between them, none
    splits one for itself as well: such a kernel has a fraction of the conversions of the two-wave kernel, in which every
    wave does (five times all of a block's, one for each form that a block can take)."""
    count = {}
    for name, code in _kernels("prefill_score_mfma.hip").items():
        form = re.search(r"score_partials_mfma_kernelIfLi%dELi\dELi(\d)ELb(\d)E" % D, name)
        if form:
            count[form.groups()] = sum(i.startswith("v_cvt_pk_bf16_f32") for i in code)
    own, shared = count[("2", "0")], [count[f] for f in (("4", "1"), ("8", "1"))]
    assert own > 0 and all(0 < n < own / 3 for n in shared), (own, shared)


def test_segment_ends_do_not_wait_for_the_stream():
    """Fused attention: the end of the next segment comes out of a register's lanes.  Where the load that fills the register
    every 64 segments is not waited for in its own branch, every end waits for all vector memory: the blocks in flight and
    the statistic just stored."""
    for name, code in _kernels("prefill_attention.hip").items():
        found = [(code[i - 1], line) for i, line in enumerate(code)
                 if line.startswith("v_readlane_b32") and code[i - 1].startswith("s_waitcnt") and "vmcnt" in code[i - 1]]
        assert not found, (name, found)
