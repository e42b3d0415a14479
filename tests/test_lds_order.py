"""Stage 3 reads the membership words of its LDS window as 16-bit halves and
clears them as 32-bit words, each lane clearing halves that other lanes read:
neither a thread's own dependencies nor the types keep the compiler from
moving the clearing up, so the source has to order the two."""
import os
import re
import subprocess

import pytest

HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_membership_words_are_read_before_they_are_cleared(tmp_path):
    from paper_2508_02751_amd import build as B
    ll = str(tmp_path / "hybrid_group.ll")
    # the kernels' accesses in source order: code as the front end emits it
    r = subprocess.run([HIPCC, *B.FLAGS, "--cuda-device-only", "-Xclang", "-disable-llvm-passes",
                        "-emit-llvm", "-S", os.path.join(B.CSRC, "hybrid_group.hip"), "-o", ll],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    text = open(ll).read()
    bodies = re.findall(r"^define amdgpu_kernel void @\S*hybrid_group_kernel.*?^}", text, re.M | re.S)
    assert len(bodies) == 2, "both forms of the kernel"
    for body in bodies:
        words, events = set(), []
        for line in body.splitlines():
            m = re.match(r"\s*(%\d+) = getelementptr inbounds \[2048 x i32\], ptr addrspacecast", line)
            if m:
                words.add(m.group(1))
            elif re.search(r"= load i16, ptr", line):
                events.append("read")
                # the halves' type may alias the words'
                tag = re.search(r"!tbaa !(\d+)", line)
                base = re.search(rf"^!{tag.group(1)} = !{{!(\d+),", text, re.M)
                assert re.search(rf'^!{base.group(1)} = !{{!"omnipotent char"', text, re.M), line
            elif (m := re.match(r"\s*store i32 0, ptr (%\d+),", line)) and m.group(1) in words:
                events.append("clear")
            elif re.search(r"call void @\S*(wave_lds_fence|__syncthreads)", line):
                events.append("fence")
        assert "read" in events and "clear" in events[events.index("read"):], events
        last = None
        for e in events:
            assert not (last == "read" and e == "clear"), events
            last = e if e in ("read", "fence") else last
