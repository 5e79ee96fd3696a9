"""Inline assembly that writes m0 (the loads that go straight to LDS take their destination from it): the statement says
so, and nothing the compiler emits holds anything else there."""
import os
import re
import subprocess

from paper_1102_0183_amd import build


def test_every_statement_that_writes_m0_declares_it():
    found = 0
    for path in build.sources():
        text = open(path).read()
        for m in re.finditer(r"asm volatile\((.*?)\);", text, flags=re.S):
            if "m0" in m.group(1).split('"::')[0]:
                found += 1
                assert m.group(1).rstrip().endswith('"m0"'), (path, m.group(0))
    assert found >= 2


def test_nothing_else_in_the_batched_pass_uses_m0(tmp_path):
    out = os.path.join(str(tmp_path), "batch.s")
    src = [s for s in build.sources() if s.endswith("cnn355_batch.hip")][0]
    subprocess.run([build.HIPCC] + [f for f in build.FLAGS if f != "-fPIC"] + ["--cuda-device-only", "-S", "-o", out, src], check=True,
                   capture_output=True)
    inside, writes = False, 0
    for line in open(out):
        if "#ASMSTART" in line:
            inside = True
        elif "#ASMEND" in line:
            inside = False
        elif re.search(r"\bm0\b", line.split(";")[0]):
            assert inside, line
            writes += 1
    assert writes > 0
