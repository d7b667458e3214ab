"""The loops that exchange data between workgroups order their stores with waits
written in inline asm.  Such a wait may only be for everything in flight: one
that leaves the last n operations out is right only while the compiler emits
exactly the n loads the source has there, which nothing holds it to (a load whose
value is not used goes, and the wait then lets a store pass)."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1810_08061_amd", "csrc")


def test_waits_count_no_operations():
    waits = {}
    for f in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        with open(f) as fh:
            for n, line in enumerate(fh, 1):
                for count in re.findall(r"vmcnt\(([^)]*)\)", line):
                    waits[f"{os.path.basename(f)}:{n}"] = count
    assert len(waits) >= 4
    assert not {k: v for k, v in waits.items() if v != "0"}
