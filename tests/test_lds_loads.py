"""Kernels that load from memory straight to LDS: other wavefronts read what a
load left there, so the loading wavefront waits for its own loads before the
barrier ahead of those reads, in the source and not by the compiler's choice."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2301_06384_amd", "csrc")
WAIT = r'asm volatile\("s_waitcnt vmcnt\(0\)" ::: "memory"\);\s*__syncthreads\(\);'


def kernels(text):
    """(name, body) of each kernel, comments removed."""
    text = re.sub(r"//[^\n]*", "", text)
    at = [m.start() for m in re.finditer(r"__global__", text)] + [len(text)]
    for a, b in zip(at, at[1:]):
        yield re.search(r"(\w+_kernel)\(", text[a:b]).group(1), text[a:b]


def test_barriers_wait_for_loads_to_lds():
    found = 0
    for f in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, f)) as fh:
            text = fh.read()
        if "global_load_lds" not in text:
            continue
        for name, body in kernels(text):
            if "global_load_lds" not in body:
                continue
            found += 1
            helper = re.search(r"auto (\w+) = \[&\]\(\) \{\s*" + WAIT, body)
            assert helper, f"{name}: no barrier that waits for the loads"
            wait = helper.group(1) + "();"
            # every call that issues loads is followed by that barrier
            main = body[helper.end():]
            calls = [m.start() for m in re.finditer(r"(?<!auto )\bload\(", main)]
            assert calls and all(main.find(helper.group(1) + "();", c) > 0 for c in calls), name
    assert found >= 1
