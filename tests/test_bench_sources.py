"""The hash that ties a counter file to the kernels it was measured on covers
every file that holds or is included by a kernel."""

import importlib.util
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1711_08935_amd", "csrc")


def test_hash_covers_every_kernel_source():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    text = {f: open(os.path.join(CSRC, f)).read() for f in os.listdir(CSRC) if f.endswith((".h", ".hip", ".cpp"))}
    kernels = {f for f, t in text.items() if "__global__" in t}
    todo, seen = list(kernels), set()
    while todo:
        f = todo.pop()
        if f in seen or f not in text:
            continue
        seen.add(f)
        todo += re.findall(r'#include "([^"]+)"', text[f])
    assert {"k_bloch.hip", "k_coulomb.hip", "k_small.hip", "k_project_mom.h"} <= kernels
    # the host file includes launch headers only and holds the static scratch array, no kernel
    assert seen - {"hub_api.hip"} <= set(bench.KERNEL_SOURCES)
