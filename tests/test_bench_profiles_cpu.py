"""CPU: what the benchmark takes a committed counter profile for.

A profile counts only while the sources of the fused kernels are the ones it was
taken on, and belongs to the kernel that the step runs."""
import os
import re

import bench

PRECS = {"fp32": ("flat32_min_sub", range(4, 9)), "fp64": ("flat64_min_sub", range(3, 9))}


def _headers(name, seen):
    text = open(os.path.join(bench.CSRC, name)).read()
    for h in re.findall(r'#include "(fdirw_\w+\.h)"', text):
        if h not in seen and os.path.exists(os.path.join(bench.CSRC, h)):
            seen.add(h)
            _headers(h, seen)
    return seen


def test_every_header_with_kernel_code_is_hashed():
    seen = _headers("fdirw_flat.hip", _headers("fdirw_kernels.hip", set()))
    code = {h for h in seen if "__device__ __forceinline__" in open(os.path.join(bench.CSRC, h)).read()}
    assert "fdirw_device.h" in code and code <= set(bench.KERNEL_SOURCES)


def test_kernel_names_follow_the_dispatch():
    text = open(os.path.join(bench.CSRC, "fdirw_api.cpp")).read()
    for prec, (fn, radii) in PRECS.items():
        body = re.search(r"static int %s\(int r\)\n{(.*?)\n}" % fn, text, re.S).group(1)
        at = {int(r): int(n) for r, n in re.findall(r"case (\d): return (\d+);", body)}
        rest = int(re.search(r"default: return (\d+);", body).group(1))
        assert bench.FLAT_MIN_SUB[prec] == {r: at.get(r, rest) for r in radii}
        for r, n in bench.FLAT_MIN_SUB[prec].items():
            assert bench.fused_kernel(prec, r, n) == "flat_line_kernel"
            assert bench.fused_kernel(prec, r, n - 1) == "line_kernel"
    assert bench.fused_kernel("fp16x32", 8, 200) == "line_kernel"
