"""The record kernels reach every plane of a record as global memory: a plane
pointer whose address space the compiler lost becomes a FLAT access, counted
with the LDS accesses and addressed through vector registers.  The kernels are
cross-compiled for gfx950 and their assembly is read; no GPU is needed."""

import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2309_04909_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"

# N, its default field, and the plane accesses of one element: the words of
# the shuffle, of the masks and of the ReLU's triple
KERNELS = [(8, "FieldPM<8, 5u>", "true", 2 + 2 + 1), (19, "FieldMersenne<19>", "false", 5 + 13),
           (19, "FieldMersenne<19>", "true", 5 + 13 + 1), (33, "FieldPM33", "false", 9 + 66)]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_no_flat_accesses(tmp_path):
    lines = ['#include "pre_kernel.h"', "namespace bc {"]
    for n, field, relu, _ in KERNELS:
        for nt in ("true", "false"):
            lines.append(f"template __global__ void k_expand<uint64_t, {n}, {field}, {relu}, {nt}>(ExpandKArgs, {field});")
            lines.append(f"template __global__ void k_drelu_pre<uint64_t, {n}, {field}, {relu}, false, {nt}>(PreKArgs, {field});")
    src, out = tmp_path / "planes.hip", tmp_path / "planes.s"
    src.write_text("\n".join(lines + ["}", ""]))
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "-mllvm", "-pragma-unroll-threshold=200000", f"-I{CSRC}",
                        "--cuda-device-only", "-S", str(src), "-o", str(out)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    counts, kernel = {}, None
    for line in out.read_text().splitlines():
        label = re.match(r"^(_ZN2bc\w+):", line)
        if label:
            kernel = counts.setdefault(label.group(1), {"flat": 0, "store": 0, "load": 0})
        elif kernel is not None:
            op = line.split()[0] if line.split() else ""
            kernel["flat"] += op.startswith("flat_")
            kernel["store"] += op.startswith("global_store")
            kernel["load"] += op.startswith("global_load")
    assert len(counts) == 4 * len(KERNELS)
    for name, c in counts.items():
        assert c["flat"] == 0, (name, c)
    for n, _, relu, planes in KERNELS:
        tag = f"Li{n}E"
        relu_tag = "Lb1E" if relu == "true" else "Lb0E"
        expand = [c for k, c in counts.items() if "k_expand" in k and tag in k and re.search(rf"E{relu_tag}Lb[01]EE", k)]
        assert len(expand) == 2 and all(c["store"] >= planes for c in expand), (n, relu, expand)
