"""Kernels that raise the device status word themselves: other workgroups of the same launch may raise it at any
moment, so the early exit has to be one decision per workgroup.  Waves that each read the word for themselves can
disagree, and those that stay wait for LDS words and barriers of those that left.  That depends on timing, so it is
looked for in the sources: in such a kernel every look at the word goes through status_of_workgroup."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_16274_amd", "csrc")
KERNELS = ["fuse_pairs", "plan_tiled_kernel", "plan_kernel", "plan_bitmap_kernel", "plan_split_kernel", "rs_sweep"]


def _kernels():
    """(name, body) of every __global__ function."""
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"__global__\s+void\s+(?:__launch_bounds__\((?:[^()]|\([^()]*\))*\)\s*)?(\w+)\s*\(", text):
            at = depth = text.index("{", m.end())
            depth, k = 0, at
            while True:
                depth += {"{": 1, "}": -1}.get(text[k], 0)
                k += 1
                if depth == 0:
                    break
            yield m.group(1), text[at:k]


def test_the_sources_are_read_as_meant():
    names = [name for name, _ in _kernels()]
    assert set(KERNELS) <= set(names) and len(names) > 60


@pytest.mark.parametrize("name", KERNELS)
def test_one_decision_per_workgroup(name):
    (body,) = [body for kernel, body in _kernels() if kernel == name]
    assert "__syncthreads" in body and re.search(r"atomicMax\((?:prm|g)\.status", body), "it raises the word and its waves meet"
    assert len(re.findall(r"read_status\(", body)) == 1 and len(re.findall(r"status_of_workgroup\(", body)) == 1
    assert not re.search(r"\*\s*(?:prm|g)\.status\b", body) and "index_wanted" not in body
