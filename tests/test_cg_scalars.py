"""The Krylov loops' device scalars: a kernel whose workgroups test S->done on entry
must not write it, unless it runs as one workgroup: a workgroup that starts late would
see the flag change between two of its waves, one of which leaves ahead of a barrier."""
import os
import re

CG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_20994_amd", "csrc", "cg.hip")


def _kernels(src):
    """name -> body of every __global__ function"""
    out = {}
    for m in re.finditer(r"__global__\s+void\s+(?:__launch_bounds__\(\w+\)\s+)?(\w+)\s*\(", src):
        at = src.index("{", m.end())
        depth, end = 0, at
        while True:
            depth += {"{": 1, "}": -1}.get(src[end], 0)
            end += 1
            if depth == 0:
                break
        out[m.group(1)] = src[at:end]
    return out


def test_no_kernel_writes_the_flag_that_its_workgroups_test():
    src = re.sub(r"//[^\n]*", "", open(CG).read())
    kernels = _kernels(src)
    testing = {k: b for k, b in kernels.items() if re.match(r"\{\s*if \(S->done\) return;", b)}
    assert {"pcg_update_kernel", "pcg_beta_final"} <= set(testing)     # the parse found them
    for name, body in testing.items():
        if re.search(r"S->done\s*=[^=]", body):
            grids = re.findall(name + r"(?:<[^<>]*>)?<<<([^,]+),", src)
            assert grids and all(g.strip() == "1" for g in grids), name
