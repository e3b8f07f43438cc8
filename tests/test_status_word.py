"""Host-side guard (no GPU) for kernels that set the call's status word themselves and whose waves meet at barriers: a wave
that reads the word on its own may see an error that another workgroup of the launch has just set, leave, and be missing in
what the others sum and share.  Such a kernel asks once per workgroup."""
import glob
import os
import re

import pytest

from paper_2209_12769_amd import build

SINGLE = re.compile(r"if \((?:a\.)?status\[0\] != 0\) return;")


def functions(text):
    """name -> (is a kernel, body) of every function of a source file."""
    out = {}
    text = re.sub(r"__launch_bounds__\([^()]*\)|__attribute__\(\((?:[^()]|\([^()]*\))*\)\)", "", text)
    for m in re.finditer(r"^[\w<>_ :*&,()\[\]]*?(\w+)\([^;{}]*\) *\{$", text, re.M | re.S):
        depth, i = 1, m.end()
        while depth:
            depth += {"{": 1, "}": -1}.get(text[i], 0)
            i += 1
        out[m.group(1)] = ("__global__" in m.group(0), text[m.end():i])
    return out


def offenders(text):
    fs = functions(text)
    reaches = {n for n, (_, b) in fs.items() if "set_error(" in b}
    reaches |= {n for n, (_, b) in fs.items() if any(re.search(rf"\b{r}(<[^;()]*>)?\(", b) for r in reaches)}
    bad = []
    for n in sorted(reaches):
        kernel, body = fs[n]
        one_workgroup = re.search(rf"hipLaunchKernelGGL\(\(?{n}[^;]*?, dim3\(1\),", text, re.S)
        if kernel and not one_workgroup and SINGLE.search(body) and ("__syncthreads" in body or "contract_one" in body):
            bad.append(n)
    return bad, reaches


def test_the_check_finds_a_wave_that_leaves():
    text = """
__global__ __launch_bounds__(256) void k_kernel(int* status) {
  if (status[0] != 0) return;
  __syncthreads();
  if (threadIdx.x == 0) set_error(status, 3);
}
"""
    assert offenders(text)[0] == ["k_kernel"]
    assert offenders(text.replace("if (status[0] != 0) return;", "if (call_failed(status)) return;"))[0] == []


@pytest.mark.parametrize("path", build.sources(), ids=os.path.basename)
def test_the_status_is_read_once_per_workgroup(path):
    assert offenders(open(path).read())[0] == []


def test_every_kernel_that_sets_an_error_was_looked_at():
    seen = set()
    for p in glob.glob(os.path.join(os.path.dirname(build.__file__), "csrc", "*.hip")):
        seen |= offenders(open(p).read())[1]
    assert {"contract_kernel", "finalize_kernel", "simulate_walk_kernel", "fo_count_kernel"} <= seen
