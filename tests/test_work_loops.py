"""Persistent kernels take their items in a loop: thread 0 adds to a counter in
device memory, leaves the item in LDS, and after a barrier every thread reads
it.  The optimiser may thread a "thread 0 only" branch at the end of an
iteration into the one at the start of the next; the other threads' way round
then leads to the barrier without passing the start, which on a GPU is an inner
loop that runs before thread 0 gets there: all wait for an item that is never
taken.  So the compiled loops are checked: whoever reads an item again has
passed the branch that takes one."""
import os
import re
import subprocess

import pytest

from paper_2607_12074_amd import build as hip

SOURCES = ["m4_batch", "m4_c4", "m4_tri", "m4_edge", "m4_local"]


def kernels(text):
    for m in re.finditer(r"^define [^\n]*amdgpu_kernel[^\n]* @(\S+?)\([^\n]*\{$", text, re.M):
        body = text[m.end():]
        yield m.group(1), body[:body.index("\n}\n")]


def blocks_of(body):
    blocks, cur = {"entry": []}, "entry"
    for line in body.splitlines():
        label = re.match(r"^([\w.]+):", line)
        if label:
            cur = label.group(1)
            blocks[cur] = []
        else:
            blocks[cur].append(line)
    succ = {}
    for name, lines in blocks.items():
        at = max((i for i, x in enumerate(lines) if re.match(r"\s+(br|switch) ", x)), default=None)
        succ[name] = [] if at is None else re.findall(r"label %([\w.]+)", "\n".join(lines[at:]))
    return blocks, succ


def reachable(succ, start, without):
    seen, todo = set(), [b for b in start if b not in without]
    while todo:
        b = todo.pop()
        if b not in seen:
            seen.add(b)
            todo += [x for x in succ[b] if x not in without]
    return seen


def work_loops(body):
    """(branch that takes an item, block that reads it, read again without it)."""
    blocks, succ = blocks_of(body)
    for name, lines in blocks.items():
        taken = set()
        for line in lines:
            m = re.match(r"\s+(%[\w.]+) = (.*)", line)
            if m and (re.match(r"atomicrmw add ptr addrspace\(1\)", m.group(2)) or
                      any(re.search(re.escape(v) + r"\b", m.group(2)) for v in taken)):
                taken.add(m.group(1))
            m = re.match(r"\s+store \S+ (%[\w.]+), ptr addrspace\(3\) (.*?), align", line)
            if not m or m.group(1) not in taken:
                continue
            branch = {b for b in blocks if name in succ[b]}
            for reader, text in blocks.items():
                if any(" = load " in x and m.group(2) in x for x in text):
                    yield branch, reader, reader in reachable(succ, succ[reader], branch)


def found_in(source, out):
    subprocess.run([hip.HIPCC] + hip.FLAGS + ["--offload-device-only", "-S", "-emit-llvm", "-o", out,
                                              source], check=True, stderr=subprocess.DEVNULL)
    with open(out) as fh:
        return [(k, *loop) for k, body in kernels(fh.read()) for loop in work_loops(body)]


@pytest.mark.parametrize("name", SOURCES)
def test_every_reader_of_an_item_passes_the_taking(name, tmp_path):
    loops = found_in(os.path.join(hip.CSRC, name + ".hip"), str(tmp_path / "k.ll"))
    assert loops, "no work loop recognised"
    for kernel, _, reader, again in loops:
        assert not again, (kernel, reader)


# the loop shape that the check is for, without and with the barrier that keeps it whole
LOOP = """#include <hip/hip_runtime.h>
__global__ void k(unsigned* work, int n, int* status, const int* skip) {
  __shared__ int item;
  for (;;) {
    %s
    if (threadIdx.x == 0) item = (int)atomicAdd(work, 1u);
    __syncthreads();
    const int i = item;
    __syncthreads();
    if (i >= n) break;
    if (skip[i]) {
      if (threadIdx.x == 0) status[i] = 9;
      continue;
    }
    atomicAdd(&status[i], (int)threadIdx.x);
    __syncthreads();
  }
}
"""


@pytest.mark.parametrize("barrier,split", [("", True), ("__syncthreads();", False)])
def test_the_check_tells_them_apart(barrier, split, tmp_path):
    src = tmp_path / "k.hip"
    src.write_text(LOOP % barrier)
    loops = found_in(str(src), str(tmp_path / "k.ll"))
    assert [again for *_, again in loops] == [split]
