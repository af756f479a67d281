"""What the compiler is told about LDS that others than the reading lane have written: read off the intermediate code, compiled for the
GPU here (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2403_19708_amd import build

CSRC = os.path.join(build.HERE, "csrc")
KERNELS = """
#include "ca_device.h"
using namespace ca;
__global__ void kernel(AttnArgs a, bf16x8 *q, const f32x16 *o) {
    __shared__ __attribute__((aligned(16))) uint8_t stage[QueryRows<%(D)d, %(style)d>::kQueryBytes];
#if %(outputs)d
    f32x16 O[%(D)d / 32];
    for (int i = 0; i < %(D)d / 32; ++i) O[i] = o[threadIdx.x * 4 + i];
    store_rows<%(D)d>(a, 0, 0, 3, 0, 31, stage, O, 0.5f);
#else
    QueryRows<%(D)d, %(style)d> rows;
    bf16x8 Q[%(D)d / 16];
    rows.fetch(a, 0, 0, 3, 0, 0, 31);
    rows.finish(stage, 0.5f, Q);
    for (int i = 0; i < %(D)d / 16; ++i) q[threadIdx.x * 8 + i] = Q[i];
#endif
}
"""


def intermediate(source):
    cmd = [build.hipcc()] + [f for f in build.FLAGS if f != "-shared" and not f.startswith("-Wl,")]
    done = subprocess.run(cmd + ["-I" + CSRC, "--cuda-device-only", "-S", "-emit-llvm", str(source), "-o", "-"], capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
    return done.stdout


@pytest.mark.parametrize("D, style, outputs", [(128, 0, 0), (128, 1, 0), (64, 0, 0), (64, 1, 0), (128, 0, 1), (64, 0, 1)])
def test_rows_handed_on_through_lds_are_read_behind_the_writes(tmp_path, D, style, outputs):
    """Lanes read what other lanes wrote: without a barrier or fences in between the compiler may move the reads to the front, whatever
    the hardware's order is."""
    source = tmp_path / "kernel.hip"
    source.write_text(KERNELS % dict(D=D, style=style, outputs=outputs))
    body = re.search(r"define [^\n]*amdgpu_kernel void @[^\n]*kernel.*?\n}", intermediate(source), re.S).group(0)
    kinds = [("store", r"store .*ptr addrspace\(3\)"), ("load", r"load .*ptr addrspace\(3\)"), ("release", r'fence syncscope\("wavefront"\) release'),
             ("barrier", r"call void @llvm.amdgcn.wave.barrier"), ("acquire", r'fence syncscope\("wavefront"\) acquire')]
    seen = [kind for line in body.splitlines() for kind, text in kinds if re.search(text, line)]
    stores, loads = seen.count("store"), seen.count("load")
    assert stores >= 4 and loads >= 4
    assert seen == ["store"] * stores + ["release", "barrier", "acquire"] + ["load"] * loads


def test_the_few_rows_kernel_reads_behind_its_waits():
    """A wavefront loads pages into a ring of its own and waits for them without a barrier: the wait itself keeps no read behind it."""
    kernels = re.findall(r"define [^\n]*amdgpu_kernel void @[^\n]*attn_rows_kernel.*?\n}", intermediate(os.path.join(CSRC, "ca_attn_rows.hip")), re.S)
    assert len(kernels) == 24
    for body in kernels:
        waits, told = 0, True
        for line in body.splitlines():
            if "call void @llvm.amdgcn.s.waitcnt(" in line:
                waits, told = waits + 1, False
            elif re.search(r"\bfence |call void asm sideeffect .*~\{memory\}", line):
                told = True
            elif re.search(r"(\bload |ds\.read\.tr).*ptr addrspace\(3\)", line):
                assert told, line
        assert waits >= 3


def test_shares_are_merged_with_their_loads_in_one_block():
    """Four shares of a row tile are in flight: their loads stand side by side and not behind a branch each, where they would wait for one another."""
    kernels = re.findall(r"define [^\n]*amdgpu_kernel void @[^\n]*combine_tiles_kernel.*?\n}", intermediate(os.path.join(CSRC, "ca_attn_dma.hip")), re.S)
    assert len(kernels) == 2
    for body in kernels:
        loads = [len(re.findall(r"= load float, ptr addrspace\(1\)", block)) for block in re.split(r"\n\d+:", body)]
        loads = [n for n in loads if n]
        assert sorted(loads) == [2 * 4] * 4 + [4 * 4] * 4           # maxima and denominators, then four sums each, of four times four shares
