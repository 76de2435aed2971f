"""The fp64 tile kernels request a slot of LDS by LDS-DMA behind the barrier that ends its reading, so no LDS read may still
be in flight at a barrier.  The compiler knows nothing of the DMA and moves products, and with them the waits for their
operands, over a barrier: checked in the assembly that it makes of the source."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_04163_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
KERNELS = ("syrk_trailing128_kernel", "syrk_trailing64_kernel", "tri_inverse_level128_kernel", "tri_inverse_level64_kernel",
           "pair_link_kernel", "hosted_kernel")


def kernels(source, tmp_path):
    """(name, instructions and labels) of every kernel in the assembly that the compiler makes of a source."""
    out = tmp_path / (source + ".s")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(out)],
                   check=True, capture_output=True)
    for m in re.finditer(r"^(_ZN4bpdq\w+):[^\n]*\n(.*?)^\.Lfunc_end", out.read_text(), re.S | re.M):
        yield m.group(1), [op for op in (line.split(";")[0].strip() for line in m.group(2).split("\n")) if op]


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")
@pytest.mark.parametrize("source", ["prepare.hip", "hessian.hip", "group_sweep_k1.hip"])
def test_m0_is_a_wait_state_old_when_an_lds_dma_load_reads_it(source, tmp_path):
    """The hardware needs one instruction between a scalar write of M0 and an LDS-DMA load, which takes its LDS address
    from there; inside one assembly string the compiler adds none."""
    loads = 0
    for name, ops in kernels(source, tmp_path):
        ops = [op for op in ops if not op.startswith(".") and not op.endswith(":")]
        for before, op in zip(ops, ops[1:]):
            if "load_lds" in op:
                loads += 1
                assert not re.match(r"s_\w+ m0\b", before), f"{name}: {before} directly before {op}"
    assert loads >= 6


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")
def test_no_lds_read_is_in_flight_at_a_barrier(tmp_path):
    seen, barriers = set(), 0
    for function, ops in kernels("prepare.hip", tmp_path):
        name = next((k for k in KERNELS if k in function), None)
        if name is None:
            continue
        seen.add(name)
        label = {op.rstrip(":"): i for i, op in enumerate(ops) if op.startswith(".LBB")}
        barriers += sum(op.startswith("s_barrier") for op in ops)
        # from behind every LDS read along every path: its wait must come before a barrier does
        todo, done = [i + 1 for i, op in enumerate(ops) if op.startswith("ds_read")], set()
        while todo:
            i = todo.pop()
            if i in done or i >= len(ops):
                continue
            done.add(i)
            op = ops[i]
            if op.startswith("s_waitcnt") and "lgkmcnt(0)" in op:
                continue
            assert not op.startswith("s_barrier"), f"{function}: an LDS read is in flight at a barrier"
            if op.startswith(("s_cbranch", "s_branch")):
                todo.append(label[op.split()[-1]])
            if not op.startswith(("s_branch", "s_endpgm")):
                todo.append(i + 1)
    assert seen == set(KERNELS) and barriers >= 9
