"""What the kernels' assembly strings leave to the source and the compiler does not look after, checked in the assembly that
it makes: the wait state between M0 and the LDS-DMA load that reads it, the age of a broadcast's operand, and the waits of
the fp64 tile kernels, which request a slot of LDS by LDS-DMA behind the barrier that ends its reading and count the memory
operations behind a request."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2602_04163_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
KERNELS = ("syrk_trailing128_kernel", "syrk_trailing64_kernel", "tri_inverse_level128_kernel", "tri_inverse_level64_kernel",
           "pair_link_kernel", "hosted_kernel", "panel_pair_kernel")
pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")


SWEEPS = sorted(s for s in build.SOURCES if s.startswith("group_sweep"))


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    """source -> [(function, its instructions and labels)], all compiled at once"""
    folder = tmp_path_factory.mktemp("asm")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]

    def compiled(source):
        out = folder / (source + ".s")
        subprocess.run([HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(out)],
                       check=True, capture_output=True)
        return [(m.group(1), [op for op in (line.split(";")[0].strip() for line in m.group(2).split("\n")) if op])
                for m in re.finditer(r"^(_ZN4bpdq\w+):[^\n]*\n(.*?)^\.Lfunc_end", out.read_text(), re.S | re.M)]

    sources = SWEEPS + ["prepare.hip", "hessian.hip"]
    with ThreadPoolExecutor(min(len(sources), os.cpu_count() or 4)) as pool:
        return dict(zip(sources, pool.map(compiled, sources))).__getitem__


def plain(ops):
    return [op for op in ops if not op.startswith(".") and not op.endswith(":")]


def paths(ops):
    """The instructions that may follow each one, and those that may precede it."""
    label = {op.rstrip(":"): i for i, op in enumerate(ops) if op.startswith(".LBB")}
    after, before = [], [[] for _ in ops]
    for i, op in enumerate(ops):
        to = [label[op.split()[-1]]] if op.startswith(("s_cbranch", "s_branch")) else []
        if not op.startswith(("s_branch", "s_endpgm")) and i + 1 < len(ops):
            to.append(i + 1)
        after.append(to)
        for j in to:
            before[j].append(i)
    return after, before


def reached(start, edges):
    seen, todo = set(), list(start)
    while todo:
        for j in edges[todo.pop()]:
            if j not in seen:
                seen.add(j)
                todo.append(j)
    return seen


@pytest.mark.parametrize("source", ["prepare.hip", "hessian.hip", "group_sweep_k1.hip"])
def test_m0_is_a_wait_state_old_when_an_lds_dma_load_reads_it(source, assembly):
    """The hardware needs one instruction between a scalar write of M0 and an LDS-DMA load, which takes its LDS address
    from there; inside one assembly string the compiler adds none."""
    loads = 0
    for name, ops in assembly(source):
        ops = plain(ops)
        for before, op in zip(ops, ops[1:]):
            if "load_lds" in op:
                loads += 1
                assert not re.match(r"s_\w+ m0\b", before), f"{name}: {before} directly before {op}"
    assert loads >= 6


def test_a_broadcast_operand_is_two_instructions_old(assembly):
    """The multiply-add that broadcasts a lane's value reads registers that no vector instruction has written in the two
    wait states before it, copies that the compiler puts in included."""
    seen = 0
    for name, ops in assembly("prepare.hip"):
        ops = plain(ops)
        for i, op in enumerate(ops):
            m = re.match(r"v_fmac_f64_dpp v\[\d+:\d+\], v\[(\d+):(\d+)\]", op)
            if not m:
                continue
            seen += 1
            young, states = [], 0
            for p in reversed(ops[:i]):
                if states >= 2:
                    break
                states += 1 + (int(p.split()[1], 0) if p.startswith("s_nop") else 0)
                w = re.match(r"v_\w+ v(?:(\d+)\b|\[(\d+):(\d+)\])", p)
                if w:
                    young += [int(w[1])] if w[1] else range(int(w[2]), int(w[3]) + 1)
            assert not {int(m[1]), int(m[2])} & set(young), f"{name}: {ops[i - 2:i + 1]}"
    assert seen >= 100


@pytest.mark.parametrize("source", SWEEPS)
def test_the_sweeps_strings_read_registers_that_are_old_enough(source, assembly):
    """A broadcast operand two wait states after the vector instruction that wrote it, and what a matrix product wrote eleven
    after it: the compiler counts neither where an assembly string reads.  (Copies between the register files count too.)"""
    strings = r"v_(fmac_f32_dpp|sub_f32_dpp|mul_f32_dpp|add_f32|mul_f32|fmac_f32|alignbit_b32)$"
    broadcasts = matrix = 0
    for name, ops in assembly(source):
        if "group_kernel" not in name or "commit" in name:
            continue
        ops = plain(ops)
        for i, op in enumerate(ops):
            word = op.split()[0]
            matrix += word.startswith("v_mfma")
            if not re.match(strings, word):
                continue
            regs = [int(r) for r in re.findall(r"\bv(\d+)\b", op)]
            broadcast = regs[1] if word.endswith("_dpp") else None
            broadcasts += broadcast is not None
            states = 0
            for p in reversed(ops[max(0, i - 12):i]):
                if states >= 11:
                    break
                w = re.match(r"v_\w+ v(?:(\d+)\b|\[(\d+):(\d+)\])", p)
                wrote = () if not w else {int(w[1])} if w[1] else set(range(int(w[2]), int(w[3]) + 1))
                assert not (states < 2 and broadcast in wrote), f"{name}: {p} .. {op}"
                assert not (p.startswith("v_mfma") and wrote & set(regs)), f"{name}: {p} .. {op}"
                states += 1 + (int(p.split()[1], 0) if p.startswith("s_nop") else 0)
    # (the fixed grid takes two broadcasts per column and matrix products for the pending columns only)
    least = (510, 96) if source.endswith("u.hip") else (1900, 800)
    assert broadcasts >= least[0] and matrix >= least[1]


def test_no_lds_read_is_in_flight_at_a_barrier(assembly):
    """Where a request may still follow, no LDS read may be in flight at a barrier.  The compiler knows nothing of the DMA and
    moves products, and with them the waits for their operands, over a barrier."""
    seen, barriers = set(), 0
    for function, ops in assembly("prepare.hip"):
        name = next((k for k in KERNELS if k in function), None)
        if name is None:
            continue
        seen.add(name)
        after, before = paths(ops)
        ahead = reached([i for i, op in enumerate(ops) if "load_lds" in op], before)
        barriers += sum(ops[i].startswith("s_barrier") for i in ahead)
        # from behind every LDS read along every path: its wait must come before a barrier does
        todo, done = [j for i in ahead if ops[i].startswith("ds_read") for j in after[i]], set()
        while todo:
            i = todo.pop()
            if i in done or i not in ahead:
                continue
            done.add(i)
            if ops[i].startswith("s_waitcnt") and "lgkmcnt(0)" in ops[i]:
                continue
            assert not ops[i].startswith("s_barrier"), f"{function}: an LDS read is in flight at a barrier"
            todo += after[i]
    assert seen == set(KERNELS) and barriers >= 9


@pytest.mark.parametrize("kernel", ["hosted_kernel", "panel_pair_kernel"])
def test_a_hosted_tile_has_the_operations_that_its_waits_count(kernel, assembly):
    """From one tile to the next there are 16 stores and 16 loads of old values: the waits for 36 and 20 let that many be
    outstanding beside the four requests of a slice.  Fewer would let a slice be read before it has landed.  (The stores
    come in three forms; the compiler may have forms share their last.)"""
    (ops,) = [ops for function, ops in assembly("prepare.hip") if kernel in function]
    after, before = paths(ops)
    waits = [i for i, op in enumerate(ops) if op.startswith("s_waitcnt vmcnt(36)")]
    assert len(waits) == 2                                      # slices 0 and 1 of a tile
    loop = reached(waits, after) & reached(waits, before)
    assert {ops[i] for i in loop if re.match(r"s_waitcnt vmcnt\((4|20|36)\) ", ops[i])} == \
        {f"s_waitcnt vmcnt({n}) lgkmcnt(0)" for n in (4, 20, 36)}
    count = lambda kind: sum(ops[i].split()[0] == kind for i in loop)
    assert count("global_load_lds_dwordx4") == 8 * 4
    assert count("global_load_dwordx2") == 16
    assert 3 * 15 + 1 <= count("global_store_dwordx2") <= 3 * 16
    assert not any(re.match(r"scratch|buffer|flat|global_(?!load_lds_dwordx4|load_dwordx2|store_dwordx2)", ops[i]) for i in loop)
