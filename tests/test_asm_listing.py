"""The kernels whose loops are inline assembly, as the compiler has set them: what it cannot see inside the statements it does not keep apart, so
the listing is looked at, along every path through it."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2509_25149_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FILES = ["gemm_f16.hip", "gemm_mx.hip"]
NO_RESULT = ("ds_write", "global_store", "scratch_store", "global_load_lds", "v_cmp", "v_readfirstlane", "v_readlane", "s_")   # no vector register is written


def registers(text):
    found = set()
    for kind, one, first, last in re.findall(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])", text):
        found.update(kind + str(i) for i in (range(int(one), int(one) + 1) if one else range(int(first), int(last) + 1)))
    return frozenset(found)


def kernels(listing):
    """{name: [(mnemonic, operands, vector registers written, read)]}; a label is ("label", name, ...)."""
    out, current = {}, None
    for line in listing.splitlines():
        line = line.split(";")[0].strip()
        if re.match(r"_Z\w+:$", line):
            current = out.setdefault(line[:-1], [])
        elif line.startswith(".Lfunc_end"):
            current = None
        elif current is None or not line:
            continue
        elif re.match(r"\.LBB\w+:$", line):
            current.append(("label", line[:-1], frozenset(), frozenset()))
        elif not line.startswith("."):
            op, _, operands = line.partition(" ") if " " in line else line.partition("\t")
            op, operands = op.strip(), operands.strip()
            first, _, rest = operands.partition(",")
            writes = frozenset() if op.startswith(NO_RESULT) else registers(first)
            reads = registers(rest if writes else operands)
            if "swap" in op:
                writes = reads = registers(operands)
            current.append((op, operands, writes, reads))
    return out


def paths(instructions, step, start):
    """step(state, instruction) -> the state behind it, hashable; every instruction is met in every state that some path reaches it in."""
    labels = {x[1]: i for i, x in enumerate(instructions) if x[0] == "label"}
    seen, todo = set(), [(0, start)]
    while todo:
        i, state = todo.pop()
        while True:
            x = instructions[i]
            if x[0] == "label":
                if (i, state) in seen:
                    break
                seen.add((i, state))
            else:
                state = step(state, x)
                if x[0] == "s_endpgm":
                    break
                if x[0] == "s_branch":
                    i = labels[x[1]]
                    continue
                if x[0].startswith("s_cbranch"):
                    todo.append((labels[x[1]], state))
            i += 1


def early_mfmas(instructions):
    """MFMAs that read a register which a vector instruction has written fewer than two instructions (or cycles of s_nop) before: through the
    builtins the compiler itself keeps the two that far apart."""
    bad = set()

    def step(recent, x):
        op, operands, writes, reads = x
        if op.startswith("v_mfma"):
            bad.update((op, operands) for _, written in recent if written & reads)
        passed = 1 + (int(operands) if op == "s_nop" else 0)
        recent = tuple((age + passed, written) for age, written in recent if age + passed < 2)
        return recent + ((0, writes),) if op.startswith("v_") and not op.startswith("v_mfma") and writes else recent

    paths(instructions, step, ())
    return bad


def touched_in_flight(instructions):
    """Instructions that read or write a register into which an LDS read may still be on its way.  Reads come back in order, so a wait for
    all but n operations leaves at most the n latest reads (others that are counted with them, scalar loads, can only make that fewer)."""
    bad = set()

    def step(pending, x):
        op, operands, writes, reads = x
        bad.update((op, operands) for into in pending if into & (writes | reads))
        if op.startswith("ds_read"):
            return pending + (writes,)
        waits = re.search(r"lgkmcnt\((\d+)\)", operands) if op == "s_waitcnt" else None
        return pending[max(0, len(pending) - int(waits.group(1))):] if waits else pending

    paths(instructions, step, ())
    return bad


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    folder = tmp_path_factory.mktemp("listings")

    def compile_one(name):
        out = str(folder / (name + ".s"))
        flags = [f for f in build.FLAGS if not f.startswith("-Rpass")]
        subprocess.run([HIPCC] + flags + ["-I", os.path.join(build.ROOT, "include"), "--cuda-device-only", "-S", os.path.join(build.CSRC, name), "-o", out],
                       check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
        with open(out) as fh:
            return kernels(fh.read())

    with ThreadPoolExecutor() as pool:
        return dict(zip(FILES, pool.map(compile_one, FILES)))


def made_up(*lines):
    return kernels("_Zk:\n" + "\n".join(lines) + "\ns_endpgm\n.Lfunc_end0:\n")["_Zk"]


def test_the_search_for_early_mfmas_finds_them():
    mfma = "v_mfma_scale_f32_16x16x128_f8f6f4 a[0:3], v[4:7], v[8:11], 0, v20, v21 op_sel:[0,0,0]"
    perm = "v_perm_b32 v20, v1, v2, v3"
    for between in ([], ["s_nop 0"], ["s_cmp_eq_u32 s0, 0"]):
        assert early_mfmas(made_up(perm, *between, mfma))
    for between in (["s_nop 1"], ["s_nop 0", "s_waitcnt lgkmcnt(0)"], ["v_mfma_f32_16x16x32_f16 v[40:43], v[4:7], v[8:11], 0", "s_nop 0"]):
        assert not early_mfmas(made_up(perm, *between, mfma))
    assert not early_mfmas(made_up("v_perm_b32 v22, v1, v2, v3", mfma))
    # around a loop's back edge
    assert early_mfmas(made_up(".LBB0_1:", mfma, "s_nop 3", perm, "s_cbranch_scc0 .LBB0_1"))


def test_the_search_for_reads_in_flight_finds_them():
    read, use = "ds_read_b128 v[4:7], v1 offset:16", "v_mfma_f32_16x16x32_f16 a[0:3], v[4:7], v[8:11], 0"
    assert touched_in_flight(made_up(read, use))
    assert touched_in_flight(made_up(read, "v_mov_b32_e32 v6, v0"))
    assert not touched_in_flight(made_up(read, "s_waitcnt lgkmcnt(0)", use))
    later = "ds_read_b128 v[12:15], v1"
    assert not touched_in_flight(made_up(read, later, "s_waitcnt vmcnt(3) lgkmcnt(1)", use))
    assert touched_in_flight(made_up(later, read, "s_waitcnt lgkmcnt(1)", use))
    assert touched_in_flight(made_up(read, "s_waitcnt vmcnt(0)", use))
    # a wait on one of two ways, and a use on the way back through a loop
    assert touched_in_flight(made_up(read, "s_cbranch_scc0 .LBB0_1", "s_waitcnt lgkmcnt(0)", ".LBB0_1:", use))
    assert touched_in_flight(made_up(".LBB0_1:", "v_mov_b32_e32 v20, v7", "s_waitcnt lgkmcnt(0)", read, "s_cbranch_scc0 .LBB0_1"))


@pytest.mark.parametrize("name", FILES)
def test_no_instruction_touches_a_register_that_an_lds_read_is_on_its_way_to(listings, name):
    """Fragment reads are in flight across the halves of a stage and the loop's back edge; the waits are not tied to the registers, so a copy or a
    spill that the compiler put there would take old values without a message."""
    checked = 0
    for kernel, instructions in listings[name].items():
        checked += sum(x[0].startswith("ds_read") for x in instructions)
        assert not touched_in_flight(instructions), kernel
    assert checked > 500


@pytest.mark.parametrize("name", FILES)
def test_no_mfma_reads_what_a_vector_instruction_has_just_written(listings, name):
    checked = 0
    for kernel, instructions in listings[name].items():
        checked += sum(x[0].startswith("v_mfma") for x in instructions)
        assert not early_mfmas(instructions), kernel
    assert checked > 1000
