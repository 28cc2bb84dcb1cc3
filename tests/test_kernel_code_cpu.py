"""The machine code that was built here for the deep-ring contraction kernels, on the CPU.

Their MFMAs are written as inline assembly, so the compiler knows neither how long a result takes to arrive nor which
operands an MFMA reads early, and puts no wait states in.  The distances that it keeps by itself around the same
instruction written as a builtin (gfx950, v_mfma_f32_16x16x32_bf16) are checked here along every path of every such kernel.
"""
import os
import re
import struct
import subprocess

import pytest

import paper_2502_04416_amd

LIB = os.path.join(os.path.dirname(paper_2502_04416_amd.__file__), "libcmoe.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"

RESULT = 8     # wait states between an MFMA and the first other use of its result
SOURCE = 2     # wait states between a vector instruction and an MFMA that reads what it wrote

REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+))(?!\w)")


def code_objects(path):
    """The gfx950 code objects in the library's offload bundles."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", data, pos - 8)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, pos)
            if data[pos + 24:pos + 24 + n].endswith(b"gfx950"):
                yield data[at + off:at + off + size]
            pos += 24 + n
        at = data.find(MAGIC, at + 1)


def registers(operand):
    out = set()
    for bank, lo, hi, one in REG.findall(operand):
        out.update((bank, r) for r in range(int(lo or one), int(hi or one) + 1))
    return frozenset(out)


def parse(listing, wanted):
    """{kernel: [(address, mnemonic, operands, branch target or None)]} of a disassembly listing."""
    kernels, current, base = {}, None, {}
    for line in listing.splitlines():
        head = re.match(r"([0-9a-f]+) <(\S+)>:", line)
        if head:
            base[head.group(2)] = int(head.group(1), 16)
            current = kernels.setdefault(head.group(2), []) if wanted in head.group(2) else None
            continue
        code = re.match(r"\s+(\w+)\s*(.*?)\s*// ([0-9A-F]+):[^<]*(?:<(\S+?)\+0x([0-9a-f]+)>)?", line)
        if current is not None and code:
            name, ops, addr, sym, off = code.groups()
            to = base[sym] + int(off, 16) if sym and "branch" in name else None
            current.append((int(addr, 16), name, ops, to))
    return kernels


def violations(code):
    """Uses of an MFMA's result, and of a vector instruction's result by an MFMA, that come too early on some path.

    The state in front of an instruction: the register sets written lately, {(set, by an MFMA): wait states since}.
    """
    index = {ins[0]: i for i, ins in enumerate(code)}
    info = []
    for _, name, ops, _ in code:
        parts = [registers(p) for p in re.split(r",(?![^\[]*\])", ops)]
        info.append((name.startswith("v_mfma"), parts, frozenset().union(*parts)))
    before = {0: {}}
    todo, found = [0], {}
    while todo:
        i = todo.pop()
        state = before[i]
        _, name, ops, to = code[i]
        mfma, parts, used = info[i]
        for (regs, by_mfma), age in state.items():
            if by_mfma:
                # (an MFMA may add to the result of another at once, if it is the whole of it)
                late = used if not mfma else parts[1] | parts[2] | (frozenset() if parts[3] == regs else parts[0] | parts[3])
                if age < RESULT and late & regs:
                    found[i] = "%s %s: %d wait states after an MFMA" % (name, ops, age)
            elif mfma and age < SOURCE and (parts[1] | parts[2] | parts[3]) & regs:
                found[i] = "%s %s: %d wait states after a source was written" % (name, ops, age)
        steps = int(ops, 0) + 1 if name == "s_nop" else 1
        after = {k: age + steps for k, age in state.items() if age + steps < (RESULT if k[1] else SOURCE)}
        if mfma:
            after[(parts[0], True)] = 0
        elif name.startswith("v_") and parts[0]:
            after[(parts[0], False)] = 0
        follow = [] if name in ("s_branch", "s_endpgm") else [i + 1]
        if to is not None:
            follow.append(index[to])
        for j in follow:
            if j >= len(code):
                continue
            known = before.get(j)
            merged = dict(after) if known is None else {k: min(known.get(k, 99), after.get(k, 99)) for k in known.keys() | after.keys()}
            if merged != known:
                before[j] = merged
                todo.append(j)
    return [found[i] for i in sorted(found)]


@pytest.fixture(scope="module")
def ring_kernels(tmp_path_factory):
    if not os.path.exists(LIB):
        import __graft_entry__
        __graft_entry__.build()
    kernels = {}
    for i, obj in enumerate(code_objects(LIB)):
        if b"grouped_gemm_bf16_ring" not in obj:
            continue
        path = tmp_path_factory.mktemp("code") / ("%d.o" % i)
        path.write_bytes(obj)
        listing = subprocess.run([OBJDUMP, "-d", str(path)], capture_output=True, text=True, check=True).stdout
        kernels.update(parse(listing, "grouped_gemm_bf16_ring"))
    return kernels


def test_mfma_results_are_waited_for(ring_kernels):
    assert len(ring_kernels) >= 13
    bad = {}
    for name, code in ring_kernels.items():
        assert sum(ins[1] == "v_mfma_f32_16x16x32_bf16" for ins in code) >= 16, name
        if violations(code):
            bad[name] = violations(code)
    assert not bad, bad


def test_mfma_results_of_the_persistent_kernel_are_waited_for(tmp_path):
    """The same distances in the persistent down contraction, whose accumulators are read between the tiles of its loop; and no
    memory access of the compiler's own inside that loop, where it would count among the transfers waited for."""
    code = {}
    for i, obj in enumerate(code_objects(LIB)):
        if b"down_stream_kernel" in obj:
            path = tmp_path / ("%d.o" % i)
            path.write_bytes(obj)
            listing = subprocess.run([OBJDUMP, "-d", str(path)], capture_output=True, text=True, check=True).stdout
            code.update(parse(listing, "down_stream_kernel"))
    past_caches = []
    for code in code.values():                      # its two forms
        mfmas = [i for i, ins in enumerate(code) if ins[1] == "v_mfma_f32_16x16x32_bf16"]
        assert len(mfmas) == 4 * 32                 # two sets of fragment registers, each for a first and a later step
        assert not violations(code)
        assert not [ins for ins in code[mfmas[0]:mfmas[-1]] if ins[1].startswith(("scratch_", "global_", "flat_"))]
        nt = {"nt" in ins[2].split() for ins in code if ins[1].startswith("buffer_store")}
        assert len(nt) == 1
        past_caches += nt
    assert sorted(past_caches) == [False, True]


def test_the_check_sees_an_early_use():
    """Straight code, a loop and a join, with the use at the distance and one wait state closer."""
    mfma = "v_mfma_f32_16x16x32_bf16", "a[0:3], v[0:3], v[4:7], a[0:3]"

    def code(*ins):
        return [(4 * i, name, ops, to) for i, (name, ops, to) in enumerate(ins)]

    def n(k):
        return "s_nop", str(k), None

    read, end = ("v_accvgpr_read_b32", "v9, a2", None), ("s_endpgm", "", None)
    assert not violations(code(mfma + (None,), n(7), read, end))
    assert violations(code(mfma + (None,), n(6), read, end))
    assert not violations(code(mfma + (None,), mfma + (None,), n(7), read, end))
    # the short way round the wait
    assert violations(code(mfma + (None,), ("s_cbranch_scc0", "", 12), n(7), read, end))
    # the read at the head of a loop, after its back edge
    assert violations(code(read, n(7), mfma + (None,), ("s_cbranch_scc0", "", 0), end))
    assert violations(code(("v_mov_b32_e32", "v1, 0", None), n(0), mfma + (None,), n(7), end))
    assert not violations(code(("v_mov_b32_e32", "v1, 0", None), n(1), mfma + (None,), n(7), end))
