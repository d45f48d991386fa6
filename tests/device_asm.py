"""The assembly of the library's kernels, for host-only tests: the compiler's view ends at inline assembly, so what it would
otherwise guarantee (wait states between dependent instructions, registers that nothing else uses) is looked at here."""
import functools
import re
import subprocess
import tempfile
from typing import NamedTuple

from paper_2511_17599_amd import build as BLD


class Inst(NamedTuple):
    op: str
    args: tuple         # operands as written, modifiers on the last one
    in_asm: bool        # from inline assembly
    block: int          # which inline assembly block of the kernel, -1 outside
    text: str


@functools.lru_cache(None)
def compiled():
    """(assembly of the device code, the compiler's remarks on what each kernel uses); one compile per process."""
    with tempfile.TemporaryDirectory() as tmp:
        out = f"{tmp}/flce.s"
        flags = [f for f in BLD.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
        res = subprocess.run([BLD.hipcc_path(), *flags, "-Rpass-analysis=kernel-resource-usage", "-S", "--offload-device-only",
                              BLD.SRC, "-o", out], capture_output=True, text=True)
        assert res.returncode == 0, res.stderr[-2000:]
        with open(out) as f:
            return f.read(), res.stderr


@functools.lru_cache(None)
def kernels():
    """{kernel name: (instructions, predecessors of each one)}"""
    return parse(compiled()[0])


def parse(text):
    found, name, insts, labels, in_asm, block = {}, None, None, None, False, -1
    for line in text.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            name, insts, labels, block = m.group(1), [], {}, -1
            found[name] = (insts, labels)
            continue
        if name is None:
            continue
        if ";#ASMSTART" in line or ";#ASMEND" in line:
            in_asm = "START" in line
            block += in_asm
            continue
        m = re.match(r"^([.\w$]+):", line)
        if m:
            labels[m.group(1)] = len(insts)
            if m.group(1).startswith(".Lfunc_end"):
                name = None
            continue
        code = re.split(r";|//", line)[0].strip()
        if not code or code.startswith("."):
            continue
        op, _, rest = code.partition(" ")
        insts.append(Inst(op, tuple(a.strip() for a in rest.split(",")) if rest.strip() else (), in_asm, block if in_asm else -1, code))
    return {n: (i, _predecessors(i, l)) for n, (i, l) in found.items() if any(x.op == "s_endpgm" for x in i)}


def _predecessors(insts, labels):
    pred = [[] for _ in insts]
    for i, x in enumerate(insts):
        if x.op not in ("s_branch", "s_endpgm") and i + 1 < len(insts):
            pred[i + 1].append(i)
        if x.op.startswith(("s_branch", "s_cbranch")) and labels.get(x.args[0], len(insts)) < len(insts):
            pred[labels[x.args[0]]].append(i)
    return pred


def registers(arg, kind):
    """The numbers of the registers of a kind ('s', 'v', 'a') that an operand names."""
    m = re.match(rf"^[-|]*{kind}(?:(\d+)|\[(\d+)(?::(\d+))?\])(?=\W|$)", arg)
    if not m:
        return set()
    first = int(m.group(1) or m.group(2))
    return set(range(first, int(m.group(3) or first) + 1))


def wait_states(x):
    return int(x.args[0], 0) + 1 if x.op == "s_nop" else 1


def before(kernel, i, states):
    """Every instruction fewer than `states` wait states ahead of instruction i, over all paths that lead there."""
    insts, pred = kernel
    best, todo = {}, [(p, 0) for p in pred[i]]
    while todo:
        j, passed = todo.pop()
        if passed >= states or best.get(j, states) <= passed:
            continue
        best[j] = passed
        todo += [(p, passed + wait_states(insts[j])) for p in pred[j]]
    return [insts[j] for j in sorted(best)]


def written_by_vector(x, kind):
    """Registers of a kind that a vector instruction writes."""
    if not x.op.startswith("v_") or not x.args:
        return set()
    two = "_co_" in x.op or x.op.startswith(("v_div_scale", "v_mad_u64", "v_mad_i64", "v_swap"))
    return set().union(*(registers(a, kind) for a in x.args[:2 if two else 1]))
