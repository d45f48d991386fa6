"""Host-only: in the kernels of the tuned bf16 loop the accumulation registers belong to the assembly that names them.

That loop keeps its accumulators in a0, a1, ... by number, which the compiler cannot see: if it ran out of vector registers
and put anything of its own there, a matrix instruction would overwrite it.  Nor may a vector instruction of the compiler's lie
between the two writes of the execution mask around masked requests, nor a write of M0 of the compiler's between the assembly that
sets it and the requests that take their LDS destination from it.  This looks at every kernel that names the registers."""
import collections
import re

import device_asm as A


def numbered(kernel):
    return any(x.in_asm and x.op == "v_mfma_f32_16x16x32_bf16" and x.args[0].startswith("a[") for x in kernel[0])


# Every kernel of the library and of its probe that has the loop, by loop and hidden-size form (contractions: whole K steps only)
LOOP_KERNELS = {"fwd_tiles_kernel": (2, 2), "recompute_kernel": (2, 2), "contract_kernel": (2, 0), "contract_pair_kernel": (1, 0)}
PROBES = {"probe_kernel": 6, "probe_half_kernel": 2, "probe_pair_kernel": 5, "probe_mfma16_kernel": 1}


def test_all_kernels_of_the_loop_are_looked_at():
    found = collections.Counter()
    for name, kernel in A.kernels().items():
        if numbered(kernel):
            m = re.search(r"(fwd_tiles|recompute|contract_pair|contract|probe_half|probe_pair|probe_mfma16|probe)_kernel", name)
            loop = re.search(r"(Fast|Small)LoopILb([01])E", name)
            found[(m.group(0),) + (loop.groups() if loop else ())] += 1
    want = collections.Counter({(k,): n for k, n in PROBES.items()})
    for k, forms in LOOP_KERNELS.items():
        for loop in ("Fast", "Small"):
            for ragged in (0, 1):
                if forms[ragged]:
                    want[(k, loop, str(ragged))] = forms[ragged]
    assert found == want


def misuse(kernel):
    """Instructions of the compiler's that name an accumulation register, or that a mask meant for requests would meet."""
    masked = False
    for x in kernel[0]:
        if x.in_asm and x.op == "s_mov_b64" and x.args[0] == "exec":
            masked = x.args[1] != "-1"
        if not x.in_asm and (masked or re.search(r"\ba(\[|\d)", x.text)):
            yield x.text


def stray_m0(kernel):
    """Requests whose M0 was last written by the compiler, on any path, or in the wait state before them."""
    insts, pred = kernel
    for i, x in enumerate(insts):
        if not (x.in_asm and x.op.startswith("buffer_load") and x.args[-1].endswith("lds")):
            continue
        seen, todo = set(), [(p, 0) for p in pred[i]]
        while todo:
            j, passed = todo.pop()
            if j in seen:
                continue
            seen.add(j)
            y = insts[j]
            if y.args and y.args[0] == "m0" and y.op.startswith("s_"):
                if not y.in_asm or passed < 1:
                    yield y.text, x.text
                continue
            todo += [(p, passed + A.wait_states(y)) for p in pred[j]]


def test_nothing_else_uses_the_accumulation_registers():
    kernels = {n: k for n, k in A.kernels().items() if numbered(k)}
    bad = {n: b for n, k in kernels.items() if (b := list(misuse(k)))}
    assert not bad, {n: b[:3] for n, b in bad.items()}


def test_requests_take_the_lds_destination_that_the_assembly_set():
    requests = 0
    for n, k in A.kernels().items():
        requests += sum(x.in_asm and x.op.startswith("buffer_load") for x in k[0])
        bad = list(stray_m0(k))
        assert not bad, (n, bad[:3])
    assert requests > 1000


def _kernel(*lines):
    return A.parse("\n".join(["_Zk:", *lines, "\ts_endpgm", ".Lfunc_end0:"]))["_Zk"]


def test_the_look_itself():
    def asm(*lines):
        return ["\t;#ASMSTART", *lines, "\t;#ASMEND"]
    load = asm("\tbuffer_load_dwordx4 v1, s[28:31], 0 offen lds")
    mfma = asm("\tv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], 0")
    assert numbered(_kernel(*mfma)) and not numbered(_kernel("\tv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], 0"))
    assert list(misuse(_kernel(*mfma, "\tv_accvgpr_write_b32 a7, v3")))
    assert list(misuse(_kernel(*asm("\ts_mov_b64 exec, s[2:3]"), "\tv_add_f32_e32 v1, v2, v3", *asm("\ts_mov_b64 exec, -1"))))
    assert not list(misuse(_kernel(*asm("\ts_mov_b64 exec, s[2:3]", "\ts_mov_b64 exec, -1"), "\tv_add_f32_e32 v1, v2, v3")))
    m0 = asm("\ts_add_i32 m0, s1, s2")
    assert not list(stray_m0(_kernel(*m0, *mfma, *load)))
    assert list(stray_m0(_kernel(*m0, *load)))
    assert list(stray_m0(_kernel(*m0, "\ts_mov_b32 m0, -1", *mfma, *load)))
    assert list(stray_m0(_kernel(".LBB0_1:", *mfma, *load, "\ts_mov_b32 m0, s9", "\ts_cbranch_scc1 .LBB0_1")))
