"""Host-only: wait states that the compiler keeps between its own instructions and does not see the need for at inline assembly.

A vector instruction's scalar result (v_readfirstlane, a comparison, a restored spill) may be read by a memory instruction five
wait states later; before that the request may run with the old descriptor, its range check among it."""
import device_asm as A


def too_early(kernel):
    """Requests of inline assembly that read a scalar register within five wait states of a vector instruction's write."""
    insts, _ = kernel
    for i, x in enumerate(insts):
        if x.in_asm and x.op.startswith("buffer_"):
            reads = set().union(*(A.registers(a.split()[0], "s") for a in x.args))
            yield from ((w.text, x.text) for w in A.before(kernel, i, 5) if A.written_by_vector(w, "s") & reads)


def test_requests_wait_for_scalars_of_vector_instructions():
    requests = sum(x.in_asm and x.op.startswith("buffer_") for insts, _ in A.kernels().values() for x in insts)
    assert requests > 1000
    bad = {n: b for n, k in A.kernels().items() if (b := list(too_early(k)))}
    assert not bad, {n: b[:2] for n, b in bad.items()}


def _kernel(*lines):
    text = "\n".join(["_Zk:", *lines, "\ts_endpgm", ".Lfunc_end0:"])
    return A.parse(text)["_Zk"]


LOAD = ["\t;#ASMSTART", "\ts_mov_b32 m0, s4", "\ts_nop 0", "\tbuffer_load_dwordx4 v1, s[28:31], 0 offen lds", "\t;#ASMEND"]


def test_the_look_itself():
    assert list(too_early(_kernel("\tv_readfirstlane_b32 s30, v3", *LOAD)))
    assert list(too_early(_kernel("\tv_readfirstlane_b32 s30, v3", "\ts_nop 1", *LOAD)))
    assert not list(too_early(_kernel("\tv_readfirstlane_b32 s30, v3", "\ts_nop 2", *LOAD)))
    assert not list(too_early(_kernel("\tv_readfirstlane_b32 s27, v3", *LOAD)))
    assert not list(too_early(_kernel("\tv_add_f32_e32 v30, v3, v4", *LOAD)))
    # around a loop: the write lies behind the request, one jump away
    assert list(too_early(_kernel(".LBB0_1:", *LOAD, "\tv_readlane_b32 s28, v3, 4", "\ts_cbranch_scc1 .LBB0_1")))
