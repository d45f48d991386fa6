"""Host-only: wait states that the compiler keeps between its own instructions and does not see the need for at inline assembly.

A vector instruction's scalar result (v_readfirstlane, a comparison, a restored spill) may be read by a memory instruction five
wait states later; before that the request may run with the old descriptor, its range check among it.  A vector instruction's
result may be an operand of a matrix instruction two wait states later (what this compiler puts between the two itself), and a matrix
instruction of 16 x 16 x 32 writes its sums within eleven."""
import device_asm as A


def too_early(kernel):
    """Requests of inline assembly that read a scalar register within five wait states of a vector instruction's write."""
    insts, _ = kernel
    for i, x in enumerate(insts):
        if x.in_asm and x.op.startswith("buffer_"):
            reads = set().union(*(A.registers(a.split()[0], "s") for a in x.args))
            yield from ((w.text, x.text) for w in A.before(kernel, i, 5) if A.written_by_vector(w, "s") & reads)


def early_operands(kernel):
    """Matrix instructions of inline assembly with an operand that a vector instruction wrote fewer than two wait states before."""
    insts, _ = kernel
    for i, x in enumerate(insts):
        if x.in_asm and x.op.startswith("v_mfma"):
            reads = set().union(*(A.registers(a, "v") for a in x.args[1:3]))
            yield from ((w.text, x.text) for w in A.before(kernel, i, 2)
                        if not w.op.startswith("v_mfma") and A.written_by_vector(w, "v") & reads)


def early_sums(kernel):
    """Plain reads of accumulation registers within eleven wait states of the matrix instruction that writes them."""
    insts, _ = kernel
    for i, x in enumerate(insts):
        if x.in_asm and x.op == "v_accvgpr_read_b32":
            reads = A.registers(x.args[1], "a")
            yield from ((w.text, x.text) for w in A.before(kernel, i, 11)
                        if w.op.startswith("v_mfma") and A.registers(w.args[0], "a") & reads)


def test_matrix_operands_and_sums_are_waited_for():
    for n, k in A.kernels().items():
        bad = list(early_operands(k)) + list(early_sums(k))
        assert not bad, (n, bad[:2])


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


def test_the_look_at_matrix_instructions_itself():
    mfma = ["\t;#ASMSTART", "\tv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], 0", "\t;#ASMEND"]
    read = ["\t;#ASMSTART", "\tv_accvgpr_read_b32 v9, a[2]", "\t;#ASMEND"]
    assert list(early_operands(_kernel("\tv_mov_b32_e32 v5, v8", *mfma)))
    assert list(early_operands(_kernel("\tv_mov_b32_e32 v5, v8", "\ts_nop 0", *mfma)))
    assert not list(early_operands(_kernel("\tv_mov_b32_e32 v5, v8", "\ts_nop 1", *mfma)))
    assert list(early_sums(_kernel(*mfma, "\ts_nop 9", *read)))
    assert not list(early_sums(_kernel(*mfma, "\ts_nop 15", *read)))
