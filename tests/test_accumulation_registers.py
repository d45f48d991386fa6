"""Host-only: in the kernels of the tuned bf16 loop the accumulation registers belong to the assembly that names them.

That loop keeps its accumulators in a0, a1, ... by number, which the compiler cannot see: if it ran out of vector registers
and put anything of its own there, a matrix instruction would overwrite it.  Nor may a vector instruction of the compiler's lie
between the two writes of the execution mask around masked requests.  This looks at the assembly of every kernel (no GPU needed).
"""
import re
import subprocess

from paper_2511_17599_amd import build as BLD


def test_nothing_else_uses_the_accumulation_registers(tmp_path):
    out = tmp_path / "flce.s"
    flags = [f for f in BLD.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([BLD.hipcc_path(), *flags, "-S", "--offload-device-only", BLD.SRC, "-o", str(out)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    kernel, in_asm, masked, seen, bad = None, False, False, set(), []
    for line in out.read_text().splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            kernel, masked = m.group(1), False
        if ";#ASMSTART" in line or ";#ASMEND" in line:
            in_asm = "START" in line
            continue
        code = line.split(";")[0].strip()
        if not code or code.startswith(".") or kernel is None:
            continue
        tuned = "FastLoop" in kernel or "SmallLoop" in kernel or "probe_half" in kernel or "probe_pair" in kernel
        if not tuned:
            continue
        if in_asm and "v_mfma_f32_16x16x32_bf16 a[" in code:
            seen.add(kernel)
        if in_asm and code.startswith("s_mov_b64 exec"):
            masked = code.split(",")[1].strip() != "-1"
        if not in_asm and (masked or re.search(r"\ba(\[|\d)", code)):
            bad.append((kernel, code))
    assert not bad, bad[:5]
    assert len(seen) >= 15      # forward, recompute, contractions on both tile edges
