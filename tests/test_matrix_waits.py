"""Wait states around matrix instructions in the built device code. The compiler places them for its own matrix instructions,
but knows nothing of those written as inline assembly (gemm_tile.h): there the source has to keep them. Read from the
disassembly of the library as it was built; needs no GPU."""
import glob
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"

# gfx950: a vector instruction's result is read by a matrix instruction two wait states later at the earliest; the result of
# v_mfma_f32_16x16x32_f16 (eight passes) is read or overwritten by a vector instruction eleven later.
WRITE_TO_MATRIX = 2
MATRIX_TO_VECTOR = 11


def _registers(operand):
    m = re.fullmatch(r"-?\|?([va])(?:(\d+)|\[(\d+):(\d+)\])\|?", operand.split()[0]) if operand else None
    if not m:
        return []
    lo, hi = (int(m[2]), int(m[2])) if m[2] else (int(m[3]), int(m[4]))
    return [(m[1], i) for i in range(lo, hi + 1)]


def violations(listing):
    """{kernel: [instruction, ...]} of a disassembly that stand closer to the write of one of their operands than they may, and the
    number of matrix instructions seen. Instructions are taken in the order of the listing, up to each jump that is always taken."""
    found, n_matrix, kernel = {}, 0, None
    written, multiplied, now = {}, {}, 0
    for line in listing.splitlines():
        head = re.match(r"^[0-9a-f]+ <(.*)>:$", line)
        if head:
            kernel, written, multiplied, now = head[1], {}, {}, 0
            continue
        ins = re.match(r"^\s+([a-z][a-z_0-9]*)\s*(.*?)\s*(?://.*)?$", line)
        if not ins or kernel is None:
            continue
        op, args = ins[1], re.split(r",\s*(?![^\[]*\])", ins[2])
        bad = False
        if op.startswith("v_mfma"):
            n_matrix += 1
            for r in (r for a in args[1:4] for r in _registers(a)):
                bad |= now - written.get(r, -99) < WRITE_TO_MATRIX
            for r in _registers(args[0]):
                multiplied[r] = now + 1
                written.pop(r, None)
        elif op.startswith("v_"):
            if "gemm_tile_kernel" in kernel:       # elsewhere the compiler sees to it, for matrix instructions of several lengths
                for r in (r for a in args for r in _registers(a)):
                    bad |= now - multiplied.get(r, -99) < MATRIX_TO_VECTOR
            for r in _registers(args[0]):
                written[r] = now + 1
                multiplied.pop(r, None)
        if bad:
            found.setdefault(kernel, []).append(line.strip())
        now += int(args[0], 0) + 1 if op == "s_nop" else 1
        if op in ("s_branch", "s_endpgm", "s_setpc_b64"):          # what follows in the listing does not follow in time
            written, multiplied = {}, {}
    return found, n_matrix


def test_the_reader_sees_a_write_that_is_too_close():
    text = "0000 <k>:\n\tv_cvt_pkrtz_f16_f32 v3, v8, v9 // 00\n\ts_nop %d // 04\n\tv_mfma_f32_16x16x32_f16 a[0:3], v[0:3], v[4:7], a[0:3] // 08\n"
    assert violations(text % 0)[0] and not violations(text % 1)[0]
    text = "0000 <gemm_tile_kernel>:\n\tv_mfma_f32_16x16x32_f16 a[0:3], v[0:3], v[4:7], a[0:3] // 00\n\ts_nop %d // 04\n\tv_accvgpr_read_b32 v1, a2 // 08\n"
    assert violations(text % 9)[0] and not violations(text % 10)[0]


def other_uses_of_m0(listing):
    """Instructions of the kernels that write m0 in inline assembly (for their loads into LDS) which read it, or write it in any other
    way: the compiler does not preserve m0 around those statements."""
    found, kernel = [], None
    for line in listing.splitlines():
        head = re.match(r"^[0-9a-f]+ <(.*)>:$", line)
        kernel = head[1] if head else kernel
        ins = line.split("//")[0].strip()
        if kernel and re.search(r"gemm_tile_kernel|verify_fused_kernel", kernel) and re.search(r"\bm0\b", ins) and not head:
            if not re.fullmatch(r"s_mov_b32 m0, (?!m0)\S+", ins):
                found.append((kernel, ins))
    return found


def test_the_reader_sees_other_uses_of_m0():
    text = "0000 <gemm_tile_kernel>:\n\ts_mov_b32 m0, s3 // 00\n\t%s // 04\n"
    assert not other_uses_of_m0(text % "s_nop 0") and other_uses_of_m0(text % "s_mov_b32 s4, m0") and other_uses_of_m0(text % "s_add_u32 m0, m0, s1")


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_waits_of_the_built_kernels(tmp_path):
    from paper_2408_05676_amd import build as b
    if not os.path.exists(b.LIB):
        b.build(verbose=False)
    shutil.copy(b.LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    objects = glob.glob(str(tmp_path / "*gfx950"))
    total, found = 0, {}
    for obj in objects:
        r = subprocess.run([OBJDUMP, "-d", "--demangle", obj], capture_output=True, text=True, check=True)
        bad, n = violations(r.stdout)
        total += n
        found.update(bad)
        assert not other_uses_of_m0(r.stdout)
    assert total > 5000, "no matrix instructions found"
    assert not found, {k: v[:2] for k, v in found.items()}
