"""The build's look at its own device assembly: no 64-bit shift takes its count
from the last vector register of a kernel's allocation."""

import os
import re
import subprocess

import pytest

from paper_1208_0277_amd import build

KERNEL = """
\t.globl\tk_one
k_one:                                  ; @k_one
; %bb.0:
\tv_mov_b32_e32 v1, 0
\t{op} v[2:3], v{count}, v[4:5]
\ts_endpgm
\t.section\t.rodata
\t.amdhsa_kernel k_one
\t\t.amdhsa_next_free_vgpr {free}
\t\t.amdhsa_accum_offset {accum}
\t.end_amdhsa_kernel
\t.text
.Lfunc_end0:
"""


def _asm(op, count, free, accum=None):
    return KERNEL.format(op=op, count=count, free=free, accum=accum or (free + 3) // 4 * 4)


@pytest.mark.parametrize("op", ["v_lshlrev_b64", "v_lshrrev_b64", "v_ashrrev_i64", "v_lshlrev_b64_e64"])
@pytest.mark.parametrize("count,free,accum,bad", [(63, 64, None, True), (63, 63 + 1, 64, True), (63, 65, None, False), (62, 64, None, False),
                                                  (31, 32, None, True), (31, 64, None, False), (55, 100, 56, True), (61, 62, None, False)])
def test_a_count_in_the_last_register_is_found(op, count, free, accum, bad):
    found = build.last_register_shifts(_asm(op, count, free, accum))
    assert [name for name, _ in found] == (["k_one"] if bad else [])


def test_other_shifts_pass():
    for op in ("v_lshlrev_b32_e32 v63, v63, v1 ;", "v_lshl_add_u64", "v_add_u64"):
        assert not build.last_register_shifts(_asm(op, 63, 64))


def test_the_compilers_assembly_is_read(tmp_path):
    """A real file's kernels, sizes and shifts are seen, and a planted one found."""
    src = os.path.join(build.HERE, "csrc", "k_prep.hip")
    out = tmp_path / "k.s"
    flags = build.FLAGS + ["-I", os.path.join(build.ROOT, "include"), "-I", os.path.join(build.HERE, "csrc")]
    subprocess.run([build.HIPCC] + flags + ["--offload-device-only", "-S", src, "-o", str(out)], check=True)
    asm = out.read_text()
    size = build.registers(asm)
    assert len(size) >= 6 and all(n % 8 == 0 and 8 <= n <= 512 for n in size.values())
    assert asm.count(".amdhsa_kernel ") == len(size)
    assert not build.last_register_shifts(asm)
    for name, body in build._FUNCTION.findall(asm):
        if name not in size:
            continue
        shift = re.search(r"v_lshlrev_b64 (v\[\d+:\d+\]), v\d+,", body)
        if shift:
            planted = body.replace(shift.group(0), f"v_lshlrev_b64 {shift.group(1)}, v{size[name] - 1},", 1)
            assert [n for n, _ in build.last_register_shifts(asm.replace(body, planted, 1))] == [name]
            return
    pytest.fail("no kernel of the file shifts 64 bits")
