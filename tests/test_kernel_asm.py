"""The GPU assembly of hand-written statements the compiler does not look
into, built from the sources here."""
import os
import re
import subprocess

import pytest

from paper_2501_16909_amd import build


@pytest.fixture(scope="module")
def decode_asm(tmp_path_factory):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = tmp_path_factory.mktemp("asm") / "k_decode.s"
    subprocess.check_call([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S",
                           os.path.join(build.CSRC, "k_decode.hip"), "-o", str(out)], stderr=subprocess.DEVNULL)
    return out.read_text()


def test_row_broadcasts_wait_for_their_operand(decode_asm):
    """Every multiply-add that takes one lane of a row stands in a statement
    that begins with the two wait states its operand needs, and in which no
    instruction writes such an operand."""
    blocks = re.findall(r"#ASMSTART\n(.*?)#ASMEND", decode_asm, flags=re.S)
    dpp = [b for b in blocks if "_dpp" in b]
    inside = sum(b.count("row_newbcast") for b in dpp)
    assert inside > 1000 and inside == decode_asm.count("row_newbcast")
    for b in dpp:
        lines = [l.split(";")[0].strip() for l in b.strip().splitlines()]
        lines = [l for l in lines if l]
        assert lines[0] == "s_nop 1", lines[0]
        ops = [re.fullmatch(r"v_fmac_f32_dpp (v\d+), (v\d+), (v\d+) row_newbcast:(\d+) row_mask:0xf bank_mask:0xf", l)
               for l in lines[1:]]
        assert all(ops) and len(ops) >= 8
        written = {m.group(1) for m in ops}
        assert not written & {m.group(2) for m in ops}
        assert not written & {m.group(3) for m in ops}
