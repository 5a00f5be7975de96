"""LDS reads that the kernels write as inline assembly, in the code that the compiler makes of them: between such a read and the wait that
covers it no instruction may touch the registers it is filling.  The compiler takes them as written at once and is free to copy them; where it
does so in front of the wait, the copy holds whatever stood there before.  Needs the compiler, no GPU."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2408_04275_amd.build import CSRC, FLAGS, HIPCC

SOURCES = ["attn_mfma.hip", "gemm_mfma.hip", "gemm_mfma_nn.hip", "gemm_mfma_tn.hip"]


def _registers(text):
    out = set()
    for bank, first, last, one in re.findall(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        out |= {bank + str(i) for i in range(int(first or one), int(last or one) + 1)}
    return frozenset(out)


def functions(listing):
    """(name, [(text, line number, inside inline assembly)]) of every function, labels included."""
    name, body, inline = None, [], False
    for number, line in enumerate(listing.splitlines(), 1):
        if ";;#ASMSTART" in line or ";;#ASMEND" in line:
            inline = "START" in line
            continue
        text = line.split(";")[0].strip()
        if re.match(r"_Z\w+:", text):
            name, body = text[:-1], []
        elif name and text.startswith(".Lfunc_end"):
            yield name, body
            name = None
        elif name and (re.match(r"\.LBB\w+:", text) or (text and not text.startswith("."))):
            body.append((text, number, inline))


def early_uses(body):
    """{line: (instruction, line of the read)} along every path.  LDS operations complete in order and lgkmcnt counts those outstanding (scalar
    loads too, which only makes a wait stricter), so behind a wait for n at most the n youngest are still out."""
    label = {text[:-1]: i for i, (text, _, _) in enumerate(body) if text.endswith(":")}
    seen, paths, found = set(), [(0, ())], {}
    while paths:
        i, out = paths.pop()
        while i < len(body):
            text, number, inline = body[i]
            op, _, operands = text.partition(" ")
            i += 1
            if text.endswith(":"):
                if (i, out) in seen:
                    break
                seen.add((i, out))
            elif op == "s_endpgm":
                break
            elif op == "s_branch":
                i = label[operands]
            elif op.startswith("s_cbranch"):
                paths.append((label[operands], out))
            elif op == "s_waitcnt":
                n = re.search(r"lgkmcnt\((\d+)\)", text)
                if n:
                    out = out[max(len(out) - int(n[1]), 0):]
                    while out and not out[0][0]:               # (the compiler waits for its own reads)
                        out = out[1:]
            else:
                touched = _registers(operands)
                for filling, read in out:
                    if filling & touched:
                        found[number] = (text, read)
                if op.startswith("ds_"):
                    filling = _registers(operands.split(",")[0]) if inline and op.startswith("ds_read") else frozenset()
                    if filling or out:
                        out = (out + ((filling, number),))[-16:]
    return found


LISTING = """_Zkernel:
	;;#ASMSTART
	ds_read_b128 v[4:7], v0 offset:16
	;;#ASMEND
	;;#ASMSTART
	ds_read_b128 v[8:11], v0 offset:32
	;;#ASMEND
	s_cbranch_vccz .LBB0_2
	{copy}
	s_waitcnt lgkmcnt(1)
	v_add_f32_e32 v1, v4, v5
.LBB0_2:
	s_waitcnt lgkmcnt(0)
	v_add_f32_e32 v1, v4, v8
	s_endpgm
.Lfunc_end0:
"""


def test_the_scan_sees_a_copy_in_front_of_the_wait():
    scan = lambda copy: [early_uses(body) for _, body in functions(LISTING.format(copy=copy))]  # noqa: E731
    assert scan("v_mov_b32_e32 v3, v12") == [{}]
    assert scan("v_mov_b64_e32 v[12:13], v[6:7]") == [{9: ("v_mov_b64_e32 v[12:13], v[6:7]", 3)}]
    assert scan("s_waitcnt lgkmcnt(1)\n\tv_mov_b32_e32 v3, v8") == [{10: ("v_mov_b32_e32 v3, v8", 6)}]


@pytest.fixture(scope="module")
def listings():
    def compile_one(source):
        r = subprocess.run([HIPCC, *FLAGS, "-S", "--cuda-device-only", os.path.join(CSRC, source), "-o", "-"], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        return r.stdout
    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        return dict(zip(SOURCES, ex.map(compile_one, SOURCES)))


@pytest.mark.parametrize("source", SOURCES)
def test_no_register_is_touched_while_a_read_fills_it(listings, source):
    reads = 0
    for name, body in functions(listings[source]):
        reads += sum(inline and text.startswith("ds_read") for text, _, inline in body)
        assert early_uses(body) == {}, name
    assert reads > 0
