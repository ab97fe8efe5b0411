"""Wait states between a matrix product and the first other instruction that touches its result, over every way through every kernel.  The hardware does
not wait for such a result (a reader that comes early gets the old value of some of its registers) and the compiler has to put other instructions or
s_nop between.  It counts them right in straight-line code, but not always across a branch: around a product behind a uniform branch it left 3 of 8, and every
fourth token of a tile had a stale sum.  Read from the assembly; CPU only."""
import re

import pytest

from tests import asm_util as A

# what the compiler leaves in straight-line code for gfx950: passes (of four cycles) of the instruction and four more; fp64 16
# passes and two (LDS and memory) or three (VALU)
_STATES = {"v_mfma_f32_16x16x32_bf16": 8, "v_mfma_i32_16x16x64_i8": 8, "v_mfma_f32_32x32x16_bf16": 12, "v_mfma_i32_32x32x32_i8": 12, "v_mfma_f64_16x16x4_f64": 18}


def _operands(text):
    return re.findall(r"[va]\[\d+:\d+\]|\b[va]\d+\b|(?<=, )-?[\d.]+", text.split(None, 1)[1])


def short_ways(p):
    """(product, reader, states) for every way from one to the other with too few of them."""
    named, found = [A.registers(t) for t in p.ins], []
    for i, text in enumerate(p.ins):
        op = text.split()[0]
        if not op.startswith(("v_mfma", "v_smfma")):
            continue
        need, result = _STATES[op], A.registers(_operands(text)[0])
        least, work = {}, [(j, 0) for j in p.after[i]]
        while work:
            j, n = work.pop()
            if n >= need or least.get(j, need) <= n:
                continue
            least[j] = n
            t = p.ins[j]
            if named[j] & result:
                # (the sum of a product that goes on is handed over inside the matrix core)
                goes_on = t.startswith(("v_mfma", "v_smfma")) and not (A.registers(_operands(t)[1]) | A.registers(_operands(t)[2])) & result
                if not goes_on:
                    found.append((text, t, n))
                continue
            n += int(t.split()[1], 0) + 1 if t.startswith("s_nop") else 1
            work += [(k, n) for k in p.after[j]]
    return found


def test_a_short_way_is_found():
    body = "\tv_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3]\n\ts_cbranch_vccnz .LBB0_2\n\ts_nop 7\n.LBB0_2:\n\ts_nop %d\n\tv_add_f32_e32 v5, v3, v5\n\ts_endpgm\n"
    assert len(short_ways(A.Program(body % 5))) == 1 and not short_ways(A.Program(body % 6))


@pytest.mark.parametrize("source", ["pact_gram.hip", "pact_centres.hip", "pact_euti.hip"])
def test_products_are_done_when_they_are_read(source):
    products = 0
    for name, body in A.kernels(source):
        if "v_mfma" in body:
            p = A.Program(body)
            products += 1
            assert not short_ways(p), name
    assert products
