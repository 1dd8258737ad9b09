"""The gradient products of attention_mfma.hip are written in inline asm, whose needs the compiler does not see.  In the code it
makes of them today (no GPU: read from this build's own assembly), along every path:

  * no vector instruction writes a product's first or second operand within 2 wait states before it, and
  * nothing but such products touches the accumulators within 19 wait states after it,

what the matrix instructions ask for (19 covers those of 16 passes; these have 8).  A register copy that another compiler
version, or a change of the kernels, puts in between shows here and not as a wrong gradient."""
import os
import re
import subprocess

import pytest

from paper_2006_16668_amd import build

BEFORE, AFTER = 2, 19


def _registers(operand):
    m = re.fullmatch(r"-?\|?([av])(?:(\d+)|\[(\d+):(\d+)\])\|?", operand.strip())
    if not m:
        return frozenset()
    first, last = (m.group(2), m.group(2)) if m.group(2) else (m.group(3), m.group(4))
    return frozenset((m.group(1), i) for i in range(int(first), int(last) + 1))


class Instruction:
    def __init__(self, text, in_asm):
        self.text = text
        self.name, _, rest = text.partition(" ")
        self.operands = [_registers(o) for o in re.split(r",\s*", rest)] if rest else []
        self.product = in_asm and self.name.startswith("v_mfma")
        self.next = []                                   # indices of the instructions that may follow
        target = re.fullmatch(r"s_c?branch\w*\s+(\S+)", text)
        self.target = target.group(1) if target else None

    @property
    def states(self):
        return int(self.text.split()[1], 0) + 1 if self.name == "s_nop" else 1

    @property
    def touched(self):
        return frozenset().union(*self.operands)

    @property
    def written(self):                                   # by a vector instruction that is no matrix product
        if not self.name.startswith("v_") or self.name.startswith("v_mfma") or not self.operands:
            return frozenset()
        return self.touched if "swap" in self.name else self.operands[0]


def _kernels(assembly):
    kernels, code, labels, in_asm = {}, None, {}, False
    for line in assembly.splitlines():
        in_asm = (in_asm or "#ASMSTART" in line) and "#ASMEND" not in line
        line = line.split(";")[0].rstrip()
        label = re.match(r"^([\w.$]+):", line)
        if label and label.group(1).startswith("_Z"):
            code, labels = [], {}
            kernels[label.group(1)] = (code, labels)
        elif label and code is not None:
            labels[label.group(1)] = len(code)
            if label.group(1).startswith(".Lfunc_end"):
                code = None
        elif code is not None and line.startswith("\t") and not line.startswith("\t."):
            code.append(Instruction(line.strip().replace("\t", " "), in_asm))
    for code, labels in kernels.values():
        for i, ins in enumerate(code):
            if ins.name not in ("s_branch", "s_endpgm", "s_setpc_b64") and i + 1 < len(code):
                ins.next.append(i + 1)
            if ins.target in labels and labels[ins.target] < len(code):
                ins.next.append(labels[ins.target])
    return {name: code for name, (code, _) in kernels.items()}


def _within(code, start, states):
    """Instructions that may be issued with fewer than `states` wait states between code[start] and them."""
    seen, todo = {}, [(n, 0) for n in code[start].next]
    while todo:
        i, passed = todo.pop()
        if passed >= states or seen.get(i, states) <= passed:
            continue
        seen[i] = passed
        todo += [(n, passed + code[i].states) for n in code[i].next]
    return seen


def check(assembly):
    """(products, what is too close to one) of every kernel"""
    found = {}
    for name, code in _kernels(assembly).items():
        products, wrong = 0, []
        for i, ins in enumerate(code):
            if ins.product:
                products += 1
                acc = ins.operands[0]
                assert acc == ins.operands[3] and len(acc) == 16
                for j in _within(code, i, AFTER):
                    other = code[j]
                    if other.product and other.operands[0] == acc and not acc & (other.operands[1] | other.operands[2]):
                        continue                         # the next product into the same accumulators
                    if acc & other.touched:
                        wrong.append((ins.text, other.text))
            elif ins.written:
                for j in _within(code, i, BEFORE):
                    if code[j].product and ins.written & (code[j].operands[1] | code[j].operands[2]):
                        wrong.append((ins.text, code[j].text))
        found[name] = (products, wrong)
    return found


SAMPLE = """_Zk:
	v_add_f32_e32 v{w}, v1, v2
{gap}	;;#ASMSTART
	v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]
	;;#ASMEND
.LBB0_1:
{tail}	v_accvgpr_read_b32 v0, a{r}
	s_cbranch_scc1 .LBB0_1
	s_endpgm
.Lfunc_end0:
"""


@pytest.mark.parametrize("w,gap,tail,r,faults", [
    (3, "", "\ts_nop 15\n\ts_nop 2\n", 3, 0), (5, "", "\ts_nop 15\n\ts_nop 2\n", 3, 1), (5, "\ts_nop 0\n", "\ts_nop 15\n\ts_nop 3\n", 3, 1),
    (11, "\ts_nop 1\n", "\ts_nop 15\n\ts_nop 2\n", 3, 0), (3, "", "\ts_nop 15\n\ts_nop 1\n", 3, 1), (3, "", "", 16, 0)])
def test_the_check_finds_what_it_looks_for(w, gap, tail, r, faults):
    (products, wrong), = check(SAMPLE.format(w=w, gap=gap, tail=tail, r=r)).values()
    assert products == 1 and len(wrong) == faults, wrong


def test_products_in_asm_have_their_wait_states(tmp_path):
    out = str(tmp_path / "attention.s")
    src = "attention_mfma.hip"
    subprocess.run([build._hipcc(), *build.FLAGS, *build.EXTRA_FLAGS[src], "-S", "--cuda-device-only", os.path.join(build.CSRC, src),
                    "-o", out], check=True, capture_output=True)
    found = check(open(out).read())
    with_products = {k: v for k, v in found.items() if v[0]}
    assert len(with_products) == 9                       # dq, and dk and dv in one form or two, of d 64 and 128, ragged or not
    for name, (products, wrong) in with_products.items():
        assert not wrong, (name, wrong[:5])
