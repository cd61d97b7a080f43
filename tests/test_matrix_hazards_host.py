"""No instruction of the built kernels touches the result of a matrix instruction that is still running.

The vector registers that a matrix instruction writes may be read or written by another instruction only so many wait states later, and the
hardware does not wait by itself.  The compiler keeps the distance along straight code, but not everywhere: it does not see into inline assembly, and
where a branch goes round some code it counts that code on the path that skips it too.  So every path of the code that runs is walked here."""
import re
import shutil
import struct
import subprocess

import pytest

from paper_2505_22179_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
# wait states between a matrix instruction and another use of its result, passes + 4
# (16x16x32 fp16: four passes, 32x32x16 fp16: eight)
NEEDED = {"v_mfma_f32_16x16x32_f16": 8, "v_mfma_f32_32x32x16_f16": 12}
REGISTER = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")
LINE = re.compile(r"^\s+(\S+)\s*(.*?)\s*//\s*([0-9A-F]+):(?:.*<(.+?)(?:\+0x([0-9a-f]+))?>)?")
LABEL = re.compile(r"^([0-9a-f]+) <(.+)>:$")


def code_objects(library):
    """the gfx950 code objects of a library: every HIP source brings a bundle"""
    blob, magic = open(library, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__"
    for at in (m.start() for m in re.finditer(re.escape(magic), blob)):
        count, = struct.unpack_from("<Q", blob, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(count if count < 16 else 0):
            offset, size, length = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + length]
            pos += 24 + length
            if name.endswith(b"gfx950") and size:
                yield blob[at + offset:at + offset + size]


def registers(text):
    out = set()
    for kind, one, first, last in REGISTER.findall(text):
        out.update((kind, i) for i in range(int(one or first), int(one or last) + 1))
    return out


class Code:
    """instructions of a listing: name, operands, indices of the ones that may follow"""

    def __init__(self, listing):
        self.name, self.operands, self.kernel, self.follow = [], [], [], []
        at, start, jumps, kernel = {}, {}, [], ""
        for line in listing:
            if (m := LABEL.match(line)):
                start[m[2]] = int(m[1], 16)
                kernel = m[2]
            elif (m := LINE.match(line)):
                at[int(m[3], 16)] = i = len(self.name)
                self.name.append(m[1])
                self.operands.append(m[2])
                self.kernel.append(kernel)
                if m[1].startswith(("s_cbranch", "s_branch")):
                    assert m[4], line
                    jumps.append((i, m[4], int(m[5] or "0", 16)))
        ends = ("s_endpgm", "s_branch", "s_setpc_b64")
        self.follow = [[] if n in ends else [i + 1] for i, n in enumerate(self.name)]
        for i, label, beyond in jumps:
            self.follow[i].append(at[start[label] + beyond])

    def touches(self, i):
        """vector registers that instruction i reads, or writes as soon as it issues"""
        name, operands = self.name[i], self.operands[i]
        if name.startswith("v_mfma"):   # chains through the third operand wait in hardware
            _, a, b, _ = re.split(r",\s*(?![^\[]*\])", operands)[:4]
            return registers(a + " " + b)
        if name.startswith("v_"):
            return registers(operands)
        if name.startswith(("ds_", "global_", "buffer_", "flat_", "scratch_")):
            loads = "read" in name or "load" in name and not operands.endswith("lds")
            return registers(operands.split(",", 1)[1] if loads and "," in operands else operands)   # a load writes much later
        return ()

    def too_early(self):
        """(matrix instruction, instruction, wait states between them) of each violation"""
        touched = {}
        for i, name in enumerate(self.name):
            if not name.startswith("v_mfma"):
                continue
            result = registers(self.operands[i].split(",")[0])
            need, best, work = NEEDED[name], {}, [(j, 0) for j in self.follow[i]]
            while work:
                j, states = work.pop()
                if states >= need or best.get(j, need) <= states:
                    continue
                best[j] = states
                if j not in touched:
                    touched[j] = self.touches(j)
                if not result.isdisjoint(touched[j]):
                    yield i, j, states
                    continue
                states += int(self.operands[j]) + 1 if self.name[j] == "s_nop" else 1
                work += [(k, states) for k in self.follow[j]]


def violations(listing):
    code = Code(listing)
    return [f"{code.kernel[j]}: {code.name[i]} {code.operands[i]} -> {code.name[j]} {code.operands[j]} after {s} wait states"
            for i, j, s in code.too_early()], code


def test_the_walk_finds_what_a_branch_goes_round():
    listing = """
0000000000000000 <k>:
	v_mfma_f32_16x16x32_f16 v[0:3], v[8:11], v[12:15], v[0:3]  // 000000000000: 00
	s_cbranch_vccnz 8                                          // 000000000008: 00 <k+0x18>
	s_nop 7                                                    // 00000000000C: 00
	v_fmac_f32_e32 v20, v21, v1                                // 000000000010: 00
	s_nop 0                                                    // 000000000014: 00
	s_waitcnt vmcnt(4)                                         // 000000000018: 00
	v_lshrrev_b32_e32 v3, 8, v30                               // 00000000001C: 00
	s_endpgm                                                   // 000000000020: 00
""".splitlines()
    found, _ = violations(listing)
    assert len(found) == 1 and "v_lshrrev_b32_e32 v3, 8, v30 after 2 wait states" in found[0]
    assert not violations([ln.replace("s_waitcnt vmcnt(4)", "s_nop 7           ") for ln in listing])[0]


@pytest.fixture(scope="module")
def found(tmp_path_factory):
    if not shutil.which(OBJDUMP):
        pytest.skip("no llvm-objdump")
    path, out, matrix, order = tmp_path_factory.mktemp("code") / "object", [], {}, {}
    for obj in code_objects(build.build(force=False)):
        path.write_bytes(obj)
        bad, code = violations(subprocess.run([OBJDUMP, "-d", str(path)], capture_output=True, text=True, check=True).stdout.splitlines())
        out += bad
        for name, operands, kernel in zip(code.name, code.operands, code.kernel):
            if name.startswith("v_mfma"):
                matrix[kernel] = matrix.get(kernel, 0) + 1
            if "tree_attn_merge" in kernel and (name.startswith("global_load") or "vmcnt" in operands):
                order.setdefault(kernel, []).append("load" if "load" in name else "wait")
    return out, matrix, order


@pytest.mark.parametrize("kernels", ["gemm_", "tree_attn_", "lm_head_"])
def test_no_result_of_a_matrix_instruction_is_touched_too_early(found, kernels):
    bad, matrix, _ = found
    assert sum(n for kernel, n in matrix.items() if kernels in kernel) > 100   # the listing was understood
    bad = [b for b in bad if kernels in b.split(":")[0]]
    assert not bad, f"{len(bad)}:\n" + "\n".join(bad[:40])


@pytest.mark.parametrize("ranges", [4, 8])
def test_the_merge_asks_for_all_partial_results_before_it_waits(found, ranges):
    """two loads per key range; one memory round trip, not one per range"""
    order, = (o for kernel, o in found[2].items() if f"tree_attn_merge_kernelILi{ranges}E" in kernel)
    assert order[:2 * ranges] == ["load"] * (2 * ranges) and "load" not in order[2 * ranges:]
