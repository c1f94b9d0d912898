"""A kernel that keeps its products in accumulation registers by number, behind the compiler's back, must not share them
with the compiler: outside of inline assembly nothing may touch them, and nothing may be spilled.  Products that its
inline MFMAs write to vector registers are the compiler's, but it counts no wait states for them: until the next fence
nothing else may read or write them (all checked on the assembly; no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2508_18182_amd import build as B


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    made = {}

    def of(source):
        if source not in made:
            asm = tmp_path_factory.mktemp("asm") / "k.s"
            subprocess.run([hipcc, *B.HIPCC_FLAGS, "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC, "-S",
                            "--offload-device-only", os.path.join(B.CSRC, source), "-o", str(asm)], check=True,
                           capture_output=True)
            made[source] = asm.read_text()
        return made[source]
    return of


def _bodies(text, kernel):
    return re.findall(r"^(_Z\S*%s\S*):.*?\n(.*?)^\.Lfunc_end" % kernel, text, re.M | re.S)


def _vector_registers(operand):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", operand) or re.fullmatch(r"v(\d+)", operand)
    return range(int(m[1]), int(m[m.lastindex]) + 1) if m else ()


def _unfenced(body):
    """Instructions outside inline assembly that touch a register which an inline MFMA wrote on some path to them, with no
    fence (the two long waits in inline assembly) in between; and the number of such MFMAs."""
    inside, blocks, label = False, {"": []}, ""           # label -> [(inline, words)], in the order of the text
    for line in body.splitlines():
        if "#ASMSTART" in line or "#ASMEND" in line:
            inside = "#ASMSTART" in line
            continue
        code = line.split(";")[0].replace(",", " ").split()
        if code and code[0].endswith(":"):
            label = code[0][:-1]
            blocks[label] = []
        elif code and not code[0].startswith("."):
            blocks[label].append((inside, code))
            if code[0].startswith("s_cbranch"):           # what follows a branch is a block of its own
                label = label + "'"
                blocks[label] = []
    names = list(blocks)
    follows = {n: [c[1] for _, c in blocks[n] if c[0].startswith(("s_branch", "s_cbranch"))] for n in names}
    for n, following in zip(names, names[1:]):
        if not blocks[n] or blocks[n][-1][1][0] not in ("s_branch", "s_endpgm"):
            follows[n].append(following)
    entering, todo, found = {n: set() for n in names}, names[:], set()
    while todo:
        n = todo.pop()
        pending = set(entering[n])
        for inline, code in blocks[n]:
            if inline and code[0] == "s_nop" and code[1] == "15":
                pending.clear()
            elif inline and code[0].startswith("v_mfma"):
                pending.update(_vector_registers(code[1]))
            elif not inline and any(pending.intersection(_vector_registers(c)) for c in code[1:]):
                found.add(" ".join(code))
        for m in follows[n]:
            if not pending <= entering[m]:
                entering[m] |= pending
                todo.append(m)
    return sorted(found), sum(c[0].startswith("v_mfma") and bool(_vector_registers(c[1])) for b in blocks.values() for _, c in b)


@pytest.mark.parametrize("source,kernel,count", [("gram_kernels.hip", "gram_region_kernel", 2)])
def test_a_fence_stands_before_what_the_compiler_does_with_products(assembly, source, kernel, count):
    bodies = _bodies(assembly(source), kernel)
    assert len(bodies) == count
    for name, body in bodies:
        found, written = _unfenced(body)
        assert not found, f"{name}: {found[:5]}"
        assert written > 100
        # the check sees a copy that is put behind the last of them
        at = [m.end() for m in re.finditer(r"v_mfma\S+ v\[\d+:\d+\].*\n.*#ASMEND\n", body)][-1]
        last = re.findall(r"v_mfma\S+ v\[(\d+):", body[:at])[-1]
        assert _unfenced(body[:at] + f"\tv_mov_b32_e32 v255, v{last}\n" + body[at:])[0]


@pytest.mark.parametrize("source,kernel,count", [("gram_kernels.hip", "gram_region_kernel", 2)])
def test_only_the_assembly_touches_them(assembly, source, kernel, count):
    text = assembly(source)
    bodies = _bodies(text, kernel)
    assert len(bodies) == count
    for name, body in bodies:
        inside, used = False, 0
        for line in body.splitlines():
            if "#ASMSTART" in line or "#ASMEND" in line:
                inside = "#ASMSTART" in line
                continue
            code = line.split(";")[0]
            touches = re.search(r"^\s+[a-z].*[\s,]a(\d+\b|\[)", code)
            used += bool(touches and inside)
            assert inside or not touches, f"{name}: {line.strip()}"
            assert "scratch_" not in code, f"{name}: {line.strip()}"
        assert used > 500
        kd = re.search(r"\.amdhsa_kernel %s\n(.*?)\.end_amdhsa_kernel" % re.escape(name), text, re.S)[1]
        free, offset = (int(re.search(r"\.amdhsa_%s (\d+)" % f, kd)[1]) for f in ("next_free_vgpr", "accum_offset"))
        assert free - offset == 256          # all of them are the kernel's
