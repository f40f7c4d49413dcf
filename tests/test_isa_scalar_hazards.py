"""Hand-written loads of the correlation kernels and the scalar registers they read: a memory instruction must not read one within five
wait states of the vector instruction that wrote it.  The compiler inserts the wait states for its own instructions and does not look into
opaque ones.  This scan follows every way through the code, branches and the back edges of loops included; the code of a loop's end is in
front of that of its beginning.  Host only (hipcc cross-compiles)."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

import test_isa_waits as waits

STATES = 5


def scalars(operands):
    out = set()
    for a, b, one in re.findall(r"s\[(\d+):(\d+)\]|\bs(\d+)\b", operands):
        out |= {int(one)} if one else set(range(int(a), int(b) + 1))
    return out


def functions(text):
    """(name, instructions, labels): an instruction is (line number, text, hand-written)."""
    name, code, labels, by_hand = None, [], {}, False
    for i, line in enumerate(text.split("\n")):
        t = line.strip()
        m = re.match(r"(_ZN2xc\w+):", t)
        if m:
            if name:
                yield name, code, labels
            name, code, labels = m.group(1), [], {}
        elif t.startswith(".Lfunc_end") and name:
            yield name, code, labels
            name = None
        elif t.startswith(";;#ASM"):
            by_hand = "START" in t
        elif re.match(r"\.L\w+:", t):
            labels[t.split(":")[0]] = len(code)
        elif name and t and t[0] not in ";.":
            code.append((i, t.split(";")[0].strip(), by_hand))
    if name:
        yield name, code, labels


def hazards(text):
    """(function, line number, load) of every hand-written load that a way through the code reaches too early."""
    found = []
    for name, code, labels in functions(text):
        loads = [n for n, (_, t, by_hand) in enumerate(code) if by_hand and t.startswith("buffer_load")]
        before = {n: [n - 1] for n in range(1, len(code)) if not code[n - 1][1].startswith(("s_branch", "s_endpgm", "s_setpc"))}
        for n, (_, t, _) in enumerate(code):
            m = re.match(r"s_c?branch\w* (\.L\w+)", t)
            if m:
                before.setdefault(labels[m.group(1)], []).append(n)
        for n in loads:
            used, seen = scalars(code[n][1].split(None, 1)[1]), {}
            todo, bad = [(p, 0) for p in before.get(n, [])], False
            while todo and not bad:
                k, distance = todo.pop()
                if distance >= STATES or seen.get(k, STATES) <= distance:
                    continue
                seen[k] = distance
                t = code[k][1]
                m = re.match(r"v_(?:readfirstlane_b32|readlane_b32|cmp\w*|\w+_co_\w+|div_scale\w*)\s+(.*)", t)
                if m and scalars(m.group(1).split(", v")[0]) & used:
                    bad = True
                nop = re.match(r"s_nop (\d+)", t)
                todo += [(p, distance + (1 + int(nop.group(1)) if nop else 1)) for p in before.get(k, [])]
            if bad:
                found.append((name, code[n][0], code[n][1]))
    return found


LOAD = "\t;;#ASMSTART\n\tbuffer_load_dwordx4 v[0:3], v4, s[16:19], 0 offen\n\t;;#ASMEND\n"


WRITE = "\tv_readlane_b32 s18, v3, 7\n"


@pytest.mark.parametrize("nop", [0, 1, 2, 3, 4])
def test_the_scan_follows_loops_and_branches(nop):
    between = "\ts_nop %d\n" % nop              # nop + 1 wait states; a branch is one
    straight = "_ZN2xc1kE:\n" + WRITE + between + LOAD + "\ts_endpgm\n"
    loop = "_ZN2xc1kE:\n.LBB0_1:\n" + between + LOAD + "\ts_nop 7\n" + WRITE + "\ts_cbranch_scc1 .LBB0_1\n\ts_endpgm\n"
    jump = "_ZN2xc1kE:\n" + WRITE + "\ts_branch .LBB0_2\n.LBB0_1:\n" + LOAD + "\ts_endpgm\n.LBB0_2:\n" + between + "\ts_cbranch_vccz .LBB0_1\n\ts_endpgm\n"
    assert [bool(hazards(t)) for t in (straight, loop, jump)] == [nop + 1 < STATES, nop + 2 < STATES, nop + 3 < STATES]
    assert not hazards("_ZN2xc1kE:\n" + WRITE + "\ts_endpgm\n" + LOAD)


@pytest.mark.skipif(not os.path.exists(waits.HIPCC), reason="hipcc not installed")
def test_hand_written_loads_read_settled_registers_on_every_way(tmp_path):
    def assembly(src):
        out = str(tmp_path / (src + ".s"))
        subprocess.run([waits.HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "--cuda-device-only", "-S", os.path.join(waits.CSRC, src), "-o", out], check=True, stderr=subprocess.DEVNULL)
        return open(out).read()

    sources = ["corr_split_kernels.hip", "corr_ws32_kernels.hip", "corr_ws_kernels.hip", "corr_row_kernels.hip"]
    with ThreadPoolExecutor(4) as ex:
        for src, text in zip(sources, ex.map(assembly, sources)):
            assert sum(1 for _, code, _ in functions(text) for _, t, by_hand in code if by_hand and t.startswith("buffer_load")) > 100
            assert not hazards(text), (src, hazards(text)[:5])
