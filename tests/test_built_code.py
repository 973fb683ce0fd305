"""Rules of the gfx950 instruction set that the compiler keeps for the instructions it knows and that instructions
written by hand have to keep by themselves, checked on the listing of the built kernels."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2504_15364_amd import binding as kd

TOOLS = "/opt/rocm/lib/llvm/bin"
CSRC = os.path.join(os.path.dirname(kd.LIB_PATH), "csrc")
# wait states between a product on the matrix pipe and another instruction that reads its result (one that
# overwrites it: one fewer)
MATRIX_WAIT = {"v_mfma_f32_32x32x16_bf16": 12, "v_mfma_f32_16x16x32_bf16": 8}
REG = re.compile(r"\b([vsa])(?:(\d+)|\[(\d+):(\d+)\])")


def registers(text):
    """The registers an operand list names, as a set of (file, number)."""
    out = set()
    for f, one, lo, hi in REG.findall(text):
        out.update((f, i) for i in range(int(one or lo), int(one or hi) + 1))
    return out


class Code:
    """One object's instructions in address order: name, operands, and the indices that may run next."""

    def __init__(self, lines):
        self.name, self.args, self.func, addr, targets = [], [], [], [], []
        where, func, base = {}, None, {}
        for l in lines:
            head = re.match(r"([0-9a-f]+) <(\S+)>:", l)
            if head:
                func = head.group(2)
                base[func] = int(head.group(1), 16)
            m = re.match(r"\s+([a-z]\w*)\s*(.*?)\s*//\s*([0-9A-F]+):.*?(?:<(\S+?)(?:\+0x([0-9a-f]+))?>)?$", l)
            if not m:
                continue
            where[int(m.group(3), 16)] = len(self.name)
            self.name.append(m.group(1))
            self.args.append(m.group(2))
            self.func.append(func)
            addr.append(int(m.group(3), 16))
            targets.append((m.group(4), int(m.group(5) or "0", 16)) if m.group(4) else None)
        self.next = []
        for i, n in enumerate(self.name):
            after = [i + 1] if i + 1 < len(self.name) and n not in ("s_endpgm", "s_branch", "s_setpc_b64") else []
            if n.startswith(("s_cbranch", "s_branch")):
                sym, off = targets[i]
                after.append(where[base[sym] + off])
            self.next.append(after)

    def after(self, i, stop):
        """Walk every path from behind instruction i; stop(j, states) is called with the wait states passed before j and
        ends the path by returning True."""
        todo, seen = [(j, 0) for j in self.next[i]], {}
        while todo:
            j, states = todo.pop()
            if seen.get(j, 1 << 30) <= states or stop(j, states):
                continue
            seen[j] = states
            passed = states + (int(self.args[j], 0) + 1 if self.name[j] == "s_nop" else 1)
            todo += [(k, passed) for k in self.next[j]]


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    out = {}
    for src in ("attention", "few", "evict"):
        obj = os.path.join(CSRC, src + ".o")
        if not (os.path.exists(obj) and os.path.exists(f"{TOOLS}/llvm-objdump")):
            pytest.skip("needs the built objects and the LLVM binary tools")
        work = tmp_path_factory.mktemp(src)
        shutil.copy(obj, work / "x.o")
        subprocess.run([f"{TOOLS}/llvm-objdump", "--offloading", "x.o"], check=True, capture_output=True, cwd=work)
        device = [p for p in work.iterdir() if "gfx950" in p.name]
        assert len(device) == 1, src
        text = subprocess.run([f"{TOOLS}/llvm-objdump", "-d", "--no-show-raw-insn", str(device[0])], check=True,
                              capture_output=True, text=True).stdout
        out[src] = Code(text.splitlines())
        assert len(out[src].name) > 1000
    return out


def test_matrix_results_are_not_touched_before_they_are_ready(listings):
    # the hardware does not hold back a reader of an unfinished product; the compiler spaces out the readers it
    # knows, and a register operand of inline assembly is not one of them
    found, products = set(), 0
    for src, code in listings.items():
        for i, n in enumerate(code.name):
            if not n.startswith("v_mfma"):
                continue
            products += 1
            need, dst = MATRIX_WAIT[n], registers(code.args[i].split(",")[0])

            def stop(j, states):
                if states >= need:
                    return True
                m = code.name[j]
                first, _, rest = code.args[j].partition(",")
                read = registers(rest if m.startswith("v_") else code.args[j])
                if not m.startswith("v_mfma") and (dst & read or (states < need - 1 and dst & registers(first))):
                    found.add((code.func[i], f"{n} {code.args[i]}", f"{m} {code.args[j]}", states))
                    return True
                return False
            code.after(i, stop)
    assert products > 1000
    assert not found, "\n".join(map(str, sorted(found)[:20]))


def test_copies_into_lds_wait_for_their_address(listings):
    # m0 holds the LDS address of a copy: one wait state between the instruction that writes it and the copy
    found, writes = set(), 0
    for src, code in listings.items():
        for i, n in enumerate(code.name):
            if not (n.startswith("s_") and re.match(r"m0\b", code.args[i])):
                continue
            writes += 1

            def stop(j, states):
                if states == 0 and "_load_lds_" in code.name[j]:
                    found.add((code.func[i], f"{n} {code.args[i]}", f"{code.name[j]} {code.args[j]}"))
                return True
            code.after(i, stop)
    assert writes > 100
    assert not found, f"{len(found)}: " + "\n".join(map(str, sorted(found)[:5]))


def test_scalar_loads_written_by_hand_wait_in_their_block():
    # to the compiler the destination of such a load holds the data at once: it may copy or reuse the register while the
    # load is on its way, unless the wait is part of the same block of assembly
    blocks = 0
    for name in sorted(os.listdir(CSRC)):
        if name.endswith((".hip", ".h")):
            for asm in re.findall(r"\basm\b(?:\s*volatile)?\s*\((.*?)\);", open(os.path.join(CSRC, name)).read(), re.S):
                if "s_load" in asm:
                    blocks += 1
                    assert "s_waitcnt" in asm, (name, asm)
    assert blocks > 0


def test_loads_are_waited_for(listings):
    # ... and where the wait is apart, because copies are to be requested in between, nothing may read or overwrite the
    # destination of a load on any path from it to a wait for its kind
    found, loads = set(), 0
    for src, code in listings.items():
        for i, n in enumerate(code.name):
            vector = n.startswith("global_load_dword")
            if not (vector or n.startswith("s_load_dword")):
                continue
            loads += 1
            dst, counter = registers(code.args[i].split(",")[0]), "vmcnt" if vector else "lgkmcnt"

            def stop(j, states):
                if code.name[j] == "s_waitcnt" and counter in code.args[j]:
                    return True
                first, _, rest = code.args[j].partition(",")
                in_order = vector and code.name[j].startswith("global_load_dword")   # loads land in the order of issue
                if dst & (registers(rest) if in_order else registers(code.args[j])):
                    found.add((code.func[i], f"{n} {code.args[i]}", f"{code.name[j]} {code.args[j]}"))
                    return True
                return False
            code.after(i, stop)
    assert loads > 500
    assert not found, f"{len(found)}: " + "\n".join(map(str, sorted(found)[:20]))
