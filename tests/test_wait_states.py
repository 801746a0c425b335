"""Direct loads to LDS are written in inline assembly, which the compiler's hazard pass does not look
into.  On gfx9 the hardware does not wait for their scalar operands either: M0 has to be written one wait
state before a load to LDS reads it, and any scalar register that a vector instruction writes five before
a vector memory instruction does.  Both are checked here over every path through the built kernels."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2209_02478_amd as mi

LLVM = "/opt/rocm/llvm/bin"
M0_STATES, SGPR_STATES = 1, 5
VECTOR_MEMORY = ("buffer_", "global_", "scratch_", "flat_")


def registers(operand):
    """Scalar registers an operand names."""
    m = re.fullmatch(r"s(\d+)", operand)
    if m:
        return {int(m.group(1))}
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    return {"vcc"} if operand.startswith("vcc") else {operand} if operand in ("m0", "exec") else set()


class Instruction:
    def __init__(self, address, text, target):
        self.address, self.text, self.target = address, text, target
        self.name, _, rest = text.partition(" ")
        self.operands = [o.strip() for part in rest.split(",") for o in [part.strip().split(" ")[0]] if o]
        self.states = int(self.operands[0], 0) + 1 if self.name == "s_nop" else 1
        self.to_lds = self.name.startswith(VECTOR_MEMORY) and (" lds" in " " + rest or "_lds_" in self.name)

    def scalar_reads(self):
        return set().union(*[registers(o) for o in self.operands]) if self.name.startswith(VECTOR_MEMORY) else set()

    def vector_writes(self):
        """Scalar registers that a vector instruction writes."""
        if not self.name.startswith("v_"):
            return set()
        two = any(part in self.name for part in ("_co_", "div_scale", "mad_u64_u32", "mad_i64_i32"))    # a carry too
        return set().union(*[registers(o) for o in self.operands[:2 if two else 1]])


def parse(disassembly):
    """Functions of a disassembly, each a list of instructions."""
    functions, current, start = {}, None, 0
    for line in disassembly.splitlines():
        m = re.match(r"^([0-9a-f]+) <(.+)>:$", line)
        if m:
            start, current = int(m.group(1), 16), functions.setdefault(m.group(2), [])
            continue
        m = re.match(r"^\s+(\S.*?)\s*// ([0-9A-F]+):(.*)$", line)
        if m and current is not None:
            target = None
            if m.group(1).startswith(("s_branch", "s_cbranch")):
                t = re.search(r"<.+?(?:\+0x([0-9a-f]+))?>\s*$", m.group(3))
                target = start + int(t.group(1) or "0", 16)
            current.append(Instruction(int(m.group(2), 16), m.group(1), target))
    return functions


def faults(code):
    """What is written too close to its reader on some path: register, wait states between, reader, writer."""
    at = {i.address: n for n, i in enumerate(code)}
    before = [[n - 1] if n and not code[n - 1].name.startswith(("s_branch", "s_endpgm", "s_setpc")) else [] for n in range(len(code))]
    for n, i in enumerate(code):
        if i.target is not None and i.target in at:
            before[at[i.target]].append(n)
    found = []
    for n, reader in enumerate(code):
        reads = reader.scalar_reads()
        if not reads and not reader.to_lds:
            continue
        stack, seen = [(p, 0) for p in before[n]], {}
        while stack:
            p, states = stack.pop()
            if states >= SGPR_STATES or seen.get(p, SGPR_STATES) <= states:
                continue
            seen[p] = states
            writer = code[p]
            if reads & writer.vector_writes():
                found.append(("sgpr", states, reader.text, writer.text))
            if reader.to_lds and states < M0_STATES and writer.name.startswith("s_") and writer.operands[:1] == ["m0"]:
                found.append(("m0", states, reader.text, writer.text))
            stack += [(q, states + writer.states) for q in before[p]]
    return found


def kernels(library, folder):
    """Functions of every gfx950 code object in a library."""
    fat = os.path.join(folder, "fat.bin")
    subprocess.check_call([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", library, os.devnull])
    with open(fat, "rb") as f:
        data = f.read()
    for n, bundle in enumerate(re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data)):
        at = bundle.end() + 8
        for _ in range(struct.unpack_from("<Q", data, bundle.end())[0]):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + length].decode()
            at += 24 + length
            if not triple.endswith("gfx950") or not size:
                continue
            path = os.path.join(folder, f"{n}.co")
            with open(path, "wb") as f:
                f.write(data[bundle.start() + offset:bundle.start() + offset + size])
            yield from parse(subprocess.check_output([f"{LLVM}/llvm-objdump", "-d", "--mcpu=gfx950", path], text=True)).items()


def sample(*lines):
    return [Instruction(4 * n, text, target) for n, (text, target) in enumerate((l, None) if isinstance(l, str) else l for l in lines)]


def test_checker():
    load = "buffer_load_dwordx4 v1, s[8:11], 0 offen lds"
    assert faults(sample("s_mov_b32 m0, s1", load))
    assert not faults(sample("s_mov_b32 m0, s1", "s_nop 0", load))
    assert faults(sample("v_readfirstlane_b32 s10, v2", "s_mov_b32 m0, s1", "s_nop 2", load))
    assert not faults(sample("v_readfirstlane_b32 s10, v2", "s_mov_b32 m0, s1", "s_nop 3", load))
    assert not faults(sample("v_readfirstlane_b32 s12, v2", "s_mov_b32 m0, s1", "s_nop 0", load))
    assert faults(sample("v_mad_u64_u32 v[2:3], s[10:11], v4, s20, 0", "s_nop 3", load))              # its carry
    assert not faults(sample("v_mad_u64_u32 v[2:3], s[10:11], v4, s20, 0", "s_nop 4", load))
    assert not faults(sample("v_mad_u64_u32 v[2:3], s[20:21], v4, s10, 0", load))
    # around a loop: the writer stands behind the load
    assert faults(sample("s_nop 4", "s_mov_b32 m0, s1", "s_nop 0", load, "v_readlane_b32 s9, v2, 1", ("s_cbranch_scc1 1", 4)))


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    if not shutil.which(f"{LLVM}/llvm-objdump"):
        pytest.skip("no disassembler")
    mi.load_library()
    code = dict(kernels(os.path.join(os.path.dirname(mi.__file__), "libmimose.so"), str(tmp_path_factory.mktemp("code"))))
    assert sum(i.to_lds for c in code.values() for i in c) > 100, "the direct loads were not found"
    return {name: faults(c) for name, c in code.items()}


def report(found):
    return "\n".join(f"{name}: {len(bad)}, first {bad[0]}" for name, bad in found.items() if bad)


def test_m0_before_loads_to_lds(built):
    text = report({name: [f for f in bad if f[0] == "m0"] for name, bad in built.items()})
    assert not text, text


def test_scalar_registers_before_vector_memory(built):
    text = report({name: [f for f in bad if f[0] == "sgpr"] for name, bad in built.items()})
    assert not text, text
