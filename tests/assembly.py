"""The gfx950 code of the built library, as the disassembler prints it: {kernel: [instruction, ...]}, for the checks of test_assembly.py."""
import os
import re
import struct
import subprocess

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
OBJCOPY = "/opt/rocm/llvm/bin/llvm-objcopy"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def kernels(library, tmp):
    fat = os.path.join(tmp, "fat")
    subprocess.run([OBJCOPY, "-O", "binary", "--only-section=.hip_fatbin", library, fat], check=True, capture_output=True)
    with open(fat, "rb") as f:
        blob = f.read()
    out, at = {}, blob.find(MAGIC)
    while at >= 0:                                         # one bundle per source file: magic, entries, each {offset, size, length of its triple, triple}
        p, (count,) = at + len(MAGIC) + 8, struct.unpack_from("<Q", blob, at + len(MAGIC))
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", blob, p)
            triple, p = blob[p + 24:p + 24 + length].decode(), p + 24 + length
            if size and "gfx950" in triple:
                obj = os.path.join(tmp, "code")
                with open(obj, "wb") as f:
                    f.write(blob[at + offset:at + offset + size])
                text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", obj], check=True, capture_output=True, text=True).stdout
                name = None
                for line in text.splitlines():
                    head = re.match(r"[0-9a-f]+ <(\S+)>:$", line)
                    if head:
                        name = head[1] if not head[1].startswith("L") else name
                        out.setdefault(name, [])
                    elif name and line.startswith("\t"):
                        out[name].append(line.split("//")[0].strip())
        at = blob.find(MAGIC, at + 1)
    return out


def registers(operand):
    """{("v", 3), ...} of an operand such as v3, s[4:7], vcc."""
    m = re.match(r"([vs])\[(\d+):(\d+)\]$", operand)
    if m:
        return {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
    m = re.match(r"([vs])(\d+)$", operand)
    return {(m[1], int(m[2]))} if m else {(operand, 0)}


def operands(instruction):
    return [o for o in re.split(r"[ ,]+", instruction)[1:] if o]


def wait_states(instruction):
    return int(instruction.split()[1], 0) + 1 if instruction.startswith("s_nop") else 1
