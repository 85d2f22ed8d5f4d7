"""What the compiler says about the kernels of the built library: the metadata of its gfx950 code objects, read from the file."""
import os
import re
import struct
import subprocess

import msgpack

from paper_2111_14255_amd import build


def objects():
    """The gfx950 code objects (ELF images) of the library's offload bundles."""
    data = open(os.environ.get("MTSCHED_LIB") or build.lib_path(), "rb").read()
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + 24)
        pos = at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<3Q", data, pos)
            target = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if size and b"gfx950" in target:
                yield data[at + offset:at + offset + size]
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", pos)


def kernels():
    """Metadata of every kernel, by mangled name."""
    out = {}
    for elf in objects():
        headers, = struct.unpack_from("<Q", elf, 32)
        n, = struct.unpack_from("<H", elf, 56)
        for i in range(n):
            kind, _, offset = struct.unpack_from("<IIQ", elf, headers + 56 * i)
            if kind != 4:                                    # PT_NOTE
                continue
            name, size, note = struct.unpack_from("<III", elf, offset)
            if note == 32:                                   # NT_AMDGPU_METADATA
                at = offset + 12 + (name + 3) // 4 * 4
                out.update({k[".name"]: k for k in msgpack.unpackb(elf[at:at + size], strict_map_key=False)["amdhsa.kernels"]})
    return out


def held_by_registers(kernel):
    """Workgroups of a kernel whose registers a compute unit holds: 512 per lane of each of four SIMDs, given out in eights."""
    waves = kernel[".max_flat_workgroup_size"] // 64
    return 512 // ((kernel[".vgpr_count"] + 7) // 8 * 8) * 4 // waves


def listings():
    """Assembly of the code objects, kernel by kernel: (name, [(address, mnemonic, operands)])."""
    for elf in objects():
        text = subprocess.run(["/opt/rocm/llvm/bin/llvm-objdump", "-d", "--mcpu=gfx950", "-"], input=elf, capture_output=True, check=True).stdout.decode()
        for part in re.split(r"\n(?=[0-9a-f]+ <)", text)[1:]:
            head, _, body = part.partition("\n")
            yield head, [(int(a, 16), m, [o.strip() for o in ops.split(",")]) for m, ops, a in re.findall(r"^\t(\S+) ?(.*?)\s*// ([0-9A-F]+):", body, re.M)]


def scalars(operand):
    """Scalar registers an operand names: s7, s[4:7], vcc, m0."""
    m = re.match(r"(?:s\[(\d+):(\d+)\]|s(\d+)$)", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1)) if m[1] else {int(m[3])}
    return {operand} if operand in ("vcc", "m0") else set()


def predecessors(code):
    """For every instruction the ones that may run just before it."""
    at = {a: i for i, (a, _, _) in enumerate(code)}
    came_from = [[] for _ in code]
    for i, (a, m, ops) in enumerate(code):
        if m not in ("s_branch", "s_endpgm", "s_setpc_b64") and i + 1 < len(code):
            came_from[i + 1].append(i)
        if m.startswith(("s_branch", "s_cbranch")):
            offset = int(re.match(r"\d+", ops[0])[0])
            came_from[at[a + 4 + 4 * (offset - 65536 if offset > 32767 else offset)]].append(i)
    return came_from


def staging_loop(code):
    """The shortest run of instructions between a branch backwards and where it goes that copies to LDS and multiplies."""
    at = {a: i for i, (a, _, _) in enumerate(code)}
    found = []
    for i, (a, m, ops) in enumerate(code):
        if m.startswith(("s_branch", "s_cbranch")):
            offset = int(re.match(r"\d+", ops[0])[0])
            j = at[a + 4 + 4 * (offset - 65536 if offset > 32767 else offset)]
            if j < i and any(w.startswith("v_mfma") for _, w, _ in code[j:i]) and any(o[-1].split()[-1:] == ["lds"] for _, _, o in code[j:i]):
                found.append(code[j:i + 1])
    return min(found, key=len)


def held_back_stores(code):
    """Stores to memory that stop at the XCD's L2 (no sc1), and stores that a wave may end without waiting for."""
    came_from = predecessors(code)
    stores = lambda m: re.match(r"(buffer|global|flat)_store", m)
    found = [(hex(a), m) for a, m, ops in code if stores(m) and "sc1" not in ops[-1].split()]
    seen, todo = set(), [i for i, (_, m, _) in enumerate(code) if m == "s_endpgm"]
    while todo:
        for j in came_from[todo.pop()]:
            a, m, ops = code[j]
            if j in seen or (m == "s_waitcnt" and "vmcnt(0)" in " ".join(ops)):
                continue
            seen.add(j)
            if stores(m):
                found.append((hex(a), m))
            todo.append(j)
    return found


def early_lds_loads(code, states=5):
    """Loads to LDS that read a scalar register which a vector instruction wrote fewer than `states` wait states before, on any path."""
    came_from = predecessors(code)
    found = []
    for i, (a, m, ops) in enumerate(code):
        if not (m.startswith("buffer_load") and ops[-1].split()[-1] == "lds"):
            continue
        reads = scalars(ops[1]) | scalars(ops[2].split()[0]) | {"m0"}
        todo = [(j, states) for j in came_from[i]]
        while todo:
            j, left = todo.pop()
            _, mj, oj = code[j]
            # results: the first operand, of additions with carry, divisions and 64-bit multiply-adds the second as well
            results = scalars(oj[0]) | (scalars(oj[1]) if re.search("_co_|div_scale|mad_[iu]64", mj) else set())
            if mj.startswith("v_") and results & reads:
                found.append((hex(a), mj))
            left -= int(oj[0], 0) + 1 if mj == "s_nop" else 1
            if left > 0:
                todo += [(k, left) for k in came_from[j]]
    return found
