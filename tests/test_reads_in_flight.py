"""The direct-to-LDS FP16 kernels read their operands from LDS with inline assembly, which the compiler takes to be complete at once:
the kernels wait themselves.  Host-only check of the built device code: no instruction may touch a register that an LDS read is still to
write.  LDS reads return in the order they were issued, so a wait for N outstanding ones covers all but the last N."""
import re
import struct
import subprocess

from paper_1705_05249_amd import gemm as G

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
KERNEL = re.compile(r"^[0-9a-f]+ <(_ZN2mg1[56]hgemm_(?:dma|pp)_kernelI\w+EvNS_8MfmaArgsE)>:$")
REGISTERS = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def device_objects():
    """the gfx950 code objects in the library that hold one of the kernels"""
    data = open(G.LIB_PATH, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        entries, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24: p + 24 + length]
            p += 24 + length
            code = data[at + offset: at + offset + size]
            if b"gfx950" in target and (b"hgemm_dma_kernel" in code or b"hgemm_pp_kernel" in code):
                yield code
        at = data.find(MAGIC, at + 1)


def kernels(path):
    """(name, [(address, instruction, branch target or None)]) of every direct-to-LDS kernel in a code object"""
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", path], check=True, capture_output=True, text=True).stdout
    name, start, body = None, 0, []
    for line in text.split("\n") + ["0 <end>:"]:
        if line.endswith(">:"):
            if name:
                yield name, body
            head = KERNEL.match(line)
            name, start, body = (head.group(1), int(line.split()[0], 16), []) if head else (None, 0, [])
        elif name and "//" in line:
            code, note = line.split("//", 1)
            target = re.search(r"<\w+(?:\+0x([0-9a-f]+))?>", note)
            body.append((int(note.split(":")[0], 16), code.strip(), start + int(target.group(1) or "0", 16) if target else None))


def registers(operands):
    found = set()
    for kind, low, high, single in REGISTERS.findall(operands):
        found.update((kind, r) for r in (range(int(low), int(high) + 1) if low else [int(single)]))
    return found


def touched_in_flight(body):
    """instructions that read or write a register which an earlier LDS read may still write; per register the number of LDS
    operations issued behind its read, the smallest over all paths to a place"""
    index = {address: i for i, (address, _, _) in enumerate(body)}
    before, work, touched, reads = {0: {}}, [0], set(), 0
    decoded = []
    for _, code, _ in body:
        op, _, operands = code.partition(" ")
        wait = re.search(r"lgkmcnt\((\d+)\)", operands) if op == "s_waitcnt" else None
        first, _, rest = operands.partition(",")
        decoded.append((op, int(wait.group(1)) if wait else None, registers(first), registers(rest)))
        reads += op.startswith("ds_read")
    while work:
        i = work.pop()
        flight = dict(before[i])
        while True:
            op, wait, first, rest = decoded[i]
            if wait is not None:
                flight = {r: age for r, age in flight.items() if age < wait}
            elif op.startswith("ds_"):
                used = rest if op.startswith("ds_read") else first | rest
                if any(r in flight for r in used):
                    touched.add(body[i][1])
                flight = {r: min(age + 1, 16) for r, age in flight.items()}
                if op.startswith("ds_read"):
                    flight.update((r, 0) for r in first)
            elif not op.startswith("s_") and any(r in flight for r in first | rest):
                touched.add(body[i][1])
            if op == "s_endpgm":
                break
            following = [i + 1] if op != "s_branch" else []
            if op.startswith(("s_cbranch", "s_branch")):
                following.append(index[body[i][2]])
            stop = len(following) != 1 or following[0] != i + 1 or following[0] in before
            for j in following if stop else ():
                known = before.get(j)
                merged = dict(flight) if known is None else {r: min(known.get(r, 99), flight.get(r, 99)) for r in known.keys() | flight.keys()}
                if merged != known:
                    before[j] = merged
                    work.append(j)
            if stop:
                break
            i = following[0]
    return reads, touched


def test_no_register_is_touched_while_a_read_may_write_it(tmp_path):
    seen, wrong = 0, {}
    for n, code in enumerate(device_objects()):
        path = tmp_path / f"{n}.co"
        path.write_bytes(code)
        for name, body in kernels(str(path)):
            reads, touched = touched_in_flight(body)
            seen += reads > 0
            if touched:
                wrong[name] = sorted(touched)[:4]
    assert seen >= 40, seen
    assert not wrong, wrong
