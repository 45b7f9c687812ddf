"""LDS and scalar-memory operations in flight in the kernels whose waits are counted by hand (table and row-lane kernels), read off the
gfx950 code of the built library: the counter those waits compare with has four bits, and the kernels are written to have at most 15
operations in flight where one of them expects some still to be."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2602_15563_amd import kmq

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler for code built here")
COUNTED = re.compile(r"gemv_lut_kernel|gemm_lut_columns_kernel|gemv_lut_loop_kernel|rowlane")
MOST = 15


def device_code(path):
    """The gfx950 code objects that hipcc put into a library."""
    data = open(path, "rb").read()
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        p = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            if size and b"gfx950" in data[p + 24:p + 24 + n]:
                yield data[at + off:at + off + size]
            p += 24 + n
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def kernels(code, path):
    """(name, [(address, mnemonic, operands)]) of every function."""
    path.write_bytes(code)
    text = subprocess.run([OBJDUMP, "-d", str(path)], capture_output=True, text=True, check=True).stdout
    name, body = None, []
    for line in text.splitlines():
        if head := re.match(r"[0-9a-f]+ <(.+)>:", line):
            if name:
                yield name, body
            name, body = head[1], []
        elif ins := re.match(r"\t(\S+)\s*(.*?)\s*// ([0-9A-F]+):", line):
            body.append((int(ins[3], 16), ins[1], ins[2]))
    if name:
        yield name, body


def most_at_counted_wait(body):
    """The most operations in flight, on any path, where an s_waitcnt that expects some to remain is met behind the first
    hand-written lookup (an address whose low byte a masked byte replaces)."""
    index = {address: i for i, (address, _, _) in enumerate(body)}
    heads, follows = {0}, {}
    first = next((i for i, (_, op, args) in enumerate(body) if op == "v_and_b32_sdwa" and "UNUSED_PRESERVE" in args), len(body))
    for i, (address, op, args) in enumerate(body):
        if op.startswith(("s_branch", "s_cbranch")):
            offset = int(args.split()[0])
            target = index[address + 4 + 4 * (offset - 65536 if offset >= 32768 else offset)]
            follows[i] = [target] if op == "s_branch" else [target, i + 1]
            heads.update([target, i + 1])
        elif op == "s_endpgm":
            follows[i] = []
            heads.add(i + 1)
    entry, work, worst = {0: 0}, [0], 0
    while work:
        i = work.pop()
        n = entry[i]
        while True:
            _, op, args = body[i]
            if op.startswith(("ds_", "s_load", "s_buffer_load", "s_scratch_load", "s_memtime", "s_memrealtime")):
                n = min(n + 1, 99)
            elif op == "s_waitcnt" and (left := re.search(r"lgkmcnt\((\d+)\)", args)):
                if 0 < int(left[1]) < MOST and i > first:
                    worst = max(worst, n)
                n = min(n, int(left[1]))
            nexts = follows.get(i)
            if nexts is None and i + 1 in heads:
                nexts = [i + 1]
            if nexts is None:
                i += 1
                continue
            for j in nexts:
                if j < len(body) and entry.get(j, -1) < n:
                    entry[j] = n
                    work.append(j)
            break
    return worst


def test_counted_waits_see_at_most_fifteen(tmp_path):
    seen, over = 0, {}
    for code in device_code(kmq.LIB_PATH):
        for name, body in kernels(code, tmp_path / "code.o"):
            if COUNTED.search(name):
                seen += 1
                n = most_at_counted_wait(body)
                if n > MOST:
                    over[name] = n
    assert seen > 100
    assert not over, f"{len(over)} of {seen} kernels, up to {max(over.values())} in flight: {sorted(over.items())[:4]}"
