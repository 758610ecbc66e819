"""Reads the gfx950 code that this repository builds (no GPU): the kernels of the built library as instruction lists, and
a walk over all their paths that follows the LDS reads a wave has in flight across its barriers."""
import os
import re
import shutil
import subprocess

import paper_2303_04759_amd as raf

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
LINE = re.compile(r"^\t(\S+)\s*(.*?)\s*// ([0-9A-F]{12}):(?:.*<(\S+?)(?:\+0x([0-9a-f]+))?>)?")


def kernels(tmp_path, contains):
    """{symbol: [(offset, opcode, operands, branch target offset or None)]} of the kernels whose symbol contains a text."""
    if not os.path.exists(raf.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    lib = shutil.copy(raf.LIB_PATH, str(tmp_path / "lib.so"))
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, stdout=subprocess.DEVNULL, cwd=str(tmp_path))
    out = {}
    for name in sorted(os.listdir(str(tmp_path))):
        if "gfx950" not in name:
            continue
        path = str(tmp_path / name)
        table = subprocess.run([OBJDUMP, "-t", path], check=True, capture_output=True, text=True).stdout
        syms = [w for w in table.split() if contains in w and not w.endswith(".kd")]
        if not syms:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--disassemble-symbols=" + ",".join(sorted(set(syms))), path], check=True,
                              capture_output=True, text=True).stdout
        code, base = None, 0
        for line in text.splitlines():
            head = re.match(r"^([0-9a-f]+) <(\S+)>:$", line)
            if head:
                base, code = int(head.group(1), 16), out.setdefault(head.group(2), [])
                continue
            m = LINE.match(line)
            if m and code is not None:
                target = int(m.group(5) or "0", 16) if m.group(4) else None
                code.append((int(m.group(3), 16) - base, m.group(1), m.group(2), target))
    return out


def _far_target(code, i):
    """Offset that a branch too far for one instruction goes to: s_getpc_b64, s_add_u32, s_addc_u32, s_setpc_b64."""
    (_, op0, reg, _), (off, op1, add, _), (_, op2, carry, _), (_, _, to, _) = code[i - 3:i + 1]
    assert (op0, op1, op2) == ("s_getpc_b64", "s_add_u32", "s_addc_u32") and reg == to, "calls are not followed"
    delta = int(add.split(",")[2], 0)
    return off + (delta - (1 << 32) if delta >= 1 << 31 else delta)


def barriers_crossed_by_lds_reads(code):
    """Over all paths of a kernel: the most workgroup barriers that a wave passes between issuing an LDS read and its first
    wait that covers the read.  Reads return in order, so a wait for lgkmcnt(n) covers all but the last n operations."""
    index = {off: i for i, (off, _, _, _) in enumerate(code)}
    worst, seen, todo = 0, set(), [(0, ())]
    while todo:
        i, fly = todo.pop()
        while True:
            if (i, fly) in seen:
                break
            seen.add((i, fly))
            _, op, args, target = code[i]
            if op.startswith("ds_"):
                fly = fly + ((0,) if op.startswith("ds_read") else (None,))
                # more in flight than the counter holds: the oldest are kept as one
                if len(fly) > 20:
                    ages = [a for a in fly[:-19] if a is not None]
                    fly = ((max(ages) if ages else None),) + fly[-19:]
            elif op.startswith("s_load") or op.startswith("s_buffer_load"):
                fly = fly + ("scalar",)     # returns out of order: only a wait for zero covers it
            elif op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", args)
                if m or args in ("0", "0x0"):
                    n = int(m.group(1)) if m else 0
                    if n == 0:
                        fly = ()
                    elif "scalar" not in fly:
                        fly = fly[-n:]
            elif op == "s_barrier":
                fly = tuple(a + 1 if isinstance(a, int) else a for a in fly)
                worst = max([worst] + [a for a in fly if isinstance(a, int)])
                if worst > 8:
                    return worst
            elif op == "s_endpgm":
                break
            assert not op.startswith("s_swappc"), "calls are not followed"
            if op == "s_setpc_b64":
                i = index[_far_target(code, i)]
                continue
            if op == "s_branch":
                i = index[target]
                continue
            if op.startswith("s_cbranch"):
                todo.append((index[target], fly))
            i += 1
    return worst
