"""Build-time check of the generated device code (runs on the build host only).

Compiles every HIP source of the library to device assembly and fails if any
instruction writes through the scalar data cache; the library uses vector
memory instructions for all its stores and atomics. Also checks that the
persistent batched step kernels keep a wave-uniform tile loop (no loop exit
taken lane by lane), which their termination relies on, and the wait states
around matrix-core products that the compiler does not keep by itself.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import re
import subprocess

# Of the scalar-memory instructions only loads are allowed: none whose name
# holds one of these words.
_SCALAR_MEMORY_WORDS = {"store", "atomic", "dcache"}


def _scalar_memory_write(op: str) -> bool:
    words = op.split("_")
    return words[0] == "s" and not _SCALAR_MEMORY_WORDS.isdisjoint(words)


def _device_asm(src: str, hipcc: str, flags, build_dir: str) -> str:
    out = os.path.join(build_dir, os.path.basename(src) + ".s")
    cmd = [hipcc, *flags, "--cuda-device-only", "-S", src, "-o", out]
    if src.endswith(".cpp"):
        cmd = [hipcc, *flags, "-x", "hip", "--cuda-device-only", "-S", src, "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"device asm failed: {' '.join(cmd)}\n{r.stderr}")
    return out


def check_device_code(srcs, jobs, hipcc, flags, build_dir) -> None:
    """Fails if the device code of any source contains a scalar-memory write."""
    with cf.ThreadPoolExecutor(jobs) as ex:
        asms = list(ex.map(lambda s_: _device_asm(s_, hipcc, flags, build_dir), srcs))
    bad = []
    for a in asms:
        with open(a) as fh:
            for ln, line in enumerate(fh, 1):
                if _scalar_memory_write(re.split(r"\s", line.strip(), maxsplit=1)[0]):
                    bad.append(f"{os.path.basename(a)}:{ln}: {line.strip()}")
    if bad:
        raise RuntimeError("scalar-memory writes in device code:\n" + "\n".join(bad[:20]))
    _check_uniform_tile_loops(asms)
    _check_matrix_core_waits(asms)


# The exec-mask update that ends a loop for some lanes only.
_LANE_LOOP_EXIT = "s_andn2_b64 exec, exec"


def _loops_with_barrier_and_lane_exit(text):
    """(kernel, loop header) for every loop that holds a barrier and is left lane by lane.

    Uses the loop annotations the compiler writes on each block label
    ("This Loop Header", "in Loop: Header=...", "Parent Loop ...")."""
    out = []
    for m in re.finditer(r"^(_Z\w+):", text, re.M):
        end = text.find(".Lfunc_end", m.end())
        lines = text[m.end():end if end > 0 else len(text)].split("\n")
        cur, parent, members = None, {}, {}
        for n, line in enumerate(lines):
            lab = re.match(r"^(\.LBB(\w+)|; %bb\.\d+):", line)
            if lab:
                nxt = lines[n + 1] if n + 1 < len(lines) else ""
                both = line + nxt
                hm = re.search(r"Header=BB(\w+)", line)
                if "This Loop Header" in both or "This Inner Loop Header" in both:
                    cur = "BB" + lab.group(2) if lab.group(2) else cur
                    pm = re.search(r"Parent Loop BB(\w+)", both)
                    if pm and lab.group(2):
                        parent[cur] = "BB" + pm.group(1)
                elif hm:
                    cur = "BB" + hm.group(1)
                elif "in Loop" not in line:
                    cur = None
            if cur:
                members.setdefault(cur, []).append(n)
        has_barrier, lane_exit = set(), set()
        for h, idx in members.items():
            for n in idx:
                if "s_barrier" in lines[n]:
                    a = h
                    while a:
                        has_barrier.add(a)
                        a = parent.get(a)
                if _LANE_LOOP_EXIT in lines[n]:
                    lane_exit.add(h)
        out += [(m.group(1), h) for h in sorted(lane_exit & has_barrier)]
    return out


def _check_uniform_tile_loops(asms) -> None:
    """No loop that holds a barrier may be left lane by lane: a lane that left
    alone would park while the rest of its wave waited at the barrier, e.g.
    for a tile index that only the parked lane fetches (the persistent batched
    step kernel's tile loop)."""
    bad = []
    for a in asms:
        with open(a) as fh:
            bad += [f"{os.path.basename(a)}: {k} loop {h}" for k, h in _loops_with_barrier_and_lane_exit(fh.read())]
    if bad:
        raise RuntimeError("barrier inside a lane-divergent loop:\n" + "\n".join(bad[:20]))


# Wait states between a matrix-core product and vector instructions on its
# registers. The compiler keeps them for its own instructions (these figures are
# what it puts behind each product on gfx950) but knows nothing of the
# instructions inside inline assembly: PASSES + 4 before its result is read or
# written (PASSES + 2 for float operands), PASSES - 1 before its C operand is
# written, and 2 from a vector write to a product that reads the register.
# Between products of different shapes on one accumulator the compiler keeps
# none: PASSES are needed (measured with K = 16 and K = 32 bfloat16 products).
_MFMA_PASSES = {
    "v_mfma_f32_16x16x16_f16": 4, "v_mfma_f32_16x16x16_bf16": 4, "v_mfma_f32_16x16x32_f16": 4,
    "v_mfma_f32_16x16x32_bf16": 4, "v_mfma_f32_32x32x8_f16": 8, "v_mfma_f32_32x32x8_bf16": 8,
    "v_mfma_f32_32x32x16_f16": 8, "v_mfma_f32_32x32x16_bf16": 8, "v_mfma_f32_16x16x4_f32": 8,
}
_MFMA_PASSES_MAX = 16
_WRITE_TO_MFMA = 2


def _vregs(operand: str) -> set:
    out = set()
    for kind, a, b, one in re.findall(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", operand):
        out |= {(kind, int(one))} if one else {(kind, i) for i in range(int(a), int(b) + 1)}
    return out


def _instructions(lines):
    """(op, operands, inside inline assembly) of a function's lines, and its labels' positions."""
    ins, labels, inline = [], {}, False
    for line in lines:
        if "#ASMSTART" in line or "#ASMEND" in line:
            inline = "#ASMSTART" in line
            continue
        text = line.split(";", 1)[0].strip()
        lab = re.match(r"^(\.?\w+):", text)
        if lab:
            labels[lab.group(1)] = len(ins)
        elif text and not text.startswith("."):
            op, _, rest = text.replace("\t", " ").partition(" ")
            ins.append((op, [o.strip() for o in rest.split(",")], inline))
    return ins, labels


def _following(ins, labels, start, states):
    """(position, wait states since the instruction at start) of what may run after it."""
    seen, todo = {}, [(start + 1, 0)]
    while todo:
        i, n = todo.pop()
        while i < len(ins) and n < states and seen.get(i, states) > n:
            seen[i] = n
            yield i, n
            op, args, _ = ins[i]
            if op in ("s_endpgm", "s_setpc_b64"):
                break
            if op.startswith(("s_cbranch", "s_branch")) and args[-1] in labels:
                todo.append((labels[args[-1]], n + 1))
                if op == "s_branch":
                    break
            n += int(args[0], 0) + 1 if op == "s_nop" else 1
            i += 1


def _matrix_core_waits(text):
    """(kernel, product, other instruction, wait states between, wait states needed) of every vector
    instruction of inline assembly too close to a matrix-core product on its registers, and of
    every product too close to one of another shape on its accumulator."""
    out = []
    for m in re.finditer(r"^(_Z\w+):", text, re.M):
        end = text.find(".Lfunc_end", m.end())
        ins, labels = _instructions(text[m.end():end if end > 0 else len(text)].split("\n"))

        def show(k):
            return ins[k][0] + " " + ", ".join(ins[k][1])

        for k, (op, args, inline) in enumerate(ins):
            if op.startswith("v_mfma"):
                passes = _MFMA_PASSES.get(op, _MFMA_PASSES_MAX)
                result, c = _vregs(args[0]), _vregs(args[3])
                after = passes + (2 if op.endswith("_f32") and op.count("f32") == 2 else 4)
                for i, n in _following(ins, labels, k, after):
                    o, a, asm = ins[i]
                    if o.startswith("v_mfma") and o != op and n < passes and _vregs(a[3]) & result:
                        out.append((m.group(1), show(k), show(i), n, passes))
                    if not asm or not o.startswith("v_") or o.startswith("v_mfma"):
                        continue
                    need = after if set().union(*map(_vregs, a)) & result else 0
                    if not need and _vregs(a[0]) & c:
                        need = passes - 1
                    if n < need:
                        out.append((m.group(1), show(k), show(i), n, need))
            elif inline and op.startswith("v_"):
                written = _vregs(args[0])
                for i, n in _following(ins, labels, k, _WRITE_TO_MFMA):
                    if ins[i][0].startswith("v_mfma") and set().union(*map(_vregs, ins[i][1][1:])) & written:
                        out.append((m.group(1), show(i), show(k), n, _WRITE_TO_MFMA))
    return out


def _check_matrix_core_waits(asms) -> None:
    """Wait states that the compiler does not keep: see _MFMA_PASSES."""
    bad = []
    for a in asms:
        with open(a) as fh:
            bad += [f"{os.path.basename(a)}: {k}: {i}: {n} wait states from {p}, {need} needed"
                    for k, p, i, n, need in _matrix_core_waits(fh.read())]
    if bad:
        raise RuntimeError(f"{len(bad)} instructions too close to a matrix-core product:\n" + "\n".join(bad[:20]))
