"""Build step: compiles the HIP sources into the C-ABI shared library, in-tree.

    python -m paper_2505_21487_amd.build            # build the library
    python -m paper_2505_21487_amd.build --check    # code-generation checks (check_register_windows, check_uniform_loads)
"""
from __future__ import annotations

import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgla_decode.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Wall", "-Wno-unused-function",
    # packed-fp32 VALU ops are not to be generated on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def sources():
    return [os.path.join(CSRC, "library.hip")]  # (one unit: see there)


def needs_build() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC)]
    deps.append(os.path.join(os.path.dirname(HERE), "include", "gla_decode.h"))
    return any(os.path.getmtime(d) > t for d in deps)


def build(verbose: bool = True, extra_flags=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + f".tmp{os.getpid()}"
    cmd = [hipcc] + HIPCC_FLAGS + list(extra_flags) + ["-o", tmp] + sources()
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


def check_register_windows(verbose: bool = True) -> list:
    """Code-generation check for the kernels that keep page-id windows in registers
    (pages of 8 tokens or fewer with the 512-dim latent).  Those registers are
    loaded asynchronously by one inline-assembly statement and must stay where
    they are until the load has landed: any copy the compiler makes of them in
    between would carry stale page ids.  Compiles those kernels to assembly and
    verifies, per kernel, that every load site names the same registers and that
    nothing else in the kernel writes them after the first site (before it they
    are set to zero).  Returns one description per kernel; raises on a violation."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    with tempfile.TemporaryDirectory() as tmp:
        asm = os.path.join(tmp, "check.s")
        cmd = [hipcc] + flags + ["--cuda-device-only", "-S", "-o", asm, os.path.join(CSRC, "check_register_windows.hip")]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd, stderr=subprocess.DEVNULL)
        text = open(asm).read()
    found = []
    for fn in re.split(r"\n(?=_ZN3gla17tuned_main_kernel\S*: ; @)", text):
        m = re.match(r"(_ZN3gla17tuned_main_kernel\S*):", fn)
        if not m or "gla_win_skip" not in fn:
            continue
        lines = fn.split(".Lfunc_end")[0].split("\n")
        sites, in_site = [], set()
        for i, line in enumerate(lines):
            if "s_cbranch_scc1 .Lgla_win_skip" not in line:
                continue
            regs, j = [], i + 1
            while "global_load_dword" in lines[j]:
                regs.append(int(re.search(r"global_load_dword v(\d+),", lines[j]).group(1)))
                in_site.add(j)
                j += 1
            sites.append((i, regs))
        first = sorted(set(tuple(r) for k, (_, r) in enumerate(sites) if k % 2 == 0))
        second = sorted(set(tuple(r) for k, (_, r) in enumerate(sites) if k % 2 == 1))
        if not sites or len(first) != 1 or len(second) != 1:
            raise RuntimeError(f"{m.group(1)}: load sites disagree on the window registers: {first} {second}")
        window = set(first[0]) | set(second[0])
        for k, line in enumerate(lines):
            t = line.strip()
            if k in in_site or not t or t[0] in ";." or t.endswith(":"):
                continue
            op, _, rest = t.partition(" ")
            if op.startswith(("s_", "ds_write", "global_store", "scratch_store", "buffer_store")):
                continue
            dst = rest.split(",")[0].strip()
            one, many = re.fullmatch(r"v(\d+)", dst), re.fullmatch(r"v\[(\d+):(\d+)\]", dst)
            written = {int(one.group(1))} if one else set(range(int(many.group(1)), int(many.group(2)) + 1)) if many else set()
            zeroed = re.fullmatch(r"v_mov_b32_e32 v\d+, 0", t) or (k < sites[0][0] and op == "v_mov_b32_e32")
            if written & window and not zeroed:
                raise RuntimeError(f"{m.group(1)}: window register written outside the load statement: {t}")
        found.append(f"{m.group(1)}: windows {first[0]} {second[0]}, {len(sites)} load sites")
    if len(found) != 2:
        raise RuntimeError(f"expected two kernels with register windows, found {len(found)}")
    if verbose:
        print("\n".join(found))
    return found


def device_code(lib: str = LIB, tool=("llvm-objdump", "-d", "--no-show-raw-insn")) -> str:
    """Disassembly of the built library's device code object, or what another tool prints of it."""
    llvm = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
    with tempfile.TemporaryDirectory() as tmp:
        fat, obj = os.path.join(tmp, "fat"), os.path.join(tmp, "gfx950.o")
        subprocess.check_call([os.path.join(llvm, "llvm-objcopy"), "--dump-section", ".hip_fatbin=" + fat, lib, os.devnull])
        subprocess.check_call([os.path.join(llvm, "clang-offload-bundler"), "--unbundle", "--type=o", "--input=" + fat,
                               "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--output=" + obj])
        return subprocess.check_output([os.path.join(llvm, tool[0]), *tool[1:], obj], text=True)


# tuned_main_kernel<DV, DN, DR, NG, WPG, KS, TOK, STAGES, PM, STREAM> in page modes 0 and 1
_UNIFORM_LOADS = re.compile(r"tuned_main_kernelI(?:Li\d+E){8}Li[01]E")


def _sgprs(operand: str) -> set:
    """Scalar registers of an operand (vcc: 106 and 107)."""
    m = re.match(r"s\[(\d+):(\d+)\]|s(\d+)\b", operand)
    if m:
        return {int(m.group(3))} if m.group(3) else set(range(int(m.group(1)), int(m.group(2)) + 1))
    return {"vcc": {106, 107}, "vcc_lo": {106}, "vcc_hi": {107}}.get(operand.split(" ")[0], set())


def check_uniform_loads(text: str) -> list:
    """Checks, in a disassembly, what the compiler does not see of direct-to-LDS loads written in assembly with a scalar base.

    In every kernel: a vector-memory instruction reads a scalar base at the earliest five wait states after a vector
    instruction wrote it, on every path to it.  In the kernels whose tile loads are assembly: m0 is written by nothing but
    "s_mov_b32 m0" with a wait state behind it, used by no load but those, and a load with an offset follows the one 1024 bytes
    before it with m0 untouched.  Returns one description per kernel of the second kind; raises on a violation."""
    found = []
    for fn in re.split(r"\n(?=[0-9a-f]+ <)", text):
        head = re.match(r"\s*([0-9a-f]+) <(\S+)>:", fn)
        if not head or "s_endpgm" not in fn:
            continue
        base, name = int(head.group(1), 16), head.group(2)
        ops, at, jumps = [], {}, {}
        for line in fn.split("\n")[1:]:
            m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):(.*)", line)
            if not m:
                continue
            at[int(m.group(3), 16)] = len(ops)
            target = re.search(r"<\S+?(?:\+0x([0-9a-f]+))?>", m.group(4)) if m.group(1).startswith(("s_cbranch", "s_branch")) else None
            if target:
                jumps.setdefault(base + int(target.group(1) or "0", 16), []).append(len(ops))
            ops.append((m.group(1), [x.strip() for x in m.group(2).split(",")]))
        into = {at[a]: src for a, src in jumps.items()}

        def before(i):  # the instructions that may run directly ahead of the i-th
            prev = [] if i == 0 or ops[i - 1][0] in ("s_branch", "s_endpgm") else [i - 1]
            return prev + into.get(i, [])

        for i, (op, args) in enumerate(ops):
            if not op.startswith(("global_", "buffer_", "scratch_")):
                continue
            regs = set().union(*[_sgprs(a) for a in args])
            todo, seen = [(j, 0) for j in before(i)] if regs else [], set()
            while todo:
                j, states = todo.pop()
                if states >= 5 or (j, states) in seen:
                    continue
                seen.add((j, states))
                o, a = ops[j]
                # (a scalar result is the first operand or, of carries, products with one and scaled divisions, the second)
                vector = re.match(r"v(\d|\[)", a[0])
                second = re.match(r"v_(add_co|addc_co|sub_co|subb_co|subrev_co|subbrev_co|div_scale|mad_[iu]64)", o)
                if o.startswith("v_") and regs & (_sgprs(a[1]) if vector and second else _sgprs(a[0])):
                    raise RuntimeError(f"{name}: {op} {', '.join(args)} reads a base written {states} wait states before by {o} {', '.join(a)}")
                todo += [(k, states + (int(a[0], 0) + 1 if o == "s_nop" else 1)) for k in before(j)]

        if not _UNIFORM_LOADS.search(name):
            continue
        offset, loads = None, 0  # offset: of the last load since m0 was written; -1024 right behind that
        for i, (op, args) in enumerate(ops):
            if "_lds_" in op:
                m = re.match(r"s\[\d+:\d+\](?: offset:(\d+))?", args[-1])
                if not op.startswith("global_load_lds") or not m or offset is None or int(m.group(1) or 0) != offset + 1024:
                    raise RuntimeError(f"{name}: {op} {', '.join(args)} is not one of the tile loads, or not behind the write of m0 meant for it")
                offset, loads = offset + 1024, loads + 1
            elif any(re.search(r"\bm0\b", a) for a in args):
                if op != "s_mov_b32" or args[0] != "m0" or ops[i + 1][0] != "s_nop":
                    raise RuntimeError(f"{name}: m0 in {op} {', '.join(args)}")
                offset = -1024
            elif op.startswith(("s_sendmsg", "s_movrel", "v_movrel", "ds_gws", "v_interp")) or "addtid" in op:
                raise RuntimeError(f"{name}: {op} uses m0")
        found.append(f"{name}: {loads} tile loads")
    return found


if __name__ == "__main__":
    if sys.argv[1:] == ["--check"]:
        check_register_windows()
        print("\n".join(check_uniform_loads(device_code())))
    else:
        build(extra_flags=sys.argv[1:])
