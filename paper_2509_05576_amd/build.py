"""Build libfobq.so (HIP, gfx950 only) in-tree with hipcc."""
from __future__ import annotations

import concurrent.futures
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libfobq.so")
SOURCES = ["api.hip", "gemm64.hip", "hessian.hip", "hessian_i8.hip", "hessian_offsets.hip", "factor.hip", "flow.hip", "quant.hip", "obq.hip", "probe.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]
# Sources whose kernels use DPP operands in inline asm (csrc/tile_block.h).  The compiler neither sees nor keeps the wait states
# that those need, so its listing is checked: with another compiler, or after a change, a copy of such an operand may land right
# in front of its use.
DPP_SOURCES = ["factor.hip", "flow.hip"]


def _registers(operand: str) -> set[int]:
    m = re.fullmatch(r"[-|]?v(?:(\d+)|\[(\d+):(\d+)\])\|?", operand.strip())
    if not m:
        return set()
    return {int(m[1])} if m[1] else set(range(int(m[2]), int(m[3]) + 1))


def dpp_hazards(listing: str) -> list[str]:
    """The instructions of an AMD listing whose DPP operand a vector instruction wrote less than two wait states before, or that come
    less than five behind a vector write of EXEC, with their line numbers.  What stands in front of a label is not known here:
    a DPP operand whose wait states reach back across one counts as a hit, too."""
    hits, before = [], []                # before: (wait states, registers written by a vector instruction, EXEC written so), None: a label
    for number, line in enumerate(listing.splitlines(), 1):
        text = re.split(r";|//", line)[0].strip()
        if not text or text.startswith("."):
            if re.match(r"\.?[A-Za-z_$][\w.$]*:", text):
                before.append(None)
            continue
        if re.match(r"[\w.$]+:", text):
            before.append(None)
            continue
        name, _, rest = text.partition(" ")
        operands = [o.strip() for o in rest.split(",")]
        if "_dpp" in name:
            source = _registers(operands[1])
            waited = 0
            for item in reversed(before):
                if waited >= 5:
                    break
                if item is None:
                    if waited < 2:
                        hits.append(f"{number}: {text} (label)")
                    break
                states, written, execs = item
                if (waited < 2 and written & source) or execs:
                    hits.append(f"{number}: {text}")
                    break
                waited += states
        written = set()
        if name.startswith("v_"):
            written = _registers(operands[0])
            if "swap" in name and len(operands) > 1:
                written |= _registers(operands[1])
        states = int(operands[0], 0) + 1 if name == "s_nop" else 1
        before.append((states, written, name.startswith("v_cmpx")))
        del before[:-8]
    return hits


def _check_dpp(src: str) -> None:
    cmd = ["hipcc", *FLAGS, "--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", "-"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0 or "_dpp" not in res.stdout:
        raise RuntimeError(f"no listing of {src} to check its DPP operands in:\n{res.stderr}")
    hits = dpp_hazards(res.stdout)
    if hits:
        raise RuntimeError(f"{src}: DPP operands used too soon after they were written:\n" + "\n".join(hits[:10]))


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    msgs = "\n".join(l for l in (res.stdout + res.stderr).splitlines()
                     if "packed-fp32-ops" not in l)  # host pass does not know the device feature
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{msgs}")
    if msgs.strip():
        print(msgs, file=sys.stderr)
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        checks = [ex.submit(_check_dpp, src) for src in DPP_SOURCES]
        objs = list(ex.map(_compile, SOURCES))
        for c in checks:
            c.result()
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stdout + res.stderr)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
