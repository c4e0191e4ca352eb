"""Shared test helpers: seeded inputs as float64, the tolerance rule and a
check of the wait states of direct-to-LDS loads in compiled kernels."""

import re
import subprocess
import tempfile

import numpy as np

from synthetic import storage_to_f64
from synthetic import workloads as W

# Tolerance per storage dtype.
TOL = {"f32": 1e-5, "f16": 2e-2, "bf16": 3e-2}


def inputs_f64(workload, dtype=None, **shape):
    dtype = dtype or W.DEFAULT_DTYPE[workload]
    specs = W.specs(workload, dtype=dtype, **shape)
    raw = W.make_inputs(specs)
    return raw, {k: storage_to_f64(v, dtype) for k, v in raw.items()}


def close(got, ref, tol):
    """Elementwise |g - r| <= tol*|r| + tol*max|r| (a relative bound per element
    plus an absolute one scaled by the output's largest magnitude); returns
    (ok, max_abs, normwise_rel) with normwise_rel = max|g - r| / max|r|."""
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    scale = float(np.max(np.abs(ref))) if ref.size else 0.0
    err = np.abs(got - ref)
    ok = bool(np.all(err <= tol * np.abs(ref) + tol * scale)) and bool(np.all(np.isfinite(got)))
    mx = float(err.max()) if err.size else 0.0
    return ok, mx, (mx / scale if scale > 0 else mx)


def close_elementwise(got, ref, rtol, atol):
    """The stricter rule |g - r| <= rtol*|r| + atol with a fixed absolute floor
    (not scaled by the output's maximum); returns (ok, max_abs, max_rel), where
    max_rel is taken over the elements with |r| > atol / rtol (where the
    relative term dominates)."""
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    err = np.abs(got - ref)
    ok = bool(np.all(err <= rtol * np.abs(ref) + atol)) and bool(np.all(np.isfinite(got)))
    big = np.abs(ref) > atol / rtol
    rel = float(np.max(err[big] / np.abs(ref[big]))) if np.any(big) else 0.0
    return ok, (float(err.max()) if err.size else 0.0), rel


OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def disassemble(code):
    """Instructions of a gfx950 code object built here, as (opcode, [operands])."""
    with tempfile.NamedTemporaryFile(suffix=".co") as f:
        f.write(code)
        f.flush()
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", f.name], capture_output=True, text=True, check=True).stdout
    out = []
    for line in text.splitlines():
        if line.startswith("\t"):
            op, _, rest = line.split("//")[0].strip().partition(" ")
            out.append((op, [t.strip() for t in rest.split(",") if t.strip()]))
    return out


def _sgprs(operand):
    m = re.fullmatch(r"s(?:(\d+)|\[(\d+):(\d+)\])", operand)
    return set() if not m else {int(m[1])} if m[1] else set(range(int(m[2]), int(m[3]) + 1))


def lds_load_faults(ins):
    """(number of direct-to-LDS loads, faults).  The loads are inline assembly,
    whose hazards the compiler does not see.  On gfx9 a scalar write of M0 (the
    load's LDS address) needs one wait state before the load, and a vector
    instruction's write of a scalar register five before a memory instruction
    that reads it (its buffer descriptor or scalar offset); nothing else may use
    M0.  Distances are counted back in program order (an instruction is one wait
    state, s_nop n is n + 1)."""
    loads = [i for i, (op, a) in enumerate(ins) if op.startswith("global_load_lds") or (a and a[-1].split()[-1] == "lds")]
    faults = []
    for i, (op, a) in enumerate(ins):
        if "m0" in a and not (op == "s_mov_b32" and a[0] == "m0" and ins[i + 1][0] == "s_nop" and i + 2 in loads):
            faults.append(f"m0: {op} {a} then {ins[i + 1]}")
    for i in loads:
        if ins[i - 2][:1] + tuple(ins[i - 2][1][:1]) != ("s_mov_b32", "m0"):
            faults.append(f"load without its own M0: {ins[i]}")
        reads = set().union(*(_sgprs(t.split()[0]) for t in ins[i][1]))
        states = 0
        for op, a in reversed(ins[:i]):
            if states >= 5:
                break
            dests = a[: 2 if "_co_" in op or "div_scale" in op else 1]
            if op.startswith("v_") and any(_sgprs(t) & reads for t in dests):
                faults.append(f"{op} {a} {states} wait states before {ins[i]}")
            states += int(a[0], 0) + 1 if op == "s_nop" else 1
    return len(loads), faults
