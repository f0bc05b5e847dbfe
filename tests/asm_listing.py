"""Assembly listings of the kernels built here, and what tests read in them.

product_hazards: the result of a matrix product in inline assembly that an
instruction touches before the matrix core has written it.  The hardware does
not wait by itself on gfx950: an instruction other than a product of the same
accumulator (same destination, as its addend) must come at least 19 wait states
after a v_mfma_f64_16x16x4_f64 and 12 after a v_mfma_f32_32x32x16_bf16, along
every path.  The compiler pads builtin products, but cannot see into inline
assembly, nor does it know that a copy or spill of its own reads a product's
result.

scalar_offset_accesses: buffer accesses with a scalar offset.  The bounds check
of a buffer resource leaves that offset out, so a row's address has to be in
the vector offset for rows past the end to read as zeros.

kernel_resources: the registers and LDS of each kernel.
"""
import os
import re
import subprocess

F64, BF16 = "v_mfma_f64_16x16x4_f64", "v_mfma_f32_32x32x16_bf16"
WAIT = {F64: 19, BF16: 12}  # wait states between a product and a read (or another write) of its result
_CACHE = {}


def listing(src):
    """The listing of a kernel source compiled with the library's own flags (None without a compiler)."""
    from paper_2609_19242_amd import build

    if src not in _CACHE:
        try:
            cc = build.hipcc()
        except RuntimeError:
            return None
        cmd = [cc, *build.flags(), *build.EXTRA_FLAGS.get(src, []), "-x", "hip", "-S", "--cuda-device-only",
               os.path.join(build.CSRC, src), "-o", "-"]
        _CACHE[src] = subprocess.run(cmd, check=True, capture_output=True, text=True).stdout
    return _CACHE[src]


_REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def _regs(operand):
    out = set()
    for m in _REG.finditer(operand):
        lo = int(m.group(2) or m.group(4))
        hi = int(m.group(3) or m.group(4))
        out |= {(m.group(1), i) for i in range(lo, hi + 1)}
    return frozenset(out)


def functions(listing):
    """{name: [(line number, label or None, mnemonic, operands)]} of a listing's functions."""
    out, name, body = {}, None, []
    for n, raw in enumerate(listing.split("\n"), 1):
        line = raw.split(";", 1)[0].split("//", 1)[0].strip()
        m = re.match(r"([.\w$]+):", line)
        if m:
            if name is None and m.group(1).startswith("_Z"):
                name, body = m.group(1), []
            elif name is not None:
                body.append((n, m.group(1), None, ()))
            line = line[m.end():].strip()
        if name is None or not line:
            continue
        if line.startswith("."):
            if line.startswith((".end_amdhsa_kernel", ".size", ".section")):
                out[name] = body
                name = None
            continue
        parts = line.split(None, 1)
        ops = tuple(o.strip() for o in re.split(r",(?![^\[]*\])", parts[1])) if len(parts) > 1 else ()
        body.append((n, None, parts[0], ops))
    return out


def product_hazards(body, product=F64, accumulators="v"):
    """[(line of the use, line of the product, wait states between)] of one function, over all its paths, for the
    products whose accumulators are in the given register file."""
    wait = WAIT[product]
    ours = lambda op, ops: op == product and ops[0].startswith(accumulators)  # noqa: E731
    at_label = {lab: i for i, (_, lab, _, _) in enumerate(body) if lab}
    found = {}
    # state: register -> (wait states still missing, line of the product); worklist over instruction indices
    seen, work = {}, [(0, {})]
    while work:
        i, state = work.pop()
        while i < len(body):
            line, label, op, ops = body[i]
            if label is not None:
                old = seen.get(i, {})
                merged = dict(old)
                for r, v in state.items():
                    if r not in merged or merged[r][0] < v[0]:
                        merged[r] = v
                if i in seen and merged == old:
                    break
                seen[i] = merged
                state = dict(merged)
                i += 1
                continue
            touched = set()
            if ours(op, ops):
                dst, addend = _regs(ops[0]), _regs(ops[3])
                touched = set(_regs(ops[1]) | _regs(ops[2]))
                if dst != addend:
                    touched |= dst | addend
                elif any(r in state for r in dst):
                    # in flight: right only if it is one product's whole result
                    if len({state[r][1] for r in dst if r in state}) > 1:
                        touched |= dst
            elif not op.startswith("s_") or "v" in "".join(ops):
                for o in ops:
                    touched |= _regs(o)
            for r in touched & state.keys():
                missing, at = state[r]
                key = (line, at)
                found[key] = max(found.get(key, 0), missing)
            passed = 1
            if op == "s_nop":
                passed = int(ops[0], 0) + 1
            state = {r: (v[0] - passed, v[1]) for r, v in state.items() if v[0] > passed}
            if ours(op, ops):
                for r in _regs(ops[0]):
                    state[r] = (wait, line)
            if op in ("s_endpgm", "s_setpc_b64"):
                break
            if op == "s_branch":
                work.append((at_label[ops[0]], state))
                break
            if op.startswith("s_cbranch"):
                work.append((at_label[ops[0]], dict(state)))
            i += 1
    return sorted((use, at, wait - missing) for (use, at), missing in found.items())


def scalar_offset_accesses(body):
    """(buffer accesses, lines of those whose scalar offset is not 0) of one function."""
    n, lines = 0, []
    for line, _, op, ops in body:
        if op is None or not re.match(r"buffer_(load|store|atomic)", op):
            continue
        n += 1
        if ops[-1].split()[0] not in ("0", "null"):
            lines.append(line)
    return n, lines


def kernel_resources(text):
    """{kernel: {field: value}} of the numeric fields in a listing's kernel metadata."""
    out = {}
    for block in text.split("  - .agpr_count:")[1:]:
        fields = dict(re.findall(r"\.(\w+):\s+(\S+)", block.split("amdhsa.target")[0]))
        out[fields["name"]] = {k: int(v) for k, v in fields.items() if v.isdigit()}
    return out
