"""What the generated gfx950 assembly must not contain.

Packed-FP32 arithmetic, and instructions that follow the write of an operand more closely than the hardware allows: the
compiler keeps these distances between its own instructions but does not look into inline assembly, on either side.
``check(text)`` takes the assembly as the compiler prints it and returns a list of findings.

Wait states (one per instruction, n + 1 for ``s_nop n``) that have to lie between a vector instruction's write and
    a DPP instruction's read of its permuted operand                              2
    a lane swap (v_permlane16_swap, v_permlane32_swap) of either operand          2
    a matrix instruction's read                                                   2
    v_readlane / v_readfirstlane                                                  1
and, for a transcendental one, any other vector instruction's read                1.
(Results of matrix instructions are not looked at: inline assembly takes none.)
"""
import functools
import re

PACKED_FP32_OPS = ("v_pk_fma_f32", "v_pk_mul_f32", "v_pk_add_f32")
_TRANSCENDENTAL = ("v_exp_", "v_log_", "v_rcp_", "v_rsq_", "v_sqrt_", "v_sin_", "v_cos_")
_TWO_RESULTS = ("v_permlane16_swap", "v_permlane32_swap", "v_swap", "v_add_co_", "v_addc_co_", "v_sub_co_", "v_subb_co_",
                "v_subrev_co_", "v_subbrev_co_", "v_mad_u64_u32", "v_mad_i64_i32", "v_div_scale_")
_NO_WAY_ON = ("s_branch", "s_endpgm", "s_setpc_b64")
_REGISTER = re.compile(r"\bv(\d+)\b|\bv\[(\d+):(\d+)\]")


@functools.lru_cache(maxsize=None)
def _registers(operands):
    """Vector registers named in an operand list."""
    out = set()
    for m in _REGISTER.finditer(operands):
        first, last = (m.group(1), m.group(1)) if m.group(1) else (m.group(2), m.group(3))
        out.update(range(int(first), int(last) + 1))
    return frozenset(out)


class _Instruction:
    __slots__ = ("line", "text", "op", "valu", "waits", "written", "target")

    def __init__(self, line, text):
        self.line, self.text = line, text
        self.op = text.split(None, 1)[0]
        self.valu = self.op.startswith("v_") and not self.op.startswith(("v_mfma", "v_nop"))
        self.waits = int(text.split()[1], 0) + 1 if self.op == "s_nop" else 1
        self.target = text.split()[-1] if self.op.startswith(("s_branch", "s_cbranch")) else None
        self.written = _registers(self._split()[0]) if self.valu else frozenset()

    def _split(self):
        """Results and sources."""
        parts = self.text[len(self.op):].split(",")
        n = 2 if self.op.startswith(_TWO_RESULTS) else 1
        return ",".join(parts[:n]), ",".join(parts[n:])

    def reads(self):
        """(registers, wait states, whether only behind transcendental instructions) of each rule that applies."""
        if not self.op.startswith("v_"):
            return
        results, sources = self._split()
        if self.op.startswith(("v_permlane16_swap", "v_permlane32_swap")):
            yield _registers(results), 2, False
        elif self.op.startswith("v_mfma"):
            yield _registers(sources), 2, False
        elif self.op.startswith(("v_readlane", "v_readfirstlane")):
            yield _registers(sources), 1, False
        elif "_dpp" in self.op:
            yield _registers(sources.split(",")[0]), 2, False
        if self.valu and not self.op.startswith(_TRANSCENDENTAL):
            yield _registers(sources) | (_registers(results) if "fmac" in self.op else frozenset()), 1, True


def _functions(text):
    """Bodies as lists of instructions and label names."""
    body, bodies = None, []
    for n, line in enumerate(text.splitlines(), 1):
        if line[:1] not in ("\t", " "):
            name = re.match(r"([\w$.]+):", line)
            if name and name.group(1).startswith(".L"):
                if body is not None:
                    body.append(name.group(1))
            elif name:
                body = []
                bodies.append((name.group(1), body))
            continue
        code = line.split(";", 1)[0].strip()
        if code and not code.startswith((".", "//")) and body is not None:
            body.append(_Instruction(n, code))
    return bodies


def _before(body, branches, at, waits):
    """Instructions with fewer than ``waits`` wait states between them and the one at ``at``, along every way to it."""
    pending, seen = [(at - 1, 0)], set()
    while pending:
        k, w = pending.pop()
        while k >= 0 and w < waits and (k, w) not in seen:
            seen.add((k, w))
            x = body[k]
            if isinstance(x, str):   # reached by jumps, and from above unless that jumps away
                pending.extend((b, w) for b in branches.get(x, ()))
                if k > 0 and not isinstance(body[k - 1], str) and body[k - 1].op in _NO_WAY_ON:
                    break
            else:
                yield x
                w += x.waits
            k -= 1


def check(text):
    """Findings, as lines of text."""
    found = ["%s used" % op for op in PACKED_FP32_OPS if op in text]
    for name, body in _functions(text):
        branches = {}
        for k, x in enumerate(body):
            if not isinstance(x, str) and x.target:
                branches.setdefault(x.target, []).append(k)
        for k, x in enumerate(body):
            if isinstance(x, str):
                continue
            for read, waits, only_transcendental in x.reads():
                for p in _before(body, branches, k, waits):
                    if p.written & read and (not only_transcendental or p.op.startswith(_TRANSCENDENTAL)):
                        found.append("%s, line %d: '%s' needs %d wait states behind '%s' (line %d)"
                                     % (name, x.line, x.text, waits, p.text, p.line))
                        break
    return found
