"""Build-time check of generated code (gfx950 assembly text) of the kernels that issue loads by hand.

csrc/decode_mfma.hip (global loads and LDS reads) and csrc/compressv.hip (LDS reads) issue some loads
by hand: the request and the hand-over of the destination registers to the compiler are separate
inline-assembly statements, with the wait between them.  In
between, the compiler believes that the destination already holds its value.  If it moves that value
(a copy into another register, a spill into the accumulation file or to scratch memory), it copies
stale contents, hands the register to something else, and the data then arrives on top of that --
wrong numbers at best, a wild address at worst.  Nothing in the language forbids such a move, so the
build reads what the compiler produced and refuses it unless, in every kernel,

  * every destination of a hand-issued `global_load_dwordx4 ... ; by hand` is handed over
    (`; by hand <registers>`) under the same name, and no instruction between the request and the
    hand-over names any of its registers;
  * no instruction between a hand-issued `ds_read_b128` (inside an inline-assembly block) and the
    next `s_waitcnt` with `lgkmcnt(0)` names a destination of such a read;
  * no scratch-memory instruction lies between a request and its hand-over;
  * the fetches from global memory into LDS are all past the caches (`nt`) or none is: which of the two a launch
    wants is a matter of the instance it calls, so that no kernel carries the code of both.

The projection kernel of csrc/compressv.hip also counts its fetches into LDS: a wait for all but the last
N of them is a wait for a tile only if the requests went out in the order that the source gives, and
to the compiler the staging buffers are unrelated memory.  verify_fetch_order reads the requests
ahead of the kernel's first wait for them.

The check follows the text in order, as the requests and hand-overs are written in straight-line code
(a wait may sit inside a branch, never a request or a hand-over); from reads at the end of a loop body
it follows the path that leaves the loop, not the back edge."""
import re
import sys

_REG = re.compile(r"\b([av])\[(\d+):(\d+)\]|\b([av])(\d+)\b")


def _regs(text):
    out = set()
    for m in _REG.finditer(text):
        if m.group(1):
            out.update((m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1))
        else:
            out.add((m.group(4), int(m.group(5))))
    return out


def _code(line):
    c = line.split(";")[0].strip()
    if not c or c.startswith(".") or c.endswith(":"):
        return ""
    return c


def check_kernel(name, lines):
    """Problems found in one kernel's lines, as strings."""
    problems = []
    pending = {}   # line number of a global request -> its destination registers
    lds_pending = {}
    in_asm = False
    n_requests = n_lds = 0
    forms = set()  # of the fetches into LDS
    for no, line in lines:
        if "#ASMSTART" in line:
            in_asm = True
            continue
        if "#ASMEND" in line:
            in_asm = False
            continue
        if "global_load_dwordx4" in line and "by hand" in line:
            m = re.search(r"global_load_dwordx4\s+(\S+?),", line)
            dst = _regs(m.group(1))
            for at, regs in pending.items():
                if regs & dst:
                    problems.append("%s: line %d requests into registers still awaited from line %d" % (name, no, at))
            pending[no] = dst
            n_requests += 1
            continue
        if "; by hand" in line and "global_load" not in line:
            m = re.search(r"; by hand\s+(\S+)", line)
            got = _regs(m.group(1)) if m else set()
            hit = [at for at, regs in pending.items() if regs == got]
            if not hit:
                problems.append("%s: line %d hands over %s, which no request names" % (name, no, m.group(1) if m else "?"))
            for at in hit:
                del pending[at]
            continue
        code = _code(line)
        if not code:
            continue
        if in_asm and code.startswith("ds_read_b128"):
            m = re.match(r"ds_read_b128\s+(\S+?),", code)
            lds_pending[no] = _regs(m.group(1))
            n_lds += 1
            continue
        if code.startswith("s_waitcnt") and "lgkmcnt(0)" in code:
            lds_pending.clear()  # (whoever issued it: nothing read from LDS is still on its way)
            continue
        if code.startswith("global_load_lds"):
            forms.add("nt" in code.split())
        named = _regs(code)
        if pending:
            if code.startswith("scratch_"):
                problems.append("%s: line %d: scratch access while hand-issued loads are awaited" % (name, no))
            for at, regs in pending.items():
                if regs & named:
                    problems.append("%s: line %d `%s` names a register awaited from line %d" % (name, no, code, at))
        for at, regs in lds_pending.items():
            if regs & named:
                problems.append("%s: line %d `%s` names a register of the LDS read at line %d" % (name, no, code, at))
        if code.startswith("s_endpgm") and (pending or lds_pending):
            problems.append("%s: requests never handed over: lines %s" % (name, sorted(pending) + sorted(lds_pending)))
    if len(forms) > 1:
        problems.append("%s: fetches into LDS both past the caches and not" % name)
    return problems, n_requests, n_lds


def check_text(text, kernel="decode_split_mfma_kernel"):
    """(problems, kernels checked, hand-issued global requests, hand-issued LDS reads) of an assembly file;
    the kernels are the functions whose mangled name contains `kernel`."""
    lines = text.split("\n")
    starts = [i for i, l in enumerate(lines) if re.match(r"_Z\S*" + re.escape(kernel) + r"\S*:\s*", l)]
    problems, kernels, total, total_lds = [], 0, 0, 0
    for k, a in enumerate(starts):
        b = len(lines)
        for j in range(a + 1, len(lines)):
            if lines[j].startswith(".Lfunc_end"):
                b = j
                break
        name = lines[a].split(":")[0]
        p, n, nl = check_kernel(name, [(i + 1, lines[i]) for i in range(a, b)])
        problems += p
        kernels += 1
        total += n
        total_lds += nl
    return problems, kernels, total, total_lds


_GEMM = re.compile(r"_Z\S*compressv_gemm_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E\S*:\s*")


def fetch_order(heads, tokens, waves, sa, sb):
    """The first requests of a wave of the projection kernel, as (byte of the staging buffers, pieces of 1 KiB): W_V of
    stage s + sb, then X of stage s + sa, for s = -sa .. -1."""
    a, b = tokens * 128, heads * 128 * 128
    out = []
    for s in range(-sa, 0):
        if s + sb >= 0:
            out.append((sa * a + (s + sb) * b, b // 1024 // waves))
        out.append(((s + sa) * a, a // 1024 // waves))
    return out


def check_fetch_order(text):
    """(problems, kernels checked) of an assembly file: do the projection kernels request their first stages in
    the order that their waits count on?"""
    lines = text.split("\n")
    problems, kernels = [], 0
    for start, line in enumerate(lines):
        m = _GEMM.match(line)
        if not m:
            continue
        kernels += 1
        _, heads, _, _, wt, mw, sa, sb = (int(x) for x in m.groups())
        name, got, m0 = line.split(":")[0], [], None
        for no in range(start + 1, len(lines)):
            code = _code(lines[no])
            if lines[no].startswith(".Lfunc_end") or code.startswith("s_barrier"):
                break
            if re.match(r"s_\S+\s+m0,", code):
                # the wave's own place in a tile is in the register, the buffer's in the literal
                at = re.match(r"s_(?:mov_b32|add_i32|add_u32)\s+m0, (s\d+)(?:, (0x[0-9a-f]+|\d+))?$", code)
                m0 = int(at.group(2) or "0", 0) if at else None
            elif code.startswith("global_load_lds_dwordx4"):
                if m0 is None:
                    problems.append("%s: line %d: where a fetch goes is not known" % (name, no + 1))
                got.append(m0)
        want = [at + 1024 * i for at, n in fetch_order(heads, wt * mw, mw * heads, sa, sb) for i in range(n)]
        if got != want:
            problems.append("%s: the first fetches go to %s, the waits count on %s" % (name, got, want))
    return problems, kernels


def verify_fetch_order(path):
    """Raises RuntimeError unless every projection kernel in the assembly file at `path` keeps its order."""
    with open(path) as f:
        problems, kernels = check_fetch_order(f.read())
    if kernels == 0:
        raise RuntimeError("%s: no projection kernel found: nothing was checked" % path)
    if problems:
        raise RuntimeError("order of fetches: %d problem(s) in %s\n%s" % (len(problems), path, "\n".join(problems[:20])))
    return kernels


def verify(path, kernel="decode_split_mfma_kernel", global_loads=True):
    """Raises RuntimeError if the assembly file at `path` breaks a rule above.  global_loads: the kernels
    are expected to hold hand-issued global loads (LDS reads are expected always)."""
    with open(path) as f:
        problems, kernels, total, total_lds = check_text(f.read(), kernel)
    if kernels == 0:
        raise RuntimeError("%s: no %s found: nothing was checked" % (path, kernel))
    if (global_loads and total == 0) or total_lds == 0:
        raise RuntimeError("%s: no hand-issued loads found in %d kernels: the check no longer sees them" % (path, kernels))
    if problems:
        raise RuntimeError("hand-issued loads: %d problem(s) in %s\n%s" % (len(problems), path, "\n".join(problems[:20])))
    return kernels, total, total_lds


if __name__ == "__main__":
    k, n, nl = verify(sys.argv[1], *(sys.argv[2:3] or ["decode_split_mfma_kernel"]), global_loads=len(sys.argv) < 3)
    print("%d kernels, %d hand-issued global loads, %d hand-issued LDS reads: registers untouched until handed over" % (k, n, nl))
