"""No instruction touches the registers of a transposing LDS read before the wave has waited for it.

Kernels issue such reads where the compiler does not track them, and wait for them by hand; a register that is free to the
compiler while a read into it is on its way (the last prefetch of a loop that nothing takes) is overwritten when the
read lands.  This follows every path through the machine code of the built library: a read is pending until an
s_waitcnt lgkmcnt(n) with at least n later LDS operations (a wave's LDS operations complete in order).  Branches on a
register pair that holds 0 or -1 on the path (a loop's exit flag) are followed as they go.  Host only."""
import glob
import os
import re
import subprocess

import pytest

from paper_1808_05567_amd import conv

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
VREG = re.compile(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b")
PAIR = re.compile(r"s\[\d+:\d+\]|vcc")
FLAG = re.compile(r"(s_and_b64|s_andn2_b64) vcc, exec, (s\[\d+:\d+\])$")


def _vregs(text):
    out = set()
    for a, b, c in VREG.findall(text):
        out.update([int(c)] if c else range(int(a), int(b) + 1))
    return frozenset(out)


def _functions(path):
    """(name, [(address, text, branch target or None)]) of the kernels with transposing reads."""
    p = subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", path], stdout=subprocess.PIPE, text=True)
    name, base, code, wanted = None, 0, [], False
    for line in p.stdout:
        if line[0] == "\t":
            text, _, rest = line.partition("//")
            at, _, where = rest.partition(":")
            if not where:  # (padding)
                continue
            text = text.strip()
            wanted = wanted or text.startswith("ds_read_b64_tr")
            target = None
            if text.startswith(("s_cbranch", "s_branch")):
                m = re.search(r"\+0x([0-9a-f]+)>", where)
                target = base + (int(m[1], 16) if m else 0)
            code.append((int(at, 16), text, target))
        elif line.startswith("0"):
            if wanted:
                yield name, code
            name, base, code, wanted = line.split("<")[1].split(">")[0], int(line[:16], 16), [], False
    if wanted:
        yield name, code
    assert p.wait() == 0


def _hazards(code):
    """(address, text, address of the read) of the instructions that touch a pending read's registers."""
    index = {at: i for i, (at, _, _) in enumerate(code)}
    leaders = {0} | {index[t] for _, _, t in code if t is not None} | \
        {i + 1 for i, (_, text, _) in enumerate(code) if text.startswith(("s_cbranch", "s_branch", "s_endpgm"))}
    flags = {m[2] for _, text, _ in code for m in [FLAG.match(text)] if m}
    dst, found = {}, {}

    def run(i, known, pending):
        """To the end of the block: its successors, what is known of the flags and what is pending there."""
        known, pending = dict(known), dict(pending)
        while True:
            at, text, target = code[i]
            op, _, args = text.partition(" ")
            if op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", args)
                if m:
                    pending = {r: n for r, n in pending.items() if n < int(m[1])}
                elif args.strip() == "0":
                    pending = {}
            elif op in ("s_cbranch_vccnz", "s_cbranch_vccz"):
                taken = known.get("vcc")
                nxt = [(target, True), (None, False)]
                if taken is not None:
                    nxt = nxt[:1] if taken == (op == "s_cbranch_vccnz") else nxt[1:]
                return [index[t] if j else i + 1 for t, j in nxt], known, pending
            elif op.startswith("s_cbranch"):
                return [index[target], i + 1], known, pending
            elif op == "s_branch":
                return [index[target]], known, pending
            elif op == "s_endpgm":
                return [], known, pending
            else:
                if pending:
                    mine = _vregs(args)
                    for r in pending:
                        if mine & dst[r]:
                            found[at, r] = text
                m = FLAG.match(text)
                if m and m[2] in known:
                    known["vcc"] = known[m[2]] != (m[1] == "s_andn2_b64")
                else:
                    for name in {p for p in PAIR.findall(args.partition(",")[0])} | ({"vcc"} if "vcc" in args else set()):
                        known.pop(name, None)
                    single = re.match(r"s(\d+)\b", args)
                    if single:
                        n = int(single[1])
                        known.pop("s[%d:%d]" % (n & ~1, n | 1), None)
                    wide = re.match(r"s\[(\d+):(\d+)\]", args)
                    if wide:
                        for n in range(int(wide[1]) & ~1, int(wide[2]) + 1, 2):
                            known.pop("s[%d:%d]" % (n, n + 1), None)
                    m = re.match(r"s_mov_b64 (s\[\d+:\d+\]), (0|-1)$", text)
                    if m and m[1] in flags:
                        known[m[1]] = m[2] == "-1"
                if op.startswith("ds_"):
                    pending = {r: min(n + 1, 16) for r, n in pending.items()}
                    if op.startswith("ds_read_b64_tr"):
                        dst[at] = _vregs(args.partition(",")[0])
                        pending[at] = 0
            i += 1
            if i in leaders:
                return [i], known, pending

    seen, work = {}, [(0, frozenset(), {})]
    while work:
        i, known, pending = work.pop()
        have = seen.get((i, known))
        if have is not None:
            if all(r in have and have[r] <= n for r, n in pending.items()):
                continue
            pending = {r: min(have.get(r, 16), pending.get(r, 16)) for r in have.keys() | pending.keys()}
        seen[i, known] = pending
        nxt, k, p = run(i, known, pending)
        work += [(j, frozenset(k.items()), p) for j in nxt]
    return [(hex(at), text, hex(r)) for (at, r), text in sorted(found.items())]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_registers_of_lds_reads_on_their_way_are_left_alone(tmp_path):
    lib = tmp_path / "lib.so"
    os.symlink(conv.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, stdout=subprocess.DEVNULL, cwd=tmp_path)
    kernels = 0
    bad = {}
    for path in sorted(glob.glob(str(tmp_path / "*gfx950"))):
        for name, code in _functions(path):
            kernels += 1
            found = _hazards(code)
            if found:
                bad[name] = (len(found), found[:3])
    assert kernels > 100, kernels
    assert not bad, "\n".join("%s: %s" % kv for kv in bad.items())
