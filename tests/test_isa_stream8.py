"""CPU-only check of the load pipeline of the matrix-core value pass over 8-bit rows: the stream's start and tile bodies, compiled
with the library's flags, have the loads and counted waits that the replay below assumes, in its order, and in the replay of
waves of one to 40 tiles every piece has arrived before its use and every strip of row numbers is there, whole, while it is
read."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2506_13059_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2506_13059_amd", "csrc", "mp_stream8.hip")
KEY_LOADS, VALUE_LOADS = 6, 4           # code rows, logit shares and scales; code rows


def _tokens(lines):
    """Loads to LDS (x: 16 bytes, y: 4), hand-written waits (number), reads of keys (k: 8 eight-byte reads) and values (t)."""
    toks, in_asm = [], False
    for ln in (x.strip() for x in lines):
        in_asm = ln.startswith(";;#ASMSTART") or (in_asm and not ln.startswith(";;#ASMEND"))
        if ln.startswith("global_load_lds_dwordx4"):
            toks.append("x")
        elif ln.startswith("global_load_lds_dword"):
            toks.append("y")
        elif in_asm and re.match(r"s_waitcnt vmcnt\(\d+\)", ln):
            toks.append(int(re.search(r"\((\d+)\)", ln).group(1)))
        elif in_asm and ln.startswith("ds_read_b64_tr_b8"):
            toks.append("t")
        elif in_asm and re.match(r"ds_read_b64 ", ln):
            toks.append("k")
        elif re.match(r"(global|buffer|scratch|flat)_", ln):
            toks.append("G")
    return toks


def _bodies(toks):
    """(wait before the keys, loads up to the wait before the values, that wait) of each tile body: 8 key reads behind a wait."""
    out = set()
    for i, t in enumerate(toks):
        if isinstance(t, int) and toks[i + 1:i + 9] == ["k"] * 8:
            j = i + 9
            loads = []
            while not isinstance(toks[j], int):
                assert toks[j] in "xy", (i, toks[i:j + 1])        # (nothing else goes to memory in between)
                loads.append(toks[j])
                j += 1
            assert toks[j + 1:j + 9] == ["t"] * 8, toks[j:j + 10]
            out.add((t, "".join(loads), toks[j]))
    return out


def _start(n, guest):
    """Loads of a wave from the wait for its first row numbers to its first tile: (what, tokens)."""
    out = [(("rows", 1), "yy")] if n > 2 else []
    for t in range(min(2, n)):
        out += [(("K", t), "xxxxxy"), (("V", t), "xxxx")]
        if t == 0 and guest:
            out.append((("guest",), "y"))           # (the first row numbers of the source that rides along)
    if n > 4:
        out.append((("rows", 2), "yy"))
    return out


def _check_starts(lines):
    """The loads that the listing has between the wait for the first row numbers and the first tile are _start's."""
    toks = _tokens(lines)
    at = [i for i, t in enumerate(toks) if t == 0 and "".join(map(str, toks[i + 1:i + 9])).startswith("yyxxxxxy")]
    assert len(at) == 1, at
    found = toks[at[0] + 1:]
    found = "".join(map(str, found[:next(i for i, t in enumerate(found) if isinstance(t, int))]))
    # (in one piece: the branches skip what a wave does not need)
    assert found == "".join(tok for _, tok in _start(5, True)), found


def _replay(n, waits, guest):
    pending, slot = [], {}

    def load(what, count):
        pending.extend([what] * count)

    def strip(s):
        slot[s & 1] = s
        load(("rows", s), 2)

    def rows(t):
        assert slot[(t >> 1) & 1] == t >> 1 and ("rows", t >> 1) not in pending, (n, t)

    def wait(k):
        del pending[:max(0, len(pending) - k)]

    strip(0)                             # (asked for before the wave knew how many rows it has)
    wait(0)
    for what, toks in _start(n, guest):
        if what[0] == "K":
            rows(what[1])
        if what[0] == "rows":
            slot[what[1] & 1] = what[1]
        load(what, len(toks))
    for t in range(n):
        ahead = min(2, n - 1 - t)
        wait(waits[ahead][0])
        assert ("K", t) not in pending, (n, t)
        if ahead == 2:
            rows(t + 2)
            load(("K", t + 2), KEY_LOADS)
        wait(waits[ahead][1])
        assert ("V", t) not in pending, (n, t)
        if ahead == 2:
            load(("V", t + 2), VALUE_LOADS)
            if t & 1 and ((t >> 1) + 3) * 2 < n:
                strip((t >> 1) + 3)
    assert not pending, n


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_every_piece_has_arrived_before_its_use(tmp_path):
    asm = tmp_path / "mp_stream8.s"
    subprocess.check_call(["hipcc", *build.FLAGS, *build.EXTRA_FLAGS.get(os.path.basename(SRC), []), "-S", "--cuda-device-only",
                           "-o", str(asm), SRC], stderr=subprocess.DEVNULL)
    lines = asm.read_text().splitlines()
    starts = [i for i, x in enumerate(lines) if re.match(r"^_ZN2mp\S*value_stream8_kernelILi\d+E\S*:", x)]
    assert len(starts) == 7
    for i in starts:
        end = next(j for j in range(i, len(lines)) if lines[j].startswith(".Lfunc_end"))
        bodies = _bodies(_tokens(lines[i:end]))
        main = [b for b in bodies if b[1]]
        last = sorted((b for b in bodies if not b[1]), reverse=True)
        assert len(main) == 1 and main[0][1] == "xxxxxy" and len(last) == 2, bodies
        waits = {2: (main[0][0], main[0][2]), 1: (last[0][0], last[0][2]), 0: (last[1][0], last[1][2])}
        _check_starts(lines[i:end])
        for n in range(1, 41):
            for guest in (False, True):
                _replay(n, waits, guest)
