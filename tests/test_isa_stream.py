"""CPU-only check of the load pipeline of the matrix-core value pass.

Its waves load straight to LDS and wait by count: "at most n loads outstanding" in front of a piece's use has to mean
that the piece has arrived.  The test compiles the kernels with the library's flags, follows the control flow of every
stream's start and every tile body for their waits and loads, checks that nothing else goes to memory in between (it would
shift the counts), and replays the loads of waves of one to twenty tiles, in the order found and with the waits found."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2506_13059_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2506_13059_amd", "csrc", "mp_stream.hip")


def _kernels(asm):
    """(heads, waves, blocks, order) of every kernel: blocks maps a label to its tokens and successors."""
    i = 0
    while i < len(asm):
        m = re.match(r"^_ZN2mp\S*value_stream_kernelILi(\d+)ELi(\d+)E\S*:", asm[i])
        i += 1
        if not m:
            continue
        blocks, label, toks, succ, in_asm, n = {}, "entry", [], [], False, 0
        while not asm[i].startswith(".Lfunc_end"):
            ln = asm[i].strip()
            i += 1
            in_asm = ln.startswith(";;#ASMSTART") or (in_asm and not ln.startswith(";;#ASMEND"))
            t = None
            if re.match(r"^\.LBB\w+:", ln):
                nxt = ln.split(":")[0]
                blocks[label] = (toks, succ + [nxt])
                label, toks, succ = nxt, [], []
            elif re.match(r"s_c?branch", ln) or ln.startswith("s_endpgm"):
                n += 1
                to = [] if ln.startswith("s_endpgm") else [ln.split()[-1]]
                if ln.startswith("s_cbranch"):
                    to.append(f"after{n}")
                blocks[label] = (toks, succ + to)
                label, toks, succ = f"after{n}", [], []
            elif ln.startswith("global_load_lds_dwordx4"):
                t = "L16"
            elif ln.startswith("global_load_lds_dword"):
                t = "L4"
            elif re.match(r"(global|buffer|scratch|flat)_", ln):
                t = "G"
            elif in_asm and re.match(r"s_waitcnt vmcnt\(\d+\)", ln):
                t = "W" + re.search(r"vmcnt\((\d+)\)", ln).group(1)
            elif in_asm and ln.startswith("ds_read_b128"):
                t = "K"
            elif ln.startswith("ds_read_b64_tr"):
                t = "T"
            if t:
                toks.append(t)
        blocks[label] = (toks, succ)
        yield int(m.group(1)), int(m.group(2)), blocks


def _paths(blocks, label, at, stop):
    """Token sequences from a place up to and including the first token that `stop` accepts (or the end)."""
    out, todo, visited = set(), [(label, at, ())], set()
    while todo:
        label, at, seen = todo.pop()
        toks, succ = blocks[label]
        for k in range(at, len(toks)):
            seen += (toks[k],)
            if stop(toks[k]):
                out.add(seen)
                break
        else:
            if not succ:
                out.add(seen)
            for s in succ:
                if (s, seen) not in visited:
                    visited.add((s, seen))
                    todo.append((s, 0, seen))
    return out


def _bodies(blocks):
    """{(has key rows, wait before them, loads before the value wait, value wait)}, and the loads behind the values"""
    found = set()
    for label, (toks, _) in blocks.items():
        for k, t in enumerate(toks):
            if not t.startswith("W"):
                continue
            ahead = _paths(blocks, label, k + 1, lambda x: x.startswith("W") or x == "T")
            if not any(p[-1:] and p[-1].startswith("W") for p in ahead) or t == "W0":
                continue        # a value wait, or the wait for the first row numbers
            for p in ahead:
                assert p and p[-1].startswith("W") and "G" not in p, p
                keys, loads, value_wait = "K" in p, [x for x in p if x[0] == "L"], int(p[-1][1:])
                assert p.count("K") in (0, 4)
                found.add((keys, int(t[1:]), tuple(loads), value_wait))
    after = set()
    for label, (toks, _) in blocks.items():
        for k, t in enumerate(toks):
            if t == "T" and toks[k:k + 8] == ["T"] * 8 and (k == 0 or toks[k - 1] != "T"):
                for p in _paths(blocks, label, k + 8, lambda x: x.startswith("W") or x == "G"):
                    after.add(tuple(x for x in p if x[0] == "L"))
    return found, after


def _start(n_tiles, key_loads, listed, guest):
    """Loads of a wave from the wait for its first row numbers to its first tile: (what, token, count)."""
    kind = "L4" if listed == "scored" else "L16"
    out = [(("strip", 1), "L4", 1)] if listed and n_tiles > 4 else []
    for t in range(min(2, n_tiles)):
        out += [(("K", t), kind, key_loads), (("V", t), "L16", 4)]
        if t == 0 and guest:
            out.append((("guest",), "L4", 1))       # (the first row numbers of the source that rides along)
    return out


def _starts(key_loads, listed, guest):
    return frozenset(tuple(tok for _, tok, count in _start(n, key_loads, listed, g) for _ in range(count))
                     for n in (1, 2, 5) for g in {False, guest}) | frozenset(
                         # (no stream of one tile has a second strip, but the code's two branches do not know that)
                         ("L4",) + tuple(tok for _, tok, count in _start(1, key_loads, listed, g) for _ in range(count))
                         for g in {False, guest} if listed)


def _compiled_starts(blocks, token):
    """The load sequences behind each `token` up to the first counted wait: a set for each place that has any."""
    found = set()
    for label, (toks, _) in blocks.items():
        for k, t in enumerate(toks):
            if t == token:
                paths = _paths(blocks, label, k + 1, lambda x: x[0] == "W" or x in ("G", "T"))
                starts = [p.count("L16") >= 4 and p[-1][0] == "W" for p in paths]
                assert token != "W0" or all(starts) or not any(starts), paths
                if all(starts):
                    found.add(frozenset(p[:-1] for p in paths))
    return found


def _replay(n_tiles, key_loads, waits, listed, guest):
    """Loads of a wave in the kernel's order; `waits[ahead]` = (before the keys' use, before the values' use)."""
    pending = []

    def load(what, count):
        pending.extend([what] * count)

    def wait(n):
        del pending[:max(0, len(pending) - n)]

    slot = {0: 0}

    def rows(t):                         # the row numbers of a tile are read: their strip is in its slot, whole
        if listed:
            assert slot[t // 4 & 1] == t // 4 and ("strip", t // 4) not in pending, (n_tiles, t)

    if listed:
        load(("strip", 0), 1)            # (asked for before the wave knew how many rows it has)
        wait(0)
    for what, _, count in _start(n_tiles, key_loads, listed, guest):
        if what[0] == "K":
            rows(what[1])
        if what[0] == "strip":
            slot[1] = 1
        load(what, count)
    for t in range(n_tiles):
        ahead = min(2, n_tiles - 1 - t)
        wait(waits[ahead][0])
        assert ("K", t) not in pending, (n_tiles, t)
        if ahead == 2:
            rows(t + 2)
            load(("K", t + 2), key_loads)
        wait(waits[ahead][1])
        assert ("V", t) not in pending, (n_tiles, t)
        if ahead == 2:
            load(("V", t + 2), 4)
            if listed and t % 4 == 1 and (t // 4 + 2) * 4 < n_tiles:
                load(("strip", t // 4 + 2), 1)
                slot[t // 4 & 1] = t // 4 + 2
    assert not pending, n_tiles          # nothing lands in LDS that the next use of it does not know of


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_every_piece_has_arrived_before_its_use(tmp_path):
    asm = tmp_path / "mp_stream.s"
    subprocess.check_call(["hipcc", *build.FLAGS, *build.EXTRA_FLAGS.get(os.path.basename(SRC), []), "-S", "--cuda-device-only",
                           "-o", str(asm), SRC], stderr=subprocess.DEVNULL)
    checked = 0
    for heads, waves, blocks in _kernels(asm.read_text().splitlines()):
        found, after = _bodies(blocks)
        for keys, key_loads, kind in ((True, 4, "L16"), (False, (16 * heads + 63) // 64, "L4")):
            bodies = {b[1:] for b in found if b[0] == keys}
            main = [b for b in bodies if b[1] == (kind,) * key_loads]
            rest = sorted((b for b in bodies if not b[1]), reverse=True)
            assert len(main) == 1 and len(rest) == 2 and len(bodies) == 3, (heads, waves, bodies)
            waits = {2: (main[0][0], main[0][2]), 1: (rest[0][0], rest[0][2]), 0: (rest[1][0], rest[1][2])}
            for n in range(1, 21):
                for listed in (True, False) if keys else ("scored",):
                    for guest in (False, True):
                        _replay(n, key_loads, waits, listed, guest)
        # every stream starts in the order of the replay: the centroid terms' (as a source of its own, and behind another
        # source's rows), the listed rows' and the plain rows', which have no row numbers to wait for
        scored = (16 * heads + 63) // 64
        assert _compiled_starts(blocks, "W0") == {_starts(scored, "scored", True), _starts(scored, "scored", False),
                                                  _starts(4, True, True)}, (heads, waves)
        assert _starts(4, False, True) in _compiled_starts(blocks, "G"), (heads, waves)
        # behind the values: the next tile's, and perhaps row numbers, in the main loop; nothing at the last two tiles
        # but the first row numbers of the stream that follows
        assert after <= {("L16",) * 4, ("L16",) * 4 + ("L4",), (), ("L4",), ("L4", "L4")}, (heads, waves, after)
        checked += 1
    assert checked == 8
