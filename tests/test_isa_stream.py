"""CPU-only check of the load pipeline of the matrix-core value pass.

Its waves load straight to LDS and wait by count: "at most n loads outstanding" in front of a piece's use has to mean
that the piece has arrived.  The test compiles the kernels, follows the control flow of every tile body for its waits
and loads, checks that nothing else goes to memory in between (it would shift the counts), and replays the loads of
waves of one to twenty tiles with the waits found."""
import os
import re
import shutil
import subprocess

import pytest

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


def _replay(n_tiles, key_loads, waits, listed):
    """Loads of a wave in the kernel's order; `waits[ahead]` = (before the keys' use, before the values' use)."""
    pending = []

    def load(what, count):
        pending.extend([what] * count)

    def wait(n):
        del pending[:max(0, len(pending) - n)]

    strips = set()
    if listed:
        strips = {0} | ({1} if n_tiles > 4 else set())       # (waited for before the first rows)
    for t in range(min(2, n_tiles)):
        load(("K", t), key_loads)
        load(("V", t), 4)
    for t in range(n_tiles):
        ahead = min(2, n_tiles - 1 - t)
        wait(waits[ahead][0])
        assert ("K", t) not in pending, (n_tiles, t)
        if ahead == 2:
            if listed:
                assert (t + 2) // 4 in strips and ("strip", (t + 2) // 4) not in pending, (n_tiles, t)
            load(("K", t + 2), key_loads)
        wait(waits[ahead][1])
        assert ("V", t) not in pending, (n_tiles, t)
        if ahead == 2:
            load(("V", t + 2), 4)
            if listed and t % 4 == 1 and (t // 4 + 2) * 4 < n_tiles:
                load(("strip", t // 4 + 2), 1)
                strips.add(t // 4 + 2)
    assert not pending, n_tiles          # nothing lands in LDS that the next use of it does not know of


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_every_piece_has_arrived_before_its_use(tmp_path):
    asm = tmp_path / "mp_stream.s"
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                           "-packed-fp32-ops", "-S", "--cuda-device-only", "-o", str(asm), SRC], stderr=subprocess.DEVNULL)
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
                for listed in (True, False):
                    _replay(n, key_loads, waits, listed)
        # behind the values: the next tile's, and perhaps row numbers, in the main loop; nothing at the last two tiles
        # but the first row numbers of the stream that follows
        assert after <= {("L16",) * 4, ("L16",) * 4 + ("L4",), (), ("L4",), ("L4", "L4")}, (heads, waves, after)
        checked += 1
    assert checked == 16
