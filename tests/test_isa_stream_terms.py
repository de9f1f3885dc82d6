"""CPU-only check of the load pipeline of the value pass whose centroid terms have a wave of their own: the tile bodies and starts of
its streams, compiled as they ship, with the replay of the kernel without such a wave."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2506_13059_amd import build
from tests import test_isa_stream as ref

SRC = os.path.join(os.path.dirname(ref.SRC), "mp_stream_terms.hip")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_every_piece_has_arrived_before_its_use(tmp_path):
    asm = tmp_path / "terms.s"
    subprocess.check_call(["hipcc", *build.FLAGS, *build.EXTRA_FLAGS.get(os.path.basename(SRC), []), "-S", "--cuda-device-only",
                           "-o", str(asm), SRC], stderr=subprocess.DEVNULL)
    text = re.sub(r"value_terms_kernelILi(\d+)E", r"value_stream_kernelILi\1ELi4E", asm.read_text())
    checked = 0
    for heads, _, blocks in ref._kernels(text.splitlines()):
        found, after = ref._bodies(blocks)
        scored = (16 * heads + 63) // 64
        for keys, key_loads, kind in ((True, 4, "L16"), (False, scored, "L4")):
            bodies = {b[1:] for b in found if b[0] == keys}
            main = [b for b in bodies if b[1] == (kind,) * key_loads]
            rest = sorted((b for b in bodies if not b[1]), reverse=True)
            assert len(main) == 1 and len(rest) == 2 and len(bodies) == 3, (heads, bodies)
            waits = {2: (main[0][0], main[0][2]), 1: (rest[0][0], rest[0][2]), 0: (rest[1][0], rest[1][2])}
            for n in range(1, 21):
                for listed in (True, False) if keys else ("scored",):
                    ref._replay(n, key_loads, waits, listed, False)
        assert ref._compiled_starts(blocks, "W0") == {ref._starts(scored, "scored", False), ref._starts(4, True, False)}, heads
        assert ref._starts(4, False, False) in ref._compiled_starts(blocks, "G"), heads
        assert after <= {("L16",) * 4, ("L16",) * 4 + ("L4",), ()}, (heads, after)
        checked += 1
    assert checked == 8
