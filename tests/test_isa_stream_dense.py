"""CPU-only check of the dense value pass's load pipeline: the tile bodies and starts of its stream, compiled as they ship, with the
replay of the kernel that serves decode steps."""
import os
import shutil
import subprocess

import pytest

from paper_2506_13059_amd import build
from tests import test_isa_stream as ref

SRC = os.path.join(os.path.dirname(ref.SRC), "mp_stream_dense.hip")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_every_piece_has_arrived_before_its_use(tmp_path):
    asm = tmp_path / "dense.s"
    subprocess.check_call(["hipcc", *build.FLAGS, *build.EXTRA_FLAGS.get(os.path.basename(SRC), []), "-S", "--cuda-device-only",
                           "-o", str(asm), SRC], stderr=subprocess.DEVNULL)
    checked = 0
    for heads, waves, blocks in ref._kernels(asm.read_text().replace("value_dense_kernel", "value_stream_kernel").splitlines()):
        found, after = ref._bodies(blocks)
        bodies = {b[1:] for b in found}
        main = [b for b in bodies if b[1] == ("L16",) * 4]
        rest = sorted((b for b in bodies if not b[1]), reverse=True)
        assert all(b[0] for b in found) and len(main) == 1 and len(rest) == 2 and len(bodies) == 3, (heads, waves, bodies)
        waits = {2: (main[0][0], main[0][2]), 1: (rest[0][0], rest[0][2]), 0: (rest[1][0], rest[1][2])}
        for n in range(1, 21):
            ref._replay(n, 4, waits, False, False)
        assert ref._starts(4, False, False) in ref._compiled_starts(blocks, "G"), (heads, waves)
        assert after <= {("L16",) * 4, ()}, (heads, waves, after)
        checked += 1
    assert checked == 16
