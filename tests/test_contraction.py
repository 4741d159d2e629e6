"""The training kernels' code does not depend on the compiler's contraction of products and
sums (CPU: compiles to gfx950 assembly, runs nothing).

Kernels that promise the same bits (forward of 256 and of 32 rows, dQ likewise, dK / dV by
blocks and by pairs) must not owe them to the compiler's choice of fused operations: with
contraction switched off it has to emit the instructions that it emits by default.
"""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2609_32712_amd import build as libbuild

pytestmark = pytest.mark.skipif(not os.path.exists(libbuild.HIPCC), reason="needs hipcc")


def _kernels(src, extra, out):
    """Instructions of every kernel of a source, compiled with the build's flags and extra."""
    flags = libbuild.FLAGS + libbuild.FILE_FLAGS.get(os.path.basename(src), [])
    subprocess.run([libbuild.HIPCC, *flags, *extra, "--cuda-device-only", "-S", src,
                    "-o", out], check=True, capture_output=True)
    res, cur = {}, None
    with open(out) as f:
        for line in f:
            m = re.match(r"(_ZN\w+):", line)
            if m:
                cur = res.setdefault(m.group(1), [])
            elif line.startswith(".Lfunc_end"):
                cur = None
            elif cur is not None and line.startswith("\t") and not line.startswith("\t."):
                cur.append(line.split(";")[0].split())
    return res


@pytest.mark.parametrize("name", ["mala_fwd.hip", "mala_bwd.hip"])
def test_training_kernels_do_not_depend_on_contraction(name, tmp_path):
    src = os.path.join(libbuild.CSRC, name)
    with ThreadPoolExecutor(2) as ex:
        std, off = ex.map(lambda a: _kernels(src, *a), (
            ([], str(tmp_path / "std.s")), (["-ffp-contract=off"], str(tmp_path / "off.s"))))
    assert any("fwd" in k or "bwd" in k for k in std) and std.keys() == off.keys()
    for k in std:
        assert len(std[k]) > 50, k
        assert std[k] == off[k], k
