"""The passes stage their packed operands straight into LDS and close a chunk with a wait that
leaves the next X tile's loads in flight.  That wait is right only if at least as many memory
operations as it leaves outstanding were issued after the staging loads: checked here in the
code that hipcc generates for gfx950 (no GPU needed)."""

import os
import re
import subprocess

import pytest

from paper_1802_08938_amd import build as b

pytestmark = pytest.mark.slow

MEM = re.compile(r"(global|flat|buffer|scratch)_(load|store|atomic)")
LDS = re.compile(r"global_load_lds|buffer_load_dword\w* .*\blds\b")


def _kernels(text):
    for m in re.finditer(r"^(_ZN4didk\w*(?:colpass|rowpass)\w*):", text, re.M):
        yield m.group(1), text[m.start():text.index("s_endpgm", m.start())].splitlines()


def test_staging_waits_cover_the_staging_loads(tmp_path):
    if not os.path.exists(b.HIPCC):
        pytest.skip("no hipcc")
    src = next(s for s in b.SOURCES if s.endswith("did_kernels.hip"))
    out = tmp_path / "k.s"
    flags = [f for f in b.FLAGS if f not in ("-shared", "-fPIC", "-Wall")]
    subprocess.run([b.HIPCC, *flags, "--cuda-device-only", "-S", src, "-o", str(out)], check=True, capture_output=True)
    barriers = 0
    for name, body in _kernels(out.read_text()):
        for i, line in enumerate(body):
            if line.strip() != "s_barrier":
                continue
            start = next((k for k in range(i - 1, -1, -1) if body[k].strip() == "s_barrier" or LDS.match(body[k].strip())), 0)
            if not LDS.match(body[start].strip()):
                continue
            barriers += 1
            after, done = 0, False  # memory operations issued after the last staging load
            for x in body[start + 1:i]:
                after += bool(MEM.match(x.strip()))
                m = re.search(r"s_waitcnt .*vmcnt\((\d+)\)", x)
                done = done or bool(m and int(m.group(1)) <= after)
            assert done, (name, i, after)
    assert barriers >= 60
