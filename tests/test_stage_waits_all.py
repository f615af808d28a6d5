"""The check of the staging waits (test_stage_waits) over each kernel's whole text: code laid out
behind an early exit is looked at too, and every column-pass and row-pass kernel has to have
staging barriers.

Like that check it reads the code in the order of its text and does not follow branches: it
finds a wait that a straight run of code does not cover, not one that only some path skips.  The
instances that read X as given wait for every load and pass it whatever the loads' number."""

import os
import re
import subprocess

import pytest

from paper_1802_08938_amd import build as b
from tests.test_stage_waits import LDS, MEM

pytestmark = pytest.mark.slow


def _kernels(text):
    for m in re.finditer(r"^(_ZN4didk\w*(?:colpass|rowpass)\w*):", text, re.M):
        yield m.group(1), [x.strip() for x in text[m.start():text.index(".Lfunc_end", m.start())].splitlines()]


def _staging_barriers(body):
    """(index, covered) of each barrier with staging loads since the barrier before it."""
    for i, line in enumerate(body):
        if line != "s_barrier":
            continue
        start = next((k for k in range(i - 1, -1, -1) if body[k] == "s_barrier" or LDS.match(body[k])), 0)
        if not LDS.match(body[start]):
            continue
        after, done = 0, False  # memory operations issued after the last staging load
        for x in body[start + 1:i]:
            after += bool(MEM.match(x))
            m = re.search(r"s_waitcnt .*vmcnt\((\d+)\)", x)
            done = done or bool(m and int(m.group(1)) <= after)
        yield i, done


def test_finds_an_uncovered_wait():
    lds, load = "buffer_load_dwordx4 v1, s[0:3], 0 offen lds", "global_load_dwordx4 v[0:3], v4, s[0:1]"
    covered = [lds, load, load, "s_waitcnt vmcnt(2) lgkmcnt(0)", "s_barrier"]
    assert [d for _, d in _staging_barriers(covered)] == [True]
    assert [d for _, d in _staging_barriers([lds, load, "s_waitcnt vmcnt(2) lgkmcnt(0)", "s_barrier"])] == [False]
    assert [d for _, d in _staging_barriers([lds, load, "s_endpgm", "s_barrier"] + covered)] == [False, True]


def test_every_pass_kernel_waits_for_its_staging(tmp_path):
    if not os.path.exists(b.HIPCC):
        pytest.skip("no hipcc")
    src = next(s for s in b.SOURCES if s.endswith("did_kernels.hip"))
    out = tmp_path / "k.s"
    flags = [f for f in b.FLAGS if f not in ("-shared", "-fPIC", "-Wall")]
    subprocess.run([b.HIPCC, *flags, "--cuda-device-only", "-S", src, "-o", str(out)], check=True, capture_output=True)
    found = {name: list(_staging_barriers(body)) for name, body in _kernels(out.read_text())}
    # (K class) x (H or not) x storage x waves, carried, grouped; row passes: class x storage, ...
    assert len(found) == 2 * 2 * 3 * 2 + 2 * 3 + 2 * 3 * 2 + 2 * 3 + 2 + 2 * 3
    for name, barriers in found.items():
        assert len(barriers) >= 2, name  # the first tile's, and a chunk's
        assert all(done for _, done in barriers), (name, barriers)
