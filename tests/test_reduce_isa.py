"""The kernels whose barriers wait for LDS accesses only (the reduced solve's and
the DP sweep), as built for gfx950: every access to LDS has to be one (ds_*).  A generic pointer
into LDS makes it a flat_* access, which passed the barrier: a parent could be
summed before its children."""

import re

import pytest

from paper_2608_01655_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    with pytest.MonkeyPatch.context() as mp:
        mp.setattr(build, "BUILD_DIR", str(tmp_path_factory.mktemp("isa")))
        with open(build.isa("pp_reduce.hip")) as fh:
            text = fh.read()
        with open(build.isa("pp_kernels.hip")) as fh:
            text += fh.read()
    found = {}
    for m in re.finditer(r"^(_ZN2pp\S*k_(?:ladder|reduce|dp)I\S*):", text, re.M):
        body = text[m.end():text.index(".Lfunc_end", m.end())]
        found[m.group(1)] = [x.split(";")[0].strip() for x in body.splitlines()]
    return found


def test_every_kernel_is_there(kernels):
    for part, count in (("k_ladder", 2), ("k_reduce", 2), ("k_dp", 1)):
        assert sum(part in x for x in kernels) >= count, (part, list(kernels))


def test_no_generic_accesses(kernels):
    for name, lines in kernels.items():
        assert not [x for x in lines if re.match(r"flat_", x)], name


def test_barriers_wait_for_lds(kernels):
    """No LDS access between the last wait and a barrier, in program text."""
    for name, lines in kernels.items():
        assert any(x.startswith("s_barrier") for x in lines)
        for q, x in enumerate(lines):
            if not x.startswith("s_barrier"):
                continue
            for y in reversed(lines[:q]):
                assert not y.startswith("ds_"), (name, q, y)
                if re.match(r"s_waitcnt.*lgkmcnt\(0\)", y):
                    break
