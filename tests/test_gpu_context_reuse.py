"""One context over changing sizes, systems, group sizes and active lists: what
it forms equals what a new context forms, bit for bit, so nothing left in its
buffers by an earlier build or walk is read."""
import sys

import numpy as np
import pytest

from paper_1507_01009_amd import ics
from gpu_helpers import gpu_run

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


# (stars, system offsets, leaf, group, every k-th star active): the sorts of one
# block and of merged runs, groups formed with the nodes and (below a leaf) by
# kernels of their own, split and whole groups, in changing order
RUNS = [(4097, None, 8, 64, 1), (700, None, 8, 64, 1), (40000, None, 8, 4, 1),
        (700, None, 8, 4, 3), (4097, None, 16, 3, 1), (40000, None, 8, 64, 7),
        (4096, [0, 1, 1, 2000, 4096], 8, 4, 1), (40000, None, 8, 128, 1),
        (9000, [0, 5000, 5000, 9000], 16, 3, 2), (1, None, 8, 64, 1), (4097, None, 8, 64, 50)]


@pytest.mark.parametrize("levels", [21, 42])
@pytest.mark.parametrize("precision", [0, 1])
def test_as_a_new_context(precision, levels):
    from paper_1507_01009_amd import binding as B
    ctx = B.Context(40000, max_systems=4, precision=precision, key_levels=levels)
    for n, off, nl, ng, every in RUNS:
        say("context reuse", precision, levels, n, off, nl, ng, every)
        pos, _, m = ics.plummer(max(n, 2), n + nl)
        pos, m = pos[:n], m[:n]
        act = None if every == 1 else np.arange(0, n, every, dtype=np.int32)
        off = None if off is None else np.array(off)
        ctx.set_sizes(nl, ng)
        a = gpu_run(pos, m, 0.01, 0.5, nl, ng, active=act, sys_off=off, ctx=ctx)
        b = gpu_run(pos, m, 0.01, 0.5, nl, ng, active=act, sys_off=off, precision=precision,
                    key_levels=levels)
        assert a["counts"] == b["counts"]
        for k, v in b["tree"].items():
            assert np.array_equal(a["tree"][k], v), (n, k)
        assert np.array_equal(a["acc"], b["acc"], equal_nan=True)
        assert np.array_equal(a["pot"], b["pot"], equal_nan=True)
        b["ctx"].close()
    ctx.close()
