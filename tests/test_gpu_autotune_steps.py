"""The autotuner varies the staged triangle roots' workgroups per CU as what they
are, the larger of tc_blocks_per_cu[1] and [2]: a setting of which only the
smaller differs is the same schedule, and is never chosen over another."""
import pytest

import graphgen
from gpu_util import build

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpm():
    import paper_2011_03135_amd as m
    m.load()
    return m


def reachable(b1, b2):
    """Settings of [1], [2] by doubling and halving their maximum."""
    seen, todo = {(b1, b2)}, [(b1, b2)]
    while todo:
        a, b = todo.pop()
        for new in (2 * max(a, b), max(a, b) // 2):
            new = min(64, max(1, new))
            s = (new, min(b, new))
            if s not in seen:
                seen.add(s)
                todo.append(s)
    return seen


@pytest.mark.parametrize("b1,b2", [(8, 4), (4, 16), (1, 1), (64, 64)])
def test_only_the_larger_is_varied(gpm, b1, b2):
    g = build(gpm, graphgen.rmat(11, seed=b1 + b2))
    for _ in range(3):
        g.set_tuning(tc_blocks_per_cu=[32, b1, b2])
        print(f"autotune from {b1}, {b2}", flush=True)
        t = tuple(g.autotune()["tc_blocks_per_cu"][1:])
        assert t in reachable(b1, b2)
