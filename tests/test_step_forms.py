"""The rule that gives the groups of a plain launch the low-latency form or the queue,
compiled for the host: limits of a group alone, on a whole card and on an eighth of it,
and groups that run side by side."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1106_2899_amd", "csrc")
LIMIT = {(0, 1): 8, (0, 2): 5, (1, 1): 4, (1, 2): 2}  # workgroups per CU of a group alone


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if not cxx:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("forms") / "forms")
    subprocess.check_call([cxx, "-O1", "-std=c++17", f"-I{CSRC}", "-o", exe, os.path.join(HERE, "step_forms.cpp")])

    def run(cases):  # (fp64, cus, [(beads, tasks, queue_only), ...])
        text = "\n".join(f"{f} {c} {len(g)} " + " ".join("%d:%d:%d" % x for x in g) for f, c, g in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        rows = [[int(x) for x in r.split()] for r in out if r]
        return [(r[0], r[1:]) for r in rows]
    return run


@pytest.mark.parametrize("cus", [256, 32])
@pytest.mark.parametrize("fp64,beads", list(LIMIT))
def test_a_group_alone(choose, fp64, beads, cus):
    most = cus * LIMIT[fp64, beads]
    got = choose([(fp64, cus, [(beads, t, 0)]) for t in (1, cus, cus + 1, most, most + 1)])
    assert got == [(1, [1]), (1, [1]), (2, [1]), (LIMIT[fp64, beads], [1]), (1, [0])]


def test_groups_side_by_side(choose):
    got = choose([
        (0, 256, [(1, 512, 0), (1, 512, 0)]),              # fit together: spread by their sum
        (0, 256, [(1, 2048, 0), (1, 2048, 0)]),            # each within its limit, not together
        (1, 256, [(1, 500, 0)] * 4 + [(2, 500, 0)]),
        (0, 256, [(1, 1000, 0), (2, 700, 0)]),
        (0, 256, [(1, 3000, 0), (1, 200, 0)]),             # one beyond its own limit
        (0, 256, [(1, 200, 0), (2, 1500, 0)]),
        (0, 256, [(2, 30000, 1), (1, 300, 0), (2, 300, 0)]),  # beside packed wavefronts
        (1, 256, [(1, 200, 0), (2, 500, 0)]),
    ])
    assert got == [(4, [1, 1]), (1, [0, 0]), (1, [0, 0, 0, 0, 1]), (1, [0, 1]), (1, [0, 1]), (1, [1, 0]),
                   (1, [0, 1, 1]), (3, [1, 1])]


def test_low_latency_workgroups_are_resident(choose):
    rng = np.random.default_rng(5)
    cases = []
    for _ in range(2000):
        n = int(rng.integers(1, 8))
        groups = [(int(rng.integers(1, 3)), int(np.exp(rng.uniform(0, 9))), 0) for _ in range(n)]
        cases.append((int(rng.integers(0, 2)), int(rng.choice([32, 64, 256])), groups))
    for (fp64, cus, groups), (per_cu, forms) in zip(cases, choose(cases)):
        used = sum(t / (cus * LIMIT[fp64, b]) for (b, t, _), on in zip(groups, forms) if on)
        assert used <= (1.25 if fp64 else 1.0) + 1e-12
        assert per_cu == (-(-sum(t for _, t, _ in groups) // cus) if all(forms) else 1)
