"""Which launch an attention call gets (split count, workspace) over whole ranges of shapes: host arithmetic, no GPU (split_choice.hip)."""
import os
import subprocess

import pytest

from paper_2506_08018_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "split_choice")
    subprocess.run(build.COMMON + [os.path.join(HERE, "split_choice.hip"), "-o", exe], check=True, capture_output=True)

    def run(calls):
        """calls: (units, G, (k_bits, v_bits), packed tiles, window tokens, ring tiles, workspace) each -> (status, splits, waves, block, pace, uses the workspace)"""
        lines = "\n".join(f"{u} 1 {G} {kb} {vb} {32 * t} {n_w} {32 * W} 0 {ws} 0" for u, G, (kb, vb), t, n_w, W, ws in calls) + "\n"
        out = subprocess.run([exe], input=lines, capture_output=True, text=True, check=True).stdout.split("\n")[:-1]
        assert len(out) == len(calls)
        return [tuple(map(int, o.split())) for o in out]

    return run


TILES = (1, 8, 24, 47, 64, 94, 96, 126, 160, 250, 375, 500, 1000)
BITS = ((1, 1), (2, 2), (3, 2), (2, 4), (3, 3), (4, 4))


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_a_call_that_needs_no_workspace_uses_none(plans, G):
    """What is accepted without a workspace leaves one that it is given alone, whatever it holds and whoever else uses it: overlapping calls may hand over the same one."""
    calls = [(u, G, bits, t, 96, 4, 0) for bits in BITS for t in TILES for u in range(1, 620)]
    alone = plans(calls)
    given = plans([c[:-1] + (-1,) for c in calls])
    unsplit = 0
    for c, a, b in zip(calls, alone, given):
        if a[0] == 0:
            unsplit += 1
            assert a == b, (c, a, b)
    assert unsplit > len(calls) // 3
