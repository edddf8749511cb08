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
        """calls: (units, G, (k_bits, v_bits), packed tiles, window tokens, ring tiles, workspace) each
        -> (status, splits, waves, block, pace, uses the workspace)"""
        lines = "\n".join(f"{u} 1 {G} {kb} {vb} {32 * t} {n_w} {32 * W} 0 {ws} 0" for u, G, (kb, vb), t, n_w, W, ws in calls) + "\n"
        out = subprocess.run([exe], input=lines, capture_output=True, text=True, check=True).stdout.split("\n")[:-1]
        assert len(out) == len(calls)
        return [tuple(map(int, o.split())) for o in out]

    return run


TILES = (1, 8, 24, 47, 64, 94, 96, 126, 160, 250, 375, 500, 1000)
BITS = ((1, 1), (2, 2), (3, 2), (2, 4), (3, 3), (4, 4))


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_a_call_that_needs_no_workspace_uses_none(plans, G):
    """What is accepted without a workspace leaves one that it is given alone, whatever it holds and whoever else uses it:
    overlapping calls may hand over the same one."""
    calls = [(u, G, bits, t, 96, 4, 0) for bits in BITS for t in TILES for u in range(1, 620)]
    alone = plans(calls)
    given = plans([c[:-1] + (-1,) for c in calls])
    unsplit = 0
    for c, a, b in zip(calls, alone, given):
        if a[0] == 0:
            unsplit += 1
            assert a == b, (c, a, b)
    assert unsplit > len(calls) // 3


def counted(plans, calls):
    """Per call the launch with the smallest workspace it is accepted with: the count without a second workgroup on any compute unit."""
    found = [None] * len(calls)
    for s in range(0, 65):
        open_ = [i for i, f in enumerate(found) if f is None]
        if not open_:
            break
        size = lambda u, G: 0 if s < 2 else (4 * u + 255) // 256 * 256 + u * s * G * 520
        for i, o in zip(open_, plans([calls[i][:-1] + (size(calls[i][0], calls[i][1]),) for i in open_])):
            if o[0] == 0:
                found[i] = o
    return found


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_more_splits_only_for_tiles_that_are_there(plans, G):
    """A ring may be mostly empty (room for steps to come): what it could hold is no work, and no reason for more workgroups than compute units."""
    calls = [(u, G, (2, 2), t, 96, W, -1) for W in (4, 100, 400) for t in (2, 20, 94, 126, 250, 500) for u in (40, 52, 56, 65, 73, 86, 94, 102)]
    more = 0
    for c, base, full in zip(calls, counted(plans, calls), plans(calls)):
        if full[1] > base[1]:
            more += 1
            live = c[3] + 3
            assert live // full[1] >= 8 and c[0] * full[1] <= 512, (c, base, full)
            assert 62 + 2 * live / full[1] < 0.92 * (60 + live / base[1]), (c, base, full)
    assert more > 10


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_more_splits_only_where_they_were_measured(plans, G):
    """From 2 splits with all group sizes, from 3 with 2 heads and more, and with few bits per Key and Value; in the middle of
    those ranges they are taken."""
    wide = 5 if G > 1 else 4
    calls = [(u, G, bits, t, 96, 4, -1) for bits in BITS + ((1, 3), (4, 1)) for t in (94, 126, 250, 500, 1000) for u in range(40, 257)]
    for c, base, full in zip(calls, counted(plans, calls), plans(calls)):
        if full[1] > base[1]:
            kb, vb = c[2]
            assert base[1] == 2 or (base[1] == 3 and G > 1), (c, base, full)
            assert kb + vb <= wide and not (G == 8 and vb > 2), (c, base, full)
            assert full[1:3] == ({2: 5, 3: 7}[base[1]], 8) and full[4:] == (1, 1), (c, base, full)
    middle = [(u, G, bits, t, 96, 4, -1) for bits in ((1, 1), (2, 2)) for u, t in ((94, 200), (94, 375)) + (((69, 500), (69, 1000)) if G > 1 else ())]
    for c, base, full in zip(middle, counted(plans, middle), plans(middle)):
        assert full[1] > base[1] > 1, (c, base, full)
