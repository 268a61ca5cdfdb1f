"""The tuner's default candidates differ in what they launch: a batched carve of
depth 4 does the same work whatever the tile's width and workgroups.  No GPU."""
from paper_1903_11785_amd import autotune


def test_each_candidate_launches_something_else():
    work = [("culled",) if t.tz == 4 else (t.tx, t.tz, t.persistent_blocks)
            for t in autotune.candidates(256)]
    assert ("culled",) in work and len(set(work)) == len(work)
