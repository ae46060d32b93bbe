"""The library's host code where the device's answers have to be scripted (a
HIP runtime in host memory, tests/hipstub): what a call clears."""
from tests import hipstub


def test_assign_clears_every_bitmap():
    """A mesh that another is copied into starts from the state between two
    rounds: of the subsegments' bitmaps (points that hold their marks, winners,
    winners on the hull) none keeps a bit of a round that did not end."""
    fills = [(int(v), int(n)) for word, v, n in hipstub.run("assign") if word == "fill"]
    cap = [n // 8 for v, n in fills if v == 0xff]  # the side slots, two per subsegment
    assert len(cap) == 1
    assert fills.count((0, 4 * (cap[0] // 32 + 1))) == 3, fills
