"""The library's host code where the device's answers have to be scripted (a
HIP runtime in host memory, tests/hipstub): what a call clears,
what it waits for after a failure, what it does without device memory or
threads, and the sizes it asks for."""
from tests import hipstub


def test_assign_clears_every_bitmap():
    """A mesh that another is copied into starts from the state between two
    rounds: of the subsegments' bitmaps (points that hold their marks, winners,
    winners on the hull) none keeps a bit of a round that did not end."""
    fills = [(int(v), int(n)) for word, v, n in hipstub.run("assign") if word == "fill"]
    cap = [n // 8 for v, n in fills if v == 0xff]  # the side slots, two per subsegment
    assert len(cap) == 1
    assert fills.count((0, 4 * (cap[0] // 32 + 1))) == 3, fills


def test_batch_waits_before_the_builders_take_over():
    """Workgroup builds of a batch whose launch fails part way may be running:
    the builder threads, which write the same meshes on streams of their own,
    begin when nothing is left on the caller's stream."""
    assert hipstub.run("launch") == [["pending", "0"]]


def test_batch_without_room_for_device_builds():
    """The library's choice to build a batch's CDTs on the device costs no
    member: without device memory for those builds (workgroups and builder
    threads) each is refined from the host's CDT, as a smaller batch's are."""
    out = [line for line in hipstub.run("scratch") if line[0] != "live"]
    assert out[0] == ["batch", "0"] and len(out) == 8
    for word, status, got, want in out[1:]:
        assert word == "member" and status == "0" and got == want, out


def test_batch_gives_its_memory_back():
    """... also where no member is left in the batch's common allocation: with
    the meshes freed, nothing the call allocated remains."""
    assert [line for line in hipstub.run("scratch") if line[0] == "live"] == [["live", "0"]]


def test_batch_without_threads():
    """Where no thread can be created the caller does their work: no exception
    leaves the C call (a batch built on the host, then one meant for the
    device)."""
    out = [line for line in hipstub.run("threads") if line[0] != "live"]
    assert out[:2] == [["batch", "0"], ["batch", "0"]] and len(out) == 9
    for word, status, got, want in out[2:]:
        assert word == "member" and status == "0" and got == want, out


def test_builder_scratch_of_large_inputs():
    """The device CDT builder's scratch holds its arrays at every size that a
    mesh can have (89 million vertices): per triangle slot at least three
    16-byte records, two 8-byte stamps and two lists of two flip candidates (16
    bytes each, twice)."""
    out = hipstub.run("sizes")
    assert len(out) == 5
    for word, nv, nbytes in out:
        assert word == "scratch" and int(nbytes) >= 2 * int(nv) * (3 * 16 + 2 * 8 + 4 * 16), (nv, nbytes)
