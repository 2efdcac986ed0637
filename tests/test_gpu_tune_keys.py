"""What a remembered shape is taken for: frames of one size whose buffers tile
alike, measured on this revision of the kernels."""
import json

import pytest
import torch

import paper_2211_00645_amd as dsk
from paper_2211_00645_amd import synth
from paper_2211_00645_amd.batch import Batch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GEO = (35.0, 0.4, 0.115)


def _stack(shape):
    return synth.blob_stack(shape, synth.blobs_for_volume(*shape), 5, device=DEV)


def test_a_volume_off_alignment_is_tuned_for_itself():
    """The shape remembered for an aligned volume of the frame is not handed to
    a volume one element off: it launches (and so fills the volume)."""
    shape = (76, 28, 272)                   # a frame no other test tunes
    st = _stack(shape)
    w, _ = dsk.plan(shape, shift=dsk.shift_px(*GEO))
    n = shape[0] * shape[1] * w
    assert (shape[1] * w) % 4 == 0
    for off in (0, 1):
        vol = torch.full((n + off,), -7.0, device=DEV)[off:].view(shape[0], shape[1], w)
        dsk.autotune(st, *GEO, out={"vol": vol}, reps=3)
        torch.cuda.synchronize()
        assert not bool((vol == -7.0).any()), off


def test_under_capture_the_other_tilings_shape_serves():
    """A stream under capture cannot be timed: a frame tuned before, whose
    volume now lies off alignment, still gets a shape."""
    shape = (60, 26, 280)                   # a frame no other test tunes
    st = _stack(shape)
    ref = dsk.deskew(st, *GEO, tune="auto")
    n = ref["vol"].numel()
    vol = torch.full((n + 1,), -7.0, device=DEV)[1:].view(ref["vol"].shape)
    out = {"vol": vol, "psum": torch.empty_like(ref["psum"]), "pmax": torch.empty_like(ref["pmax"])}
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dsk.deskew(st, *GEO, tune="auto", out=out)
    for _ in range(3):
        for t in out.values():
            t.fill_(-7.0)
        graph.replay()
        torch.cuda.synchronize()
        for k in ("vol", "psum", "pmax"):
            assert torch.equal(out[k], ref[k]), k


def test_entries_of_earlier_kernels_are_not_taken(tmp_path, monkeypatch):
    """nt_store 0 is no candidate: a tuned shape with it came from the file."""
    stale = dict(block=256, per_thread=8, nt_store=0, unroll=1, wg_per_cu=0, pace_gbs=0, ms=1e-6,
                 mode=0)

    shape = (68, 22, 268)                   # a frame no other test tunes
    st = _stack(shape)
    path = tmp_path / "fwd.json"
    w, _ = dsk.plan(shape, shift=dsk.shift_px(*GEO))
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    old = f"{arch}/fwd/u16/68x22x268/w{w}/vsm/uniform"
    path.write_text("{\n" + f'  "{old}": ' + json.dumps(stale) + "\n}\n")
    monkeypatch.setenv("DSK_TUNE_CACHE", str(path))
    assert dsk.autotune(st, *GEO, reps=3)["tune"]["nt_store"] == 1
    assert json.loads(path.read_text())[old] == stale        # kept for the library it is of
    monkeypatch.delenv("DSK_TUNE_CACHE")

    stacks = [_stack((20, 12, 70)), _stack((9, 30, 64))]
    first, second = tmp_path / "a.json", tmp_path / "b.json"
    b = Batch(stacks, [GEO] * 2, psum=False, cache_path=first)
    b.close()
    batch = [k for k in json.loads(first.read_text()) if "/jobs" in k]
    assert len(batch) == 1 and batch[0].split("/")[1].startswith("k")
    arch, _, rest = batch[0].split("/", 2)
    second.write_text("{\n" + f'  "{arch}/{rest}": ' + json.dumps(stale) + "\n}\n")
    b = Batch(stacks, [GEO] * 2, psum=False, cache_path=second)
    assert b.tune["nt_store"] == 1
    b.close()
