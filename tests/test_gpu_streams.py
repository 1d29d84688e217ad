"""Which of an engine's calls wait for which, by what is done when: heads and encodes beside a depth head, or a caller's kernel, of tens of
milliseconds.

In a process of its own, with five hardware queues: one each for the default stream and an engine's four, since streams that share
one run in turn whatever the engine does (the other tests' process has made dozens of streams)."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
import json, sys
import numpy as np
import torch
import paper_2508_11584_amd as vpe
import vpe_inputs as vi
from paper_2508_11584_amd.synthetic import make_engine

SPEC = vi.ModelSpec("long_head", dim=64, depth=4, heads=1, mlp_hidden=64, img_h=518, img_w=518, taps=(1, 2, 3, 4), head_ch=1024,
                    dtype="bf16", batch=12)
image = torch.from_numpy(vi.make_batch(SPEC, 31)).cuda()

def engine(kinds, **kw):
    eng, _, _ = make_engine(SPEC, 30, kinds=kinds, **kw)
    for _ in range(2):                                   # (the first launches load code)
        fh = eng.encode(image)
        for h in range(len(kinds)):
            eng.run_head(h, fh)
        eng.sync()
    return eng

def ready(eng, fh):
    while eng.frame_ready(fh) == vpe.VPE_BUSY:
        pass

found = {}

# a long head on an idle engine, then the next frame
eng = engine(("depth",))
eng.run_head(0, eng.encode(image))
ready(eng, eng.encode(image))
found["long head done when the next encode was"] = eng.head_done(0)
eng.sync()
eng.close()

# a short head behind a long one: called on the same frame, then polled on the next
eng = engine(("depth", "det"), ring_slots=4)
fh = eng.encode(image)
eng.run_head(0, fh)
eng.run_head(1, fh)
eng.wait_head(1)
found["long head done when the short one called behind it was"] = eng.head_done(0)
eng.sync()
eng.run_head(0, eng.encode(image))
ready(eng, eng.encode(image))
assert eng.run_head_latest(1)[0] == vpe.VPE_OK
eng.wait_head(1)
found["long head done when the polled one was"] = eng.head_done(0)
eng.sync()
eng.close()

# a short head that shares a long one's stream (three for four heads): behind it on an older frame, then called on the newest
eng = engine(("depth", "depth", "depth", "seg"), ring_slots=8)
older = eng.encode(image)
eng.run_head(0, older)
newest = eng.encode(image)
eng.run_head(3, older)
eng.run_head(3, newest)
ready(eng, eng.encode(image))
found["long head done when the encode behind a short one was"] = eng.head_done(0)
eng.sync()
eng.close()

# three lanes: an encode into a slot that a long head reads waits for it, and a short head for that encode; other lanes do not
eng = engine(("depth", "seg"), encoder_lanes=3, ring_slots=5)
eng.run_head(0, eng.encode(image))
for _ in range(4):
    eng.encode(image)
for _ in range(2):
    eng.run_head(1, eng.encode(image))
for _ in range(3):
    fh = eng.encode(image)
ready(eng, fh)
found["long head done when another lane's encode was"] = eng.head_done(0)
eng.sync()
eng.close()

# a short head beside 20 ms or more of the caller's own work on the borrowed encoder stream (the next frame's copy, say), asked for
# again or kept from before
def borrowed_work(stream):
    with torch.cuda.stream(torch.cuda.ExternalStream(stream)):
        torch.cuda._sleep(50_000_000)
        done = torch.cuda.Event()
        done.record()
    return done

eng = engine(("seg",), ring_slots=4)
kept = eng.next_encode_stream()
for name, ask in (("asked for again", eng.next_encode_stream), ("kept", lambda: kept)):
    fh = eng.encode(image)
    work = borrowed_work(ask())
    eng.run_head(0, fh)
    eng.wait_head(0)
    found["caller's work done when the head was, stream " + name] = work.query()
    eng.sync()
    torch.cuda.synchronize()
eng.close()

# a run behind the caller's work on a stream it named; the head's next run waits for that run, the encode behind must not
eng = engine(("seg",), ring_slots=4)
mine = torch.cuda.Stream()
fh = eng.encode(image)
work = borrowed_work(mine.cuda_stream)
eng.run_head(0, fh, mine)
eng.run_head(0, eng.encode(image))
ready(eng, eng.encode(image))
found["caller's work done when the second next encode was"] = work.query()
eng.sync()
torch.cuda.synchronize()
eng.close()
print(json.dumps(found))
"""


@pytest.fixture(scope="module")
def found():
    r = subprocess.run([sys.executable, "-c", PROGRAM], cwd=ROOT, env={**os.environ, "GPU_MAX_HW_QUEUES": "5"}, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
    print(r.stdout, flush=True)
    return json.loads(r.stdout.splitlines()[-1])


def test_a_long_head_does_not_hold_the_next_encode(found):
    assert not found["long head done when the next encode was"]


def test_short_heads_do_not_wait_for_a_long_one(found):
    assert not found["long head done when the short one called behind it was"]
    assert not found["long head done when the polled one was"]


def test_a_short_head_behind_a_long_one_does_not_hold_the_next_encode(found):
    assert not found["long head done when the encode behind a short one was"]


def test_lanes_do_not_wait_for_each_other_through_a_short_head(found):
    assert not found["long head done when another lane's encode was"]


def test_heads_do_not_wait_for_the_callers_work_on_a_borrowed_stream(found):
    assert not found["caller's work done when the head was, stream asked for again"]
    assert not found["caller's work done when the head was, stream kept"]


def test_encodes_do_not_wait_for_the_callers_work_in_front_of_a_head(found):
    assert not found["caller's work done when the second next encode was"]
