"""What the sampler loops ask of the HIP runtime, on a stand-in for it that runs nothing (fake_hip.c): the order of
the kernels and the streams they go to, and what a call does when the runtime refuses something.  No GPU is needed,
and orders that would race on one can be looked at without running them."""
import ctypes
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["gcc", "-O1", "-w", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "fake_hip.c")], check=True)
    return so


HEAD = '''
import ctypes, os, sys
sys.path.insert(0, {root!r})
F = ctypes.CDLL({so!r}, mode=ctypes.RTLD_GLOBAL)
F.fake_log.restype = ctypes.c_char_p
from paper_2609_30096_amd import synth, track
L = track.lib()
BASE = 1 << 40  # device addresses; nothing reads them
shape = synth.TINY_LATENT
sc = synth.SamplerConfig(steps=3, shift=3.0, guidance=5.0)
LARGE, SMALL = synth.TINY_LARGE, synth.TINY_SMALL


def model(cfg, ws=None, extra=0):
    h = ctypes.c_void_p()
    c = track.config_c(cfg)
    n = L.track_weights_bytes(ctypes.byref(c))
    assert L.track_model_create(ctypes.byref(c), ctypes.c_void_p(BASE), n, ctypes.byref(h)) == 0
    need = L.track_workspace_bytes(h, ctypes.byref(track.shape_c(shape)), 2)
    if ws is not None:
        assert L.track_model_set_workspace(h, ctypes.c_void_p(ws), need + extra) == 0
    return h, need


def ptrs(*a):
    return (ctypes.c_void_p * len(a))(*a)


def calibrate(l, s, M=1):
    x, c = [BASE + (1 << 32) + 4096 * i for i in range(M)], [BASE + (2 << 32) + 4096 * i for i in range(M)]
    return L.track_calibrate(l, s, ctypes.byref(track.shape_c(shape)), M, ptrs(*x), ptrs(*c),
                             ctypes.c_void_p(BASE + (3 << 32)), ctypes.byref(track.sampler_c(sc)), None, None, None,
                             ctypes.c_void_p(0x77))


def sample(l, s, mask):
    return L.track_sample(l, s, (ctypes.c_uint8 * sc.steps)(*mask), ctypes.byref(track.shape_c(shape)),
                          ctypes.byref(track.sampler_c(sc)), ctypes.c_void_p(BASE + (1 << 32)),
                          ctypes.c_void_p(BASE + (2 << 32)), ctypes.c_void_p(BASE + (3 << 32)),
                          ctypes.c_void_p(BASE + (4 << 32)), ctypes.c_void_p(0x77))


def log():
    t = F.fake_log().decode().splitlines()
    F.fake_clear()
    return [l.split() for l in t]


# P: a model's context formed (its RoPE tables), f: a forward pass begun, other kernels not shown
def passes(lg):
    return "".join("P" if "rope_tables" in n else "f" for op, n, st in lg
                   if op == "launch" and ("rope_tables" in n or "mod_tables" in n))


def streams(lg):
    return {{st for op, n, st in lg if op == "launch"}}


def err():
    return L.track_last_error().decode()
'''


def run(fake, body):
    code = HEAD.format(root=ROOT, so=fake) + body
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_calibrate_on_disjoint_workspaces(fake):
    """A small pair's two models run on two streams; each context is formed once per sample.  Attached sizes that
    reach into each other beyond what the layouts need (one arena handed out in pieces) count as disjoint."""
    run(fake, '''
for ws_s in (BASE + (5 << 32), BASE + (6 << 32)):
    l, n = model(LARGE, BASE + (5 << 32) - (1 << 24), extra=1 << 25)
    s, _ = model(SMALL, ws_s)
    assert n < 1 << 24
    assert calibrate(l, s, M=2) == 0, err()
    lg = log()
    assert passes(lg) == "PP" + 6 * "f" + "PP" + 6 * "f", passes(lg)
    assert len(streams(lg)) == 2 and "77" in streams(lg)
    assert sample(l, s, [0, 1, 0]) == 0, err()
    assert passes(log()) == "PfPff"
''')


def test_calibrate_on_overlapping_workspaces(fake):
    """The small model's workspace inside the large one's scratch: each forward pass follows its own model's context,
    everything on the caller's stream."""
    run(fake, '''
import dataclasses
big = dataclasses.replace(LARGE, dim=512, heads=16, ffn_dim=2048)
l, nl = model(big, BASE + (5 << 32))
s, ns = model(SMALL, BASE + (5 << 32) + 256)
assert ns + 256 < nl - (1 << 20)   # before the large model's trajectory state at the end
assert calibrate(l, s, M=2) == 0, err()
lg = log()
assert passes(lg) == 12 * "Pf", passes(lg)
assert streams(lg) == {"77"}
assert sample(l, s, [1, 0, 0]) == 0, err()
assert passes(log()) == "PfPff"
''')


def test_calibrate_without_a_second_stream(fake):
    """Where the runtime refuses the second stream, its events or the query before them, the call runs on one."""
    run(fake, '''
l, _ = model(LARGE, BASE + (5 << 32))
s, _ = model(SMALL, BASE + (6 << 32))
for name in (b"hipStreamCreateWithFlags", b"hipEventCreateWithFlags", b"hipStreamIsCapturing"):
    F.fake_fail(name, 1)
    assert calibrate(l, s) == 0, (name, err())
    lg = log()
    assert passes(lg) == "PfPfffff", (name, passes(lg))
    assert streams(lg) == {"77"}, name
assert calibrate(l, s) == 0 and len(streams(log())) == 2
''')


def test_progress_callback_may_use_the_models(fake):
    """A progress callback can run the small model on another prompt, or write the embeddings: the contexts are formed
    anew after it, in sampling and calibration."""
    run(fake, '''
l, _ = model(LARGE, BASE + (5 << 32))
s, _ = model(SMALL, BASE + (6 << 32))
seen = []
def preview(user, j, k, n):
    seen.append((j, k))
    st = L.track_dit_forward(s, ctypes.byref(track.shape_c(shape)), ctypes.c_void_p(BASE), 500.0,
                             ctypes.c_void_p(BASE + (7 << 32)), None, 1.0, ctypes.c_void_p(BASE + (8 << 32)),
                             ctypes.c_void_p(0x77))
    assert st == 0, err()
track.set_progress(lambda j, k, n: preview(None, j, k, n))
assert sample(l, s, [1, 1, 0]) == 0, err()
lg = log()
assert passes(lg) == 3 * "PfPf", passes(lg)   # a step, the preview
assert calibrate(l, s) == 0, err()
lg = log()
assert passes(lg) == 3 * "PPffPf", passes(lg)
assert seen == [(-1, 0), (-1, 1), (-1, 2), (0, 0), (0, 1), (0, 2)]
track.set_progress(None)
assert sample(l, s, [1, 1, 0]) == 0, err()
assert passes(log()) == "PffPf"
''')


def test_band_energy_without_pinned_memory(fake):
    """Refused pinned memory falls back to a copy from the workspace; a slot that a kernel may still write, because the
    call failed before it was waited for, is not handed to the next call."""
    run(fake, '''
w = L.track_band_workspace_bytes(ctypes.byref(track.shape_c(shape)), 1, 2, 2)
out = (ctypes.c_double * 6)()
def bands():
    return L.track_op_band_energy(ctypes.byref(track.shape_c(shape)), 1, 2, 2, 2, 5.0, ctypes.c_void_p(BASE),
                                  ctypes.c_void_p(BASE + (1 << 32)), ctypes.c_void_p(BASE + (2 << 32)), w, out,
                                  ctypes.c_void_p(0x77))
def ops():
    return [op for op, n, st in log() if op in ("copy", "hostmalloc")]
F.fake_fail(b"hipHostMalloc", 1)
assert bands() == 0, err()
assert ops() == ["hostmalloc", "copy"]
assert bands() == 0 and ops() == ["hostmalloc"]
assert bands() == 0 and ops() == []            # the slot is kept
for name in (b"hipStreamSynchronize", b"hipLaunchKernel"):
    F.fake_fail(name, 1)
    assert bands() == track.E_DEVICE
    ops()
    F.hipGetLastError()
    assert bands() == 0 and ops() == ["hostmalloc"]
''')


def test_forward_of_very_many_blocks(fake):
    """The text values of all blocks are transposed together: more blocks than a grid's third dimension holds (65535)
    take more than one launch."""
    run(fake, '''
shape = synth.LatentShape(16, 1, 4, 4, 3)
many = synth.DiTConfig(blocks=33000, dim=128, heads=1, head_dim=128, ffn_dim=64, text_dim=64, dtype=synth.BF16)
m, _ = model(many, BASE + (5 << 32))
st = L.track_dit_forward(m, ctypes.byref(track.shape_c(shape)), ctypes.c_void_p(BASE), 500.0, ctypes.c_void_p(BASE),
                         ctypes.c_void_p(BASE), 2.0, ctypes.c_void_p(BASE), ctypes.c_void_p(0x77))
assert st == 0, err()
''')
