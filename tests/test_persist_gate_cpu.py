"""The order of several models' persistent launches on one device, on the host: the library runs on a stand-in
for the HIP runtime (hip_stub.c) that logs launches, event waits and synchronisations.  Two kernels that each need
every compute unit must not be in flight side by side: with two models alive, every launch waits for the event of
the one before it, also while one of the models is being destroyed."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = r'''
import ctypes, os, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
stub.stub_log.restype = ctypes.c_char_p
SYNC = ctypes.CFUNCTYPE(ctypes.c_int)
import workloads as wl
from paper_2606_08094_amd import vla
CFG = wl.PI0_BF16.with_(n_layers=1, d_model=512, head_dim=64, d_ff=2048, d_prefix=512, prefix_len=40, n_steps=1)
P, L = CFG.prefix_len, vla.lib()
buf = ctypes.create_string_buffer((16 << 20) + 256)
mem = (ctypes.addressof(buf) + 255) // 256 * 256   # one zeroed block stands for every weight and buffer

def model():
    return vla.Model(CFG, {n: mem for n in vla.weight_order(CFG)})

def denoise(m, stream):
    m.denoise(mem, m.kv_cache_bytes(1, P), 1, P, mem, mem, [1.0, 0.0], None, None, mem, stream)

def events():
    out = [l.split() for l in stub.stub_log().decode().splitlines()]
    stub.stub_clear()
    return [(w, int(s, 16), int(e, 16)) for w, s, e in out if w != "kernel"]
'''

CASES = {
    # one model alone: no events
    "one_model": r'''
a = model()
denoise(a, 0x10); events()
denoise(a, 0x10); denoise(a, 0x20)
assert [e[:2] for e in events()] == [("persist", 0x10), ("persist", 0x20)]
''',
    # two models: each launch between a wait for the last one's event and its own record
    "two_models": r'''
a, b = model(), model()
denoise(a, 0x10); denoise(b, 0x20); events()
denoise(a, 0x10); denoise(b, 0x20)
got = events()
assert [e[:2] for e in got] == [(w, s) for s in (0x10, 0x20) for w in ("wait", "persist", "record")], got
assert len({e[2] for e in got if e[0] != "persist"}) == 1, got
''',
    # a launch of one model while the other, with a kernel in flight, is being destroyed: until the device has
    # synchronised, it still waits for that kernel
    "destroy": r'''
a, b = model(), model()
denoise(a, 0x10); denoise(b, 0x20); denoise(b, 0x20); events()
def launch():
    denoise(a, 0x10)
    return 0
cb = SYNC(launch)
stub.stub_on_sync(cb)
b.close()
got = events()
assert [e[0] for e in got] == ["sync", "wait", "persist", "record"], got
denoise(a, 0x10)   # alone again
assert [e[0] for e in events()] == ["persist"]
''',
    # a captured call cannot wait for an event of work outside its capture: it goes in without events, in the
    # caller's order; a stream whose state cannot be told gets no launch at all
    "capture": r'''
a, b = model(), model()
denoise(a, 0x10); denoise(b, 0x20); events()
stub.stub_capture(1, 0)
denoise(a, 0x10)
assert [e[:2] for e in events()] == [("persist", 0x10)]
stub.stub_capture(0, 0)
denoise(b, 0x20)
assert [e[0] for e in events()] == ["wait", "persist", "record"]
stub.stub_capture(0, 906)
try:
    denoise(a, 0x10)
except vla.VlaError as e:
    assert vla.STATUS[e.status] == "VLA_E_DEVICE", e
else:
    raise AssertionError("accepted")
assert events() == []
denoise(a, 0)      # the null stream is never captured
assert [e[0] for e in events()] == ["wait", "persist", "record"]
''',
    # each device has its own order, whatever its number
    "devices": r'''
a, b = model(), model()
denoise(a, 0x10); denoise(b, 0x20)
for dev in (3, 70):
    stub.stub_device(dev)
    denoise(a, 0x10); events()
    denoise(b, 0x20)
    assert [e[0] for e in events()] == ["wait", "persist", "record"], dev
''',
}


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    if not os.path.exists(os.path.join(ROOT, "paper_2606_08094_amd", "libvla.so")):
        pytest.skip("libvla.so not built")
    so = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "hip_stub.c")], check=True)
    return so


@pytest.mark.parametrize("case", sorted(CASES))
def test_launch_order(stub, case):
    r = subprocess.run([sys.executable, "-c", PRELUDE + CASES[case], stub], cwd=ROOT, capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
