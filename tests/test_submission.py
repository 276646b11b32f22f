"""What is enqueued for a batch, and what its record says of it: host code, followed without a GPU.  tests/native/runtime_standin.cpp stands in for the HIP runtime and
keeps time: a kernel takes 5 us, a stamp 2, the host link brings 53 bytes a ns, the host takes none.  Every program runs in a process of its own.
"""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_28175_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"
pytestmark = pytest.mark.skipif(not os.path.exists(CLANG), reason="ROCm clang++ not found")

SETUP = """
import ctypes, sys
standin = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)            # ahead of the runtime that the library brings along
sys.path.insert(0, sys.argv[2])
import numpy as np
import paper_2604_28175_amd as S
from paper_2604_28175_amd import binding
import synth
standin.standin_notes.restype = ctypes.c_char_p
HP, LP, COPY = [0x1000], [0x2000], [0x3000, 0x4000]                     # streams: names, for the stand-in
def context(n_copy=2):
    d = binding.CtxDesc()
    d.device, d.n_hp, d.n_lp, d.n_copy = 0, 1, 1, n_copy
    d.hp_streams[0], d.lp_streams[0] = HP[0], LP[0]
    for i in range(n_copy):
        d.copy_streams[i] = COPY[i]
    c = S.Context.__new__(S.Context)
    c.handle = ctypes.c_void_p()
    assert binding.lib.strait_ctx_create(ctypes.byref(d), ctypes.byref(c.handle)) == 0
    return c
def notes():
    return [l.split() for l in standin.standin_notes().decode().splitlines()]
def lengths(md, batch):
    return np.full(batch, md.hyper[4], np.int32) if md.arch == synth.ARCH_ENCODER else None
"""


@pytest.fixture(scope="session")
def standin(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("standin") / "standin.so")
    subprocess.run([CLANG, "-std=c++17", "-O1", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    os.path.join(ROOT, "tests", "native", "runtime_standin.cpp"), "-o", lib], check=True)
    return lib


def run(standin, program):
    r = subprocess.run([sys.executable, "-c", SETUP + program, standin, ROOT], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
    return r.stdout


def test_parts_of_a_large_batch_begin_on_16_bytes(standin):
    """Images whose bytes, and token sequences whose statistics, are no multiples of 16: every staged batch of 9 MB and more is taken, in parts that the kernels can
    read, or whole."""
    out = run(standin, """
c = context()
took = {}
for name, md, batches in (("250", synth.mobilenet_v2(1, hw=250), list(range(24, 129))), ("226", synth.mobilenet_v2(1, hw=226), list(range(28, 129))),
                          ("30", synth.tiny_cnn(1, hw=30), [1746, 1747, 1801, 2500, 3000]), ("1250", synth.mobilenet_v2(1, hw=1250), [1, 2, 3, 4, 5, 9]),
                          ("sequences of 37", synth.encoder(1, layers=2, hidden=64, heads=1, ffn=256, seq=37), [2000, 2001, 2350]),
                          ("197 tokens of 192", synth.vit(1, hw=224, classes=100, layers=2, hidden=192, heads=3, ffn=768), list(range(31, 40)))):
    m = c.load(synth.pack(md), max(batches), 1)
    for b in batches:
        notes()
        m.wait(m.submit(S.PRIO_LOW, m.staging(0, b), lengths(md, b), m.new_output(b)))
        standin.standin_idle()
        n = notes()
        sent = [int(l[1]) for l in n if l[0] == "memcpy"]
        assert sum(sent) in (m.io_bytes(b)[0], 0), (name, b, sent)
        one = m.io_bytes(1)[0]
        assert all(s % one == 0 for s in sent)
        took[name] = max(took.get(name, 0), len(sent))
        starts = [sum(sent[:i]) for i in range(len(sent))]
        assert all(s % 16 == 0 for s in starts), (name, b, starts)
    m.free()
print(took)
assert took["250"] > 3 and took["226"] > 3 and took["30"] > 1 and took["sequences of 37"] > 1 and took["197 tokens of 192"] > 1
""")
    print(out)


def test_a_batch_is_done_when_its_input_s_end_is_stamped(standin):
    """The stamp that ends an input's transfer lies in front of what the kernels wait for, or, of an input in parts, is waited for itself: the record that is read holds
    this batch's, and a late stamp is not written into a later batch's."""
    run(standin, """
import time
c = context()
md = synth.mobilenet_v2(1)
m = c.load(synth.pack(md), 64, 1)
x = np.zeros((64, 224, 224, 3), np.float16)
for prio in (S.PRIO_LOW, S.PRIO_HIGH):
    notes()
    m.wait(m.submit(prio, x, None, m.new_output(64)))
    standin.standin_idle()
    n = notes()
    end = [i for i, l in enumerate(n) if l[:2] == ["stamp", "9"]]                    # (8 and 9: a transfer's start and end)
    assert len(end) == 1 and ["record", n[end[0]][2]] in [[l[0], l[2]] for l in n[end[0]:] if l[0] == "record"]
    for late in (True, False):
        if late:
            standin.standin_hold_stamp(9)
        t = m.submit(prio, m.staging(0, 64), None, m.new_output(64))
        assert sum(l[0] == "memcpy" for l in notes()) > 1
        if late:
            time.sleep(0.05)
            assert not m.poll(t)                                                     # its result is there
            standin.standin_release()
        r = m.wait(t)
        assert r.total_ms > 0
        standin.standin_idle()
""")


def test_a_batch_in_parts_counts_on_both_copy_streams(standin):
    """While a low-priority batch's parts are on both copy streams, another input finds neither of them empty, and a small high-priority one goes in on its compute
    stream, also where that has work: on a copy stream it would wait for half of the parts.  Everything is counted down again."""
    run(standin, """
c = context()
md, small = synth.mobilenet_v2(1), synth.resnet50(1)
lp = c.load(synth.pack(md), 128, 1)
big = c.load(synth.pack(md), 64, 2)
hp = c.load(synth.pack(small), 8, 3)
x = np.zeros((64, 224, 224, 3), np.float16)
for again in range(2):
    notes()
    standin.standin_hold()
    a = hp.submit(S.PRIO_HIGH, hp.staging(0, 8), None, hp.new_output(8))
    l = lp.submit(S.PRIO_LOW, lp.staging(0, 128), None, lp.new_output(128))
    assert sum(n[0] == "memcpy" for n in notes()) > 4
    b = hp.submit(S.PRIO_HIGH, hp.staging(1, 8), None, hp.new_output(8))             # behind the first, on a stream that is not idle
    assert [n[2] for n in notes() if n[0] == "copy_in"] == ["0x1000"]
    o = big.submit(S.PRIO_LOW, x, None, big.new_output(64))                          # ordinary memory: pieces only where the stream is empty
    sent = [n for n in notes() if n[0] == "memcpy"]
    assert len(sent) == 1, sent
    standin.standin_release()
    for m, t in ((hp, a), (hp, b), (lp, l), (big, o)):
        m.wait(t)
    standin.standin_idle()
    notes()
    big.wait(big.submit(S.PRIO_LOW, x, None, big.new_output(64)))
    assert sum(n[0] == "memcpy" for n in notes()) > 1                                # alone again
    standin.standin_hold()
    a = hp.submit(S.PRIO_HIGH, hp.staging(0, 8), None, hp.new_output(8))
    b = hp.submit(S.PRIO_HIGH, hp.staging(1, 8), None, hp.new_output(8))
    standin.standin_release()
    assert [n[2] in ("0x3000", "0x4000") for n in notes() if n[0] == "copy_in"] == [False, True]
    hp.wait(a), hp.wait(b)
    standin.standin_idle()
""")


def test_what_the_scheduling_policy_is_fed_is_a_transfer_and_then_kernels(standin):
    """The policy adds a batch's transfer to its kernels (Eq. 1 to 3, 6).  Profiles, and batches of the serving front end, are not begun before their input is complete."""
    run(standin, """
c = context()
md, batch = synth.mobilenet_v2(1), 64
m = c.load(synth.pack(md), batch, 1)
def kernels_us(n):
    first, last = [i for i, l in enumerate(n) if l[0] == "memcpy"][0], [i for i, l in enumerate(n) if l[0] == "memcpy"][-1]
    return 5 * sum(l[0] == "kernel" for l in n), first == last
notes()
m.wait(m.submit(S.PRIO_LOW, m.staging(0, batch), None, m.new_output(batch)))         # a program's own: in parts
standin.standin_idle()
parted, whole = kernels_us(notes())
assert not whole
p = S.profile_model(m, S.PRIO_LOW, batch, 1)
n = notes()
us = 5 * sum(l[0] == "kernel" for l in n) / 4                                       # three to warm up, one that counts
assert sum(l[0] == "memcpy" for l in n) == 4
assert abs(p.t_kernel_isol_ns - 1e3 * us) <= 2e3 + 10 and us < parted, (p.t_kernel_isol_ns, us, parted)
standin.standin_idle()
sched = S.Scheduler(1)
profs = [(1e6, 1000, 1e6, [0.1] * 5, 0.1, 0.1)] * batch
sched.set_profile(7, S.PRIO_LOW, profs)
srv = S.Server(sched, 2, 100000)
srv.add_model(m, 7, S.PRIO_LOW, batch, 10_000_000_000, 50_000_000)
x, out = np.zeros((batch, 224, 224, 3), np.float16), np.zeros((batch, m.io_bytes(1)[1]), np.uint8)
srv.start()
warm = notes()
assert max(int(l[1]) for l in warm if l[0] == "memcpy") == m.io_bytes(batch)[0]
for i in range(batch):
    srv.request(7, x[i], out[i])
srv.wait_idle(20.0)
n = notes()
assert sum(int(l[1]) for l in n if l[0] == "memcpy") == m.io_bytes(batch)[0]
assert sum(l[0] == "memcpy" for l in n) == 1, [l for l in n if l[0] == "memcpy"]
r = srv.results()
assert len(r) == batch and all(q.status == 0 and q.batch == batch for q in r), [(q.status, q.batch) for q in r]
srv.stop()
""")


def test_a_result_leaves_by_sixteen_workgroups_where_nothing_runs_beside_it(standin):
    """Eight leave the launches of other streams' batches alone, but take up to 15 % longer."""
    run(standin, """
c = context()
md, small = synth.encoder(1, layers=1), synth.resnet50(1)
m, hp = c.load(synth.pack(md), 64, 3), c.load(synth.pack(small), 8, 1)
def out_grids():
    return [int(l[-1]) for l in notes() if l[0] == "copy_out" and int(l[1]) > 1 << 20]
def batch(i, b):
    return m.submit(S.PRIO_LOW, m.staging(i, b), lengths(md, b), m.new_output(b))
for b in (8, 64):                                                                    # behind its kernels; on a copy stream
    notes()
    m.wait(batch(0, b))
    assert out_grids() == [16], b
    standin.standin_hold()
    two = [batch(i, b) for i in range(2)]                                            # one behind the other on one stream
    standin.standin_release()
    for t in two:
        m.wait(t)
    assert out_grids() == [16, 16] if b == 8 else 8 in out_grids(), b                # (of the second nothing is left when the first is through, or it is)
    standin.standin_idle()
standin.standin_hold()
h = hp.submit(S.PRIO_HIGH, hp.staging(0, 8), None, hp.new_output(8))
t = batch(0, 8)
standin.standin_release()
m.wait(t), hp.wait(h)
assert out_grids() == [8]
""")
