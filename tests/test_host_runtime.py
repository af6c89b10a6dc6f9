"""The library's host code without a device: a child process runs it on the
runtime of fake_hip.c (device memory in host memory, kernels that only enter a
log), so that slot bounds, launch shapes and failure paths can be looked at."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes as C
import numpy as np
from paper_2406_14512_amd import ffpic
from paper_2406_14512_amd import workloads as W
F = C.CDLL(None)
F.fake_name.restype = C.c_char_p
F.fake_grid.restype = C.c_uint32
F.fake_h2d4.restype = C.POINTER(C.c_int32)
F.fake_fail.argtypes = [C.c_char_p]

def launches(part):
    names = [F.fake_name(k).decode() for k in range(F.fake_count())]
    return [(n, F.fake_grid(k, 0), F.fake_grid(k, 1)) for k, n in enumerate(names) if part in n]

def system(precision, n, cap=None, nth=64, **over):
    w = W.tiny_dipole(n)
    w.nr = w.nth = nth
    d = w.desc()
    d["precision"] = precision
    d.update(over)
    sim = ffpic.Sim(d, capacity=[cap or n] * 2)
    for s in range(2):
        sim.load_particles(s, w.particles(s))
    F.fake_clear()
    return w, sim
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    from paper_2406_14512_amd import ffpic
    try:
        ffpic.lib()
    except ImportError:
        from paper_2406_14512_amd import build
        build.build()
    so = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.run(["gcc", "-O1", "-w", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "fake_hip.c")], check=True)

    def run(body):
        env = dict(os.environ, LD_PRELOAD=so, PYTHONPATH=ROOT)
        env.pop("FFPIC_TUNING_CACHE", None)
        r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body)], env=env,
                           cwd=ROOT, capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
    return run


@pytest.mark.parametrize("precision", [0, 1])
def test_load_appends_behind_the_devices_count(fake, precision):
    """A sort on the device lowers its slot count and not the host's bound: a
    load after it appends at the count, or the slots between the two, which
    hold stale particles, would be sorted in as live."""
    fake(f"""
    w, sim = system({precision}, 100, cap=200)
    count = F.fake_h2d4()              # of species 1, the last one loaded
    assert count[0] == 100 and sim.n(1) == 100
    count[0] = 60                      # forty left, and a sort dropped them
    p = w.particles(1)
    sim.load_particles(1, {{k: v[:10] for k, v in p.items()}})
    assert sim.n(1) == 70, sim.n(1)
    """)


@pytest.mark.parametrize("precision", [0, 1])
def test_failed_copies_are_waited_for(fake, precision):
    """A call whose k-th queued copy is refused returns the error after waiting
    for the ones before it, which read or write the caller's memory."""
    fake(f"""
    w, sim = system({precision}, 50, cap=100)
    image = sim.save()
    p = w.particles(1)
    calls = dict(
        save=sim.save, restore=lambda: sim.restore(image), field=lambda: sim.field(ffpic.ER),
        particles=lambda: sim.particles(0), diagnostics=lambda: sim.diagnostics(poynting=True),
        load=lambda: sim.load_particles(1, {{k: v[:10] for k, v in p.items()}}))
    for name, call in calls.items():
        failed = 0
        for k in range(100):
            F.fake_clear()
            F.fake_fail_copy(k)
            try:
                call()
            except ffpic.FfpicError as e:
                assert e.code == ffpic.EHIP
                assert F.fake_copies_pending() == 0, (name, k)
                failed += 1
            else:
                break
        assert failed >= 2, name
        F.fake_fail_copy(-1)
    """)


@pytest.mark.parametrize("precision", [0, 1])
def test_failed_capture_leaves_no_placement(fake, precision):
    """A capture that ends between a step's sort and its push never ran: the
    next push is a plain one, and places by no order."""
    fake(f"""
    w, sim = system({precision}, 50)
    F.fake_fail(b"k_push")
    try:
        sim.step(1)
        assert False
    except ffpic.FfpicError as e:
        assert e.code == ffpic.EHIP
    assert launches("k_bucket_dest"), "the sort left its placement to the push"
    F.fake_fail(b"")
    F.fake_clear()
    sim.run_phases(ffpic.PHASE_PUSH)
    push = launches("k_push")
    assert push and all("Lb0EE" in n for n, _, _ in push), push
    """)


@pytest.mark.parametrize("mode,kernel", [(1, "k_push32IL"), (2, "k_push32_group")])
def test_failed_batch_capture_leaves_no_placement(fake, mode, kernel):
    fake(f"""
    w = W.tiny_dipole(50)
    w.nr = w.nth = 64
    d = w.desc()
    d["precision"] = 1
    b = ffpic.Batch([d, d], [[50, 50]] * 2)
    for v in b.views:
        for s in range(2):
            v.load_particles(s, w.particles(s))
    b.set_graph({mode})
    F.fake_clear()
    F.fake_fail(b"{kernel}")
    try:
        b.step(1)
        assert False
    except ffpic.FfpicError as e:
        assert e.code == ffpic.EHIP
    assert launches("k_bucket_dest") and launches("{kernel}")
    F.fake_fail(b"")
    for v in b.views:
        F.fake_clear()
        v.run_phases(ffpic.PHASE_PUSH)
        push = launches("k_push32")
        assert push and all("Lb0EE" in n for n, _, _ in push), push
    """)


def test_push_chunk_setting_is_taken(fake):
    """ffpic_set_push_chunk gives the particles per thread of every push, also of
    species that would take fewer without it (one, for 1e5 slots)."""
    fake("""
    n = 50_000
    w, sim = system(1, n)
    sim.run_phases(ffpic.PHASE_PUSH)
    assert [g for _, *g in launches("k_push32")] == [[-(-n // 256), 2]]
    for ppt in (8, 16, 32):
        sim.set_push_chunk(ppt)
        F.fake_clear()
        sim.run_phases(ffpic.PHASE_PUSH)
        assert [g for _, *g in launches("k_push32")] == [[-(-n // (256 * ppt)), 2]], ppt
        F.fake_clear()
        sim.step(1)            # no graph captured with another chunk is replayed
        assert [g for _, *g in launches("k_push32")] == [[-(-n // (256 * ppt)), 2]], ppt
    """)


def test_grouped_push_chunk_setting_is_taken(fake):
    fake("""
    n = 50_000
    w = W.tiny_dipole(n)
    w.nr = w.nth = 64
    d = w.desc()
    d["precision"] = 1
    b = ffpic.Batch([d, d], [[n, n]] * 2)
    for v in b.views:
        for s in range(2):
            v.load_particles(s, w.particles(s))
    b.set_graph(2)
    items = {0: 4 * -(-n // 256)}
    items.update({p: 4 * -(-n // (256 * p)) for p in (8, 16, 32)})
    for ppt in (0, 8, 16, 32):
        b.set_grouped_chunk(ppt)
        F.fake_clear()
        b.step(1)
        assert [g[0] for _, *g in launches("k_push32_group")] == [min(items[ppt], 1024)], ppt
    """)


def test_tuner_times_only_chunks_that_differ(fake):
    fake("""
    w, sim = system(1, 50_000)
    t = sim.autotune(1e9)
    assert list(t["timed"]["push_ppt"]) == [16] and t["push_ppt"] == 16, t
    sim.set_push_chunk(8)
    t = sim.autotune(1e9)
    assert list(t["timed"]["push_ppt"]) == [16] and t["push_ppt"] == 16, t
    F.fake_clear()
    sim.run_phases(ffpic.PHASE_PUSH)
    assert [g for _, *g in launches("k_push32")] == [[-(-50_000 // 256), 2]]
    """)
