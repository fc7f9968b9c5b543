"""Whose scratch a call that is spread over workgroups uses, asked on the host: tests/host/scratch_driver.cpp stands in for the HIP
runtime and prints what each call asks of it (no kernel runs and no device is needed)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LIB_DIR = os.path.join(ROOT, "paper_2503_14985_amd")
CALLS = ("gemm", "tiles", "tall", "mha", "paged", "few")       # decode GEMM, tile GEMM (and of 44 rows), attention, paged decode in many ranges and in few


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    exe = str(tmp_path_factory.mktemp("scratch") / "scratch_driver")
    cmd = [HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-x", "hip", os.path.join(ROOT, "tests", "host", "scratch_driver.cpp"),
           "-x", "none", "-o", exe, os.path.join(LIB_DIR, "libmlt.so"), "-Wl,-rpath," + LIB_DIR, "-pthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    env = {k: v for k, v in os.environ.items() if not k.startswith("MLT_")}

    def run(calls):
        """[(call, stream)] -> [(kernel, events)], in one process"""
        r = subprocess.run([exe], input="".join("%s %s\n" % c for c in calls), capture_output=True, text=True, timeout=600, env=env)
        assert r.returncode == 0, r.stderr[-2000:]
        out = [line.split(": ") for line in r.stdout.splitlines()]
        assert len(out) == len(calls) and all(head.startswith("0 ") for head, _ in out), r.stdout
        return [(head[2:], events.split()) for head, events in out]
    return run


def launches(events):
    return [e for e in events if e[0] == "L"]


@pytest.mark.parametrize("call", CALLS)
def test_a_stream_keeps_its_own_buffer(ask, call):
    """Allocated at the first call of each stream (and its counters zeroed there by one launch), then kept."""
    got = ask([(call, s) for s in ("0", "0", "1", "2", "1", "2", "0")])
    plain = [e[0] for e in got[1][1]]
    assert "split" in got[0][0] and plain in (["L"], ["L", "L"])
    for i, (name, events) in enumerate(got):
        assert name == got[0][0] and [e[0] for e in events] == (["A", "L"] if i in (0, 2, 3) else []) + plain


@pytest.mark.parametrize("call", CALLS)
def test_each_thread_has_its_own_buffer_on_hip_stream_per_thread(ask, call):
    """One handle, but another stream in each thread: with one buffer for the handle, calls that overlap would write and read it at
    the same time."""
    ref, *got = ask([(call, "0"), (call, "0")] + [(call, "P%d" % t) for t in (1, 1, 2, 2, 2, 3)])[1:]
    for i, (name, events) in enumerate(got):
        assert name == ref[0] and events == (["A", "LP"] if i in (0, 2, 5) else []) + ["LP"] * len(ref[1])


@pytest.mark.parametrize("call", CALLS)
def test_more_threads_than_buffers(ask, call):
    """From the 33rd thread on a GEMM brings memory of its own (and a second kernel adds its parts), the others run unsplit; the
    streams' buffers are not used up by threads."""
    *got, last = ask([(call, "P%d" % t) for t in range(34)] + [(call, "5")])
    assert [events[0] for _, events in got] == ["A"] * 32 + [got[32][1][0]] * 2
    assert got[32][1] == (["aP", "LP", "LP", "fP"] if call in ("gemm", "tiles", "tall") else ["LP"]) and last[1][0] == "A"


@pytest.mark.parametrize("call", CALLS)
def test_a_call_that_is_recorded_allocates_nothing(ask, call):
    (_, events), = ask([(call, "c")])
    assert len(launches(events)) == len(events) == 1


def test_a_recorded_call_without_its_split_takes_the_kernel_that_is_better_without(ask):
    """44 x 7296 x 11456: four parts on 64 x 128 tiles; not split the streaming kernel takes half the time."""
    (tiles, _), (stream, _) = ask([("tall", "0"), ("tall", "c")])
    assert tiles == "gemm_nt_64x128x64_w2x4_k2_splitk4" and stream == "gemm_nt_skinny_stream"
