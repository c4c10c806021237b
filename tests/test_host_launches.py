"""What the library's host side allocates, frees, waits for and launches, in
which order, on the CPU: a child process loads libccl.so over a stand-in for
the HIP runtime (hip_recorder.cpp) that logs those calls and runs no kernel."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1712_09789_amd", "libccl.so")

PRELUDE = """
import collections, ctypes, sys, threading
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
p, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
rec.rec_limit.argtypes = [i64]
rec.rec_take.argtypes, rec.rec_take.restype = [ctypes.c_char_p, i64], i64
lib.ccl_label.argtypes = [p, i32, i32, i64, i32, p, p]
lib.ccl_label_3d.argtypes = [p, i32, i32, i32, i64, i64, i32, p, p]
lib.ccl_replay_last.argtypes = [i32, i32, p]
IN, OUT = 1 << 32, 1 << 36
Event = collections.namedtuple("Event", "what thread stream ptr value")

def take():
    buf = ctypes.create_string_buffer(1 << 22)
    assert rec.rec_take(buf, len(buf)) < len(buf)
    rows = [l.split() for l in buf.value.decode().splitlines()]
    return [Event(w, int(t), int(s, 16), int(a, 16), int(v)) for w, t, s, a, v in rows]

def image(H, W, conn=8, stream=None, at=0):
    assert lib.ccl_label(IN + at, H, W, W, conn, OUT + 4 * at, stream) == 0

def volume(D, H, W, conn=26, stream=None, at=0):
    assert lib.ccl_label_3d(IN + at, D, H, W, W, H * W, conn, OUT + 4 * at, stream) == 0
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rec") / "libhip_recorder.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-w", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_1712_09789_amd", "csrc"),
                    os.path.join(ROOT, "tests", "hip_recorder.cpp"), "-o", out], check=True)

    def run(code):
        r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(code), out, LIB],
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr

    return run


@pytest.mark.parametrize("H,W,grouped", [(4096, 4096, 1), (200, 200, 1), (640, 480, 0), (50, 60, 0)])
def test_relabel_after_a_replayed_local_step_follows_nodes(recorder, H, W, grouped):
    # the relabel takes the slots for forest nodes: the launch that wrote them
    # last has to be a local step without merge groups, or the merge itself
    recorder(f"""
        image({H}, {W})
        first = [e for e in take() if e.what.startswith("launch")]
        assert any(e.what == "launch:k_block" for e in first) == bool({grouped})
        for kinds in ((0, 2), (0, 0, 2, 2), (2, 0, 2), (0, 2, 0, 2)):
            image({H}, {W})
            for k in kinds:
                assert lib.ccl_replay_last(k, 2, None) == 0
        image({H}, {W})
        lib.ccl_replay_last(2, 1, None)
        nodes = False
        for e in take():
            if e.what == "launch:k_local":
                nodes = e.value == 0
            elif e.what == "launch:k_block":
                nodes = True
            elif e.what == "launch:k_final":
                assert nodes
    """)


def test_replays_launch_that_kernel_alone(recorder):
    recorder("""
        image(4096, 4096)
        take()
        lib.ccl_replay_last(2, 3, None)
        assert [e.what for e in take()] == ["launch:k_final"] * 3
        lib.ccl_replay_last(0, 3, None)
        assert [e.what for e in take()] == ["launch:k_local"] * 3
        lib.ccl_replay_last(2, 0, None)
        assert take() == []
    """)


@pytest.mark.parametrize("call", ["volume(64, 64, 64, 6, st, at)", "volume(64, 64, 64, 26, st, at)",
                                  "image(1500, 1600, 8, st, at)", "image(300, 300, 4, st, at)"])
@pytest.mark.parametrize("st", [None, 0x5000])
def test_calls_of_two_threads_on_one_stream_do_not_mix(recorder, call, st):
    # the launches of a call share a workspace with those of every other call
    # on the stream, so no other call's may come between them
    recorder(f"""
        st = {st}
        def calls(at):
            for _ in range(12):
                {call}
        calls(0)
        per_call = len([e for e in take() if e.what.startswith("launch")]) // 12
        assert per_call >= 3
        rec.rec_delay_us(300)
        threads = [threading.Thread(target=calls, args=(t << 20,)) for t in (1, 2, 3)]
        for t in threads: t.start()
        for t in threads: t.join()
        log = [e for e in take() if e.what.startswith("launch")]
        assert len(log) == 3 * 12 * per_call
        for i in range(0, len(log), per_call):
            assert len({{e.thread for e in log[i:i + per_call]}}) == 1, log[i:i + per_call]
        assert len({{e.thread for e in log}}) == 3
    """)


@pytest.mark.parametrize("conn", [6, 26])
def test_a_workspace_is_in_nobodys_use_when_it_is_freed(recorder, conn):
    # threads label growing volumes on one stream and on others while another
    # one gives the workspaces back: a launch uses a buffer that is there, and a
    # buffer goes after a wait that follows its last launch
    recorder(f"""
        rec.rec_delay_us(100)
        def calls(st, at):
            for k in range(1, 13):
                volume(16 * k, 32, 64, {conn}, st, at)
                image(70 * k, 300, 8, st, at)
        def release():
            for _ in range(20):
                assert lib.ccl_release_workspace(0) == 0
        threads = [threading.Thread(target=calls, args=(st, t << 24)) for t, st in
                   enumerate((0x5000, 0x5000, 0x6000))] + [threading.Thread(target=release)]
        for t in threads: t.start()
        for t in threads: t.join()
        lib.ccl_release_workspace(0)
        size, freed = {{}}, 0
        dirty = set()  # (stream, workspace) of launches not waited for
        for e in take():
            if e.what == "malloc":
                size[e.ptr] = e.value
            elif e.what.startswith("launch"):
                assert any(b <= e.ptr < b + n for b, n in size.items()), e
                dirty.add((e.stream, e.ptr))
            elif e.what == "wait":
                dirty = {{d for d in dirty if d[0] != e.stream}}
            elif e.what == "wait_device":
                dirty.clear()
            elif e.what == "free":
                n = size.pop(e.ptr)
                assert not any(e.ptr <= at < e.ptr + n for _, at in dirty), e
                freed += 1
        assert freed > 3 and not size
    """)


@pytest.mark.parametrize("conn", [6, 26])
def test_volumes_on_the_per_thread_stream_share_nothing(recorder, conn):
    # hipStreamPerThread is one handle for a stream of each thread
    recorder(f"""
        volume(64, 64, 64, {conn}, 2)
        assert [e.what for e in take()] == ["launch:k_vlocal", "launch:k_vmerge", "launch:k_vfinal"]
    """)


@pytest.mark.parametrize("conn", [6, 26])
def test_volumes_without_a_workspace_are_labelled_in_place(recorder, conn):
    # no memory for a first workspace, then for a larger one; the call succeeds,
    # and goes back to a workspace once it can be had
    recorder(f"""
        here = ["launch:k_vlocal", "launch:k_vmerge", "launch:k_vfinal"]
        there = ["launch:k_wlocal", "launch:k_wmerge", "launch:k_wfinal"]
        launches = lambda: [e.what for e in take() if e.what.startswith("launch")]
        rec.rec_limit(1000)
        volume(64, 64, 64, {conn})
        assert launches() == here
        rec.rec_limit(1 << 40)
        volume(64, 64, 64, {conn})
        assert launches() == there
        rec.rec_limit(1000)
        volume(200, 300, 300, {conn})
        assert launches() == here
        rec.rec_limit(1 << 40)
        volume(200, 300, 300, {conn})
        assert launches() == there
    """)


@pytest.mark.parametrize("conn,per_brick", [(6, 37460), (26, 14036)])
def test_kept_volume_workspaces_are_reported(recorder, conn, per_brick):
    recorder(f"""
        for f in (lib.ccl_workspace_cached, lib.ccl_volume_workspace_cached):
            f.argtypes, f.restype = [p], i64
        held = lambda st=None: (lib.ccl_workspace_cached(st), lib.ccl_volume_workspace_cached(st))
        assert held() == (0, 0)
        image(300, 300)
        images = held()[0]
        assert images > 0 and held()[1] == 0
        take()
        volume(33, 40, 70, {conn})  # 3 x 3 x 2 bricks
        allocated = sum(e.value for e in take() if e.what == "malloc")
        assert held() == (images, allocated) and held(0x5000) == (0, 0)
        need = 18 * {per_brick}
        assert 1.25 * need <= allocated <= 1.25 * (need + 5 * 256)
        volume(16, 16, 64, {conn})
        assert held() == (images, allocated)
        lib.ccl_release_workspace(0)
        assert held() == (0, 0)
    """)


@pytest.mark.parametrize("conn", [6, 26])
def test_rules_of_the_volume_paths(recorder, conn):
    # 32 rows; more than 4096 bricks less than a third full
    recorder(f"""
        for shape, path in (((1, 31, 500), "v"), ((1, 32, 500), "w"), ((31, 1, 500), "v"),
                            ((4, 8, 500), "w"), ((2, 16, 64 * 4096), "w"),
                            ((2, 16, 64 * 4096 + 1), "v"), ((6, 16, 64 * 4096 + 1), "w")):
            volume(*shape, {conn})
            got = [e.what for e in take() if e.what.startswith("launch")]
            assert got and all(k.startswith("launch:k_" + path) for k in got), (shape, got)
    """)
