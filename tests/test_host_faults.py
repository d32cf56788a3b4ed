"""Error paths and waits of the library's host code, on the CPU: its four translation units compiled against a HIP runtime on host
memory (fake_hip.cpp) in which any call can be made to fail."""
import ctypes as C
import os
import random
import subprocess
import threading

import numpy as np
import pytest

from paper_2211_13939_amd import binding, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
N_MEL = synth.DIMS["n_mel"]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake") / "libfake.so")
    csrc = os.path.join(ROOT, "paper_2211_13939_amd", "csrc")
    # -Bsymbolic: the HIP runtime of this process is not in the way
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    # (the HIP compiler's own words, in postnet.cpp)
                    "-Wno-unused-result", "-D__align__(n)=__attribute__((aligned(n)))", "-DHIP_SYMBOL(x)=((const void*)x)", os.path.join(ROOT, "tests", "fake_hip.cpp")]
                   + [os.path.join(csrc, f) for f in ("tts_pool.cpp", "encoder.cpp", "postnet.cpp", "vocoder.cpp")] + ["-o", out], check=True)
    L = C.CDLL(out)
    for f in ("pool", "encoder", "postnet", "vocoder"):
        getattr(L, f"tts_{f}_workspace_bytes").restype = C.c_size_t
    L.tts_last_error.restype = C.c_char_p
    for f in ("tts_pool_destroy", "tts_encoder_destroy", "tts_postnet_destroy", "tts_vocoder_destroy"):
        getattr(L, f).restype = None
        getattr(L, f).argtypes = [C.c_void_p]
    L.fake_fail.argtypes = [C.c_char_p, C.c_int, C.c_int]
    L.fake_calls.argtypes = [C.c_char_p]
    L.fake_capture.argtypes = [C.c_void_p]
    return L


@pytest.fixture(autouse=True)
def _reset(lib):
    lib.fake_reset()


def _arena(nbytes):
    raw = np.zeros(nbytes + 256, np.uint8)
    return raw, C.c_void_p(raw.ctypes.data + (-raw.ctypes.data) % 256)


class FakePool:
    def __init__(self, lib, weights, max_pool=4, max_steps=64, chunk=8, stream=1, segments=False, max_enc_len=16, bf16=None):
        self.L, self.chunk = lib, chunk
        cfg = binding.make_config(synth.DIMS, max_pool=max_pool, max_enc_len=max_enc_len, max_steps=max_steps, chunk_frames=chunk, use_graph=segments,
                                  bf16=segments if bf16 is None else bf16)
        n = int(lib.tts_pool_workspace_bytes(C.byref(cfg)))
        self._arena, at = _arena(n)
        w = binding.TtsWeights(*[weights[k].ctypes.data_as(C.POINTER(C.c_float)) for k in binding.WEIGHT_FIELDS])
        self.h = C.c_void_p()
        assert lib.tts_pool_create(C.byref(cfg), C.byref(w), at, C.c_size_t(n), C.c_void_p(stream), C.byref(self.h)) == 0, lib.tts_last_error()

    def add(self, n_steps, length=3):
        enc, rid = np.zeros((length, synth.DIMS["enc_dim"]), np.float32), C.c_int64()
        assert self.L.tts_pool_add_request(self.h, enc.ctypes.data_as(C.c_void_p), length, n_steps, C.byref(rid)) == 0
        return rid.value

    def step_n(self, n):
        assert self.L.tts_pool_step_n(self.h, n, None) == 0

    def sync(self):
        assert self.L.tts_pool_sync(self.h) == 0

    def drain(self, rid):
        """(status, first value of every frame, finished)"""
        buf, n, fin = np.full((self.chunk, N_MEL), np.nan, np.float32), C.c_int(-1), C.c_int(-1)
        rc = self.L.tts_pool_drain_chunk(self.h, C.c_int64(rid), buf.ctypes.data_as(C.c_void_p), C.byref(n), C.byref(fin))
        if rc:
            return rc, None, None
        got = buf[:n.value]
        assert (got == got[:, :1]).all()
        return rc, got[:, 0].tolist(), bool(fin.value)

    def close(self):
        self.L.tts_pool_destroy(self.h)


def _frames(n_steps, first, count):
    return [1000.0 * n_steps + f for f in range(first, first + count)]


class FakeEncoder:
    def __init__(self, lib):
        self.L = lib
        cfg = binding.make_encoder_config(max_tokens=64, max_len=64)
        w = binding.TtsEncoderWeights()
        src = synth.make_encoder_weights()
        keep = self._keep = []

        def ptr(a):
            keep.append(np.ascontiguousarray(a, np.float32))
            return keep[-1].ctypes.data_as(C.POINTER(C.c_float))

        for t in range(4):
            w.tables[t] = ptr(src["tables"][t])
        for i in range(3):
            w.conv_w[i], w.conv_b[i] = ptr(src["conv_w"][i]), ptr(src["conv_b"][i])
        for d, k in enumerate("fb"):
            w.w_ih[d], w.w_hh[d], w.b[d] = ptr(src["w_ih_" + k]), ptr(src["w_hh_" + k]), ptr(src["b_" + k])
        n = int(lib.tts_encoder_workspace_bytes(C.byref(cfg)))
        self._arena, at = _arena(n)
        self.h = C.c_void_p()
        assert lib.tts_encoder_create(C.byref(cfg), C.byref(w), at, C.c_size_t(n), C.c_void_p(1), C.byref(self.h)) == 0, lib.tts_last_error()

    def run(self):
        ids, lens = synth.encoder_ids(7, 1).astype(np.int32), np.array([7], np.int32)
        out = np.zeros((7, 512), np.float32)
        return self.L.tts_encoder_run(self.h, ids.ctypes.data_as(C.POINTER(C.c_int)), lens.ctypes.data_as(C.POINTER(C.c_int)), 1,
                                      out.ctypes.data_as(C.c_void_p))

    def close(self):
        self.L.tts_encoder_destroy(self.h)


@pytest.mark.parametrize("before", [0, 1, 2, 3])
@pytest.mark.parametrize("what,nth", [("launch_encoder", 1), ("hipEventRecord", 2)])
def test_encoder_call_that_fails_on_the_way_is_through_with_its_ids(lib, before, what, nth):
    """A call whose launches fail after the first kernel has been queued: that kernel still reads the ids in pinned memory, which
    neither the next call may rewrite nor the end of the encoder free before the stream has got there."""
    enc = FakeEncoder(lib)
    for _ in range(before):
        assert enc.run() == 0
    lib.fake_fail(what.encode(), nth, 1)
    assert enc.run() == binding.TTS_E_HIP
    for _ in range(3):
        assert enc.run() == 0
    assert lib.fake_violations() == 0
    lib.fake_fail(what.encode(), nth, 1)
    assert enc.run() == binding.TTS_E_HIP
    enc.close()
    assert lib.fake_violations() == 0


def test_drain_whose_bookkeeping_fails_leaves_no_chunk_behind_that_was_never_made(lib, weights_fp32):
    """Slot 1 is frozen after 5 frames of a step call of 8.  The drain of request 0 brings both chunks to the host, sees the
    fault and fails to read what the device lost: request 1's chunk of 8 frames, 3 of them never made, must not be handed out."""
    pool = FakePool(lib, weights_fp32)
    a, b = pool.add(24), pool.add(23)
    lib.fake_freeze(1, 5)
    pool.step_n(8)
    lib.fake_fail(b"hipMemcpyAsync", 1, 1)
    assert pool.drain(a)[0] == binding.TTS_E_HIP
    assert pool.drain(b) == (0, _frames(23, 0, 5), True)
    assert pool.drain(a) == (0, _frames(24, 0, 8), False)
    pool.step_n(16)
    assert pool.drain(a) == (0, _frames(24, 8, 8), False)
    assert pool.drain(a) == (0, _frames(24, 16, 8), True)
    assert pool.drain(b) == (0, [], True)
    pool.close()


def test_what_the_device_lost_is_not_forgotten_by_a_wait_that_fails(lib, weights_fp32):
    """Slot 1 is frozen after 5 frames of 8.  The wait for the device's marks fails: the next call still finds them."""
    pool = FakePool(lib, weights_fp32)
    a, b = pool.add(24), pool.add(23)
    lib.fake_freeze(1, 5)
    pool.step_n(8)
    lib.fake_fail(b"hipStreamSynchronize", 2, 1)          # (the first wait is the chunks')
    assert pool.drain(a)[0] == binding.TTS_E_HIP
    assert pool.drain(b) == (0, _frames(23, 0, 5), True)
    pool.close()


@pytest.mark.parametrize("times", [1, 2])
def test_pool_without_pinned_memory_for_its_chunks(lib, weights_fp32, times):
    """Where the pinned staging buffer cannot be had (the second pinned allocation; the first is the status word), the pool makes
    do with less of it, or none: it is created, and its drains hand out the same frames."""
    lib.fake_fail(b"hipHostMalloc", 2, times)
    pool = FakePool(lib, weights_fp32)
    a, b = pool.add(20), pool.add(11)
    pool.step_n(8)
    assert pool.drain(a) == (0, _frames(20, 0, 8), False)
    assert pool.drain(a) == (0, [], False)
    pool.step_n(12)
    assert pool.drain(b) == (0, _frames(11, 0, 8), False)
    assert pool.drain(a) == (0, _frames(20, 8, 8), False)
    assert pool.drain(b) == (0, _frames(11, 8, 3), True)
    assert pool.drain(a) == (0, _frames(20, 16, 4), True)
    c = pool.add(24)
    lib.fake_freeze(2, 5)
    pool.step_n(8)
    assert pool.drain(c) == (0, _frames(24, 0, 5), True)
    pool.close()


def test_every_drain_that_hands_out_frames_waits_for_the_stream(lib, weights_fp32):
    """A caller may take a drain that handed out frames for a wait, also when an earlier drain had brought the chunk along; and a
    request that further steps have frozen meanwhile is reported as finished by that drain already."""
    pool = FakePool(lib, weights_fp32)
    a, b = pool.add(24), pool.add(23)
    pool.step_n(8)
    for rid in (a, b):
        before = lib.fake_calls(b"hipStreamSynchronize")
        assert pool.drain(rid)[1] == _frames(24 if rid == a else 23, 0, 8)
        assert lib.fake_calls(b"hipStreamSynchronize") > before
    pool.step_n(8)
    assert pool.drain(a) == (0, _frames(24, 8, 8), False)         # brings b's frames 8 .. 15 along
    lib.fake_freeze(1, 16)
    pool.step_n(8)
    assert pool.drain(b) == (0, _frames(23, 8, 8), True)
    lib.fake_fail(b"hipStreamSynchronize", 1, 1)
    assert pool.drain(a)[0] == binding.TTS_E_HIP
    assert pool.drain(a) == (0, _frames(24, 16, 8), True)
    pool.close()


def test_pools_of_one_thread_that_are_waited_for_cost_each_other_nothing(lib, weights_fp32):
    """Pools whose steps are segments (two-byte) and one whose steps are launches of their own, each waited for before the next is used:
    nothing is recorded and nobody waits."""
    pools = [FakePool(lib, weights_fp32, stream=1, segments=True), FakePool(lib, weights_fp32, stream=2, segments=True),
             FakePool(lib, weights_fp32, stream=3)]
    before = [lib.fake_calls(f) for f in (b"hipEventRecord", b"hipStreamWaitEvent")]
    for k in range(3):
        for p in pools:
            rid = p.add(8)
            p.step_n(8)
            assert p.drain(rid) == (0, _frames(8, 0, 8), True)
    assert lib.fake_segments() == 6 and lib.fake_unordered() == 0
    assert [lib.fake_calls(f) for f in (b"hipEventRecord", b"hipStreamWaitEvent")] == before
    for p in pools:
        p.close()


@pytest.mark.parametrize("busy", [0, 1])
def test_segments_of_several_pools_follow_each_other(lib, weights_fp32, busy):
    """One thread, nobody waited for: a segment is ordered behind the other pools' launches so far, a step behind their segments."""
    lib.fake_busy(busy)
    pools = [FakePool(lib, weights_fp32, stream=1, segments=True), FakePool(lib, weights_fp32, stream=2, segments=True),
             FakePool(lib, weights_fp32, stream=3), FakePool(lib, weights_fp32, stream=2)]
    r = random.Random(3)
    for p in pools:
        for n in (60, 50):
            p.add(n)
    for _ in range(80):
        p = r.choice(pools)
        p.step_n(r.randrange(1, 4))
        if r.random() < 0.2:
            r.choice(pools).sync()
    us = (C.c_float * 6)()
    assert lib.tts_pool_kernel_times(pools[2].h, 2, us, 6, None) == 0
    pools[0].step_n(1)
    assert lib.fake_segments() > 10 and lib.fake_unordered() == 0
    for p in pools:
        p.close()


def test_segments_of_pools_of_several_threads_follow_each_other(lib, weights_fp32):
    """A thread per pool, one of them created while the others step, one thread that ends and hands its pool on."""
    pools = [FakePool(lib, weights_fp32, stream=1, segments=True, max_steps=4096), FakePool(lib, weights_fp32, stream=2, segments=True, max_steps=4096)]
    errors = []

    def drive(p, seed, calls):
        try:
            r = random.Random(seed)
            p.add(4000)
            for _ in range(calls):
                p.step_n(r.randrange(1, 4))
                if r.random() < 0.3:
                    p.sync()
        except BaseException as e:
            errors.append(e)

    def late():
        try:
            p = FakePool(lib, weights_fp32, stream=3, max_steps=4096)
            drive(p, 7, 100)
            p.close()
        except BaseException as e:
            errors.append(e)

    lib.fake_busy(1)
    drive(pools[0], 1, 3)                      # this thread alone, not waited for
    threads = [threading.Thread(target=drive, args=(pools[0], 2, 200)), threading.Thread(target=drive, args=(pools[1], 3, 200)),
               threading.Thread(target=late)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    drive(pools[1], 4, 20)
    assert not errors
    assert lib.fake_segments() > 100 and lib.fake_unordered() == 0
    for p in pools:
        p.close()


def test_segment_beside_a_stream_that_is_being_captured(lib, weights_fp32):
    """A stream that its owner is capturing is left alone, by the same thread and by another one."""
    a, b = FakePool(lib, weights_fp32, stream=1, segments=True), FakePool(lib, weights_fp32, stream=2, segments=True)
    a.add(40), b.add(40)
    a.step_n(2)
    a.sync()
    a.step_n(2)
    lib.fake_busy(1)
    lib.fake_capture(1)
    before = [lib.fake_calls(f) for f in (b"hipEventRecord", b"hipStreamWaitEvent", b"hipStreamSynchronize")]
    b.step_n(2)
    assert [lib.fake_calls(f) for f in (b"hipEventRecord", b"hipStreamWaitEvent", b"hipStreamSynchronize")] == before
    t = threading.Thread(target=b.step_n, args=(2,))
    t.start()
    t.join()
    assert lib.fake_calls(b"hipStreamSynchronize") == before[2]
    lib.fake_capture(None)
    a.close()
    b.close()


def test_captured_call_takes_its_steps_one_by_one(lib, weights_fp32):
    """(The runtime of this test has no graphs: steps that were captured as a graph would fail the call.)"""
    a, b = FakePool(lib, weights_fp32, stream=1, segments=True), FakePool(lib, weights_fp32, stream=2, segments=True)
    ra, rb = a.add(20), b.add(20)
    a.step_n(2)
    b.step_n(2)
    segments, waits = lib.fake_segments(), lib.fake_calls(b"hipStreamWaitEvent")
    lib.fake_busy(1)
    lib.fake_capture(1)
    a.step_n(7)
    lib.fake_capture(None)
    assert lib.fake_segments() == segments == 2 and lib.fake_calls(b"hipStreamWaitEvent") == waits
    a.step_n(11)
    b.step_n(18)
    assert lib.fake_segments() == 4
    for p, r in ((a, ra), (b, rb)):
        got = [f for _ in range(3) for f in p.drain(r)[1]]
        assert got == _frames(20, 0, 20)
        p.close()


@pytest.mark.parametrize("bf16,slots", [(False, 16), (True, 16), (True, 48)])
def test_what_a_segment_goes_by_does_not_change_while_it_runs(lib, weights_fp32, bf16, slots):
    """Requests that end with a segment's first step, inside it, with its last step and behind it, that leave, that move to lower slots, that
    are lost: a workgroup that starts steps after the others counts the same steps as they do."""
    pool = FakePool(lib, weights_fp32, max_pool=slots, max_steps=80, segments=True, bf16=bf16)
    rids = [pool.add(n) for n in ([1, 2, 3, 7, 8, 9, 40, 41, 64, 80] * 5)[:slots]]
    ninth = rids[9]
    for k, n in enumerate((2, 6, 2, 6, 24, 30, 64)):
        pool.step_n(n)
        assert lib.fake_stale() == 0, k
        if k in (2, 4):                                   # of those that have ended half leave, and others come
            n_done = 0
            for rid in list(rids):
                got, done = C.c_int(), C.c_int()
                assert lib.tts_pool_frames(pool.h, C.c_int64(rid), C.byref(got), C.byref(done)) == 0
                n_done += done.value and rid != ninth
                if done.value and rid != ninth and n_done % 2:
                    assert lib.tts_pool_retire(pool.h, C.c_int64(rid)) == 0
                    rids.remove(rid)
            rids += [pool.add(n) for n in (2, 30, 31)]
        if k == 3:
            lib.fake_freeze(9, 20)                        # (of 80 frames, there from the beginning)
    assert lib.fake_segments() == 7
    lost = C.c_int()
    assert lib.tts_pool_sync(pool.h) == binding.TTS_E_LOST
    assert lib.tts_pool_lost(pool.h, C.c_int64(ninth), C.byref(lost)) == 0 and lost.value
    if slots > 16:
        assert lib.tts_pool_moves(pool.h) > 0
    pool.close()


# slots spanned, longest text -> fewest steps of a call that are one launch (None: never)
FEWEST = [(1, 1024, 1), (16, 1024, 1), (17, 320, 1), (32, 321, 2), (17, 640, 2), (32, 641, 3), (20, 768, 3), (20, 769, 8), (32, 896, 8), (17, 897, None),
          (32, 1024, None), (33, 160, 2), (48, 161, 3), (33, 320, 3), (48, 321, 8), (48, 352, 8), (33, 353, 16), (48, 384, 16), (33, 385, None),
          (48, 1024, None)]


@pytest.mark.parametrize("slots,longest,fewest", FEWEST)
def test_steps_are_one_launch_where_that_is_the_faster_form(lib, weights_fp32, slots, longest, fewest):
    """One text of that length among short ones, in the highest slot.  (Steps as launches of their own would be graphs, which the runtime
    of this test does not have: such a call fails.)"""
    pool = FakePool(lib, weights_fp32, max_pool=48, max_steps=200, chunk=40, segments=True, max_enc_len=1024)
    for k in range(slots - 1):
        pool.add(200)
    pool.add(200, longest)

    def as_one(n):
        before = lib.fake_segments()
        rc = lib.tts_pool_step_n(pool.h, n, None)
        assert rc == (0 if lib.fake_segments() > before else binding.TTS_E_HIP)
        return lib.fake_segments() > before

    assert [as_one(n) for n in range(1, 18)] == [fewest is not None and n >= fewest for n in range(1, 18)]
    assert as_one(40) == (fewest is not None)
    pool.close()


def test_neighbours_event_that_cannot_be_had(lib, weights_fp32):
    """A wait that cannot be queued: the call says so and steps nothing; an event that cannot be recorded: the stream is waited for."""
    a, b = FakePool(lib, weights_fp32, stream=1, segments=True), FakePool(lib, weights_fp32, stream=2, segments=True)
    ra, rb = a.add(8), b.add(8)
    lib.fake_busy(1)
    a.step_n(2)
    lib.fake_fail(b"hipStreamWaitEvent", 1, 1)
    assert lib.tts_pool_step_n(b.h, 2, None) == binding.TTS_E_HIP
    n = C.c_int()
    assert lib.tts_pool_frames(b.h, C.c_int64(rb), C.byref(n), None) == 0 and n.value == 0
    b.step_n(2)
    t = threading.Thread(target=a.step_n, args=(2,))
    t.start()
    t.join()
    lib.fake_fail(b"hipEventRecord", 1, 1)
    b.step_n(2)
    a.step_n(4)
    b.step_n(4)
    assert lib.fake_unordered() == 0
    assert a.drain(ra) == (0, _frames(8, 0, 8), True) and b.drain(rb) == (0, _frames(8, 0, 8), True)
    a.close()
    b.close()


@pytest.mark.parametrize("module", ["pool", "encoder", "postnet", "vocoder"])
def test_what_an_object_starts_with_is_there_when_it_has_been_made(lib, weights_fp32, module):
    """The first call goes to the object's own stream, which does not wait for the default stream's fills."""
    if module == "pool":
        FakePool(lib, weights_fp32, segments=True).close()
    elif module == "encoder":
        FakeEncoder(lib).close()
    else:
        if module == "postnet":
            cfg, w = binding.make_postnet_config(max_columns=64), binding.TtsPostnetWeights()
        else:
            cfg, w = binding.make_vocoder_config(overlap=4, max_chunk=8, max_requests=2, max_batch=2), binding.TtsVocoderWeights()
        zeros = np.zeros(512 * 512 * 16, np.float32)                     # (as large as the largest tensor)
        at = (C.c_void_p * (C.sizeof(w) // 8)).from_buffer(w)
        for i in range(len(at)):
            at[i] = zeros.ctypes.data
        n = int(getattr(lib, f"tts_{module}_workspace_bytes")(C.byref(cfg)))
        raw, arena = _arena(n)
        h = C.c_void_p()
        create = getattr(lib, f"tts_{module}_create")
        assert create(C.byref(cfg), C.byref(w), arena, C.c_size_t(n), C.c_void_p(1), C.byref(h)) == 0, lib.tts_last_error()
        getattr(lib, f"tts_{module}_destroy")(h)
    assert lib.fake_filling() == 0
