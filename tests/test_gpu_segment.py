"""Steps as one launch (csrc/segment.hip: two-byte pools whose running requests lie in the first 48 slots) against the same steps
as launches of their own (use_graph=False): the same bits, frames and carried state."""
import numpy as np
import pytest

from paper_2211_13939_amd import binding, synth
from tests.helpers import make_pool, say

pytestmark = pytest.mark.gpu


def _both(weights, lengths, frames, calls, max_pool=16, max_enc_len=1024, spoil=None, later=(), forms=(True, False)):
    """The job in either form: frames of every request, its state and its stop logits, and the launches of segments.  A pool without
    graphs takes every step as launches of its own."""
    wl = synth.small_workload(len(lengths), 5, 90, 8, 8, seed=31, bf16=True)
    out = []
    for use_graph in forms:
        pool = make_pool(wl, weights, max_pool=max_pool, max_enc_len=max_enc_len, max_steps=80, chunk_frames=40, use_graph=use_graph)
        rng = np.random.default_rng(5)
        enc = [synth.round_to_bf16(rng.standard_normal((L, wl.dims["enc_dim"])).astype(np.float32)) for L in lengths]
        if spoil is not None:
            enc[0].view(np.uint32)[lengths[0] // 2, 3] = spoil
        n_first = len(lengths) - len(later)
        ids = pool.add_requests(enc[:n_first], frames[:n_first])
        for k, n in enumerate(calls):
            ids += [pool.add_request(enc[n_first + j], frames[n_first + j]) for j, at in enumerate(later) if at == k]
            pool.step_n(n)
        pool.sync()
        mel = [pool.drain_all(r) for r in ids]
        state = [{name: pool.get_state(r, name) for name in binding.STATE} for r in ids]
        stop = [pool.stop_logits(r, 0, m.shape[0]) for r, m in zip(ids, mel)]
        assert (pool.segments() > 0) == use_graph
        out.append((mel, state, stop, pool.segments()))
        pool.close()
    return out


def _same(out, frames):
    (mel, state, stop, _), (mel1, state1, stop1, _) = out
    for i, n in enumerate(frames):
        assert mel[i].shape[0] == n
        np.testing.assert_array_equal(mel[i], mel1[i])
        np.testing.assert_array_equal(stop[i], stop1[i])
        for name in binding.STATE:
            np.testing.assert_array_equal(state[i][name], state1[i][name], err_msg=name)


@pytest.mark.parametrize("lengths,frames,calls", [
    ([1], [2], [2]),                                                       # the smallest
    ([165], [41], [3, 1, 37]),                                             # odd calls, a single step among them
    ([17, 512, 513], [5, 80, 44], [64, 16]),                               # rows kept in registers end at 512 positions
    ([1024, 16, 1023, 15], [33, 2, 64, 65], [1, 32, 31, 1]),               # the longest texts; ends inside a call and at its end
    ([31 + 40 * i for i in range(8)], [40 - i for i in range(8)], [40]),   # eight slots: one request per XCD
    ([33 + 20 * i for i in range(9)], [12 + i for i in range(9)], [7, 13]),
    ([20 + 9 * i for i in range(16)], [10 + 3 * i for i in range(16)], [20, 35]),
    ([600, 321, 320, 17] + [30 + 5 * i for i in range(13)], [40] * 17, [1, 39]),   # a second tile: two workgroups a request, 320 positions in registers
    ([25 + 6 * i for i in range(32)], [8 + i for i in range(32)], [16, 23]),
    ([300, 129, 128, 257] + [20 + 4 * i for i in range(29)], [5 + i for i in range(33)], [20, 17]),   # a third: one a request, 128 positions
    ([896, 17] + [320 + 30 * i for i in range(16)], [40] * 18, [8, 32]),                               # the longest texts of two tiles, and of three
    ([384, 385 - 16] + [20 + 8 * i for i in range(35)], [40] * 37, [16, 24]),
    ([20 + 5 * i for i in range(48)], [48 - i for i in range(48)], [13, 35]),
], ids=lambda v: None)
def test_segment_equals_steps(lengths, frames, calls, weights_bf16):
    say(f"case: segments of {calls} steps, texts of {lengths}, frames {frames}")
    out = _both(weights_bf16, lengths, frames, calls, max_pool=16 if len(lengths) <= 16 else 48)
    _same(out, frames)
    assert out[0][3] == sum(n > 1 or len(lengths) <= 16 or (len(lengths) <= 32 and max(lengths) <= 320) for n in calls)


def test_segments_between_steps_of_a_larger_pool(weights_bf16):
    """With a 49th request the pool's steps are launches of their own; they become segments again, of fewer tiles, when requests have
    ended and the pool is packed."""
    say("case: 12 requests, 40 more for eight steps, ten of them for longer, segments again")
    lengths = [20 + 2 * i for i in range(52)]
    frames = [60] * 12 + [20] * 10 + [8] * 30
    out = _both(weights_bf16, lengths, frames, [15, 8, 12, 25], max_pool=64, max_enc_len=160, later=[1] * 40)
    _same(out, frames)
    assert out[0][3] == 3


@pytest.mark.parametrize("spoil", [0xFFFFFFFF, 0x7F800000, 0x7FC00000])
def test_segment_with_values_that_are_no_numbers(spoil, weights_bf16):
    """A word that the workgroups hand each other is taken for empty while all of its bits are set: a value of that pattern must not
    keep a reader waiting, and another request must not notice."""
    say(f"case: an encoder output with the bits {spoil:#x} beside an ordinary one")
    frames = [24, 24]
    (mel, _, _, _), = _both(weights_bf16, [30, 40], frames, [24], max_enc_len=64, spoil=spoil, forms=(True,))
    (clean, _, _, _), = _both(weights_bf16, [30, 40], frames, [24], max_enc_len=64, forms=(True,))
    assert mel[0].shape == (24, 80) and not np.array_equal(mel[0], clean[0])
    np.testing.assert_array_equal(mel[1], clean[1])


def test_segment_with_a_large_attention_vector(weights_bf16):
    """Energies beyond the bound of the one-pass softmax take the form with the maximum."""
    say("case: attention vector times 40")
    w = dict(weights_bf16)
    w["v"] = w["v"] * 40
    assert np.abs(w["v"]).sum() > 30
    frames = [20, 33]
    _same(_both(w, [70, 600], frames, [33]), frames)


def _job(n, weights, max_pool, frames, use_graph=True, seed=0):
    """A pool of n requests and the frames they give alone on the GPU."""
    rng = np.random.default_rng(seed)
    lengths = [int(x) for x in rng.integers(5, 90, size=n)]
    enc = [synth.round_to_bf16(rng.standard_normal((L, 512)).astype(np.float32)) for L in lengths]
    wl = synth.small_workload(n, 5, 90, 8, 8, seed=31, bf16=weights["bf16"])
    make = lambda: make_pool(wl, weights["w"], max_pool=max_pool, max_enc_len=90, max_steps=80, chunk_frames=40, use_graph=use_graph)
    pool = make()
    ids = pool.add_requests(enc, [frames] * n)
    pool.step_n(frames)
    pool.sync()
    want = [pool.drain_all(r) for r in ids]
    pool.close()
    pool = make()
    return pool, pool.add_requests(enc, [frames] * n), want


@pytest.mark.parametrize("n", [1, 16, 20, 32, 40, 48])
def test_segments_beside_other_work(n, weights_bf16):
    """Another stream keeps the compute units busy with products that end by themselves: a segment's workgroups start late, in parts; the
    frames do not change and no wait runs out."""
    import torch
    say(f"case: segments of {n} slots while a second stream runs large matrix products")
    pool, ids, want = _job(n, dict(w=weights_bf16, bf16=True), 48, 24)
    side = torch.cuda.Stream(device=pool.device)
    a = torch.randn(4096, 4096, device=pool.device)
    with torch.cuda.stream(side):
        for _ in range(40):
            a = (a @ a) * 1e-4
    for k in (4, 1, 7, 12):
        pool.step_n(k)
    pool.sync()                      # raises if a wait ran out
    side.synchronize()
    assert pool.segments() == (4 if n <= 32 else 3)                        # (a single step of three tiles: launches of its own)
    for r, w in zip(ids, want):
        np.testing.assert_array_equal(pool.drain_all(r), w)
    pool.close()


@pytest.mark.parametrize("threads", [False, True])
def test_segments_of_several_pools(threads, weights_bf16, weights_fp32):
    """Pools of one and of three tiles, and a fp32 pool whose steps are launches of their own, stepped in turn without a wait, by one
    thread and by a thread each: the frames of each alone."""
    import threading
    say(f"case: three pools, {'a thread each' if threads else 'one thread'}")
    jobs = [_job(3, dict(w=weights_bf16, bf16=True), 16, 64, seed=1), _job(40, dict(w=weights_bf16, bf16=True), 48, 64, seed=2),
            _job(5, dict(w=weights_fp32, bf16=False), 16, 64, seed=3)]
    errors = []

    def drive(pool, counts):
        try:
            for k in counts:
                pool.step_n(k)
        except BaseException as e:
            errors.append(e)

    if threads:
        ts = [threading.Thread(target=drive, args=(job[0], [1, 3] * 16)) for job in jobs]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
    else:
        for _ in range(16):
            for job in jobs:
                drive(job[0], [1, 3])
    assert not errors
    for pool, ids, want in jobs:
        pool.sync()                  # raises if a wait ran out
        assert pool.segments() == {3: 32, 40: 16, 5: 0}[len(ids)]           # (of the 40, single steps are launches of their own)
        for r, w in zip(ids, want):
            np.testing.assert_array_equal(pool.drain_all(r), w)
        pool.close()


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("n", [1, 6, 7])
def test_captured_steps(n, bf16, weights_bf16, weights_fp32):
    """A call on a stream that is being captured, its graph launched once, between calls that are not."""
    import torch
    say(f"case: {n} steps captured, {'bf16' if bf16 else 'fp32'}")
    pool, ids, want = _job(3, dict(w=weights_bf16 if bf16 else weights_fp32, bf16=bf16), 16, 40)
    pool.step_n(5)
    pool.sync()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=pool.stream):
        pool.step_n(n)
    assert pool.segments() == int(bf16)
    with torch.cuda.stream(pool.stream):
        graph.replay()
    pool.step_n(35 - n)
    pool.sync()
    for r, w in zip(ids, want):
        np.testing.assert_array_equal(pool.drain_all(r), w)
    del graph
    pool.close()
