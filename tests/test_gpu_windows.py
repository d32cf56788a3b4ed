"""Chunks of several requests handed to the device with one launch (tts_pool_chunk_windows) against one call per request, and vocoder samples
written straight to pinned host memory."""
import numpy as np
import pytest

from paper_2211_13939_amd import binding, synth
from tests.helpers import make_pool, say

pytestmark = pytest.mark.gpu

CTX, CHUNK = 10, 8


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 17])
def test_windows_together_equal_windows_one_by_one(n, offset, weights_fp32):
    """Requests that end inside a chunk, at its end and later, one whose chunk is not ready; a destination that is aligned to 16 bytes and
    one that is aligned to a float."""
    import torch
    say(f"case: windows of {n} requests, {offset} floats into the buffer")
    wl = synth.small_workload(n, 5, 60, 40, 40, seed=5)
    frames = [(12, 16, 40, 3)[i % 4] for i in range(n)]
    pools = [make_pool(wl, weights_fp32, max_pool=32, max_enc_len=64, max_steps=40, chunk_frames=CHUNK) for _ in range(2)]
    ids = [p.add_requests([wl.encoder_outputs(i) for i in range(n)], frames) for p in pools]
    bufs = []
    for p in pools:
        with torch.cuda.stream(p.stream):
            bufs.append(torch.full((n * (CTX + CHUNK) * 80 + 4,), float("nan"), device="cuda")[offset:])
    for steps in (4, 4, 3, 5, 8):
        for p in pools:
            p.step_n(steps)
        together = pools[0].chunk_windows(ids[0], CTX, bufs[0][:n * (CTX + CHUNK) * 80])
        single, row = [], 0
        for rid in ids[1]:
            single.append(pools[1].chunk_window(rid, CTX, bufs[1][row * 80:][:(CTX + CHUNK) * 80]))
            row += sum(single[-1][:2])
        assert together == single
        for p in pools:
            p.sync()
        a, b = (x[:row * 80].cpu().numpy() for x in bufs)
        assert np.isfinite(a).all()
        np.testing.assert_array_equal(a, b)
    for p in pools:
        p.close()


def test_windows_of_requests_that_are_not_there(weights_fp32):
    import torch
    say("case: an unknown request, one that is named twice, too many")
    wl = synth.small_workload(2, 5, 20, 8, 8, seed=5)
    pool = make_pool(wl, weights_fp32, max_pool=4, max_enc_len=24, max_steps=8, chunk_frames=CHUNK)
    a, b = pool.add_requests([wl.encoder_outputs(i) for i in range(2)], [8, 8])
    pool.step_n(8)
    buf = torch.empty(300 * (CTX + CHUNK), 80, device="cuda")
    for rids, code in (([a, 99], binding.TTS_E_NOTFOUND), ([a, b, a], binding.TTS_E_INVAL), ([a] * 257, binding.TTS_E_INVAL), ([], binding.TTS_E_INVAL)):
        with pytest.raises(binding.TtsError) as e:
            pool.chunk_windows(rids, CTX, buf)
        assert e.value.code == code
    assert pool.chunk_windows([b, a], CTX, buf) == [(0, 8, True)] * 2          # nothing was handed out before
    pool.close()


@pytest.mark.parametrize("bf16,requests", [(True, 1), (True, 40), (False, 2)])
def test_samples_to_pinned_memory(bf16, requests):
    """Both tilings of the last layer."""
    import torch
    say(f"case: samples of {requests} requests to pinned memory")
    voc = binding.Vocoder(binding.make_vocoder_config(overlap=4, max_chunk=40, max_requests=requests, max_batch=requests, bf16=bf16),
                          synth.make_vocoder_weights(bf16=bf16))
    size = requests * 44 * binding.VOCODER_HOP
    with torch.cuda.stream(voc.stream):
        mel = torch.randn(requests * 40, 80, device="cuda")
        dev = torch.zeros(size, device="cuda")
    host = torch.zeros(size).pin_memory()
    whole = [binding.VOCODER_FIRST | binding.VOCODER_LAST] * requests
    for to in (dev, host):
        n = sum(voc.run_device(mel, [40] * requests, list(range(requests)), whole, to))
    voc.stream.synchronize()
    assert n == requests * 40 * binding.VOCODER_HOP
    np.testing.assert_array_equal(host[:n].numpy(), dev[:n].cpu().numpy())
    voc.close()


def test_buffers_of_a_loop_that_is_dropped_with_a_round_on_its_way(weights_fp32):
    """The vocoder stores a round's samples to pinned memory: nobody else is given that memory before it has."""
    import gc
    import torch
    from paper_2211_13939_amd import stream
    say("case: an overlapped loop that is dropped while its vocoder round is queued")
    wl = synth.small_workload(2, 10, 50, 24, 24, seed=53)
    pool = make_pool(wl, weights_fp32, chunk_frames=12, max_pool=2)
    side = torch.cuda.Stream(device=pool.device)
    pn = binding.Postnet(binding.make_postnet_config(max_columns=2 * (12 + CTX)), *synth.make_postnet_weights(), stream=side)
    voc = binding.Vocoder(binding.make_vocoder_config(overlap=4, max_chunk=12, max_requests=2, max_batch=2), synth.make_vocoder_weights(), stream=side)
    be = stream.GpuPostnetBackend(pool, pn, lambda i: wl.encoder_outputs(i), wl.n_steps, 12, CTX, vocoder=voc, on_audio=lambda i, a: None, overlap=True)
    for i in range(2):
        be.add(i)
    with torch.cuda.stream(side):
        a = torch.ones(8192, 8192, device="cuda")
        for _ in range(20):
            a = (a @ a) * 1e-4
    be.run(12)
    assert be.pending() and not side.query()
    size, mine = be._sets[0]["h_audio"].numel(), {st["h_audio"].data_ptr() for st in be._sets}
    del be
    gc.collect()
    others = [torch.empty(size, pin_memory=True) for _ in range(6)]
    done = side.query()
    assert done or not mine & {t.data_ptr() for t in others}
    torch.cuda.synchronize()
    voc.close()
    pn.close()
    pool.close()
