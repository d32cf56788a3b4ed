"""Device time of a PostNet or vocoder call, which its launches stamp themselves: within the time between two events around the call,
for every form a call's first and last launch take, also for a short call behind a longer one and for replays of a captured call."""
import pytest

from paper_2211_13939_amd import binding, synth
from tests.helpers import say

pytestmark = pytest.mark.gpu


def _check(obj, call, torch):
    """Two events around the call, with the stream busy before it (so the host's pace is not part of it).  Events cost a few us themselves,
    and the workgroups that share a stamp may store it in any order: a tenth and 12 us below are left to that."""
    with torch.cuda.stream(obj.stream):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        call()
        busy = torch.ones(4096, 4096, device="cuda")
        for _ in range(3):
            busy = busy @ busy
        a.record()
        call()
        b.record()
    b.synchronize()
    between, own = a.elapsed_time(b) * 1e3, obj.elapsed_ms() * 1e3
    say(f"  {own:.1f} us, {between:.1f} us between events")
    assert 0 < own <= between + 0.05
    assert own >= 0.9 * between - 12
    return own


@pytest.mark.parametrize("bf16,windows", [(True, 1), (True, 14), (True, 30), (True, 64), (True, 300), (False, 6), (False, 40), (False, 100)])
def test_postnet_call(bf16, windows):
    """One launch; layers, the last of them by either kernel; more windows than one list holds."""
    import torch
    ws, bs = synth.make_postnet_weights(bf16=bf16)
    pn = binding.Postnet(binding.make_postnet_config(max_columns=windows * 50, bf16=bf16), ws, bs)
    with pytest.raises(binding.TtsError):
        pn.elapsed_ms()
    with torch.cuda.stream(pn.stream):
        mel = torch.randn(windows * 50, 80, device="cuda")
        out = torch.zeros(windows * 40, 80, device="cuda")
    say(f"case PostNet of {windows} windows, {'bf16' if bf16 else 'fp32'}")
    long = _check(pn, lambda: pn.run_device(mel, [50] * windows, [10] * windows, out), torch)
    if windows > 30:
        assert _check(pn, lambda: pn.run_device(mel, [50], [10], out), torch) < long
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=pn.stream):
        pn.run_device(mel, [50] * windows, [10] * windows, out)
    for _ in range(3):
        with torch.cuda.stream(pn.stream):
            graph.replay()
        assert 0.5 * long < pn.elapsed_ms() * 1e3 < 2 * long + 12
    pn.close()


@pytest.mark.parametrize("bf16,requests", [(True, 1), (True, 64), (False, 3)])
def test_vocoder_call(bf16, requests):
    import torch
    voc = binding.Vocoder(binding.make_vocoder_config(overlap=8, max_chunk=40, max_requests=requests, max_batch=requests, bf16=bf16),
                          synth.make_vocoder_weights(bf16=bf16))
    with torch.cuda.stream(voc.stream):
        mel = torch.randn(requests * 40, 80, device="cuda")
        audio = torch.zeros(requests * 48 * binding.VOCODER_HOP, device="cuda")
    say(f"case vocoder of {requests} requests, {'bf16' if bf16 else 'fp32'}")
    whole = [binding.VOCODER_FIRST | binding.VOCODER_LAST] * requests
    long = _check(voc, lambda: voc.run_device(mel, [40] * requests, list(range(requests)), whole, audio), torch)
    if requests > 1:
        assert _check(voc, lambda: voc.run_device(mel, [3], [0], whole[:1], audio), torch) < long
    voc.close()


@pytest.mark.parametrize("module", ["postnet of 3 windows", "postnet of 60 windows", "vocoder"])
def test_a_call_that_was_only_captured_has_no_time(module):
    """Neither that of a call before it nor none at all; its graph's launches have theirs, and a call behind them has its own."""
    import torch
    say(f"case captured calls, {module}")
    n = 60 if "60" in module else 3
    if module == "vocoder":
        obj = binding.Vocoder(binding.make_vocoder_config(overlap=8, max_chunk=40, max_requests=n, max_batch=n, bf16=True), synth.make_vocoder_weights(bf16=True))
    else:
        obj = binding.Postnet(binding.make_postnet_config(max_columns=n * 50, bf16=True), *synth.make_postnet_weights(bf16=True))
    with torch.cuda.stream(obj.stream):
        mel = torch.randn(n * 50, 80, device="cuda")
        out = torch.zeros(n * 48 * binding.VOCODER_HOP, device="cuda")
    whole = [binding.VOCODER_FIRST | binding.VOCODER_LAST] * n

    def call(k):
        if module == "vocoder":
            obj.run_device(mel, [40] * k, list(range(k)), whole[:k], out)
        else:
            obj.run_device(mel, [50] * k, [10] * k, out)

    for before in (False, True):
        if before:
            call(1)
            assert obj.elapsed_ms() > 0
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=obj.stream):
            call(n)
        with pytest.raises(binding.TtsError) as e:
            obj.elapsed_ms()
        assert e.value.code == binding.TTS_E_INVAL
        for _ in range(2):
            with torch.cuda.stream(obj.stream):
                graph.replay()
            assert obj.elapsed_ms() > 0
    call(1)
    assert obj.elapsed_ms() > 0
    torch.cuda.synchronize()
    obj.close()
