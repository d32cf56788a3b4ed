"""A small call's convolutions as one launch, whose workgroups hand each other their outputs: the same bits as layer by layer, at the
edges of column tiles, column groups and of the forms with one, two and three times as many tiles a workgroup; call after call of
changing sizes (the words of one call are emptied by the next), under capture, and where the workgroups wait once or not at all for
each other and form what they need themselves."""
import numpy as np
import pytest

from paper_2211_13939_amd import binding, synth
from tests.helpers import say

pytestmark = pytest.mark.gpu

EDGES = {True: (1, 15, 16, 17, 31, 33, 255, 256, 257, 511, 512, 513, 767, 768, 769), False: (1, 15, 16, 17, 127, 128, 129, 255, 256, 257, 383, 384, 385)}


def _windows(columns, rng):
    wins = []
    while sum(wins) < columns:
        wins.append(min(int(rng.integers(1, 60)), columns - sum(wins)))
    return wins, [int(rng.integers(0, w)) for w in wins]


def _postnet(bf16, max_columns=1024):
    ws, bs = synth.make_postnet_weights(bf16=bf16)
    return binding.Postnet(binding.make_postnet_config(max_columns=max_columns, bf16=bf16), ws, bs)


# capacities whose largest call has more columns in its groups than whole groups of the largest size would
FULL = [(True, n) for n in (257, 288, 449, 450, 480)] + [(False, n) for n in (129, 144, 225, 240)]


@pytest.mark.parametrize("bf16,columns", FULL)
def test_postnet_made_for_exactly_the_call(bf16, columns):
    """Several calls in a row: each of the two sets of words in its turn."""
    import torch
    rng = np.random.default_rng(columns)
    pn = _postnet(bf16, max_columns=columns)
    for call in range(4):
        wins, keeps = _windows(columns, rng)
        say(f"case PostNet made for {columns} columns, call {call} of {columns} in {len(wins)} windows, {'bf16' if bf16 else 'fp32'}")
        with torch.cuda.stream(pn.stream):
            mel = torch.from_numpy(rng.standard_normal((columns, 80)).astype(np.float32)).cuda()
            got, want = (torch.full((columns - sum(keeps), 80), float("nan"), device="cuda") for _ in range(2))
            pn.run_device(mel, wins, keeps, got)
            pn.run_device(mel, wins, keeps, want, static=True)
        pn.stream.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())
    assert pn.one_launch_calls() == 4
    pn.close()


@pytest.mark.parametrize("bf16,columns", FULL)
def test_encoder_made_for_exactly_the_call(bf16, columns):
    """Against the same requests in a larger call of a larger encoder, layer by layer."""
    weights = synth.make_encoder_weights(bf16=bf16)
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=columns, max_len=columns, bf16=bf16), weights)
    large = binding.Encoder(binding.make_encoder_config(max_tokens=1152, max_len=640, bf16=bf16), weights)
    more = synth.encoder_ids(600, 99)
    for call, lens in enumerate(([columns], [columns // 3, 1, columns - columns // 3 - 1], [columns // 2, columns - columns // 2])):
        say(f"case encoder made for {columns} tokens, call {call} of {lens}, {'bf16' if bf16 else 'fp32'}")
        ids = [synth.encoder_ids(l, 7 * call + i) for i, l in enumerate(lens)]
        for a, b in zip(enc.run(ids), large.run(ids + [more])):
            np.testing.assert_array_equal(a, b)
    assert enc.one_launch_calls() == 3 and large.one_launch_calls() == 0
    enc.close()
    large.close()


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("polls", [None, 1, 0])
def test_postnet_calls_as_one_launch(polls, bf16):
    """Against tts_postnet_run_static, whose calls are a launch per layer, twice over: with the words of other sizes before.  polls = 1:
    most workgroups take what is not there from the counter; 0: every workgroup forms all it needs by itself."""
    import torch
    rng = np.random.default_rng(71)
    pn = _postnet(bf16)
    if polls is not None:
        pn.set_wait_polls(polls)
    for columns in EDGES[bf16] + EDGES[bf16][::-2] + (24, 96, 300, 500, 3):
        wins, keeps = _windows(columns, rng) if columns not in (24, 96, 300, 500) else ([columns // 4] * 4, [0] * 4)
        say(f"case postnet as one launch: {columns} columns in {len(wins)} windows, {'bf16' if bf16 else 'fp32'}, polls {polls}")
        with torch.cuda.stream(pn.stream):
            mel = torch.from_numpy(rng.standard_normal((columns, 80)).astype(np.float32)).cuda()
            got, want = (torch.full((columns - sum(keeps), 80), float("nan"), device="cuda") for _ in range(2))
            before = pn.one_launch_calls()
            pn.run_device(mel, wins, keeps, got)
            assert pn.one_launch_calls() == before + (columns <= (768 if bf16 else 384))
            pn.run_device(mel, wins, keeps, want, static=True)
        pn.stream.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())
        if not any(keeps):
            say("  ... its results where its input lies")
            pn.run_device(mel, wins, keeps, mel)
            pn.stream.synchronize()
            np.testing.assert_array_equal(mel.cpu().numpy(), want.cpu().numpy())
    pn.close()


@pytest.mark.parametrize("bf16", [True, False])
def test_postnet_call_captured_and_replayed(bf16):
    """Whose turn the two sets of words are lies on the device: replays, with calls of other sizes between them."""
    import torch
    rng = np.random.default_rng(72)
    pn = _postnet(bf16)
    wins, keeps = [50, 17, 3], [10, 0, 2]
    say(f"case postnet as one launch under capture, {'bf16' if bf16 else 'fp32'}")
    with torch.cuda.stream(pn.stream):
        mel = torch.zeros((70, 80), device="cuda")
        got, want, other = (torch.zeros((n, 80), device="cuda") for n in (58, 58, 200))
        pn.run_device(mel, wins, keeps, got)
    pn.stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=pn.stream):
        pn.run_device(mel, wins, keeps, got)
    for i in range(5):
        with torch.cuda.stream(pn.stream):
            mel.copy_(torch.from_numpy(rng.standard_normal((70, 80)).astype(np.float32)))
            graph.replay()
            if i % 2:
                pn.run_device(torch.zeros((200, 80), device="cuda"), [200], [0], other)
            pn.run_device(mel, wins, keeps, want, static=True)
        pn.stream.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())
    del graph
    pn.close()


@pytest.mark.parametrize("bf16,edges", [(True, (1, 16, 17, 255, 256, 257, 511, 512)), (False, (1, 16, 17, 127, 128, 129, 256, 257, 383, 384))])
@pytest.mark.parametrize("polls", [None, 1, 0])
def test_encoder_calls_as_one_launch(bf16, edges, polls):
    """Against the same requests in a call with one more, long one, which is too large for one launch; polls as above."""
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=1152, max_len=640, bf16=bf16), synth.make_encoder_weights(bf16=bf16))
    more = synth.encoder_ids(600, 99)
    for columns in edges:
        say(f"case encoder as one launch: {columns} tokens, {'bf16' if bf16 else 'fp32'}, polls {polls}")
        lens = [columns] if columns < 40 else [columns // 3, 1, columns - columns // 3 - 1]
        ids = [synth.encoder_ids(l, i) for i, l in enumerate(lens)]
        if polls is not None:
            enc.set_wait_polls(polls)
        before = enc.one_launch_calls()
        got = enc.run(ids)
        want = enc.run(ids + [more])
        assert enc.one_launch_calls() == before + 1
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a, b)
    enc.close()
