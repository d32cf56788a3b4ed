"""Steps as one launch (csrc/segment.hip: two-byte pools whose running requests lie in the first 48 slots) against the same steps
as launches of their own (use_graph=False): the same bits, frames and carried state."""
import numpy as np
import pytest

from paper_2211_13939_amd import binding, synth
from tests.helpers import make_pool, say

pytestmark = pytest.mark.gpu


def _both(weights, lengths, frames, calls, max_pool=16, max_enc_len=1024, spoil=None, later=(), forms=(True, False)):
    """The job in either form: frames of every request and, of those that did not have to be retired on the way, the state."""
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
        out.append((mel, state, stop))
        pool.close()
    return out


def _same(out, frames):
    (mel, state, stop), (mel1, state1, stop1) = out
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
    ([20 + 5 * i for i in range(48)], [48 - i for i in range(48)], [13, 35]),
], ids=lambda v: None)
def test_segment_equals_steps(lengths, frames, calls, weights_bf16):
    say(f"case: segments of {calls} steps, texts of {lengths}, frames {frames}")
    _same(_both(weights_bf16, lengths, frames, calls, max_pool=16 if len(lengths) <= 16 else 48), frames)


def test_segments_between_steps_of_a_larger_pool(weights_bf16):
    """With a 49th request the pool's steps are launches of their own; they become segments again, of fewer tiles, when requests have
    ended and the pool is packed."""
    say("case: 12 requests, 40 more for eight steps, ten of them for longer, segments again")
    lengths = [20 + 2 * i for i in range(52)]
    frames = [60] * 12 + [20] * 10 + [8] * 30
    _same(_both(weights_bf16, lengths, frames, [15, 8, 12, 25], max_pool=64, max_enc_len=160, later=[1] * 40), frames)


@pytest.mark.parametrize("spoil", [0xFFFFFFFF, 0x7F800000, 0x7FC00000])
def test_segment_with_values_that_are_no_numbers(spoil, weights_bf16):
    """A word that the workgroups hand each other is taken for empty while all of its bits are set: a value of that pattern must not
    keep a reader waiting, and another request must not notice."""
    say(f"case: an encoder output with the bits {spoil:#x} beside an ordinary one")
    frames = [24, 24]
    (mel, _, _), = _both(weights_bf16, [30, 40], frames, [24], max_enc_len=64, spoil=spoil, forms=(True,))
    (clean, _, _), = _both(weights_bf16, [30, 40], frames, [24], max_enc_len=64, forms=(True,))
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
