"""The vocoder's tilings follow the windows of a call: a request's samples are the bits it has alone, whatever they are."""
import numpy as np
import pytest

from paper_2211_13939_amd import binding, synth

pytestmark = pytest.mark.gpu
WHOLE_REQUEST = binding.VOCODER_FIRST | binding.VOCODER_LAST


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("frames", [1, 16, 17, 33, 48])        # half a tile of 64 channels holds 17 frames, a whole window 48
def test_bits_do_not_depend_on_the_tiling(frames, bf16):
    w = synth.make_vocoder_weights(bf16=bf16)
    mel = lambda i, n: np.random.default_rng([frames, i]).standard_normal((n, synth.DIMS["n_mel"])).astype(np.float32)
    mine = mel(0, frames)
    out = []
    for max_chunk in (max(frames, 4), 72):
        voc = binding.Vocoder(binding.make_vocoder_config(overlap=4, max_chunk=max_chunk, max_requests=100, max_batch=100, bf16=bf16), w)
        for n in (1, 2, 7, 25, 45, 64, 100):
            for longest in {frames, max_chunk}:
                others = [mel(i, longest if i == 1 else frames) for i in range(1, n)]
                out.append(voc.run([mine] + others, list(range(n)), [WHOLE_REQUEST] * n)[0])
        voc.close()
    assert np.isfinite(out[0]).all() and np.abs(out[0]).max() > 0
    for o in out[1:]:
        np.testing.assert_array_equal(out[0], o)
