"""Acoustic encoder on the GPU against the CPU oracle (oracle/encoder_oracle.c), through the C ABI."""
import numpy as np
import pytest

from paper_2211_13939_amd import binding, synth
from tests.helpers import TOL_BF16, TOL_F32, make_pool, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
def test_ragged_batch_matches_oracle(bf16):
    """Six requests of 1 .. 77 tokens in one call (several column tiles, ragged ends, a one-token request; fewer
    requests than MFMA columns): F_enc of every request equals the oracle's, which encodes each request alone."""
    from oracle import oracle as orc
    w = synth.make_encoder_weights(bf16=bf16)
    W = orc.EncoderWeights(w)
    lens = [1, 5, 16, 17, 77, 33]
    ids = [synth.encoder_ids(L, 100 + i) for i, L in enumerate(lens)]
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=256, max_len=100, bf16=bf16), w)
    say(f"case encoder: requests of {lens} tokens, {'bf16' if bf16 else 'fp32'}")
    got = enc.run(ids)
    worst = 0.0
    for a, g in zip(ids, got):
        want = orc.encoder(W, a)
        assert g.shape == want.shape
        worst = max(worst, float(np.abs(g - want).max()))
    say(f"  max abs err {worst:.3e} on F_enc in (-1, 1), {enc.elapsed_ms() * 1e3:.0f} us")
    assert worst <= (TOL_BF16 if bf16 else TOL_F32)
    enc.close()


@pytest.mark.parametrize("n_tokens", [1, 2, 33, 300])
def test_a_call_of_one_request_matches_oracle_bf16(n_tokens):
    """The usual call at join time: one request (one column of a column tile of the convolutions, two workgroups of the
    recurrence): one token, two tokens and a request that feeds h back 300 times."""
    from oracle import oracle as orc
    w = synth.make_encoder_weights(bf16=True)
    ids = synth.encoder_ids(n_tokens, 500 + n_tokens)
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=320, max_len=300, bf16=True), w)
    say(f"case encoder: one request of {n_tokens} tokens, bf16")
    got = enc.run([ids])[0]
    want = orc.encoder(orc.EncoderWeights(w), ids)
    assert got.shape == want.shape
    err = float(np.abs(got - want).max())
    say(f"  max abs err {err:.3e}")
    assert err <= TOL_BF16
    enc.close()


def test_more_requests_than_mfma_columns_and_long_request():
    """20 requests (more than the 16 columns of a column tile) and one of 300 tokens, bf16."""
    from oracle import oracle as orc
    w = synth.make_encoder_weights(bf16=True)
    W = orc.EncoderWeights(w)
    rng = np.random.default_rng(7)
    lens = [int(x) for x in rng.integers(3, 40, size=19)] + [300]
    ids = [synth.encoder_ids(L, 200 + i) for i, L in enumerate(lens)]
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=1024, max_len=300, bf16=True), w)
    say(f"case encoder: 20 requests, {sum(lens)} tokens, longest 300, bf16")
    got = enc.run(ids)
    worst = 0.0
    for k in (0, 7, 15, 16, 18, 19):
        worst = max(worst, float(np.abs(got[k] - orc.encoder(W, ids[k])).max()))
    say(f"  max abs err {worst:.3e}, {enc.elapsed_ms() * 1e3:.0f} us")
    assert worst <= TOL_BF16
    enc.close()


@pytest.mark.parametrize("bf16", [True, False])
def test_result_does_not_depend_on_batch_composition(bf16):
    """Bitwise, whatever the call.  The convolutions and the input projection have one kernel for small calls - all calls here,
    see the next test - and one for large ones, which sum in one order.  The recurrence does so, too: with two-byte weights
    every request has workgroups of its own, with fp32 weights a unit's sum does not depend on how many workgroups share a
    direction and how many requests share them."""
    w = synth.make_encoder_weights(bf16=bf16)
    ids = [synth.encoder_ids(L, 300 + i) for i, L in enumerate((40, 9, 23, 61, 5, 33))]
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=512, max_len=100, bf16=bf16), w)
    say(f"case encoder batch composition, {'bf16' if bf16 else 'fp32'}")
    alone = enc.run([ids[2]])[0]
    np.testing.assert_array_equal(alone, enc.run([ids[2]])[0])
    pair = enc.run([ids[3], ids[2]])[1]
    np.testing.assert_array_equal(pair, enc.run([ids[2], ids[0]])[0])
    np.testing.assert_array_equal(alone, pair)
    four = enc.run([ids[0], ids[1], ids[2], ids[3]])[2]
    np.testing.assert_array_equal(four, enc.run(ids)[2])
    np.testing.assert_array_equal(four, enc.run([ids[2], ids[5], ids[4]])[0])
    np.testing.assert_array_equal(four, alone)
    enc.close()


@pytest.mark.parametrize("bf16", [True, False])
def test_result_does_not_depend_on_the_size_of_the_call(bf16):
    """Calls of a few column tiles and of more and more of them (both kernels of the convolutions and of the input projection, every
    number of column tiles per workgroup of the large calls' one): a request's F_enc is, bit for bit, the one it has alone."""
    w = synth.make_encoder_weights(bf16=bf16)
    lens = [130, 33, 1, 160, 77, 150] + [int(x) for x in np.random.default_rng(41).integers(1, 300, size=40)]
    ids = [synth.encoder_ids(L, 3100 + i) for i, L in enumerate(lens)]
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=8192, max_len=300, bf16=bf16), w)
    alone = [enc.run([a])[0] for a in ids[:6]]
    for tiles in (35, 64, 65, 100, 128, 129, 159, 160, 161, 300):
        n = max(k for k in range(6, len(ids) + 1) if sum(lens[:k]) <= 16 * tiles)
        last = 16 * tiles - 7 - sum(lens[:n])             # the call ends inside its last tile
        call = ids[:n] + ([synth.encoder_ids(min(last, 300), 3200 + tiles)] if last > 0 else [])
        say(f"case encoder, {'bf16' if bf16 else 'fp32'}: {len(call)} requests, {sum(a.shape[1] for a in call) / 16:.1f} column tiles")
        for want, got in zip(alone, enc.run(call)):
            np.testing.assert_array_equal(got, want)
    enc.close()


def test_bad_calls_are_rejected():
    w = synth.make_encoder_weights()
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=64, max_len=40), w)
    good = synth.encoder_ids(10, 1)
    bad = good.copy(); bad[1, 3] = 4                     # the prosody tables have four rows
    for case in ([bad], [synth.encoder_ids(41, 2)], [synth.encoder_ids(40, 3), synth.encoder_ids(30, 4)]):
        with pytest.raises(binding.TtsError) as e:
            enc.run(case)
        assert e.value.code == binding.TTS_E_INVAL
    neg = good.copy(); neg[0, 0] = -1
    with pytest.raises(binding.TtsError):
        enc.run([neg])
    assert enc.run([good])[0].shape == (10, 512)
    enc.close()


def test_encoder_output_feeds_the_pool_on_device(weights_fp32):
    """Eq. 1 then Eq. 2 without leaving the device: F_enc of two requests goes from the encoder's output buffer
    straight into tts_pool_add_request; the mel frames equal the oracle decoder run on the oracle encoder's F_enc."""
    import torch
    from oracle import oracle as orc
    we = synth.make_encoder_weights()
    We = orc.EncoderWeights(we)
    lens, steps = [37, 12], [14, 9]
    ids = [synth.encoder_ids(L, 400 + i) for i, L in enumerate(lens)]
    wl = synth.small_workload(2, 12, 37, 9, 14, seed=3)
    pool = make_pool(wl, weights_fp32, max_pool=2, max_enc_len=64, max_steps=16)
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=64, max_len=64), we, stream=pool.stream)
    d_f = torch.empty((sum(lens), 512), dtype=torch.float32, device=pool.device)
    starts = enc.run_device(ids, d_f)
    rids = [pool.add_request(d_f[s:s + L], n) for s, L, n in zip(starts, lens, steps)]
    pool.step_n(max(steps))
    Wd = orc.Weights(weights_fp32)
    worst = 0.0
    say(f"case encoder -> pool on device: tokens {lens}, steps {steps}")
    for rid, a, n in zip(rids, ids, steps):
        f_enc = orc.encoder(We, a).astype(np.float32)
        ref, _, _, _ = orc.pool_decode(wl.dims, Wd, [f_enc], [n], n)
        got = pool.drain_all(rid)
        assert got.shape == (n, 80)
        worst = max(worst, float(np.abs(got - ref[0]).max()))
    say(f"  max abs err {worst:.3e}")
    assert worst <= TOL_F32
    enc.close()
    pool.close()


def test_serving_loop_with_encoder_at_join_matches_oracle(weights_fp32):
    """The arrival-driven loop with module E in front: every request joins with its token ids, the encoder produces
    F_enc on the device at join time, the decoder runs on it.  Mel frames equal the oracle chain (encoder, decoder)."""
    from oracle import oracle as orc
    from paper_2211_13939_amd import stream
    n, chunk = 4, 8
    wl = synth.small_workload(n, 8, 45, 11, 30, seed=61)
    ids = [synth.encoder_ids(int(L), 700 + i) for i, L in enumerate(wl.enc_len)]
    we = synth.make_encoder_weights()
    pool = make_pool(wl, weights_fp32, chunk_frames=chunk, max_pool=3, max_enc_len=64)
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=64, max_len=64), we, stream=pool.stream)
    join = stream.EncoderAtJoin(enc, lambda i: ids[i], 64)
    got = {i: [] for i in range(n)}

    class Collect(stream.GpuBackend):
        def run(self, k):
            self.pool.step_n(k)
            chunk_ids, fin_ids = [], []
            for rid, s in self.live.items():
                s["done"] = min(s["total"], s["done"] + k)
                if s["done"] - s["drained"] >= self.chunk or s["done"] == s["total"]:
                    while True:
                        frames, fin = self.pool.drain_chunk(rid)
                        s["drained"] += frames.shape[0]
                        if frames.shape[0]:
                            got[s["index"]].append(frames.copy())
                            chunk_ids.append(rid)
                        if fin:
                            fin_ids.append(rid)
                        if fin or frames.shape[0] == 0 or s["done"] - s["drained"] < self.chunk:
                            break
            self.pool.sync()
            return None, chunk_ids, fin_ids

    be = Collect(pool, join, wl.n_steps, chunk)
    say(f"case serving loop with encoder at join: tokens {wl.enc_len.tolist()}, steps {wl.n_steps.tolist()}, pool of 3")
    res = stream.simulate(be, np.array([0.0, 0.0, 1e-4, 3e-3]), wl.n_steps, chunk, join_every=1, max_pool=3)
    assert not np.isnan(res.last_chunk_latency_s).any()
    We, Wd = orc.EncoderWeights(we), orc.Weights(weights_fp32)
    worst = 0.0
    for i in range(n):
        T = int(wl.n_steps[i])
        f_enc = orc.encoder(We, ids[i]).astype(np.float32)
        ref, _, _, _ = orc.pool_decode(wl.dims, Wd, [f_enc], [T], T)
        mel = np.concatenate(got[i])
        assert mel.shape == (T, 80)
        worst = max(worst, float(np.abs(mel - ref[0]).max()))
    say(f"  max abs err {worst:.3e}")
    assert worst <= TOL_F32
    enc.close()
    pool.close()


def test_largest_batch_and_a_very_long_request():
    """256 requests in one call (eight of them share a group of workgroups of the recurrence) and, in another call, one request
    of 1000 tokens (the recurrence runs 1000 dependent steps), fp32."""
    from oracle import oracle as orc
    w = synth.make_encoder_weights()
    W = orc.EncoderWeights(w)
    rng = np.random.default_rng(29)
    lens = [int(x) for x in rng.integers(1, 12, size=256)]
    ids = [synth.encoder_ids(L, 800 + i) for i, L in enumerate(lens)]
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=4096, max_len=1000), w)
    say(f"case encoder largest batch: 256 requests, {sum(lens)} tokens; then one request of 1000 tokens")
    got = enc.run(ids)
    worst = 0.0
    for k in (0, 15, 16, 100, 255):
        worst = max(worst, float(np.abs(got[k] - orc.encoder(W, ids[k])).max()))
    long_ids = synth.encoder_ids(1000, 999)
    g = enc.run([long_ids])[0]
    worst_long = float(np.abs(g - orc.encoder(W, long_ids)).max())
    say(f"  max abs err {worst:.3e} (batch), {worst_long:.3e} (1000 tokens)")
    assert worst <= TOL_F32 and worst_long <= TOL_F32
    with pytest.raises(binding.TtsError):
        enc.run(ids + [ids[0]])                # 257 requests
    enc.close()


def test_largest_batch_bf16():
    """256 requests in one call in the two-byte mode: 512 workgroups of the recurrence, two per CU's worth of the chip."""
    from oracle import oracle as orc
    w = synth.make_encoder_weights(bf16=True)
    W = orc.EncoderWeights(w)
    rng = np.random.default_rng(31)
    lens = [int(x) for x in rng.integers(1, 40, size=256)]
    ids = [synth.encoder_ids(L, 1200 + i) for i, L in enumerate(lens)]
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=256 * 40, max_len=64, bf16=True), w)
    say(f"case encoder largest batch, bf16: 256 requests, {sum(lens)} tokens")
    got = enc.run(ids)
    worst = 0.0
    for k in (0, 1, 127, 128, 200, 255):
        assert got[k].shape == (lens[k], 512)
        worst = max(worst, float(np.abs(got[k] - orc.encoder(W, ids[k])).max()))
    say(f"  max abs err {worst:.3e}, {enc.elapsed_ms() * 1e3:.0f} us")
    assert worst <= TOL_BF16
    # bit for bit what smaller calls give
    np.testing.assert_array_equal(got[200], enc.run(ids[150:])[50])
    np.testing.assert_array_equal(got[200], enc.run([ids[200]])[0])
    enc.close()


def test_shared_recurrence_fp32():
    """fp32 weights: how many workgroups share a direction, and how many requests share them, follows from the number of
    requests (every boundary of that rule is here); the order of a sum does not, so results equal those of a request alone."""
    w = synth.make_encoder_weights()
    lens = [3, 1, 8, 2, 5] + [1 + i % 3 for i in range(124)]
    ids = [synth.encoder_ids(L, 1500 + i) for i, L in enumerate(lens)]
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=1024, max_len=16), w)
    alone = {k: enc.run([ids[k]])[0] for k in (0, 1, 2, 7, 8, 15, 31, 63, 128)}
    for n in (2, 8, 9, 16, 17, 32, 33, 64, 65, 128, 129):
        say(f"case encoder, fp32: {n} requests share the recurrence")
        got = enc.run(ids[:n])
        for k in alone:
            if k < n:
                np.testing.assert_array_equal(got[k], alone[k])
    enc.close()


@pytest.mark.parametrize("n", [1, 9, 65])
def test_shared_recurrence_that_gives_up_fp32(n):
    """Workgroups whose partners keep them waiting give up (here at once: no polls are allowed); the call's results are the
    same, bit for bit, and so are those of the call behind it."""
    w = synth.make_encoder_weights()
    ids = [synth.encoder_ids(3 + 7 * i % 20, 1700 + i) for i in range(n)]
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=2048, max_len=32), w)
    want = enc.run(ids)
    say(f"case encoder, fp32: {n} requests, no polls")
    enc.set_wait_polls(0)
    got = enc.run(ids)
    enc.set_wait_polls(1 << 12)
    for a, b, c in zip(want, got, enc.run(ids)):
        np.testing.assert_array_equal(a, b)
        np.testing.assert_array_equal(a, c)
    enc.close()


@pytest.mark.parametrize("polls", [1, 2, 3, 4, 6])
def test_shared_recurrence_that_gives_up_on_the_way_fp32(polls):
    """A few polls are sometimes enough and sometimes not: workgroups give up in the middle of a chain, at steps of their own,
    while their waves may be a step apart.  Every wave leaves at the same step, and the results are the same bits."""
    w = synth.make_encoder_weights()
    ids = [synth.encoder_ids(L, 2100 + i) for i, L in enumerate([90, 4, 33, 61, 1, 17, 48, 25, 70] * 4)]
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=2048, max_len=96), w)
    want = {n: enc.run(ids[:n]) for n in (1, 9, 36)}
    enc.set_wait_polls(polls)
    for n in want:
        say(f"case encoder, fp32: {n} requests, {polls} polls")
        for a, b in zip(want[n], enc.run(ids[:n])):
            np.testing.assert_array_equal(a, b)
    enc.close()


@pytest.mark.parametrize("n,at", [(20, 7), (40, 6), (40, 39), (100, 41), (160, 83), (160, 159)])
def test_shared_recurrence_of_a_long_request_among_short_ones_fp32(n, at):
    """A request of 300 tokens whose companions - alone in its group of workgroups (20 requests), or one, three and seven others
    (40, 100, 160) - end hundreds of steps before it, while the words through which h travels are reused 150 times: the same
    bits as alone, and the oracle's values."""
    from oracle import oracle as orc
    w = synth.make_encoder_weights()
    lens = [1 + (5 * i) % 8 for i in range(n)]
    lens[at] = 300
    ids = [synth.encoder_ids(L, 2300 + i) for i, L in enumerate(lens)]
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=1280, max_len=300), w)
    say(f"case encoder, fp32: request {at} of {n} has 300 tokens, the others up to 8")
    got = enc.run(ids)
    for k in sorted({0, at - 1, at, min(at + 1, n - 1), n - 1}):
        np.testing.assert_array_equal(got[k], enc.run([ids[k]])[0])
    err = float(np.abs(got[at] - orc.encoder(orc.EncoderWeights(w), ids[at])).max())
    say(f"  max abs err {err:.3e}")
    assert err <= TOL_F32
    enc.close()


@pytest.mark.parametrize("bf16,lens", [(False, [400, 399, 400, 66]), (False, [1, 640, 640]), (False, [640, 640, 640, 640, 1]),
                                       (True, [400, 89]), (True, [400, 239]), (True, [1, 330, 310, 640, 7])])
def test_input_projection_of_large_calls(bf16, lens):
    """Calls on the far side of the line from which the convolutions (fp32 25 tiles, two-byte 33) or the input projection (two-byte 25 tiles,
    fp32 160: the calls of 31 and 161) take whole column tiles, with two, four and seven of them per workgroup in the projection, a whole
    and a barely begun last tile: the oracle's values for every request."""
    from oracle import oracle as orc
    w = synth.make_encoder_weights(bf16=bf16)
    W = orc.EncoderWeights(w)
    ids = [synth.encoder_ids(L, 2600 + i) for i, L in enumerate(lens)]
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=2561, max_len=640, bf16=bf16), w)
    say(f"case encoder large calls: {lens} tokens, {'bf16' if bf16 else 'fp32'}")
    for k, got in enumerate(enc.run(ids)):
        assert np.abs(got - orc.encoder(W, ids[k])).max() <= (TOL_BF16 if bf16 else TOL_F32)
    enc.close()


@pytest.mark.parametrize("max_tokens", [64, 100, 400])
def test_requests_that_join_together_are_encoded_together(weights_fp32, max_tokens):
    """Requests that arrive at one time go through the encoder in as few calls as its token limit and the join's buffer allow
    (64, 100 and 400 tokens against 45 + 11 + 30 + 1 + 44 + 20), and each one's frames equal those of a join of its own (small calls, fp32;
    large ones below)."""
    from paper_2211_13939_amd import stream
    lens, steps = [45, 11, 30, 1, 44, 20], [9, 8, 17, 5, 12, 16]
    ids = [synth.encoder_ids(L, 2800 + i) for i, L in enumerate(lens)]
    wl = synth.small_workload(len(lens), 8, 45, 5, 17, seed=67)
    enc_w, got, calls = synth.make_encoder_weights(), [], []
    for together in (False, True):
        pool = make_pool(wl, weights_fp32, chunk_frames=8, max_pool=4, max_enc_len=64, max_steps=20)
        enc = binding.Encoder(binding.make_encoder_config(max_tokens=max_tokens, max_len=45), enc_w, stream=pool.stream)
        run_device, frames = enc.run_device, {i: [] for i in range(len(lens))}
        enc.run_device = lambda a, out: calls.append((together, len(a))) or run_device(a, out)
        join = stream.EncoderAtJoin(enc, lambda i: ids[i], 45)
        be = stream.GpuBackend(pool, join if together else lambda i: join(i), steps, 8)
        drain = pool.drain_chunk

        def keep(rid):
            f, fin = drain(rid)
            frames[be.live[rid]["index"]].append(f.copy())
            return f, fin
        pool.drain_chunk = keep
        say(f"case encoder, joins {'together' if together else 'one by one'}: {lens} tokens, at most {max_tokens} a call")
        stream.simulate(be, np.zeros(len(lens)), steps, 8, max_pool=4)
        got.append([np.concatenate(frames[i]) for i in range(len(lens))])
        enc.close()
        pool.close()
    assert [f.shape[0] for f in got[0]] == steps
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
    assert [n for t, n in calls if not t] == [1] * len(lens)
    assert sum(n for t, n in calls if t) == len(lens) and max(n for t, n in calls if t) == (2 if max_tokens == 64 else 4)


@pytest.mark.parametrize("bf16", [True, False])
def test_large_joins_equal_joins_of_their_own(bf16):
    """Six requests that join together with 877 tokens, 55 column tiles in one call of the encoder (the kernel of large calls) where each
    alone has up to 10 (the kernel of small ones): every F_enc is, bit for bit, that of a join of its own."""
    from paper_2211_13939_amd import stream
    lens = [150, 130, 160, 143, 150, 144]
    ids = [synth.encoder_ids(L, 3300 + i) for i, L in enumerate(lens)]
    enc = binding.Encoder(binding.make_encoder_config(max_tokens=1024, max_len=160, bf16=bf16), synth.make_encoder_weights(bf16=bf16))
    join = stream.EncoderAtJoin(enc, lambda i: ids[i], 160)
    say(f"case encoder at join, {'bf16' if bf16 else 'fp32'}: {lens} tokens together and one by one")
    import torch
    together, groups = {}, []
    with torch.cuda.stream(enc.stream):
        for group, encs in join.many(range(len(lens))):
            groups.append(len(group))
            together.update((i, f.cpu().numpy()) for i, f in zip(group, encs))
        for i in range(len(lens)):
            np.testing.assert_array_equal(together[i], join(i).cpu().numpy())
    assert groups == [6]
    enc.close()
