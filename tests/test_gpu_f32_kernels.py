"""The fp32 model's matrix-core kernels where their dispatch and tile edges
lie: 16 segments take the 128 x 128 GEMM tiles (at least 512 of them), one
segment the 64 x 64 tiles, both with partial last tiles (1500 rows, a head of
an odd number of ids). A result is the same sum over k in the same order with
either tile, so a segment's logits do not depend on its pass (bit-exact), and
they match the oracle within the fp32 tolerance."""
import numpy as np
import pytest

from paper_2507_01021_amd import binding, synth

from parity import TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_vocab", [2, 255, 258])
def test_f32_pass_equals_solo_and_oracle(n_vocab):
    from oracle import model as M
    import oracle
    shape = synth.CTC_TINY.with_(n_enc=1, n_vocab=n_vocab)
    W = synth.make_weights(shape, 0)
    segs = synth.fixed_batch(shape, [16000 + 29000 * i for i in range(16)], 1500, seed=41)
    with binding.Context(synth.pack_blob(W), max_slots=16, max_encode_batch=16) as ctx:
        ctx.encode(segs, list(range(16)))
        got = [ctx.debug_copy(binding.T_CTC_LOGITS, i, (1500, n_vocab)) for i in range(16)]
        for i in (0, 7, 15):
            ctx.encode([segs[i]], [0])
            assert np.array_equal(got[i], ctx.debug_copy(binding.T_CTC_LOGITS, 0, (1500, n_vocab))), i
    E = M.encoder(W, shape, oracle.log_mel_segment(segs[7].audio, shape.n_mels)[None])[0]
    want = E @ W["ctc.w"].astype(np.float64).T + W["ctc.b"]
    err = (np.abs(got[7] - want).max(axis=1) / np.abs(want).max(axis=1)).max()
    print(f"n_vocab {n_vocab}: logits rel err {err:.2e}", flush=True)
    assert err < TOL["f32"]
