"""The bf16 encoder GEMMs take one of four tile sizes by the number of
workgroups a launch has (1 segment: mostly 64 x 64, 5: 128 x 128, 32: 256 x
256 or 256 x 128), every one with partial last tiles (1500 rows per segment).
A result is the same sum over k in the same order with every tile, so a
segment's encoder output does not depend on the size of its pass (bit-exact).
The solo passes are checked against the oracle in test_gpu_parity."""
import numpy as np
import pytest

from paper_2507_01021_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [384, 512, 768, 1280])
def test_pass_sizes_give_identical_encoder_outputs(d):
    shape = synth.BASE.with_(d=d, n_head=d // 64, n_enc=1, n_dec=1, n_vocab=64)
    W = synth.make_weights(shape, 0)
    segs = synth.fixed_batch(shape, [16000 * (1 + i % 29) for i in range(32)], 1, seed=71)
    for s in segs:
        s.prompt = [1]
    look = [0, 4, 31]
    with binding.Context(synth.pack_blob(W), max_slots=128, max_encode_batch=32) as ctx:
        ctx.encode(segs, list(range(32)))
        full = {i: ctx.debug_copy(binding.T_ENC_OUT, i, (1500, d)) for i in look}
        ckv = ctx.debug_copy(binding.T_CROSS_K, 4, (1, d // 64, 1500, 64))
        for i in look:
            ctx.encode([segs[i]], [32 + i])
            assert np.array_equal(full[i], ctx.debug_copy(binding.T_ENC_OUT, 0, (1500, d))), i
        assert np.array_equal(ckv, ctx.debug_copy(binding.T_CROSS_K, 36, (1, d // 64, 1500, 64)))
        ctx.encode(segs[:5], list(range(64, 69)))
        assert np.array_equal(full[4], ctx.debug_copy(binding.T_ENC_OUT, 4, (1500, d)))
    assert all(np.all(np.isfinite(v)) and np.abs(v).max() > 0 for v in full.values())
    print(f"d {d}: passes of 1, 5 and 32 identical", flush=True)
