"""The bf16 encoder GEMMs take one of four tile sizes by the number of
workgroups a launch has (1 segment: mostly 64 x 64, 5: 128 x 128, 32: 256 x
256 or, at widths up to 640, 256 x 128; the test makes sure that its passes
take all of them), every one with partial last tiles (1500 rows per segment).
A result is the same sum over k in the same order with every tile, so a
segment's encoder output does not depend on the size of its pass (bit-exact).
The solo passes are checked against the oracle in test_gpu_parity."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2507_01021_amd import binding, synth

pytestmark = pytest.mark.gpu


def tiles(d, n):
    """The tiles that the launches of a pass of n segments take: the conv stem,
    a layer's GEMMs over the larger half of the pass, the cross K/V GEMMs."""
    def tile(MA, MB, K, batch=1):
        return binding.test_kernel_choice(binding.CHOICE_ENC_GEMM, binding.DTYPE_BF16, MA, MB, K, batch)
    M = 1500 * (n - n // 2)
    return [tile(d, 3000, 384, n), tile(d, 1500, 3 * d, n), tile(2 * d, M, d), tile(M, d, d), tile(d, M, d),
            tile(4 * d, M, d), tile(d, M, 4 * d), tile(1500 * n, d, d), tile(d, 1500 * n, d)]


@pytest.mark.parametrize("d", [384, 512, 768, 1024, 1280, 1536, 2048])
def test_pass_sizes_give_identical_encoder_outputs(d):
    solo, five, full = tiles(d, 1), tiles(d, 5), tiles(d, 32)
    want = {384: {64, 128, 256, 384}, 512: {64, 128, 256, 384}}.get(d, {64, 128, 256} if d <= 1280 else {128, 256})
    assert set(solo + five + full) == want
    assert sum(a != b for a, b in zip(solo, full)) >= 6
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


CHILD = """
from paper_2507_01021_amd import binding
import test_gpu_encoder_bits as bits
try:
    print("digest", bits.digest(bits.CASES["base"][0]))
except binding.WhisperError as e:
    print("error", e.status)
"""


@pytest.mark.parametrize("var,value", [("WHISPER_GEMM_TILE", "64"), ("WHISPER_GEMM_TILE", "128"),
                                       ("WHISPER_GEMM_TILE", "256"), ("WHISPER_GEMM_TILE", "384"),
                                       ("WHISPER_GEMM_H", "0"), ("WHISPER_GEMM_H", "1"), ("WHISPER_GEMM_TILE", "100")])
def test_forced_tiles_give_the_same_bits(var, value):
    """The switches are read once per process: each in a child of its own."""
    import test_gpu_encoder_bits as bits
    here = os.path.dirname(os.path.abspath(__file__))
    env = {**os.environ, var: value, "PYTHONPATH": os.pathsep.join([os.path.dirname(here), here])}
    out = subprocess.run([sys.executable, "-c", CHILD], env=env, capture_output=True, text=True, timeout=100, check=True)
    want = f"error {binding.E_INVAL}" if value == "100" else "digest " + bits.CASES["base"][1]
    print(var, value, out.stdout.strip(), flush=True)
    assert out.stdout.strip().splitlines()[-1] == want
