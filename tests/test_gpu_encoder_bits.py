"""Encoder outputs of the bf16 model bit for bit: the digests are those of the
encoder attention that adds a query's softmax weights tile by tile over its
four lanes. Another order of any fp32 sum of the encoder (attention, GEMM,
norm) changes low bits of the layers after it and with them the digest, though
it stays within every tolerance. Inputs are uniform noise, so that they do not
depend on the host's sine."""
import hashlib

import numpy as np
import pytest

from paper_2507_01021_amd import binding, synth

pytestmark = pytest.mark.gpu

CASES = {
    "base": (synth.BASE.with_(n_enc=3, n_dec=1, n_vocab=64),
             "3d6bc3e68b26c1918f1eeb419fd0522d0aeac281d18be9ab781b8041d6e42383"),
    "large": (synth.LARGE_V3.with_(n_enc=2, n_dec=1, n_vocab=64),
              "01611d068c523a3a89f16291486ca1d0e09b4909fcad0b515c9a0269898deaac"),
}


def digest(shape):
    W = synth.make_weights(shape, 0)
    rng = np.random.default_rng(17)
    segs = [synth.Segment(rng.uniform(-0.5, 0.5, n).astype(np.float32), i, i, [1], 1)
            for i, n in enumerate((16000, 123457, 480000))]
    with binding.Context(synth.pack_blob(W), max_slots=3) as ctx:
        ctx.encode(segs, [0, 1, 2])
        out = [ctx.debug_copy(binding.T_ENC_OUT, i, (1500, shape.d)) for i in range(3)]
    assert all(np.all(np.isfinite(o)) and np.abs(o).max() > 0 for o in out)
    return hashlib.sha256(b"".join(o.tobytes() for o in out)).hexdigest()


@pytest.mark.parametrize("name", list(CASES))
def test_encoder_outputs_keep_their_bits(name):
    shape, want = CASES[name]
    got = digest(shape)
    print(name, got, flush=True)
    assert got == want
