"""Decode steps whose cross-attention is split by chunk (few rows and heads)
against unsplit ones: a slot's logits do not depend on the other rows of its
step (bit-exact), so stepping the slots in batches on both sides of each
model's limit, alone, and through the allocation-free step must agree."""
import numpy as np
import pytest

from paper_2507_01021_amd import binding, synth

pytestmark = pytest.mark.gpu

CASES = {
    # (shape, rows): split up to 80 (row, head) pairs in bf16, 96 in fp32, 16 rows at most
    "base": (synth.BASE, [1, 5, 10, 11, 17]),          # 8 heads: 10 rows split, 11 not
    "large": (synth.LARGE_V3.with_(n_vocab=1000), [1, 4, 5]),  # 20 heads: 4 rows split, 5 not
    "tiny": (synth.TINY, [1, 16, 17]),                 # 6 heads, fp32: 16 rows split, 17 not
    "wide": (synth.TINY.with_(d=2048, n_head=32, n_vocab=500), [1, 3, 4]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_split_steps_equal_unsplit(name):
    shape, rows = CASES[name]
    shape = shape.with_(n_enc=1, n_dec=2)
    W = synth.make_weights(shape, 0)
    n = max(rows)
    segs = synth.fixed_batch(shape, [16000 * (2 + i) for i in range(n)], 40, seed=61)
    rng = np.random.default_rng(6)
    for s in segs:
        s.prompt = rng.integers(0, shape.n_vocab, 3).tolist()
    ref = None
    with binding.Context(synth.pack_blob(W), max_slots=n) as ctx:
        for k in rows + [0]:
            ctx.encode(segs, list(range(n)))
            got = []
            for step in range(5):
                forced = np.arange(n) % shape.n_vocab
                lg = np.empty((n, shape.n_vocab), np.float32)
                for at in range(0, n, max(k, 1)):
                    part = list(range(at, min(n, at + max(k, 1))))
                    if k == 0:  # alone, the first two steps allocation-free
                        if step < 2:
                            ctx.decode_step_noalloc(part)
                            lg[part] = 0
                            continue
                    lg[part] = ctx.decode_step(part, forced=forced[part], logits=True)[1]
                got.append(lg)
            got = np.stack(got)
            if ref is None:
                ref = got
            assert np.array_equal(ref[2:], got[2:]), (name, k)
            print(f"{name}: {k or 1} rows a step{'' if k else ', allocation-free'}: equal", flush=True)
            for s in range(n):  # run the slots to their end
                while True:
                    try:
                        ctx.decode_step([s])
                    except binding.WhisperError as e:
                        assert e.status == binding.E_STATE
                        break


@pytest.mark.parametrize("name,rows", [("base", [1, 2, 3, 4, 5, 6, 10]), ("large", [2, 4]), ("tiny", [1, 2, 5, 10, 11]),
                                       ("wide", [1, 2, 3])])
def test_allocation_free_split_steps_equal_regular_ones(name, rows):
    """The allocation-free step keeps the chunks' results in the activations of
    its MLP: as many rows as fit there (five of 16 in bf16, ten in fp32) are
    split, on both sides of that limit. Two such steps, then the logits of a
    regular one against three regular steps."""
    shape = CASES[name][0].with_(n_enc=1, n_dec=2, n_vocab=1000)
    W = synth.make_weights(shape, 0)
    n = max(rows)
    segs = synth.fixed_batch(shape, [16000 * (2 + i) for i in range(n)], 40, seed=62)
    for i, seg in enumerate(segs):
        seg.prompt = [1 + i]
    with binding.Context(synth.pack_blob(W), max_slots=n) as a, binding.Context(synth.pack_blob(W), max_slots=n) as b:
        a.encode(segs, list(range(n)))
        b.encode(segs, list(range(n)))
        for k in rows:
            part = list(range(n - k, n))
            for _ in range(2):
                a.decode_step(part)
                b.decode_step_noalloc(part)
            ta, la = a.decode_step(part, logits=True)
            tb, lb = b.decode_step(part, logits=True)
            assert np.all(np.isfinite(la)) and np.array_equal(la, lb) and np.array_equal(ta, tb), (name, k)
            print(f"{name}: {k} rows allocation-free: equal", flush=True)
