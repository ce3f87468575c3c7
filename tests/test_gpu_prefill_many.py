"""Prefill of many rows: the projections' and the cross-attention's variants
for many rows (many_kernel, skinny_ln_kernel with 32 weight rows,
cross_attn_rows_kernel), those that few rows keep, and the boundary between
two chunks of 2048 rows, which falls inside a slot's prompt. Each of them keeps
the order of every sum of the one-position step, so the logits after a
prefilled prompt equal those of the prompt fed one position per step bit for
bit."""
import numpy as np
import pytest

from paper_2507_01021_amd import binding, synth

pytestmark = pytest.mark.gpu

CASES = {
    # few rows: one workgroup per row
    "base-short": (synth.BASE, [2, 3, 5, 2]),
    "tiny-short": (synth.TINY, [2, 3, 5, 2]),
    # enough of them to share a workgroup in fp32, not in bf16
    "base-three": (synth.BASE, [4] * 16),
    "tiny-three": (synth.TINY, [4] * 16),
    # rows: one group, a group edge, a full and a partial 64-row group
    "base-few": (synth.BASE, [2, 9, 10, 66, 130]),
    # 2300 rows: two chunks, the second starting inside a prompt
    "base-chunks": (synth.BASE, [447, 440, 1, 300, 391, 8, 447, 275]),
    "tiny-chunks": (synth.TINY, [447, 440, 1, 300, 391, 8, 447, 275]),
    # the widest model
    "wide": (synth.BASE.with_(d=2048, n_head=32, n_enc=1, n_dec=2, n_vocab=1000), [129, 300]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_prefill_of_many_rows_equals_steps(name):
    shape, lens = CASES[name]
    if name != "wide":
        shape = shape.with_(n_enc=1, n_dec=2, n_vocab=4000)
    W = synth.make_weights(shape, 0)
    blob = synth.pack_blob(W)
    n = len(lens)
    segs = synth.fixed_batch(shape, [min(480000, 16000 * (3 + 3 * i)) for i in range(n)], 1, seed=51)
    rng = np.random.default_rng(5)
    for s, k in zip(segs, lens):
        s.prompt = rng.integers(0, shape.n_vocab, k).tolist()
    got = {}
    for pf in (0, 1):
        with binding.Context(blob, max_slots=n, prefill=pf) as ctx:
            ctx.encode(segs, list(range(n)))
            rows = []
            for i, k in enumerate(lens):
                for _ in range(0 if pf else k - 1):
                    ctx.decode_step([i])
                rows.append(ctx.decode_step([i], logits=True)[1][0].copy())
        got[pf] = rows
        print(f"{name}: prefill {pf} done", flush=True)
    for i in range(n):
        assert np.all(np.isfinite(got[1][i]))
        assert np.array_equal(got[0][i], got[1][i]), (name, i, lens[i])
