"""whisper_ctx_set_stream: a context on the caller's streams computes what it
does on its own, ordered with the caller's work there; choosing a stream costs
no device work, does not wait for the stream chosen and leaves a pending error
of the caller alone."""
import ctypes as C
import time

import numpy as np
import pytest

from paper_2507_01021_amd import binding, synth

pytestmark = pytest.mark.gpu

SHAPE = synth.BASE.with_(n_enc=2, n_dec=2, n_vocab=4000)
N = 33  # two decode chains; two parts per encoder pass


@pytest.fixture(scope="module")
def blob():
    return synth.pack_blob(synth.make_weights(SHAPE, 0))


def segments():
    segs = synth.fixed_batch(SHAPE, [16000 * (1 + i % 7) for i in range(N)], 6, seed=23)
    rng = np.random.default_rng(3)
    for s in segs:
        s.prompt = rng.integers(0, SHAPE.n_vocab, 2).tolist()
    return segs


def steps(ctx, segs, device_audio=None):
    """Encoder outputs, then logits of every step of all slots."""
    ctx.encode(segs, list(range(N)), device_audio)
    out = [ctx.debug_copy(binding.T_ENC_OUT, 0, (1500, SHAPE.d))]
    for _ in range(7):
        out.append(ctx.decode_step(list(range(N)), logits=True)[1])
    return out


def equal(a, b):
    return len(a) == len(b) and all(np.array_equal(x, y) for x, y in zip(a, b))


def hip():
    for line in open("/proc/self/maps"):
        if "libamdhip64" in line:
            return C.CDLL(line.split()[-1])
    raise AssertionError("no HIP runtime in this process")


def test_callers_streams_compute_the_same(blob):
    import torch
    segs = segments()
    with binding.Context(blob, max_slots=N) as ctx:
        want = steps(ctx, segs)
        queue = ctx.transcribe(segs)
        streams = [torch.cuda.Stream() for _ in range(5)]
        for i, s in enumerate([*streams, None, streams[0]]):
            ctx.set_stream(s.cuda_stream if s else None)
            assert equal(want, steps(ctx, segs)), i
            got = ctx.transcribe(segs)
            assert all(np.array_equal(a["tokens"], b["tokens"]) for a, b in zip(queue, got)), i
            print(f"stream {i}: equal", flush=True)


def test_work_is_ordered_with_the_callers(blob):
    """Audio that the caller's stream writes after a long kernel is what the
    encoder reads; a token buffer is read on that stream right after the step."""
    import torch
    segs = segments()
    with binding.Context(blob, max_slots=N) as ctx:
        want = steps(ctx, segs)
        s = torch.cuda.Stream()
        ctx.set_stream(s.cuda_stream)
        src = [torch.from_numpy(x.audio).cuda() for x in segs]
        dst = [torch.full_like(x, 0.25) for x in src]
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            torch.cuda._sleep(20_000_000)
            for a, b in zip(dst, src):
                a.copy_(b)
        assert equal(want, steps(ctx, segs, [x.data_ptr() for x in dst]))
        ctx.encode(segs, list(range(N)))
        tok = torch.full((N,), -7, dtype=torch.int32, device="cuda")
        seen = []
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            for _ in range(7):
                torch.cuda._sleep(1_000_000)
                ctx.decode_step_noalloc(list(range(N)), tok.data_ptr())
                seen.append(tok.clone())
        s.synchronize()
        for step in range(1, 7):
            assert np.array_equal(seen[step].cpu().numpy(), want[1 + step].argmax(1)), step


def test_choosing_a_stream_waits_for_nothing_of_it_and_keeps_errors(blob):
    import torch
    lib = hip()
    lib.hipGetLastError.restype = lib.hipSetDevice.restype = C.c_int
    streams = [torch.cuda.Stream() for _ in range(8)]
    with binding.Context(blob, max_slots=N) as ctx:
        with torch.cuda.stream(streams[0]):
            torch.cuda._sleep(100_000_000)
        ctx.set_stream(streams[0].cuda_stream)
        assert not streams[0].query()  # still busy
        streams[0].synchronize()
        took = []
        for i in range(200):
            t = time.perf_counter()
            ctx.set_stream(streams[i % 8].cuda_stream)
            took.append(time.perf_counter() - t)
        print(f"set_stream: median {1e6 * np.median(took):.1f} us, largest {1e6 * max(took):.1f} us", flush=True)
        # no launch and no wait: a kernel launched and waited for takes more than 10 us
        assert np.median(took) < 8e-6
        assert lib.hipGetLastError() == 0
        err = lib.hipSetDevice(9999)
        assert err != 0
        ctx.set_stream(streams[1].cuda_stream)
        assert lib.hipGetLastError() == err
        assert lib.hipGetLastError() == 0


def test_two_contexts_on_streams_of_their_own(blob):
    import torch
    segs = segments()
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with binding.Context(blob, max_slots=N) as x, binding.Context(blob, max_slots=N) as y:
        want = steps(x, segs)
        x.set_stream(a.cuda_stream)
        y.set_stream(b.cuda_stream)
        x.encode(segs, list(range(N)))
        y.encode(segs[::-1], list(range(N)))
        for step in range(7):
            p = x.decode_step(list(range(N)), logits=True)[1]
            q = y.decode_step(list(range(N)), logits=True)[1]
            assert np.array_equal(p, want[1 + step]) and np.array_equal(q, want[1 + step][::-1]), step


def test_step_captured_on_the_callers_stream(blob):
    """An allocation-free step recorded into a graph of the caller's, replayed
    with eager work and synchronisations between the replays."""
    import torch
    segs = segments()
    with binding.Context(blob, max_slots=N) as ctx:
        want = steps(ctx, segs)
        ctx.encode(segs, list(range(N)))
        s = torch.cuda.Stream()
        ctx.set_stream(s.cuda_stream)
        tok = torch.full((N,), -7, dtype=torch.int32, device="cuda")
        ctx.decode_step_noalloc(list(range(N)))  # inside the prompt; not captured
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            ctx.decode_step_noalloc(list(range(N)), tok.data_ptr())
        for step in range(1, 6):
            tok.fill_(-7)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(tok.cpu().numpy(), want[1 + step].argmax(1)), step
