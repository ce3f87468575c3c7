"""The engine's dispatch rules on the host: which kernel variant a launch of
given sizes takes."""
import os

import pytest

from paper_2507_01021_amd import binding
from paper_2507_01021_amd.binding import DTYPE_BF16, DTYPE_F32

WIDTHS = [384, 512, 768, 1024, 1280, 1536, 2048]


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(binding.LIB_PATH):
        pytest.skip("library not built (python -m paper_2507_01021_amd.build)")
    return binding.load()


def projections(d):
    """(output features, split-K parts, waves) of a decoder layer's projections."""
    return [(3 * d, 1, 4), (d, 4, 4), (d, 1, 8), (d, 1, 4), (4 * d, 1, 4), (d, 8, 4)]


def many(dtype, MA, KS, n, NW):
    return binding.test_kernel_choice(binding.CHOICE_DEC_PROJ, dtype, MA, KS, n, NW)


@pytest.mark.parametrize("dtype", [DTYPE_F32, DTYPE_BF16])
def test_steps_of_few_rows_keep_the_skinny_kernel(dtype):
    for d in WIDTHS:
        for MA, KS, NW in projections(d):
            if NW == 8 and dtype == DTYPE_F32:
                continue
            for n in (1, 16, 17, 64):
                assert many(dtype, MA, KS, n, NW) == 0, (d, MA, KS, n, NW)


def test_prefill_chunks_take_the_kernel_for_many_rows():
    # 2048 rows: every projection from d = 768 on; 1520 rows: all but the residual projection
    for MA, KS, NW in projections(768):
        if (MA, KS, NW) == (768, 1, 4):
            continue  # 192 workgroups of a short reduction
        assert many(DTYPE_BF16, MA, KS, 2048, NW) == 1, (MA, KS, NW)
        assert many(DTYPE_BF16, MA, KS, 1520, NW) == (NW == 4), (MA, KS, NW)


def shared(dtype, slots, per_slot, H):
    groups = slots * ((per_slot + 7) // 8)
    return binding.test_kernel_choice(binding.CHOICE_PREFILL_CROSS, dtype, slots * per_slot, H, groups)


@pytest.mark.parametrize("dtype", [DTYPE_F32, DTYPE_BF16])
def test_short_prompts_keep_one_row_per_workgroup(dtype):
    """One row per slot (a prompt of two tokens) never pays for eight, and few
    (row, head) pairs run at once anyway."""
    for H in (6, 8, 12, 16, 20, 24, 32):
        for slots in range(1, 129):
            assert shared(dtype, slots, 1, H) == 0, (H, slots)
        if dtype == DTYPE_BF16:
            for slots in range(1, 33):
                assert shared(dtype, slots, 2, H) == 0, (H, slots)
            assert shared(dtype, 4, 5, H) == 0, H


@pytest.mark.parametrize("dtype", [DTYPE_F32, DTYPE_BF16])
def test_long_prompts_share_their_slots_rows(dtype):
    for H in (6, 8, 12, 16, 20, 24, 32):
        for slots in (1, 4, 16, 32):
            per = 223 if slots > 1 else 440
            assert shared(dtype, slots, min(per, 2048 // slots), H) == 1, (H, slots)


def tile(MA, MB, K, batch=1, dtype=DTYPE_BF16):
    return binding.test_kernel_choice(binding.CHOICE_ENC_GEMM, dtype, MA, MB, K, batch)


def test_gemm_tiles():
    # a 128 x 128 tile for 144 of them, 64 x 64 below
    assert tile(128 * 12, 128 * 11, 1280) == 64 and tile(128 * 12, 128 * 12, 1280) == 128
    # one round of 256 x 256 from 144 tiles on
    assert tile(256 * 11, 256 * 13, 1280) == 128 and tile(256 * 12, 256 * 12, 1280) == 256
    # further rounds 60 % full, 308 of 512, unless the reduction is long
    assert tile(256 * 308, 256, 1280) == 256 and tile(256 * 307, 256, 1280) == 128
    assert tile(256 * 307, 256, 2047) == 128 and tile(256 * 257, 256, 2048) == 256
    # short reductions: 75 % full, 384 of 512, else 750 tiles of 256 x 128
    assert tile(256, 128 * 749, 640) == 128 and tile(256, 128 * 750, 640) == 384
    assert tile(256 * 384, 256, 640) == 256 and tile(256 * 383, 256, 640) == 384
    assert tile(256, 128 * 750, 704) == 256
    # the 256 x 256 kernel needs two K tiles
    assert tile(256 * 16, 256 * 16, 128) == 256 and tile(256 * 16, 256 * 16, 64) == 128
    assert tile(128 * 22, 128 * 23, 384, dtype=DTYPE_F32) == 64 and tile(128 * 32, 128 * 16, 384, dtype=DTYPE_F32) == 128


def test_bad_choice_arguments_are_refused():
    for args in [(binding.CHOICE_DEC_PROJ, DTYPE_BF16, 1280, 1, 0, 4), (binding.CHOICE_DEC_PROJ, DTYPE_F32, 1280, 1, 1, 8),
                 (binding.CHOICE_DEC_PROJ, 2, 1280, 1, 1, 4), (binding.CHOICE_DEC_PROJ, DTYPE_BF16, 1280, 1, 1), (99, 0, 1),
                 (binding.CHOICE_ENC_GEMM, DTYPE_BF16, (1 << 20) + 1, 256, 256, 1)]:
        with pytest.raises(binding.WhisperError) as e:
            binding.test_kernel_choice(*args)
        assert e.value.status == binding.E_INVAL
