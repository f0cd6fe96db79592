"""The shape rules that choose a kernel, at points where both sides were measured."""

import pytest

from routes import f32_loops, f32_parts, f32_small, gsum_rows, skinny_down, skinny_logits

# (vocab, tokens, hidden): 32-row blocks measured faster than the ring, and slower
FEW = [(2000, 1, 512), (2000, 1, 8192), (8192, 32, 4096), (10000, 16, 4096), (16384, 8, 8192), (16384, 24, 4096),
       (4096, 64, 2048), (2000, 128, 8192), (4096, 128, 1024), (3000, 129, 4096), (2000, 256, 512), (1000, 512, 2048),
       (48000, 8, 2048), (6000, 48, 8192), (8192, 96, 1024), (33000, 8, 4096), (48000, 4, 5120)]
MANY = [(32000, 1, 4096), (32000, 8, 4096), (32000, 1, 5120), (32000, 64, 8192), (12000, 32, 5120), (20000, 16, 2048),
        (6000, 64, 4096), (10000, 33, 1024), (6000, 128, 4096), (8192, 128, 4096), (3000, 256, 4096), (2000, 500, 4096),
        (32000, 230, 5120), (64000, 500, 8192), (58000, 1, 4096), (33000, 16, 4096)]


@pytest.mark.parametrize("vocab,n,h", FEW)
def test_few_rows_take_small_blocks(vocab, n, h):
    assert skinny_logits(vocab, n, h)


@pytest.mark.parametrize("vocab,n,h", MANY)
def test_many_rows_take_the_ring(vocab, n, h):
    assert not skinny_logits(vocab, n, h)


def test_down_projection():
    assert skinny_down(512, 1, 1344) and skinny_down(1024, 250, 1024) and skinny_down(2048, 128, 2048)
    assert not skinny_down(2048, 250, 2048) and not skinny_down(5120, 8, 13824) and not skinny_down(2048, 1, 5504)


def test_row_sums_of_the_logit_gradient():
    for n, v in [(2048, 4000), (2048, 64000), (3008, 32000), (4096, 8000), (4096, 16000), (4096, 28000), (8192, 20000)]:
        assert gsum_rows(False, n, v) == 32
    for n, v in [(4096, 32000), (8192, 16000), (8192, 24000), (8192, 32000)]:
        assert gsum_rows(False, n, v) == 128


# (128 x 128 tiles, 64 x 64 tiles, K) where the small tiles measured faster, and slower
@pytest.mark.parametrize("tiles,small,k", [(16, 64, 512), (128, 512, 1000), (144, 517, 512), (260, 1040, 512), (352, 1408, 2048),
                                           (520, 2072, 2304)])
def test_f32_small_tiles(tiles, small, k):
    assert f32_small(tiles, small, k)


@pytest.mark.parametrize("tiles,small,k", [(204, 810, 128), (175, 686, 128), (180, 720, 512), (256, 1024, 512), (380, 1520, 128),
                                           (630, 2375, 128), (671, 2541, 448), (720, 2880, 768), (1008, 4032, 512)])
def test_f32_large_tiles(tiles, small, k):
    assert not f32_small(tiles, small, k)


def test_f32_parts_where_the_tiles_come_out_even():
    assert [f32_parts(*t) for t in [(207, 765), (175, 686), (380, 1520), (128, 512)]] == [4] * 4
    assert [f32_parts(*t) for t in [(256, 1024), (630, 2375), (720, 2880), (1008, 4032)]] == [1] * 4


def test_f32_loops():
    assert [t for t in (256, 512, 513, 768, 769, 1024, 1025, 1280, 1281) if f32_loops(t)] == [513, 768, 1025, 1280]
