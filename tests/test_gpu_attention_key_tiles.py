"""The bf16 attention around the edges of its tiles: 16 keys of a score tile, 32 of a value fragment, 64 of a block, 16 virtual rows
(query row, head of the kv group) of an accumulator - and groups of heads that straddle them."""
import pytest

from test_gpu_kernels import attention_case

pytestmark = pytest.mark.gpu

KEYS = [1, 4, 5, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 79, 80, 81, 127, 128, 129, 191, 192, 193]


@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (3, 1), (5, 1), (7, 1), (14, 2), (16, 1), (17, 1), (24, 8)])
def test_key_counts_around_the_tiles(Hq, Hkv):
    attention_case("bf16", Hq, Hkv, 128, [(193, [k - 1 for k in KEYS])], seed=101 + Hq)


@pytest.mark.parametrize("Hq,Hkv,rows", [(7, 1, 2), (7, 1, 3), (7, 1, 18), (7, 1, 19), (4, 1, 4), (4, 1, 5), (16, 1, 1), (16, 1, 9),
                                         (5, 1, 26), (2, 2, 129)])
def test_rows_around_the_row_tiles(Hq, Hkv, rows):
    """Row counts one row short of, at and past a 16-row accumulator tile or a workgroup's 128 virtual rows."""
    attention_case("bf16", Hq, Hkv, 128, [(300, list(range(300 - rows, 300)))], seed=7 * rows + Hq)


@pytest.mark.parametrize("Hq,Hkv", [(7, 1), (8, 2)])
def test_requests_that_meet_inside_a_row_tile(Hq, Hkv):
    reqs = [(16, [0, 15]), (33, [32]), (64, [-1, 63, 31]), (65, [64, 0]), (130, list(range(110, 130)))]
    attention_case("bf16", Hq, Hkv, 128, reqs, seed=19)
