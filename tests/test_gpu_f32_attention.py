"""The two fp32 attention kernels around the counts where one takes over from the other, and values that only some of the rows of a
workgroup see."""
import math

import numpy as np
import pytest
import torch

from oracle import vlc_oracle as orc
import paper_2512_12977_amd as vlc
from helpers import assert_close
from test_gpu_kernels import attention_case

pytestmark = pytest.mark.gpu
DEV = "cuda"


# (row, head) pairs on both sides of 640, where 16 of them begin to share a workgroup, and of 32768, where its wavefronts become one
@pytest.mark.parametrize("Hq,n", [(1, 639), (1, 640), (5, 127), (5, 128), (8, 4095), (8, 4096)])
@pytest.mark.parametrize("D", [64, 128])
def test_attention_around_the_pair_counts(D, Hq, n):
    some = [-1, 0, 1, 15, 16, 30, 31, 32, 63, 64, 127, 128, 159]
    attention_case("f32", Hq, 1, D, [(160, [some[i % len(some)] for i in range(n // 2)]), (161, [some[-1 - i % 9] for i in range(n - n // 2)])],
                   seed=n)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("copies", [4, 40])
def test_attention_values_that_a_row_does_not_see(D, copies):
    """An infinity and a NaN among the values of a key count for the rows that see the key and leave the others alone, also where
    these share a workgroup with them (copies = 40) and where the key is the one that a step is filled up with."""
    lens = [1, 31, 32, 33, 64, 70, 99, 100] * copies
    rng = np.random.default_rng(D + copies)
    n, Hq, Hkv, S = len(lens), 4, 2, 100
    q, K = rng.standard_normal((n, Hq, D)).astype(np.float32), rng.standard_normal((S, Hkv, D)).astype(np.float32)
    V = rng.standard_normal((S, Hkv, D)).astype(np.float32)
    V[99, 0, 3], V[69, 0, 7], V[32, 1, D - 1] = np.inf, np.nan, -np.inf
    out = torch.zeros((n, Hq, D), device=DEV)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    vlc.vlc_sparse_q_attention(dev(q), dev(K), dev(V), dev(np.zeros(n, dtype=np.int32)), dev(np.asarray(lens, dtype=np.int32)),
                               1.0 / math.sqrt(D), out)
    got = out.cpu().numpy().astype(np.float64)
    Vf = np.where(np.isfinite(V), V, 0.0).astype(np.float64)
    want = orc.attention_rows(q.astype(np.float64), K.astype(np.float64), Vf, np.asarray(lens), 1.0 / math.sqrt(D))
    L = np.asarray(lens)
    for head, d, key, odd in ((slice(0, 2), 3, 99, np.inf), (slice(0, 2), 7, 69, np.nan), (slice(2, 4), D - 1, 32, -np.inf)):
        sees = L > key
        np.testing.assert_array_equal(got[sees][:, head, d], np.full((int(sees.sum()), 2), odd))
        assert np.all(np.isfinite(got[~sees][:, head, d]))
        tmp = got[:, head, d]
        tmp[sees] = want[sees][:, head, d]
        got[:, head, d] = tmp
    assert_close(got, want, "f32", "the finite elements")


# Requests of few rows, so that a workgroup of 16 (row, head) pairs has rows of several: (requests, rows of each, heads, kv heads).
# One after the other on MFMA tiles where a tile has few requests (three rows of two heads each: three or four of them), or pair by
# pair; on four wavefronts or one per tile (from 32768 pairs on), the pairs on those of one workgroup or of four (up to 128 tiles).
SHORT = [(60, 3, 4, 2), (800, 3, 4, 2), (2800, 3, 4, 2), (800, 1, 2, 2), (5000, 1, 2, 2), (17000, 1, 2, 2), (641, 1, 1, 1)]


def short_requests(D, requests, rows, Hq, Hkv, seed):
    """Rows of 1 to 76 keys, zero-length ones among them; requests look at overlapping parts of 2000 keys from slots of their own."""
    rng = np.random.default_rng(seed)
    i = np.repeat(np.arange(requests), rows)
    starts, lens = 37 * i % 1921, 1 + i % 37 + 19 * (np.arange(len(i)) % rows)
    lens[5::97] = 0
    q = rng.standard_normal((len(i), Hq, D)).astype(np.float32)
    K, V = [rng.standard_normal((2000, Hkv, D)).astype(np.float32) for _ in range(2)]
    return starts, lens, q, K, V


def attended(starts, lens, q, K, V):
    """(rows, GPU result, oracle's) of every row, of some thousands where there are more; the oracle gets zeros for what is no number."""
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    out, scale = torch.full(q.shape, 3.0, device=DEV), 1.0 / math.sqrt(q.shape[2])
    vlc.vlc_sparse_q_attention(dev(q), dev(K), dev(V), dev(starts.astype(np.int32)), dev(lens.astype(np.int32)), scale, out)
    Kf, Vf = [np.where(np.isfinite(a), a, 0.0).astype(np.float64) for a in (K, V)]
    rows = np.arange(0, len(lens), 1 + len(lens) // 3000)
    want = np.concatenate([orc.attention_rows(q[i:i + 1].astype(np.float64), Kf[a:a + max(L, 1)], Vf[a:a + max(L, 1)], np.asarray([L]), scale)
                           for i, a, L in zip(rows, starts[rows], lens[rows])])
    return rows, out.cpu().numpy().astype(np.float64)[rows], want


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("requests,rows,Hq,Hkv", SHORT)
def test_attention_of_short_requests(D, requests, rows, Hq, Hkv):
    """Values that are no numbers count in the rows that see them and in no other, whatever request shares the workgroup."""
    starts, lens, q, K, V = short_requests(D, requests, rows, Hq, Hkv, 5 + D)
    odd = {(key, key % Hkv, 3 * key % D): [np.inf, -np.inf, np.nan][key % 3] for key in range(11, 2000, 173)}
    for at, value in odd.items():
        V[at] = value
    checked, got, want = attended(starts, lens, q, K, V)
    first, end, g = starts[checked], (starts + lens)[checked], Hq // Hkv
    for (key, kvh, d), value in odd.items():
        sees = (first <= key) & (key < end)
        heads = slice(g * kvh, g * kvh + g)
        np.testing.assert_array_equal(got[sees][:, heads, d], np.full((int(sees.sum()), g), value))
        for h in range(g * kvh, g * kvh + g):
            got[sees, h, d] = want[sees, h, d]
    assert_close(got, want, "f32", "the finite elements")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("requests,rows,Hq,Hkv", SHORT)
def test_attention_nan_scores_of_short_requests(D, requests, rows, Hq, Hkv):
    """A key that is no number makes the rows that see it NaN, in the heads of its kv head, and no others."""
    starts, lens, q, K, V = short_requests(D, requests, rows, Hq, Hkv, 6 + D)
    keys = range(11, 2000, 173)
    for key in keys:
        K[key, key % Hkv, 5 * key % D] = np.nan
    checked, got, want = attended(starts, lens, q, K, V)
    nan = np.zeros(got.shape, dtype=bool)
    for key in keys:
        sees = (starts[checked] <= key) & (key < (starts + lens)[checked])
        nan[sees, Hq // Hkv * (key % Hkv):Hq // Hkv * (key % Hkv + 1)] = True
    np.testing.assert_array_equal(np.isnan(got), nan)
    assert_close(np.where(nan, 0.0, got), np.where(nan, 0.0, want), "f32", "the rows that do not see such a key")
