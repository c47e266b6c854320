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
