"""The offline weight quantizer where short rows of many channels take workgroups of 256 threads with four lanes a start: the row
lengths and counts around that rule, against the oracle, with rows that crowd into few cells or are fitted almost exactly among them,
and more starts than a workgroup takes at once."""
import numpy as np
import pytest
import torch

import paper_2505_18663_amd as dvdq
from test_gpu_bgr import DEV, _exact_listing_error, compare

pytestmark = pytest.mark.gpu


def rows_of_every_kind(N, K):
    rng = np.random.default_rng(N + K)
    w = rng.standard_normal((N, K)) * 0.02
    g = rng.standard_normal((7, K))
    w[0] = np.where(rng.random(K) < 0.9, 0.0, g[0])
    w[1] = 5.0 + 1e-3 * g[1]
    w[2] = np.round(g[2] * 4) / 8
    w[3] = 0.25 * (rng.integers(0, 16, K) - 6) + 1e-7 * g[3]
    w[4] = g[4] * 0.02 + np.eye(1, K, 1)[0] * 1e6
    w[5] = g[5] * 1e-30
    w[6] = np.exp(3 * g[6])
    w[7] = -0.25
    return w.astype(np.float32)


@pytest.mark.parametrize("N,K", [(257, 2), (300, 34), (260, 510), (257, 4608), (257, 4610), (512, 4610), (513, 4610), (513, 6144), (513, 6146)])
@pytest.mark.parametrize("search", [dvdq.BGR_LISTING, dvdq.BGR_BEST_OF_ALL])
def test_row_lengths_and_counts_around_the_rule(N, K, search):
    print(compare(rows_of_every_kind(N, K), f"N{N} K{K} search{search}", n_steps=9, max_refine=3, search=search))


@pytest.mark.parametrize("n_steps,K", [(127, 96), (131, 96), (300, 258)])   # 64 starts at a time, half of n_steps altogether
def test_more_starts_than_a_workgroup_takes_at_once(n_steps, K):
    print(compare(rows_of_every_kind(300, K), f"n_steps{n_steps} K{K}", n_steps=n_steps, max_refine=4))


@pytest.mark.parametrize("K", [6, 1536, 4608])
def test_row_error_is_rounded_once(K):
    """As for the other row lengths: 1.5 * 2^-53 and the yardstick's own 1e-17."""
    w = rows_of_every_kind(257, K)
    w = w[[1, 5, 6, 8, 9, 10]].repeat(50, axis=0)[:257]
    _, _, _, err = dvdq.bgr_quantize(torch.from_numpy(w).to(DEV), n_steps=20, max_refine=1, eps=0.0, want_error=True,
                                     search=dvdq.BGR_LISTING)
    err = err.cpu().numpy()
    rel = []
    for i in range(0, 257, 50):
        x = _exact_listing_error(w[i], 20, 1)
        rel.append(abs(float((np.longdouble(err[i]) - x) / x)))
        assert np.array_equal(err[i:i + 50], np.full(len(err[i:i + 50]), err[i]))
    print(f"K{K}:", " ".join(f"{r:.1e}" for r in rel))
    assert max(rel) <= 2e-16, rel
