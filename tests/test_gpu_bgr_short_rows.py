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


@pytest.mark.parametrize("N,K,n_steps,max_refine,threads", [
    (513, 2, 9, 3, 256), (600, 34, 9, 3, 256), (520, 510, 9, 3, 256), (513, 5376, 9, 3, 256), (512, 34, 9, 3, 512), (512, 4608, 9, 3, 512),
    (257, 2, 80, 3, 256), (300, 34, 80, 3, 256), (257, 2048, 80, 1, 256), (257, 2048, 79, 1, 512), (257, 2050, 99, 3, 512), (260, 4608, 100, 3, 256),
    (260, 4608, 100, 2, 512), (260, 4610, 100, 3, 512), (256, 2048, 80, 1, 1024), (513, 5378, 99, 1, 512), (513, 5378, 100, 1, 256),
    (513, 6144, 100, 0, 256), (513, 6146, 100, 0, 512)])
@pytest.mark.parametrize("search", [dvdq.BGR_LISTING, dvdq.BGR_BEST_OF_ALL])
def test_row_lengths_and_counts_around_the_rule(N, K, n_steps, max_refine, threads, search):
    assert dvdq.bench_bgr_choice(N, K, n_steps, max_refine) == threads
    print(compare(rows_of_every_kind(N, K), f"N{N} K{K} search{search}", n_steps=n_steps, max_refine=max_refine, search=search))


@pytest.mark.parametrize("n_steps,K", [(127, 96), (131, 96), (300, 258)])   # 64 starts at a time, half of n_steps altogether
def test_more_starts_than_a_workgroup_takes_at_once(n_steps, K):
    assert dvdq.bench_bgr_choice(300, K, n_steps, 4) == 256
    print(compare(rows_of_every_kind(300, K), f"n_steps{n_steps} K{K}", n_steps=n_steps, max_refine=4))


@pytest.mark.parametrize("K", [6, 1536, 4608])
def test_row_error_is_rounded_once(K):
    """As for the other row lengths: 1.5 * 2^-53 and the yardstick's own 1e-17."""
    assert dvdq.bench_bgr_choice(513, K, 20, 1) == 256
    w = rows_of_every_kind(513, K)
    w = w[[1, 5, 6, 8, 9, 10]].repeat(100, axis=0)[:513]
    _, _, _, err = dvdq.bgr_quantize(torch.from_numpy(w).to(DEV), n_steps=20, max_refine=1, eps=0.0, want_error=True,
                                     search=dvdq.BGR_LISTING)
    err = err.cpu().numpy()
    rel = []
    for i in range(0, 513, 100):
        x = _exact_listing_error(w[i], 20, 1)
        rel.append(abs(float((np.longdouble(err[i]) - x) / x)))
        assert np.array_equal(err[i:i + 100], np.full(len(err[i:i + 100]), err[i]))
    print(f"K{K}:", " ".join(f"{r:.1e}" for r in rel))
    assert max(rel) <= 2e-16, rel
