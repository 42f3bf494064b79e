"""Kernels chosen by a rule on sizes, at the sizes where the rule or the kernel can go wrong: edges of tiles, remainders,
the smallest and the largest of each range (one parametrised test per kernel, against the oracle)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import dapq_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import dapq_harness
    return dapq_harness


def announce(text):
    print(f"[case] {text}", flush=True)


def problem_bits(seed, layers, lens, Hq, Hkv, N):
    rng = np.random.default_rng(seed)
    tokens = int(sum(lens))
    draw = lambda *s: W.to_bf16_bits(rng.standard_normal(s, dtype=np.float32))  # noqa: E731
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return draw(layers, len(lens), Hq, N, 128), draw(layers, tokens, Hkv, 128), draw(layers, tokens, Hkv, 128), cu


def oracle_lse2(q, k, Hkv, cu):
    """log2 of every row's softmax normaliser, float64: [layers, batch, Hq, N]."""
    layers, batch, Hq, N, d = q.shape
    out = np.zeros((layers, batch, Hq, N))
    for l in range(layers):
        for b in range(batch):
            for h in range(Hq):
                x = O.bf16_bits_to_f64(q[l, b, h]) @ O.bf16_bits_to_f64(k[l, cu[b]:cu[b + 1], h // (Hq // Hkv)]).T / np.sqrt(d)
                m = x.max(axis=1)
                out[l, b, h] = (m + np.log(np.exp(x - m[:, None]).sum(axis=1))) / np.log(2)
    return out


# chunks of 128 keys per sequence (the smallest calls): runs of 8 chunks, 16 classes of runs, one wave per run up to 16
@pytest.mark.parametrize("lens", [[1024], [1025], [8 * 128 * 2], [8 * 128 * 16], [8 * 128 * 16 + 1], [8 * 128 * 33 + 77],
                                  [20000, 1, 1100]], ids=str)
def test_normalisers_merged_over_many_chunks(H, lens):
    """The fp32 sums of a row's chunks, merged by several waves: |error| <= 2e-4 in the log2 domain (the bar of the
    other tests of the normaliser: 1.4e-4 relative on a sum of up to 2^17 positive terms), for a row count that is not
    a multiple of the 64 rows of a workgroup, and the same bits from two calls."""
    announce(f"normalisers over {lens}")
    q, k, v, cu = problem_bits(3, 1, lens, 4, 1, 17)
    prob = H.Problem(q, k, v, 1, cu if len(lens) > 1 else None, "thd")
    lse = prob.stats()
    assert torch.equal(lse, prob.stats())
    assert np.abs(lse.cpu().numpy() - oracle_lse2(q, k, 1, cu)).max() < 2e-4
