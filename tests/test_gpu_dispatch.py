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
        for b in (b for b in range(batch) if cu[b] < cu[b + 1]):
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


# rows around the tiles of 32 and the eight waves' first and second tiles; groups that fill one head tile of 4, several
@pytest.mark.parametrize("g", [1, 3, 4, 5, 8, 12])
@pytest.mark.parametrize("rows", [1, 15, 17, 32, 33, 256, 257, 300, 513, 530, 800])
def test_decode_tiles_and_head_groups(H, rows, g):
    """|error| <= 1e-5 max|v| + 1e-4 |o|, the bar of the other decode tests.  Heads of one call hold different numbers
    of rows (an empty one among them); the queries are not 16-byte aligned; in the last head a key of the second round of
    tiles lies hundreds of binades above everything before it, so the running reference has to move."""
    announce(f"decode rows={rows} g={g}")
    rng = np.random.default_rng(rows * 16 + g)
    budget, hkv, batch = rows + 3, 2, 2
    counts = np.array([[rows, max(1, rows // 2)], [0, rows]], dtype=np.int32)
    f = lambda *s: rng.standard_normal(s, dtype=np.float32)  # noqa: E731
    q, k, v = f(batch, hkv * g, 128), f(batch, hkv, budget, 128), f(batch, hkv, budget, 128)
    k[1, 1, min(rows - 1, 270)] = 60.0 * q[1, g]
    k[1, 1, rows // 3] = -60.0 * q[1, g]
    qb, kb, vb = (W.to_bf16_bits(x) for x in (q, k, v))
    store = torch.zeros(q.size + 1, dtype=torch.bfloat16, device="cuda")
    store[1:] = H.dev_bf16(qb).reshape(-1)
    out = torch.full((1, batch, hkv * g, 128), float("nan"), dtype=torch.float32, device="cuda")
    shape = H.D.make_shape(n_layers=1, batch=batch, n_q_heads=hkv * g, n_kv_heads=hkv, n_pseudo=1, total_tokens=batch,
                           scale=128 ** -0.5)
    H.D.dapq_decode_attention(shape, store[1:], H.dev_bf16(kb), H.dev_bf16(vb), torch.from_numpy(counts).cuda(), budget, out)
    got = out.cpu().numpy()[0].astype(np.float64)
    q64, k64, v64 = (O.bf16_bits_to_f64(x) for x in (qb, kb, vb))
    for b in range(batch):
        for h in range(hkv * g):
            n = counts[b, h // g]
            if n == 0:
                assert (got[b, h] == 0).all()
                continue
            x = k64[b, h // g, :n] @ q64[b, h] / np.sqrt(128)
            w = np.exp(x - x.max())
            want = (w / w.sum()) @ v64[b, h // g, :n]
            bound = 1e-5 * np.abs(v64[b, h // g, :n]).max() + 1e-4 * np.abs(want)
            assert (np.abs(got[b, h] - want) <= bound).all(), (b, h)


def decode_call(H, q, k, v, counts, layers=1):
    """One decode step; q [batch, Hq, 128], k and v [batch, Hkv, budget, 128] (bf16 bits), counts [batch, Hkv]: [batch, Hq, 128]."""
    batch, hq, hkv, budget = q.shape[0], q.shape[1], k.shape[1], k.shape[2]
    out = torch.full((batch, hq, 128), float("nan"), dtype=torch.float32, device="cuda")
    shape = H.D.make_shape(n_layers=layers, batch=batch // layers, n_q_heads=hq, n_kv_heads=hkv, n_pseudo=1,
                           total_tokens=batch // layers, scale=128 ** -0.5)
    H.D.dapq_decode_attention(shape, H.dev_bf16(q), H.dev_bf16(k), H.dev_bf16(v),
                              torch.from_numpy(np.ascontiguousarray(counts, dtype=np.int32)).cuda(), budget, out)
    return out.cpu().numpy().astype(np.float64)


def decode_want(q, k, v, counts):
    """The same in float64."""
    q, k, v = (O.bf16_bits_to_f64(x) for x in (q, k, v))
    g = q.shape[1] // k.shape[1]
    want = np.zeros(q.shape)
    for b, h in np.ndindex(q.shape[:2]):
        n = counts[b, h // g]
        if n:
            x = k[b, h // g, :n] @ q[b, h] / np.sqrt(128)
            w = np.exp(x - x.max())
            want[b, h] = (w / w.sum()) @ v[b, h // g, :n]
    return want


# the numbers of heads at which the slices change (up to 32 heads, up to 128, more), tiles of 4 and of 8 query heads
@pytest.mark.parametrize("layers,batch,hkv", [(1, 4, 8), (3, 11, 1), (2, 8, 8), (1, 43, 3), (1, 50, 8)])
@pytest.mark.parametrize("g", [1, 4, 8, 12])
@pytest.mark.parametrize("rows", [1, 33, 257, 983])
def test_decode_slices(H, rows, g, layers, batch, hkv):
    """|error| as in the other decode tests, for heads that are full, half full, nearly empty and empty; what lies past the count is
    no number or infinite and is not looked at."""
    announce(f"decode: {layers * batch * hkv} heads, rows={rows} g={g}")
    rng = np.random.default_rng(rows + g)
    n = layers * batch
    f = lambda *s: rng.standard_normal(s, dtype=np.float32)  # noqa: E731
    q, k, v = (W.to_bf16_bits(x) for x in (2 * f(n, hkv * g, 128), f(n, hkv, rows, 128), f(n, hkv, rows, 128)))
    counts = np.array([rows, (rows + 1) // 2, 1, 0, rows - 1])[np.arange(n * hkv) % 5].reshape(n, hkv)
    want = decode_want(q, k, v, counts)
    past = np.arange(rows)[None, None, :, None] >= counts[:, :, None, None]
    got = decode_call(H, q, np.where(past, np.uint16(0x7FC1), k), np.where(past, np.uint16(0xFF80), v), counts, layers)
    assert (np.abs(got - want) <= 1e-5 * np.abs(O.bf16_bits_to_f64(v)).max() + 1e-4 * np.abs(want)).all()
    assert (got[want == 0] == 0).all()


# the lines between four, two and one slice: by the number of heads (64, 128; long caches: 24, 48 and, from 5 query heads per KV head
# on, 64) and by heads x rows (from 5 on, by heads x heads x rows)
@pytest.mark.parametrize("heads,rows,g", [(64, 1408, 4), (64, 1409, 4), (65, 40, 4), (24, 4096, 2), (25, 4096, 2), (128, 896, 4),
                                          (128, 897, 4), (129, 100, 1), (48, 4096, 1), (49, 4096, 1), (128, 1088, 8), (128, 1089, 5),
                                          (64, 2500, 8), (65, 2500, 8)])
def test_decode_lines_between_slices(H, heads, rows, g):
    """|error| as in the other decode tests, for full and half full heads."""
    announce(f"decode: {heads} heads, rows={rows} g={g}")
    rng = np.random.default_rng(heads + rows)
    f = lambda *s: rng.standard_normal(s, dtype=np.float32)  # noqa: E731
    q, k, v = (W.to_bf16_bits(x) for x in (2 * f(heads, g, 128), f(heads, 1, rows, 128), f(heads, 1, rows, 128)))
    counts = np.array([rows, rows // 2])[np.arange(heads) % 2].reshape(heads, 1)
    want = decode_want(q, k, v, counts)
    got = decode_call(H, q, k, v, counts, 1)
    assert (np.abs(got - want) <= 1e-5 * np.abs(O.bf16_bits_to_f64(v)).max() + 1e-4 * np.abs(want)).all()


@pytest.mark.parametrize("heads,rows,g", [(128, 704, 8), (128, 705, 5), (100, 1153, 8), (100, 1154, 8)])
def test_decode_lines_of_many_query_heads(H, heads, rows, g):
    test_decode_lines_between_slices(H, heads, rows, g)


# the three slice counts (up to 32 heads, up to 128, more), both head tiles
@pytest.mark.parametrize("batch", [2, 9, 33])
@pytest.mark.parametrize("g", [4, 5])
def test_decode_rows_that_weigh_nothing(H, g, batch):
    """Rows whose logits are -inf (a key of that channel at the largest value, against a query as large) weigh 0 wherever they
    lie: in all of a wave's first tile, in its last, everywhere but in one row.  |error| as in the other decode tests."""
    announce(f"decode: -inf logits, g={g} batch={batch}")
    rng = np.random.default_rng(g)
    rows, hkv = 600, 4
    f = lambda *s: rng.standard_normal(s, dtype=np.float32)  # noqa: E731
    q, k, v = f(batch, hkv * g, 128), f(batch, hkv, rows, 128), f(batch, hkv, rows, 128)
    q[..., 5], k[..., 5] = 3e38, 0.0
    for kv, gone in enumerate((slice(0, 400), slice(256, 288), slice(500, 600), slice(1, 600))):
        k[:, kv, gone, 5] = -3e38
    q, k, v = (W.to_bf16_bits(x) for x in (q, k, v))
    counts = np.full((batch, hkv), rows)
    got, want = decode_call(H, q, k, v, counts), decode_want(q, k, v, counts)     # (-1e77 in float64: weight 0 as well)
    assert (np.abs(got - want) <= 1e-5 * np.abs(O.bf16_bits_to_f64(v)).max() + 1e-4 * np.abs(want)).all()


@pytest.mark.parametrize("batch", [2, 9, 33])
@pytest.mark.parametrize("g", [4, 5])
def test_decode_infinite_values(H, g, batch):
    """An infinite value makes its channel infinite in every query head that gives its row a weight, whichever bits of the weight's
    significand are set; the other channels are not touched (|error| as in the other decode tests)."""
    announce(f"decode: infinite values, g={g} batch={batch}")
    rng = np.random.default_rng(g)
    rows, hkv = 70, 4
    f = lambda *s: rng.standard_normal(s, dtype=np.float32)  # noqa: E731
    q, k, v = f(batch, hkv * g, 128), f(batch, hkv, rows, 128), f(batch, hkv, rows, 128)
    k[:, 1] = 0.0                         # all weights 1: their second and third part are 0
    q, k, v = (W.to_bf16_bits(x) for x in (q, k, v))
    counts = np.full((batch, hkv), rows)
    want = decode_want(q, k, v, counts)
    bound = 1e-5 * np.abs(O.bf16_bits_to_f64(v)).max() + 1e-4 * np.abs(want)
    for channel in (3, 64, 127):
        v[:, :, channel % rows, channel] = 0x7F80
        want[..., channel] = np.inf
    v[:, :, 40, 90] = 0xFF80
    want[..., 90] = -np.inf
    got = decode_call(H, q, k, v, counts)
    infinite = np.isinf(want)
    assert np.array_equal(got[infinite], want[infinite])
    assert (np.abs(got[~infinite] - want[~infinite]) <= bound[~infinite]).all()


@pytest.mark.parametrize("batch", [2, 9, 33])
@pytest.mark.parametrize("rise", [5, 14, 40, 59, 61, 300])
@pytest.mark.parametrize("size", [1e33, 1.0, 1e-30])
def test_decode_logits_that_rise_late(H, size, rise, batch):
    """Rows late in the cache whose logits lie `rise` binades above the others', and values of up to `size`: the sums must not leave the
    range of fp32 on the way.  |error| as in the other decode tests, and 2^-22 max|v| per binade of the logits: an fp32
    logit of `rise` binades is known to about two units of its last place, 2^-23 rise, and with it the ratio of two weights."""
    announce(f"decode: a logit {rise} binades higher late, values of {size}, batch={batch}")
    rng = np.random.default_rng(rise)
    rows, hkv, g = 700, 4, 4
    f = lambda *s: rng.standard_normal(s, dtype=np.float32)  # noqa: E731
    q, k = f(batch, hkv * g, 128), 0.1 * f(batch, hkv, rows, 128)
    v = np.float32(size) * (2 * rng.random((batch, hkv, rows, 128), dtype=np.float32) - 1)
    q[..., 7], k[..., 7] = 8.0, 0.0
    k[:, :, (600, 300, 37, 699), 7] = rise * np.log(2) * np.sqrt(128) / 8
    q, k, v = (W.to_bf16_bits(x) for x in (q, k, v))
    counts = np.full((batch, hkv), rows)
    got, want = decode_call(H, q, k, v, counts), decode_want(q, k, v, counts)
    assert (np.abs(got - want) <= (1e-5 + rise * 2.0 ** -22) * np.abs(O.bf16_bits_to_f64(v)).max() + 1e-4 * np.abs(want)).all()


def test_decode_step_of_very_many_heads(H):
    """2^24 + 2^19 heads of one row each: the output is the row's value, within 2^-21 of itself (weight times value over weight: three
    sums and a quotient in fp32, 2^-24 each).  One tensor of 4.4 GB is queries, keys and values at once; the output takes 8.9 GB."""
    announce("decode: 17.3 million heads")
    layers, batch, hkv = 33, 1024, 512
    x = torch.randn((layers * batch * hkv, 128), dtype=torch.bfloat16, device="cuda")
    count = torch.ones(layers * batch * hkv, dtype=torch.int32, device="cuda")
    count[-1] = 0
    out = torch.empty(x.shape, dtype=torch.float32, device="cuda")
    shape = H.D.make_shape(n_layers=layers, batch=batch, n_q_heads=hkv, n_kv_heads=hkv, n_pseudo=1, total_tokens=batch,
                           scale=128 ** -0.5)
    H.D.dapq_decode_attention(shape, x, x, x, count, 1, out)
    assert (out[-1] == 0).all()
    for a, b in zip(out[:-1].split(1 << 20), x[:-1].float().split(1 << 20)):
        assert ((a - b).abs() <= 2.0 ** -21 * b.abs()).all()


# few workgroups: keys around the sub-blocks and tiles of 128, rows around the row blocks of 32, the eight waves (256) and the
# 512 rows whose partials pass 2 merges itself; more than 64 sequences (their chunk prefix lies in device memory), empty ones
@pytest.mark.parametrize("rows", [1, 31, 33, 74, 257, 512, 520])
@pytest.mark.parametrize("lens", [[513], [1025], [5000], [640, 640], [1, 33, 127, 128, 129, 0, 700],
                                  [(7 * i) % 150 for i in range(67)]], ids=lambda lens: f"{len(lens)}x{max(lens)}")
def test_scores_of_small_calls(H, lens, rows):
    """Scores within 1e-3 of the oracle's and normalisers within 2e-4 in the log2 domain (the bars of the other score
    tests), the bits of dapq_score from the two separate entry points, and a key hundreds of binades above the others."""
    announce(f"small score call: {lens} rows={rows}")
    g = 2 if rows % 2 == 0 else 1
    q, k, v, cu = problem_bits(rows, 1, lens, 2 * g, 2, rows // g)
    last = int(cu[np.argmax(lens) + 1]) - 1
    k[0, last, 1] = W.to_bf16_bits(30.0 * O.bf16_bits_to_f64(q[0, int(np.argmax(lens)), g, 0]))
    for layout, ragged in (("thd", len(set(lens)) > 1), ("hnd", True)):
        prob = H.Problem(q, k, v, 2, cu if ragged else None, layout)
        S = prob.score()
        assert torch.equal(S, prob.score_split())
        H.assert_scores_close(S.cpu().numpy(), O.score(q, k, 2, cu), f"{lens} rows={rows} {layout}")
    live = [b for b, n in enumerate(lens) if n]
    err = np.abs(prob.stats().cpu().numpy()[:, live] - oracle_lse2(q, k, 2, cu)[:, live])
    assert err.max() < 2e-4


# tiles of 128 and 256 keys, the last ones short, and of 128 keys whose queries do not go through LDS (40000); one to five row
# blocks, shared out to eight waves in one to eight parts, and nine, in two trips
@pytest.mark.parametrize("rows", [32, 64, 96, 128, 160, 257])
@pytest.mark.parametrize("lens", [[9000], [20001], [40000], [3000, 0, 77, 2100]], ids=lambda lens: f"{len(lens)}x{max(lens)}")
def test_tiles_of_small_calls(H, lens, rows):
    """The oracle's scores within 1e-3 and its normalisers within 2e-4 in the log2 domain, and the bits of dapq_score from the two
    separate entry points, with a key hundreds of binades above the others."""
    announce(f"tiles: {lens} rows={rows}")
    q, k, v, cu = problem_bits(rows, 1, lens, 2, 2, rows)
    b = int(np.argmax(lens))
    k[0, int(cu[b]) + lens[b] // 2, 1] = W.to_bf16_bits(30.0 * O.bf16_bits_to_f64(q[0, b, 1, 0]))
    prob = H.Problem(q, k, v, 2, cu if len(lens) > 1 else None, "thd")
    S = prob.score()
    assert torch.equal(S, prob.score_split())
    H.assert_scores_close(S.cpu().numpy(), O.score(q, k, 2, cu), f"{lens} rows={rows}")
    live = [i for i, n in enumerate(lens) if n]
    assert np.abs(prob.stats().cpu().numpy()[:, live] - oracle_lse2(q, k, 2, cu)[:, live]).max() < 2e-4


@pytest.mark.parametrize("batch", [2, 64, 65])
def test_small_ragged_calls_write_no_chunk_prefix(H, batch):
    """Up to 64 sequences every wave of the tile form finds its chunk by itself: neither pass writes the prefix of the chunk
    counts, the first batch + 1 words of the workspace; more sequences need it in both passes."""
    announce(f"chunk prefix of {batch} sequences")
    lens = [(7 * i) % 150 + 1 for i in range(batch)]
    q, k, v, cu = problem_bits(batch, 1, lens, 2, 2, 16)
    prob = H.Problem(q, k, v, 2, cu, "thd")
    lse = prob.stats()
    for call in (prob.score, prob.stats, lambda: H.D.dapq_score_accumulate(prob.shape, prob.q, prob.k, lse, torch.empty(
            (1, 2, prob.tokens), dtype=torch.float32, device="cuda"), prob.ws)):
        prob.ws.fill_(0xA5)
        call()
        kept = bool((prob.ws[:4 * (batch + 1)] == 0xA5).all())
        assert kept == (batch <= 64)


def test_scores_of_very_many_sequences(H):
    """2^26 + 100 sequences of one key each: every score is the number of query rows.  Keys of 17 GB, a workspace of 35 GB."""
    announce("scores of 67 million sequences")
    batch = (1 << 26) + 100
    cu = torch.arange(batch + 1, dtype=torch.int32, device="cuda")
    k = torch.zeros((batch, 128), dtype=torch.bfloat16, device="cuda")
    q = torch.ones((2, 128), dtype=torch.bfloat16, device="cuda")
    shape = H.D.make_shape(n_layers=1, batch=batch, n_q_heads=2, n_kv_heads=1, n_pseudo=1, total_tokens=batch, cu_seqlens=cu,
                           k_strides=(0, 0, 0, 128), q_strides=(0, 0, 128, 128), scale=128 ** -0.5)
    ws = torch.empty(H.D.workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    ws.fill_(0xFF)
    S = torch.empty((1, 1, batch), dtype=torch.float32, device="cuda")
    H.D.dapq_score(shape, q, k, S, ws)
    assert (S == 2.0).all()


@pytest.mark.parametrize("rows", [128, 200])
def test_small_ragged_scores_in_a_workspace_sized_for_longer_ones(H, rows):
    """A workspace that holds the wave form's sums only: the oracle's scores within 1e-3 (the bar of the other score tests), the same
    bits from the two separate entry points, and nothing written past the end of it."""
    announce(f"small workspace: rows={rows}")
    lens = [3000, 1, 4000, 0, 2500, 700, 3300, 2047]
    q, k, v, cu = problem_bits(rows, 2, lens, 2, 2, rows)
    prob = H.Problem(q, k, v, 2, cu, "thd")
    prob.shape.n_layers, prob.shape.k_stride_layer, prob.shape.q_stride_layer = 16, 0, 0        # 16 times the first layer
    want = H.D.workspace_bytes(prob.shape)
    prob.shape.total_tokens = 40000
    ws_bytes = H.D.workspace_bytes(prob.shape)
    prob.shape.total_tokens = prob.tokens
    assert ws_bytes < want
    whole = torch.full((want,), 0xA5, dtype=torch.uint8, device="cuda")
    S, T = (torch.full((16, 2, prob.tokens), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2))
    H.D.dapq_score(prob.shape, prob.q, prob.k, S, whole[:ws_bytes])
    lse = torch.empty((16, len(lens), 2, rows), dtype=torch.float32, device="cuda")
    H.D.dapq_score_stats(prob.shape, prob.q, prob.k, lse, whole[:ws_bytes])
    H.D.dapq_score_accumulate(prob.shape, prob.q, prob.k, lse, T, whole[:ws_bytes])
    assert torch.equal(S, T) and torch.equal(S, S[:1].expand_as(S))
    assert (whole[ws_bytes:] == 0xA5).all()
    H.assert_scores_close(S[:1].cpu().numpy(), O.score(q[:1], k[:1], 2, cu), f"rows={rows}")


# 2^23 workgroups of 512 threads are the 2^32 threads that an axis of a launch does not hold; as many single waves are 2^26
@pytest.mark.parametrize("batch,rows", [((1 << 23) + 37, 33), ((1 << 26) + 101, 2)], ids=["one workgroup a sequence", "one wave a sequence"])
def test_scores_of_very_many_dense_sequences(H, batch, rows):
    """A key to a sequence, with a channel of its own value, and queries that overlap from sequence to sequence: every score is the number
    of rows, and every normaliser the logit, of 8 bits times 8 bits.  The second: keys of 17 GB, a workspace of 35 GB."""
    announce(f"scores of {batch} dense sequences, rows={rows}")
    seq = torch.arange(batch, device="cuda")
    value = ((seq * 37) % 251 + 1).to(torch.bfloat16)
    k = torch.zeros((batch, 128), dtype=torch.bfloat16, device="cuda")
    k[:, 0] = value
    q = (torch.arange(batch * 8 + rows * 128, device="cuda") % 253 - 126).to(torch.bfloat16)
    shape = H.D.make_shape(n_layers=1, batch=batch, n_q_heads=1, n_kv_heads=1, n_pseudo=rows, total_tokens=batch,
                           k_strides=(0, 0, 0, 128), q_strides=(0, 8, 0, 128), scale=1.0 / 128)
    ws = torch.empty(H.D.workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    ws.fill_(0xFF)
    lse = torch.full((batch, rows), float("nan"), dtype=torch.float32, device="cuda")
    S, T = (torch.full((batch,), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2))
    H.D.dapq_score(shape, q, k, S, ws)
    H.D.dapq_score_stats(shape, q, k, lse, ws)
    H.D.dapq_score_accumulate(shape, q, k, lse, T, ws)
    assert torch.equal(S, T) and (S - rows).abs().max() < 1e-3 * rows
    worst = 0.0
    for row in range(rows):
        want = q[row * 128: row * 128 + batch * 8: 8].float() * value.float() * (1.4426950408889634 / 128)
        worst = max(worst, float((lse[:, row] - want).abs().max()))
    assert worst < 2e-4


def score_values(kind, rng, n):
    x = rng.random(n, dtype=np.float32)
    if kind == "octaves":
        return np.exp2(40 * x - 30).astype(np.float32)
    if kind == "one value":
        return np.full(n, 0.37, dtype=np.float32)
    if kind == "three values":
        return np.floor(3 * x).astype(np.float32)
    if kind == "half zero":
        return np.where(x < 0.5, 0, x).astype(np.float32)
    if kind.startswith("crowd"):  # most keys share a value that is not the least: all but one or two, half of them, a third
        y = np.where(x < {"crowd": 1.1, "crowd of half": 0.5, "crowd of a third": 0.33}[kind], np.float32(1), x)
        y[n // 2], y[n // 3] = 0.01, 50.0
        return y.astype(np.float32)
    if kind == "neighbours":      # consecutive floats below a single far larger one
        y = np.nextafter(np.float32(1), np.float32(2)) + np.float32(2 ** -23) * np.floor(300 * x)
        y[n // 2] = 1e30
        return y.astype(np.float32)
    y = np.float32(1e3) * (x - np.float32(0.5))     # both signs, both zeros, both infinities
    y[::7], y[1::7] = 0.0, -0.0
    y[n // 3], y[n // 2] = np.inf, -np.inf
    return y


# the selection closes in on the threshold by bins of the span of the keys: spans of 0 to 2^32, bins that hold one value or
# most of them, more and fewer than the 64 candidates that one wave ranks, at the lengths where the variants change
@pytest.mark.parametrize("kind", ["octaves", "one value", "three values", "half zero", "neighbours", "signs", "crowd",
                                  "crowd of half", "crowd of a third"])
@pytest.mark.parametrize("n", [1, 33, 64, 65, 1000, 8192, 8193, 16385, 32768, 40000, 140001])
def test_selection_over_distributions(H, n, kind):
    """The retained positions are the oracle's, bit for bit (selection compares the given scores; equal ones lowest
    position first; -0 and +0 are told apart by neither, so the zeros of one input all have the same sign)."""
    announce(f"selection of {n}: {kind}")
    rng = np.random.default_rng(n)
    S = np.stack([score_values(kind, rng, n) for _ in range(2)])[None]
    if kind == "signs":
        S[S == 0] = 0.0
    q = np.zeros((1, 1, 2, 1, 128), dtype=np.uint16)
    k = np.zeros((1, n, 2, 128), dtype=np.uint16)
    prob = H.Problem(q, k, k, 2, None, "hnd")
    for budget in sorted({b for b in (1, 63, 64, 65, n // 30, n // 2, n - 1) if 1 <= b < max(n, 2) and b <= 15000}):
        for pooled in (False, True):
            P = np.stack([O.pool(S[0, kv], 7) for kv in range(2)]) if pooled and kind != "signs" else S[0]
            dev = torch.from_numpy(S).cuda()
            idx, count = (prob.pool_topk(dev, 7, budget, want_pooled=n > 65536, pieces=True)[:2] if pooled and kind != "signs"
                          else prob.topk(dev, budget))
            for kv in range(2):
                got = idx.cpu().numpy()[0, 0, kv][:int(count[0, 0, kv])]
                assert np.array_equal(got, O.topk(P[kv].astype(np.float64), budget)), (budget, pooled, kv)


# waves with and without negative scores in one head (their keys are formed differently), waves that are full, partly filled and
# empty; as many equal keys at the threshold as one list of candidates holds, one fewer and one more, spread and side by side
@pytest.mark.parametrize("equal", [63, 64, 65])
@pytest.mark.parametrize("n", [70, 2047, 2048, 2050, 8191, 16384, 32767, 40000])
def test_selection_of_mixed_waves(H, n, equal):
    """The retained positions are the oracle's, bit for bit, with budgets that take none, some and all of the equal keys."""
    announce(f"selection of {n}, {equal} equal")
    rng = np.random.default_rng(n + equal)
    S = rng.random((1, 2, n), dtype=np.float32)
    S[0, 0, n // 3: n // 3 + n // 7] -= np.float32(2.0)
    above = n // 40
    order = np.argsort(-S[0], axis=1, kind="stable")
    S[0, 0, order[0, above: above + equal]] = np.float32(0.97)                     # spread
    S[0, 0, order[0, :above]] = np.float32(1.5) + S[0, 0, order[0, :above]]
    S[0, 1, n // 2: n // 2 + min(equal, n - n // 2)] = np.float32(7.0)             # side by side
    q = np.zeros((1, 1, 2, 1, 128), dtype=np.uint16)
    k = np.zeros((1, n, 2, 128), dtype=np.uint16)
    prob = H.Problem(q, k, k, 2, None, "hnd")
    dev = torch.from_numpy(S).cuda()
    for budget in sorted({b for b in (1, above, above + 1, above + equal - 1, above + equal, above + equal + 1, 30) if 1 <= b < n}):
        idx, count = prob.topk(dev, budget)
        for kv in range(2):
            got = idx.cpu().numpy()[0, 0, kv][:int(count[0, 0, kv])]
            assert np.array_equal(got, O.topk(S[0, kv].astype(np.float64), budget)), (budget, kv)


# ragged batches too large for the tile form (more than 65536 units): the kernels of two, four, seven and eight row blocks, two row groups
# of eight, up to and beyond the 64 sequences that a wave looks up by itself
@pytest.mark.parametrize("batch", [40, 64, 65, 100])
@pytest.mark.parametrize("rows", [33, 128, 200, 250, 512])
def test_ragged_batches_in_the_wave_form(H, rows, batch):
    """Every layer is the same problem (layer strides of 0): all layers have the same bits, and the first has the oracle's
    scores within 1e-3 (the bar of the other score tests)."""
    announce(f"ragged wave form: rows={rows} batch={batch}")
    lens = [(37 * b) % 211 for b in range(batch - 1)] + [1500]
    q, k, v, cu = problem_bits(batch, 1, lens, 2, 2, rows)
    prob = H.Problem(q, k, v, 2, cu, "thd")
    tokens = int(cu[-1])
    layers = 66000 // (2 * (tokens // 128 + batch) * ((rows + 31) // 32)) + 1
    shape = H.D.make_shape(n_layers=layers, batch=batch, n_q_heads=2, n_kv_heads=2, n_pseudo=rows, total_tokens=tokens,
                           cu_seqlens=prob.cu, k_strides=(0, 0, 128, 256), q_strides=(0, 2 * rows * 128, rows * 128, 128),
                           scale=128 ** -0.5)
    ws = torch.empty(H.D.workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    S = torch.full((layers, 2, tokens), float("nan"), dtype=torch.float32, device="cuda")
    H.D.dapq_score(shape, prob.q, prob.k, S, ws)
    assert torch.equal(S, S[:1].expand_as(S))
    H.assert_scores_close(S[:1].cpu().numpy(), O.score(q, k, 2, cu), f"rows={rows} batch={batch}")


# dense batches whose chunks are no powers of two: eight per sequence, shorter than the power of two; four and two, longer (sums in
# two steps; up to 256 rows both passes in one kernel); three and one; several sequences; the last chunk with a partial sub-block or short;
# a wave of two to eight row blocks, two row groups of five
@pytest.mark.parametrize("rows", [33, 96, 128, 160, 192, 224, 250, 300])
@pytest.mark.parametrize("layers,batch,length", [(64, 1, 3001), (128, 1, 5000), (170, 1, 2900), (70, 7, 1111), (25, 3, 2017)])
def test_equal_chunks_of_dense_batches(H, layers, batch, length, rows):
    """Every layer is the same problem (layer strides of 0), with a key hundreds of binades above the others: the oracle's scores within
    1e-3 and normalisers within 2e-4 in the log2 domain, the same bits in every layer and from the two separate entry points."""
    announce(f"equal chunks: {layers} layers, {batch} x {length} keys, rows={rows}")
    lens = [length] * batch
    q, k, v, cu = problem_bits(rows, 1, lens, 2, 2, rows)
    k[0, 2 * length // 3, 1] = W.to_bf16_bits(30.0 * O.bf16_bits_to_f64(q[0, 0, 1, 0]))
    prob = H.Problem(q, k, v, 2, None, "thd")
    tokens = batch * length
    shape = H.D.make_shape(n_layers=layers, batch=batch, n_q_heads=2, n_kv_heads=2, n_pseudo=rows, total_tokens=tokens,
                           k_strides=(0, 0, 128, 256), q_strides=(0, 2 * rows * 128, rows * 128, 128), scale=128 ** -0.5)
    ws = torch.full((H.D.workspace_bytes(shape),), 0xA5, dtype=torch.uint8, device="cuda")
    S, T = (torch.full((layers, 2, tokens), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2))
    lse = torch.full((layers, batch, 2, rows), float("nan"), dtype=torch.float32, device="cuda")
    H.D.dapq_score(shape, prob.q, prob.k, S, ws)
    H.D.dapq_score_stats(shape, prob.q, prob.k, lse, ws)
    H.D.dapq_score_accumulate(shape, prob.q, prob.k, lse, T, ws)
    assert torch.equal(S, T) and torch.equal(S, S[:1].expand_as(S)) and torch.equal(lse, lse[:1].expand_as(lse))
    H.assert_scores_close(S[:1].cpu().numpy(), O.score(q, k, 2, cu), f"{layers} {lens} rows={rows}")
    assert np.abs(lse[:1].cpu().numpy() - oracle_lse2(q, k, 2, cu)).max() < 2e-4


# one chunk of at most 128 keys, or of 129: on both sides of the kernel for short prompts, which has nearly all of these, and of the waves
@pytest.mark.parametrize("rows", [64, 65, 128, 129, 192, 193, 256])
@pytest.mark.parametrize("layers,batch,length", [(2, 3, 1), (3, 1, 33), (1, 2, 127), (2, 2, 128), (2, 2, 129), (1365, 3, 40), (1366, 3, 40)])
def test_chunks_of_few_keys(H, layers, batch, length, rows):
    """As above."""
    test_equal_chunks_of_dense_batches(H, layers, batch, length, rows)


# what it leaves to waves that start with fragments: six to eight row blocks, more than 512 heads, an odd number of chunks (a wave to a workgroup);
# both passes in one kernel up to 8192 of them, with more through the ring; three row groups, in separate launches
@pytest.mark.parametrize("layers,batch,length,rows", [
    (87, 3, 128, 192), (87, 3, 97, 161), (1366, 3, 128, 192), (87, 3, 128, 224), (87, 3, 65, 193), (1366, 3, 65, 224), (87, 3, 128, 256),
    (87, 3, 33, 256), (87, 3, 64, 225), (1366, 3, 64, 256), (172, 3, 128, 576), (172, 3, 64, 672), (172, 3, 33, 768), (172, 3, 1, 600)])
def test_few_keys_in_waves(H, layers, batch, length, rows):
    """As above."""
    test_equal_chunks_of_dense_batches(H, layers, batch, length, rows)


# short prompts, all of a head in one workgroup: edges of sub-blocks and row blocks (eight waves make eight, four, two parts or one of them), queries
# through LDS and (more than 320 keys) not; the lines between it and the waves: 256 heads, 512, two workgroups to a compute unit
@pytest.mark.parametrize("layers,batch,length,rows", [
    (1, 1, 1, 1), (1, 1, 32, 32), (1, 2, 33, 31), (3, 1, 256, 33), (1, 1, 512, 32), (2, 1, 511, 64), (1, 1, 300, 65), (1, 2, 384, 96),
    (1, 1, 385, 97), (1, 1, 448, 128), (1, 1, 449, 128), (2, 1, 319, 129), (1, 1, 320, 160), (1, 1, 321, 160), (1, 1, 384, 193),
    (1, 1, 352, 256), (1, 2, 384, 256), (1, 1, 385, 256), (128, 1, 129, 250), (129, 1, 128, 250), (129, 1, 129, 250), (64, 4, 96, 200),
    (64, 5, 40, 70), (257, 1, 64, 33), (257, 1, 32, 32), (86, 3, 224, 64), (86, 3, 225, 64)])
def test_short_prompts(H, layers, batch, length, rows):
    """As above."""
    test_equal_chunks_of_dense_batches(H, layers, batch, length, rows)


# whole sub-blocks of a short prompt whose logits overflow to -inf (bf16's lowest value in a key, as a mask would have it): a wave's only one,
# its first one, its last one; a prompt of a sub-block and a key
@pytest.mark.parametrize("length,rows,masked", [(96, 33, (32, 64)), (256, 32, (0, 32)), (300, 250, (0, 64)), (300, 65, (288, 300)), (33, 20, (0, 32))])
def test_short_prompts_with_masked_keys(H, length, rows, masked):
    """The oracle's scores within 1e-3 and normalisers within 2e-4 in the log2 domain: the masked keys add nothing to any row."""
    announce(f"masked keys {masked} of {length}, rows={rows}")
    q, k, v, cu = problem_bits(rows, 1, [length], 2, 2, rows)
    q[..., 0] = W.to_bf16_bits(np.full(q.shape[:-1], 2.0, dtype=np.float32))
    k[0, masked[0]:masked[1]] = 0
    k[0, masked[0]:masked[1], :, 0] = 0xFF7F
    prob = H.Problem(q, k, v, 2, None, "thd")
    S = prob.score()
    assert torch.isfinite(S).all() and not S[:, :, masked[0]:masked[1]].any()
    H.assert_scores_close(S.cpu().numpy(), O.score(q, k, 2, cu), f"{length} rows={rows}")
    assert np.abs(prob.stats().cpu().numpy() - oracle_lse2(q, k, 2, cu)).max() < 2e-4


# the same in the other forms: tiles of one sub-block, of several with a part to each, two at a time and several times two, with the queries straight
# from memory; the waves of a dense batch in separate launches and in one, with 64 keys too, and of a ragged batch; a whole tile, chunk or prompt
@pytest.mark.parametrize("rows,lens,layers,ragged,masked", [
    (250, [1024], 1, False, [(0, 32), (100, 170)]), (16, [5000], 1, False, [(0, 32), (128, 320), (4990, 5000)]),
    (128, [5000], 1, False, [(64, 96), (200, 500)]), (250, [16384], 1, False, [(0, 64), (256, 352), (1024, 1300)]),
    (250, [5000], 8, False, [(0, 64), (1000, 1500)]), (40, [513], 1, False, [(0, 40)]), (60, [1000, 70, 33], 2, True, [(0, 64), (1000, 1070)]),
    (250, [3001], 64, False, [(0, 32), (400, 1000), (2990, 3001)]), (128, [1500] * 3, 100, False, [(0, 40), (700, 1600), (3000, 4500)]),
    (256, [64], 300, False, [(0, 32)]), (33, [700, 0, 33, 1500], 1000, True, [(0, 32), (700, 1100)]),
    (250, [211] * 20 + [1500], 100, True, [(0, 33), (211, 422), (4220, 4900)])])
def test_masked_keys(H, rows, lens, layers, ragged, masked):
    """As above, in every layer and from the two separate entry points (layer strides of 0); a prompt of masked keys alone has scores of 0."""
    announce(f"masked keys {masked} of {layers} x {lens}, rows={rows}")
    q, k, v, cu = problem_bits(rows, 1, lens, 2, 2, rows)
    q[..., 0] = W.to_bf16_bits(np.full(q.shape[:-1], 2.0, dtype=np.float32))
    hidden = np.zeros(int(cu[-1]), dtype=bool)
    for first, end in masked:
        hidden[first:end] = True
    k[0, hidden] = 0
    k[0, hidden, :, 0] = 0xFF7F
    prob = H.Problem(q, k, v, 2, cu if ragged else None, "thd")
    tokens, batch = int(cu[-1]), len(lens)
    shape = H.D.make_shape(n_layers=layers, batch=batch, n_q_heads=2, n_kv_heads=2, n_pseudo=rows, total_tokens=tokens, cu_seqlens=prob.cu,
                           k_strides=(0, 0, 128, 256), q_strides=(0, 2 * rows * 128, rows * 128, 128), scale=128 ** -0.5)
    ws = torch.full((H.D.workspace_bytes(shape),), 0xA5, dtype=torch.uint8, device="cuda")
    S, T = (torch.full((layers, 2, tokens), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2))
    lse = torch.full((layers, batch, 2, rows), float("nan"), dtype=torch.float32, device="cuda")
    H.D.dapq_score(shape, prob.q, prob.k, S, ws)
    H.D.dapq_score_stats(shape, prob.q, prob.k, lse, ws)
    H.D.dapq_score_accumulate(shape, prob.q, prob.k, lse, T, ws)
    assert torch.equal(S, T) and torch.equal(S, S[:1].expand_as(S)) and torch.equal(lse, lse[:1].expand_as(lse))
    S, lse, logs = S[0].cpu().numpy(), lse[0].cpu().numpy(), oracle_lse2(q, k, 2, cu)[0]
    assert not S[:, hidden].any()
    for b in range(batch):
        here = slice(int(cu[b]), int(cu[b + 1]))
        if not hidden[here].all():
            H.assert_scores_close(S[None, :, here], O.score(q[:, b:b + 1], k[:, here], 2), f"sequence {b} of {lens}, rows={rows}")
            assert np.abs(lse[b] - logs[b]).max() < 2e-4


# the pseudo tokens' own block: the only key that the first row sees, a sub-block, the last keys
@pytest.mark.parametrize("rows,masked", [(20, (0, 1)), (40, (0, 33)), (130, (0, 40)), (64, (50, 64))])
def test_masked_pseudo_keys(H, rows, masked):
    """The oracle's scores over the extended sequence within 1e-3."""
    announce(f"masked pseudo keys {masked}, rows={rows}")
    q, k, v, cu = problem_bits(rows, 1, [300], 2, 2, rows)
    q[..., 0] = W.to_bf16_bits(np.full(q.shape[:-1], 2.0, dtype=np.float32))
    kp = problem_bits(rows + 1, 1, [1], 2, 2, rows)[0]
    kp[:, :, :, masked[0]:masked[1]] = 0
    kp[:, :, :, masked[0]:masked[1], 0] = 0xFF7F
    S = H.Problem(q, k, v, 2, None, "thd").score_extended(kp)
    H.assert_scores_close(S.cpu().numpy(), O.score(q, k, 2, cu, None, kp), f"masked pseudo keys, rows={rows}")


@pytest.mark.parametrize("rows", [33, 96, 128, 160, 192, 224, 250])
@pytest.mark.parametrize("layers,batch,length", [(160, 2, 700), (100, 3, 1500), (40, 5, 3000)])
def test_one_or_two_chunks_in_one_kernel(H, layers, batch, length, rows):
    """One chunk of a sequence, or two, longer than the power of two (sums in two steps): as above."""
    test_equal_chunks_of_dense_batches(H, layers, batch, length, rows)


# calls whose own workspace would be larger than that of a larger shape, which they are given: longer chunks (sums in one step and, where
# they are longer than the power of two, in two; one chunk per sequence; two row groups), fewer segments
@pytest.mark.parametrize("rows,lens,layers,larger,ragged", [
    (250, [4402], 28, 48, False), (250, [1491] * 3, 42, 64, False), (33, [1592] * 3, 41, 64, False), (33, [980] * 3, 72, 128, False),
    (300, [1617] * 7, 20, 24, False), (300, [1293] * 7, 6, 8, False), (128, [4418], 18, 24, False),
    (300, [2000, 0, 7, 3000, 401, 31, 70], 116, 128, True), (250, [3000, 3, 504], 66, 100, True), (128, [4660], 117, 128, True)])
def test_calls_in_the_workspace_of_a_larger_shape(H, rows, lens, layers, larger, ragged):
    """The oracle's scores and normalisers (the bars of the other score tests), the same bits in every layer and from the two separate
    entry points; every layer is the same problem (layer strides of 0)."""
    announce(f"workspace of {larger} layers: {layers} of {len(lens)}x{max(lens)}, rows={rows}")
    q, k, v, cu = problem_bits(rows + layers, 1, lens, 2, 2, rows)
    b = int(np.argmax(lens))
    k[0, int(cu[b]) + 2 * lens[b] // 3, 1] = W.to_bf16_bits(30.0 * O.bf16_bits_to_f64(q[0, b, 1, 0]))
    prob = H.Problem(q, k, v, 2, cu if ragged else None, "thd")
    tokens = int(cu[-1])

    def shape(n_layers):
        return H.D.make_shape(n_layers=n_layers, batch=len(lens), n_q_heads=2, n_kv_heads=2, n_pseudo=rows, total_tokens=tokens,
                              cu_seqlens=prob.cu, k_strides=(0, 0, 128, 256), q_strides=(0, 2 * rows * 128, rows * 128, 128),
                              scale=128 ** -0.5)
    room = H.D.workspace_bytes(shape(larger))
    assert room < H.D.workspace_bytes(shape(layers))
    guard = torch.full((room + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    ws = guard[:room]
    S, T = (torch.full((layers, 2, tokens), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2))
    lse = torch.full((layers, len(lens), 2, rows), float("nan"), dtype=torch.float32, device="cuda")
    H.D.dapq_score(shape(layers), prob.q, prob.k, S, ws)
    H.D.dapq_score_stats(shape(layers), prob.q, prob.k, lse, ws)
    H.D.dapq_score_accumulate(shape(layers), prob.q, prob.k, lse, T, ws)
    assert (guard[room:] == 0xA5).all()
    assert torch.equal(S, T) and torch.equal(S, S[:1].expand_as(S)) and torch.equal(lse, lse[:1].expand_as(lse))
    H.assert_scores_close(S[:1].cpu().numpy(), O.score(q, k, 2, cu), f"{lens} rows={rows}")
    live = [i for i, n in enumerate(lens) if n]
    assert np.abs(lse[:1].cpu().numpy()[:, live] - oracle_lse2(q, k, 2, cu)[:, live]).max() < 2e-4


# segments that begin and end inside sequences, take in several, empty ones among them, or hold one sub-block; a head of one key
@pytest.mark.parametrize("rows", [33, 128, 250, 300])
@pytest.mark.parametrize("lens", [[1, 0, 31, 32, 33, 0, 0, 64, 900, 5, 0, 1300, 0], [0, 2500, 0, 65], [1], [0, 3, 0]],
                         ids=lambda lens: f"{len(lens)}x{max(lens)}")
def test_segments_of_ragged_batches(H, rows, lens):
    """Enough layers of the same problem for the wave form, with a key hundreds of binades above the others (its piece is summed
    again): the oracle's scores and normalisers (the bars of the other score tests), the same bits in every layer and from the two
    separate entry points."""
    announce(f"segments: {lens} rows={rows}")
    q, k, v, cu = problem_bits(rows, 1, lens, 2, 2, rows)
    tokens = int(cu[-1])
    layers = 66000 // (2 * (tokens // 128 + len(lens)) * ((rows + 31) // 32)) + 1
    b = int(np.argmax(lens))
    if tokens > 1:
        k[0, int(cu[b]) + 3 * lens[b] // 5, 1] = W.to_bf16_bits(30.0 * O.bf16_bits_to_f64(q[0, b, 1, 0]))
    prob = H.Problem(q, k, v, 2, cu, "thd")
    shape = H.D.make_shape(n_layers=layers, batch=len(lens), n_q_heads=2, n_kv_heads=2, n_pseudo=rows, total_tokens=tokens,
                           cu_seqlens=prob.cu, k_strides=(0, 0, 128, 256), q_strides=(0, 2 * rows * 128, rows * 128, 128),
                           scale=128 ** -0.5)
    ws_bytes = H.D.workspace_bytes(shape)
    ws = torch.full((ws_bytes,), 0xA5, dtype=torch.uint8, device="cuda")
    S, T = (torch.full((layers, 2, tokens), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2))
    lse = torch.full((layers, len(lens), 2, rows), float("nan"), dtype=torch.float32, device="cuda")
    H.D.dapq_score(shape, prob.q, prob.k, S, ws)
    H.D.dapq_score_stats(shape, prob.q, prob.k, lse, ws)
    H.D.dapq_score_accumulate(shape, prob.q, prob.k, lse, T, ws)
    assert torch.equal(S, T) and torch.equal(S, S[:1].expand_as(S)) and torch.equal(lse, lse[:1].expand_as(lse))
    if tokens:
        H.assert_scores_close(S[:1].cpu().numpy(), O.score(q, k, 2, cu), f"{lens} rows={rows}")
    live = [i for i, n in enumerate(lens) if n]
    err = np.abs(lse[:1].cpu().numpy()[:, live] - oracle_lse2(q, k, 2, cu)[:, live])
    assert not live or err.max() < 2e-4


# fewer channel pairs than a wave has lanes, one wave, a few; heads up to the most a launch takes
@pytest.mark.parametrize("rows,heads,d", [(1, 65536, 64), (1, 100000, 64), (1, 65535 * 8, 8), (2, 9000, 64), (1, 3, 128), (3, 1025, 24)])
def test_rotation_of_many_heads(H, rows, heads, d):
    """The oracle's bits, as in the other tests of the rotation."""
    announce(f"rotation: {rows} rows, {heads} heads of {d}")
    rng = np.random.default_rng(heads)
    x = W.to_bf16_bits(rng.standard_normal((rows, heads, d), dtype=np.float32))
    pos = rng.integers(0, 140000, rows)
    assert np.array_equal(H.rope_gpu(x, pos, 500000.0), O.rope_apply(x, pos, 500000.0))


@pytest.mark.parametrize("offset", [0, 4, 8])
def test_candidates_of_long_heads_off_16_bytes(H, offset):
    """A workspace that starts `offset` bytes past a 16-byte boundary gives the oracle's positions too."""
    announce(f"selection in pieces, workspace {offset} bytes off")
    n, budget = 100000, 1000
    S = np.random.default_rng(offset).random((1, 2, n), dtype=np.float32)
    zero = np.zeros((1, n, 2, 128), dtype=np.uint16)
    prob = H.Problem(np.zeros((1, 1, 2, 1, 128), dtype=np.uint16), zero, zero, 2, None, "hnd")
    need = H.D.topk_workspace_bytes(prob.shape, budget)
    ws = torch.full((need + 16,), 0xA5, dtype=torch.uint8, device="cuda")[offset:offset + need]
    idx = torch.empty((1, 1, 2, budget), dtype=torch.int32, device="cuda")
    count = torch.empty((1, 1, 2), dtype=torch.int32, device="cuda")
    H.D.dapq_topk(prob.shape, torch.from_numpy(S).cuda(), budget, None, idx, count, ws)
    for kv in range(2):
        assert np.array_equal(idx.cpu().numpy()[0, 0, kv], O.topk(S[0, kv].astype(np.float64), budget))


# a wave holds two to eight row blocks, the row groups of a head as many each: the last rows of one number and the first of the next,
# one to three groups; both passes in one kernel, in separate launches, and in segments of a ragged batch
@pytest.mark.parametrize("lens,layers,ragged", [([700, 700], 130, False), ([5100], 30, False), ([1500, 0, 33, 800, 64], 200, True)],
                         ids=["one kernel", "launches", "segments"])
@pytest.mark.parametrize("rows", [64, 65, 96, 97, 129, 160, 161, 192, 193, 224, 225, 257, 321, 449, 513])
def test_row_blocks_of_a_wave(H, rows, lens, layers, ragged):
    """Every layer is the same problem (layer strides of 0): the oracle's scores within 1e-3, with and without the pseudo tokens' own keys
    in the normaliser, the same bits in every layer and from the two separate entry points."""
    announce(f"row blocks: rows={rows} {lens}")
    q, k, v, cu = problem_bits(rows, 1, lens, 1, 1, rows)
    prob = H.Problem(q, k, v, 1, cu if ragged else None, "thd")
    tokens = int(cu[-1])
    layers = layers * 513 // rows if ragged else layers                                     # beyond the tile form
    shape = H.D.make_shape(n_layers=layers, batch=len(lens), n_q_heads=1, n_kv_heads=1, n_pseudo=rows, total_tokens=tokens,
                           cu_seqlens=prob.cu, k_strides=(0, 0, 128, 128), q_strides=(0, rows * 128, rows * 128, 128), scale=128 ** -0.5)
    if not ragged:  # (dense calls of up to 1024 tiles of 128 keys may take the tile form)
        assert len(lens) == 2 or layers * -(-tokens // 128) > 1024
        assert H.D.score_single_launch(shape) == (len(lens) == 2 and rows <= 256)
    ws = torch.full((H.D.workspace_bytes(shape),), 0xA5, dtype=torch.uint8, device="cuda")
    S, T, X = (torch.full((layers, 1, tokens), float("nan"), dtype=torch.float32, device="cuda") for _ in range(3))
    lse = torch.full((layers, len(lens), 1, rows), float("nan"), dtype=torch.float32, device="cuda")
    H.D.dapq_score(shape, prob.q, prob.k, S, ws)
    H.D.dapq_score_stats(shape, prob.q, prob.k, lse, ws)
    H.D.dapq_score_accumulate(shape, prob.q, prob.k, lse, T, ws)
    assert torch.equal(S, T) and torch.equal(S, S[:1].expand_as(S))
    H.assert_scores_close(S[:1].cpu().numpy(), O.score(q, k, 1, cu), f"rows={rows}")
    kp = W.to_bf16_bits(np.random.default_rng(rows).standard_normal((1, len(lens), 1, rows, 128), dtype=np.float32))
    H.D.dapq_score_stats_extend(shape, prob.q, H.dev_bf16(kp), (0, rows * 128, rows * 128, 128), lse)
    H.D.dapq_score_accumulate(shape, prob.q, prob.k, lse, X, ws)
    assert torch.equal(X, X[:1].expand_as(X))
    H.assert_scores_close(X[:1].cpu().numpy(), O.score(q, k, 1, cu, None, kp), f"extended, rows={rows}")


# more keys than the caches hold until pass 2 (of up to four row blocks 384 MB, of more 1536 MB of a dense and 768 MB of a ragged batch): what
# pass 1 leaves in the caches starts inside a chunk, whose last sub-block is partial; two to eight row blocks
@pytest.mark.parametrize("lens,layers,ragged", [([24101], 256, False), ([61003], 101, False), ([9000, 0, 33, 15000, 70], 256, True)],
                         ids=["one kernel", "launches", "segments"])
@pytest.mark.parametrize("rows", [40, 96, 128, 160, 200, 224, 256])
def test_keys_that_stream(H, rows, lens, layers, ragged):
    """Every layer is the same problem (layer strides of 0): the oracle's scores within 1e-3, the same bits in every layer and from the
    two separate entry points."""
    announce(f"streamed keys: rows={rows} {lens}")
    assert layers * sum(lens) * 256 >= 1536e6
    q, k, v, cu = problem_bits(rows, 1, lens, 1, 1, rows)
    prob = H.Problem(q, k, v, 1, cu if ragged else None, "thd")
    tokens = int(cu[-1])
    shape = H.D.make_shape(n_layers=layers, batch=len(lens), n_q_heads=1, n_kv_heads=1, n_pseudo=rows, total_tokens=tokens,
                           cu_seqlens=prob.cu, k_strides=(0, 0, 128, 128), q_strides=(0, rows * 128, rows * 128, 128), scale=128 ** -0.5)
    assert H.D.score_single_launch(shape) == (layers == 256 and not ragged)
    ws = torch.full((H.D.workspace_bytes(shape),), 0xA5, dtype=torch.uint8, device="cuda")
    S, T = (torch.full((layers, 1, tokens), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2))
    lse = torch.full((layers, len(lens), 1, rows), float("nan"), dtype=torch.float32, device="cuda")
    H.D.dapq_score(shape, prob.q, prob.k, S, ws)
    H.D.dapq_score_stats(shape, prob.q, prob.k, lse, ws)
    H.D.dapq_score_accumulate(shape, prob.q, prob.k, lse, T, ws)
    assert torch.equal(S, T) and torch.equal(S, S[:1].expand_as(S))
    H.assert_scores_close(S[:1].cpu().numpy(), O.score(q, k, 1, cu), f"rows={rows}")


def selection_call(H, S, batch, width, budget, pieces):
    """dapq_pool_topk over scores [layers][heads][batch * length]: positions, counts and pooled scores on the host."""
    layers, heads, tokens = S.shape
    shape = H.D.make_shape(n_layers=layers, batch=batch, n_q_heads=heads, n_kv_heads=heads, n_pseudo=1, total_tokens=tokens, scale=1.0)
    n = H.D.topk_workspace_bytes(shape, budget) if pieces else 0
    ws = torch.full((n,), 0xA5, dtype=torch.uint8, device="cuda") if n else None
    dev = torch.from_numpy(S).cuda()
    idx = torch.full((layers, batch, heads, budget), -7, dtype=torch.int32, device="cuda")
    count = torch.full((layers, batch, heads), -7, dtype=torch.int32, device="cuda")
    pooled = torch.full_like(dev, float("nan"))
    H.D.dapq_pool_topk(shape, dev, width, budget, None, idx, count, pooled, workspace=ws)
    return idx.cpu().numpy(), count.cpu().numpy(), pooled.cpu().numpy()


def check_selection(S, batch, width, budget, got, sample):
    idx, count, pooled = got
    length = S.shape[2] // batch
    for l, b, h in sample:
        P = O.pool(S[l, h, b * length:(b + 1) * length].astype(np.float64), width)
        want = O.topk(P, budget)
        assert np.array_equal(pooled[l, h, b * length:(b + 1) * length].astype(np.float64), P), (l, b, h)
        assert count[l, b, h] == len(want) and np.array_equal(idx[l, b, h, :len(want)], want), (l, b, h)
        assert (idx[l, b, h, len(want):] == -7).all()


# the lengths around every variant's limit, as many heads as compute units and more, scores on and off 16 bytes (sequences of an odd length
# follow each other), waves of the last one full, partly filled and empty
@pytest.mark.parametrize("heads", [4, 300])
@pytest.mark.parametrize("length", [1, 3, 511, 513, 2047, 2048, 2049, 4095, 4097, 8191, 8192, 8193, 16383, 16385, 32767])
def test_selection_variants(H, length, heads):
    """The pooled scores and retained positions are the oracle's, bit for bit."""
    announce(f"selection variants: {heads} x 2 of {length}")
    rng = np.random.default_rng(length + heads)
    S = rng.lognormal(0.0, 0.5, (heads // 4, 2, 2 * length)).astype(np.float32)
    sample = [(0, 0, 0), (0, 1, 1), (heads // 4 - 1, 1, 0)]
    for width, budget in ((7, max(1, length // 5)), (1, 40), (9, length + 3)):
        check_selection(S, 2, width, budget, selection_call(H, S, 2, width, budget, False), sample)


# pieces whose survivors fit the area they go out through and not; candidate lists of every merge kernel, of whole quads and not
@pytest.mark.parametrize("length,budget", [(40001, 100), (40000, 4000), (65539, 4097), (65536, 16000), (65536, 16449), (70001, 20000), (70000, 20001)])
def test_survivors_of_pieces(H, length, budget):
    """The pooled scores and retained positions are the oracle's, bit for bit."""
    announce(f"survivors of pieces: {budget} of {length}")
    rng = np.random.default_rng(budget)
    S = rng.lognormal(0.0, 0.5, (2, 2, length)).astype(np.float32)
    for width in (1, 7):
        check_selection(S, 1, width, budget, selection_call(H, S, 1, width, budget, True), [(0, 0, 0), (1, 0, 1)])


# ragged batches of many heads much shorter than their kernel could hold, whose scores come straight from memory, and as many as still go
# through LDS; heads on and off 16 bytes, empty, of one key, longer than a wave holds and as long as the workgroup
@pytest.mark.parametrize("lens,layers,pieces", [
    ([0, 1, 37, 601, 2049, 1300, 8, 3000], 65, False),              # 256 threads, 1040 heads
    ([0, 1, 37, 601, 2049, 1300, 8, 3000], 64, False),              # 1024
    ([5, 8192, 0, 13, 640, 1, 66, 2100], 65, True),                 # and a longer total: the same kernel beside the pieces
    ([5, 8192, 0, 13, 640, 1, 66, 2100], 33, False),                # 512 threads, 528 heads
    ([16000, 3, 0, 129, 32, 1, 64, 31], 33, False)])
def test_short_heads_of_ragged_batches(H, lens, layers, pieces):
    """The pooled scores and retained positions are the oracle's, bit for bit."""
    announce(f"short heads: {layers} x 2 of {lens}, pieces {pieces}")
    rng = np.random.default_rng(layers + lens[0])
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    S = rng.lognormal(0.0, 0.5, (layers, 2, int(cu[-1]))).astype(np.float32)
    dev, cu_dev = torch.from_numpy(S).cuda(), torch.from_numpy(cu).cuda()
    for width, budget in ((7, 300), (1, 40), (9, 9000)):
        shape = H.D.make_shape(n_layers=layers, batch=len(lens), n_q_heads=2, n_kv_heads=2, n_pseudo=1, total_tokens=int(cu[-1]),
                               cu_seqlens=cu_dev, scale=1.0)
        n = H.D.topk_workspace_bytes(shape, budget) if pieces else 0
        assert bool(n) == pieces
        ws = torch.full((n,), 0xA5, dtype=torch.uint8, device="cuda") if n else None
        idx = torch.full((layers, len(lens), 2, budget), -7, dtype=torch.int32, device="cuda")
        count = torch.full((layers, len(lens), 2), -7, dtype=torch.int32, device="cuda")
        pooled = torch.full_like(dev, float("nan"))
        H.D.dapq_pool_topk(shape, dev, width, budget, None, idx, count, pooled, workspace=ws)
        got, counts, P = idx.cpu().numpy(), count.cpu().numpy(), pooled.cpu().numpy()
        for l, h in ((0, 0), (layers // 2, 1), (layers - 1, 0)):
            for b in range(len(lens)):
                head = slice(int(cu[b]), int(cu[b + 1]))
                want_p = O.pool(S[l, h, head].astype(np.float64), width)
                want = O.topk(want_p, budget)
                assert np.array_equal(P[l, h, head].astype(np.float64), want_p), (l, h, b)
                assert counts[l, b, h] == len(want) and np.array_equal(got[l, b, h, :len(want)], want), (l, h, b)
                assert (got[l, b, h, len(want):] == -7).all()


# bytes moved around the lines of the non-temporal hints (8 MB: 128 heads of 64 rows; 192 MB: 3072 of 64), budgets around a workgroup's
# 32 rows; heads that keep nothing, less than the budget, all of it
@pytest.mark.parametrize("heads,budget", [(2, 1), (2, 33), (128, 63), (128, 64), (3072, 63), (3072, 64), (2049, 97)], ids=str)
@pytest.mark.parametrize("ragged", [False, True])
def test_gather_with_and_without_streaming_hints(heads, budget, ragged):
    import paper_2603_11564_amd as D
    announce(f"gather of {heads} heads, budget {budget}, ragged {ragged}")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(heads + budget)
    L, H = 130, 4
    cu = torch.tensor([0, 101, L], dtype=torch.int32, device="cuda") if ragged else None
    batch = 2 if ragged else 1
    layers = (heads + H * batch - 1) // (H * batch)
    # every layer reads the same keys and values (layer stride 0)
    k = torch.randint(-32768, 32767, (H, L, 128), dtype=torch.int16, device="cuda", generator=gen)
    v = torch.randint(-32768, 32767, (H, L, 128), dtype=torch.int16, device="cuda", generator=gen)
    strides = (0, 0, L * 128, 128)
    shape = D.make_shape(n_layers=layers, batch=batch, n_q_heads=H, n_kv_heads=H, n_pseudo=1, total_tokens=L, cu_seqlens=cu,
                         k_strides=strides, v_strides=strides, scale=1.0)
    lens = [101, L - 101] if ragged else [L]
    idx = torch.stack([torch.randint(0, n, (layers, H, budget), dtype=torch.int32, device="cuda", generator=gen) for n in lens], 1)
    count = torch.randint(0, budget + 1, (layers, batch, H), dtype=torch.int32, device="cuda", generator=gen)
    count[0], count[-1] = budget, budget - 1
    out = [torch.full((layers, batch, H, budget, 128), 77, dtype=torch.int16, device="cuda") for _ in range(2)]
    D.dapq_gather(shape, k, v, idx, count, budget, out[0], out[1])
    start = torch.tensor([0, 101], device="cuda")[:batch].view(1, batch, 1, 1)
    kept = torch.arange(budget, device="cuda") < count[..., None]
    for got, src in zip(out, (k, v)):
        want = src[torch.arange(H, device="cuda").view(1, 1, H, 1), idx + start]
        want[~kept] = 77  # slots past the count stay as they were
        assert torch.equal(got, want)


# 128 MB of caches, one sweep over them or (more than 8 query heads) several
@pytest.mark.parametrize("heads,rows,g", [(256, 976, 4), (256, 977, 4), (256, 977, 1), (300, 851, 8), (256, 977, 9)])
def test_decode_caches_that_stream(H, heads, rows, g):
    test_decode_lines_between_slices(H, heads, rows, g)


# 4 MB of results, runs of heads that are not whole trips of four
@pytest.mark.parametrize("rows,heads", [(64, 255), (64, 256), (64, 259), (1031, 19)])
def test_rotation_that_streams(H, rows, heads):
    test_rotation_of_many_heads(H, rows, heads, 128)
