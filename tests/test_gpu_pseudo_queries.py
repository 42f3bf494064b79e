"""GPU parity of dapq_pseudo_queries (gather of the copied tokens' rows, query projection on MFMA, head split,
rotation) against the float64 oracle, through the C ABI.

Comparison rule.  The oracle rounds the exact sum e to bf16; the kernel rounds an fp32 accumulation a of the
same exact products.  |a - e| is bounded by the accumulation error acc_tol (4 sqrt(hidden) 2^-24 sum|x w|:
n exact products, n - 1 roundings of partial sums, taken at the usual square-root growth with a factor 4), so
every result must lie within ulp_bf16/2 + acc_tol of e (ulp taken at |e| + acc_tol), can differ from the oracle's
bits only where e is that close to a rounding boundary (well under 1 % of the elements), and then by one bf16 step.  After the
rotation (bit-exact for equal inputs) the same holds with two inputs per output."""
import sys

import numpy as np
import pytest
import torch

import workloads as W
from qproj_shapes import SPLIT_SHAPES
from oracle import dapq_oracle as O

pytestmark = pytest.mark.gpu


def announce(msg):
    print(f"[gpu-case] {msg}", file=sys.__stderr__, flush=True)


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import dapq_harness
    return dapq_harness


def bf16_ulp(v):
    """Spacing of bf16 (8 significant bits) at |v| (normal range)."""
    e = np.floor(np.log2(np.maximum(np.abs(v), 2.0 ** -120)))
    return 2.0 ** (e - 7)


def run_case(H, seed, layers, tokens, hidden, Hq, d, tok, positions=None, pairing=0, theta=500000.0,
             x_pad=0, w_pad=0, shared_x=False, q_pad_rows=0):
    """One call of the entry point; returns device output bits [layers, Hq, rows, d] and the host inputs."""
    F = Hq * d
    rows = len(tok)
    x_bits = np.stack([W.projection_rows(seed, l, tokens, hidden) for l in range(1 if shared_x else layers)])
    w_bits = np.stack([W.query_weight(seed, l, F, hidden) for l in range(layers)])
    # padded strides: rows of x / w sit in wider rows whose tail holds NaN patterns that must never be read
    xs, wsr = hidden + x_pad, hidden + w_pad
    x_dev = np.full((x_bits.shape[0], tokens, xs), 0x7FC0, dtype=np.uint16)
    x_dev[:, :, :hidden] = x_bits
    w_dev = np.full((layers, F, wsr), 0x7FC0, dtype=np.uint16)
    w_dev[:, :, :hidden] = w_bits
    x_t, w_t = H.dev_bf16(x_dev), H.dev_bf16(w_dev)
    tok_t = torch.tensor(tok, dtype=torch.int32, device="cuda")
    pos_t = None if positions is None else torch.tensor(positions, dtype=torch.int32, device="cuda")
    q_rows = rows + q_pad_rows
    q_t = H.dev_bf16(np.full((layers, Hq, q_rows, d), 0x7FC1, dtype=np.uint16))
    desc = H.D.Qproj(n_layers=layers, rows=rows, hidden=hidden, n_q_heads=Hq, head_dim=d, total_tokens=tokens,
                     x_stride_layer=0 if shared_x else tokens * xs, x_stride_token=xs,
                     w_stride_layer=F * wsr, w_stride_row=wsr,
                     q_stride_layer=Hq * q_rows * d, q_stride_head=q_rows * d, q_stride_row=d)
    ws = torch.empty(max(H.D.pseudo_queries_workspace_bytes(desc), 16), dtype=torch.uint8, device="cuda")
    H.D.dapq_pseudo_queries(desc, x_t, tok_t, w_t, pos_t, theta, pairing, q_t, ws)
    torch.cuda.synchronize()
    got = H.host_bits(q_t)
    assert (got[:, :, rows:] == 0x7FC1).all(), "rows past `rows` were written"
    return got[:, :, :rows], x_bits, w_bits


def check_projection(got_bits, x_bits, w_bits, tok, Hq, hidden, shared_x=False):
    layers = w_bits.shape[0]
    tok = np.asarray(tok)
    worst_equal = 1.0
    for l in range(layers):
        xb = x_bits[0 if shared_x else l]
        valid = (tok >= 0) & (tok < xb.shape[0])
        # (the library reads indices past the end as rows without a source; the method knows no such index)
        want_bits = O.pseudo_queries(xb, np.where(valid, tok, -1), w_bits[l], Hq)
        x = O.bf16_bits_to_f64(xb)
        w = O.bf16_bits_to_f64(w_bits[l])
        xg = np.where(valid[:, None], x[np.clip(tok, 0, xb.shape[0] - 1)], 0.0)
        e = (xg @ w.T).reshape(len(tok), Hq, -1).transpose(1, 0, 2)
        acc_tol = 4.0 * np.sqrt(hidden) * 2.0 ** -24 * (np.abs(xg) @ np.abs(w).T).reshape(len(tok), Hq, -1).transpose(1, 0, 2)
        got = O.bf16_bits_to_f64(got_bits[l])
        want = O.bf16_bits_to_f64(want_bits)
        assert np.isfinite(got).all()
        ulp = bf16_ulp(np.abs(e) + acc_tol)          # the accumulated value may sit a binade above a tiny exact sum
        assert (np.abs(got - e) <= 0.5 * ulp + acc_tol).all(), f"layer {l}: outside half an ulp of the exact sum"
        assert (np.abs(got - want) <= ulp + acc_tol).all()
        if (~valid).any():
            assert (got_bits[l][:, ~valid] == 0).all()
        worst_equal = min(worst_equal, float((got_bits[l] == want_bits).mean()))
    return worst_equal


SHAPES = [
    # layers, tokens, hidden, Hq, d, rows
    (1, 9, 64, 1, 8, 5),          # one partial feature tile, one partial row block, one hidden block
    (2, 50, 128, 3, 32, 33),      # 96 features: last wave half empty; 33 rows: second row block nearly empty
    (1, 70, 192, 5, 32, 64),      # 160 features; three hidden blocks (the ring drains mid-way)
    (3, 40, 256, 2, 64, 65),      # two sweeps of rows, the second with one row
    (1, 300, 1024, 4, 128, 130),  # three sweeps; head_dim 128
    (1, 31, 320, 2, 128, 32),     # exactly one row block (one-block variant)
    (2, 64, 64, 8, 16, 1),        # a single row
    (1, 40, 1088, 2, 64, 40),     # 17 hidden blocks dealt to two waves per tile (9 + 8), sums added from the workspace
    (1, 100, 4096, 8, 128, 64),   # one layer of a 4096-wide model: eight waves per tile
    (2, 30, 2048, 1, 72, 7),      # 72 features: a tile with 8 live features, four-way split
]


@pytest.mark.parametrize("case", range(len(SHAPES)))
def test_projection_matches_oracle(H, case):
    layers, tokens, hidden, Hq, d, rows = SHAPES[case]
    announce(f"pseudo queries: projection case {case} {SHAPES[case]}")
    r = np.random.default_rng(300 + case)
    tok = r.integers(0, tokens, rows).tolist()
    got, x_bits, w_bits = run_case(H, 40 + case, layers, tokens, hidden, Hq, d, tok)
    equal = check_projection(got, x_bits, w_bits, tok, Hq, hidden)
    assert equal > 0.99, equal


@pytest.mark.parametrize("seed", range(48))
def test_projection_random_shapes(H, seed):
    """Seeded random shapes: layers, rows, hidden blocks, head counts and sizes, padded strides, missing sources,
    one x for all layers or one per layer -- every combination of kernel variant, sweep count and hidden split that
    small shapes can reach."""
    r = np.random.default_rng(5000 + seed)
    layers = int(r.integers(1, 4))
    rows = int(r.choice([1, 2, 31, 32, 33, 63, 64, 65, 96, 129, int(r.integers(1, 200))]))
    hidden = 64 * int(r.choice([1, 2, 3, 5, 8, 16, 17, 33, 40]))
    Hq = int(r.integers(1, 9))
    d = int(r.choice([8, 16, 24, 32, 64, 128]))
    tokens = int(r.integers(1, 120))
    tok = r.integers(-1, tokens, rows).tolist()
    x_pad, w_pad = int(r.choice([0, 8, 64])), int(r.choice([0, 8, 72]))
    shared = bool(r.integers(0, 2))
    announce(f"pseudo queries random {seed}: layers {layers} rows {rows} hidden {hidden} Hq {Hq} d {d} tokens {tokens} "
             f"pads {x_pad},{w_pad} shared_x {shared}")
    got, x_bits, w_bits = run_case(H, 900 + seed, layers, tokens, hidden, Hq, d, tok, x_pad=x_pad, w_pad=w_pad,
                                   shared_x=shared, q_pad_rows=int(r.integers(0, 3)))
    equal = check_projection(got, x_bits, w_bits, tok, Hq, hidden, shared_x=shared)
    assert equal > 0.98, equal


def test_projection_many_waves_variants(H):
    """Grids of 1024 and more waves take the four-tile variants: 32 layers x 4096 features, 64 rows and 32 rows."""
    for rows in (64, 32, 100):
        announce(f"pseudo queries: four-tile variant, rows={rows}")
        layers, tokens, hidden, Hq, d = 32, 20, 128, 32, 128
        tok = np.random.default_rng(rows).integers(0, tokens, rows).tolist()
        got, x_bits, w_bits = run_case(H, 77, layers, tokens, hidden, Hq, d, tok)
        assert check_projection(got, x_bits, w_bits, tok, Hq, hidden) > 0.99


def test_projection_sources_strides_and_shared_rows(H):
    announce("pseudo queries: missing sources, padded strides, one x for all layers")
    layers, tokens, hidden, Hq, d = 2, 25, 192, 3, 32
    tok = [3, -1, 24, 0, 0, -1, 7, 25, 1000, 24]      # -1: no source; 25, 1000: past the end -> zero rows
    got, x_bits, w_bits = run_case(H, 51, layers, tokens, hidden, Hq, d, tok, x_pad=64, w_pad=8, q_pad_rows=3)
    assert check_projection(got, x_bits, w_bits, tok, Hq, hidden) > 0.99
    got, x_bits, w_bits = run_case(H, 52, layers, tokens, hidden, Hq, d, tok[:5], shared_x=True)
    assert check_projection(got, x_bits, w_bits, tok[:5], Hq, hidden, shared_x=True) > 0.99
    # an empty prompt: no tokens at all, every pseudo token without a source
    desc = H.D.Qproj(n_layers=1, rows=4, hidden=64, n_q_heads=1, head_dim=32, total_tokens=0, x_stride_layer=0,
                     x_stride_token=64, w_stride_layer=32 * 64, w_stride_row=64, q_stride_layer=4 * 32,
                     q_stride_head=4 * 32, q_stride_row=32)
    x_t = H.dev_bf16(np.zeros((1, 64), dtype=np.uint16))
    w_t = H.dev_bf16(W.query_weight(1, 0, 32, 64))
    q_t = H.dev_bf16(np.full((1, 4, 32), 0x7FC1, dtype=np.uint16))
    H.D.dapq_pseudo_queries(desc, x_t, torch.full((4,), -1, dtype=torch.int32, device="cuda"), w_t, None, 1.0, 0, q_t)
    torch.cuda.synchronize()
    assert (H.host_bits(q_t) == 0).all()
    # no rows: nothing is written
    desc.rows = 0
    q_t = H.dev_bf16(np.full((1, 4, 32), 0x7FC1, dtype=np.uint16))
    H.D.dapq_pseudo_queries(desc, x_t, torch.zeros(1, dtype=torch.int32, device="cuda"), w_t, None, 1.0, 0, q_t)
    torch.cuda.synchronize()
    assert (H.host_bits(q_t) == 0x7FC1).all()


@pytest.mark.parametrize("pairing", [0, 1])
def test_rotated_queries_match_oracle_and_the_two_calls(H, pairing):
    announce(f"pseudo queries: with rotation, pairing={pairing}")
    layers, tokens, hidden, Hq, d, rows = 3, 60, 256, 4, 128, 48
    r = np.random.default_rng(9 + pairing)
    tok = r.integers(0, tokens, rows).tolist()
    pos = (r.integers(0, 140000, rows)).tolist()
    got, x_bits, w_bits = run_case(H, 61, layers, tokens, hidden, Hq, d, tok, positions=pos, pairing=pairing)
    pre, _, _ = run_case(H, 61, layers, tokens, hidden, Hq, d, tok)
    name = "half" if pairing == 0 else "interleaved"
    for l in range(layers):
        # one call = projection, then dapq_rope_apply on its output: bit for bit
        pre_t = H.dev_bf16(pre[l].transpose(1, 0, 2))                       # [rows, Hq, d]
        out_t = torch.empty_like(pre_t)
        H.D.dapq_rope_apply(pre_t, out_t, torch.tensor(pos, dtype=torch.int32, device="cuda"), rows, Hq, d, Hq * d, d,
                            500000.0, pairing)
        torch.cuda.synchronize()
        assert np.array_equal(H.host_bits(out_t).transpose(1, 0, 2), got[l])
        # and the oracle's rotated queries: equal except where the projection sat on a rounding boundary
        want_bits = O.pseudo_queries(x_bits[l], tok, w_bits[l], Hq, positions=pos, pairing=name)
        g, w_ = O.bf16_bits_to_f64(got[l]), O.bf16_bits_to_f64(want_bits)
        p = O.bf16_bits_to_f64(O.pseudo_queries(x_bits[l], tok, w_bits[l], Hq))
        if pairing == 0:
            mag = np.maximum(np.abs(p[..., : d // 2]), np.abs(p[..., d // 2:]))
            mag = np.concatenate([mag, mag], axis=-1)
        else:
            mag = np.maximum(np.abs(p[..., 0::2]), np.abs(p[..., 1::2])).repeat(2, axis=-1)
        assert (np.abs(g - w_) <= 2.0 * bf16_ulp(np.sqrt(2.0) * mag)).all()
        assert (got[l] == want_bits).mean() > 0.98


# workspaces with room for 2, 4, 8 and 16 planes of sums, which are rotated as they are added up (how many a call writes: the shapes by plan
# below); channel pairs that do not fill a workgroup, head sizes that do not fill a feature tile, one and several sweeps and layers
@pytest.mark.parametrize("pairing", [0, 1])
@pytest.mark.parametrize("hidden,splits", [(1024, 2), (2048, 4), (4096, 8), (8192, 16)])
@pytest.mark.parametrize("layers,Hq,d,rows", [(1, 3, 72, 37), (2, 2, 128, 65), (1, 1, 8, 1)])
def test_rotated_queries_of_split_calls(H, layers, Hq, d, rows, hidden, splits, pairing):
    """One call = the projection (without positions), then dapq_rope_apply on its output: bit for bit, with missing sources, padded
    strides and rows past the end left alone; and the projection is the oracle's (check_projection)."""
    announce(f"pseudo queries: rotation, room for {splits} planes, {layers} layers, {Hq} heads of {d}, {rows} rows, pairing {pairing}")
    r = np.random.default_rng(hidden + rows)
    tokens = 20
    tok = r.integers(-1, tokens, rows).tolist()
    pos = r.integers(0, 140000, rows).tolist()
    desc = H.D.Qproj(n_layers=layers, rows=rows, hidden=hidden, n_q_heads=Hq, head_dim=d, total_tokens=tokens, x_stride_layer=0,
                     x_stride_token=hidden, w_stride_layer=0, w_stride_row=hidden, q_stride_layer=0, q_stride_head=rows * d,
                     q_stride_row=d)
    block = 64 if rows > 32 else 32
    assert H.D.pseudo_queries_workspace_bytes(desc) == splits * layers * (-(-rows // block) * block) * (-(-Hq * d // 64) * 64) * 4
    args = dict(x_pad=8, w_pad=8, q_pad_rows=2)
    got, x_bits, w_bits = run_case(H, 80, layers, tokens, hidden, Hq, d, tok, positions=pos, pairing=pairing, **args)
    pre, _, _ = run_case(H, 80, layers, tokens, hidden, Hq, d, tok, **args)
    check_projection(pre, x_bits, w_bits, tok, Hq, hidden)
    for l in range(layers):
        turned = H.rope_gpu(np.ascontiguousarray(pre[l].transpose(1, 0, 2)), pos, 500000.0, pairing)
        assert np.array_equal(turned.transpose(1, 0, 2), got[l])


@pytest.mark.parametrize("shape", SPLIT_SHAPES, ids=lambda shape: "x".join(map(str, shape)))
def test_every_number_of_planes(H, shape):
    """The projection is the oracle's (check_projection), its rotation is dapq_rope_apply's, bit for bit."""
    layers, Hq, d, rows, hidden = shape
    announce(f"pseudo queries: {SPLIT_SHAPES[shape]} waves and planes, {shape}")
    r = np.random.default_rng(hidden + rows)
    tok, pos = r.integers(0, 40, rows).tolist(), r.integers(0, 140000, rows).tolist()
    pre, x_bits, w_bits = run_case(H, 82, layers, 40, hidden, Hq, d, tok)
    got, _, _ = run_case(H, 82, layers, 40, hidden, Hq, d, tok, positions=pos)
    check_projection(pre, x_bits, w_bits, tok, Hq, hidden)
    for l in range(layers):
        turned = H.rope_gpu(np.ascontiguousarray(pre[l].transpose(1, 0, 2)), pos, 500000.0)
        assert np.array_equal(turned.transpose(1, 0, 2), got[l])


# hidden axes dealt to one and to four waves of a workgroup, in equal shares and with shares that are short or empty
@pytest.mark.parametrize("hidden", [1024, 1088, 1344, 2240, 4096, 5120, 6208])
@pytest.mark.parametrize("layers,Hq,d,rows", [(1, 8, 128, 64), (3, 2, 72, 30), (9, 16, 128, 33), (1, 5, 64, 130)])
def test_shares_of_the_hidden_axis(H, layers, Hq, d, rows, hidden):
    """The projection is the oracle's (check_projection), its rotation is dapq_rope_apply's, bit for bit."""
    announce(f"pseudo queries: shares of {hidden}, {layers} layers, {Hq} heads of {d}, {rows} rows")
    r = np.random.default_rng(hidden + rows)
    tok, pos = r.integers(0, 40, rows).tolist(), r.integers(0, 140000, rows).tolist()
    pre, x_bits, w_bits = run_case(H, 81, layers, 40, hidden, Hq, d, tok)
    got, _, _ = run_case(H, 81, layers, 40, hidden, Hq, d, tok, positions=pos)
    check_projection(pre, x_bits, w_bits, tok, Hq, hidden)
    for l in range(layers):
        turned = H.rope_gpu(np.ascontiguousarray(pre[l].transpose(1, 0, 2)), pos, 500000.0)
        assert np.array_equal(turned.transpose(1, 0, 2), got[l])


def test_queries_feed_the_score_path(H):
    """token indices -> queries -> scores: the chain of Sec. 4.1 and 4.2 on the device against the same chain in the
    oracle.  The device's queries may differ from the oracle's by one bf16 step where the projection sat on a
    rounding boundary (checked above: under 1 % of the elements); one such step moves a logit by at most
    2^-8 |q_c k_c| / sqrt(d) < 3e-3 here, so the scores are compared at 5e-3 instead of the 1e-3 that holds
    for equal queries."""
    announce("pseudo queries: chained into dapq_score")
    layers, L, hidden, Hq, Hkv, d, m, n = 1, 700, 256, 4, 2, 128, 4, 28
    N = m + n
    r = np.random.default_rng(123)
    k_bits = W.to_bf16_bits(r.standard_normal((layers, L, Hkv, d)))
    x_bits = W.projection_rows(5, 0, L, hidden)
    w_bits = W.query_weight(5, 0, Hq * d, hidden)
    q0 = np.zeros((layers, 1, Hq, N, d), dtype=np.uint16)
    prob = H.Problem(q0, k_bits, k_bits, Hkv, None, "thd")
    tok = torch.empty((1, N), dtype=torch.int32, device="cuda")
    pos = torch.empty((1, N), dtype=torch.int32, device="cuda")
    H.D.dapq_pseudo_tokens(prob.shape, m, n, tok, pos)
    desc = H.D.Qproj(n_layers=1, rows=N, hidden=hidden, n_q_heads=Hq, head_dim=d, total_tokens=L, x_stride_layer=0,
                     x_stride_token=hidden, w_stride_layer=0, w_stride_row=hidden, q_stride_layer=Hq * N * d,
                     q_stride_head=N * d, q_stride_row=d)
    ws = torch.empty(max(H.D.pseudo_queries_workspace_bytes(desc), 16), dtype=torch.uint8, device="cuda")
    H.D.dapq_pseudo_queries(desc, H.dev_bf16(x_bits), tok, H.dev_bf16(w_bits), pos, 500000.0, 0, prob.q, ws)
    S = prob.score().cpu().numpy().astype(np.float64)
    src, want_pos = O.pseudo_tokens(L, m, n)
    q_want = O.pseudo_queries(x_bits, src, w_bits, Hq, positions=want_pos)           # [Hq, N, d]
    assert (H.host_bits(prob.q)[0, 0] == q_want).mean() > 0.98
    S_want = O.score(q_want[None, None], k_bits, Hkv)
    assert np.isfinite(S).all()
    assert (np.abs(S - S_want) <= 5e-3 * np.abs(S_want)).all()


# 96 MB of weights, which one sweep of up to 64 rows reads; waves of two and of four feature tiles, of one and of two row blocks
@pytest.mark.parametrize("layers,hidden,rows", [(11, 4096, 64), (12, 4096, 64), (12, 4096, 20), (12, 4096, 65), (96, 512, 64), (96, 512, 20)])
def test_weights_that_stream(H, layers, hidden, rows):
    announce(f"streamed weights: {layers} layers, hidden {hidden}, {rows} rows")
    rng = np.random.default_rng(layers + rows)
    tok = rng.integers(0, 70, rows)
    got, x, w = run_case(H, layers, layers, 70, hidden, 8, 128, tok)
    assert check_projection(got, x, w, tok, 8, hidden) > 0.98
