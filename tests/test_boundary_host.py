"""The C-ABI boundary without a GPU: the library loads, exports what include/dapq.h declares,
and rejects bad arguments on the host before anything is enqueued."""
import ctypes as C
import os
import random
import re

import pytest

import paper_2603_11564_amd as D
from paper_2603_11564_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ERR_INVALID, ERR_UNSUPPORTED, ERR_WORKSPACE, ERR_HIP = -1, -2, -3, -4


@pytest.fixture(scope="module")
def lib():
    return D.load_library()


def good_shape(**kw):
    args = dict(n_layers=2, batch=1, n_q_heads=32, n_kv_heads=8, n_pseudo=64, total_tokens=4096,
                k_strides=(4096 * 8 * 128, 0, 128, 8 * 128), v_strides=(4096 * 8 * 128, 0, 128, 8 * 128),
                q_strides=(32 * 64 * 128, 32 * 64 * 128, 64 * 128, 128), scale=128 ** -0.5)
    args.update(kw)
    return D.make_shape(**args)


def test_header_and_library_agree(lib):
    header = open(os.path.join(ROOT, "include", "dapq.h")).read()
    declared = set(re.findall(r"\b(dapq_[a-z0-9_]+)\s*\(", header))
    assert declared == set(binding.EXPORTS)
    for name in declared:
        assert hasattr(lib, name), name
    # the struct mirror has the layout the header describes (6 int32, int64, pointer, 12 int64, float)
    assert C.sizeof(binding.Shape) == 6 * 4 + 8 + 8 + 12 * 8 + 8


def test_workspace_bytes_is_a_function_of_the_shape(lib):
    a = D.workspace_bytes(good_shape())
    assert a > 0 and a % 256 == 0 and a == D.workspace_bytes(good_shape())
    assert D.workspace_bytes(good_shape(n_layers=4)) > a
    assert D.workspace_bytes(good_shape(head_dim=64)) == 0
    assert b"head_dim" in lib.dapq_last_error()
    assert D.workspace_bytes(good_shape(n_q_heads=30)) == 0


def test_workspace_bytes_over_a_sweep_of_shapes(lib):
    """The launch plan (chunking, workspace carving) is pure host arithmetic: walk it over small, huge, ragged and
    degenerate shapes.  Under the host sanitizers (tests/test_host_sanitizers.py) this is where an overflow or an
    out-of-range shift in that arithmetic would show."""
    seen = 0
    for layers in (1, 32, 80, 8191):
        for tokens in (0, 1, 31, 4096, 131072, 2 ** 31 - 8):
            for n_pseudo in (1, 64, 512, 32768):
                for batch, ragged in ((1, False), (8, False), (8, True), (65535, True)):
                    if not ragged and tokens % batch:
                        continue
                    s = good_shape(n_layers=layers, batch=batch, n_pseudo=n_pseudo, total_tokens=tokens,
                                   cu_seqlens=None)
                    if ragged:
                        s.cu_seqlens = FAKE          # never dereferenced by the plan
                    b = D.workspace_bytes(s)
                    assert b % 256 == 0
                    if layers * 8 <= 65535:
                        assert b > 0, (layers, tokens, n_pseudo, batch, ragged, lib.dapq_last_error())
                    seen += 1
    assert seen > 300


def test_topk_workspace_bytes(lib):
    """The optional workspace of the selection calls: nothing unless a head can be longer than 32768 keys; then two
    candidate lists of heads x pieces x budget 4-byte entries and a count per piece (pieces of 32768 keys)."""
    def align(n):
        return (n + 255) // 256 * 256
    assert D.topk_workspace_bytes(good_shape(), 983) == 0                                   # 4096 keys per head
    assert D.topk_workspace_bytes(good_shape(total_tokens=32768), 983) == 0                 # one piece: one workgroup
    assert D.topk_workspace_bytes(good_shape(total_tokens=65536), 983) == 2 * align(16 * 2 * 983 * 4) + align(16 * 2 * 4)
    long_heads = good_shape(n_layers=3, total_tokens=131072)                                # 3 x 1 x 8 heads, 4 pieces
    assert D.topk_workspace_bytes(long_heads, 3932) == 2 * align(24 * 4 * 3932 * 4) + align(24 * 4 * 4)
    assert D.topk_workspace_bytes(good_shape(total_tokens=65537), 5) == 2 * align(16 * 3 * 5 * 4) + align(16 * 3 * 4)
    assert D.topk_workspace_bytes(long_heads, 20000) == 0          # 4 x 20000 candidates are more than a merge holds
    assert D.topk_workspace_bytes(long_heads, 0) == 0
    ragged = good_shape(batch=8, total_tokens=78821)
    ragged.cu_seqlens = FAKE                                                                # never dereferenced here
    assert D.topk_workspace_bytes(ragged, 512) == 2 * align(2 * 8 * 8 * 3 * 512 * 4) + align(2 * 8 * 8 * 3 * 4)


def test_score_single_launch_follows_the_launch_plan(lib):
    """dapq_score runs both passes in one kernel exactly when a (layer, sequence, KV head) is one workgroup: a dense
    batch, at most 256 query rows per KV head, at most 4 key chunks per sequence."""
    assert D.score_single_launch(good_shape(n_layers=32, total_tokens=32768))                # the 8B shape: 4 chunks of 8192
    assert D.score_single_launch(good_shape(n_layers=32, total_tokens=32768, n_pseudo=32))
    assert D.score_single_launch(good_shape(n_layers=1, total_tokens=512))                   # 4 chunks of 128
    assert D.score_single_launch(good_shape(n_layers=1, total_tokens=100))                   # one chunk
    assert D.score_single_launch(good_shape(n_layers=1, batch=3, total_tokens=1200))         # 4 chunks for each of 3
    assert not D.score_single_launch(good_shape(n_layers=1, total_tokens=1024))              # 8 chunks of 128
    assert D.score_single_launch(good_shape(n_layers=1, total_tokens=300))                   # 3 chunks: three waves
    assert not D.score_single_launch(good_shape(n_layers=1, total_tokens=600))               # 5 chunks
    assert not D.score_single_launch(good_shape(n_layers=32, total_tokens=32768, n_pseudo=128))   # two row groups
    ragged = good_shape(batch=4, total_tokens=400)
    ragged.cu_seqlens = FAKE                                                                 # never dereferenced here
    assert not D.score_single_launch(ragged)
    with pytest.raises(D.DapqError):
        D.score_single_launch(good_shape(n_q_heads=30))


def test_few_chunks_of_a_sequence_stay_in_one_kernel(lib):
    """Where one to four chunks of a sequence leave some of the chip idle in the only round, or a last round nearly empty, one kernel with
    one start-up is still faster than three launches with fuller rounds: five prompts of 2265 keys, 16 layers, 256 rows 245 us in four
    chunks each, 277 in five and 281 in six; five of 2316, 8 layers, 128 rows 72 us in two and 94 in six."""
    def five(layers, keys, group, n):
        return good_shape(n_layers=layers, batch=5, n_q_heads=8 * group, n_pseudo=n, total_tokens=5 * keys,
                          k_strides=(5 * keys * 8 * 128, 0, 128, 8 * 128),
                          q_strides=(5 * 8 * group * n * 128, 8 * group * n * 128, n * 128, 128))
    for layers, keys, group, n in ((16, 2265, 8, 32), (16, 2811, 4, 64), (8, 2316, 4, 32), (8, 696, 4, 32), (8, 1906, 1, 16)):
        assert D.score_single_launch(five(layers, keys, group, n)), (layers, keys, group, n)
    # long prompts fill their rounds (465 us in six chunks, 556 in two); the tiles of small calls stay tiles
    assert not D.score_single_launch(five(8, 10983, 4, 37))
    assert not D.score_single_launch(good_shape(n_layers=1, total_tokens=640))


FAKE = 0x1000  # never dereferenced: every call below must fail validation first


def call(lib, fn, *args):
    return getattr(lib, fn)(*args)


def test_invalid_arguments_are_rejected_on_the_host(lib):
    s = good_shape()
    ws = D.workspace_bytes(s)
    sp = C.byref(s)
    assert lib.dapq_score(sp, None, FAKE, FAKE, FAKE, ws, None) == ERR_INVALID
    assert b"q is NULL" in lib.dapq_last_error()
    assert lib.dapq_score(sp, FAKE, FAKE, FAKE, FAKE, ws - 1, None) == ERR_WORKSPACE
    assert lib.dapq_score(sp, FAKE + 2, FAKE, FAKE, FAKE, ws, None) == ERR_UNSUPPORTED      # misaligned q
    assert lib.dapq_score(None, FAKE, FAKE, FAKE, FAKE, ws, None) == ERR_INVALID
    bad = good_shape(n_q_heads=30)
    assert lib.dapq_score(C.byref(bad), FAKE, FAKE, FAKE, FAKE, 1 << 30, None) == ERR_INVALID
    bad = good_shape(head_dim=64)
    assert lib.dapq_score(C.byref(bad), FAKE, FAKE, FAKE, FAKE, 1 << 30, None) == ERR_UNSUPPORTED
    bad = good_shape(k_strides=(4096 * 8 * 128, 0, 132, 8 * 128))
    assert lib.dapq_score(C.byref(bad), FAKE, FAKE, FAKE, FAKE, 1 << 30, None) == ERR_UNSUPPORTED
    bad = good_shape(scale=0.0)
    assert lib.dapq_score_stats(C.byref(bad), FAKE, FAKE, FAKE, FAKE, 1 << 30, None) == ERR_INVALID
    bad = good_shape(n_pseudo=0)
    assert lib.dapq_score_accumulate(C.byref(bad), FAKE, FAKE, FAKE, FAKE, FAKE, 1 << 30, None) == ERR_INVALID
    bad = good_shape(batch=3, total_tokens=4096)                     # dense batch must divide evenly
    assert lib.dapq_pool(C.byref(bad), FAKE, FAKE + 64, 7, None) == ERR_INVALID

    assert lib.dapq_pool(sp, FAKE, FAKE + 64, 4, None) == ERR_INVALID          # even width
    assert lib.dapq_pool(sp, FAKE, FAKE + 64, 65, None) == ERR_INVALID
    assert lib.dapq_pool(sp, FAKE, FAKE, 7, None) == ERR_INVALID               # aliasing
    assert lib.dapq_pool(sp, None, FAKE, 7, None) == ERR_INVALID
    assert lib.dapq_topk(sp, FAKE, 0, None, FAKE, FAKE, None, 0, None) == ERR_INVALID
    assert lib.dapq_topk(sp, FAKE, 8, None, None, FAKE, None, 0, None) == ERR_INVALID
    assert lib.dapq_gather(sp, FAKE, FAKE, FAKE, FAKE, 0, FAKE, FAKE, None) == ERR_INVALID
    assert lib.dapq_gather(sp, FAKE, FAKE + 2, FAKE, FAKE, 8, FAKE, FAKE, None) == ERR_UNSUPPORTED
    assert lib.dapq_gather(sp, FAKE, None, FAKE, FAKE, 8, FAKE, FAKE, None) == ERR_INVALID

    assert lib.dapq_rope_apply(None, FAKE, FAKE, 4, 2, 128, 256, 128, 5e5, 0, None) == ERR_INVALID
    assert lib.dapq_rope_apply(FAKE, FAKE, FAKE, 4, 2, 127, 256, 128, 5e5, 0, None) == ERR_INVALID
    assert lib.dapq_rope_apply(FAKE, FAKE, FAKE, 4, 2, 128, 256, 128, 5e5, 2, None) == ERR_INVALID
    assert lib.dapq_rope_apply(FAKE, FAKE, FAKE, 4, 2, 128, 256, 128, -1.0, 0, None) == ERR_INVALID
    assert lib.dapq_rope_apply(FAKE, FAKE, FAKE, 4, 2, 128, 256, 64, 5e5, 0, None) == ERR_INVALID
    assert lib.dapq_rope_apply(FAKE, FAKE, FAKE, 0, 2, 128, 256, 128, 5e5, 0, None) == 0       # nothing to do


def test_invalid_arguments_of_the_entry_points_around_the_step(lib):
    s = good_shape()
    sp = C.byref(s)
    i64 = C.c_int64
    # extended normaliser
    kp = (i64(8 * 64 * 128), i64(8 * 64 * 128), i64(64 * 128), i64(128))
    assert lib.dapq_score_stats_extend(sp, FAKE, None, *kp, FAKE, None) == ERR_INVALID
    assert lib.dapq_score_stats_extend(sp, FAKE, FAKE, *kp, None, None) == ERR_INVALID
    assert lib.dapq_score_stats_extend(sp, FAKE, FAKE + 4, *kp, FAKE, None) == ERR_UNSUPPORTED          # misaligned keys
    assert lib.dapq_score_stats_extend(sp, FAKE, FAKE, kp[0], kp[1], kp[2], i64(64), FAKE, None) == ERR_INVALID   # row < d
    assert lib.dapq_score_stats_extend(sp, FAKE, FAKE, kp[0], kp[1], i64(132), kp[3], FAKE, None) == ERR_UNSUPPORTED
    # pooling + selection in one call
    assert lib.dapq_pool_topk(sp, FAKE, 4, 8, None, FAKE, FAKE, None, None, 0, None) == ERR_INVALID             # even width
    assert lib.dapq_pool_topk(sp, FAKE, 7, 0, None, FAKE, FAKE, None, None, 0, None) == ERR_INVALID             # budget
    assert lib.dapq_pool_topk(sp, FAKE, 7, 8, None, FAKE, FAKE, FAKE, None, 0, None) == ERR_INVALID             # pooled aliases scores
    assert lib.dapq_pool_topk(sp, FAKE, 11, 8, None, FAKE, FAKE, None, None, 0, None) == ERR_UNSUPPORTED        # needs the buffer
    assert b"pooled" in lib.dapq_last_error()
    long_heads = good_shape(total_tokens=70000, k_strides=(70000 * 8 * 128, 0, 128, 8 * 128),
                            v_strides=(70000 * 8 * 128, 0, 128, 8 * 128))
    assert lib.dapq_pool_topk(C.byref(long_heads), FAKE, 7, 8, None, FAKE, FAKE, None, None, 0, None) == ERR_UNSUPPORTED
    # recall
    assert lib.dapq_recall(sp, FAKE, FAKE, 8, FAKE, FAKE, 8, None, None, None) == ERR_INVALID
    assert lib.dapq_recall(sp, FAKE, FAKE, 0, FAKE, FAKE, 8, FAKE, None, None) == ERR_INVALID
    assert lib.dapq_recall(sp, None, FAKE, 8, FAKE, FAKE, 8, FAKE, None, None) == ERR_INVALID
    # decode step over the compact cache
    assert lib.dapq_decode_attention(sp, FAKE, FAKE, FAKE, FAKE, 8193, FAKE, None) == ERR_UNSUPPORTED
    assert lib.dapq_decode_attention(sp, FAKE, FAKE, FAKE, FAKE, 0, FAKE, None) == ERR_UNSUPPORTED
    assert lib.dapq_decode_attention(sp, FAKE, FAKE + 8, FAKE, FAKE, 64, FAKE, None) == ERR_UNSUPPORTED  # misaligned cache
    assert lib.dapq_decode_attention(sp, FAKE, FAKE, FAKE, None, 64, FAKE, None) == ERR_INVALID
    bad = good_shape(scale=float("nan"))
    assert lib.dapq_decode_attention(C.byref(bad), FAKE, FAKE, FAKE, FAKE, 64, FAKE, None) == ERR_INVALID


def test_invalid_arguments_of_the_pseudo_query_projection(lib):
    def desc(**kw):
        f = dict(n_layers=2, rows=64, hidden=4096, n_q_heads=32, head_dim=128, total_tokens=1000, x_stride_layer=1000 * 4096,
                 x_stride_token=4096, w_stride_layer=4096 * 4096, w_stride_row=4096, q_stride_layer=32 * 64 * 128,
                 q_stride_head=64 * 128, q_stride_row=128)
        f.update(kw)
        return C.byref(D.Qproj(**f))
    call = lib.dapq_pseudo_queries
    dbl = C.c_double
    assert call(None, FAKE, FAKE, FAKE, None, dbl(5e5), 0, FAKE, None, 0, None) == ERR_INVALID
    assert call(desc(), None, FAKE, FAKE, None, dbl(5e5), 0, FAKE, None, 0, None) == ERR_INVALID
    assert call(desc(), FAKE, None, FAKE, None, dbl(5e5), 0, FAKE, None, 0, None) == ERR_INVALID
    assert call(desc(), FAKE, FAKE, FAKE, None, dbl(5e5), 0, None, None, 0, None) == ERR_INVALID
    assert call(desc(n_layers=0), FAKE, FAKE, FAKE, None, dbl(5e5), 0, FAKE, None, 0, None) == ERR_INVALID
    assert call(desc(rows=-1), FAKE, FAKE, FAKE, None, dbl(5e5), 0, FAKE, None, 0, None) == ERR_INVALID
    assert call(desc(hidden=4000), FAKE, FAKE, FAKE, None, dbl(5e5), 0, FAKE, None, 0, None) == ERR_UNSUPPORTED     # not a multiple of 64
    assert b"hidden" in lib.dapq_last_error()
    assert call(desc(head_dim=12, q_stride_row=16, q_stride_head=1024), FAKE, FAKE, FAKE, None, dbl(5e5), 0, FAKE, None, 0, None) == ERR_UNSUPPORTED
    assert call(desc(x_stride_token=2048), FAKE, FAKE, FAKE, None, dbl(5e5), 0, FAKE, None, 0, None) == ERR_INVALID  # rows overlap
    assert call(desc(w_stride_row=4100), FAKE, FAKE, FAKE, None, dbl(5e5), 0, FAKE, None, 0, None) == ERR_UNSUPPORTED  # not 16-byte rows
    assert call(desc(q_stride_row=64), FAKE, FAKE, FAKE, None, dbl(5e5), 0, FAKE, None, 0, None) == ERR_INVALID
    assert call(desc(), FAKE + 2, FAKE, FAKE, None, dbl(5e5), 0, FAKE, None, 0, None) == ERR_UNSUPPORTED             # misaligned x
    assert call(desc(total_tokens=1 << 20), FAKE, FAKE, FAKE, None, dbl(5e5), 0, FAKE, None, 0, None) == ERR_UNSUPPORTED  # 8 GiB layer
    assert b"4 GiB" in lib.dapq_last_error()
    # a single layer is split along the hidden axis and needs the workspace; all 32 layers at once do not
    one = dict(n_layers=1)
    need = D.pseudo_queries_workspace_bytes(D.Qproj(**{**dict(n_layers=1, rows=64, hidden=4096, n_q_heads=32, head_dim=128,
                                                              total_tokens=1000, x_stride_layer=0, x_stride_token=4096,
                                                              w_stride_layer=0, w_stride_row=4096, q_stride_layer=0,
                                                              q_stride_head=64 * 128, q_stride_row=128)}))
    assert need == 8 * 64 * 4096 * 4                      # eight hidden splits of fp32 sums
    assert call(desc(**one), FAKE, FAKE, FAKE, None, dbl(5e5), 0, FAKE, None, 0, None) == ERR_WORKSPACE
    assert call(desc(**one), FAKE, FAKE, FAKE, None, dbl(5e5), 0, FAKE, FAKE, need - 1, None) == ERR_WORKSPACE
    assert D.pseudo_queries_workspace_bytes(D.Qproj(n_layers=32, rows=64, hidden=4096, n_q_heads=32, head_dim=128,
                                                    total_tokens=1000, x_stride_layer=0, x_stride_token=4096,
                                                    w_stride_layer=0, w_stride_row=4096, q_stride_layer=0,
                                                    q_stride_head=64 * 128, q_stride_row=128)) == 0
    assert D.pseudo_queries_workspace_bytes(D.Qproj(n_layers=1, rows=64, hidden=100)) == 0   # invalid: the call says why
    assert call(desc(), FAKE, FAKE, FAKE, FAKE, dbl(0.0), 0, FAKE, None, 0, None) == ERR_INVALID                       # theta
    assert call(desc(), FAKE, FAKE, FAKE, FAKE, dbl(5e5), 2, FAKE, None, 0, None) == ERR_INVALID                       # pairing


def test_score_plan_covers_every_shape(lib):
    """The launch plan is a pure function of the shape; its workspace figure pins the split it chose."""
    def ws(**kw):
        return D.workspace_bytes(good_shape(**kw))
    lse = 2 * 1 * 32 * 64 * 4
    # 2 layers x 8 KV heads x 4096 keys, 256 rows: 128-key chunks -> 32 chunks per head, (ref, sum) per row and chunk;
    # in front of them the chunk prefix of the sequences, 256 bytes, and 256 that nothing uses
    assert ws() == 256 + 256 + 2 * 8 * 32 * 256 * 8 + lse
    # 512 rows per KV head: two row groups; one extra plane of column sums
    big = dict(n_pseudo=128, q_strides=(32 * 128 * 128, 32 * 128 * 128, 128 * 128, 128))
    lse2 = 2 * 1 * 32 * 128 * 4
    assert ws(**big) == 256 + 256 + 2 * 8 * 32 * 512 * 8 + lse2 + 2 * 8 * 4096 * 4
    # very many rows are still planned (row groups on the grid), absurdly many are refused
    assert ws(n_pseudo=4096, q_strides=(32 * 4096 * 128, 32 * 4096 * 128, 4096 * 128, 128)) > 0
    assert ws(n_pseudo=1 << 19) == 0 and b"rows per KV head" in lib.dapq_last_error()


def test_many_heads_of_few_rows_are_not_refused(lib):
    """dapq_rope_apply takes up to 65535 runs of 8 heads, however few rows there are: the call gets as far as its launch, which
    reports that there is no GPU here."""
    if os.path.exists("/dev/kfd"):
        pytest.skip("would be launched, with pointers that are none")
    for rows, heads, d in ((1, 65536, 64), (1, 100000, 64), (1, 65535 * 8, 8), (3, 65535 * 8, 128)):
        assert lib.dapq_rope_apply(FAKE, FAKE, FAKE, rows, heads, d, heads * d, d, 5e5, 0, None) == ERR_HIP, lib.dapq_last_error()


def test_a_workspace_sized_for_a_longer_batch_serves_shorter_ones(lib):
    """Small ragged batches like more workspace than larger ones, and run without it: the call gets as far as its launch, which
    reports that there is no GPU here."""
    if os.path.exists("/dev/kfd"):
        pytest.skip("would be launched, with pointers that are none")

    def ragged(tokens):
        s = good_shape(n_layers=4, batch=8, n_pseudo=32, total_tokens=tokens, k_strides=(tokens * 8 * 128, 0, 128, 8 * 128),
                       q_strides=(8 * 32 * 32 * 128, 32 * 32 * 128, 32 * 128, 128))
        s.cu_seqlens = FAKE                                                                  # never dereferenced here
        return s
    # (the first three: what these batches asked for when every shape ran in the kernels for larger ones)
    for tokens, enough in ((16384, 1442304), (20000, 1704448), (25000, 1999360), (29696, D.workspace_bytes(ragged(32768)))):
        sp = C.byref(ragged(tokens))
        assert enough < D.workspace_bytes(ragged(tokens))
        assert lib.dapq_score(sp, FAKE, FAKE, FAKE, FAKE, enough, None) == ERR_HIP, lib.dapq_last_error()
        assert lib.dapq_score_stats(sp, FAKE, FAKE, FAKE, FAKE, enough, None) == ERR_HIP, lib.dapq_last_error()
        assert lib.dapq_score_accumulate(sp, FAKE, FAKE, FAKE, FAKE, FAKE, enough, None) == ERR_HIP, lib.dapq_last_error()
        assert lib.dapq_score(sp, FAKE, FAKE, FAKE, FAKE, 1 << 18, None) == ERR_WORKSPACE


def test_a_workspace_sized_for_a_larger_shape_serves_smaller_ones(lib):
    """Fewer layers, sequences, heads, rows or keys can make a plan of more partial sums: in the workspace of the larger shape such a call
    makes do with fewer chunks (dense) or segments (ragged).  It gets as far as its launch, which reports that there is no GPU here."""
    if os.path.exists("/dev/kfd"):
        pytest.skip("would be launched, with pointers that are none")

    def shape(layers, batch, kv_heads, group, n, keys, ragged):  # keys: of a sequence, of a ragged batch all
        tokens = keys if ragged else keys * batch
        s = D.make_shape(n_layers=layers, batch=batch, n_q_heads=kv_heads * group, n_kv_heads=kv_heads, n_pseudo=n, total_tokens=tokens,
                         k_strides=(tokens * kv_heads * 128, 0, 128, kv_heads * 128),
                         q_strides=(batch * kv_heads * group * n * 128, kv_heads * group * n * 128, n * 128, 128), scale=128 ** -0.5)
        s.cu_seqlens = FAKE if ragged else None                                             # never dereferenced here
        return s

    def serves(large, small, ragged):
        room, sp = D.workspace_bytes(shape(*large, ragged)), C.byref(shape(*small, ragged))
        for rc in (lib.dapq_score(sp, FAKE, FAKE, FAKE, FAKE, room, None),
                   lib.dapq_score_stats(sp, FAKE, FAKE, FAKE, FAKE, room, None),
                   lib.dapq_score_accumulate(sp, FAKE, FAKE, FAKE, FAKE, FAKE, room, None)):
            assert rc == ERR_HIP, (large, small, ragged, lib.dapq_last_error())

    serves((1, 1, 8, 4, 32, 20800), (1, 1, 8, 4, 32, 19400), False)
    serves((2, 1, 8, 4, 64, 40314), (2, 1, 8, 4, 64, 36685), False)
    serves((32, 16, 8, 4, 32, 93604), (32, 13, 8, 4, 32, 93604), False)
    serves((16, 5, 8, 4, 32, 865), (15, 5, 8, 4, 32, 865), True)
    serves((257, 1, 1, 4, 64, 384), (256, 1, 1, 4, 64, 384), False)                         # one chunk a wave, then three
    rng = random.Random(3)
    for _ in range(1500):
        ragged = rng.random() < 0.5
        large = [rng.choice((1, 2, 8, 15, 16, 32, 80)), int(2 ** rng.uniform(0, 8)), rng.choice((1, 2, 3, 4, 8)),
                 rng.choice((1, 2, 4, 5, 8)), rng.choice((7, 16, 32, 37, 64, 128, 256)), int(2 ** rng.uniform(0, 17))]
        small = list(large)
        for i in rng.sample(range(6), rng.choice((1, 1, 2, 6))):
            small[i] = max(1, int(large[i] * rng.uniform(0.3, 1.0)))
        serves(large, small, ragged)
    # a call is not made to do with anything: a workspace that fills less than half the chip with waves is one for another call
    long = shape(1, 1, 8, 4, 64, 1 << 17, False)
    assert lib.dapq_score(C.byref(long), FAKE, FAKE, FAKE, FAKE, D.workspace_bytes(long) // 3, None) == ERR_WORKSPACE


def test_binding_raises_with_the_library_message():
    with pytest.raises(D.DapqError) as e:
        D.dapq_pool(good_shape(), None, None, 7, stream=0)
    assert e.value.code == ERR_INVALID and "NULL" in str(e.value)


def test_product_path_does_not_touch_the_oracle():
    for root, _, files in os.walk(os.path.join(ROOT, "paper_2603_11564_amd")):
        for f in files:
            if f.endswith((".py", ".hip", ".h")):
                text = open(os.path.join(root, f)).read()
                assert "oracle" not in text, f
    assert "oracle" not in open(os.path.join(ROOT, "include", "dapq.h")).read()
    assert "paper_2603_11564_amd" not in open(os.path.join(ROOT, "oracle", "dapq_oracle.py")).read()


def test_header_is_plain_c_and_links_from_a_c_program(tmp_path):
    """include/dapq.h compiles as strict C99 on its own, its structs have the sizes the ctypes mirrors assume, and
    a C program linked against libdapq.so reaches every declared entry point (no compute call: nothing here needs
    a GPU)."""
    import subprocess
    header = open(os.path.join(ROOT, "include", "dapq.h")).read()
    names = sorted(set(re.findall(r"\b(dapq_[a-z0-9_]+)\s*\(", header)))
    src = tmp_path / "abi.c"
    src.write_text(
        '#include "dapq.h"\n#include <stdio.h>\n#include <string.h>\n'
        "int main(void) {\n"
        "  void (*fns[])(void) = {" + ", ".join(f"(void (*)(void)){n}" for n in names) + "};\n"
        "  size_t i, n = sizeof fns / sizeof fns[0];\n"
        "  for (i = 0; i < n; ++i) if (!fns[i]) return 1;\n"
        "  if (dapq_workspace_bytes(NULL) != 0) return 2;            /* invalid shape: 0, and a message */\n"
        "  if (strlen(dapq_last_error()) == 0) return 3;\n"
        "  if (dapq_gather(NULL, NULL, NULL, NULL, NULL, 1, NULL, NULL, NULL) != DAPQ_ERR_INVALID_ARG) return 4;\n"
        '  printf("%zu %zu %zu\\n", n, sizeof(dapq_shape), sizeof(dapq_qproj));\n'
        "  return 0;\n}\n")
    exe = tmp_path / "abi"
    libdir = os.path.dirname(binding.lib_path())
    subprocess.run(["gcc", "-std=c99", "-pedantic", "-Wall", "-Wextra", "-Werror",
                    "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe), binding.lib_path(),
                    f"-Wl,-rpath,{libdir}", "-Wl,-rpath,/opt/rocm/lib", "-Wl,--allow-shlib-undefined"],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    assert int(out[0]) == len(binding.EXPORTS)
    assert int(out[1]) == C.sizeof(binding.Shape) and int(out[2]) == C.sizeof(binding.Qproj)
