"""The calls that go through the extension module: each reaches its own function of the library with its arguments in order.  On the host: every
call is refused by the library's argument checks, whose message names the argument, before anything touches a GPU."""
import ctypes as C
import os
import subprocess
import sys
import sysconfig

import pytest
import torch

import paper_2603_11564_amd as D

T = torch.empty(64, dtype=torch.uint8)  # (never dereferenced: the calls fail before)
N = None


def shape(**kw):
    a = dict(n_layers=1, batch=1, n_q_heads=8, n_kv_heads=8, n_pseudo=4, total_tokens=64, k_strides=(8192, 0, 0, 128),
             v_strides=(8192, 0, 0, 128), q_strides=(4096, 4096, 512, 128), scale=0.1)
    a.update(kw)
    return D.make_shape(**a)


def desc():
    return D.Qproj(n_layers=1, rows=4, hidden=64, n_q_heads=1, head_dim=8, total_tokens=4, x_stride_token=64, w_stride_row=64,
                   q_stride_head=32, q_stride_row=8)


@pytest.mark.parametrize("call,message", [
    (lambda: D.dapq_rope_apply(T, T, N, 4, 1, 128, 128, 512, 5e5, 0, 0), "pos must not be NULL"),
    (lambda: D.dapq_rope_apply(T, T, T, 4, 1, 126 + 1, 128, 512, 5e5, 0, 0), r"head_dim \(127\)"),
    (lambda: D.dapq_rope_apply(T, T, T, 4, 1, 128, 128, 512, -1.0, 0, 0), "theta must be"),
    (lambda: D.dapq_rope_apply(T, T, T, 4, 1, 128, 128, 64, 5e5, 0, 0), r"stride_head \(64\)"),
    (lambda: D.dapq_rope_apply(T, T, T, 4, 1, 128, -5, 512, 5e5, 0, 0), r"stride_row \(-5\)"),
    (lambda: D.dapq_rope_apply(T, T, T, 4, 1, 128, 128, 512, 5e5, 2, 0), "pairing must be"),
    (lambda: D.dapq_score(shape(), T, T, N, T, 0), "scores is NULL"),
    (lambda: D.dapq_score(shape(total_tokens=4096), T, T, T, N, 0), "workspace is NULL"),
    (lambda: D.dapq_score_static(shape(scale=-1.0), T, T, T, 0), "scale must be"),
    (lambda: D.dapq_score_stats(shape(), T, T, N, T, 0), "lse2 is NULL"),
    (lambda: D.dapq_score_accumulate(shape(), T, T, T, N, T, 0), "scores is NULL"),
    (lambda: D.dapq_score_accumulate(shape(), T, T, T, T, N, 0), "workspace is NULL"),
    (lambda: D.dapq_score_stats_extend(shape(), T, T, (0, 0, 0, 64), T, 0), r"kp_stride_row \(64\)"),
    (lambda: D.dapq_score_stats_extend(shape(), T, T, (0, 0, 0, 128), N, 0), "lse2 is NULL"),
    (lambda: D.dapq_pool(shape(), T, T.clone(), 6, 0), r"\(6\)"),
    (lambda: D.dapq_pool(shape(), T, T, 7, 0), "pooled must not alias"),
    (lambda: D.dapq_topk(shape(), T, -3, N, T, T, N, 0), r"budget \(-3\)"),
    (lambda: D.dapq_topk(shape(), T, 8, N, T, N, N, 0), "count must not be NULL"),
    (lambda: D.dapq_pool_topk(shape(), T, 4, 8, N, T, T, N, 0, N), r"width \(4\)"),
    (lambda: D.dapq_pool_topk(shape(), T, 3, 8, N, T, T, T, 0, N), "pooled must not alias"),
    (lambda: D.dapq_gather(shape(), T, T, T, T, -8, T, T, 0), r"budget \(-8\)"),
    (lambda: D.dapq_gather(shape(), T, T, T, T, 8, T, N, 0), "v_out must not be NULL"),
    (lambda: D.dapq_recall(shape(), T, T, 8, T, T, 8, N, N, 0), "NULL"),
    (lambda: D.dapq_decode_attention(shape(), T, T, T, T, 9000, T, 0), r"budget \(9000\)"),
    (lambda: D.dapq_pseudo_tokens(shape(), 1, 2, T, T, 0), r"first_m \(1\) \+ last_n \(2\)"),
    (lambda: D.dapq_pseudo_queries(desc(), T, T, T, T, -1.0, 0, T, N, 0), "finite theta"),
    (lambda: D.dapq_pseudo_queries(desc(), T, T, T, T, 5e5, 3, T, N, 0), "pairing 0 or 1"),
    (lambda: D.dapq_pseudo_queries(desc(), T, N, T, T, 5e5, 0, T, N, 0), "token_idx"),
])
def test_calls_reach_the_library(call, message):
    with pytest.raises(D.DapqError, match=message):
        call()


def test_arguments_of_the_wrong_kind_are_refused():
    for bad, error in ((lambda: D.dapq_gather(shape(), 4096, T, T, T, 8, T, T, 0), AttributeError),
                       (lambda: D.dapq_gather(shape(), T, T, T, T, 8.0, T, T, 0), TypeError),
                       (lambda: D.dapq_gather(desc(), T, T, T, T, 8, T, T, 0), TypeError),
                       (lambda: D.dapq_gather(bytearray(C.sizeof(D.Shape)), T, T, T, T, 8, T, T, 0), TypeError),
                       (lambda: D.dapq_gather(shape(), T, T, T, T, 8, T, T, "stream"), AttributeError),
                       (lambda: D.dapq_pseudo_queries(shape(), T, T, T, T, 5e5, 0, T, N, 0), TypeError)):
        with pytest.raises(error):
            bad()
    assert C.sizeof(D.Shape) != C.sizeof(D.Qproj)


def test_numbers_of_other_kinds_are_converted():
    for theta, pairing in (("-1", 0.0), (torch.tensor(-1.0), "0"), (-1, True)):
        with pytest.raises(D.DapqError, match="finite theta"):
            D.dapq_pseudo_queries(desc(), T, T, T, T, theta, pairing, T, N, 0)


class Larger(D.Shape):
    _fields_ = [("tag", C.c_int64)]


class Thing:
    def __init__(self, **kw):
        self.__dict__.update(kw)


def larger():
    s = Larger()
    C.memmove(C.byref(s), C.byref(shape()), C.sizeof(D.Shape))
    return s


@pytest.mark.parametrize("call,message", [
    (lambda: D.dapq_gather(shape(), T, T, T, T, C.c_int32(-8), T, T, 0), r"budget \(-8\)"),
    (lambda: D.dapq_gather(shape(), T, T, T, T, Thing(_as_parameter_=-8), T, T, 0), r"budget \(-8\)"),
    (lambda: D.dapq_gather(larger(), T, T, T, T, -8, T, T, 0), r"budget \(-8\)"),
    (lambda: D.dapq_gather(shape(), T, T, T, T, -8, T, T, Thing(cuda_stream=None)), r"budget \(-8\)"),
    (lambda: D.dapq_gather(shape(), T, T, T, T, -8, T, T, Thing(cuda_stream=C.c_void_p(0))), r"budget \(-8\)"),
    (lambda: D.dapq_gather(shape(), T, T, T, T, 8, T, Thing(data_ptr=lambda: None), 0), "v_out must not be NULL"),
    (lambda: D.dapq_score(larger(), Thing(data_ptr=lambda: C.c_void_p(4096)), T, N, T, 0), "scores is NULL"),
    (lambda: D.dapq_score_accumulate(larger(), T, T, T, T, N, 0), "workspace is NULL"),
    (lambda: D.dapq_score_stats_extend(shape(), T, T, (0, 0, 0, C.c_int64(64)), T, 0), r"kp_stride_row \(64\)"),
    (lambda: D.dapq_pool_topk(larger(), T, 4, 8, N, T, T, N, 0, N), r"width \(4\)"),
    (lambda: D.dapq_rope_apply(T, T, T, 4, 1, 128, C.c_int64(-5), 512, 5e5, 0, 0), r"stride_row \(-5\)"),
    (lambda: D.dapq_pseudo_queries(desc(), T, T, T, T, -1.0, 0, T, Thing(data_ptr=lambda: C.c_void_p(0), numel=lambda: 4, element_size=lambda: 1), 0),
     "finite theta"),
])
def test_arguments_that_ctypes_converts(call, message):
    """Numbers and addresses as ctypes objects, descriptors with fields of the caller's, handles of None: each reaches the library."""
    with pytest.raises(D.DapqError, match=message):
        call()


def test_arguments_that_ctypes_refuses():
    for bad in (lambda: D.dapq_gather(shape(), T, T, T, T, 8.0, T, T, 0), lambda: D.dapq_gather(shape(), T, T, T, T, C.c_int64(8), T, T, 0),
                lambda: D.dapq_gather(desc(), T, T, T, T, 8, T, T, 0), lambda: D.dapq_score(C.pointer(shape()), T, T, T, T, 0)):
        with pytest.raises(C.ArgumentError):
            bad()


def test_extension_module_belongs_to_this_python():
    """Its file name carries the interpreter's binary interface, and nothing lies beside it that another interpreter would load instead;
    where there is none the library does not load."""
    D.load_library()
    path = sys.modules["paper_2603_11564_amd._native"].__file__
    suffix = sysconfig.get_config_var("EXT_SUFFIX")
    assert suffix != ".so" and os.path.basename(path) == "_native" + suffix
    assert not os.path.exists(os.path.join(os.path.dirname(path), "_native.so"))
    r = subprocess.run([sys.executable, "-c", "import sys; sys.modules['paper_2603_11564_amd._native'] = None\n"
                                              "import paper_2603_11564_amd as D; D.load_library()"],
                       capture_output=True, text=True, cwd=os.path.dirname(os.path.dirname(path)))
    assert r.returncode == 1 and "is not built for this Python" in r.stderr


@pytest.mark.parametrize("cxx", ["env g++", "", None])
def test_extension_module_builds_with_any_compiler_command(cxx, tmp_path, monkeypatch):
    """With arguments in CXX, without CXX, and (None) where there is no g++."""
    from paper_2603_11564_amd import build
    target = str(tmp_path / "module.so")
    monkeypatch.setattr(build, "NATIVE_LIB", target)
    monkeypatch.setenv("CXX", cxx or "")
    if cxx is None:
        which = build.shutil.which
        monkeypatch.setattr(build.shutil, "which", lambda name, **kw: None if name == "g++" else which(name, **kw))
    assert build.build_native() == target and os.path.getsize(target) > 0
