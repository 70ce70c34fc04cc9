"""The native part of the binding (csrc/lx_call.cpp), without a GPU: what reaches the C functions, recorded by functions bound in
their place, and what is refused before them.  CPU tensors serve: only their attributes are read."""
import ctypes as C
import os
import sysconfig

import pytest
import torch

NAMES = ("lx_mask_compact", "lx_mask_compact_pair", "lx_attn_combine_patterns", "lx_mlp_predict_mask", "lx_sparse_ffn_fwd",
         "lx_sparse_ffn_bwd_dx", "lx_sparse_ffn_lora_fwd", "lx_sparse_ffn_lora_bwd", "lx_sparse_attn_fwd", "lx_sparse_attn_bwd_dx",
         "lx_sparse_attn_bwd_dx_noalloc")
STREAM = 0x7A0


@pytest.fixture
def calls():
    """(module, list of (name, arguments) of the calls made, status to return)."""
    from paper_2510_15964_amd import build
    build.ensure()
    from paper_2510_15964_amd import lx
    seen, status, keep, addr = [], [0], [], {}
    for n in NAMES:
        types = getattr(lx._lib, n).argtypes
        # structures and arrays arrive as pointers
        plain = [t if t in (C.c_int, C.c_int32, C.c_int64, C.c_float, C.c_size_t) else C.c_void_p for t in types]

        def record(*args, _n=n, _t=types):
            out = []
            for v, t in zip(args, _t):
                if t is C.POINTER(lx.lx_blocklist):
                    v = None if v is None else C.cast(v, t).contents.nnz_cap
                elif t is C.POINTER(C.c_int64):
                    v = tuple(C.cast(v, t)[k] for k in range(3))
                out.append(v)
            seen.append((_n, out))
            return status[0]
        f = C.CFUNCTYPE(C.c_int, *plain)(record)
        keep.append(f)
        addr[n] = C.cast(f, C.c_void_p).value

    def bind(a, stream):
        lx._call.bind(a, lx._DTYPES, lx.LxError, stream, torch.uint8, torch.float32, torch.int32)
    bind(addr, lambda: STREAM)
    yield lx, seen, status
    bind({n: C.cast(getattr(lx._lib, n), C.c_void_p).value for n in lx.EXPORTS}, lx._stream)


def bf(*shape):
    return torch.zeros(shape, dtype=torch.bfloat16)


def header(lx, cap):
    z = torch.zeros(4, dtype=torch.int32)
    return lx.BlockList(1, 4, z, z.clone(), cap)


def p(t):
    return t.data_ptr()


def test_ffn_arguments(calls):
    lx, seen, _ = calls
    X, Wu, Wd, Y, H, bu, bd, Wut, Wdt = bf(128, 192), bf(256, 192), bf(192, 256), bf(128, 192), bf(9), bf(256), bf(192), bf(192, 256), bf(256, 192)
    ws, bl = torch.zeros(10, dtype=torch.float32), header(lx, 7)
    assert lx.lx_sparse_ffn_fwd(X, Wu, Wd, bl, 64, 32, Y, H, b_up=bu, b_down=bd, workspace=ws) is Y
    assert lx.lx_sparse_ffn_fwd(X, Wu, Wd, bl, 64, 64, Y, None) is Y
    assert lx.lx_sparse_ffn_bwd_dx(Y, H, Wu, Wd, bl, 64, 32, X, ws, W_up_t=Wut, W_down_t=Wdt) is X
    assert lx.lx_sparse_ffn_bwd_dx(Y, H, None, None, bl, 64, 32, X, None, W_up_t=Wut, W_down_t=Wdt) is X
    size = [lx.LX_BF16, 128, 192, 256, 64]
    assert seen == [
        ("lx_sparse_ffn_fwd", size + [32, p(X), p(Wu), p(bu), p(Wd), p(bd), 7, p(Y), p(H), p(ws), 40, STREAM]),
        ("lx_sparse_ffn_fwd", size + [64, p(X), p(Wu), None, p(Wd), None, 7, p(Y), None, None, 0, STREAM]),
        ("lx_sparse_ffn_bwd_dx", size + [32, p(Y), p(H), p(Wu), p(Wd), p(Wut), p(Wdt), 7, p(X), p(ws), 40, STREAM]),
        ("lx_sparse_ffn_bwd_dx", size + [32, p(Y), p(H), None, None, p(Wut), p(Wdt), 7, p(X), None, 0, STREAM])]


def test_lora_and_predictor_arguments(calls):
    lx, seen, _ = calls
    T, d, F = 64, 128, 512
    X, dY, Wu, Wd, A, B, Y, H, U, Wut, Wdt, dX = (bf(T, d).half(), bf(T, d).half(), bf(F, d), bf(d, F), bf(64, d), bf(F, 64), bf(T, d), bf(5),
                                                  bf(T, 64), bf(d, F), bf(F, d), bf(T, d))
    dA, dB, ws, bl = torch.zeros(64, d), torch.zeros(F, 64), torch.zeros(33, dtype=torch.uint8), header(lx, 3)
    lx.lx_sparse_ffn_lora_fwd(X, Wu, A, B, Wd, bl, Y, H, U, ws)
    lx.lx_sparse_ffn_lora_bwd(X, dY, H, U, Wut, Wdt, A, B, bl, dX, dA, dB, ws)
    mask, Wa = torch.zeros(1, 64, dtype=torch.uint8), bf(64, d)
    assert lx.lx_mlp_predict_mask(X, Wa, 0.5, T, mask=mask) is mask
    size = [lx.LX_F16, T, d, F, 64, 64]
    assert seen == [
        ("lx_sparse_ffn_lora_fwd", size + [p(X), p(Wu), p(A), p(B), p(Wd), 3, p(Y), p(H), p(U), p(ws), 33, STREAM]),
        ("lx_sparse_ffn_lora_bwd", size + [p(X), p(dY), p(H), p(U), p(Wut), p(Wdt), p(A), p(B), 3, p(dX), p(dA), p(dB), p(ws), 33, STREAM]),
        ("lx_mlp_predict_mask", [lx.LX_F16, T, d, 64, T, p(X), p(Wa), 0.5, p(mask), STREAM])]
    with pytest.raises(AssertionError):
        lx.lx_sparse_ffn_lora_fwd(X, Wu, bf(63, d), B, Wd, bl, Y, H, U, ws)
    with pytest.raises(AssertionError):
        lx.lx_sparse_ffn_lora_bwd(X, dY, H, U, Wut, Wdt, A, B, bl, dX, dA.half(), dB, ws)
    with pytest.raises(AssertionError):
        lx.lx_mlp_predict_mask(X, Wa[:, :64], 0.5, T, mask=mask)
    assert len(seen) == 3


def test_attention_arguments(calls):
    lx, seen, _ = calls
    B, Hh, S, D = 2, 3, 128, 64
    Q, K, V, O, dO, dQ, dK, dV = (torch.zeros(B, S, Hh, D).transpose(1, 2) for _ in range(8))
    LSE, ws, act = torch.zeros(B, Hh, S), torch.zeros(12, dtype=torch.uint8), torch.zeros(Hh, dtype=torch.uint8)
    rows, cols = header(lx, 5), header(lx, 6)
    assert lx.lx_sparse_attn_fwd(Q, K, V, rows, 0.25, True, O, LSE) == (O, LSE)
    lx.lx_sparse_attn_bwd_dx(Q, K, V, O, LSE, dO, rows, cols, 0.25, False, dQ, dK, dV, ws, mask_batch=2, head_active=act)
    lx.lx_sparse_attn_bwd_dx_noalloc(Q, K, V, O, LSE, dO, rows, cols, 0.25, True, dQ, dK, dV, head_active=act)
    size, st = [lx.LX_F32, B, Hh, S, D, 0.25], (S * Hh * D, D, Hh * D)
    tensors = [p(Q), p(K), p(V), p(O), p(LSE), p(dO), st, 5, 6]
    assert seen == [
        ("lx_sparse_attn_fwd", size + [1, p(Q), p(K), p(V), st, 5, 1, None, p(O), p(LSE), STREAM]),
        ("lx_sparse_attn_bwd_dx", size + [0] + tensors + [2, p(act), p(dQ), p(dK), p(dV), p(ws), 12, STREAM]),
        ("lx_sparse_attn_bwd_dx_noalloc", size + [1] + tensors + [1, p(act), p(dQ), p(dK), p(dV), STREAM])]
    other = torch.zeros(B, Hh, S, D)                       # other strides, other shape, last stride not one
    for bad in (other, Q[:, :, :64], Q[:1]):
        with pytest.raises(AssertionError):
            lx.lx_sparse_attn_fwd(Q, bad, V, rows, 0.25, True, O, LSE)
    with pytest.raises(AssertionError):
        lx.lx_sparse_attn_fwd(*[other.transpose(2, 3)] * 3, rows, 0.25, True, other.transpose(2, 3), LSE)
    assert len(seen) == 3


def test_pattern_and_mask_tensors_are_checked(calls):
    lx, seen, _ = calls
    out = header(lx, 4)
    with pytest.raises(AssertionError):                    # not on the GPU
        lx.lx_mask_compact(torch.zeros(2, 2, dtype=torch.uint8), out=out)
    with pytest.raises(AssertionError):
        lx.lx_mask_compact_pair(torch.zeros(2, 2, dtype=torch.uint8), out=(out, out))
    with pytest.raises(AssertionError):
        lx.lx_mask_compact(torch.zeros(2, 2), out=out)
    with pytest.raises(AssertionError):
        lx.lx_attn_combine_patterns(out, None, 1, torch.zeros(2, dtype=torch.int32), out=(out, None))
    assert seen == []


class GpuMask:
    """A tensor's attributes, of one on the GPU."""
    is_cuda, dtype = True, torch.uint8

    def __init__(self, t):
        self.t, self.shape = t, t.shape

    def __getattr__(self, name):
        return getattr(self.t, name)


def test_compaction_arguments(calls):
    lx, seen, _ = calls
    m, out, other = GpuMask(torch.zeros(2, 3, 5, 7, dtype=torch.uint8)), header(lx, 4), header(lx, 4)
    o, q = [p(out.row_ptr), p(out.col_idx)], [p(other.row_ptr), p(other.col_idx)]
    assert lx.lx_mask_compact(m, out=out) is out
    lx.lx_mask_compact(m, transpose=True, nnz_cap=9, out=out)
    assert lx.lx_mask_compact_pair(m, out=(out, other)) == (out, other)
    hp = GpuMask(torch.zeros(6, dtype=torch.int32))
    hp.dtype = torch.int32
    lx.lx_attn_combine_patterns(header(lx, 2), header(lx, 3), 1, hp, out=(out, other))
    lx.lx_attn_combine_patterns(header(lx, 2), None, 1, hp, nnz_cap=0, out=(out, None))
    assert seen == [
        ("lx_mask_compact", [p(m), 6, 5, 7, 35, 7, 1] + o + [210, STREAM]),
        ("lx_mask_compact", [p(m), 6, 7, 5, 35, 1, 7] + o + [9, STREAM]),
        ("lx_mask_compact_pair", [p(m), 6, 5, 7, 35, 7, 1] + o + q + [210, STREAM]),
        ("lx_attn_combine_patterns", [2, 3, 1, 1, p(hp), 6] + o + q + [6, STREAM]),
        ("lx_attn_combine_patterns", [2, None, 1, 1, p(hp), 6] + o + [None, None, 1, STREAM])]


def test_errors(calls):
    lx, seen, status = calls
    X, W, bl = bf(64, 64), bf(64, 64), header(lx, 1)
    status[0] = lx.LX_ERR_WORKSPACE
    with pytest.raises(lx.LxError) as e:
        lx.lx_sparse_ffn_fwd(X, W, W, bl, 64, 64, X, X)
    assert e.value.status == lx.LX_ERR_WORKSPACE and str(e.value) == "lx_sparse_ffn_fwd: LX_ERR_WORKSPACE"
    del seen[:]
    with pytest.raises(lx.LxError) as e:
        lx.lx_sparse_ffn_fwd(X.double(), W, W, bl, 64, 64, X, X)
    assert e.value.status == lx.LX_ERR_UNSUPPORTED and "torch.float64" in str(e.value)
    with pytest.raises(ValueError, match="expected 2, got 1"):
        lx.lx_sparse_ffn_fwd(X[0], W, W, bl, 64, 64, X, X)
    with pytest.raises(ValueError, match="too many values"):
        lx.lx_sparse_ffn_fwd(X[None], W, W, bl, 64, 64, X, X)
    with pytest.raises(TypeError):
        lx.lx_sparse_ffn_fwd(X, W, W, bl, 64.0, 64, X, X)
    with pytest.raises(AttributeError):
        lx.lx_sparse_ffn_fwd(X, W, 5, bl, 64, 64, X, X)
    assert seen == []


def test_masks_of_many_dimensions(calls):
    lx, seen, _ = calls
    out, other = header(lx, 4), header(lx, 4)
    m = GpuMask(torch.zeros([2, 3] + [1] * 14 + [5, 7], dtype=torch.uint8))
    lx.lx_mask_compact(m, out=out)
    lx.lx_mask_compact_pair(m, out=(out, other))
    assert [(n, a[:7]) for n, a in seen] == [("lx_mask_compact", [p(m), 6, 5, 7, 35, 7, 1]),
                                             ("lx_mask_compact_pair", [p(m), 6, 5, 7, 35, 7, 1])]
    del seen[:]
    with pytest.raises(AssertionError):                    # no row and column
        lx.lx_mask_compact(GpuMask(torch.zeros(7, dtype=torch.uint8)), out=out)
    with pytest.raises(ZeroDivisionError):
        lx.lx_mask_compact(GpuMask(torch.zeros(2, 0, 7, dtype=torch.uint8)), out=out)
    assert seen == []


class Held:
    def __init__(self, v):
        self._as_parameter_ = v


@pytest.mark.parametrize("sixteen", [16, 2 ** 70 + 16, C.c_int32(16), Held(16), Held(C.c_int32(16)), torch.tensor(16)])
def test_numbers_convert_as_in_the_prototype(calls, sixteen):
    lx, seen, _ = calls
    X, bl = bf(64, 64), header(lx, 1)
    Q, LSE = torch.zeros(1, 2, 64, 64), torch.zeros(1, 2, 64)
    lx.lx_sparse_ffn_fwd(X, X, X, bl, sixteen, 64, X, X)
    lx.lx_sparse_attn_fwd(Q, Q, Q, bl, 0.25, False, Q, LSE, mask_batch=sixteen)
    assert seen[0][1][4] == 16 and seen[1][1][12] == 16
    assert C.CFUNCTYPE(C.c_int, C.c_int32)(lambda v: v)(sixteen) == 16      # (ctypes itself)


@pytest.mark.parametrize("quarter,value", [(0.25, 0.25), (C.c_float(0.25), 0.25), (Held(0.25), 0.25), (1, 1.0), (torch.tensor(0.25), 0.25),
                                           (1e300, float("inf"))])
def test_reals_convert_as_in_the_prototype(calls, quarter, value):
    lx, seen, _ = calls
    Q, LSE, bl = torch.zeros(1, 2, 64, 64), torch.zeros(1, 2, 64), header(lx, 1)
    lx.lx_sparse_attn_fwd(Q, Q, Q, bl, quarter, False, Q, LSE)
    lx.lx_mlp_predict_mask(bf(64, 64), bf(64, 64), quarter, 64, mask=LSE)
    assert seen[0][1][5] == value and seen[1][1][7] == value


def test_wrong_types_are_ctypes_errors(calls):
    lx, seen, _ = calls
    X, bl = bf(64, 64), header(lx, 1)
    Q, LSE = torch.zeros(1, 2, 64, 64), torch.zeros(1, 2, 64)
    for wrong in (64.0, None, "64", C.c_int64(64), Held(64.0)):
        with pytest.raises(C.ArgumentError):
            lx.lx_sparse_ffn_fwd(X, X, X, bl, wrong, 64, X, X)
    for wrong in (None, "1", C.c_double(1.0), 10 ** 400):
        with pytest.raises(C.ArgumentError):
            lx.lx_sparse_attn_fwd(Q, Q, Q, bl, wrong, False, Q, LSE)
    other = header(lx, 1)
    other.c = lx.lx_compact_job()                          # a structure, of another type
    with pytest.raises(C.ArgumentError):
        lx.lx_sparse_ffn_fwd(X, X, X, other, 64, 64, X, X)
    with pytest.raises(lx.LxError):                        # an unsupported dtype comes first
        lx.lx_sparse_ffn_fwd(X.double(), X, X, bl, 64.0, 64, X, X)
    assert seen == []


def test_the_module_is_of_this_interpreter():
    from paper_2510_15964_amd import build
    build.ensure()
    from paper_2510_15964_amd import lx
    assert build.CALL == lx.CALL_PATH == lx._call.__file__
    assert os.path.basename(build.CALL) == "_lx_call" + sysconfig.get_config_var("EXT_SUFFIX")
    assert sysconfig.get_config_var("SOABI") in build.CALL


@pytest.mark.parametrize("there", [(), ("LIB",), ("CALL",), ("LIB", "CALL")])
def test_built_unless_both_files_are_there(monkeypatch, tmp_path, there):
    from paper_2510_15964_amd import build
    built = []
    monkeypatch.setattr(build, "build", lambda: built.append(1))
    for f in ("LIB", "CALL"):
        monkeypatch.setattr(build, f, str(tmp_path / f))
        if f in there:
            (tmp_path / f).touch()
    build.ensure()
    assert len(built) == (0 if len(there) == 2 else 1)


def test_a_second_copy_of_the_binding_leaves_the_first_alone():
    import importlib.util
    from paper_2510_15964_amd import build
    build.ensure()
    from paper_2510_15964_amd import lx
    spec = importlib.util.spec_from_file_location("lx_again", lx.__file__)
    again = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(again)
    X = bf(64, 64)
    for m in (lx, again, lx):
        with pytest.raises(m.LxError):
            m.lx_sparse_ffn_fwd(X.double(), X, X, m.BlockList(1, 4, X, X, 1), 64, 64, X, X)
