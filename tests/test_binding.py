"""The binding's argument marshalling: what it binds, passes and refuses."""
import ctypes
import types

import numpy as np
import pytest
import torch


@pytest.fixture(scope="module")
def px():
    import paper_2607_22595_amd as px
    return px


def function(px, args, c_args):
    abs_ = ctypes.cast(ctypes.CDLL(None).abs, ctypes.c_void_p).value
    return px._call.Function("abs", abs_, args, c_args, {"Route": px.XmixRoute})


def test_ints_dims_and_bits(px):
    f = function(px, "x:int b:bits(n)", "x")
    assert f(-5, [1, 2]) == 5 and f(-7, range(3)) == 7 and f(3, ()) == 3
    assert function(px, "x:int b:bits(n)", "n")(-5, [4] * 40) == 40  # the C side refuses it
    g = function(px, "n:dim b:bits(n)", "n")
    assert g(2, (8, 9)) == 2
    with pytest.raises(AssertionError):
        g(3, (8, 9))
    for n in (-1, -7):  # no size: it must not pass as whatever comes after it
        with pytest.raises(AssertionError):
            g(n, (8, 9))
    with pytest.raises(TypeError):
        f("a", [1])
    with pytest.raises(TypeError):
        f(1, ["a"])
    with pytest.raises(TypeError):
        f(1)


@pytest.mark.parametrize("args,c_args", [("x:zz", "x"), ("x", "x"), ("x:int", "y"), ("x:i32[", "x"),
                                         ("x:struct(None)", "x"), ("x:rt", "x")])
def test_bad_specifications_are_refused(px, args, c_args):
    with pytest.raises(ValueError):
        function(px, args, c_args)


def test_tensors_without_gpu_storage_are_refused(px):
    f = function(px, "t?:*", "t")
    assert f(None) == 0
    with pytest.raises(ValueError):
        f(torch.zeros(3))
    with pytest.raises(AssertionError):
        f(np.zeros(3))


def test_streams(px):
    f = function(px, "s:stream", "s")
    for handle in (7, np.int64(7), np.uint64(7), types.SimpleNamespace(cuda_stream=7)):
        assert f(handle) == 7
    with pytest.raises(TypeError):
        f(object())


def test_structs_are_of_their_class(px):
    """A ring, a dictionary or anything else in a route's place is refused before
    its memory is taken for a route, and the other way round."""
    rt, ring = px.Route(8, 2, "cpu"), px.Ring(4, 32, "cpu")
    t = torch.zeros(8)  # (not on the GPU: what gets past the structs ends there)
    dic = types.SimpleNamespace(struct=px.XmixSaeDict())
    for wrong in (ring, dic, types.SimpleNamespace(struct=ctypes.c_int64())):
        for call in (lambda r: px.xmix_route_gate(r, 0, t, t),
                     lambda r: px.xmix_route_trigger(r, 0, t, torch.zeros(8), 8),
                     lambda r: px._call.Function("f", 1, "r:struct(R)", "r", {"R": px.XmixRoute})(r)):
            with pytest.raises(TypeError):
                call(wrong)
    f = function(px, "r:struct(Route) x:int", "x")
    assert f(rt, 3) == 3 and f(types.SimpleNamespace(struct=rt.struct), 4) == 4
    with pytest.raises(AttributeError):
        f(object(), 3)
    # the address is the struct's own
    seen = []
    take = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.POINTER(px.XmixRoute))(
        lambda p: seen.append((ctypes.addressof(p.contents), p.contents.T_max)) or 0)
    g = px._call.Function("take", ctypes.cast(take, ctypes.c_void_p).value, "r:rt(Route)", "r",
                          {"Route": px.XmixRoute})
    assert g(rt) == 0 and seen == [(ctypes.addressof(rt.struct), 8)]


def recorded(px, f):
    """The Function f with its C entry point replaced by one that keeps the route
    it is given, and the list that it keeps it in."""
    args, c_args, structs = f.spec
    at, seen = c_args.split().index("route"), []
    take = ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_uint64] * 24)(
        lambda *c: seen.append(px.XmixRoute.from_buffer_copy(
            ctypes.string_at(c[at], ctypes.sizeof(px.XmixRoute)))) or 0)
    g = px._call.Function("recorded", ctypes.cast(take, ctypes.c_void_p).value, args, c_args, structs)
    g_keep.append(take)
    return g, seen


g_keep = []  # the callbacks, which their Functions do not hold


@pytest.mark.gpu
@pytest.mark.parametrize("rows,slots", [(5, 5), (8, 8), (11, 8)])
def test_route_is_cut_to_the_rows_there_are(px, rows, slots):
    """A kernel may read every row and request id of its route's slots, whether or
    not the token carries a bit: of a tensor with fewer, so many are passed on."""
    rt, z = px.Route(8, 2), lambda *s: torch.zeros(s, device="cuda")
    h, w, b = z(rows, 64), z(2, 64), z(2)
    token, seen = recorded(px, px._probe_score_token)
    token(h, rt, w, b, [0, 1], px.XMIX_PROBE_TOKEN, None, 0, z(2, rows), z(2, rows), None, None)
    span, seen_s = recorded(px, px._probe_score_span)
    span(h, rt, w, b, [0, 1], px.XMIX_PROBE_MEAN, z(4), 3, z(2, 3), z(2, 3), z(64), None)
    steer, seen_q = recorded(px, px._steer_apply)
    steer(z(8, 64), rt, z(rows), w, [0, 1], z(4, 2), None)
    for r in (seen, seen_s, seen_q):
        assert len(r) == 1 and r[0].T_max == slots and r[0].n_apps == 2
        assert r[0].tok_mask == rt.tok_mask.data_ptr() and r[0].app_tokens == rt.app_tokens.data_ptr()
    assert rt.struct.T_max == 8


@pytest.mark.gpu
def test_probes_of_a_tensor_with_the_valid_rows_only(px):
    """The scores of a batch whose activations end at its last valid token."""
    T, n, d = 64, 37, 256
    g = torch.Generator().manual_seed(3)
    h, w = torch.randn((T, d), generator=g).cuda(), torch.randn((3, d), generator=g).cuda()
    b, sub = torch.randn(3, generator=g).cuda(), torch.full((4,), 7, dtype=torch.int32, device="cuda")
    req = torch.repeat_interleave(torch.arange(4, dtype=torch.int32), T // 4).cuda()
    cu = torch.tensor([0, 16, 30, 37, 37], dtype=torch.int32, device="cuda")
    rt = px.Route(T, 3)
    px.xmix_route_build(req, torch.tensor([n], dtype=torch.int32, device="cuda"), sub, rt,
                        torch.zeros(1, dtype=torch.int32, device="cuda"))
    for mode, out in ((px.XMIX_PROBE_TOKEN, T), (px.XMIX_PROBE_MEAN, 4), (px.XMIX_PROBE_LAST, 4)):
        got = []
        for x in (h, h[:n].clone()):
            cols = x.shape[0] if mode == px.XMIX_PROBE_TOKEN else out
            o = [torch.full((3, cols), 9.0, device="cuda") for _ in range(2)]
            ws = torch.zeros(max(px.probe_workspace(T, 3, mode), 1), dtype=torch.uint8, device="cuda")
            px.xmix_probe_score(x, rt, w, b, [0, 1, 2], mode, *o, cu_seqlens=cu, ws=ws)
            got.append([v[:, :min(n, cols)] for v in o])
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
        assert not torch.any(got[0][0][:, :3] == 9.0)


@pytest.mark.gpu
def test_gpu_tensors_are_checked(px):
    rt = px.Route(8, 2)
    h = torch.zeros((8, 64), dtype=torch.bfloat16, device="cuda")
    v, alpha = torch.zeros((2, 64), dtype=torch.bfloat16, device="cuda"), torch.zeros((4, 2)).cuda()
    req = torch.zeros(8, dtype=torch.int32, device="cuda")
    px.xmix_steer_apply(h, rt, req, v, [0, 1], alpha)
    px.xmix_steer_apply(h, rt, req, v[0], [0], alpha[:, :1].contiguous())   # one vector as a row
    px.xmix_steer_apply(h, rt, req, v, (1, 0), alpha, stream=torch.cuda.Stream())
    for bad, err in [((h[:7], rt, req, v, [0, 1], alpha), AssertionError),
                     ((h, rt, req, v.float(), [0, 1], alpha), AssertionError),
                     ((h, rt, req, v[:, :32].contiguous(), [0, 1], alpha), AssertionError),
                     ((h, rt, req, v, [0], alpha), AssertionError),
                     ((h, rt, req, v, [0, 1], alpha.half()), AssertionError),
                     ((h, rt, req, v, [0, 1], alpha.cpu()), ValueError),
                     ((h.t(), rt, req, v, [0, 1], alpha), ValueError),
                     ((h.half(), rt, req, v, [0, 1], alpha), TypeError),
                     ((h, rt, req, v, [0, 2], alpha), px.XmixError)]:
        with pytest.raises(err):
            px.xmix_steer_apply(*bad)
    torch.cuda.synchronize()
