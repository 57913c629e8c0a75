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
