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


def calls(px):
    """Every call that is marshalled natively: its arguments, the wrong ones of
    each (a check fails), and those whose absence the C entry point reports."""
    T, d, n, p, R, E, k, m, z = 8, 256, 2, 3, 4, 16, 4, 256, dict(device="cuda")
    bf, i32 = torch.bfloat16, torch.int32

    def t(*shape, dtype=torch.float32):
        return torch.zeros(shape, dtype=dtype, **z)

    rt, req, sub, tv, err = px.Route(T, 8), t(T, dtype=i32), t(R, dtype=i32), t(1, dtype=i32), t(1, dtype=i32)
    h, v, w, b, alpha = t(T, d, dtype=bf), t(n, d, dtype=bf), t(p, d, dtype=bf), t(p), t(R, n)
    lg, W = t(p, T), px.xmix_sae_pack_encoder(t(m, d, dtype=bf))
    ids, ring = t(T, dtype=i32), px.Ring(16, 16 + 6 * k)
    ws = torch.zeros(px.sae_encode_workspace(T, d, m, k), dtype=torch.uint8, device="cuda")
    bad_h = [t(T - 1, d, dtype=bf), t(T, 2 * d, dtype=bf), t(T, d), t(T, 1, d, dtype=bf)]
    bad_v = [t(n, d), t(n, d // 2, dtype=bf)]
    bad_alpha = [t(R, n + 1), t(R * n), t(R, n, dtype=bf)]
    bad_w = [t(p, d), t(p + 1, d, dtype=bf), t(p, d // 2, dtype=bf)]
    bad_lg = [t(p, T + 1), t(p + 1, T), t(p * T)]
    steer = dict(vecs=v, app_bits=[0, 1], alpha=alpha)
    bad_steer = dict(vecs=bad_v, app_bits=[[0], [0, 1, 2]], alpha=bad_alpha)
    both = dict(vecs=v, steer_bits=[0, 1], alpha=alpha, w=w, b=b, probe_bits=[2, 3, 4], logit_out=lg,
                score_out=t(p, T))
    bad_both = dict(vecs=bad_v, steer_bits=[[0]], alpha=bad_alpha, w=bad_w, b=[b.to(bf)],
                    probe_bits=[[2]], logit_out=bad_lg, score_out=bad_lg)
    probe = dict(h=h, route=rt, w=w, b=b, app_bits=[2, 3, 4], mode=px.XMIX_PROBE_TOKEN, logit_out=lg,
                 score_out=t(p, T))
    bad_probe = dict(h=bad_h[:3], w=bad_w, b=[b.to(bf)], app_bits=[[2]], logit_out=bad_lg)
    span = dict(probe, mode=px.XMIX_PROBE_LAST, logit_out=t(p, R), score_out=t(p, R),
                cu_seqlens=t(R + 1, dtype=i32))
    bad_span = dict(bad_probe, h=[t(T, 2 * d, dtype=bf), t(T, d)], logit_out=[t(p, R + 1), t(p, T)],
                    cu_seqlens=[t(0, dtype=i32), t(R, dtype=i32)])
    enc = dict(h=h, route=rt, app_bit=0, W=W, b_enc=t(m, dtype=bf), b_dec=t(d, dtype=bf), c_fold=None,
               k=k, idx_out=t(T, k, dtype=i32), val_out=t(T, k, dtype=bf), ws=ws)
    bad_enc = dict(h=bad_h[:1] + bad_h[2:], k=[k + 1, -1], idx_out=[t(T, k), t(T, k + 1, dtype=i32)],
                   val_out=[t(T, k), t(T + 1, k, dtype=bf)])
    ring_args = dict(req_of_token=req, layer_id=0, app_id=0, ring=ring)
    bad_req = [t(T + 1, dtype=i32), t(T)]
    return {
        px.xmix_route_build: (dict(req_of_token=req, T_valid=tv, sub_mask=sub, route=rt, err_word=err),
                              dict(req_of_token=bad_req, T_valid=[t(1)], sub_mask=[t(R)]),
                              ["err_word"]),
        px.xmix_route_gate: (dict(route=rt, app_bit=0, signal=t(T), threshold=t(1)),
                             dict(signal=[t(T, dtype=bf)], threshold=[t(1, dtype=i32)]), []),
        px.xmix_route_trigger: (dict(route=rt, app_bit=0, token_ids=ids, vocab_bits=t(4, dtype=i32),
                                     vocab_size=100),
                                dict(token_ids=[t(T)], vocab_bits=[t(3, dtype=i32)]), []),
        px.xmix_steer_apply: (dict(h=h, route=rt, req_of_token=req, **steer),
                              dict(h=bad_h, **bad_steer), ["req_of_token"]),
        px.xmix_steer_probe: (dict(h=h, route=rt, req_of_token=req, **both),
                              dict(h=bad_h, **bad_both), ["req_of_token"]),
        px.xmix_route_steer_probe: (dict(req_of_token=req, T_valid=tv, sub_mask=sub, route=rt,
                                         err_word=err, h=h, **both),
                                    dict(req_of_token=bad_req, h=bad_h, **bad_both),
                                    ["T_valid", "err_word"]),
        px.xmix_router_write: (dict(logits=t(T, E), route=rt, app_bits=[0, 1], offsets=t(n, E)),
                               dict(logits=[t(T - 1, E), t(T, E + 1)], app_bits=[[0]],
                                    offsets=[t(n, E + 1), t(n + 1, E), t(n, E, dtype=bf)]), []),
        px.xmix_probe_score: (probe, bad_probe, ["score_out"]),
        (lambda **a: px.xmix_probe_score(**a)): (span, bad_span, ["score_out"]),
        px.xmix_sae_encode_topk: (enc, bad_enc, []),
        px.xmix_sae_encode_topk_ring: (dict(enc, **ring_args), dict(bad_enc, req_of_token=bad_req), []),
    }


@pytest.mark.gpu
def test_every_call_checks_its_arguments(px):
    for fn, (args, wrong, absent) in calls(px).items():
        fn(**args)
        for name, values in wrong.items():
            for v in values:
                with pytest.raises((AssertionError, TypeError)):
                    fn(**dict(args, **{name: v}))
        for name in absent:
            with pytest.raises(px.XmixError):
                fn(**dict(args, **{name: None}))
        for name, v in args.items():
            if isinstance(v, torch.Tensor):
                with pytest.raises(ValueError):
                    fn(**dict(args, **{name: v.cpu()}))
                if v.dim() == 2 and v.shape[0] > 1:
                    with pytest.raises(ValueError):
                        fn(**dict(args, **{name: v.t().contiguous().t()}))
            elif isinstance(v, (px.Route, px.Ring, px.SaeDict)):
                other = px.Ring(4, 32) if not isinstance(v, px.Ring) else px.Route(8, 8)
                with pytest.raises(TypeError):
                    fn(**dict(args, **{name: other}))
    torch.cuda.synchronize()
