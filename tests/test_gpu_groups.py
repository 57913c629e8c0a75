"""Kernels that take several token slots per workgroup, at the edges of their
groups and of the rules that choose between the kernels: the oracle's results,
and the same bits from a launch that takes one slot per workgroup."""
import numpy as np
import pytest
import torch

import oracle
import synth
from parity import bf16_f64, check_probe, check_residual, torch_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def px():
    import paper_2607_22595_amd as px
    return px


def dev(a):
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(a.view(np.int32) if a.dtype == np.uint32 else a).cuda()


def build(px, req, T_valid, sub, n_apps):
    rt = px.Route(len(req), n_apps)
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    px.xmix_route_build(dev(req), torch.tensor([T_valid], dtype=torch.int32, device="cuda"),
                        dev(sub), rt, err)
    return rt, err


def batch(T, n_apps, p=0.5, seed=0, R=None):
    rng = np.random.default_rng(seed)
    R = T if R is None else R
    req = np.sort(rng.integers(0, R, T)).astype(np.int32)
    sub = np.zeros(R, np.uint32)
    for a in range(n_apps):
        sub |= (rng.random(R) < p).astype(np.uint32) << np.uint32(a)
    return rng, req, sub


@pytest.mark.parametrize("T,R_max", [(1, 1), (1023, 7), (1025, 9), (8191, 30), (8192, 8192),
                                     (8193, 5), (20001, 300)])
def test_route_build_batches(px, T, R_max):
    """One slot, a chunk and a batch of chunks more or less by one."""
    rng, req, sub = batch(T, 32, seed=T, R=R_max)
    req[rng.integers(0, T, 3)] = -1
    req[rng.integers(0, T, 2)] = R_max + 1
    for tv in (T, T // 2, T + 1):
        rt, err = build(px, req, tv, sub, 32)
        tm, cnt, lists, e = oracle.route(req, tv, sub, 32)
        assert np.array_equal(rt.tok_mask.cpu().numpy().view(np.uint32), tm)
        assert np.array_equal(rt.app_count.cpu().numpy(), cnt)
        assert np.array_equal(rt.app_tokens.cpu().numpy(), lists)
        assert int(err.item()) == e


@pytest.mark.parametrize("T,d,n_steer,dtype", [
    (5, 8, 1, "bf16"), (4095, 264, 5, "bf16"), (4096, 264, 5, "bf16"), (4098, 1000, 9, "bf16"),
    (2049, 2056, 32, "bf16"), (7, 4, 3, "f32"), (4097, 260, 5, "f32"), (2047, 1028, 4, "f32")])
def test_steer_token_groups(px, T, d, n_steer, dtype):
    rng, req, sub = batch(T, n_steer, p=0.3, seed=T)
    bf = dtype == "bf16"
    draw = synth.normal_bf16 if bf else synth.normal_f32
    h, v = draw("g/h", (T, d), 1.0), draw("g/v", (n_steer, d), 0.2)
    alpha = rng.uniform(-8, 8, (T, n_steer)).astype(np.float32)
    rt, _ = build(px, req, T, sub, n_steer)
    hd = dev(h)
    px.xmix_steer_apply(hd, rt, dev(req), dev(v), range(n_steer), dev(alpha))
    tm = oracle.route(req, T, sub, n_steer)[0]
    ref = oracle.steer(h, tm, req, v, list(range(n_steer)), alpha)
    got = torch_bits(hd) if bf else hd.cpu().numpy()
    # fp64 sums of a few exact products, rounded once: the oracle's own value
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("T", [64, 4096])
def test_steer_rounding_over_the_whole_range(px, T):
    """Zeros, subnormal results, halfway ties, the top of the range, infinities
    and NaN: one rounding from fp64, as the oracle's."""
    d = 64
    rng = np.random.default_rng(T)
    h = rng.integers(0, 1 << 16, (T, d)).astype(np.uint16)   # every kind of bf16
    v = rng.integers(0, 1 << 16, (1, d)).astype(np.uint16)
    v[0, :16] = 0
    v[0, 16:24] = 0x0080                                      # 2^-126
    alpha = np.exp2(rng.integers(-20, 3, (T, 1))).astype(np.float32)
    alpha[::5] = 0.0
    req = np.arange(T, dtype=np.int32)
    rt, _ = build(px, req, T, np.ones(T, np.uint32), 1)
    hd = dev(h)
    px.xmix_steer_apply(hd, rt, dev(req), dev(v), [0], dev(alpha))
    ref = oracle.steer(h, np.ones(T, np.uint32), req, v, [0], alpha)
    got, nan = torch_bits(hd), np.isnan(bf16_f64(ref))
    assert np.array_equal(np.isnan(bf16_f64(got)), nan)
    assert np.array_equal(got[~nan], ref[~nan])


@pytest.mark.parametrize("T,d,n_probe,R", [(2047, 264, 4, 5), (2048, 264, 1, 70), (2050, 4104, 5, 64),
                                           (2049, 264, 8, 63), (2300, 520, 9, 129)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_probe_token_groups(px, T, d, n_probe, R, dtype):
    """Per-token and mean-pooled probes on either side of the group rule; spans
    that end inside a group, empty ones and one past the slots."""
    rng = np.random.default_rng(T + n_probe)
    cu = np.sort(rng.integers(0, T, R + 1)).astype(np.int32)
    cu[0], cu[R - 1:] = 0, T
    cu[R // 2] = cu[R // 2 - 1]                                # an empty span
    req = np.full(T, -1, np.int32)
    for r in range(R):
        req[cu[r]:cu[r + 1]] = r
    sub = (rng.random((R, n_probe)) < 0.6) @ (1 << np.arange(n_probe, dtype=np.uint64))
    sub = sub.astype(np.uint32)
    bf = dtype == "bf16"
    draw = synth.normal_bf16 if bf else synth.normal_f32
    h, w = draw("p/h", (T, d), 1.0), draw("p/w", (n_probe, d), d ** -0.5)
    b = rng.normal(0, 0.3, n_probe).astype(np.float32)
    bits = list(range(n_probe))
    rt, _ = build(px, req, T, sub, n_probe)
    tm = oracle.route(req, T, sub, n_probe)[0]
    hd, wd, bd = dev(h), dev(w), dev(b)

    def call(mode, n_out, hh, route, cu_d=None):
        out = [torch.full((n_probe, n_out), float("nan"), device="cuda") for _ in range(2)]
        nb = px.probe_workspace(route.T_max, n_probe, mode)
        ws = torch.full((max(nb, 1),), 0xFF, dtype=torch.uint8, device="cuda")
        px.xmix_probe_score(hh, route, wd, bd, bits, mode, *out, cu_seqlens=cu_d, ws=ws)
        return [o.cpu().numpy() for o in out]

    hf, wf = (bf16_f64(h), bf16_f64(w)) if bf else (h.astype(np.float64), w.astype(np.float64))
    absdot = np.abs(wf) @ np.abs(hf).T
    lg, sg = call(px.XMIX_PROBE_TOKEN, T, hd, rt)
    lr, sr = oracle.probe_token(h, tm, w, b, bits)
    assert np.array_equal(np.isnan(lg), np.isnan(lr))
    check_probe(lg, sg, lr, sr, ~np.isnan(lr), absdot)
    # the same bits from launches of fewer slots than the group rule asks for
    for t0 in (0, 1001):
        n = min(700, T - t0)
        part, _ = build(px, req[t0:t0 + n], n, sub, n_probe)
        lp, _ = call(px.XMIX_PROBE_TOKEN, n, dev(h[t0:t0 + n]), part)
        assert np.array_equal(lp, lg[:, t0:t0 + n], equal_nan=True)
    lg, sg = call(px.XMIX_PROBE_MEAN, R, hd, rt, dev(cu))
    lr, sr = oracle.probe_mean(h, tm, w, b, bits, cu)
    assert np.array_equal(np.isnan(lg), np.isnan(lr))
    floor = np.stack([[absdot[q, cu[r]:cu[r + 1]].mean() if cu[r + 1] > cu[r] else 0.0
                       for r in range(R)] for q in range(n_probe)])
    check_probe(lg, sg, lr, sr, ~np.isnan(lr), floor)


@pytest.mark.parametrize("R", [2047, 2048, 2050])
@pytest.mark.parametrize("d,n_probe,dtype", [(264, 4, "bf16"), (4104, 5, "bf16"), (1028, 9, "f32")])
def test_probe_last_request_groups(px, R, d, n_probe, dtype):
    """Last-token probes on either side of the group rule: empty spans at each
    place of a group and a whole group of them, spans that end past the slots,
    and the bits of launches of fewer requests."""
    rng = np.random.default_rng(R + d)
    size = rng.integers(1, 4, R)
    for j in range(4):
        size[40 + 4 * j + j] = 0                               # at place j of a group
    size[80:84] = 0
    cu = np.concatenate([[0], np.cumsum(size)]).astype(np.int32)
    T = int(cu[-1])
    req = np.repeat(np.arange(R), size).astype(np.int32)
    cu[R - 1:] += 2                                            # these two end past the slots
    sub = (rng.random((R, n_probe)) < 0.5) @ (1 << np.arange(n_probe, dtype=np.uint64))
    sub = sub.astype(np.uint32)
    bf = dtype == "bf16"
    draw = synth.normal_bf16 if bf else synth.normal_f32
    h, w = draw("l/h", (T, d), 1.0), draw("l/w", (n_probe, d), d ** -0.5)
    b = rng.normal(0, 0.3, n_probe).astype(np.float32)
    bits = list(range(n_probe))
    rt, _ = build(px, req, T, sub, n_probe)
    tm = oracle.route(req, T, sub, n_probe)[0]
    hd, wd, bd = dev(h), dev(w), dev(b)

    def call(cu_d):
        out = [torch.full((n_probe, len(cu_d) - 1), float("nan"), device="cuda")
               for _ in range(2)]
        px.xmix_probe_score(hd, rt, wd, bd, bits, px.XMIX_PROBE_LAST, *out,
                            cu_seqlens=dev(cu_d))
        return [o.cpu().numpy() for o in out]

    lg, sg = call(cu)
    lr, sr = oracle.probe_last(h, tm, w, b, bits, np.minimum(cu, T))
    lr[:, cu[1:] > T] = np.nan                                 # not the oracle's to read
    assert np.array_equal(np.isnan(lg), np.isnan(lr))
    assert np.isnan(lr[:, 40]).all() and np.isnan(lr[:, 80:84]).all() and np.isnan(lr[:, -1]).all()
    hf, wf = (bf16_f64(h), bf16_f64(w)) if bf else (h.astype(np.float64), w.astype(np.float64))
    absdot = (np.abs(wf) @ np.abs(hf).T)[:, np.clip(cu[1:] - 1, 0, T - 1)]
    check_probe(lg, sg, lr, sr, ~np.isnan(lr), absdot)
    for r0 in (0, 1001):
        lp, _ = call(cu[r0:r0 + 1001])
        assert np.array_equal(lp, lg[:, r0:r0 + 1000], equal_nan=True)


@pytest.mark.parametrize("T,d,k,n_clamp,n_apps", [(1, 8, 1, 1, 1), (5, 264, 64, 16, 3),
                                                  (4097, 264, 32, 5, 9), (130, 4104, 8, 4, 2)])
def test_clamp_token_groups(px, T, d, k, n_clamp, n_apps):
    """Clamps of single calls and of a batched call (more apps than one launch
    takes) over whole and partial groups; clamp ids outside the dictionary,
    ids that the encode selected, and an unused slot (-1) in its output."""
    m = 512
    rng, req, sub = batch(T, n_apps, p=0.6, seed=T + k)
    h = synth.normal_bf16("c/h", (T, d), 1.0)
    rt, _ = build(px, req, T, sub, n_apps)
    tm = oracle.route(req, T, sub, n_apps)[0]
    apps, ref = [], h.copy()
    one = dev(h)
    for a in range(n_apps):
        W = synth.normal_bf16(f"c/W{a}", (m, d), d ** -0.5)
        idx = np.argsort(rng.random((T, m)), axis=1)[:, :k].astype(np.int32)
        val = synth.normal_bf16(f"c/val{a}", (T, k), 2.0) & np.uint16(0x7FFF)
        ids = rng.choice(m, n_clamp, replace=False).astype(np.int32)
        idx[T // 2, 0] = ids[0]
        idx[T // 2, k - 1] = -1 if k > 1 else ids[0]
        vals = rng.normal(5, 2, n_clamp).astype(np.float32)
        ids_ref, vals_ref = ids, vals
        if n_clamp > 1:      # an id outside the dictionary clamps nothing
            ids_ref, vals_ref = ids[:-1].copy(), vals[:-1]
            ids[-1] = m + 3 if a % 2 else -1
        da = [dev(x) for x in (idx, val, W, ids, vals)]
        delta = torch.zeros((T, d), dtype=torch.float32, device="cuda")
        px.xmix_sae_clamp_decode(one, rt, a, *da, delta)
        prev = ref
        ref, dref = oracle.clamp_decode(prev, tm, a, idx, val, W, ids_ref, vals_ref,
                                        want_delta=True)
        got, dg = torch_bits(one), delta.cpu().numpy()
        rows = (tm >> np.uint32(a)) & 1 == 1
        assert np.array_equal(got[~rows], prev[~rows])
        # n_clamp fp32 multiply-adds: each within 2^-24 of the sum of magnitudes
        worst = np.abs(vals).sum() + 64 * n_clamp
        assert np.all(np.abs(dg[rows] - dref[rows]) <= n_clamp * 2.0 ** -23 * worst)
        for t in np.nonzero(rows)[0][:: max(1, T // 50)]:
            check_residual(got[t], ref[t], dref[t])
        ref = got.copy()          # the next app starts from the same rows
        apps.append((a, *da, delta.clone()))
    many = dev(h)
    again = [(*a[:6], torch.zeros_like(a[6])) for a in apps]
    px.xmix_sae_clamp_decode_multi(many, rt, again)
    assert torch.equal(many.view(torch.int16), one.view(torch.int16))
    for a, b in zip(apps, again):
        assert torch.equal(a[6], b[6])


@pytest.mark.parametrize("T,d,n_clamp", [(1024, 4096, 7), (1025, 4096, 7), (1030, 4096, 2),
                                         (4096, 4096, 2), (4097, 4096, 2), (8203, 520, 16),
                                         (2046, 2056, 3), (513, 8200, 5)])
def test_clamp_launches_of_every_size_agree(px, T, d, n_clamp):
    """A launch of many rows (four tokens per workgroup where the rule says so,
    groups with no, some and all of their tokens subscribed) leaves the bits that
    launches of a few hundred rows leave (one token per workgroup), for one app
    and for three; some of its rows against the oracle."""
    m, k, n_apps = 300, 24, 3
    rng, req, sub = batch(T, n_apps, p=0.4, seed=T + d)
    sub[:64] = np.where(np.arange(64) < 32, 0, 7)   # whole groups of none and of all
    req[:64] = np.arange(64)
    tm = oracle.route(req, T, sub, n_apps)[0]
    h = synth.normal_bf16("c/h", (T, d), 1.0)
    apps = []
    for a in range(n_apps):
        idx = np.argsort(rng.random((T, m)), axis=1)[:, :k].astype(np.int32)
        val = synth.normal_bf16(f"c/val{a}", (T, k), 2.0) & np.uint16(0x7FFF)
        apps.append((idx, val, synth.normal_bf16(f"c/W{a}", (m, d), d ** -0.5),
                     rng.choice(m, n_clamp, replace=False).astype(np.int32),
                     rng.normal(5, 2, n_clamp).astype(np.float32)))

    def run(t0, n):
        one, many = dev(h[t0:t0 + n]), dev(h[t0:t0 + n])
        rt, _ = build(px, req[t0:t0 + n], n, sub, n_apps)
        args = []
        for a, (idx, val, W, ids, vals) in enumerate(apps):
            x = [dev(v) for v in (idx[t0:t0 + n], val[t0:t0 + n], W, ids, vals)]
            args.append((a, *x, torch.zeros((n, d), dtype=torch.float32, device="cuda")))
        for x in args:
            px.xmix_sae_clamp_decode(one, rt, *x)
        deltas = [x[6].clone() for x in args]
        px.xmix_sae_clamp_decode_multi(many, rt, args)
        assert torch.equal(many.view(torch.int16), one.view(torch.int16))
        assert all(torch.equal(x[6], y) for x, y in zip(args, deltas))
        return torch_bits(one), [x.cpu().numpy() for x in deltas]

    got, deltas = run(0, T)
    for t0 in range(0, T, 512):
        n = min(512, T - t0)
        part, dp = run(t0, n)
        assert np.array_equal(part, got[t0:t0 + n])
        assert all(np.array_equal(x, y[t0:t0 + n]) for x, y in zip(dp, deltas))
    assert np.array_equal(got[(tm & 7) == 0], h[(tm & 7) == 0])
    idx, val, W, ids, vals = apps[0]
    rows = np.nonzero(tm & 1)[0][::97]
    _, ref = oracle.clamp_decode(h[rows], np.ones(len(rows), np.uint32), 0, idx[rows], val[rows],
                                 W, ids, vals, want_delta=True)
    # n_clamp fp32 multiply-adds: each within 2^-24 of the sum of magnitudes
    worst = np.abs(vals).sum() + 64 * n_clamp
    assert np.all(np.abs(deltas[0][rows] - ref) <= n_clamp * 2.0 ** -23 * worst)


@pytest.mark.parametrize("widths", [(4,), (12, 16), (1024, 4), (1036, 20), (4096, 1028), (2, 6),
                                    (2048, 10)])
@pytest.mark.parametrize("off", [0, 4])
def test_readback_row_sizes(px, widths, off):
    """Segments around the 16-byte unit and the wave's 4 KB turn, on sources at
    a 4-byte offset, into a ring that wraps."""
    T, cap = 301, 200
    rng, req, sub = batch(T, 1, p=0.7, seed=sum(widths))
    rt, _ = build(px, req, T, sub, 1)
    tm = oracle.route(req, T, sub, 1)[0]
    segs, host = [], []
    for n in widths:
        raw = rng.integers(0, 256, T * n + 16).astype(np.uint8)
        segs.append(torch.from_numpy(raw).cuda()[off:off + T * n].view(T, n))
        host.append(raw[off:off + T * n].reshape(T, n))
    ring = px.Ring(cap, 16 + sum(widths))
    slots, head = np.zeros((cap, 16 + sum(widths)), np.uint8), 0
    for _ in range(3):
        px.xmix_readback_compact(segs, rt, 0, dev(req), 3, 5, ring)
        slots, head = oracle.compact(host, tm, 0, req, 3, 5, slots, head)
        assert int(ring.head[0].item()) == head and int(ring.head[1].item()) == 0
        assert np.array_equal(ring.slots.cpu().numpy(), slots)


@pytest.mark.parametrize("T,n,cap", [(4500, 64, 4700), (9000, 36, 5000), (2300, 4100, 2000),
                                     (1300, 8196, 900)])
def test_readback_more_rows_than_workgroups(px, T, n, cap):
    """Rows that the workgroups take in turns, by one, two and four waves a row."""
    rng, req, sub = batch(T, 1, p=0.95, seed=n)
    rt, _ = build(px, req, T, sub, 1)
    tm = oracle.route(req, T, sub, 1)[0]
    raw = rng.integers(0, 256, (T, n)).astype(np.uint8)
    ring = px.Ring(cap, 16 + n)
    slots, head = np.zeros((cap, 16 + n), np.uint8), 0
    for _ in range(2):
        px.xmix_readback_compact([dev(raw)], rt, 0, dev(req), 3, 5, ring)
        slots, head = oracle.compact([raw], tm, 0, req, 3, 5, slots, head)
        assert int(ring.head[0].item()) == head and int(ring.head[1].item()) == 0
        assert np.array_equal(ring.slots.cpu().numpy(), slots)


@pytest.mark.parametrize("sbits,pbits", [([0, 1, 2], [3, 4]), ([5, 6], [0, 1, 2]), ([6, 2, 4], [3, 0]),
                                         ([1, 3], [6, 5, 4]), ([31, 0], [30, 31]), ([30, 31], [0])])
def test_app_bits_in_any_order(px, sbits, pbits):
    """Consecutive bits (one shift) and every other order, in the three kernels."""
    T, d = 70, 264
    rng, req, sub = batch(T, 32, p=0.4, seed=len(sbits) + 7 * pbits[0])
    h = synth.normal_bf16("b/h", (T, d), 1.0)
    v, w = synth.normal_bf16("b/v", (len(sbits), d), 0.2), synth.normal_bf16("b/w", (len(pbits), d), 0.1)
    alpha = rng.uniform(-8, 8, (T, len(sbits))).astype(np.float32)
    b = np.zeros(len(pbits), np.float32)
    rt, _ = build(px, req, T, sub, 32)
    tm = oracle.route(req, T, sub, 32)[0]
    ref = oracle.steer(h, tm, req, v, sbits, alpha)
    lr, _ = oracle.probe_token(h, tm, w, b, pbits)
    for fused in (False, True):
        hd = dev(h)
        out = [torch.full((len(pbits), T), float("nan"), device="cuda") for _ in range(2)]
        if fused:
            px.xmix_steer_probe(hd, rt, dev(req), dev(v), sbits, dev(alpha), dev(w), dev(b), pbits,
                                *out)
        else:
            px.xmix_probe_score(hd, rt, dev(w), dev(b), pbits, px.XMIX_PROBE_TOKEN, *out)
            px.xmix_steer_apply(hd, rt, dev(req), dev(v), sbits, dev(alpha))
        assert np.array_equal(torch_bits(hd), ref)
        got = out[0].cpu().numpy()
        assert np.array_equal(np.isnan(got), np.isnan(lr))
        # 264 fp32 multiply-adds of terms of about 0.1
        assert np.nanmax(np.abs(got - lr)) <= 264 * 2.0 ** -24 * 100


@pytest.mark.parametrize("T,d,n_steer,n_probe,dtype", [
    (1, 8, 1, 1, "bf16"), (130, 4088, 4, 4, "bf16"), (70, 4104, 5, 5, "bf16"),
    (1024, 4096, 2, 3, "bf16"), (1025, 4096, 2, 3, "bf16"),   # up to 8 MB of rows, and past it
    (33, 8200, 8, 8, "bf16"), (40, 2056, 3, 9, "bf16"), (64, 2052, 4, 8, "f32"),
    (1025, 2048, 1, 4, "f32")])
@pytest.mark.parametrize("gap", [1, 2])
def test_steer_probe_early_rows(px, T, d, n_steer, n_probe, dtype, gap):
    """The fused pass on either side of the rule that reads rows before their
    masks, rows that end inside, at and past a turn of 512 slices, app bits
    side by side and apart: the oracle's rows, and the probe kernel's bits."""
    n = gap * (n_steer + n_probe)
    rng, req, sub = batch(T, n, p=0.4, seed=T + d)
    bf = dtype == "bf16"
    draw = synth.normal_bf16 if bf else synth.normal_f32
    h, v = draw("e/h", (T, d), 1.0), draw("e/v", (n_steer, d), 0.2)
    w = draw("e/w", (n_probe, d), d ** -0.5)
    h[::3, -1] = 0x7F80 if bf else np.inf                     # some rows end in an infinity
    alpha = rng.uniform(-4, 4, (T, n_steer)).astype(np.float32)
    b = rng.normal(0, 0.3, n_probe).astype(np.float32)
    sbits = [gap * s for s in range(n_steer)]
    pbits = [gap * (n_steer + p) for p in range(n_probe)]
    rt, _ = build(px, req, T, sub, n)
    tm = oracle.route(req, T, sub, n)[0]
    hd, wd, bd, vd, rd, ad = dev(h), dev(w), dev(b), dev(v), dev(req), dev(alpha)
    sep = [torch.full((n_probe, T), float("nan"), device="cuda") for _ in range(2)]
    px.xmix_probe_score(hd, rt, wd, bd, pbits, px.XMIX_PROBE_TOKEN, *sep)
    fused = [torch.full((n_probe, T), float("nan"), device="cuda") for _ in range(2)]
    px.xmix_steer_probe(hd, rt, rd, vd, sbits, ad, wd, bd, pbits, *fused)
    for a, c in zip(fused, sep):
        assert np.array_equal(a.cpu().numpy(), c.cpu().numpy(), equal_nan=True)
    ref = oracle.steer(h, tm, req, v, sbits, alpha)
    got = torch_bits(hd) if bf else hd.cpu().numpy()
    assert np.array_equal(got, ref)
    lr, sr = oracle.probe_token(h, tm, w, b, pbits)
    fin = np.isfinite(lr)
    hf, wf = (bf16_f64(h), bf16_f64(w)) if bf else (h.astype(np.float64), w.astype(np.float64))
    hf[::3, -1] = 0.0
    absdot = np.abs(wf) @ np.abs(hf).T
    check_probe(fused[0].cpu().numpy(), fused[1].cpu().numpy(), lr, sr, fin, absdot)


@pytest.mark.parametrize("n_steer,n_probe", [(1, 2), (2, 2), (2, 3), (2, 4), (2, 5), (3, 2),
                                             (3, 4), (9, 2)])
@pytest.mark.parametrize("T,d,dtype", [(65, 4100, "f32"), (513, 4096, "f32"), (40, 4104, "bf16")])
def test_steer_probe_few_apps(px, T, d, n_steer, n_probe, dtype):
    """The numbers of probes and of steering vectors where the fused pass changes
    how many it asks for together, rows of more than one turn of 512 slices."""
    test_steer_probe_early_rows(px, T, d, n_steer, n_probe, dtype, 1)


def test_rows_of_more_column_slices_than_a_grid_holds(px):
    """A row of 65537 workgroups' columns: steering and a clamp, against torch on
    the columns where a grid's y would end and on the last ones."""
    d = (1 << 27) + 2056
    at = torch.tensor([0, 1, 32768 * 2048 - 1, 32768 * 2048, 65535 * 2048 + 5, 65536 * 2048 - 1,
                       65536 * 2048, d - 9, d - 8, d - 1], device="cuda")
    rt, _ = build(px, np.zeros(1, np.int32), 1, np.array([3], np.uint32), 2)
    W = torch.empty((1, d), dtype=torch.bfloat16, device="cuda")
    for c in range(0, d, 1 << 24):                     # small whole numbers, exact in bf16
        n = min(1 << 24, d - c)
        W[0, c:c + n] = ((torch.arange(n, device="cuda") + c // 512) % 61).to(torch.bfloat16)
    h = torch.zeros((1, d), dtype=torch.bfloat16, device="cuda")
    px.xmix_steer_apply(h, rt, dev(np.zeros(1, np.int32)), W, [0],
                        torch.full((1, 1), 2.0, device="cuda"))
    assert torch.equal(h[0, at], 2 * W[0, at])
    assert torch.equal(h, 2 * W)
    idx = torch.full((1, 1), -1, dtype=torch.int32, device="cuda")
    args = (1, idx, torch.zeros((1, 1), dtype=torch.bfloat16, device="cuda"), W,
            torch.zeros(1, dtype=torch.int32, device="cuda"), torch.ones(1, device="cuda"))
    px.xmix_sae_clamp_decode(h, rt, *args)
    assert torch.equal(h, 3 * W)
    px.xmix_sae_clamp_decode_multi(h, rt, [args])
    assert torch.equal(h, 4 * W)
