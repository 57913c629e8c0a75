"""The decode encode's ways to cut its work: whole, halved and quartered slices,
tiles of 32, 64, 128 and 256 tokens, at the edges of the rules that choose
between them, against the oracle; and the same bits from every one of them, from
the prefill encode and from the batched call."""
import numpy as np
import pytest
import torch

import oracle
import synth
from parity import check_topk, torch_bits

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


class Enc:
    """One SAE app's device buffers."""

    def __init__(self, px, s, T, d):
        self.px, self.s, self.T = px, s, T
        self.W = px.xmix_sae_pack_encoder(dev(s.W_enc))
        self.be, self.bd = dev(s.b_enc), dev(s.b_dec)
        self.c = torch.empty(s.m, dtype=torch.float32, device="cuda")
        px.xmix_sae_fold_bias(self.W, self.be, self.bd, self.c)
        # NaN patterns: nothing of the workspace may be read before it is written
        self.ws = torch.full((px.sae_encode_workspace(T, d, s.m, s.k),), 0xFF, dtype=torch.uint8,
                             device="cuda")
        self.reset()

    def reset(self):
        self.idx = torch.full((self.T, self.s.k), -7, dtype=torch.int32, device="cuda")
        self.val = torch.zeros((self.T, self.s.k), dtype=torch.bfloat16, device="cuda")

    def single(self, h, rt, bit):
        self.px.xmix_sae_encode_topk(h, rt, bit, self.W, self.be, self.bd, self.c, self.s.k,
                                     self.idx, self.val, self.ws)

    def app(self, bit):
        return self.px.SaeApp(bit, self.W, self.be, self.bd, self.c, self.s.k, self.idx, self.val,
                              self.ws)

    def result(self):
        return self.idx.cpu().numpy(), torch_bits(self.val)


def route(px, T, sub, n_apps):
    rt = px.Route(T, n_apps)
    px.xmix_route_build(dev(np.arange(T, dtype=np.int32)),
                        torch.tensor([T], dtype=torch.int32, device="cuda"), dev(sub), rt,
                        torch.zeros(1, dtype=torch.int32, device="cuda"))
    return rt


# 16384, 16640, 32768 and 33024 latents: the last of each cut and the first of
# the next; widths of one window (256), of a number of windows that four does
# not divide (768, 1280), and with a remainder of every cut
@pytest.mark.parametrize("m,d,T,n", [
    (256, 256, 8, 1), (4096, 256, 33, 32), (4096, 768, 64, 33), (16384, 1280, 70, 64),
    (16384, 512, 128, 65), (16384, 256, 200, 129), (16384, 768, 512, 512),
    (16640, 768, 40, 31), (16640, 1280, 130, 130), (32768, 256, 512, 256), (32768, 512, 512, 257),
    (32768, 256, 400, 391), (33024, 512, 129, 128), (33024, 256, 129, 129), (33024, 768, 300, 257),
    (4096, 512, 513, 513), (1024, 256, 1024, 1000), (65536, 256, 140, 140)])
def test_decode_cuts_match_the_oracle(px, m, d, T, n):
    k = 32
    wl = synth.make("c3", d=d, m=m, k=k, T=T, n_sub=n, seed=m + T)
    s, hb = wl.layers[0].saes[0], wl.layers[0].h
    e, h = Enc(px, s, T, d), dev(hb)
    rt = route(px, T, wl.sub, 1)
    e.single(h, rt, 0)
    idx, val = e.result()
    toks = np.nonzero(wl.sub & 1)[0]
    assert np.all(idx[np.setdiff1d(np.arange(T), toks)] == -7)
    # the first and last token of every tile and wave share, and a few between
    at = sorted({0, n - 1} | {q for b in range(32, n, 32) for q in (b - 1, b)})
    sample = toks[at]
    ref, _, _, pre = oracle.sae_encode(hb, sample, s.W_enc, s.b_enc, s.b_dec, k, want_pre=True)
    for q, t in enumerate(sample):
        check_topk(idx[t], val[t], ref[q], pre[q], k)
    # every other token of the tile: as a batch of its own tokens alone
    few = np.zeros(T, np.uint32)
    few[toks[:: max(1, n // 20)]] = 1
    if n > 40:
        e2 = Enc(px, s, T, d)
        e2.single(h, route(px, T, few, 1), 0)
        i2, v2 = e2.result()
        rows = np.nonzero(few)[0]
        assert np.array_equal(i2[rows], idx[rows]) and np.array_equal(v2[rows], val[rows])


@pytest.mark.parametrize("T,p,ms", [(20, 0.5, (4096, 4096, 7680)), (300, 0.7, (16640, 4096, 33024)),
                                    (300, 0.3, (33024, 33024, 256)), (700, 0.5, (4096, 33024))])
@pytest.mark.parametrize("routed", [False, True])
def test_batched_cuts_match_single_calls(px, T, p, ms, routed):
    d, k = 256, 16
    wl = synth.make("c5", d=d, T=T, m=256, k=k, p=p, n_steer=1, n_probe=1, n_clamp_apps=len(ms))
    h = dev(wl.layers[0].h)
    saes = [synth.make("c3", d=d, m=m, k=k, T=2, n_sub=1, seed=i).layers[0].saes[0]
            for i, m in enumerate(ms)]
    enc = [Enc(px, s, T, d) for s in saes]
    rt = route(px, T, wl.sub, wl.n_apps)
    for i, e in enumerate(enc):
        e.single(h, rt, 2 + i)
    ref = [e.result() for e in enc]
    for e in enc:
        e.reset()
    if routed:
        rt2 = px.Route(T, wl.n_apps)
        px.xmix_route_sae_encode_topk_multi(
            dev(wl.req), torch.tensor([T], dtype=torch.int32, device="cuda"), dev(wl.sub), rt2,
            torch.zeros(1, dtype=torch.int32, device="cuda"), h,
            [e.app(2 + i) for i, e in enumerate(enc)])
        assert torch.equal(rt2.app_tokens, rt.app_tokens)
        assert torch.equal(rt2.app_count, rt.app_count)
        assert torch.equal(rt2.tok_mask, rt.tok_mask)
    else:
        px.xmix_sae_encode_topk_multi(h, rt, [e.app(2 + i) for i, e in enumerate(enc)])
    for e, (i, v) in zip(enc, ref):
        gi, gv = e.result()
        assert np.array_equal(gi, i) and np.array_equal(gv, v)
    for i, s in enumerate(saes):
        toks = np.nonzero((wl.sub >> np.uint32(2 + i)) & 1)[0][::29]
        r, _, _, pre = oracle.sae_encode(wl.layers[0].h, toks, s.W_enc, s.b_enc, s.b_dec, k,
                                         want_pre=True)
        for q, t in enumerate(toks):
            check_topk(ref[i][0][t], ref[i][1][t], r[q], pre[q], k)


@pytest.mark.parametrize("m,T,n_tied", [(4096, 6, 3), (16640, 40, 12)])
def test_repair_of_cut_slices(px, m, T, n_tied):
    """Whole 256-latent slices tied far above the rest: their parts report the
    bound, and the repair redoes whole slices."""
    d, k = 256, 16
    wl = synth.make("c3", d=d, m=m, k=k, T=T, n_sub=T, n_outliers=0)
    s = wl.layers[0].saes[0]
    W = s.W_enc.reshape(m, d).copy()
    row = synth.normal_bf16("t/row", (d,), 0.3)
    for q in range(n_tied):
        W[256 * (2 * q + 1):256 * (2 * q + 2)] = row
    s.W_enc, s.b_enc = W, np.zeros(m, np.uint16)
    hb = (synth.bf16_bits_to_f32(wl.layers[0].h) + 2 * np.sign(synth.bf16_bits_to_f32(row)))
    hb = torch.from_numpy(hb).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    e = Enc(px, s, T, d)
    e.single(dev(hb), route(px, T, wl.sub, 1), 0)
    idx, val = e.result()
    for t in range(T):       # the tie takes the lowest latents
        assert idx[t].tolist() == list(range(256, 256 + k))
        assert len(set(val[t].tolist())) == 1


@pytest.mark.parametrize("m,T,n", [(4096, 70, 64), (16384, 300, 200), (24576, 512, 300)])
def test_a_workspace_for_whole_slices(px, m, T, n):
    """A workspace that only holds whole slices is taken, by the single, the staged
    and the batched call, with the same results."""
    d, k = 512, 32
    wl = synth.make("c3", d=d, m=m, k=k, T=T, n_sub=n, seed=m)
    s, h, rt = wl.layers[0].saes[0], dev(wl.layers[0].h), route(px, T, wl.sub, 1)
    e = Enc(px, s, T, d)
    e.single(h, rt, 0)
    ref = e.result()
    cap = min(64, 4 * max(2, -(-2 * k * 256 // m) + 1))
    whole = m * 4 + -(-T * (m // 256) * (8 + 8 * cap) // 256) * 256
    assert whole < e.ws.numel()
    area = e.ws
    e.ws = area[:whole]
    guard = area[whole:].fill_(0x5A)
    for call in (lambda: e.single(h, rt, 0),
                 lambda: px.xmix_sae_encode_topk_multi(h, rt, [e.app(0)]),
                 lambda: (px.xmix_sae_encode_candidates(h, rt, 0, e.W, e.be, e.bd, e.c, k, e.ws),
                          px.xmix_sae_merge_topk(h, rt, 0, e.W, e.c, k, e.idx, e.val, e.ws))):
        e.reset()
        call()
        got = e.result()
        assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])
    assert bool((guard == 0x5A).all())


def test_workspace_of_every_cut_stays_in_the_static_array(px):
    """What xmix_sae_encode_topk_noalloc took with whole slices, it still takes."""
    for m in (256, 4096, 16384, 16640, 32768, 33024, 65536):
        for k in (1, 16, 64):
            for T in (1, 100, 512, 513, 1024):
                t = max(2, -(-2 * k * 256 // m) + 1)
                whole = m * 4 + T * (m // 256) * (8 + 8 * min(64, 4 * t))
                if whole <= px.XMIX_STATIC_SCRATCH_BYTES:
                    assert px.sae_encode_workspace(T, 4096, m, k) <= px.XMIX_STATIC_SCRATCH_BYTES


def tied(s, n_tied, d):
    """s with every second one of its first slices a single repeated row, which
    the merge can only settle by recomputing slices; the latents of its second half
    are those of the first with the halves of their rows exchanged."""
    W = s.W_enc.reshape(s.m, d).copy()
    W[s.m // 2:] = np.roll(W[:s.m // 2], d // 2, axis=1)
    row = synth.normal_bf16("t/tied", (d,), 0.06)
    for q in range(n_tied):
        W[256 * (2 * q + 1):256 * (2 * q + 2)] = row
    s.W_enc = W
    return s


@pytest.mark.parametrize("m,d,n_tied", [(4096, 768, 0), (4096, 256, 4), (16640, 512, 0),
                                        (16640, 256, 9), (33024, 256, 0), (65536, 256, 0)])
def test_a_token_is_encoded_alike_in_every_batch(px, m, d, n_tied):
    """One token's candidates come from narrow, whole, big or prefill tiles by the
    batch that it is in, and perhaps from a recomputed slice: the indices and
    values are the same bits.  The two halves of a token's row are equal, so that
    every latent has a twin whose pre-activation differs by the rounding of its sum
    alone: another order of summation shows in the indices."""
    k, n = 24, 1100
    wl = synth.make("c3", d=d, m=m, k=k, T=n, n_sub=n, seed=m + d)
    rows = wl.layers[0].h.copy()
    rows[:, d // 2:] = rows[:, :d // 2]
    s, h = tied(wl.layers[0].saes[0], n_tied, d), dev(rows)
    enc = {T: Enc(px, s, T, d) for T in (8, 60, 100, 128, 200, 400, 512, 700, 1024, n)}
    e = enc[n]
    e.single(h, route(px, n, np.ones(n, np.uint32), 1), 0)   # prefill
    idx, val = e.result()
    for T, e in enc.items():
        for live in {T, max(1, T // 3), max(1, T - 70)}:
            first = (37 * T + live) % (n - T + 1)
            sub = np.zeros(T, np.uint32)
            sub[:live] = 1
            e.reset()
            e.single(h[first:first + T].contiguous(), route(px, T, sub, 1), 0)
            i, v = e.result()
            rows = slice(first, first + live)
            assert np.array_equal(i[:live], idx[rows]) and np.array_equal(v[:live], val[rows]), (T, live)
    # beside other apps, which leave the batch fewer cuts
    for T in (60, 400):
        e, others = enc[T], [Enc(px, s, T, d) for _ in range(4)]
        e.reset()
        px.xmix_sae_encode_topk_multi(h[:T].contiguous(), route(px, T, np.full(T, 31, np.uint32), 5),
                                      [e.app(0)] + [o.app(1 + q) for q, o in enumerate(others)])
        i, v = e.result()
        assert np.array_equal(i, idx[:T]) and np.array_equal(v, val[:T])
