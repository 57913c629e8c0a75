"""Candidate emission of the encode at the edges of its plan, against the oracle."""
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


@pytest.mark.parametrize("m,k", [(256, 8), (512, 64), (768, 64), (1024, 64), (2048, 32), (4096, 8),
                                 (4096, 64), (8192, 64), (16384, 64)])
@pytest.mark.parametrize("T", [70, 1030])
def test_encode_emission_plans(px, m, k, T):
    """Shares of the winners per 256-latent tile from a whole tile down to one
    value, with and without a lower bound on a tile's count."""
    wl = synth.make("c3", d=256, m=m, k=k, T=T, n_sub=60, seed=m + k)
    s, h = wl.layers[0].saes[0], wl.layers[0].h
    rt = px.Route(T, 1)
    px.xmix_route_build(dev(wl.req), torch.tensor([T], dtype=torch.int32, device="cuda"),
                        dev(wl.sub), rt, torch.zeros(1, dtype=torch.int32, device="cuda"))
    W = px.xmix_sae_pack_encoder(dev(s.W_enc))
    idx = torch.full((T, k), -7, dtype=torch.int32, device="cuda")
    val = torch.zeros((T, k), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(px.sae_encode_workspace(T, 256, m, k), dtype=torch.uint8, device="cuda")
    px.xmix_sae_encode_topk(dev(h), rt, 0, W, dev(s.b_enc), dev(s.b_dec), None, k, idx, val, ws)
    toks = oracle.route(wl.req, T, wl.sub, 1)[2][0][:60]
    idx_ref, _, _, pre = oracle.sae_encode(h, toks, s.W_enc, s.b_enc, s.b_dec, k, want_pre=True)
    gi, gv = idx.cpu().numpy(), torch_bits(val)
    for q, t in enumerate(toks):
        check_topk(gi[t], gv[t], idx_ref[q], pre[q], k)


# few tiles (128-token ones), the last count and dictionary that take them, and
# more: 65 slices x 1030 tokens are 585 tiles of 128, 65 x 1537 would be 845
@pytest.mark.parametrize("m,n,T", [(256, 1, 1025), (1024, 127, 1100), (1024, 128, 1100),
                                   (1024, 129, 1100), (2048, 257, 1100), (16640, 1030, 1030),
                                   (16640, 1537, 1600), (16640, 1536, 1600), (33024, 1030, 1100)])
def test_prefill_tile_sizes(px, m, n, T):
    d, k = 256, 16
    wl = synth.make("c3", d=d, m=m, k=k, T=T, n_sub=n, seed=m + n)
    s, h = wl.layers[0].saes[0], wl.layers[0].h
    rt = px.Route(T, 1)
    px.xmix_route_build(dev(wl.req), torch.tensor([T], dtype=torch.int32, device="cuda"),
                        dev(wl.sub), rt, torch.zeros(1, dtype=torch.int32, device="cuda"))
    W = px.xmix_sae_pack_encoder(dev(s.W_enc))
    idx = torch.full((T, k), -7, dtype=torch.int32, device="cuda")
    val = torch.zeros((T, k), dtype=torch.bfloat16, device="cuda")
    # NaN patterns: staged rows past the live tiles are not written, nor read
    ws = torch.full((px.sae_encode_workspace(T, d, m, k),), 0xFF, dtype=torch.uint8, device="cuda")
    px.xmix_sae_encode_topk(dev(h), rt, 0, W, dev(s.b_enc), dev(s.b_dec), None, k, idx, val, ws)
    toks = np.nonzero(wl.sub & 1)[0]
    gi, gv = idx.cpu().numpy(), torch_bits(val)
    assert np.all(gi[np.setdiff1d(np.arange(T), toks)] == -7)
    at = sorted({0, n - 1} | {q for b in range(64, n, 64) for q in (b - 1, b)})
    ref, _, _, pre = oracle.sae_encode(h, toks[at], s.W_enc, s.b_enc, s.b_dec, k, want_pre=True)
    for q, t in enumerate(toks[at]):
        check_topk(gi[t], gv[t], ref[q], pre[q], k)
