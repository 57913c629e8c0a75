"""Host-side checks of the encode kernels' workgroup-to-tile maps.

The launch grids and the slot -> (latent tile, token tile) maps below are
the ones the encode kernels compute from blockIdx; every tile of the
problem must be visited exactly once and no slot may land outside it."""
import numpy as np
import pytest


def decode_map(n, n_nt, grid):
    """sae_stream_kernel and sae_stream_apps_kernel: workgroup w runs units w,
    w + grid, ...; the token tiles of eight slices are laid together, the slices
    fastest."""
    for w in range(grid):
        for u in range(w, n * n_nt, grid):
            if n_nt == 1:
                yield u, 0
                continue
            grp = u // (8 * n_nt)
            r = u - grp * 8 * n_nt
            width = min(8, n - 8 * grp)
            yield 8 * grp + r % width, r // width


def prefill_map(n_mt, n_nt, bt_=8, bl_=4):
    """sae_gemm_kernel: 256 latents x 256 tokens per tile, in XCD blocks."""
    m8 = (n_mt + 7) // 8
    nbt = (n_nt + bt_ - 1) // bt_
    nbl = (m8 + bl_ - 1) // bl_
    for L in range(8 * nbt * nbl * bt_ * bl_):
        xcd, slot = L % 8, L // 8
        b, p = slot // (bt_ * bl_), slot % (bt_ * bl_)
        bt, bl = b % nbt, b // nbt
        lt, nt = bl_ * bl + p // bt_, bt_ * bt + p % bt_
        if nt >= n_nt or lt >= m8:
            continue
        mt = xcd * m8 + lt
        if mt < n_mt:
            yield mt, nt


def _cover(gen, n_mt, n_nt):
    seen = np.zeros((n_mt, n_nt), np.int32)
    for mt, nt in gen:
        assert 0 <= mt < n_mt and 0 <= nt < n_nt
        seen[mt, nt] += 1
    return seen


@pytest.mark.parametrize("m,T", [(256, 1), (65536, 256), (65536, 512), (1024, 300), (768, 1000),
                                 (131072, 1024), (2560, 4000)])
@pytest.mark.parametrize("cut,tok", [(1, 128), (1, 256), (2, 128), (4, 128)])
def test_decode_map_covers_every_tile_once(m, T, cut, tok):
    n, n_nt = m // 256 * cut, (T + tok - 1) // tok
    for grid in {n, min(256, n * n_nt), 7}:
        assert (_cover(decode_map(n, n_nt, grid), n, n_nt) == 1).all()


@pytest.mark.parametrize("m,T", [(2048, 300), (65536, 512), (2560, 1000), (18688, 400)])
def test_token_tiles_of_a_slice_share_an_xcd(m, T):
    """Workgroups are dealt to the 8 XCDs in turn: of the full groups of eight
    slices, every token tile of a slice runs on the same one."""
    n, n_nt = m // 256, (T + 127) // 128
    xcd = {}
    for u in range(n // 8 * 8 * n_nt):
        grp, r = divmod(u, 8 * n_nt)
        xcd.setdefault(8 * grp + r % 8, set()).add(u % 8)
    assert len(xcd) == n // 8 * 8 and all(len(x) == 1 for x in xcd.values())


@pytest.mark.parametrize("m,T", [(256, 1025), (1024, 1500), (2048, 2100), (2560, 1025),
                                 (131072, 8192), (65536, 3000), (768, 1300)])
def test_prefill_map_covers_every_tile_once(m, T):
    n_mt, n_nt = m // 256, (T + 255) // 256
    assert (_cover(prefill_map(n_mt, n_nt), n_mt, n_nt) == 1).all()
