"""gemm_xs_kernel (16x16 MFMAs) on the CPU: no spill traffic where its waits are hand-counted, the
designed instruction mix of its main loops, and the index formulas of its LDS tiles, restated."""
import re

import pytest

from test_kernel_build import _blocked_decode, _blocked_from_k, _main_loop, asm  # noqa: F401

TYPES = ("DF16b", "DF16_", "f")
VARIANTS = [(0, 0, 0), (0, 0, 1), (1, 0, 0), (1, 0, 1), (2, 1, 0), (3, 2, 0)]  # epilogue, A layout, K check
# BM, BN, waves along M and N.
TILES = {"Tile256": (256, 256, 2, 4), "Tile128": (128, 256, 1, 4), "Tile64": (64, 64, 2, 2),
         "Tile128x64": (128, 64, 1, 2)}
# fp32 runs 64 x 64 and 128 x 256 alone; 128 x 64 is for logits.
KERNELS = [(t, e, a, c, tile) for t in TYPES for e, a, c in VARIANTS for tile in TILES
           if (t != "f" or tile in ("Tile64", "Tile128")) and (tile != "Tile128x64" or e < 2)]


def test_only_reachable_tiles_are_built(asm):  # noqa: F811
    assert not re.search(r"^_ZN3lce14gemm_xb_kernelIf", asm, re.M)
    built = set(re.findall(r"^_ZN3lce14gemm_xs_kernelIfLi\d+ELi\d+ELb\dENS_4TileILi(\d+)ELi(\d+)E", asm, re.M))
    assert built == {("64", "64"), ("128", "256")}


@pytest.mark.parametrize("t,e,a,c,tile", KERNELS)
def test_main_loop(asm, t, e, a, c, tile):  # noqa: F811
    bm, bn, wm, wn = TILES[tile]
    name = (f"_ZN3lce14gemm_xs_kernelI{t}Li{e}ELi{a}ELb{c}ENS_4TileILi{bm}ELi{bn}ELi{wm}ELi{wn}EEEEEvNS_8GemmArgsE")
    code = _main_loop(asm, name, with_prologue=True)
    assert not [x for x in code if x.startswith("scratch_") or re.match(r"buffer_(load|store)\S*\s.*\boff\b", x)]
    loop = _main_loop(asm, name)
    count = lambda f: sum(1 for x in loop if f(x))  # noqa: E731
    ni, nj, nl = bm // wm // 16, bn // wn // 16, bm // (8 * wm * wn)
    # Two K-tiles per trip, two K-quads each; fp32 takes four MFMA steps per K-quad.
    assert count(lambda x: x.startswith("v_mfma")) == 4 * ni * nj * (4 if t == "f" else 1)
    assert count(lambda x: x.startswith("buffer_load") and x.endswith("lds")) == 2 * nl
    assert count(lambda x: x.startswith("buffer_load") and not x.endswith("lds")) == 4 * nj
    assert count(lambda x: x.startswith("ds_read_b64_tr_b16")) == (8 * ni if t != "f" and a else 0)


@pytest.mark.parametrize("t", ["DF16b", "DF16_"])
@pytest.mark.parametrize("tile", ["Tile256", "Tile128", "Tile64"])
def test_dw_preload_is_in_flight_together(asm, t, tile):  # noqa: F811
    """The earlier chunks' dW of an accumulating tile: every piece requested before any is waited for."""
    bm, bn, wm, wn = TILES[tile]
    name = f"_ZN3lce14gemm_xs_kernelI{t}Li3ELi2ELb0ENS_4TileILi{bm}ELi{bn}ELi{wm}ELi{wn}EEEEEvNS_8GemmArgsE"
    code = _main_loop(asm, name, with_prologue=True)
    code = code[:next(i for i, x in enumerate(code) if x.startswith("buffer_load") and x.endswith("lds"))]
    loads = [i for i, x in enumerate(code) if re.match(r"(global|buffer)_load_dwordx4", x)]
    assert len(loads) == bm // wm // 16 * (bn // wn // 16) // 2
    assert not [x for x in code[loads[0]:loads[-1]] if x.startswith("s_waitcnt") and "vmcnt" in x]


def _swz_k(r):
    return (r ^ (r >> 3)) & 7


def _swz_mn16(bm, k):
    if bm == 64:
        return (2 if k & 2 else 0) ^ (4 if k & 8 else 0)
    return (2 if k & 1 else 0) ^ (4 if k & 2 else 0) ^ (8 if k & 8 else 0)


def _transposed(got):
    """What lane l receives of a ds_read_b64_tr_b16: in its 16-lane group, element l%4 of lanes 4e + (l%16)/4."""
    return {l: [got[16 * (l >> 4) + 4 * e + (l & 15) // 4][l % 4] for e in range(4)] for l in range(64)}


def _conflict_free(addrs, size):
    """Each half of the wave (32 lanes of `size` bytes) covers every 4-byte bank of 256 bytes at most
    size / 8 times (b64 reads: once)."""
    for half in (addrs[:32], addrs[32:]):
        banks = [(x // 4 + i) % 64 for x in half for i in range(size // 4)]
        assert max(banks.count(b) for b in set(banks)) <= size // 8


@pytest.mark.parametrize("tile", TILES)
def test_k_contiguous_tile(tile):
    bm, _, wm, wn = TILES[tile]
    kw, nl = wm * wn, bm // (8 * wm * wn)
    stored = {}
    for w in range(kw):
        for j in range(nl):
            for l in range(64):
                slot_x = (l & 7) ^ (l >> 3) ^ ((nl * w) & 7)
                stored[(nl * w + j) * 1024 + 16 * l] = (8 * nl * w + (l >> 3) + 8 * j, slot_x ^ j)
    assert len(stored) == bm * 8
    for m in range(wm):
        wsub = m * (bm // wm)
        for i in range(bm // wm // 16):
            for u in range(2):
                for l in range(64):
                    r = wsub + (l & 15)
                    xa = r * 128 + (((l >> 4) ^ _swz_k(r) ^ ((4 * u) ^ (2 * i % 8))) << 4)
                    assert stored[xa + 2048 * i] == (r + 16 * i, 4 * u + (l >> 4))


@pytest.mark.parametrize("tile", ["Tile256", "Tile128", "Tile64"])
def test_mn_contiguous_16bit_tile(tile):
    bm, _, wm, wn = TILES[tile]
    kw, nl, pitch = wm * wn, bm // (8 * wm * wn), 2 * bm
    lanes, rows = pitch // 16, 1024 // pitch
    xor_j = {256: lambda j: 4 if j & 1 else 0, 128: lambda j: 8 if j & 2 else 0, 64: lambda j: 4 if j else 0}[bm]
    stored = {}
    for w in range(kw):
        for j in range(nl):
            for l in range(64):
                kr = 64 // kw * w + rows * j + l // lanes
                slot = (l % lanes) ^ _swz_mn16(bm, (64 // kw * w) | (l // lanes)) ^ xor_j(j)
                for e in range(8):
                    stored[(nl * w + j) * 1024 + 16 * l + 2 * e] = (kr, 8 * slot + e)
    for m in range(wm):
        wsub = m * (bm // wm)
        for i in range(bm // wm // 16):
            for u in range(2):
                got = [{}, {}]
                for s in range(2):
                    addrs = []
                    for l in range(64):
                        g, ip = l >> 4, l & 15
                        r0 = 8 * g + (ip >> 2)
                        slot = (wsub // 8 + 2 * i + ((ip & 3) >> 1)) ^ _swz_mn16(bm, r0)
                        addrs.append(r0 * pitch + 16 * slot + 8 * (ip & 1) + (32 * u + 4 * s) * pitch)
                        got[s][l] = [stored[addrs[-1] + 2 * e] for e in range(4)]
                    _conflict_free(addrs, 8)
                lo, hi = _transposed(got[0]), _transposed(got[1])
                for l in range(64):
                    k0 = 32 * u + 8 * (l >> 4)
                    assert lo[l] + hi[l] == [(k0 + k, wsub + 16 * i + (l & 15)) for k in range(8)]


@pytest.mark.parametrize("tile", ["Tile256", "Tile128", "Tile64"])
def test_blocked_16bit_tile(tile):
    bm, _, wm, wn = TILES[tile]
    kw, nl = wm * wn, bm // (8 * wm * wn)
    stored = {}  # LDS byte -> (token, id): piece P of fragment (b, c) is token 32 b + P%32, ids 16 c + 8 (P/32) ..
    for w in range(kw):
        for j in range(nl):
            b, c = w // (kw // 2), (w % (kw // 2)) * nl + j
            for l in range(64):
                piece = l ^ (4 * (l >> 5))
                for e in range(8):
                    stored[(nl * w + j) * 1024 + 16 * l + 2 * e] = (32 * b + piece % 32, 16 * c + 8 * (piece // 32) + e)
    for m in range(wm):
        wsub = m * (bm // wm)
        for i in range(bm // wm // 16):
            for u in range(2):
                got = [{}, {}]
                for s in range(2):
                    addrs = []
                    for l in range(64):
                        g, ip = l >> 4, l & 15
                        h = (ip & 3) >> 1
                        xa = (wsub // 16) * 1024 + 16 * (8 * g + (ip >> 2) + 4 * h + 32 * h) + 8 * (ip & 1)
                        addrs.append((xa ^ (64 * s)) + 64 * bm * u + 1024 * i)
                        got[s][l] = [stored[addrs[-1] + 2 * e] for e in range(4)]
                    _conflict_free(addrs, 8)
                lo, hi = _transposed(got[0]), _transposed(got[1])
                for l in range(64):
                    k0 = 32 * u + 8 * (l >> 4)
                    assert lo[l] + hi[l] == [(k0 + k, wsub + 16 * i + (l & 15)) for k in range(8)]


@pytest.mark.parametrize("esz", [2, 4])
def test_blocked_b_fragment(esz):
    """A 16-column fragment's loads find chunk l/16 of column l%16 of the K-quad in the 32-column layout."""
    N, K = 64, 256 // esz
    KP, NB = K * esz // 32, N // 32
    layout = _blocked_from_k(N, K, esz, KP, NB)  # byte of a 16-byte piece -> (column, first K)
    for j in range(4):
        for u in range(KP // 2):
            for l in range(64):
                off = (l >> 5) * 1024 + (((l >> 4) & 1) * 32 + (l & 15)) * 16 + (j & 1) * 256
                off += ((j >> 1) * KP + 2 * u) * 1024
                assert layout[off] == (16 * j + (l & 15), (64 * u + 16 * (l >> 4)) // esz)


def test_regroup16():
    """v_permlane32_swap then v_permlane16_swap give lane group g elements 8g .. 8g + 7; backwards, the start."""
    def swap(a, b, width):  # odd groups of `width` lanes of a with the even ones of b
        a, b = list(a), list(b)
        for l in range(64):
            if (l // width) % 2 == 0:
                a[l + width], b[l] = b[l], a[l + width]
        return a, b
    for e in range(2):  # dword e of a lane's x (its group's elements 4g ..) and y (16 + 4g ..)
        x = [(l & 15, 4 * (l >> 4) + 2 * e) for l in range(64)]
        y = [(l & 15, 16 + 4 * (l >> 4) + 2 * e) for l in range(64)]
        lo, hi = swap(*swap(x, y, 32), 16)
        assert lo == [(l & 15, 8 * (l >> 4) + 2 * e) for l in range(64)]
        assert hi == [(l & 15, 8 * (l >> 4) + 4 + 2 * e) for l in range(64)]
        assert swap(*swap(lo, hi, 16), 32) == (x, y)


@pytest.mark.parametrize("tile", ["Tile128", "Tile64"])
@pytest.mark.parametrize("KP", [32, 16032])
def test_blocked_fp32_loader_fetches_the_mn_loaders_pieces(tile, KP):
    """fp32 blocked A: load j of wave w, lane l fetches the piece (K-row, ids) that the MN-contiguous loader puts
    in the same LDS slot, inside the descriptor's range (the tile's ids in the K-tile's one token block), and the
    fragment reads find their rows."""
    bm, _, wm, wn = TILES[tile]
    kw, nl, esz, pitch = wm * wn, bm // (8 * wm * wn), 4, 4 * bm
    lanes, rows = pitch // 16, 1024 // pitch
    stored = {}
    for w in range(kw):
        for j in range(nl):
            for l in range(64):
                kr = 32 // kw * w + l // lanes
                off = kr * 16 + j * rows * 16 + ((l % lanes) << 9)
                assert _blocked_decode(off, KP, esz) == (kr + rows * j, 4 * (l % lanes))
                assert off + 16 <= bm * esz * 32
                for e in range(4):
                    stored[(nl * w + j) * 1024 + 16 * l + 4 * e] = (kr + rows * j, 4 * (l % lanes) + e)
    assert len(stored) == 32 * bm
    for m in range(wm):
        wsub = m * (bm // wm)
        for i in range(bm // wm // 16):
            for u in range(2):
                for l in range(64):
                    for s in range(4):
                        at = 4 * (l >> 4) * pitch + (wsub + (l & 15)) * 4 + (16 * u + s) * pitch + 64 * i
                        assert stored[at] == (16 * u + 4 * (l >> 4) + s, wsub + 16 * i + (l & 15))


@pytest.mark.parametrize("esz", [2, 4])
def test_lse_epilogue_stores_e_blocked(esz):
    """The LSE_BWD epilogue of a wave at (mw, nw): the token and first id of every 16-byte piece that lane l stores
    for blocks i (16-bit: i and i + 1) and j."""
    KP = 64 if esz == 2 else 128
    for mw, nw in ((0, 0), (32, 32), (128, 192), (768, 224)):
        for j in range(4):
            for i in range(0, 8, 2 if esz == 2 else 1):
                for l in range(64):
                    g, r16 = l >> 4, l & 15
                    e_blk = ((nw + 16 * j) >> 5) * KP * 1024 + (l >> 5) * 1024
                    e_blk += ((g & 1) * 32 + r16 + 16 * (j & 1)) * 16
                    off = e_blk + ((mw + 16 * i) >> (4 if esz == 2 else 3)) * 1024
                    ids = 8 * g if esz == 2 else 4 * g  # 16-bit: after regroup16, 8 ids of the 32 of two blocks
                    assert _blocked_decode(off, KP, esz) == (nw + 16 * j + r16, mw + 16 * i + ids)
