"""CPU replica of what the FP32 part products and the row kernels copy and
read (csrc/stream.hip, tile.hip, rows.hip), beside test_dma_maps.py, whose
operand classes it uses:

* the three-part table SK3: its slots, fragments and global addresses;
* every tile of the streaming core, taken from the source: its waves' share of
  each stage's DMA, its addresses for the workloads' shapes, its ring and wait
  counts replayed in issue order, its LDS;
* the short-reduction kernel in FP32 (eight waves, three-part tiles) and the
  split of a row block's columns over blocks;
* the SH row kernel's copies between rows and LDS rows with padding;
* the register-staged core's 16-byte reads of lines and rows.
"""
import os
import re

import pytest

from test_dma_maps import (KS, LAYERS, SBK, SKc, SKh, VOXELS, astat_ok, check_k_contiguous, pad32, tile_starts)

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1808_01517_amd", "csrc")
LDS_PER_CU = 160 * 1024


def source(name):
    return open(os.path.join(CSRC, name)).read()


def tiles():
    """(BM, BN, waves, ring) of every SCfg in the source."""
    found = {tuple(int(x) for x in m) for m in re.findall(r"SCfg<(\d+), (\d+), (\d+), (\d+), (\d+)>", source("stream.hip"))}
    return sorted((bm, bn, wm * wn, ns) for bm, bn, wm, wn, ns in found)


F32_TILES = [(256, 144, 8, 2), (256, 96, 8, 2), (64, 144, 4, 2), (128, 48, 4, 3), (64, 48, 4, 4)]
BF16_TILES = [(128, 144, 4, 3), (128, 48, 4, 3), (256, 96, 4, 3), (64, 48, 4, 8)]


def test_the_tiles_are_those_of_the_source():
    assert tiles() == sorted(set(F32_TILES + BF16_TILES))


class SK3:
    """Three bfloat16 parts per row, each as SKh: part i of (r, k) at
    p[r * 3 ldp + i ldp + k]; LDS holds the parts' tiles one after another."""

    def __init__(self, ldp, rows):
        self.ld, self.rows = ldp, rows
        self.unit = 16
        self.esize = 2

    def slots(self, BR):
        return 3 * BR * SBK * 2 // 16

    def prk(self, s, BR):
        part, q = divmod(s, BR * 4)
        r = q >> 2
        return part, r, 8 * ((q & 3) ^ ((r >> 1) & 3))

    def lane_off(self, s, r0, BR):
        part, r, k = self.prk(s, BR)
        gr = r0 + r if r0 + r < self.rows else self.rows - 1
        return ((gr - r0) * 3 * self.ld + part * self.ld + k) * 2

    def base(self, r0, k0):
        return (r0 * 3 * self.ld + k0) * 2

    def frag3(self, BR, rg, q16, g4):
        r = rg * 16 + q16
        at = r * SBK + ((g4 ^ ((r >> 1) & 3)) << 3)
        return [[(i * BR * SBK + at + e, (i, r, 8 * g4 + e)) for e in range(8)] for i in range(3)]


@pytest.mark.parametrize("BR", [32, 48, 96, 144])
def test_three_part_stage(BR):
    op = SK3(160, 4096)
    lds = {}
    for s in range(op.slots(BR)):
        part, r, k = op.prk(s, BR)
        for e in range(8):
            assert 8 * s + e not in lds
            lds[8 * s + e] = (part, r, k + e)
    assert set(lds.values()) == {(p, r, k) for p in range(3) for r in range(BR) for k in range(SBK)}
    for rg in range(BR // 16):
        for q16 in range(16):
            for g4 in range(4):
                for part in op.frag3(BR, rg, q16, g4):
                    for at, want in part:
                        assert lds[at] == want


@pytest.mark.parametrize("layer", LAYERS)
@pytest.mark.parametrize("BN", [32, 48, 96, 144])
def test_three_part_addresses(layer, BN):
    C, O, Ki, Ko = layer
    for K, N in ((C * Ki, O * Ko), (O * Ko, C * Ki)):
        if BN == 32 and not astat_ok(K, N):
            continue
        ld = pad32(K)
        op = SK3(ld, N)
        for r0 in tile_starts(N, BN):
            for k0 in sorted({0, (ld // SBK - 1) * SBK}):  # the padded table is copied whole
                for s in range(op.slots(BN)):
                    o = op.lane_off(s, r0, BN)
                    a = op.base(r0, k0) + o
                    assert 0 <= o < 2 ** 32 and 0 <= a and a + 16 <= N * 3 * ld * 2


@pytest.mark.parametrize("V", VOXELS)
def test_activation_addresses_of_every_tile(V):
    for C, O, Ki, Ko in LAYERS:
        for K in (C * Ki, O * Ko):
            for BM in sorted({t[0] for t in F32_TILES + BF16_TILES}):
                if K % 4 == 0:
                    check_k_contiguous(SKc(True, K, V), BM, V, K, V * K * 4)
                elif BM == 256:
                    check_k_contiguous(SKc(False, K, V), BM, V, K, V * K * 4)
                if K % 8 == 0:
                    check_k_contiguous(SKh(K, V), BM, V, K, V * K * 2)


def operands(tile, f32):
    """The (A, B) slot counts a tile of that precision is used with."""
    bm, bn = tile[:2]
    b = SK3(4096, 4096) if f32 else SKh(4096, 4096)
    for a in (SKc(True, 4096, 4096), SKc(False, 4096, 4096)) + (() if f32 else (SKh(4096, 4096),)):
        yield a.slots(bm), b.slots(bn), bm * SBK * a.esize, b.slots(bn) * 16


@pytest.mark.parametrize("tile,f32", [(t, True) for t in F32_TILES] + [(t, False) for t in BF16_TILES])
def test_rings_and_waits(tile, f32):
    """Each wave's instructions of a stage are wave, wave + NW, ..; its waits
    allow at most what it issued after the stage it waits for, and a slot is
    refilled only after the barrier behind its last read."""
    bm, bn, NW, ns = tile
    for sa, sb, abytes, bbytes in operands(tile, f32):
        nia, nib = (sa + 63) // 64, (sb + 63) // 64
        niw = nia // NW + nib // NW
        NS = ns if (ns - 2) * niw < 64 else 2
        D = NS - 1
        assert (D - 1) * niw < 64 and NS * (abytes + bbytes) <= LDS_PER_CU
        covered = sorted(i for w in range(NW) for i in range(w, nia, NW))
        assert covered == list(range(nia))
        for wave in range(NW):
            per = len(range(wave, nia, NW)) + len(range(wave, nib, NW))
            assert per >= niw
            for niter in (0, 1, 2, 3, D, D + 1, 2 * D + 3):
                log, held = [], {}

                def issue(it, log=log, held=held, per=per, NS=NS):
                    held[it % NS] = it
                    log += [it] * per

                for s in range(min(D, niter)):
                    issue(s)
                for it in range(niter):
                    imm = (D - 1) * niw if it + D <= niter else 0
                    last = max(i for i, x in enumerate(log) if x == it)
                    assert imm <= len(log) - 1 - last, (wave, it, imm)
                    if it + D < niter:
                        assert held.get((it + D) % NS, it - 1) == it - 1  # read before this barrier
                        issue(it + D)
                    assert held[it % NS] == it


def test_short_reductions_in_three_parts():
    BN, ldb, N, NW, TM, D = 32, 160, 1440, 8, 2, 1
    text = source("stream.hip")
    assert re.search(r"constexpr int NW = F32 \? 8 : 4;", text) and "#define DLM_ASTAT_D_F32 1" in text
    op = SK3(ldb, N)
    ni = op.slots(BN) // 64
    nit = KS * ni
    slab = op.slots(BN) * 16
    seen, top = set(), 0
    for wave in range(NW):
        for q in range(wave, nit, NW):
            sl, ins = divmod(q, ni)
            for lane in range(64):
                s = ins * 64 + lane
                lds = sl * slab + ins * 1024 + 16 * lane
                assert lds not in seen
                seen.add(lds)
                part, r, k = op.prk(s, BN)
                glob = op.lane_off(s, 0, BN) + sl * SBK * 2
                assert glob == (r * 3 * ldb + part * ldb + SBK * sl + k) * 2
                top = max(top, glob)
    assert sorted(seen) == list(range(0, KS * slab, 16))
    assert (N // BN - 1) * BN * 3 * ldb * 2 + top + 16 <= N * 3 * ldb * 2
    side = 1440 * 4 + 16 * TM * NW * (1440 // 16) * 2
    assert (D + 1) * KS * slab + side <= LDS_PER_CU
    # waits: after the DMA of tile t the wave issued the stores of tile t - 1
    stores = TM * BN // 16
    for tiles_ in (1, 2, 3, 45):
        for wave in range(NW):
            nq = len(range(wave, nit, NW))
            log = [("dma", 0)] * nq
            for t in range(tiles_):
                if t >= D:
                    last = max(i for i, e in enumerate(log) if e == ("dma", t))
                    assert stores <= len(log) - 1 - last
                if t + D < tiles_:
                    log += [("dma", t + D)] * nq
                log += [("st", t)] * stores


@pytest.mark.parametrize("columns", [32, 96, 448, 1440])
@pytest.mark.parametrize("blocks", [1, 3, 32, 255, 256])
def test_row_blocks_share_their_columns(columns, blocks):
    tiles_ = columns // 32
    share = min(256 // blocks, tiles_) if blocks < 256 else 1
    got = []
    for y in range(share):
        t0 = tiles_ * y // share
        got += range(t0, tiles_ * (y + 1) // share)
    assert got == list(range(tiles_))


# ------------------------------------------------------------- SH row kernel
def stride(n):
    return n + 4 if n % 8 == 0 else n


def magic(d):
    return 0 if d < 2 else ((1 << 32) + d - 1) // d


@pytest.mark.parametrize("n", [1, 3, 4, 7, 8, 16, 45, 90, 96, 135, 270, 272, 384, 504, 512])
def test_row_copies(n):
    """Every LDS element of nv rows is copied once, from its own place, and
    nothing beyond the rows is read; pieces are found by the magic division."""
    st = stride(n)
    for nv in (1, 2, 31, 32, 64, 96):
        if nv * st * 4 > 64 * 1024:
            continue
        mg, cs, last = magic(st // 4), st >> 2, (n >> 2) - 1
        lds = {}
        for i in range(nv * st >> 2):
            src = 4 * i
            if st != n:
                r = i * mg >> 32
                assert r == i // cs
                c = i - r * cs
                src = r * n + 4 * min(c, last)
            assert src + 4 <= nv * n
            for e in range(4):
                lds[4 * i + e] = src + e
        for t in range(nv * st & 3):
            lds[4 * (nv * st >> 2) + t] = 4 * (nv * st >> 2) + t
        for r in range(nv):
            for k in range(n):
                assert lds[r * st + k] == r * n + k
        out = {}
        mg, cs = magic(n // 4), n >> 2
        for i in range(nv * n >> 2):
            at = 4 * i
            if st != n:
                r = i * mg >> 32
                assert r == i // cs
                at = r * st + 4 * (i - r * cs)
            for e in range(4):
                out[4 * i + e] = lds[at + e]
        for t in range(nv * n & 3):
            out[4 * (nv * n >> 2) + t] = lds[4 * (nv * n >> 2) + t]
        assert out == {i: i for i in range(nv * n)}


# ------------------------------------------------- register-staged core
TBK = 32


def runs(items, NT):
    per = (items + NT - 1) // NT
    for tid in range(NT):
        for i in range(per):
            e = tid + i * NT
            yield tid, i, e if e < items else items - 1


@pytest.mark.parametrize("BR,NT,rows,lines", [
    (128, 256, 1, 40), (128, 256, 3, 33), (128, 256, 135, 64), (144, 256, 136, 95), (144, 256, 4, 70), (256, 512, 300, 45),
    (64, 256, 5, 32), (144, 256, 143, 32), (128, 256, 129, 31),
])
def test_line_reads_stay_inside(BR, NT, rows, lines):
    """Lines: 16-byte runs along the rows of k-lines, ld = rows; a stage is read
    without a look at any bound only where whole() allows it."""
    ld, items = rows, TBK * BR // 4
    step = NT // (BR // 4) if NT % (BR // 4) == 0 and items % NT == 0 else 0
    for r0 in range(0, rows + 1, BR):
        for k0 in range(0, lines, TBK):
            kend = lines
            whole = ld >= 4 and k0 + TBK <= min(kend, lines - 1)
            for tid, i, e in runs(items, NT):
                row, k = 4 * (e % (BR // 4)), e // (BR // 4)
                if step:  # one offset for all of a thread's runs
                    f = tid
                    assert row == 4 * (f % (BR // 4)) and k == f // (BR // 4) + i * step
                if whole:
                    o = (k0 + k) * ld + min(r0 + row, rows - 1)
                    assert 0 <= o and o + 4 <= lines * ld
                else:
                    for j in range(4):
                        o = min(k0 + k, kend - 1) * ld + min(r0 + row + j, rows - 1)
                        assert 0 <= o < lines * ld


@pytest.mark.parametrize("BR,NT,rows,P", [(128, 256, 135, 33), (144, 256, 136, 64), (144, 256, 1, 100), (128, 256, 129, 31)])
def test_row_reads_stay_inside(BR, NT, rows, P):
    """Rows: 16-byte runs along k of rows of P."""
    for r0 in range(0, rows + 1, BR):
        for k0 in range(0, P, TBK):
            whole = k0 + TBK <= P
            for _, _, e in runs(BR * TBK // 4, NT):
                r, k = min(r0 + e // (TBK // 4), rows - 1), k0 + 4 * (e % (TBK // 4))
                if whole:
                    assert r * P + k + 4 <= rows * P
                else:
                    for j in range(4):
                        assert min(k + j, P - 1) < P
