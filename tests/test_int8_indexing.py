"""Host-side replay of the streaming kernel's int8 form (k_wide.hip; no GPU).

It multiplies pairs of 16 x 32 tiles (one v_mfma_i32_16x16x64_i8 each) in
chunks of four tiles, whose slot holds them even when they are full.  This test
replays the schedule with the constants read from the kernel source and the
tile offsets of real encodings from the oracle, and checks that every tile is
multiplied once, that chunks start at multiples of four, and that every value
piece, LDS window and offsets lane lies inside its buffer.  It also replays a
lane's four nibble windows (aligned dword pair + v_alignbyte_b32 + the selector
table + v_perm_b32) and compares the expanded operand with the dense int8 row."""
import os
import re

import numpy as np
import pytest

import synth

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2405_03594_amd", "csrc", "k_wide.hip")
TC = 4


def _slot():
    src = open(SRC).read()
    for line in ("constexpr int TC = kQ ? 4 : 2;",
                 "const int P = (S + TC - 1) / TC, L = (P + W - 1) / W;",
                 "kbeg = TC * (wave * L < P ? wave * L : P);",
                 "kend = kbeg + TC * L < S ? kbeg + TC * L : S;",
                 "const int t = ob + lane < kend ? ob + lane : kend;",
                 "if (c1 - ob + TC > kWave - 1) {",
                 "a0[b] = (XB * o[0]) & ~15u;",
                 "np[b] = (int)((XB * o[TC] - a0[b] + 15u) >> 4);",
                 "if (np[b] > 2 * kWave && lane == 0)",
                 "uint32_t p = before + t0 + ((t1 - t0) & (0u - (uint32_t)(fg >> 1)));"):
        assert line in src, f"kernel changed: update this replay ({line})"
    m = re.search(r"constexpr int kWideSlot = (\d+) \+ (\d+);", src)
    return int(m.group(1)) + int(m.group(2))


def _ranges(S, W):
    P = -(-S // TC)
    L = -(-P // W)
    out = []
    for w in range(W):
        kbeg = TC * min(w * L, P)
        kend = min(kbeg + TC * L, S)
        out.append((min(kbeg, kend), kend))
    return out


def _chunks(tob, kbeg, kend):
    out, ob = [], kbeg
    for c0 in range(kbeg, kend, TC):
        if c0 > kbeg and c0 - ob + TC > 63:
            ob = c0
        window = [int(tob[min(ob + i, kend)]) for i in range(64)]
        r = c0 - ob
        assert r + TC <= 63
        o = window[r:r + TC + 1]                          # tiles past the range: its end
        a0 = o[0] & ~15
        out.append((c0, a0, (o[TC] - a0 + 15) >> 4, o))
    return out


@pytest.mark.parametrize("W", [4, 8, 16])
@pytest.mark.parametrize("N,K,s", [(16, 16, 0.5), (33, 48, 0.0), (20, 272, 0.7), (16, 4096, 0.0), (32, 4112, 0.7),
                                   (16, 11008, 0.5), (17, 512, 1.0), (16, 65552, 0.7)])
def test_int8_schedule_stays_in_bounds(orc, N, K, s, W):
    slot = _slot()
    Wq, mask, _ = synth.int8_weight(5 + N + K, N, K, s)
    if s == 0.0:
        mask[::16, 0] = 0                                 # full tiles off a 16-byte boundary
    T = orc.pack_tiled(Wq, "i8", mask)
    S, B = -(-K // 32), -(-N // 16)
    value_bytes = -(-T.nnz // 16) * 16 + 16
    for b in range(B):
        tob = T.tile_offsets[b * S:(b + 1) * S + 1]
        covered = np.zeros(S, dtype=np.int64)
        for kbeg, kend in _ranges(S, W):
            assert kbeg % TC == 0 or kbeg == kend         # empty ranges are clamped to the end
            for c0, a0, pieces, o in _chunks(tob, kbeg, kend):
                covered[c0:min(c0 + TC, kend)] += 1
                assert pieces <= 129 and 16 * pieces <= slot
                assert a0 + 16 * max(pieces, 1) <= value_bytes    # (lanes past the chunk read its first piece again)
                for t in o:                               # a window starts at most at a tile's end, and reads 8 bytes
                    assert ((t - a0) & ~3) + 8 <= slot
        assert (covered == 1).all()


def _popc(x):
    return bin(int(x) & 0xFFFFFFFF).count("1")


def _sel(nib):
    out = 0
    for j in range(4):
        b = _popc(nib & ((1 << j) - 1)) if (nib >> j) & 1 else 12
        out |= b << (8 * j)
    return out


def _perm(s0, s1, sel):
    src = int(s1).to_bytes(4, "little") + int(s0).to_bytes(4, "little")
    out = 0
    for j in range(4):
        b = (sel >> (8 * j)) & 0xFF
        assert b < 8 or b == 12
        out |= (src[b] if b < 8 else 0) << (8 * j)
    return out


@pytest.mark.parametrize("N,K,s", [(16, 16, 0.5), (20, 272, 0.7), (33, 96, 0.0), (17, 528, 0.9)])
def test_int8_lane_expansion_matches_dense_rows(orc, N, K, s):
    slot = _slot()
    Wq, mask, _ = synth.int8_weight(41 + N, N, K, s)
    T = orc.pack_tiled(Wq, "i8", mask)
    vals = np.concatenate([T.values.view(np.uint8), np.zeros(32, np.uint8)])
    dense = np.where(mask.astype(bool), Wq, 0).astype(np.int8).view(np.uint8)
    S, B = -(-K // 32), -(-N // 16)
    bm = T.bitmask.reshape(-1)

    def alignbyte(hi, lo, sh):
        return ((int(hi) << 32 | int(lo)) >> (8 * (sh & 3))) & 0xFFFFFFFF

    for b in range(B):
        tob = T.tile_offsets[b * S:(b + 1) * S + 1]
        for kbeg, kend in _ranges(S, 8):
            for c0, a0, npieces, to in _chunks(tob, kbeg, kend):
                stage = np.zeros(slot, np.uint8)
                stage[:16 * npieces] = vals[a0:a0 + 16 * npieces]
                cn = min(TC, kend - c0)
                for q in range(-(-cn // 2)):
                    for lane in range(64):
                        fr, fg = lane & 15, lane >> 4
                        tsel, half = fg >> 1, fg & 1
                        j = 2 * q + tsel
                        t = b * S + c0 + j
                        words = [int(bm[t * 16 + r]) if j < cn else 0 for r in range(16)]
                        w = words[fr]
                        # values before this lane's: the 16-column group before (all rows), then rows above fr
                        o = to[j] + sum(_popc((words[r] >> (16 * g)) & 0xFFFF) for g in range(half) for r in range(16)) + \
                            sum(_popc((words[r] >> (16 * half)) & 0xFFFF) for r in range(fr))
                        got = []
                        for i in range(4):
                            nib = (w >> (16 * half + 4 * i)) & 15
                            p = o - a0
                            d = p & ~3
                            lo = int(stage[d:d + 4].view(np.uint32)[0])
                            hi = int(stage[d + 4:d + 8].view(np.uint32)[0])
                            got.append(_perm(0, alignbyte(hi, lo, p), _sel(nib)))
                            o += _popc(nib)
                        got = np.array(got, dtype=np.uint32).view(np.uint8)
                        n, k0 = b * 16 + fr, 32 * (c0 + j) + 16 * half
                        exp = np.zeros(16, np.uint8)
                        if n < N and j < cn and k0 < K:
                            seg = dense[n, k0:min(k0 + 16, K)]
                            exp[:seg.size] = seg
                        assert np.array_equal(got, exp), (b, c0 + j, lane)
