"""CPU model of the weight gradients formed inside the last pass
(csrc/whtmix_wgrad.hip): the product layout, the LDS addresses of the exchange
and of the staged dY / X tile, the operand pairing of every matrix
instruction, and the channel transform left to the final sum."""
import numpy as np
import pytest
from scipy.linalg import hadamard

SHAPES = [(A, cb) for A in range(11, 16) for cb in range(4, 8)]


class Wg:
    """The constants of the kernel's Wg<A, CB>, re-derived."""

    def __init__(self, A, cb):
        self.A, self.cb, self.C = A, cb, 1 << cb
        self.TW, self.SB = A - 11, cb - 4
        self.SW = min(self.SB, self.TW)
        self.SR = self.SB - self.SW
        self.RT = 5 - self.SR
        self.REM = A - 5 - cb
        self.WB = max(self.TW, 3)
        self.E = self.WB - self.TW
        self.NCHB = A - cb - 3
        self.QB = cb + self.RT
        self.SHIFT = (16 - (1 << (self.QB - 5))) & 63
        self.XCH = (1 << A) + (1 << (A - 5)) + self.SHIFT * ((1 << (A - self.QB)) - 1)

    @property
    def ok(self):
        return self.RT >= 3 and 0 <= self.REM <= self.RT

    def at(self, t):
        return t + (t >> 5) + self.SHIFT * (t >> self.QB)

    def base(self, t):
        lane, w = t & 63, t >> 6
        return ((lane & 15) | ((w & ((1 << self.SW) - 1)) << 4) | ((lane >> 4) << self.QB)
                | ((w >> self.SW) << (self.QB + 2)))

    def reg(self, k):
        return ((k & ((1 << self.SR) - 1)) << (4 + self.SW)) | ((k >> self.SR) << self.cb)

    @staticmethod
    def plane(nb, cb, j, n, chunk):
        """16-byte unit of chunk `chunk` of channel NNB j + n."""
        row = ((j << (cb - 4)) | n) << nb
        return row + ((j >> nb) << nb if nb < 4 else 0) + (chunk ^ (j & ((1 << min(nb, 4)) - 1)))

    @staticmethod
    def plane_units(nb, cb):
        return (16 << (cb - 4 + nb)) + ((15 >> nb) << nb if nb < 4 else 0)

    def stage(self, nb, lv, cg, quad):
        """(half-word address, channel) of the writes of stage_quad."""
        nnb = 1 << (self.cb - 4)
        for i in range(1 << lv):
            if nnb >= 1 << lv:
                j, n = cg // (nnb >> lv), ((cg & ((nnb >> lv) - 1)) << lv) + i
            else:
                j, n = cg * ((1 << lv) // nnb) + i // nnb, i % nnb
            c = (cg << lv) + i
            assert c == nnb * j + n
            byte = 16 * (self.plane(nb, self.cb, j, 0, quad >> 1) + (n << nb)) + 8 * (quad & 1)
            assert byte + 8 <= 16 * self.plane_units(nb, self.cb)
            yield byte // 2, c


def test_shapes_covered():
    left_out = [s for s in SHAPES if not Wg(*s).ok]
    assert left_out == [(11, 7), (15, 4)]


@pytest.mark.parametrize("shape", [s for s in SHAPES if Wg(*s).ok])
def test_layout_exchange_and_operands(shape):
    w = Wg(*shape)
    A, cb, C = w.A, w.cb, w.C
    threads = np.arange(1 << (A - 5))
    k = np.arange(32)
    # the product layout holds every tile element once
    idx = w.base(threads)[:, None] + w.reg(k)[None, :]
    assert np.array_equal(np.sort(idx.ravel()), np.arange(1 << A))
    # exchange: injective, in bounds, register offsets additive on both sides
    el = np.arange(1 << A)
    assert len(np.unique(w.at(el))) == 1 << A and w.at(el).max() < w.XCH
    assert np.array_equal(w.at(w.base(threads))[:, None] + w.at(w.reg(k))[None, :], w.at(idx))
    std = threads[:, None] + (k << (A - 5))[None, :]     # layout A-5
    assert np.array_equal(w.at(threads)[:, None] + w.at(k << (A - 5))[None, :], w.at(std))
    # layout A-5 registers are token bits; the token bits below are product-
    # layout register bits [SR, SR + REM)
    assert A - 5 >= cb
    assert [int(w.reg(1 << (w.SR + j))) for j in range(w.REM)] == [1 << (cb + j)
                                                                  for j in range(w.REM)]
    # reads of the product layout: 64 lanes on 64 banks, for every register
    banks = w.at(idx[:64, 0]) % 64
    assert len(np.unique(banks)) == 64

    # the staged tile (bf16 in one round; the planes of float32 in two halves
    # of the tokens, one round where there is one k step): 8-byte writes of four
    # tokens, then every operand read pairs the tokens of the register operand
    tok_of = idx >> cb
    for bf16 in (True, False):
        rounds = 1 if bf16 or w.RT == 3 else 2
        nb = w.NCHB - (rounds == 2)
        lv = 3 if bf16 else 2
        steps = 1 << (w.RT - 3)
        for h in range(rounds):
            half = {}
            for t in range(1 << (A - 5)):
                cg, u = t & ((1 << (cb - lv)) - 1), t >> (cb - lv)
                for hh in ([0] if bf16 else [0, 1] if rounds == 1 else [h]):
                    # the load's first token, with the half's bit put back
                    uq = u if bf16 else ((u & ((1 << (w.RT - 3)) - 1))
                                         | ((u >> (w.RT - 3)) << (w.RT - 2)))
                    tok0 = 4 * uq + (hh << (w.RT - 1))
                    assert ((tok0 + 3) << cb) + (cg << lv) + (1 << lv) <= 1 << A
                    quad = u if bf16 or rounds == 2 else (u << 1) | hh
                    for a, c in w.stage(nb, lv, cg, quad):
                        for e in range(4):
                            assert a + e not in half
                            half[a + e] = (tok0 + e, c)
            assert len(half) == (1 << A) // rounds
            for t in range(1 << (A - 5)):
                lane, wave = t & 63, t >> 6
                j, q, tw = lane & 15, lane >> 4, wave >> w.SW
                for s in range(h * steps // rounds, (h + 1) * steps // rounds):
                    chunk = (s | (q << (w.RT - 3)) | (tw << (w.RT - 1)) if rounds == 1 else
                             (s - h * steps // rounds) | (q << (w.RT - 4)) | (tw << (w.RT - 2)))
                    for n in (0, C // 16 - 1):
                        unit = w.plane(nb, cb, j, 0, chunk) + (n << nb)
                        got = [half[8 * unit + e] for e in range(8)]
                        assert got == [(int(tok_of[t, (8 * s + e) << w.SR]), C // 16 * j + n)
                                       for e in range(8)]
                    if lane == 0:   # the 16 lanes of an operand read: 16 bank groups
                        assert len({w.plane(nb, cb, k, 0, chunk) % 16 for k in range(16)}) == 16
    # the strips of the registers: channel 16 (strip0 | sr << SW) + i
    for t in (0, 63, (1 << (A - 5)) - 1):
        strip0 = (t >> 6) & ((1 << w.SW) - 1)
        for sr in range(1 << w.SR):
            assert (int(idx[t, sr]) & (C - 1)) == 16 * (strip0 | (sr << w.SW)) + (t & 15)


def test_channel_inverse_commutes_with_the_token_sum():
    """Z'^T dY = H_C (U^T dY) for U = Z' H_C (the channel inverse undone), the
    transform wgrad_final_kernel applies to the summed C x C matrix."""
    rng = np.random.default_rng(5)
    tokens, C = 32, 16
    u, d = rng.standard_normal((tokens, C)), rng.standard_normal((tokens, C))
    H = hadamard(C).astype(float)
    assert np.allclose((u @ H).T @ d, H @ (u.T @ d))


class Wd:
    """The constants of the direct form's Wd<A, CB>."""

    def __init__(self, A, cb):
        self.A, self.cb = A, cb
        self.TW, self.SB = A - 11, cb - 4
        self.SW = min(self.SB, self.TW)
        self.SR = self.SB - self.SW
        self.LB = A - 6 - self.SW
        self.RT = self.LB - self.SR
        self.NCHB = A - cb - 3

    plane, plane_units = staticmethod(Wg.plane), staticmethod(Wg.plane_units)

    @property
    def ok(self):
        return Wg(self.A, self.cb).ok and self.LB <= 6

    def base(self, t):
        lane, strips = t & 63, t >> 6
        return (lane & 15) | (strips << 4) | ((lane >> 4) << self.cb)

    def reg(self, k):
        tok = k >> self.SR
        return (((k & ((1 << self.SR) - 1)) << (4 + self.SW)) | ((tok & 3) << (self.cb + self.RT))
                | ((tok >> 2) << (self.cb + 2)))


def swap(idx, lane_bit, j):
    """v_permlane16/32_swap on register pairs (k, k | 1 << j): lane bit
    lane_bit and register bit j change places."""
    out = idx.copy()
    lanes = np.arange(64)
    lo, hi = lanes[(lanes >> lane_bit) & 1 == 0], lanes[(lanes >> lane_bit) & 1 == 1]
    for k in range(idx.shape[1]):
        if not k & (1 << j):
            out[hi, k] = idx[lo, k | (1 << j)]
            out[lo, k | (1 << j)] = idx[hi, k]
    return out


@pytest.mark.parametrize("shape", [s for s in SHAPES if Wd(*s).ok])
def test_direct_form(shape):
    w = Wd(*shape)
    A, cb, C = w.A, w.cb, 1 << w.cb
    VV, threads = 1 << w.LB, 64 << w.SW
    t_all, k = np.arange(threads), np.arange(VV)
    idx = w.base(t_all)[:, None] + w.reg(k)[None, :]
    assert np.array_equal(np.sort(idx.ravel()), np.arange(1 << A))
    # transformed: register token bits, then the two traded in from the lanes
    done = {int(np.log2(w.reg(1 << j))) for j in range(w.SR, w.LB)}
    waves = []
    for wv in range(1 << w.SW):
        x = idx[64 * wv:64 * wv + 64]
        x = swap(swap(x, 4, w.SR), 5, w.SR + 1)
        waves.append(x)
    for j in (w.SR, w.SR + 1):
        done |= {int(np.log2(abs(int(waves[0][0, 1 << j]) - int(waves[0][0, 0]))))}
    assert done == set(range(cb, A))
    for bf16 in (True, False):
        rounds = 1 if bf16 or w.RT == 3 else 2
        nb = w.NCHB - (rounds == 2)
        lv = 3 if bf16 else 2
        np_ = VV * (2 if bf16 else 4) // 16 // rounds
        qs = threads >> (cb - lv)
        assert qs >= 1 and np_ % 4 == 0
        B = w.RT - 3
        steps = 1 << (w.RT - 3)
        for h in range(rounds):
            half = {}
            for t in range(threads):
                cg, q0 = t & ((1 << (cb - lv)) - 1), t >> (cb - lv)
                for m in range(np_ // 4):
                    quad = q0 + m * qs
                    full = quad if rounds == 1 else ((quad & ((1 << B) - 1)) | (h << B)
                                                     | ((quad >> B) << (B + 1)))
                    assert (full << (cb + 2)) + (3 << cb) + (cg << lv) + (1 << lv) <= 1 << A
                    for a, c in Wg.stage(w, nb, lv, cg, quad):
                        for e in range(4):
                            assert a + e not in half
                            half[a + e] = (4 * full + e, c)
            assert len(half) == (1 << A) // rounds
            for wv in range(1 << w.SW):
                for lane in range(64):
                    j, q = lane & 15, lane >> 4
                    for s in range(h * steps // rounds, (h + 1) * steps // rounds):
                        chunk = (s | (q << (w.RT - 3)) if rounds == 1 else
                                 (s - h * steps // rounds) | (q << (w.RT - 4)))
                        for n in (0, C // 16 - 1):
                            unit = Wg.plane(nb, cb, j, 0, chunk) + (n << nb)
                            got = [half[8 * unit + e] for e in range(8)]
                            for sr in (0, (1 << w.SR) - 1):
                                el = [int(waves[wv][lane, sr | ((8 * s + e) << w.SR)])
                                      for e in range(8)]
                                assert [(v >> cb, C // 16 * j + n) for v in el] == got
                                # the operand's row: channel 16 strip + lane mod 16
                                assert {v & (C - 1) for v in el} == {
                                    16 * (wv | (sr << w.SW)) + (lane & 15)}
