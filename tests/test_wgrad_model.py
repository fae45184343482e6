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
    def swz(nb, c):
        sh = 4 - nb if nb < 4 else 0
        return ((c >> sh) ^ (c >> 3)) & ((1 << min(nb, 4)) - 1)


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
                    for i in range(1 << lv):
                        c = (cg << lv) + i
                        byte = (16 * ((cg << (nb + lv)) + (i << nb)
                                      + ((quad >> 1) ^ w.swz(nb, cg << lv) ^ w.swz(nb, i)))
                                + 8 * (quad & 1))
                        assert byte + 8 <= (2 << A) // rounds
                        for e in range(4):
                            assert byte // 2 + e not in half
                            half[byte // 2 + e] = (tok0 + e, c)
            assert len(half) == (1 << A) // rounds
            for t in range(1 << (A - 5)):
                lane, wave = t & 63, t >> 6
                j, q, tw = lane & 15, lane >> 4, wave >> w.SW
                for s in range(h * steps // rounds, (h + 1) * steps // rounds):
                    chunk = (s | (q << (w.RT - 3)) | (tw << (w.RT - 1)) if rounds == 1 else
                             (s - h * steps // rounds) | (q << (w.RT - 4)) | (tw << (w.RT - 2)))
                    xo = chunk ^ w.swz(nb, j)
                    for n in (0, C // 16 - 1):
                        unit = (j << nb) + (xo ^ w.swz(nb, 16 * n)) + (16 * n << nb)
                        got = [half[8 * unit + e] for e in range(8)]
                        assert got == [(int(tok_of[t, (8 * s + e) << w.SR]), 16 * n + j)
                                       for e in range(8)]
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
